"""CPU test of the bucket slot reservation (csrc/reserve.h): the rule against
64-bit arithmetic, and workgroups that go on reserving in a full bucket as
far as the expansion lets them."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1610_07902_amd", "csrc")

PROGRAM = r"""
#include "reserve.h"
#include <cstdio>
#include <vector>
using namespace spv;
int main() {
    const int64_t big = INT32_MAX;
    const std::vector<int64_t> caps = {0, 1, 5, 8191, 8192, 1 << 30, big - 8192, big - 1, big};
    const std::vector<int64_t> counts = {1, 2, 64, 1024, 8191, 8192};
    for (int64_t cap : caps)
        for (int64_t n : counts)
            for (int64_t at : {int64_t(0), cap, big, big + 1, int64_t(UINT32_MAX) - 8192, int64_t(UINT32_MAX)})
                for (int64_t d = -8200; d <= 8200; ++d) {
                    const int64_t taken = at + d;
                    if (taken < 0 || taken > int64_t(UINT32_MAX)) continue;
                    if (slots_fit((int32_t)(uint32_t)taken, (int32_t)n, (int32_t)cap) != (taken + n <= cap)) {
                        std::printf("taken %lld n %lld cap %lld\n", (long long)taken, (long long)n, (long long)cap);
                        return 1;
                    }
                }
    // every workgroup takes whole chunks of one bucket until one does not fit
    for (int64_t cap : caps) {
        uint32_t counter = 0;
        int64_t given = 0, asked = 0;
        std::vector<char> over(kExpandMaxGrid, 0);
        for (bool more = true; more;) {
            more = false;
            for (int w = 0; w < kExpandMaxGrid; ++w) {
                if (over[w]) continue;
                more = true;
                const uint32_t taken = counter;
                counter += kExpandMaxChunk;
                asked += kExpandMaxChunk;
                if (slots_fit((int32_t)taken, kExpandMaxChunk, (int32_t)cap)) {
                    if (taken != given) return std::printf("slot %u given twice\n", taken), 1;
                    given += kExpandMaxChunk;
                } else {
                    over[w] = 1;
                }
            }
        }
        if (given > cap || asked != (int64_t)counter) return std::printf("counter wrapped, cap %lld\n", (long long)cap), 1;
    }
    std::puts("ok");
}
"""


def test_reservation_rule(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout
