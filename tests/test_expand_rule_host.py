"""CPU test of when the expansion takes a call and how it cuts it into tiles
(csrc/expand_rule.h): over matrices from even to skewed, calls from one entry
to all and every chunk shape, no choice of columns gives one workgroup's tile
much more than its share, even matrices are always taken, and tiles are neither
thinner than a chunk where there are many nor thicker where there are few."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1610_07902_amd", "csrc")

PROGRAM = r"""
#include "expand_rule.h"
#include <cstdio>
using namespace spv;
#define FAIL(...) return std::printf(__VA_ARGS__), 1
int main() {
    const int shapes[][2] = {{256, 4}, {256, 8}, {256, 16}, {512, 4}, {512, 8}, {1024, 4}, {1024, 8}};
    int64_t taken = 0, refused = 0;
    for (int64_t n : {1, 2, 777, 1 << 15, 1 << 20, 1 << 26})
        for (double mean : {0.0, 0.3, 3.8, 6.9, 16.0, 57.5, 300.0, 1000.0})
            for (int64_t longest : {0, 1, 7, 40, 64, 200, 600, 2047, 2048, 100000})
                for (const auto& sh : shapes)
                    for (int gmax : {64, 256, 512, 2048, 4096})
                        for (int64_t f : {int64_t(-1), int64_t(0), int64_t(1), int64_t(16), int64_t(500), n / 100, n / 10, n}) {
                            const int64_t nnz = (int64_t)(mean * n);
                            if (f > n || longest * n < nnz || longest > nnz) continue;
                            const int block = sh[0], chunk = sh[0] * sh[1];
                            const int cus = gmax < 256 ? gmax : 256;
                            const ExpandTiles t = expand_tiles(n, nnz, longest, f, block, chunk, gmax, cus);
                            (t.taken ? taken : refused)++;
                            const double m = mean > 1.0 ? mean : 1.0;
                            if (t.taken && longest > 2047) FAIL("column of %lld taken\n", (long long)longest);
                            if (!t.taken && longest <= 2047 && longest <= 2 * m) FAIL("even matrix refused\n");
                            if (t.per_min < 1 || t.per_max < t.per_min || t.per_max > block) FAIL("bounds\n");
                            if (t.per < 1 || t.per > t.per_max || t.grid < 1 || t.grid > gmax) FAIL("tile\n");
                            if (!t.taken) continue;
                            // the widest tile of the call, and how many of them one workgroup gets
                            const int64_t most_f = f < 0 ? n : f;
                            int64_t per = t.per;
                            if (f < 0) {
                                const int64_t wide = (int64_t)t.grid * t.per_max, rounds = (most_f + wide - 1) / wide;
                                per = (most_f + t.grid * rounds - 1) / (t.grid * rounds);
                                per = per > t.per_max ? t.per_max : per < t.per_min ? t.per_min : per;
                            }
                            const double extra = (double)per * longest - 2.0 * per * m;
                            if (extra > 8192.0 && extra > 2.0 * chunk && per > 1)
                                FAIL("tile of %lld: longest %lld mean %g chunk %d f %lld\n", (long long)per,
                                     (long long)longest, mean, chunk, (long long)f);
                            const int64_t tiles = (most_f + per - 1) / per;
                            // several tiles: each filled (evenly dealt out by rounds: half filled at
                            // least), or the whole workgroup wide
                            if (tiles > (f < 0 ? t.grid : cus) && per < block &&
                                per * m < (f < 0 ? 0.4 : 0.8) * chunk - m)
                                FAIL("%lld thin tiles on %d workgroups\n", (long long)tiles, t.grid);
                            // fewer tiles than compute units: none of more than a chunk, or of several columns
                            if (f > 0 && tiles < cus / 2 && per > 1 && per * m > chunk)
                                FAIL("%lld tiles of %g products\n", (long long)tiles, per * m);
                        }
    if (!taken || !refused) FAIL("taken %lld refused %lld\n", (long long)taken, (long long)refused);
    std::puts("ok");
}
"""


def test_no_tile_gets_much_more_than_its_share(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout
