// Persistent BFS levels for small frontiers on low-degree graphs.
//
// A high-diameter graph (a 3-D grid: hundreds of levels, frontiers of a few
// thousand vertices) spends almost all of a level's time in launch and
// phase latency of the three bucketing kernels.  While the frontier stays
// at or below kTinyFrontier vertices, this kernel runs level after level in
// one cooperative launch, with ONE grid-wide barrier per level.
//
// min-select2nd (parents: select2nd with x value = vertex id, so a new
// vertex's parent is its smallest frontier in-neighbour, as in the
// level-synchronous SpMSpV).  One 64-bit word per vertex holds level << 32 |
// parent, and every edge (u, v) out of F(L) is ONE atomic minimum with
// (L + 1) << 32 | u: a word at kUndiscovered means the lane found v and
// appends it, a word of level L + 1 keeps the smaller parent, a word of an
// earlier level is smaller already and stays.  Vertices visited before the
// launch hold 0.  Levels, parents and visited bits are written from the
// words when the launch ends, in one pass over them that also puts them
// back to kUndiscovered (-0.0: the words are the HBM accumulator's fp64
// cells, empty between calls).
//
// or-and (levels only): the lane whose atomic OR first sets v's visited
// bit owns v, writes its level and appends it.
//
// A level is a chain of dependent round trips to memory, so what counts is
// their number.  Each workgroup keeps the part of the frontier it discovered
// in LDS and goes on from there: no list to write, count and read back, and
// the column bounds and neighbours of the next level's vertices are loaded
// while the barrier is under way.  What remains is one atomic per edge and
// the barrier, whose arrivals add up the next frontier's length.  A workgroup
// whose part outgrows its threads asks for the parts to be dealt out evenly
// again, which goes through a list in memory and one more barrier.  Updates of
// one word queue at about 10 ns each, so arrivals are counted in groups.
// Measured on a 256^3 grid with parents (766 levels): 14.8 ms with two
// bitmaps, a minimum per vertex, a commit of every frontier vertex (two loads
// and two atomics per edge, four scattered writes per vertex) and a shared
// list with one counter update per wave; 9.7 ms with one word per vertex and
// one counter update per workgroup; 8.4 ms with the frontier kept in LDS (11.0
// us per level; 6.9 on a 128^3 grid, 3.5 on a path, the barrier and one
// atomic alone).
//
// Results are those of the bucketing path (same levels, same minimum
// parents); only the order of the frontier list differs.  The kernel stops
// when the frontier empties or outgrows kTinyFrontier, commits it, and
// leaves it in front[0] with its length and level in the control block for
// the bucketing path.

#include "internal.h"

namespace spv {

namespace {

constexpr int kPBlock = 512;
constexpr int kPList = 4096;   // frontier vertices a workgroup keeps in LDS
constexpr int kPShare = kPBlock;   // a longer part asks for a new deal
constexpr int kSpinLimit = 1 << 22;
// Barrier words, each on a cache line of its own (workgroups that wait poll
// the published word while others update the counters): the two list
// counters, groups that arrived and arrivals of each group, four 64-bit
// words each (one per barrier modulo 4), and the published word once per
// group, so that a line is polled by one group's workgroups only.
// Workgroup b belongs to group b mod kGroups, one die's workgroups.
constexpr int kLine = 32;   // 128-byte L2 line in 32-bit words
constexpr int kGroups = 8;
constexpr int kCount = 0, kRoot = 2 * kLine, kArrive = 3 * kLine, kGen = kArrive + kGroups * kLine;
static_assert(kGen + kGroups * kLine <= kPersistBarWords, "barrier words");
// Arrival words: arrivals in bits 63:48, requests for a new deal in 47:36,
// the sum of the workgroups' frontier parts in 35:0.  Published: the barrier
// number's low 16 bits in 63:48, then the same fields.
constexpr int kArriveShift = 48, kDealShift = 36;
constexpr uint64_t kSumMask = (1ull << kDealShift) - 1;
constexpr uint64_t kDealMask = 0xfffull << kDealShift;
constexpr uint64_t kUndiscovered = 0x8000000000000000ull;

__device__ __forceinline__ int32_t ldc(const int32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ldu(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stc(int32_t* p, int32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ldc64(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stc64(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stcu(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Grid barrier that also adds up one value per workgroup (all workgroups are
// resident: cooperative launch).  The last arrival of a group adds the
// group's word to the root, the last group publishes the sums.  Barrier k
// uses word k mod 4 of every counter; workgroup 0 clears word (k + 2) mod 4
// before it arrives at barrier k (its last use, barrier k - 2, is complete,
// and its next one starts after barrier k).
// Every value that crosses workgroups in this kernel is
// written and read with device-scope atomics, which are coherent without
// cache maintenance, so the barrier only has to wait for this workgroup's
// own memory operations to complete: no L2 write-back or invalidation (which
// on a multi-die GPU would touch the whole L2 of a die at every barrier).
// That wait is explicit: a workgroup-scope fence does not wait for vector
// memory operations on gfx950 (the waves of a workgroup share one CU), so
// every wave waits for its own outstanding loads, stores and atomics
// (s_waitcnt vmcnt(0)) before the workgroup barrier, and only then does
// thread 0 publish the arrival.
// A wait past kSpinLimit polls sets ERR_SPIN and returns false; the caller
// then leaves the kernel, so every later barrier of the others times out
// too and no wave can hang.
//
// grid_arrive / grid_wait: thread 0 of each workgroup, between workgroup
// barriers.  The published word (0 after a time-out).
__device__ __forceinline__ void grid_arrive(uint32_t* bar, uint32_t gen, uint64_t add) {
    const int k = (int)(gen & 3u);
    if (blockIdx.x == 0) {
        const int c = (k + 2) & 3;
        for (int g = 0; g < kGroups; ++g) stc64(reinterpret_cast<uint64_t*>(&bar[kArrive + g * kLine]) + c, 0ull);
        stc64(reinterpret_cast<uint64_t*>(&bar[kRoot]) + c, 0ull);
        wait_vmem();
    }
    const uint32_t grp = blockIdx.x % kGroups;
    const uint64_t members = (gridDim.x - grp + kGroups - 1) / kGroups;
    const uint64_t groups = gridDim.x < kGroups ? gridDim.x : kGroups;
    auto* arrive = reinterpret_cast<unsigned long long*>(&bar[kArrive + grp * kLine]) + k;
    auto* root = reinterpret_cast<unsigned long long*>(&bar[kRoot]) + k;
    constexpr uint64_t low = (1ull << kArriveShift) - 1;
    const uint64_t mine = (1ull << kArriveShift) | add;
    const uint64_t w = atomicAdd(arrive, mine) + mine;
    if (w >> kArriveShift != members) return;
    const uint64_t up = (1ull << kArriveShift) | (w & low);
    const uint64_t r = atomicAdd(root, up) + up;
    if (r >> kArriveShift != groups) return;
    const uint64_t word = (uint64_t)((gen + 1u) & 0xffffu) << kArriveShift | (r & low);
    for (int g = 0; g < kGroups; ++g) stc64(reinterpret_cast<uint64_t*>(&bar[kGen + g * kLine]), word);
}
__device__ __forceinline__ uint64_t grid_wait(const uint32_t* bar, uint32_t gen, uint32_t* err) {
    const uint64_t want = (gen + 1u) & 0xffffu;
    const auto* word = reinterpret_cast<const uint64_t*>(&bar[kGen + (blockIdx.x % kGroups) * kLine]);
    for (int spins = 0;; ++spins) {
        const uint64_t w = ldc64(word);
        if (w >> kArriveShift == want) return w | 1ull << 63;
        if (spins > kSpinLimit) {
            atomicOr(err, ERR_SPIN);
            return 0ull;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}
// The whole barrier with nothing to add; false after a time-out.
__device__ bool grid_sync(uint32_t* bar, uint32_t& gen, uint32_t* err) {
    __shared__ int s_ok;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    wait_vmem();
    __syncthreads();
    if (threadIdx.x == 0) {
        grid_arrive(bar, gen, 0ull);
        s_ok = grid_wait(bar, gen, err) != 0ull;
    }
    ++gen;
    __syncthreads();
    return s_ok != 0;
}

template <bool MIN>
__global__ __launch_bounds__(kPBlock) void k_bfs_persistent(PersistArgs a) {
    constexpr int K = 8;   // neighbours per lane in flight
    __shared__ int32_t s_list[2][kPList];   // this workgroup's part of F(L) and of F(L+1)
    __shared__ int32_t s_n[2], s_end[2];    // vertices found for each, and how many of them are in s_list
    __shared__ int32_t s_first;
    __shared__ uint64_t s_word;
    int32_t f = ldc(&a.ctrl->f);
    if (f <= 0 || f > kTinyFrontier) return;   // the same value in every workgroup
    int32_t lvl = ldc(&a.ctrl->level);         // level of the frontier in front[0]
    const int lane = threadIdx.x & 63;
    int32_t* const level = reinterpret_cast<int32_t*>(
        __hip_atomic_load(reinterpret_cast<const uint64_t*>(&a.ctrl->bfs_level), __ATOMIC_RELAXED,
                          __HIP_MEMORY_SCOPE_AGENT));
    int32_t* const parent = reinterpret_cast<int32_t*>(
        __hip_atomic_load(reinterpret_cast<const uint64_t*>(&a.ctrl->bfs_parent), __ATOMIC_RELAXED,
                          __HIP_MEMORY_SCOPE_AGENT));
    uint32_t* const err = &a.ctrl->err;
    const int64_t stride = (int64_t)gridDim.x * kPBlock;
    // Slots of a list in memory: waves are dealt to the workgroups in turn, so
    // a short one uses every compute unit.
    const int64_t p0 = ((int64_t)(threadIdx.x / 64) * gridDim.x + blockIdx.x) * 64 + lane;
    uint32_t gen = 0;
    int cur = 0;     // F(L): s_list[cur]
    int deal = 1;    // list in memory of the next deal: front[deal], its counter bar[kCount + kLine * deal]
    if (threadIdx.x < 2) {
        s_n[threadIdx.x] = 0;
        s_end[threadIdx.x] = kPList;
    }
    if (MIN) {
        // vertices visited before this launch: the smallest word
        const int64_t words = ((int64_t)a.n + 31) / 32;
        for (int64_t w = p0; w < words; w += stride) {
            uint32_t bits = ldu(&a.visited[w]);
            while (bits) {
                const int bit = __ffs(bits) - 1;
                bits &= bits - 1u;
                if (w * 32 + bit < a.n) stc64(&a.state[w * 32 + bit], 0ull);
            }
        }
        if (!grid_sync(a.bar, gen, err)) return;
    } else {
        __syncthreads();
    }
    // Vertices found by a wave (claim[j]: v[j]) join this workgroup's part of
    // the list s_list[to]; past its end they go to the next deal's list.
    auto append = [&](const int32_t (&v)[K], const bool (&claim)[K], int to) {
        uint64_t vote[K];
        int total = 0;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            vote[j] = __ballot(claim[j]);
            total += (int)__popcll(vote[j]);
        }
        if (!total) return;
        int32_t first = 0;
        if (lane == 0) first = atomicAdd(&s_n[to], total);
        first = __shfl(first, 0, 64);
        const bool fits = first + total <= kPList;   // uniform in the wave
        if (!fits) {   // and neither does any later one
            if (lane == 0) {
                if (first <= kPList) s_end[to] = first;   // one wave: the entries in LDS end here
                first = atomicAdd(reinterpret_cast<int32_t*>(&a.bar[kCount + kLine * deal]), total);
            }
            first = __shfl(first, 0, 64);
        }
        const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int32_t at = first + (int)__popcll(vote[j] & below);
            if (claim[j]) {
                if (fits) s_list[to][at] = v[j];
                else stc(&a.front[deal][at], v[j]);
            }
            first += (int)__popcll(vote[j]);
        }
        if (!fits) wait_vmem();
    };
    // This workgroup's share of a list of f vertices, f <= kTinyFrontier (at
    // most kPList of them: the launch has at least kTinyFrontier / kPList
    // workgroups).
    auto take = [&](const int32_t* list, int to) {
        for (int64_t p = p0; p - lane < f; p += stride) {
            const int32_t u = p < f ? ldc(&list[p]) : -1;
            const uint64_t have = __ballot(u >= 0);
            int32_t first = 0;
            if (lane == 0) first = atomicAdd(&s_n[to], (int)__popcll(have));
            first = __shfl(first, 0, 64);
            if (u >= 0) s_list[to][first + (int)__popcll(have & ((1ull << lane) - 1ull))] = u;
        }
    };
    take(a.front[0], cur);
    __syncthreads();
    int32_t part = s_n[cur];
    int32_t u, q, len, v[K];   // this thread's first vertex of the level, its column and first neighbours
    auto fetch = [&](int32_t i) {
        u = i < part ? s_list[cur][i] : -1;
        q = 0;
        len = 0;
        if (u >= 0) {
            q = a.colptr[u];
            len = a.colptr[u + 1] - q;
        }
#pragma unroll
        for (int j = 0; j < K; ++j) v[j] = j < len ? a.rowids[q + j] : -1;
    };
    fetch(threadIdx.x);
    for (;;) {
        const int to = cur ^ 1;
        // Lanes step through their vertices' neighbour lists together
        // (degrees are small here), K neighbours per lane in flight.
        for (int32_t off = 0; off < part; off += kPBlock) {
            if (off > 0) fetch(off + threadIdx.x);
            int32_t mx = len;
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) mx = max(mx, __shfl_xor(mx, d, 64));
            for (int k0 = 0; k0 < mx; k0 += K) {
                if (k0 > 0) {
#pragma unroll
                    for (int j = 0; j < K; ++j) v[j] = k0 + j < len ? a.rowids[q + k0 + j] : -1;
                }
                bool claim[K];
                if (MIN) {
                    const uint64_t key = (uint64_t)(uint32_t)(lvl + 1) << 32 | (uint32_t)u;
                    uint64_t old[K];
#pragma unroll
                    for (int j = 0; j < K; ++j)
                        old[j] = v[j] >= 0 ? atomicMin(reinterpret_cast<unsigned long long*>(&a.state[v[j]]), key) : 0ull;
#pragma unroll
                    for (int j = 0; j < K; ++j) claim[j] = old[j] == kUndiscovered;
                } else {
                    // Levels only: the first lane to set v's visited bit owns
                    // v and writes its level at once.
                    uint32_t old[K];
#pragma unroll
                    for (int j = 0; j < K; ++j)
                        old[j] = v[j] >= 0 ? atomicOr(&a.visited[v[j] >> 5], 1u << (v[j] & 31)) : 0xffffffffu;
#pragma unroll
                    for (int j = 0; j < K; ++j) claim[j] = !((old[j] >> (v[j] & 31)) & 1u);
#pragma unroll
                    for (int j = 0; j < K; ++j)
                        if (claim[j]) level[v[j]] = lvl + 1;
                }
                append(v, claim, to);
            }
        }
        __syncthreads();   // F(L+1)'s part is complete; F(L)'s list and count are free
        cur = to;
        part = min(s_n[cur], s_end[cur]);
        if (threadIdx.x == 0) {
            s_n[cur ^ 1] = 0;
            s_end[cur ^ 1] = kPList;
            grid_arrive(a.bar, gen, (uint64_t)(s_n[cur] > kPShare) << kDealShift | (uint64_t)(uint32_t)s_n[cur]);
        }
        fetch(threadIdx.x);   // while the others arrive
        if (threadIdx.x == 0) s_word = grid_wait(a.bar, gen, err);
        ++gen;
        __syncthreads();
        const uint64_t w = s_word;
        if (w == 0ull) return;   // timed out: so will every other workgroup
        f = (int32_t)(w & kSumMask);
        ++lvl;
        const bool last = f == 0 || f > kTinyFrontier;
        if (f > 0 && ((w & kDealMask) || last)) {
            // every part to the list in memory, behind what did not fit LDS
            if (threadIdx.x == 0)
                s_first = part > 0 ? atomicAdd(reinterpret_cast<int32_t*>(&a.bar[kCount + kLine * deal]), part) : 0;
            __syncthreads();
            for (int32_t i = threadIdx.x; i < part; i += kPBlock) stc(&a.front[deal][s_first + i], s_list[cur][i]);
            // the other list's counter: last used before the previous deal's barrier
            if (blockIdx.x == 0 && threadIdx.x == 0) stcu(&a.bar[kCount + kLine * (deal ^ 1)], 0u);
            if (!grid_sync(a.bar, gen, err)) return;
            deal ^= 1;
            if (!last) {
                if (threadIdx.x == 0) {
                    s_n[cur] = 0;
                    s_end[cur] = kPList;
                }
                __syncthreads();
                take(a.front[deal ^ 1], cur);
                __syncthreads();
                part = s_n[cur];
                fetch(threadIdx.x);
            }
        }
        if (last) break;
    }
    // Levels, parents and visited bits of what this launch discovered; the
    // words go back to kUndiscovered.  Consecutive vertices per wave.
    if (MIN) {
        const int64_t n64 = ((int64_t)a.n + 63) & ~int64_t(63);
        for (int64_t v = p0; v < n64; v += stride) {
            const uint64_t w = v < a.n ? ldc64(&a.state[v]) : kUndiscovered;
            const uint64_t seen = __ballot(w != kUndiscovered);
            if (!seen) continue;
            if (w != kUndiscovered) {
                if (w != 0ull) {
                    level[v] = (int32_t)(w >> 32);
                    if (parent) parent[v] = (int32_t)(uint32_t)w;
                }
                stc64(&a.state[v], kUndiscovered);
            }
            const int64_t at = v >> 5;   // two bitmap words per wave, all their vertices here
            if ((lane & 31) == 0 && v < a.n) stcu(&a.visited[at], (uint32_t)(seen >> (lane & 32)));
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        stc(&a.ctrl->f, f);
        stc(&a.ctrl->level, lvl);
    }
    // Hand the frontier back in front[0].
    if (f > 0 && deal == 0) {   // it was dealt to front[1]
        for (int64_t p = p0; p < f; p += stride) stc(&a.front[0][p], ldc(&a.front[1][p]));
    }
}

}  // namespace

int persistent_grid(int num_cu) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_bfs_persistent<true>, kPBlock, 0) != hipSuccess ||
        per_cu < 1)
        return 0;
    int per_cu2 = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu2, k_bfs_persistent<false>, kPBlock, 0) != hipSuccess ||
        per_cu2 < 1)
        return 0;
    if (per_cu2 < per_cu) per_cu = per_cu2;
    if (per_cu > 1) per_cu = 1;   // fewer arrivals per barrier; small frontiers need few threads
    const int grid = per_cu * num_cu;
    // a deal gives every workgroup at most kPList vertices, and arrivals fit their fields
    return (int64_t)grid * kPList < 2 * kTinyFrontier || grid > 1024 ? 0 : grid;
}

hipError_t launch_bfs_persistent(const PersistArgs& a, bool min_semiring, int grid, hipStream_t s) {
    void* args[] = {const_cast<PersistArgs*>(&a)};
    const void* fn = min_semiring ? reinterpret_cast<const void*>(k_bfs_persistent<true>)
                                  : reinterpret_cast<const void*>(k_bfs_persistent<false>);
    return hipLaunchCooperativeKernel(fn, dim3(grid), dim3(kPBlock), args, 0, s);
}

}  // namespace spv
