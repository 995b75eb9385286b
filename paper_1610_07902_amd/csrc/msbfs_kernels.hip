// Multi-source BFS in the pull direction (bottom-up), bit-parallel over the
// sources.  The paper names switching SpMSpV-driven BFS to the matrix-driven
// direction as future work (Conclusions); with many sources one pull step
// serves all of them: source s owns bit s % 64 of word s / 64 of every
// vertex's frontier and seen masks (G = ceil(nsrc / 64) words per vertex,
// stored vertex-major: word g of vertex v at v * G + g).
//
// A vertex v not yet seen by some sources scans its row (the in-neighbours
// u, ascending) and takes, for every such source, the first u whose frontier
// mask has the source's bit: with ascending rows that is the smallest
// frontier in-neighbour, the parent the push direction's min-select2nd
// gives.  The scan stops once every unseen source is found.  Rows of up to
// kMsLong entries are scanned packed, 32 vertices per wave; rows of up to
// kMsHuge entries by one wave each, longer ones by a workgroup.
//
// Switching a search from push to pull converts its state once: the
// per-source visited bitmaps become the seen masks (transposed), the
// per-source frontier lists become frontier masks.

#include "device_ops.h"

namespace spv {

namespace {

constexpr int kMsBlock = 256;

__device__ __forceinline__ uint64_t group_valid(int nsrc, int g) {
    const int k = nsrc - 64 * g;
    return k >= 64 ? ~0ull : ((1ull << k) - 1ull);
}

__device__ __forceinline__ uint64_t wave_or64(uint64_t v) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) v |= __shfl_xor(v, d);
    return v;
}

// Tell the host that the step found something.  One flag, stored only while
// it reads unset: an add of every wave's count to one word serialised there
// (about 12 ns each, 16K waves: 200 us of every large step of 64 searches on
// scale 20, whatever else the step did).
__device__ __forceinline__ void ms_report(const MsArgs& a, uint32_t found) {
    if (found && (threadIdx.x & (kWave - 1)) == 0 && !ld_acquire64(a.found_any)) st_release64(a.found_any, 1ull);
}

// 64 x 64 bit transpose across a wave: lane i's bit k becomes lane k's bit i
// (swap of off-diagonal blocks, block size halved each round).
__device__ __forceinline__ uint64_t wave_transpose64(uint64_t x) {
    const int lane = threadIdx.x & (kWave - 1);
    uint64_t m = 0x00000000ffffffffull;
#pragma unroll
    for (int j = 32; j >= 1; j >>= 1) {
        const uint64_t y = __shfl_xor(x, j);
        x = (lane & j) ? (x & ~m) | ((y >> j) & m) : (x & m) | ((y & m) << j);
        m ^= m << (j >> 1);
    }
    return x;
}

// Rows of up to kMsLong entries.  One wave covers 32 consecutive vertices;
// the entries of those that still miss a source are packed one after the
// other and taken 64 at a time, so lanes stay full whatever the row lengths
// and column ids come in whole lines.  A step's frontier words are turned
// into one word per source (bit transpose); lane s then takes, per row of
// the step, the first entry with its source's bit, and keeps the parent in
// LDS (slot [source][row], padded against bank conflicts).  kMsUnroll steps
// of loads are in flight, the next ones' column ids loaded ahead.
//
// Afterwards the wave stores source by source, so each store instruction
// writes consecutive vertices of one source's level and parent rows (a whole
// 128-byte line) instead of scattered words.
//
// Bound by memory: the two large steps of 64 searches on scale 20 move about
// 1 GB each (frontier words that miss L2, and lines of level and parent
// written in part) in 270 us.  32 vertices per wave keep 18 waves' LDS on a
// compute unit and a store instruction on whole lines; 64 vertices per wave
// took 295 + 276 + 93 us against 274 + 264 + 79 for the three largest steps,
// 16 (half lines) 330 + 323 + 108, one thread per row 311 + 275 + 212.
constexpr int kMsUnroll = 4;
constexpr int kMsRows = 32;   // vertices per wave

template <bool PARENT>
__global__ __launch_bounds__(kWave) void k_ms_pull_pack(MsArgs a) {
    __shared__ uint32_t s_par[PARENT ? 64 : 1][kMsRows + 1];
    __shared__ int32_t s_first[kMsRows];
    const int g = blockIdx.y;
    const uint64_t valid = group_valid(a.nsrc, g);
    const int lane = threadIdx.x;
    uint32_t cnt = 0;
    for (int64_t base = (int64_t)blockIdx.x * kMsRows; base < a.n; base += (int64_t)gridDim.x * kMsRows) {
        const int64_t v = base + lane;
        const bool in = lane < kMsRows && v < a.n;
        const int64_t vc = in ? v : a.n - 1;
        const int64_t at = vc * a.G + g;
        const int32_t b = a.rowptr[vc], len = a.rowptr[vc + 1] - b;
        const uint64_t seen = a.seen[at];
        const bool mine = in && len <= kMsLong;   // longer rows belong to the other kernels
        const uint64_t unseen = mine && len > 0 ? valid & ~seen : 0ull;
        // packed positions: row r owns [s_first[r], s_first[r] + len) when it misses a source
        const int32_t l = unseen ? len : 0;
        int32_t x = l;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int32_t y = __shfl_up(x, d);
            if (lane >= d) x += y;
        }
        const int32_t total = __shfl(x, kWave - 1);
        const int32_t delta = b - (x - l);   // entry number minus packed position
        __syncthreads();   // the previous rows' reads are done (one wave: no wait)
        if (lane < kMsRows) s_first[lane] = x - l;
        __syncthreads();
        uint64_t left = unseen;   // sources this lane's row still misses
        auto locate = [&](int32_t p0, int32_t (&rp)[kMsUnroll], uint32_t (&u)[kMsUnroll]) {
#pragma unroll
            for (int c = 0; c < kMsUnroll; ++c) {
                const int32_t p = min(p0 + c * kWave + lane, total - 1);
                int r = 0;   // the last row starting at or before p (rows with nothing packed start at their successor)
#pragma unroll
                for (int d = kMsRows / 2; d >= 1; d >>= 1)
                    if (s_first[r + d] <= p) r += d;
                rp[c] = r;
                u[c] = a.colids[p + __shfl(delta, r)];
            }
        };
        auto resolve = [&](uint32_t u, uint64_t f, int32_t rp) {
            const uint64_t any = __ballot(f != 0ull);
            if (!any) return;
            const uint64_t t = wave_transpose64(f);
            const int r0 = __builtin_amdgcn_readfirstlane(rp), r1 = __builtin_amdgcn_readlane(rp, kWave - 1);
            uint64_t rows = __ballot(left != 0ull && lane >= r0 && lane <= r1);
            while (rows) {   // uniform: the rows of this step that miss a source
                const int r = __ffsll((unsigned long long)rows) - 1;
                rows &= rows - 1ull;
                const uint64_t where = __ballot(rp == r);
                if (!(where & any)) continue;
                const uint64_t miss = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)left, r) |
                                      (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(left >> 32), r) << 32;
                const uint64_t hit = (miss >> lane) & 1ull ? t & where : 0ull;
                const uint64_t found = __ballot(hit != 0ull);
                if (!found) continue;
                if (PARENT) {
                    const uint32_t pu = (uint32_t)__shfl((int)u, hit ? __ffsll((unsigned long long)hit) - 1 : 0);
                    if (hit) s_par[lane][r] = pu;
                }
                if (lane == r) left &= ~found;
            }
        };
        if (total > 0) {
            int32_t rp[kMsUnroll], rn[kMsUnroll];
            uint32_t u[kMsUnroll], un[kMsUnroll];
            locate(0, rn, un);
            for (int32_t p0 = 0; p0 < total; p0 += kMsUnroll * kWave) {
                uint64_t f[kMsUnroll];
                const uint64_t alive = __ballot(left != 0ull);
#pragma unroll
                for (int c = 0; c < kMsUnroll; ++c) {
                    u[c] = un[c];
                    rp[c] = rn[c];
                    // a row whose sources are all found needs no more words
                    f[c] = 0ull;
                    if (p0 + c * kWave + lane < total && ((alive >> rp[c]) & 1ull))
                        f[c] = a.fcur[(int64_t)u[c] * a.G + g];
                }
                if (p0 + kMsUnroll * kWave < total) locate(p0 + kMsUnroll * kWave, rn, un);
#pragma unroll
                for (int c = 0; c < kMsUnroll; ++c) resolve(u[c], f[c] & valid, rp[c]);
            }
        }
        const uint64_t found = unseen & ~left;
        if (mine) {
            a.fnext[at] = found;
            if (found) {
                a.seen[at] = seen | found;
                cnt = 1;
            }
        }
        __syncthreads();
        // source-major stores of the new levels and parents, kPer sources at a time
        constexpr int kPer = kWave / kMsRows;
        const int row = lane & (kMsRows - 1), sub = lane / kMsRows;
        const uint64_t fr = __shfl(found, row);
        const uint64_t any = wave_or64(found);   // uniform
        for (int s0 = 0; s0 < 64; s0 += kPer) {
            if (!((any >> s0) & ((1ull << kPer) - 1ull))) continue;
            const int sb = s0 + sub;
            if ((fr >> sb) & 1ull) {
                const int64_t o = (int64_t)(64 * g + sb) * a.n + base + row;
                a.level[o] = a.lvl;
                if (PARENT) a.parent[o] = (int32_t)s_par[sb][row];
            }
        }
    }
    ms_report(a, (uint32_t)(__ballot(cnt != 0) != 0ull));
}

// Entries [b, e) of one row against the frontier masks, by one wave: lane s
// returns the first (smallest) in-neighbour whose mask has source s's bit,
// or kNoPar.  Sources outside `unseen` are not looked for; the scan stops
// once all of them are found.
//
// Bound by the chain colids -> frontier word of a step, so a step takes 64
// entries first (most rows end there) and then kMsSteps * 64, their loads in
// flight together, with the next step's column ids loaded ahead.  All
// sources of 64 entries are resolved together by one bit transpose (lane s
// then holds source s's entries as bits); with few sources left a ballot
// per source is cheaper.
constexpr uint32_t kNoPar = 0xffffffffu;
constexpr int kMsSteps = 4;
constexpr int kMsFewSources = 12;   // 12 ballots cost about what the 12 lane exchanges of a transpose do

__device__ __forceinline__ uint32_t ms_scan_row(const MsArgs& a, int g, int32_t b, int32_t e, uint64_t unseen) {
    const int lane = threadIdx.x & (kWave - 1);
    uint32_t par = kNoPar;
    uint64_t left = unseen;   // uniform
    auto resolve = [&](uint32_t u, uint64_t f) {
        f &= left;
        if (!__ballot(f != 0ull)) return;
        if (__popcll(left) > kMsFewSources) {
            const uint64_t t = wave_transpose64(f);
            const uint32_t pu = (uint32_t)__shfl((int)u, t ? __ffsll((unsigned long long)t) - 1 : 0);
            if (t) par = pu;
            left &= ~__ballot(t != 0ull);
        } else {
            uint64_t rest = left;
            while (rest) {
                const int s = __ffsll((unsigned long long)rest) - 1;
                rest &= rest - 1ull;
                const uint64_t lanes = __ballot((f >> s) & 1ull);
                if (lanes) {
                    const uint32_t pu = (uint32_t)__shfl((int)u, __ffsll((unsigned long long)lanes) - 1);
                    if (lane == s) par = pu;
                    left &= ~(1ull << s);
                }
            }
        }
    };
    // positions are unsigned: the look-ahead may pass 2^31 - 1
    const uint32_t end = (uint32_t)e;
    auto entry = [&](uint32_t k) { return a.colids[k < end ? k : end - 1u]; };   // clamped: loads stay unconditional
    auto word = [&](uint32_t u, uint32_t k) {
        const uint64_t w = a.fcur[(int64_t)u * a.G + g];
        return k < end ? w : 0ull;
    };
    uint32_t k = (uint32_t)(b + lane);
    {
        const uint32_t u = entry(k);
        uint32_t un[kMsSteps];   // ids of the next step, in flight with this one's words
#pragma unroll
        for (int c = 0; c < kMsSteps; ++c) un[c] = entry(k + kWave * (1 + c));
        resolve(u, word(u, k));
        k += kWave;
        while (left && k - (uint32_t)lane < end) {
            uint32_t uc[kMsSteps];
            uint64_t w[kMsSteps];
#pragma unroll
            for (int c = 0; c < kMsSteps; ++c) uc[c] = un[c];
#pragma unroll
            for (int c = 0; c < kMsSteps; ++c) w[c] = word(uc[c], k + kWave * c);
#pragma unroll
            for (int c = 0; c < kMsSteps; ++c) un[c] = entry(k + kWave * (kMsSteps + c));
#pragma unroll
            for (int c = 0; c < kMsSteps; ++c)
                if (left) resolve(uc[c], w[c]);
            k += kMsSteps * kWave;
        }
    }
    return par;
}

// A found row's outputs: lane s stores source s's level and parent.
template <bool PARENT>
__device__ __forceinline__ uint32_t ms_store_row(const MsArgs& a, int g, int32_t v, int64_t at, uint64_t seen,
                                                 uint32_t par) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t found = __ballot(par != kNoPar);
    if (par != kNoPar) {
        const int64_t o = (int64_t)(64 * g + lane) * a.n + v;
        a.level[o] = a.lvl;
        if (PARENT) a.parent[o] = (int32_t)par;
    }
    if (lane == 0) {
        a.fnext[at] = found;
        if (found) a.seen[at] = seen | found;
    }
    return (uint32_t)__popcll(found);
}

// Rows of kMsLong + 1 to kMsHuge entries, one wave each.
template <bool PARENT>
__global__ __launch_bounds__(kMsBlock) void k_ms_pull_long(MsArgs a) {
    const int g = blockIdx.y;
    const uint64_t valid = group_valid(a.nsrc, g);
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t nwaves = (int64_t)gridDim.x * (kMsBlock / kWave);
    const int32_t count = a.long_count[0];
    uint32_t cnt = 0;   // uniform
    for (int64_t r = (int64_t)blockIdx.x * (kMsBlock / kWave) + threadIdx.x / kWave; r < count; r += nwaves) {
        const int32_t v = a.long_rows[r];
        const int32_t b = a.rowptr[v], e = a.rowptr[v + 1];
        const int64_t at = (int64_t)v * a.G + g;
        const uint64_t seen = a.seen[at];
        const uint64_t unseen = valid & ~seen;
        if (unseen) cnt |= ms_store_row<PARENT>(a, g, v, at, seen, ms_scan_row(a, g, b, e, unseen));
        else if (lane == 0) a.fnext[at] = 0ull;
    }
    ms_report(a, cnt);
}

// Rows longer than kMsHuge entries, one workgroup each: every wave scans a
// contiguous part of the row, and the smallest in-neighbour per source over
// the waves is the row's (entries are ascending).  One wave alone walks a
// hub row's entries in one chain: on scale 20 the longest row held a step
// for 1.1 ms with 64 entries per dependent step.
constexpr int kMsHugeBlock = 1024;

template <bool PARENT>
__global__ __launch_bounds__(kMsHugeBlock) void k_ms_pull_huge(MsArgs a) {
    constexpr int NW = kMsHugeBlock / kWave;
    __shared__ uint32_t s_par[64];
    const int g = blockIdx.y;
    const uint64_t valid = group_valid(a.nsrc, g);
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = threadIdx.x / kWave;
    const int32_t count = a.long_count[1];
    uint32_t cnt = 0;
    for (int32_t r = (int32_t)blockIdx.x; r < count; r += (int32_t)gridDim.x) {
        const int32_t v = a.long_rows[a.long_cap - 1 - r];   // listed from the array's end
        const int32_t b = a.rowptr[v], e = a.rowptr[v + 1];
        const int64_t at = (int64_t)v * a.G + g;
        const uint64_t seen = a.seen[at];
        const uint64_t unseen = valid & ~seen;
        if (!unseen) {   // the same in every wave
            if (threadIdx.x == 0) a.fnext[at] = 0ull;
            continue;
        }
        if (threadIdx.x < 64) s_par[threadIdx.x] = kNoPar;
        __syncthreads();
        const int32_t part = ((e - b + NW - 1) / NW + kWave - 1) & ~(kWave - 1);
        const int32_t pb = (int32_t)min((int64_t)e, (int64_t)b + (int64_t)wid * part);
        const int32_t pe = (int32_t)min((int64_t)e, (int64_t)pb + part);
        if (pb < pe) {
            const uint32_t par = ms_scan_row(a, g, pb, pe, unseen);
            if (par != kNoPar) atomicMin(&s_par[lane], par);
        }
        __syncthreads();
        if (wid == 0) cnt |= ms_store_row<PARENT>(a, g, v, at, seen, s_par[lane]);
        __syncthreads();   // s_par is set again for the next row
    }
    if (wid == 0) ms_report(a, cnt);
}

// Rows longer than kMsLong entries, listed once per handle: those of up to
// kMsHuge entries from the array's start (count[0] of them), longer ones from
// its end (count[1]).  Both fit: each row has more than kMsLong of the nnz
// entries.
__global__ void k_ms_long_rows(const int32_t* rowptr, int32_t n, int32_t* rows, int32_t cap, int32_t* count) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const int32_t len = rowptr[v + 1] - rowptr[v];
        if (len > kMsHuge) rows[cap - 1 - atomicAdd(&count[1], 1)] = (int32_t)v;
        else if (len > kMsLong) rows[atomicAdd(&count[0], 1)] = (int32_t)v;
    }
}

// Seen masks from the per-source visited bitmaps (source s's bitmap at
// visited + s * mask_words).  A vertex with an empty row can never be
// reached in the pull direction: it is marked seen by every source so no
// later step reads its row.  A wave takes 64 vertices: lane s reads source
// s's bits of them and a transpose turns these into a mask per vertex.  With
// one load per vertex and source this took 50 us for 64 sources on a scale-20
// graph, so 13.
__global__ void k_ms_seen(MsArgs a, const uint32_t* visited, int32_t mask_words) {
    const int g = blockIdx.y;
    const uint64_t valid = group_valid(a.nsrc, g);
    const int ns = a.nsrc - 64 * g < 64 ? a.nsrc - 64 * g : 64;
    const int lane = threadIdx.x & (kWave - 1);
    for (int64_t v0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) & ~63ll; v0 < a.n;
         v0 += (int64_t)gridDim.x * blockDim.x) {
        const int64_t v = v0 + lane;
        const int64_t vc = v < a.n ? v : a.n - 1;
        const uint32_t* w = visited + (int64_t)(64 * g + min(lane, ns - 1)) * mask_words + (v0 >> 5);
        const uint32_t lo = w[0], hi = w[v0 + 32 < a.n ? 1 : 0];
        const bool empty = a.rowptr[vc + 1] == a.rowptr[vc];
        const uint64_t of_source = lane < ns ? (v0 + 32 < a.n ? (uint64_t)hi << 32 : 0ull) | lo : 0ull;
        const uint64_t bits = wave_transpose64(of_source);
        if (v < a.n) a.seen[v * a.G + g] = empty ? valid : bits;
    }
}

// Frontier masks from the per-source frontier lists (source s's entries at
// [xoff[s], xoff[s+1]) of front) into fm, cleared before.
__global__ __launch_bounds__(kMsBlock) void k_ms_front(MsArgs a, const int32_t* front, const int64_t* xoff,
                                                       uint64_t* fm) {
    __shared__ int64_t s_off[kMaxBatch + 1];
    for (int i = threadIdx.x; i <= a.nsrc; i += kMsBlock) s_off[i] = xoff[i];
    __syncthreads();
    const int64_t total = s_off[a.nsrc];
    for (int64_t p = (int64_t)blockIdx.x * kMsBlock + threadIdx.x; p < total; p += (int64_t)gridDim.x * kMsBlock) {
        int lo = 0, hi = a.nsrc - 1;   // the source whose range holds p
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_off[mid] <= p) lo = mid;
            else hi = mid - 1;
        }
        const int32_t v = front[p];
        if (v >= 0 && v < a.n)
            atomicOr(reinterpret_cast<unsigned long long*>(&fm[(int64_t)v * a.G + (lo >> 6)]), 1ull << (lo & 63));
    }
}

// Sum of the column lengths (out-degrees) of every entry of the frontier
// lists: the push direction's work for the next level.
__global__ __launch_bounds__(kMsBlock) void k_ms_degsum(const int32_t* front, const int64_t* xoff, int nsrc,
                                                        const int32_t* colptr, int32_t n, unsigned long long* out) {
    const int64_t total = xoff[nsrc];
    unsigned long long sum = 0;
    for (int64_t p = (int64_t)blockIdx.x * kMsBlock + threadIdx.x; p < total; p += (int64_t)gridDim.x * kMsBlock) {
        const int32_t v = front[p];
        if (v >= 0 && v < n) sum += (unsigned long long)(colptr[v + 1] - colptr[v]);
    }
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) sum += __shfl_xor(sum, d);
    // one add per workgroup: adds to one word queue at 6 to 12 ns each
    __shared__ unsigned long long s_sum[kMsBlock / kWave];
    if ((threadIdx.x & (kWave - 1)) == 0) s_sum[threadIdx.x / kWave] = sum;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < kMsBlock / kWave; ++w) sum += s_sum[w];
    if (sum) atomicAdd(out, sum);
}

inline unsigned grid_for_n(int64_t n, int cap) {
    int64_t g = (n + kMsBlock - 1) / kMsBlock;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (unsigned)g;
}

}  // namespace

hipError_t launch_ms_long_rows(const int32_t* rowptr, int32_t n, int32_t* rows, int32_t cap, int32_t* count,
                               hipStream_t s) {
    hipLaunchKernelGGL(k_ms_long_rows, dim3(grid_for_n(n, 4096)), dim3(kMsBlock), 0, s, rowptr, n, rows, cap, count);
    return hipGetLastError();
}

hipError_t launch_ms_to_pull(const MsArgs& a, const uint32_t* visited, int32_t mask_words, const int32_t* front,
                             const int64_t* xoff, uint64_t* fm, hipStream_t s) {
    hipLaunchKernelGGL(k_ms_seen, dim3(grid_for_n(a.n, 8192), a.G), dim3(kMsBlock), 0, s, a, visited, mask_words);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ms_front, dim3(4096), dim3(kMsBlock), 0, s, a, front, xoff, fm);
    return hipGetLastError();
}

template <bool PARENT>
static hipError_t ms_pull(const MsArgs& a, dim3 gp, dim3 gl, dim3 gh, hipStream_t s) {
    hipLaunchKernelGGL(k_ms_pull_huge<PARENT>, gh, dim3(kMsHugeBlock), 0, s, a);
    hipLaunchKernelGGL(k_ms_pull_pack<PARENT>, gp, dim3(kWave), 0, s, a);
    hipLaunchKernelGGL(k_ms_pull_long<PARENT>, gl, dim3(kMsBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_ms_pull(const MsArgs& a, bool parent, int num_cu, hipStream_t s) {
    int64_t gpack = (a.n + kMsRows - 1) / kMsRows;
    if (gpack > 65536) gpack = 65536;
    if (gpack < 1) gpack = 1;
    const dim3 gp((unsigned)gpack, a.G), gl((unsigned)(8 * num_cu), a.G), gh((unsigned)num_cu, a.G);
    // the longest rows first: they take the longest
    return parent ? ms_pull<true>(a, gp, gl, gh, s) : ms_pull<false>(a, gp, gl, gh, s);
}

hipError_t launch_ms_degsum(const int32_t* front, const int64_t* xoff, int nsrc, const int32_t* colptr, int32_t n,
                            unsigned long long* out, hipStream_t s) {
    hipLaunchKernelGGL(k_ms_degsum, dim3(512), dim3(kMsBlock), 0, s, front, xoff, nsrc, colptr, n, out);
    return hipGetLastError();
}

}  // namespace spv
