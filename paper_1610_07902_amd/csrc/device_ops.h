// Device helpers shared by the bucketing kernels, the one-launch multiply
// and the masked multiply: agent-scope control-word access, the decoupled
// look-back, block-wide scans, reading x values, the semiring's Mult, and
// the merge's tile accumulation.  Not installed.
#pragma once

#include "internal.h"

namespace spv {

constexpr uint64_t LB_AGG = 1ull << 62;
constexpr uint64_t LB_INC = 2ull << 62;
constexpr uint64_t LB_VAL = (1ull << 62) - 1;
constexpr int kSpinMax = 1 << 20;

__device__ __forceinline__ uint64_t ld_acquire64(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_release64(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Control words written by an earlier kernel (plain stores or atomics) are
// read with agent-scope atomic loads, never through the scalar cache.
__device__ __forceinline__ int32_t ld_ctrl(const int32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t* ld_ctrl_ptr(int32_t* const* p) {
    return reinterpret_cast<int32_t*>(__hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void st_ctrl(int32_t* p, int32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_ctrl_u(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A waiting call's results to the host (system scope: pinned memory), by one
// thread of the call's last kernel; an error bit that this kernel itself
// raises is reported by raise_err, wherever it happens.
__device__ __forceinline__ void report_nnz(Report* rep, const Ctrl* ctrl, int64_t nnz) {
    if (!rep) return;
    const uint32_t err = __hip_atomic_load(&ctrl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&rep->nnz, nnz, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&rep->err, err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&rep->state, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void raise_err(uint32_t* err, uint32_t bits, Report* rep) {
    atomicOr(err, bits);
    if (rep) __hip_atomic_store(&rep->bad, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

// Decoupled look-back over per-tile state words (status in bits 63:62,
// value in 61:0).  Called by all 64 lanes of one wave.  Publishes `agg` for
// `tile`, returns the exclusive prefix and publishes the inclusive one.  K
// words per lane and round trip: predecessors that all finish at about the
// same time leave only sums, which one round of 64 * K covers.
// A wait that exceeds kSpinMax polls sets ERR_SPIN and returns a partial
// prefix rather than hanging.
__device__ __forceinline__ void publish_sum(uint64_t* st, int tile, uint64_t agg) {
    st_release64(&st[tile], (tile == 0 ? LB_INC : LB_AGG) | (agg & LB_VAL));
}

template <int K = 1>
__device__ inline uint64_t lookback(uint64_t* st, int tile, uint64_t agg, uint32_t* err, Report* rep = nullptr) {
    const int lane = threadIdx.x & (kWave - 1);
    if (lane == 0) publish_sum(st, tile, agg);
    if (tile == 0) return 0;
    uint64_t excl = 0;
    int base = tile - 1;
    int spins = 0;
    for (bool done = false; !done;) {
        uint64_t w[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int idx = base - k * kWave - lane;
            w[k] = idx >= 0 ? ld_acquire64(&st[idx]) : LB_INC;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint64_t status = w[k] >> 62;
            const uint64_t inc_mask = __ballot(status == 2);
            const uint64_t empty_mask = __ballot(status == 0);
            const uint64_t need = inc_mask ? (((inc_mask & (~inc_mask + 1)) << 1) - 1) : ~0ull;
            if (empty_mask & need) {   // not there yet: look again from here
                if (++spins > kSpinMax) {
                    if (lane == 0) raise_err(err, ERR_SPIN, rep);
                    done = true;
                }
                __builtin_amdgcn_s_sleep(1);
                break;
            }
            const uint64_t v = ((need >> lane) & 1ull) ? (w[k] & LB_VAL) : 0ull;
            excl += wave_sum_u64(v);
            if (inc_mask) {
                done = true;
                break;
            }
            base -= kWave;
        }
    }
    if (lane == 0) st_release64(&st[tile], LB_INC | ((excl + agg) & LB_VAL));
    return excl;
}

template <int BLOCK>
__device__ __forceinline__ uint64_t block_exclusive_u64(uint64_t v, uint64_t* s_tmp, uint64_t& total) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = threadIdx.x / kWave;
    uint64_t x = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint64_t y = __shfl_up(x, d, kWave);
        if (lane >= d) x += y;
    }
    if (lane == kWave - 1) s_tmp[wid] = x;
    __syncthreads();
    // every lane reads the wave totals (broadcast reads, independent of
    // each other) instead of one thread summing them in sequence
    uint64_t pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < BLOCK / kWave; ++w) {
        const uint64_t t = s_tmp[w];
        pre += w < wid ? t : 0;
        tot += t;
    }
    total = tot;
    __syncthreads();   // s_tmp is reused by the next scan
    return pre + x - v;
}

// Inclusive sum over the wave's lanes with data-parallel moves (shifts within
// rows of 16 lanes, then the rows' last lanes broadcast): register moves
// where __shfl_up goes through LDS six times in a row.
__device__ __forceinline__ int wave_inclusive_i32(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return x;
}

// Every load of the array is issued before this point and every use comes
// after it: neither a later condition nor the register allocator's ordering
// turns the loads into a chain of single round trips.
template <typename T, int K>
__device__ __forceinline__ void loaded(T (&v)[K]) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < K; ++i) asm volatile("" : "+v"(v[i]));
}

template <int BLOCK>
__device__ __forceinline__ int block_exclusive_i32(int v, int* s_tmp, int& total) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = threadIdx.x / kWave;
    const int x = wave_inclusive_i32(v);
    if (lane == kWave - 1) s_tmp[wid] = x;
    __syncthreads();
    // every lane reads the wave totals (broadcast reads, independent of
    // each other) instead of one thread summing them in sequence
    int pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < BLOCK / kWave; ++w) {
        const int t = s_tmp[w];
        pre += w < wid ? t : 0;
        tot += t;
    }
    total = tot;
    __syncthreads();   // s_tmp is reused by the next scan
    return pre + x - v;
}

// The call's statistics from the expansion phase's per-workgroup sums, by one
// workgroup of the merge.
template <int BLOCK>
__device__ __forceinline__ void collect_stats(const MergeArgs& a) {
    __shared__ int64_t s_w[BLOCK / kWave];
    __shared__ int32_t s_c[BLOCK / kWave], s_l[BLOCK / kWave];
    int64_t w = 0;
    int32_t c = 0, l = 0;
    for (int i = threadIdx.x; i < a.stat_n; i += BLOCK) {
        const ExpandStat st = a.stat[i];
        w += st.products;
        c += st.columns;
        l = max(l, st.longest);
    }
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) {
        w += __shfl_xor(w, d, kWave);
        c += __shfl_xor(c, d, kWave);
        l = max(l, __shfl_xor(l, d, kWave));
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        s_w[threadIdx.x / kWave] = w;
        s_c[threadIdx.x / kWave] = c;
        s_l[threadIdx.x / kWave] = l;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 1; k < BLOCK / kWave; ++k) {
        w += s_w[k];
        c += s_c[k];
        l = max(l, s_l[k]);
    }
    if (w > a.nnz) raise_err(&a.ctrl->err, ERR_BUCKET_OVERFLOW, a.rep);
    st_ctrl(&a.ctrl->W_last, w > a.nnz ? 0 : (int32_t)w);
    st_ctrl(&a.ctrl->fnz_last, c);
    st_ctrl(&a.ctrl->maxlen_last, l);
}

template <int XMODE>
__device__ __forceinline__ uint32_t x_value(const void* x_val, int p, int32_t j) {
    if constexpr (XMODE == XV_BITS32) return reinterpret_cast<const uint32_t*>(x_val)[p];
    else if constexpr (XMODE == XV_INDEX) return (uint32_t)j;
    else if constexpr (XMODE == XV_U8) return reinterpret_cast<const uint8_t*>(x_val)[p] ? 1u : 0u;
    else return 1u;
}

// The semiring's Mult of a stored entry's value and an x value.
template <int SR>
__device__ __forceinline__ uint32_t mult_value(float av, uint32_t xbits) {
    if constexpr (SR == SR_PLUS_TIMES) return __float_as_uint(__fmul_rn(av, __uint_as_float(xbits)));
    else if constexpr (SR == SR_MIN_SELECT2ND) return xbits;
    else return (av != 0.0f ? 1u : 0u) & (xbits != 0u ? 1u : 0u);
}

template <int SR>
__device__ __forceinline__ uint32_t mult(const float* values, int32_t q, uint32_t xbits) {
    if constexpr (SR == SR_PLUS_TIMES) {
        const float av = values ? values[q] : 1.0f;
        return __float_as_uint(__fmul_rn(av, __uint_as_float(xbits)));
    } else if constexpr (SR == SR_MIN_SELECT2ND) {
        return xbits;
    } else {
        const uint32_t av = values ? (values[q] != 0.0f ? 1u : 0u) : 1u;
        return av & (xbits != 0u ? 1u : 0u);
    }
}

template <int SR>
__device__ __forceinline__ uint32_t identity() {
    if constexpr (SR == SR_PLUS_TIMES) return 0u;            // +0.0f
    else if constexpr (SR == SR_MIN_SELECT2ND) return 0x7fffffffu;
    else return 0u;
}

template <int SR>
__device__ __forceinline__ void accumulate(uint32_t* cell, uint32_t v) {
    if constexpr (SR == SR_PLUS_TIMES) atomicAdd(reinterpret_cast<float*>(cell), __uint_as_float(v));
    else if constexpr (SR == SR_MIN_SELECT2ND) atomicMin(reinterpret_cast<int*>(cell), (int)v);
    else atomicOr(cell, v);
}

template <int SR>
__device__ __forceinline__ void store_value(void* y_val, int64_t o, uint32_t v) {
    if constexpr (SR == SR_OR_AND) reinterpret_cast<uint8_t*>(y_val)[o] = (uint8_t)(v != 0u);
    else reinterpret_cast<uint32_t*>(y_val)[o] = v;
}



// Tile accumulation.  Measured on gfx950 (random addresses in a 128 KB
// tile, every lane of 256 workgroups of 1024 threads): an LDS add of a
// 64-bit float retires about 2 lanes per cycle per compute unit, and keeps
// that rate when a third of the lanes hit a few dozen hub rows; a 32-bit
// float add retires about a third of a lane per cycle, and a
// compare-and-swap loop on a 32-bit word about 1.9 on distinct rows but half
// a lane once hub rows make lanes retry.  So plus-times accumulates every
// row in fp64 and rounds it to fp32 once, when y is written: faster, and the
// rounding error no longer grows with the number of terms of a row (fp32
// sums of a few hundred thousand terms in arbitrary order drift past 1e-5).
// An fp64 cell starts at -0.0, which only a sum whose every term is -0.0
// reproduces: such a product also sets the row's bitmap bit, and every other
// touched row is the one whose cell is no longer -0.0 (a ballot pass after
// the accumulation sets its bit).  min and or use their native integer
// atomics and set the bitmap bit with every entry.
constexpr uint64_t kNegZero64 = 0x8000000000000000ull;

// The adds alone, for rows whose bits are set already.
template <int SR, int K>
__device__ __forceinline__ void add_values(const uint32_t (&r)[K], const uint32_t (&v)[K], const bool (&ok)[K],
                                           uint32_t* spa) {
#pragma unroll
    for (int u = 0; u < K; ++u) {
        if (!ok[u]) continue;
        if constexpr (SR == SR_PLUS_TIMES)
            atomicAdd(&reinterpret_cast<double*>(spa)[r[u]], (double)__uint_as_float(v[u]));
        else accumulate<SR>(&spa[r[u]], v[u]);
    }
}

// Adds and bitmap bits of a long bucket, without a branch per entry: a lane
// that has none adds the neutral value to one of the first 32 cells.
// mark: plus-times sets every entry's bit here (a bucket with few entries,
// where one atomic per entry is cheaper than the ballot pass over the whole
// tile); otherwise only those of -0.0 products, and touched_bits64 finds the
// rest.
template <int SR, int K>
__device__ __forceinline__ void add_rows(const uint32_t (&r)[K], const uint32_t (&v)[K], const bool (&ok)[K],
                                         uint32_t* spa, uint32_t* bm, bool mark = false) {
    constexpr bool kSum = SR == SR_PLUS_TIMES;
    const uint32_t kNone = kSum ? 0x80000000u : identity<SR>();
    bool bits = !kSum || mark;
#pragma unroll
    for (int u = 0; u < K; ++u) {
        const uint32_t c = ok[u] ? r[u] : threadIdx.x & 31u;
        const uint32_t w = ok[u] ? v[u] : kNone;
        if constexpr (kSum) {
            atomicAdd(&reinterpret_cast<double*>(spa)[c], (double)__uint_as_float(w));
            bits |= ok[u] & (v[u] == kNone);
        } else {
            accumulate<SR>(&spa[c], w);
        }
    }
    if (!__any(bits)) return;
#pragma unroll
    for (int u = 0; u < K; ++u) {
        const uint32_t c = ok[u] ? r[u] : threadIdx.x & 31u;
        atomicOr(&bm[c >> 5], ok[u] & (!kSum | mark | (v[u] == kNone)) ? 1u << (c & 31u) : 0u);
    }
}

// One row's entries, summed in a register per lane instead of in the row's
// LDS cell.  Lanes of a wave that add to one cell wait for each other, and a
// hub row brings a good part of every wave's lanes there.
template <int SR>
struct HubSum {
    uint32_t row = ~0u;   // matches no row
    bool any = false;     // this lane took an entry
    uint32_t acc = identity<SR>();
    double sum = -0.0;

    // Takes the row's entries out of r, v, ok.  -0.0 products stay with the
    // cells, where they set the row's bit.
    template <int K>
    __device__ __forceinline__ void take(const uint32_t (&r)[K], const uint32_t (&v)[K], bool (&ok)[K]) {
#pragma unroll
        for (int u = 0; u < K; ++u) {
            bool hit = ok[u] & (r[u] == row);
            if constexpr (SR == SR_PLUS_TIMES) {
                hit &= v[u] != 0x80000000u;
                sum += hit ? (double)__uint_as_float(v[u]) : -0.0;
            } else if constexpr (SR == SR_MIN_SELECT2ND) {
                acc = hit ? (uint32_t)min((int)acc, (int)v[u]) : acc;
            } else {
                acc |= hit ? v[u] : 0u;
            }
            any |= hit;
            ok[u] &= !hit;
        }
    }
    // adds what the wave's lanes took to the row (all 64 lanes)
    __device__ __forceinline__ void flush(uint32_t* spa, uint32_t* bm) {
        if (!__any(any)) return;
        const int lane = threadIdx.x & (kWave - 1);
        if constexpr (SR == SR_PLUS_TIMES) {
            for (int d = kWave / 2; d; d >>= 1) sum += __shfl_xor(sum, d);
            if (lane == 0) atomicAdd(&reinterpret_cast<double*>(spa)[row], sum);
        } else {
            for (int d = kWave / 2; d; d >>= 1) {
                const uint32_t o = __shfl_xor(acc, d);
                if constexpr (SR == SR_MIN_SELECT2ND) acc = (uint32_t)min((int)acc, (int)o);
                else acc |= o;
            }
            if (lane == 0) {
                accumulate<SR>(&spa[row], acc);
                atomicOr(&bm[row >> 5], 1u << (row & 31u));
            }
        }
    }
};

// The most frequent of kTry rows sampled from a wave's K * 64 entries, as
// count << 16 | row (rows < 2^15), for a maximum over waves.
template <int K>
__device__ __forceinline__ uint32_t frequent_row(const uint32_t (&r)[K], const bool (&ok)[K]) {
    constexpr int kTry = 4;
    uint32_t best = 0;
    const int wid = threadIdx.x / kWave;
#pragma unroll
    for (int c = 0; c < kTry; ++c) {
        const uint32_t cand = __builtin_amdgcn_readlane(r[c % K], (c * kWave / kTry + wid) & (kWave - 1));
        int n = 0;
#pragma unroll
        for (int u = 0; u < K; ++u) n += __popcll(__ballot(ok[u] && r[u] == cand));
        if (n) best = max(best, (uint32_t)n << 16 | cand);
    }
    return best;
}

// Bitmap bits of the fp64 cells a plus-times entry reached (cell no longer
// -0.0): a wave reads kTouched runs of 64 consecutive cells (conflict-free
// 8-byte LDS reads, all in flight together), lane s keeps the ballot of run s,
// and each writes its two bitmap words at the end (nothing else writes them
// after the accumulation).  With a read-modify-write of the bitmap per run
// the pass over a 16384-row tile took 6 us, so 1.
constexpr int kTouched = 8;
template <int BLOCK>
__device__ __forceinline__ void touched_bits64(const uint32_t* spa, uint32_t* bm, int rows) {
    const uint64_t* c64 = reinterpret_cast<const uint64_t*>(spa);
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = threadIdx.x / kWave;
    for (int c0 = wid * kTouched * kWave; c0 < rows; c0 += BLOCK * kTouched) {
        uint64_t cell[kTouched], mine = 0;
#pragma unroll
        for (int s = 0; s < kTouched; ++s) cell[s] = c64[min(c0 + s * kWave + lane, rows - 1)];
#pragma unroll
        for (int s = 0; s < kTouched; ++s) {
            const uint64_t b = __ballot(cell[s] != kNegZero64 && c0 + s * kWave + lane < rows);
            mine = lane == s ? b : mine;
        }
        const int c = c0 + lane * kWave;   // first row of this lane's run
        if (lane < kTouched && c < rows) {
            bm[c >> 5] |= (uint32_t)mine;
            if (c + 32 < rows) bm[(c >> 5) + 1] |= (uint32_t)(mine >> 32);
        }
    }
}

// Append the taken entries of one tile of BLOCK * K list positions (item i of
// thread t is position i * BLOCK + t) to a list in position order: ballots
// give each wave its counts per item, one exclusive scan over (item, wave)
// in LDS places them, and the tile takes its slots with ONE counter update.
// A counter update per wave and item instead (23K updates of one word for
// 1.5M entries) serialised at the counter: 150 us against about 15 us for
// the step with one per tile.  s_cnt holds K * BLOCK / 64 + 1 ints.
template <int BLOCK, int K>
__device__ __forceinline__ void append_tile(const bool (&take)[K], const int32_t (&idx)[K], const uint32_t (&val)[K],
                                            int32_t* x_idx, uint32_t* x_val, int32_t* counter, int* s_cnt) {
    constexpr int NW = BLOCK / kWave, N = K * NW;
    static_assert(N <= kWave, "the (item, wave) counts are scanned by one wave");
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = threadIdx.x / kWave;
    int below[K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const uint64_t vote = __ballot(take[i]);
        below[i] = (int)__popcll(vote & ((1ull << lane) - 1ull));
        if (lane == 0) s_cnt[i * NW + wid] = (int)__popcll(vote);
    }
    __syncthreads();
    if (wid == 0) {
        const int c = lane < N ? s_cnt[lane] : 0;
        int x = c;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int y = __shfl_up(x, d, kWave);
            if (lane >= d) x += y;
        }
        const int total = __shfl(x, kWave - 1, kWave);
        int first = 0;
        if (lane == 0 && total > 0) first = atomicAdd(counter, total);
        first = __shfl(first, 0, kWave);
        if (lane < N) s_cnt[lane] = first + x - c;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < K; ++i)
        if (take[i]) {
            const int p = s_cnt[i * NW + wid] + below[i];
            x_idx[p] = idx[i];
            x_val[p] = val[i];
        }
    __syncthreads();   // s_cnt is reused by the next tile
}

// End of a list-building step (PageRank, connected components): the last
// workgroup to finish publishes the next x's length and counts the multiply
// that just ran if it had input.  Every append's counter update returned
// before its workgroup's arrival, so the last arrival sees them all.
__device__ __forceinline__ void finish_step(Ctrl* ctrl) {
    if (threadIdx.x != 0) return;
    if (atomicAdd(&ctrl->step_done, 1u) + 1u != gridDim.x) return;
    const int32_t fp = ld_ctrl(&ctrl->f);
    if (fp > 0) st_ctrl(&ctrl->level, ld_ctrl(&ctrl->level) + 1);
    st_ctrl(&ctrl->f, ld_ctrl(&ctrl->gen_count));
    st_ctrl(&ctrl->gen_count, 0);
    st_ctrl_u(&ctrl->step_done, 0u);
}

// Tiles of the list-building steps: 256 threads, 8 entries each, all of a
// thread's loads in flight together.
constexpr int kStepBlock = 256;
constexpr int kStepItems = 8;
constexpr int kStepTile = kStepBlock * kStepItems;
inline int step_grid(int64_t count) {
    int64_t g = (count + kStepTile - 1) / kStepTile;
    if (g < 1) g = 1;
    if (g > 2048) g = 2048;
    return (int)g;
}

}  // namespace spv
