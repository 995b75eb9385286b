// Steps (a) and (b) of one y <- A x in one kernel: every selected column's
// entries become (row, Mult) pairs in row-range buckets (Algorithm 1, step
// 1), without the column tables and the product prefix of the two-kernel
// form going through memory.
//
// A workgroup takes tiles of consecutive x entries (one per thread at most),
// reads their column ranges, compacts the non-empty ones into an LDS table
// and works through the tile's products in chunks of BLOCK * ITEMS.  A
// chunk's products find their column by rank: one bit per column start, so
// product k's column is the number of set bits up to k.  The rest is the
// bucketing's: row ids and values are gathered with consecutive lanes on
// consecutive products, ranked in an LDS bucket histogram, one slot range per
// touched bucket is reserved with one global atomic, and the chunk is
// counting-sorted in LDS and written out in bucket runs.
//
// For matrices whose columns are even enough that no tile holds many chunks
// more than the others (expand_rule.h).  Else the two-kernel form's equal
// product chunks are the better split.  (Cutting long
// columns into queued pieces for idle or reserved workgroups was measured on
// scale 22 at 1 %: 30 to 38 us against 30.5 for scan and scatter, the queue's
// counters and waits costing what the scan did.)
//
// Why one kernel: the scan is a chain of round trips (x, column bounds,
// look-back across workgroups, tables out), and the bucketing begins with
// three more to read the tables back.  Nothing here needs the products'
// global positions: bucket slots are reserved, and the sums W needs are
// written per workgroup and added up by the merge.  Measured on a 64^3 grid, 50
// columns: scan 7.9 + scatter 4.5 us against 5.3 us.

#include <hip/hip_ext.h>

#include "device_ops.h"
#include "expand_rule.h"

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>

namespace spv {

namespace {

// Packed (count, sum) block scan: sum of at most 1024 lengths of at most
// kLongCol fits 21 bits, the count of non-empty columns the 11 above.
constexpr int kSumBits = 21;
constexpr int kNoSlot = -1;   // the bucket's run is dropped (overflow)
static_assert(1024ll * kLongCol < (1ll << kSumBits), "packed scan");

template <int BLOCK, int ITEMS, int SR, int XMODE>
__global__ __launch_bounds__(BLOCK) void k_expand(ExpandArgs a) {
    constexpr int C = BLOCK * ITEMS;
    static_assert(C <= kExpandMaxChunk, "bound of the fill counters");
    constexpr int WORDS = C / 32;   // column-start bits of a chunk
    extern __shared__ __align__(16) uint32_t lds_expand[];
    const int nb = a.nb;
    uint2* const stage = reinterpret_cast<uint2*>(lds_expand);                  // [C + 64] sort buffer
    int32_t* const hist = reinterpret_cast<int32_t*>(stage + C + kWave);        // [nb + 64] counts, then global slot base
    int32_t* const loff = hist + nb + kWave;                                    // [nb] chunk-local bucket offsets
    int32_t* const s_off = loff + nb;                                           // [BLOCK + 1] product offset of each column
    int32_t* const s_start = s_off + BLOCK + 1;                                 // [BLOCK] its first entry in A
    uint32_t* const s_xv = reinterpret_cast<uint32_t*>(s_start + BLOCK);        // [BLOCK] its x value
    uint32_t* const bits = s_xv + BLOCK;                                        // [WORDS] column starts in the chunk
    int32_t* const pre = reinterpret_cast<int32_t*>(bits + WORDS);              // [WORDS] columns before each word
    __shared__ int s_tmp[BLOCK / kWave + 1];
    __shared__ int s_base;
    __shared__ int s_over;   // a run of this workgroup did not fit its bucket
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wid = tid / kWave;

    const int f = a.f_dev ? ld_ctrl(a.f_dev) : a.f_host;
    // merge look-back words of this call; frontier bookkeeping
    for (int i = blockIdx.x * BLOCK + tid; i < a.lb3_n; i += gridDim.x * BLOCK) a.lb3[i] = 0;
    if (blockIdx.x == 0 && tid == 0) {
        if (!a.f_dev) st_ctrl(&a.ctrl->f, f);
        if (a.bump_level && f > 0) st_ctrl(&a.ctrl->level, ld_ctrl(&a.ctrl->level) + 1);
    }
    for (int i = tid; i < nb + kWave; i += BLOCK) hist[i] = 0;
    for (int i = tid; i < WORDS; i += BLOCK) bits[i] = 0u;
    if (tid == 0) s_over = 0;
    const int tl = a.tile_log2;
    // x entries per tile: the host's choice, or for a device-known f the same
    // number of tiles for every workgroup, as few as the tiles' bounds allow
    int per = a.per_tile;
    if (a.f_dev) {
        const int wide = (int)gridDim.x * a.per_max;   // of one round of tiles
        const int all = (int)gridDim.x * max(1, (f + wide - 1) / wide);
        per = max(a.per_min, (f + all - 1) / all);
    }
    const int ntiles = (f + per - 1) / per;

    // the slots [base, top) of the bucket this thread reserves for
    int base = 0, top = 0;
    if (nb <= BLOCK && tid < nb) {
        const int r0 = tid << tl;
        base = a.rcp[r0];
        top = a.rcp[(int)min((int64_t)r0 + (int64_t(1) << tl), (int64_t)a.m)];
    }

    // The products of `ncols` columns in the LDS table, `total` in all.  After
    // a run that did not fit (repeated x indices, reported) nothing more is
    // added, which bounds the fill counters.
    auto bucket_products = [&](int ncols, int total) {
        if (tid == 0) s_base = 0;
        __syncthreads();   // the table and the cleared bits are written
        for (int q0 = 0; q0 < total; q0 += C) {
            const int cnt = min(C, total - q0);
            if (tid < ncols) {
                const int o = s_off[tid] - q0;
                if (o >= 0 && o < C) atomicOr(&bits[o >> 5], 1u << (o & 31));
            }
            __syncthreads();
            if (wid == 0) {   // columns before each word
                constexpr int PER = WORDS / kWave > 0 ? WORDS / kWave : 1;
                int p[PER], sum = 0;
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const int w = lane * PER + i;
                    p[i] = w < WORDS ? __popc(bits[w]) : 0;
                    sum += p[i];
                }
                const int x = wave_inclusive_i32(sum);
                int run = s_base + x - sum;
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    const int w = lane * PER + i;
                    if (w < WORDS) pre[w] = run;
                    run += p[i];
                }
                if (lane == kWave - 1) s_base = run;   // read by this wave's lanes above (in order)
            }
            __syncthreads();
            // (1) gather + rank, lanes on consecutive products.  Every load,
            // LDS atomic and LDS read below is unconditional (a product past
            // the chunk or dropped by the mask counts in a counter of its
            // lane's own and is sorted to a slot of its lane's own), and each
            // group is issued as a whole before its first use: left to the
            // compiler, conditions become branches and the groups chains of
            // single LDS round trips.
            int32_t row[ITEMS], slot[ITEMS];
            uint32_t val[ITEMS];
            bool ok[ITEMS];
            {
                int32_t col[ITEMS], before[ITEMS];
                uint32_t word[ITEMS], xcol[ITEMS];
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) {
                    const int k = i * BLOCK + tid;
                    word[i] = bits[k >> 5];
                    before[i] = pre[k >> 5];
                }
                loaded(word);
                loaded(before);
                const uint32_t upto = (2u << (tid & 31)) - 1u;
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) col[i] = before[i] + __popc(word[i] & upto) - 1;
                int32_t st[ITEMS], of[ITEMS];
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) {
                    st[i] = s_start[col[i]];
                    of[i] = s_off[col[i]];
                    xcol[i] = s_xv[col[i]];
                }
                loaded(st);
                loaded(of);
                loaded(xcol);
                int32_t q[ITEMS];
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) {
                    const int k = i * BLOCK + tid;
                    ok[i] = k < cnt;
                    q[i] = ok[i] ? st[i] + (q0 + k - of[i]) : 0;
                }
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) row[i] = a.rowids[q[i]];
                if (SR != SR_MIN_SELECT2ND && a.values) {
                    float av[ITEMS];
#pragma unroll
                    for (int i = 0; i < ITEMS; ++i) av[i] = a.values[q[i]];
                    loaded(av);
#pragma unroll
                    for (int i = 0; i < ITEMS; ++i) val[i] = mult_value<SR>(av[i], xcol[i]);
                } else {
#pragma unroll
                    for (int i = 0; i < ITEMS; ++i) val[i] = mult_value<SR>(1.0f, xcol[i]);
                }
                loaded(row);
            }
            if (a.mask) {
                uint32_t mw[ITEMS];
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) mw[i] = a.mask[(uint32_t)row[i] >> 5];
                loaded(mw);
#pragma unroll
                for (int i = 0; i < ITEMS; ++i)
                    ok[i] = ok[i] && ((mw[i] >> (row[i] & 31)) & 1u) == (uint32_t)a.mask_keep;
            }
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) slot[i] = atomicAdd(&hist[ok[i] ? row[i] >> tl : nb + lane], 1);
            loaded(slot);
            __syncthreads();
            for (int i = tid; i < WORDS; i += BLOCK) bits[i] = 0u;
            // (2) chunk-local offsets and one slot reservation per touched
            // bucket, whose round trip overlaps the counting sort (3)
            auto sort = [&]() {
                int32_t o[ITEMS];
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) o[i] = loff[ok[i] ? row[i] >> tl : 0];
                loaded(o);
#pragma unroll
                for (int i = 0; i < ITEMS; ++i)
                    stage[ok[i] ? o[i] + slot[i] : C + lane] = make_uint2((uint32_t)row[i], val[i]);
            };
            int kept;
            if (nb <= BLOCK) {
                const int b = tid;
                const int n = b < nb ? hist[b] : 0;
                const int e = block_exclusive_i32<BLOCK>(n, s_tmp, kept);
                int g[1] = {0};
                if (b < nb) loff[b] = e;
                if (n > 0) g[0] = atomicAdd(&a.cursor[b], n);
                __syncthreads();
                sort();
                loaded(g);   // not before the sort
                if (n > 0) {
                    if (!slots_fit(g[0], n, top - base)) {
                        atomicOr(&a.ctrl->err, ERR_BUCKET_OVERFLOW);
                        s_over = 1;
                        hist[b] = kNoSlot;
                    } else {
                        hist[b] = base + g[0];
                    }
                }
                __syncthreads();
            } else {
                int carry = 0;
                for (int b0 = 0; b0 < nb; b0 += BLOCK) {
                    const int b = b0 + tid;
                    const int n = b < nb ? hist[b] : 0;
                    int tot;
                    const int e = block_exclusive_i32<BLOCK>(n, s_tmp, tot);
                    if (b < nb) {
                        loff[b] = carry + e;
                        if (n > 0) {
                            const int r0 = b << tl;
                            const int base = a.rcp[r0];
                            const int cap = a.rcp[(int)min((int64_t)r0 + (int64_t(1) << tl), (int64_t)a.m)] - base;
                            const int g = atomicAdd(&a.cursor[b], n);
                            if (!slots_fit(g, n, cap)) {
                                atomicOr(&a.ctrl->err, ERR_BUCKET_OVERFLOW);
                                s_over = 1;
                                hist[b] = kNoSlot;
                            } else {
                                hist[b] = base + g;
                            }
                        }
                    }
                    carry += tot;
                }
                kept = carry;
                __syncthreads();
                sort();
                __syncthreads();
            }
            // (4) coalesced write-out of the bucket runs
            {
                uint2 e[ITEMS];
                int gb[ITEMS], lo[ITEMS];
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) e[i] = stage[i * BLOCK + tid];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) {
                    const int b = i * BLOCK + tid < kept ? (int)e[i].x >> tl : 0;
                    gb[i] = hist[b];
                    lo[i] = loff[b];
                }
                loaded(gb);
                loaded(lo);
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) {
                    const int t = i * BLOCK + tid;
                    if (t < kept && gb[i] != kNoSlot) a.buckets[(int64_t)gb[i] + (t - lo[i])] = e[i];
                }
            }
            __syncthreads();
            if (q0 + C < total && s_over) break;   // uniform: set before a barrier that every thread has passed
            for (int i = tid; i < nb; i += BLOCK) hist[i] = 0;
        }
    };

    int64_t sum_w = 0;
    int32_t sum_c = 0, lmax = 0;
    // One tile's x entry of this thread: its column's first entry and length.
    auto column = [&](int tile, int32_t* st, int32_t* len, uint32_t* xv) {
        const int64_t p = (int64_t)tile * per + tid;
        const bool in = tid < per && p < f;
        const int32_t j = in ? a.x_idx[p] : -1;
        const bool inr = j >= 0 && j < a.n;
        *xv = in ? x_value<XMODE>(a.x_val, (int)p, j) : 0u;
        *st = 0;
        *len = 0;
        if (a.dcsc) {
            // DCSC: find column j among the stored ones through its chunk of
            // the column index (a few candidates), else it is empty.
            if (inr) {
                const int c = j >> a.dc_shift;
                int32_t lo = a.dc_aux[c];
                const int32_t end = a.dc_aux[c + 1];
                int32_t hi = end;
                while (lo < hi) {
                    const int32_t mid = (lo + hi) >> 1;
                    if (a.dc_jc[mid] < j) lo = mid + 1;
                    else hi = mid;
                }
                if (lo < end && a.dc_jc[lo] == j) {
                    *st = a.colptr[lo];
                    *len = a.colptr[lo + 1] - *st;
                }
            }
        } else {
            const int32_t jc = inr ? j : 0;
            const int32_t b0 = a.colptr[jc], b1 = a.colptr[jc + 1];
            *st = b0;
            *len = inr ? b1 - b0 : 0;
        }
        if (in && !inr) atomicOr(&a.ctrl->err, ERR_X_RANGE);
    };
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        int32_t st, len;
        uint32_t xv;
        column(tile, &st, &len, &xv);
        sum_w += len;
        sum_c += len > 0;
        lmax = max(lmax, len);
        int packed;
        const int e = block_exclusive_i32<BLOCK>(len | (len > 0 ? 1 << kSumBits : 0), s_tmp, packed);
        if (len > 0) {
            const int c = e >> kSumBits;
            s_off[c] = e & ((1 << kSumBits) - 1);
            s_start[c] = st;
            s_xv[c] = xv;
        }
        bucket_products((int)((uint32_t)packed >> kSumBits), packed & ((1 << kSumBits) - 1));
        __syncthreads();   // the table is written again
        if (tile + (int)gridDim.x < ntiles && s_over) break;
    }
    // this workgroup's share of the call's statistics (added up by the merge)
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) {
        sum_w += __shfl_xor(sum_w, d, kWave);
        sum_c += __shfl_xor(sum_c, d, kWave);
        lmax = max(lmax, __shfl_xor(lmax, d, kWave));
    }
    __syncthreads();
    int64_t* const s_w = reinterpret_cast<int64_t*>(stage);
    int32_t* const s_c = reinterpret_cast<int32_t*>(s_w + BLOCK / kWave);
    if (lane == 0) {
        s_w[wid] = sum_w;
        s_c[2 * wid] = sum_c;
        s_c[2 * wid + 1] = lmax;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < BLOCK / kWave; ++w) {
            sum_w += s_w[w];
            sum_c += s_c[2 * w];
            lmax = max(lmax, s_c[2 * w + 1]);
        }
        ExpandStat st;
        st.products = sum_w;
        st.columns = sum_c;
        st.longest = lmax;
        a.stat[blockIdx.x] = st;
    }
}

template <typename K>
hipError_t allow_lds(K kernel, size_t bytes) {
    if (bytes <= 65536) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)bytes);
}

template <int B, int I>
struct Shape {
    static constexpr int block = B, items = I;
};

// Calls op with the kernel of a (block, items, semiring, x mode); the value
// of op, or `none` for a combination that does not exist.
template <typename R, typename Op>
R with_kernel(int block, int items, int semiring, int xmode, R none, Op op) {
    auto by_mode = [&](auto shape) -> R {
        constexpr int B = decltype(shape)::block, I = decltype(shape)::items;
        if (semiring == SR_PLUS_TIMES) return xmode == XV_BITS32 ? op(k_expand<B, I, SR_PLUS_TIMES, XV_BITS32>) : none;
        if (semiring == SR_MIN_SELECT2ND) {
            if (xmode == XV_BITS32) return op(k_expand<B, I, SR_MIN_SELECT2ND, XV_BITS32>);
            return xmode == XV_INDEX ? op(k_expand<B, I, SR_MIN_SELECT2ND, XV_INDEX>) : none;
        }
        if (xmode == XV_U8) return op(k_expand<B, I, SR_OR_AND, XV_U8>);
        return xmode == XV_TRUE ? op(k_expand<B, I, SR_OR_AND, XV_TRUE>) : none;
    };
    switch (block * 16 + items) {
        case 256 * 16 + 4: return by_mode(Shape<256, 4>{});
        case 256 * 16 + 8: return by_mode(Shape<256, 8>{});
        case 256 * 16 + 16: return by_mode(Shape<256, 16>{});
        case 512 * 16 + 4: return by_mode(Shape<512, 4>{});
        case 512 * 16 + 8: return by_mode(Shape<512, 8>{});
        case 1024 * 16 + 4: return by_mode(Shape<1024, 4>{});
        case 1024 * 16 + 8: return by_mode(Shape<1024, 8>{});
    }
    return none;
}

}  // namespace

size_t expand_lds_bytes(int nb, int block, int items) {
    const size_t chunk = size_t(block) * items;
    return (chunk + kWave) * 8 + (size_t(nb) * 2 + kWave) * 4 + (size_t(block) * 3 + 1) * 4 + chunk / 32 * 8;
}

// Workgroups one compute unit holds at once, as the runtime computes it from
// the kernel's registers, LDS and threads.
int expand_resident(int semiring, int xmode, int block, int items, int nb) {
    static std::mutex mu;
    static std::map<std::tuple<int, int, int, int, int, int>, int> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = -1;
    const auto key = std::make_tuple(dev, semiring, xmode, block, items, nb);
    {
        std::lock_guard<std::mutex> g(mu);
        const auto it = cache.find(key);
        if (it != cache.end()) return it->second;
    }
    const size_t lds = expand_lds_bytes(nb, block, items);
    int n = with_kernel(block, items, semiring, xmode, 1, [&](auto kern) {
        int r = 0;
        if (allow_lds(kern, lds) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&r, reinterpret_cast<const void*>(kern), block, lds) !=
                hipSuccess)
            return 1;
        return r;
    });
    if (n < 1) n = 1;
    std::lock_guard<std::mutex> g(mu);
    cache[key] = n;
    return n;
}

hipError_t launch_expand(const ExpandArgs& a, int semiring, int xmode, int block, int items, int grid, hipStream_t s,
                         const LaunchEvents* ev) {
    if (grid < 1 || grid > kExpandMaxGrid || a.per_tile < 1 || a.per_tile > block || a.per_min < 1 ||
        a.per_max < a.per_min || a.per_max > block)
        return hipErrorInvalidValue;
    const size_t lds = expand_lds_bytes(a.nb, block, items);
    return with_kernel(block, items, semiring, xmode, hipErrorInvalidValue, [&](auto kern) {
        const hipError_t e = allow_lds(kern, lds);
        if (e != hipSuccess) return e;
        if (ev) hipExtLaunchKernelGGL(kern, dim3(grid), dim3(block), (uint32_t)lds, s, ev->start, ev->stop, 0, a);
        else hipLaunchKernelGGL(kern, dim3(grid), dim3(block), lds, s, a);
        return hipGetLastError();
    });
}

}  // namespace spv
