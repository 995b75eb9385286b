// Connected components by data-driven label propagation around the SpMSpV
// hot path (the paper's introduction lists connected components among the
// data-driven uses of SpMSpV):
//   label(v) = v for every vertex; the first x lists every vertex with an
//   out-edge, valued by its label;
//   each step: y = A x over min-select2nd (y(i) = the smallest label among
//   x's in-neighbours of i); every i with y(i) < label(i) takes y(i) and
//   joins the next x (when it has out-edges); stop when x is empty.
// At the fixed point label(v) = the smallest vertex that reaches v (for a
// symmetric A, the smallest vertex of v's component).  Only the entries of
// the current x and y are touched per step; x is appended tile by tile in
// any order (one counter update per tile).

#include "device_ops.h"

namespace spv {

namespace {

__global__ void k_cc_reset(Ctrl* ctrl) {
    if (threadIdx.x == 0) {
        ctrl->f = 0;
        ctrl->level = 0;
        ctrl->gen_count = 0;
        ctrl->nnz_y = 0;
        ctrl->step_done = 0;
    }
}

// Both kernels are bound by memory; x takes one counter update per tile
// (append_tile, measured on the PageRank step).
__global__ __launch_bounds__(kStepBlock) void k_cc_init(int32_t n, const int32_t* colptr, int32_t* label,
                                                        int32_t* x_idx, uint32_t* x_val, Ctrl* ctrl) {
    __shared__ int s_cnt[kWave];
    for (int64_t b = (int64_t)blockIdx.x * kStepTile; b < n; b += (int64_t)gridDim.x * kStepTile) {
        int32_t j[kStepItems];
        uint32_t v[kStepItems];
        bool take[kStepItems];
#pragma unroll
        for (int i = 0; i < kStepItems; ++i) {
            const int64_t p = b + i * kStepBlock + threadIdx.x;
            j[i] = (int32_t)(p < n ? p : n - 1);
            v[i] = (uint32_t)j[i];
            take[i] = colptr[j[i] + 1] > colptr[j[i]] && p < n;
        }
#pragma unroll
        for (int i = 0; i < kStepItems; ++i) label[j[i]] = j[i];
        append_tile<kStepBlock, kStepItems>(take, j, v, x_idx, x_val, &ctrl->gen_count, s_cnt);
    }
    finish_step(ctrl);
}

__global__ __launch_bounds__(kStepBlock) void k_cc_update(const int32_t* colptr, int32_t* label, const int32_t* y_idx,
                                                          const int32_t* y_val, int32_t* x_idx, uint32_t* x_val,
                                                          Ctrl* ctrl) {
    __shared__ int s_cnt[kWave];
    const int64_t cnt = __hip_atomic_load(&ctrl->nnz_y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int32_t f = ld_ctrl(&ctrl->f);
    if (f <= 0) return;   // the multiply was a no-op; y holds stale entries
    for (int64_t b = (int64_t)blockIdx.x * kStepTile; b < cnt; b += (int64_t)gridDim.x * kStepTile) {
        int32_t j[kStepItems], y[kStepItems], old[kStepItems], len[kStepItems];
        uint32_t v[kStepItems];
        bool take[kStepItems];
#pragma unroll
        for (int i = 0; i < kStepItems; ++i) {
            const int64_t p = b + i * kStepBlock + threadIdx.x;
            const int64_t pc = p < cnt ? p : cnt - 1;
            j[i] = y_idx[pc];
            y[i] = y_val[pc];
        }
#pragma unroll
        for (int i = 0; i < kStepItems; ++i) {
            old[i] = label[j[i]];
            len[i] = colptr[j[i] + 1] - colptr[j[i]];
        }
#pragma unroll
        for (int i = 0; i < kStepItems; ++i) {
            // j appears once in y: no other thread writes its label
            const bool lower = b + i * kStepBlock + threadIdx.x < cnt && y[i] < old[i];
            if (lower) label[j[i]] = y[i];
            take[i] = lower && len[i] > 0;
            v[i] = (uint32_t)y[i];
        }
        append_tile<kStepBlock, kStepItems>(take, j, v, x_idx, x_val, &ctrl->gen_count, s_cnt);
    }
    finish_step(ctrl);
}

}  // namespace

hipError_t launch_cc_init(int32_t n, const int32_t* colptr, int32_t* label, int32_t* x_idx, int32_t* x_val,
                          Ctrl* ctrl, hipStream_t s) {
    hipLaunchKernelGGL(k_cc_reset, dim3(1), dim3(64), 0, s, ctrl);
    hipLaunchKernelGGL(k_cc_init, dim3(step_grid(n)), dim3(kStepBlock), 0, s, n, colptr, label, x_idx,
                       reinterpret_cast<uint32_t*>(x_val), ctrl);
    return hipGetLastError();
}

hipError_t launch_cc_update(int32_t n, const int32_t* colptr, int32_t* label, const int32_t* y_idx,
                            const int32_t* y_val, int32_t* x_idx, int32_t* x_val, Ctrl* ctrl, hipStream_t s) {
    hipLaunchKernelGGL(k_cc_update, dim3(step_grid(n)), dim3(kStepBlock), 0, s, colptr, label, y_idx, y_val, x_idx,
                       reinterpret_cast<uint32_t*>(x_val), ctrl);
    return hipGetLastError();
}

}  // namespace spv
