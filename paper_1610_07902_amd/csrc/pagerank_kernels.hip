// Data-driven (delta) PageRank around the SpMSpV hot path.  The paper names
// PageRank among the data-driven uses of SpMSpV, where a vertex stops
// sending updates once its value has converged (Introduction); the rule
// implemented is:
//   rank = 0, delta = (1 - d) / n everywhere, every vertex active;
//   each step: rank += delta; x = { (j, d * delta(j) / outdeg(j)) : j active,
//   outdeg(j) > 0 }; delta = A x (plus-times SpMSpV, structural pattern);
//   j is active next when delta(j) > tol * rank(j) (rank before adding).
// Only the entries of the current x and y are touched per step.  The x list
// is appended tile by tile in any order (one counter update per tile).

#include "device_ops.h"

namespace spv {

namespace {

// Both kernels are bound by memory: k_pr_update reads y, rank and both column
// bounds of each touched vertex and writes rank and the next x (28 bytes
// each).  Measured on 1.5M touched vertices: 150 us with one counter update
// per wave and a kernel to publish the length, about 15 us with one per tile
// (append_tile) and the last workgroup publishing.
__global__ __launch_bounds__(kStepBlock) void k_pr_init(int32_t n, const int32_t* colptr, float d, float* rank,
                                                        int32_t* x_idx, uint32_t* x_val, Ctrl* ctrl) {
    __shared__ int s_cnt[kWave];
    const float base = (1.0f - d) / (float)n;
    for (int64_t b = (int64_t)blockIdx.x * kStepTile; b < n; b += (int64_t)gridDim.x * kStepTile) {
        int32_t j[kStepItems], len[kStepItems];
        uint32_t v[kStepItems];
        bool take[kStepItems];
#pragma unroll
        for (int i = 0; i < kStepItems; ++i) {
            const int64_t p = b + i * kStepBlock + threadIdx.x;
            j[i] = (int32_t)(p < n ? p : n - 1);
            len[i] = colptr[j[i] + 1] - colptr[j[i]];
            take[i] = p < n && len[i] > 0;
        }
#pragma unroll
        for (int i = 0; i < kStepItems; ++i) {
            rank[j[i]] = base;   // a clamped position writes the last vertex's value again
            v[i] = __float_as_uint(take[i] ? d * base / (float)len[i] : 0.f);
        }
        append_tile<kStepBlock, kStepItems>(take, j, v, x_idx, x_val, &ctrl->gen_count, s_cnt);
    }
    finish_step(ctrl);
}

__global__ __launch_bounds__(kStepBlock) void k_pr_update(const int32_t* colptr, float d, float tol, float* rank,
                                                          const int32_t* y_idx, const float* y_val, int32_t* x_idx,
                                                          uint32_t* x_val, Ctrl* ctrl) {
    __shared__ int s_cnt[kWave];
    const int64_t cnt = __hip_atomic_load(&ctrl->nnz_y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int32_t f = ld_ctrl(&ctrl->f);
    if (f <= 0) return;   // the multiply was a no-op; y holds stale entries
    for (int64_t b = (int64_t)blockIdx.x * kStepTile; b < cnt; b += (int64_t)gridDim.x * kStepTile) {
        int32_t j[kStepItems], len[kStepItems];
        float y[kStepItems], r[kStepItems];
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
            r[i] = rank[j[i]];
            len[i] = colptr[j[i] + 1] - colptr[j[i]];
        }
#pragma unroll
        for (int i = 0; i < kStepItems; ++i) {
            const bool in = b + i * kStepBlock + threadIdx.x < cnt;
            if (in) rank[j[i]] = r[i] + y[i];
            take[i] = in && y[i] > tol * r[i] && len[i] > 0;
            v[i] = __float_as_uint(take[i] ? d * y[i] / (float)len[i] : 0.f);
        }
        append_tile<kStepBlock, kStepItems>(take, j, v, x_idx, x_val, &ctrl->gen_count, s_cnt);
    }
    finish_step(ctrl);
}

__global__ void k_pr_reset(Ctrl* ctrl) {
    if (threadIdx.x == 0) {
        ctrl->f = 0;
        ctrl->level = 0;
        ctrl->gen_count = 0;
        ctrl->nnz_y = 0;
        ctrl->step_done = 0;
    }
}

}  // namespace

hipError_t launch_pr_init(int32_t n, const int32_t* colptr, float d, float* rank, int32_t* x_idx, float* x_val,
                          Ctrl* ctrl, hipStream_t s) {
    hipLaunchKernelGGL(k_pr_reset, dim3(1), dim3(64), 0, s, ctrl);
    hipLaunchKernelGGL(k_pr_init, dim3(step_grid(n)), dim3(kStepBlock), 0, s, n, colptr, d, rank, x_idx,
                       reinterpret_cast<uint32_t*>(x_val), ctrl);
    return hipGetLastError();
}

hipError_t launch_pr_update(int32_t n, const int32_t* colptr, float d, float tol, float* rank, const int32_t* y_idx,
                            const float* y_val, int32_t* x_idx, float* x_val, Ctrl* ctrl, hipStream_t s) {
    hipLaunchKernelGGL(k_pr_update, dim3(step_grid(n)), dim3(kStepBlock), 0, s, colptr, d, tol, rank, y_idx, y_val,
                       x_idx, reinterpret_cast<uint32_t*>(x_val), ctrl);
    return hipGetLastError();
}

}  // namespace spv
