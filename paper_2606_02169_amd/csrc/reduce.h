// Deterministic FP64 block reductions for wave64 (no atomics): a fixed pattern of lane moves inside each
// wave, then the waves' partials summed in wave order.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace mrmf {

// v moved across lanes by one DPP pattern (rows outside row_mask contribute 0), one 32-bit half at a time
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_move(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<uint32_t>(u)), CTRL, ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<uint32_t>(u >> 32)), CTRL, ROW_MASK, 0xf,
                                               false);
    return __builtin_bit_cast(double, (static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32) |
                                          static_cast<uint64_t>(static_cast<uint32_t>(lo)));
}

// Sums over the 64 lanes of a wave (all active) with a fixed pattern of DPP moves (lane pairs 1 and 2 apart, the
// half and full row mirrors, then the row broadcasts of lanes 15 and 31), which stay in the vector unit where
// __shfl goes through LDS; the totals end in lane 63.
template <int NV>
__device__ __forceinline__ void wave_sum(double (&v)[NV]) {
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_move<0xB1, 0xf>(v[k]);   // quad_perm [1, 0, 3, 2]
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_move<0x4E, 0xf>(v[k]);   // quad_perm [2, 3, 0, 1]
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_move<0x141, 0xf>(v[k]);  // row_half_mirror
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_move<0x140, 0xf>(v[k]);  // row_mirror: every lane holds its row's sum
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_move<0x142, 0xa>(v[k]);  // row_bcast:15 into rows 1 and 3
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_move<0x143, 0xc>(v[k]);  // row_bcast:31 into rows 2 and 3
}

__device__ __forceinline__ double wave_sum(double v) {
    double a[1] = {v};
    wave_sum<1>(a);
    return a[0];
}

// The waves' sums of v in lds[wave * NV + k] (NV * blockDim / 64 doubles), after a barrier.
template <int NV>
__device__ __forceinline__ void block_sum_lds(double (&v)[NV], double* lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    wave_sum<NV>(v);
    if (lane == 63) {
#pragma unroll
        for (int k = 0; k < NV; ++k) lds[wave * NV + k] = v[k];
    }
    __syncthreads();
}

// Sums v over the block; the result is valid in thread 0.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* lds) {
    const int nw = (blockDim.x + 63) >> 6;
    block_sum_lds<NV>(v, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            double s = 0.0;
            for (int w = 0; w < nw; ++w) s += lds[w * NV + k];
            v[k] = s;
        }
    }
    __syncthreads();
}

// The sum of v[0] over the block, in every thread.
template <int NV>
__device__ __forceinline__ double block_total(double (&v)[NV], double* lds) {
    const int nw = (blockDim.x + 63) >> 6;
    block_sum_lds<NV>(v, lds);
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += lds[w * NV];
    __syncthreads();
    return s;
}

}  // namespace mrmf
