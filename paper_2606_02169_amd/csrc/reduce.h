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

// Sum over the 64 lanes of a wave with a fixed pattern of DPP moves (lane pairs 1 and 2 apart, the half and full row
// mirrors, then the row broadcasts of lanes 15 and 31); the total ends in lane 63.
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_move<0xB1, 0xf>(v);   // quad_perm [1, 0, 3, 2]
    v += dpp_move<0x4E, 0xf>(v);   // quad_perm [2, 3, 0, 1]
    v += dpp_move<0x141, 0xf>(v);  // row_half_mirror
    v += dpp_move<0x140, 0xf>(v);  // row_mirror: every lane holds its row's sum
    v += dpp_move<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_move<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return v;                      // lane 63: the wave's sum
}

// Sums over the 64 lanes of a wave (all active) as the tree of lane distances 32, 16, 8, 4, 2, 1; every lane holds the
// totals.  Below 16 the partner's value comes by a DPP move inside the vector unit instead of a shuffle through LDS: a
// rotation of the 16 lanes of a row by 8, by 4 (lanes 8 apart already hold the same sum), then swaps inside quads.
template <int NV>
__device__ __forceinline__ void wave_tree(double (&v)[NV]) {
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += __shfl_xor(v[k], 32, 64);
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += __shfl_xor(v[k], 16, 64);
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_move<0x128, 0xf>(v[k]);  // row_ror:8
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_move<0x124, 0xf>(v[k]);  // row_ror:4
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_move<0x4E, 0xf>(v[k]);   // quad_perm [2, 3, 0, 1]
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] += dpp_move<0xB1, 0xf>(v[k]);   // quad_perm [1, 0, 3, 2]
}

// The same sums (distances 32, 16, 8, 4, 2, 1) for many values, NV a multiple of 16: the lanes share them out as the
// distances halve, so that NV moves do what wave_tree does with 6 NV.  v[j], j < NV / 16, ends as value
// wave_share(lane, NV) + j, the same in the four lanes of a quad.
__device__ __forceinline__ int wave_share(int lane, int nv) {
    return (lane >> 5 & 1) * (nv / 2) + (lane >> 4 & 1) * (nv / 4) + (lane >> 3 & 1) * (nv / 8) + (lane >> 2 & 1) * (nv / 16);
}

template <int NV>
__device__ __forceinline__ void wave_tree_shared(double (&v)[NV], int lane) {
    static_assert(NV % 16 == 0, "halved four times");
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        const int d = 32 >> l, n = NV >> (l + 1);
        const bool up = (lane & d) != 0;
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const double give = up ? v[k] : v[n + k], keep = up ? v[n + k] : v[k];
            v[k] = keep + (d == 8 ? dpp_move<0x128, 0xf>(give) : __shfl_xor(give, d, 64));  // row_ror:8
        }
    }
#pragma unroll
    for (int k = 0; k < NV / 16; ++k) {
        v[k] += dpp_move<0x4E, 0xf>(v[k]);  // quad_perm [2, 3, 0, 1]
        v[k] += dpp_move<0xB1, 0xf>(v[k]);  // quad_perm [1, 0, 3, 2]
    }
}

// Sums v over the block (the waves' trees, then in wave order); the result is valid in thread 0.  `lds` must hold
// NV * (blockDim / 64) doubles.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    wave_tree<NV>(v);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) lds[wave * NV + k] = v[k];
    }
    __syncthreads();
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

}  // namespace mrmf
