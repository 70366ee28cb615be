// Device-side pieces of the GEMMs whose operands both lie in MFMA operand order
// (ls_prefill.hip, ls_gemm_rows.hip).
#pragma once
#include "ls_gemm_dev.h"

namespace ls {

// acc += (16 x k)(k x 16) of one k step (KSTEP values of k), x the A operand
template <typename WT>
__device__ __forceinline__ void mfma_one(const u32x4& x, const u32x4& y, f32x4& acc) {
    if constexpr (sizeof(WT) == 2) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, x), __builtin_bit_cast(f16x8, y), acc, 0,
                                                     0, 0);
    } else {
        const f32x4 a = __builtin_bit_cast(f32x4, x), b = __builtin_bit_cast(f32x4, y);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc, 0, 0, 0);
    }
}

// eight (fp16) or four (fp32) consecutive values in the compute dtype: 16 bytes
template <typename WT>
__device__ __forceinline__ u32x4 pack16(const float* v) {
    if constexpr (sizeof(WT) == 2)
        return u32x4{pack_h2(v[0], v[1]), pack_h2(v[2], v[3]), pack_h2(v[4], v[5]), pack_h2(v[6], v[7])};
    else
        return __builtin_bit_cast(u32x4, f32x4{v[0], v[1], v[2], v[3]});
}

// Values k .. k + 15 of row m (k a multiple of 16) into an activation buffer of K columns
template <typename WT>
__device__ __forceinline__ void store_act16(void* base, int m, int k, int K, const float* v) {
    constexpr int VEC = WTraits<WT>::VEC;
#pragma unroll
    for (int e = 0; e < 16; e += VEC) *(u32x4*)((WT*)base + opd_elem<WT>(m, k + e, K)) = pack16<WT>(v + e);
}

}  // namespace ls
