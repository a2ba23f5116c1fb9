// Decode of MXFP4 weights in registers, shared by the streaming tiles (expert_ffn_mx_tiles.h)
// and the GEMM tiles (expert_gemm.hip).  Internal linkage, as there.
#pragma once

#include <hip/hip_runtime.h>

namespace spice {
namespace {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// E8M0 block scale -> fp32 2^(s - 127): the exponent field for s >= 1, the subnormal
// 2^-127 for s = 0, NaN for s = 255; the conversion applies it exactly.
// Bit 22 marks both special cases; without a compare, which the compiler turned into branches
// between the loads and the MFMAs.
__device__ __forceinline__ float e8m0(uint32_t s) {
    const uint32_t special = (((s + 1u) & 0xFEu) - 1u) >> 31;  // s is 0 or 255
    return __uint_as_float((s << 23) | (special << 22));
}

// 8 E2M1 codes (4 bytes, low nibble first) times the block scale -> 8 bf16, one MFMA A operand.
__device__ __forceinline__ u32x4_t mx_decode8(uint32_t w, float scale) {
    const bf16x2_t p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, scale, 0);
    const bf16x2_t p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, scale, 1);
    const bf16x2_t p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, scale, 2);
    const bf16x2_t p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, scale, 3);
    return u32x4_t{__builtin_bit_cast(uint32_t, p0), __builtin_bit_cast(uint32_t, p1),
                   __builtin_bit_cast(uint32_t, p2), __builtin_bit_cast(uint32_t, p3)};
}

// 32 codes (16 bytes) -> four MFMA A operands: op[k] holds elements 8k .. 8k+7 (bytes 4k .. 4k+3).
__device__ __forceinline__ void mx_decode(u32x4_t raw, float scale, u32x4_t (&op)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) op[k] = mx_decode8(raw[k], scale);
}

}  // namespace
}  // namespace spice
