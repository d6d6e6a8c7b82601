// tvl_quant_device.h -- device code shared by the kernels over block-quantised
// weights: decoding, buffer descriptors, the swizzled x layout in LDS and the
// reduction over lane groups.
#pragma once

#include "tvl_device.h"

namespace tvl {
namespace {

#define TVL_LDS __attribute__((address_space(3)))
__device__ __forceinline__ float sbyte(unsigned v, int b) { return (float)(int)(signed char)(v >> (8 * b)); }

// 8-bit: sum_j q_j x_j over the 16 columns of one 16-byte weight vector
__device__ __forceinline__ float qdot8(const u4 w, const f4 (&xv)[4])
{
    float ta = 0.f, tb = 0.f;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const unsigned v = w[d];
        ta = fmaf(sbyte(v, 0), xv[d].x, ta);
        tb = fmaf(sbyte(v, 1), xv[d].y, tb);
        ta = fmaf(sbyte(v, 2), xv[d].z, ta);
        tb = fmaf(sbyte(v, 3), xv[d].w, tb);
    }
    return ta + tb;
}

// q / 16 for the signed nibble in bits 3:0 of byte B of v
#define TVL_NIB16(B)                                                                              \
    __device__ __forceinline__ float nib16_##B(unsigned v)                                        \
    {                                                                                             \
        float r;                                                                                  \
        asm("v_cvt_off_f32_i4_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #B \
            : "=v"(r) : "v"(v));                                                                  \
        return r;                                                                                 \
    }
TVL_NIB16(0)
TVL_NIB16(1)
TVL_NIB16(2)
TVL_NIB16(3)
#undef TVL_NIB16

// 4-bit: sum_j q_j x_j / 16 over the 32 columns of one 16-byte vector.  Dword
// d holds columns 8d .. 8d+7, column 8d + 2b in the low nibble of byte b and
// 8d + 2b + 1 in its high nibble.  Per 8 codes: one shift, 8 conversions and
// 8 FMAs.
__device__ __forceinline__ float qdot4(const u4 w, const f4 (&xv)[8])
{
    float ta = 0.f, tb = 0.f; // even columns; odd columns
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const unsigned lo = w[d], hi = w[d] >> 4;
        const f4 x0 = xv[2 * d], x1 = xv[2 * d + 1];
        ta = fmaf(nib16_0(lo), x0.x, ta);
        tb = fmaf(nib16_0(hi), x0.y, tb);
        ta = fmaf(nib16_1(lo), x0.z, ta);
        tb = fmaf(nib16_1(hi), x0.w, tb);
        ta = fmaf(nib16_2(lo), x1.x, ta);
        tb = fmaf(nib16_2(hi), x1.y, tb);
        ta = fmaf(nib16_3(lo), x1.z, ta);
        tb = fmaf(nib16_3(hi), x1.w, tb);
    }
    return ta + tb;
}

// Buffer descriptor (CDNA V#) over [base, base + bytes): raw addressing, the
// gfx9-family default format word.  Loads through it take a 32-bit per-lane
// offset and a scalar offset, so R rows cost R offset registers instead of
// R 64-bit pointers, and the chunk advance is one scalar add.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, int64_t bytes)
{
    const int n = bytes > 0x7fffffff ? 0x7fffffff : (int)bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, n, 0x00020000);
}
constexpr int kBufNT = 2; // cache policy: non-temporal (streamed once)

// the f4 of x at column col (a multiple of 4) in the swizzled LDS layout:
// f4 j lives at 16-byte slot (j with its low 3 bits XORed by bits 5:3)
__device__ __forceinline__ f4 lds_x4(const TVL_LDS float *xl, int col)
{
    const int j = col >> 2;
    const int slot = (j & ~7) | ((j ^ (j >> 3)) & 7);
    return *(const TVL_LDS f4 *)(xl + 4 * slot);
}

// Reduce R values per lane over each group of G consecutive lanes (R <= G,
// both powers of two).  On return lane l holds the group total of value
// (l % G) / (G / R).
template <int R, int G>
__device__ __forceinline__ float reduce_group(float (&v)[R], int lane)
{
    static_assert(R <= G && G <= kWave, "R <= G <= 64");
    halve_all<R, G / 2>(v, lane);
#pragma unroll
    for (int o = G / (2 * R); o >= 1; o >>= 1)
        v[0] += __shfl_xor(v[0], o);
    return v[0];
}

}  // namespace
}  // namespace tvl
