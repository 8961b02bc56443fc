// The activation in a kernel's epilogue: results requantised four at a time and stored as the next layer's blocked input.
#pragma once
#include "act_requant.h"
#include "kernels.h"

namespace c2i8 {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int act16 __attribute__((ext_vector_type(16)));   // a 32 x 32 MFMA result

// Four values activated, a byte each.  A sum that saturates comes out the same: it is clipped to 127 anyway (2^31 / 2^24 = 128).  The shift, the
// clip to int8 and the packing of two values are one instruction: 11 in all where four act_requant and their packing are some 40 --
// on the 32 x 32 results of a shallow layer that was more time than their MFMAs take.
__device__ __forceinline__ unsigned act_requant4(int x0, int x1, int x2, int x3, int shift, int relu)
{
    if (shift > 24) {
        const int y[4] = {act_requant(x0, shift, relu), act_requant(x1, shift, relu), act_requant(x2, shift, relu), act_requant(x3, shift, relu)};
        return (unsigned)(y[0] & 0xFF) | (unsigned)(y[1] & 0xFF) << 8 | (unsigned)(y[2] & 0xFF) << 16 | (unsigned)(y[3] & 0xFF) << 24;
    }
    const int half = shift > 0 ? 1 << (shift - 1) : 0, least = relu ? 0 : (int)0x80000000;
    x0 = max(__builtin_elementwise_add_sat(x0, half), least), x1 = max(__builtin_elementwise_add_sat(x1, half), least);
    x2 = max(__builtin_elementwise_add_sat(x2, half), least), x3 = max(__builtin_elementwise_add_sat(x3, half), least);
    const unsigned lo = (unsigned short)__builtin_amdgcn_ashr_pk_i8_i32(x0, x1, shift), hi = (unsigned short)__builtin_amdgcn_ashr_pk_i8_i32(x2, x3, shift);
    return lo | hi << 16;
}

// The first `left` of a dword's four bytes, zeros behind them.
__device__ __forceinline__ unsigned act_keep(unsigned y, int left)
{
    return left >= 4 ? y : left <= 0 ? 0u : y & ((1u << 8 * left) - 1);
}

// A 32 x 32 MFMA result (lane: column lane % 32, rows 8 g + 4 (lane / 32) + 0..3) whose rows are channels: both lanes of a column trade half of
// what they hold, and each is left with 16 consecutive channels, 16 (lane / 32) on, activated -- one 16-byte piece instead of four dwords 8 bytes
// apart.  With the four at a time above, the general kernel's fused activations on blocked input take 0.90 of the time they took value by value and dword by
// dword (1247 drawn layers; 64 images 64 x 56 x 56 -> 64, 3x3: 29.8 -> 24.0 us; 1024 images 22 x 28 x 28 -> 256, 1x1: 131 -> 62).  left: channels there are from row 0 on; zeros from there.  Lanes l and l + 32 both active, or neither.
__device__ __forceinline__ v4i act_block16(const act16 &d, int left, int lane, int shift, int relu)
{
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    unsigned y[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) y[g] = act_requant4(d[4 * g], d[4 * g + 1], d[4 * g + 2], d[4 * g + 3], shift, relu);
    if (left < 32) {
#pragma unroll
        for (int g = 0; g < 4; ++g) y[g] = act_keep(y[g], left - 8 * g - 4 * (lane >> 5));
    }
    const v2u a = __builtin_amdgcn_permlane32_swap(y[0], y[2], false, false), b = __builtin_amdgcn_permlane32_swap(y[1], y[3], false, false);
    return v4i{(int)a[0], (int)a[1], (int)b[0], (int)b[1]};
}

// Whether the 32 channels from k on (k in a row of 32) are the last there are and the first half of a block of 64: the other half, zeros, is nobody else's
// to write where a workgroup has 32 channels.  (A clear of the whole output before the stage took 1.5 to 7 us.)
__device__ __forceinline__ bool act_half_left(int k, int K, int cb_log2) { return cb_log2 == 6 && (k & 32) == 0 && (k & ~31) + 32 >= K; }

// Four consecutive output channels k .. k+3 of pixel (n, p, q) -- what one lane holds in v%4 of an MFMA
// result block -- activated and stored as one dword of the blocked tensor; channels from K on are zeros.
__device__ __forceinline__ void act_store4(const ActOut &e, int n, int p, int q, int k, int K, int x0, int x1, int x2, int x3)
{
    if (k >= e.Cb << e.cb_log2) return;
    const size_t pix = ((size_t)n * e.Cb + (k >> e.cb_log2)) * e.Hp * e.Wp + (size_t)(p + e.pad) * e.Wp + (q + e.pad);
    int8_t *dst = e.out + (pix << e.cb_log2) + (k & ((1 << e.cb_log2) - 1));
    *reinterpret_cast<unsigned *>(dst) = act_keep(act_requant4(x0, x1, x2, x3, e.shift, e.relu), K - k);
    if (act_half_left(k, K, e.cb_log2)) *reinterpret_cast<unsigned *>(dst + 32) = 0;
}
// The 32 channels from k on of a 32 x 32 result, two pieces of 16 bytes (act_block16).
__device__ __forceinline__ void act_store32(const ActOut &e, int n, int p, int q, int k, int K, int lane, const act16 &d)
{
    const auto y = act_block16(d, K - k, lane, e.shift, e.relu);
    k += 16 * (lane >> 5);
    if (k >= e.Cb << e.cb_log2) return;
    const size_t pix = ((size_t)n * e.Cb + (k >> e.cb_log2)) * e.Hp * e.Wp + (size_t)(p + e.pad) * e.Wp + (q + e.pad);
    int8_t *dst = e.out + (pix << e.cb_log2) + (k & ((1 << e.cb_log2) - 1));
    *reinterpret_cast<v4i *>(dst) = y;
    if (act_half_left(k, K, e.cb_log2)) *reinterpret_cast<v4i *>(dst + 32) = v4i{0, 0, 0, 0};
}

}  // namespace c2i8
