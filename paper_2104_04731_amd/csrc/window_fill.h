// Device pieces of the GEMM stages that read the network's own tensors: input pixels turned around into pixel-major LDS
// records, and raw 3x3 weights brought into depth order.  Used by resident_mfma.hip and band_mfma.hip.
#pragma once
#include "rewrite_bodies.h"

namespace c2i8 {

// The input pixels a workgroup keeps: of image n0 the `len0` pixels from lo0 on, of every image behind it its first
// full8 pixels (the last one's may be fewer); slots in all, each range a multiple of 8.
struct WindowRange {
    int n0, lo0, len0, full8, slots;
    unsigned mg_full8;
};
__device__ __forceinline__ void window_slot(const WindowRange &w, int s, int *n, int *lin)
{
    *n = w.n0;
    *lin = w.lo0 + s;
    if (s >= w.len0) {
        const int r = s - w.len0, d = fast_div_any(r, w.full8, w.mg_full8);
        *n = w.n0 + 1 + d;
        *lin = r - d * w.full8;
    }
}

// The tensor a window is filled from.
struct WindowSource {
    const int8_t *src;
    long long img_bytes, src_bytes;   // of an image, of the tensor
    int C1, HW;                       // last channel, pixels of an image
    int pstride;                      // pixel-major: bytes from pixel to pixel
};

typedef unsigned long long u64_a1 __attribute__((aligned(1)));
typedef unsigned u32_a1 __attribute__((aligned(1)));

// Eight pixels of four channels (a channel per 64-bit value) -> eight records' dwords, `pitch` bytes apart.
__device__ __forceinline__ void put_4x8(const unsigned long long (&v)[4], unsigned char *d, int pitch)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const unsigned r0 = (unsigned)(v[0] >> (32 * h)), r1 = (unsigned)(v[1] >> (32 * h));
        const unsigned r2 = (unsigned)(v[2] >> (32 * h)), r3 = (unsigned)(v[3] >> (32 * h));
        const unsigned lo01 = __builtin_amdgcn_perm(r1, r0, 0x05010400), hi01 = __builtin_amdgcn_perm(r1, r0, 0x07030602);
        const unsigned lo23 = __builtin_amdgcn_perm(r3, r2, 0x05010400), hi23 = __builtin_amdgcn_perm(r3, r2, 0x07030602);
        *reinterpret_cast<unsigned *>(d) = __builtin_amdgcn_perm(lo23, lo01, 0x05040100);
        *reinterpret_cast<unsigned *>(d + pitch) = __builtin_amdgcn_perm(lo23, lo01, 0x07060302);
        *reinterpret_cast<unsigned *>(d + 2 * pitch) = __builtin_amdgcn_perm(hi23, hi01, 0x05040100);
        *reinterpret_cast<unsigned *>(d + 3 * pitch) = __builtin_amdgcn_perm(hi23, hi01, 0x07060302);
        d += 4 * pitch;
    }
}

// NCHW -> records.  Unit: 4 channels x 8 pixels, neighbouring lanes on neighbouring channel quads (a record's pieces fall
// into different banks; the planes' lines are shared by the units that follow in the same workgroup).  cq: channel quads
// of a record; bytes past the last channel are zero.  (Bound by the loads where several waves share a SIMD -- without its
// LDS writes it takes as long -- and by the instruction count of a lone wave, hence the short path: one image, nothing
// past the tensor's end, whole quads only: scalar bases and one 32-bit offset per unit.)
template <int NT, int B>
__device__ __forceinline__ void window_from_nchw(const WindowSource &t, const WindowRange &w, int cq, unsigned mg_cq, unsigned char *win, int pitch, int tid)
{
    const int units = cq * (w.slots >> 3);
    const long long img0 = (long long)w.n0 * t.img_bytes;
    if (w.slots == w.len0 && t.C1 + 1 == 4 * cq && img0 + (long long)t.C1 * t.HW + w.lo0 + w.slots <= t.src_bytes) {
        const int8_t *const b0 = t.src + img0 + w.lo0, *const b1 = b0 + t.HW, *const b2 = b1 + t.HW, *const b3 = b2 + t.HW;
        for (int u0 = tid; u0 < units; u0 += NT * B) {   // B: units per thread and round of loads
            unsigned long long v[B][4];
            int dst[B];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int u = u0 + b * NT;
                if (u < units) {
                    const int g = fast_div_any(u, cq, mg_cq), c4 = (u - g * cq) * 4;
                    const unsigned off = (unsigned)(c4 * t.HW + g * 8);
                    dst[b] = g * 8 * pitch + c4;
                    v[b][0] = *reinterpret_cast<const u64_a1 *>(b0 + off);
                    v[b][1] = *reinterpret_cast<const u64_a1 *>(b1 + off);
                    v[b][2] = *reinterpret_cast<const u64_a1 *>(b2 + off);
                    v[b][3] = *reinterpret_cast<const u64_a1 *>(b3 + off);
                }
            }
#pragma unroll
            for (int b = 0; b < B; ++b)
                if (u0 + b * NT < units) put_4x8(v[b], win + dst[b], pitch);
        }
        return;
    }
    for (int u0 = tid; u0 < units; u0 += NT * B) {
        unsigned long long v[B][4];
        int dst[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int u = min(u0 + b * NT, units - 1), g = fast_div_any(u, cq, mg_cq), c4 = (u - g * cq) * 4;
            int n, lin;
            window_slot(w, g * 8, &n, &lin);
            dst[b] = g * 8 * pitch + c4;
            const long long img = (long long)n * t.img_bytes;
            const int8_t *base = t.src + img;
            const long long left = t.src_bytes - 8 - img;
            const int last = left > 0x7FFFFFFFLL ? 0x7FFFFFFF : (int)left;  // may be negative in a tiny last image: still in the tensor
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int want = min(c4 + i, t.C1) * t.HW + lin, at = min(want, last);
                v[b][i] = *reinterpret_cast<const u64_a1 *>(base + at) >> (8 * (want - at));
                if (c4 + i > t.C1) v[b][i] = 0;
            }
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            if (u0 + b * NT >= units) break;
            put_4x8(v[b], win + dst[b], pitch);
        }
    }
}

// Pixel-major source (NHWC) -> records: 16-byte pieces, neighbouring lanes on neighbouring pieces.
// u16: pieces of a record (what lies past the last channel is the next pixel's: its weights are zero).
template <int NT, int B>
__device__ __forceinline__ void window_from_pixels(const WindowSource &t, const WindowRange &w, int u16, unsigned mg_u16, unsigned char *win, int pitch, int tid)
{
    const int units = u16 * w.slots;
    for (int u0 = tid; u0 < units; u0 += NT * B) {
        v4i v[B];
        int dst[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int u = min(u0 + b * NT, units - 1), s = fast_div_any(u, u16, mg_u16), j = u - s * u16;
            int n, lin;
            window_slot(w, s, &n, &lin);
            dst[b] = s * pitch + j * 16;
            lin = min(lin, t.HW - 1);
            const long long img = (long long)n * t.img_bytes;
            const long long left = t.src_bytes - 16 - img;
            const int last = left > 0x7FFFFFFFLL ? 0x7FFFFFFF : (int)left;
            const int want = lin * t.pstride + j * 16, at = min(want, last);
            v4i x;
            __builtin_memcpy(&x, t.src + img + at, 16);
            v[b] = want != at ? shift_piece(x, at - want) : x;
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            if (u0 + b * NT >= units) break;
            *reinterpret_cast<v4i *>(win + dst[b]) = v[b];
        }
    }
}

// Raw 3x3 weights: 4 channels x 9 taps of one row are 36 consecutive bytes (byte 9c + t).  raw9_load fetches them (rows past
// the last one and channels past the last one: zeros), raw9_tap<T> picks tap T's dword of four channels out of them: three
// byte permutes.
__host__ __device__ __forceinline__ void raw9_load(const int8_t *wt, int K, int C, int k, int quad, unsigned (&d)[9])
{
#pragma unroll
    for (int i = 0; i < 9; ++i) d[i] = 0;
    const int valid = k < K ? min(C - quad * 4, 4) * 9 : 0;   // bytes that belong to this row's channels
    if (valid <= 0) return;
    const int8_t *p = wt + (long long)k * C * 9 + (long long)quad * 36;
    // 36 bytes are left in the tensor: behind a row's last channels come the next rows, and four of them (the shortest is
    // nine bytes) always suffice.  One row is not enough where a row has a single channel.
    if (min(K - k, 4) * C * 9 - quad * 36 >= 36) {
        const v4i_a1 x0 = *reinterpret_cast<const v4i_a1 *>(p), x1 = *reinterpret_cast<const v4i_a1 *>(p + 16);
        d[0] = x0[0], d[1] = x0[1], d[2] = x0[2], d[3] = x0[3], d[4] = x1[0], d[5] = x1[1], d[6] = x1[2], d[7] = x1[3];
        d[8] = *reinterpret_cast<const u32_a1 *>(p + 32);
    } else {   // the tensor's last bytes
#pragma unroll
        for (int i = 0; i < 9; ++i)
            for (int b = 0; b < 4; ++b)
                if (i * 4 + b < valid) d[i] |= (unsigned)(unsigned char)p[i * 4 + b] << (8 * b);
    }
}
__host__ __device__ __forceinline__ void raw9_mask(int C, int quad, unsigned (&d)[9])
{
    const int valid = min(C - quad * 4, 4) * 9;
    if (valid < 36 && valid > 0) {
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int keep = valid - 4 * i;
            d[i] &= keep >= 4 ? 0xFFFFFFFFu : keep <= 0 ? 0u : (1u << (8 * keep)) - 1u;
        }
    }
}
template <int T>
__device__ __forceinline__ unsigned raw9_tap(const unsigned (&d)[9])
{
    constexpr int p0 = T, p1 = 9 + T, p2 = 18 + T, p3 = 27 + T;
    const unsigned lo = __builtin_amdgcn_perm(d[p1 >> 2], d[p0 >> 2], 0x0C0C0000u | (4u + (p1 & 3)) << 8 | (p0 & 3));
    const unsigned hi = __builtin_amdgcn_perm(d[p3 >> 2], d[p2 >> 2], 0x0C0C0000u | (4u + (p3 & 3)) << 8 | (p2 & 3));
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

}  // namespace c2i8
