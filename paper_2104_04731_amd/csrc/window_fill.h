// Device pieces of the GEMM stages that read the network's own tensors: input pixels turned around into pixel-major LDS
// records (the raw 3x3 weights' pieces are in rewrite_bodies.h).
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

// The ranges of a workgroup's pixels [m0, m1): per image from the first pixel any valid tap reads to the last, starts a
// multiple of 8.  n1: its last image.
template <typename A>
__device__ __forceinline__ WindowRange tile_window(const A &a, int m0, int m1, int *n1_out)
{
    const int n0 = fast_div_any(m0, a.PQ, a.mg_PQ), n1 = fast_div_any(m1 - 1, a.PQ, a.mg_PQ);
    auto first_of = [&](int pq) {
        const int p = fast_div_any(pq, a.Q, a.mg_Q), q = pq - p * a.Q;
        const int row = p * a.stride - a.pad, col = q * a.stride - a.pad;
        return (row < 0 ? 0 : row * a.W + min(max(col, 0), a.W - 1)) & ~7;
    };
    auto end_of = [&](int pq) {
        const int p = fast_div_any(pq, a.Q, a.mg_Q), q = pq - p * a.Q;
        const int row = p * a.stride - a.pad + (a.R - 1) * a.dil, col = q * a.stride - a.pad + (a.S - 1) * a.dil;
        return row >= a.H ? a.HW : row * a.W + max(min(a.W - 1, col), -1) + 1;
    };
    const int lo0 = first_of(m0 - n0 * a.PQ);
    const int len0 = max(((n1 > n0 ? end_of(a.PQ - 1) : end_of(m1 - 1 - n0 * a.PQ)) - lo0 + 7) & ~7, 0);
    const int len_last = n1 > n0 ? max((end_of(m1 - 1 - n1 * a.PQ) + 7) & ~7, 0) : 0;
    *n1_out = n1;
    return WindowRange{n0, lo0, len0, a.full8, len0 + (n1 > n0 ? (n1 - n0 - 1) * a.full8 + len_last : 0), a.mg_full8};
}

// The tensor a window is filled from.
struct WindowSource {
    const int8_t *src;
    long long img_bytes, src_bytes;   // of an image, of the tensor
    int C1, HW;                       // last channel, pixels of an image
    int pstride;                      // pixel-major: bytes from pixel to pixel
    int wide = 4;                     // 64-byte runs: units of a run and channel quad, or 0: not taken
};

// WindowSource::wide for planes of HW pixels: no runs on less than 64, where one holds the ends of several images' rows.  With runs -> without:
// 65 layers on 7 x 7 and 7 x 8 whose channels fill no quad 1.05 in the mean (503 images 114 x 7 x 7 -> 32 1x1 8.1 -> 7.2 us), 100 with whole
// quads 1.02, windows of two small images among them 1.05 (92 layers on 25 to 56 pixels, mostly 1x1 stride 2; 24 images 256 x 7 x 7 -> 64 5.56 -> 5.23,
// 5 images 512 x 5 x 5 -> 55 7.2 -> 5.8, at best 0.91).  From 64 pixels on the runs win: 226 layers on 64 to 462 pixels 0.93.
// Made on the host: a test of the plane's size in the kernel cost it 360 bytes of code and calls of 8 us 3 %, a factor among its arguments 0.5 %.
static inline int window_wide_units(long long HW) { return HW >= 64 ? 4 : 0; }

typedef unsigned long long u64_a1 __attribute__((aligned(1)));

// Four pixels of four channels (a channel per dword) -> four records' dwords, `pitch` bytes apart.
__device__ __forceinline__ void put_4x4(unsigned r0, unsigned r1, unsigned r2, unsigned r3, unsigned char *d, int pitch)
{
    const unsigned lo01 = __builtin_amdgcn_perm(r1, r0, 0x05010400), hi01 = __builtin_amdgcn_perm(r1, r0, 0x07030602);
    const unsigned lo23 = __builtin_amdgcn_perm(r3, r2, 0x05010400), hi23 = __builtin_amdgcn_perm(r3, r2, 0x07030602);
    *reinterpret_cast<unsigned *>(d) = __builtin_amdgcn_perm(lo23, lo01, 0x05040100);
    *reinterpret_cast<unsigned *>(d + pitch) = __builtin_amdgcn_perm(lo23, lo01, 0x07060302);
    *reinterpret_cast<unsigned *>(d + 2 * pitch) = __builtin_amdgcn_perm(hi23, hi01, 0x05040100);
    *reinterpret_cast<unsigned *>(d + 3 * pitch) = __builtin_amdgcn_perm(hi23, hi01, 0x07060302);
}

// Eight pixels of four channels (a channel per 64-bit value).
__device__ __forceinline__ void put_4x8(const unsigned long long (&v)[4], unsigned char *d, int pitch)
{
    put_4x4((unsigned)v[0], (unsigned)v[1], (unsigned)v[2], (unsigned)v[3], d, pitch);
    put_4x4((unsigned)(v[0] >> 32), (unsigned)(v[1] >> 32), (unsigned)(v[2] >> 32), (unsigned)(v[3] >> 32), d + 4 * pitch, pitch);
}

// The form for windows of many pixels: a unit is 4 channels x 16 pixels, four lanes take 64 bytes of a channel row in 16-byte
// loads, the next four the next quad's.  What decides there is how many cache lines a load instruction names: one whose lanes
// are a channel plane apart each (the form below) takes 20 to 65 cycles, one of these 14 (64 images 56 x 56, 64 -> 64: 18.0 -> 15.9 us;
// 16 images 72 x 56 x 56 -> 96, stride 2: 9.7 -> 8.1).  The LDS stores of four lanes meet in the same banks, which costs
// about what the loads do.  false, nothing done: a load could pass the tensor's end.
template <int NT, int B, typename Place>
__device__ __forceinline__ bool window_wide_nchw(const WindowSource &t, const WindowRange &w, int cq, unsigned mg_cq, Place &&place, int pitch, int tid)
{
    const int8_t *const src = t.src + (long long)w.n0 * t.img_bytes;
    const long long left = t.src_bytes - (long long)w.n0 * t.img_bytes;
    const bool padded = t.C1 + 1 != 4 * cq;
    // (the last image's rows of the last channels, rounded up to 16 pixels, are the last bytes any unit asks for)
    const int over = w.slots - w.len0, images = over > 0 ? fast_div_any(over - 1, w.full8, w.mg_full8) + 1 : 0;
    const int last_end = images ? over - (images - 1) * w.full8 : w.lo0 + w.len0;
    const bool inside = (long long)images * t.img_bytes + (long long)t.C1 * t.HW + last_end + 8 <= left;
    if (!inside) return false;
    constexpr int U = B / 2;   // units per thread and round of loads
    const int units = ((w.slots + 63) >> 6) * 4 * cq;
    for (int u0 = tid; u0 < units; u0 += NT * U) {
        v4i v[U][4];
        int at[U], c4[U];
#pragma unroll
        for (int b = 0; b < U; ++b) {
            const int u = u0 + b * NT, rest = u >> 2, run = fast_div_any(rest, cq, mg_cq);
            c4[b] = (rest - run * cq) * 4;
            at[b] = u < units ? (run * 4 + (u & 3)) * 16 : w.slots;
            if (at[b] < w.slots) {
                int n, lin;
                window_slot(w, at[b], &n, &lin);
                const int8_t *const p = src + (long long)(n - w.n0) * t.img_bytes + lin;
                const int ahead = at[b] < w.len0 ? w.len0 - at[b] : w.full8 - lin;   // slots of this image's range from here on
                if (ahead >= 16 || at[b] + 8 >= w.slots) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) __builtin_memcpy(&v[b][i], p + (long long)min(c4[b] + i, t.C1) * t.HW, 16);
                } else {   // the other eight pixels begin the next image
                    const int8_t *const p2 = src + (long long)(n + 1 - w.n0) * t.img_bytes;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const long long c = (long long)min(c4[b] + i, t.C1) * t.HW;
                        unsigned long long x[2];
                        x[0] = *reinterpret_cast<const u64_a1 *>(p + c);
                        x[1] = *reinterpret_cast<const u64_a1 *>(p2 + c);
                        __builtin_memcpy(&v[b][i], x, 16);
                    }
                }
            }
        }
#pragma unroll
        for (int b = 0; b < U; ++b)
            if (at[b] < w.slots) {
                if (padded)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (c4[b] + i > t.C1) v[b][i] = v4i{0, 0, 0, 0};
                unsigned char *const d = place(at[b], c4[b]);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e < 2 || at[b] + 8 < w.slots)
                        put_4x4((unsigned)v[b][0][e], (unsigned)v[b][1][e], (unsigned)v[b][2][e], (unsigned)v[b][3][e], d + 4 * e * pitch, pitch);
            }
    }
    return true;
}

__host__ __device__ static inline bool window_takes_runs(int slots, int cq, int wide, int threads, bool deep = false)
{
    const int runs = (slots + 63) >> 6;
    return (slots >= 128 || slots * 5 >= runs * 256 || (deep && cq > 64 && slots > 32)) && runs * cq * wide >= threads;
}

// NCHW -> records; bytes past the last channel are zero.  cq: channel quads of a record.  The form for few pixels: a unit is 4
// channels x 8 pixels, neighbouring lanes on neighbouring channel quads (a record's pieces fall into different banks), no
// lane without work.  (Bound by the instruction count of a lone wave, hence the short path: one image, nothing past the
// tensor's end, whole quads only: scalar bases and one 32-bit offset per unit.)  The other form from 128 pixels on, or where
// its runs of 64 are four fifths full, if it has work for every thread: below, its idle lanes cost more than its loads save
// (2 images 292 x 20 x 20 -> 66, 88 pixels: 8.2 us, 9.4 with it; 15 images 256 x 7 x 7 -> 26: 9.4 and 9.0; 8 images 64 x 7 x 7 ->
// 130: 4.7 and 4.9).
// DEEP (the stream kernel): above 256 channels whatever the idle lanes.  A window's channel rows are then more cache lines than the L1 holds, and the
// form for few pixels comes back to each of them once per eight pixels: 450 launches on 72 to 96 pixels of 512 channels 0.915 of the time in the
// mean, at best 0.77 (134 on 40 and 48 pixels 0.947; 5 to 7 chunks of 64 channels 0.96 to 0.98).  Planes of less than 64 pixels: 1.02, at worst 1.4.
// place(slot, channel): where a record's dword of four channels goes.  RUNS: the other form is compiled in.
template <int NT, int B, bool RUNS, bool DEEP, typename Place>
__device__ __forceinline__ void window_from_nchw_to(const WindowSource &t, const WindowRange &w, int cq, unsigned mg_cq, Place &&place, int pitch, int tid)
{
    if (RUNS && window_takes_runs(w.slots, cq, t.wide, NT, DEEP) && window_wide_nchw<NT, B>(t, w, cq, mg_cq, place, pitch, tid)) return;
    const int units = cq * (w.slots >> 3);
    const long long img0 = (long long)w.n0 * t.img_bytes;
    if (w.slots == w.len0 && t.C1 + 1 == 4 * cq && img0 + (long long)t.C1 * t.HW + w.lo0 + w.slots <= t.src_bytes) {
        const int8_t *const b0 = t.src + img0 + w.lo0, *const b1 = b0 + t.HW, *const b2 = b1 + t.HW, *const b3 = b2 + t.HW;
        for (int u0 = tid; u0 < units; u0 += NT * B) {   // B: units per thread and round of loads
            unsigned long long v[B][4];
            unsigned char *dst[B];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int u = u0 + b * NT;
                if (u < units) {
                    const int g = fast_div_any(u, cq, mg_cq), c4 = (u - g * cq) * 4;
                    const unsigned off = (unsigned)(c4 * t.HW + g * 8);
                    dst[b] = place(g * 8, c4);
                    v[b][0] = *reinterpret_cast<const u64_a1 *>(b0 + off);
                    v[b][1] = *reinterpret_cast<const u64_a1 *>(b1 + off);
                    v[b][2] = *reinterpret_cast<const u64_a1 *>(b2 + off);
                    v[b][3] = *reinterpret_cast<const u64_a1 *>(b3 + off);
                }
            }
#pragma unroll
            for (int b = 0; b < B; ++b)
                if (u0 + b * NT < units) put_4x8(v[b], dst[b], pitch);
        }
        return;
    }
    for (int u0 = tid; u0 < units; u0 += NT * B) {
        unsigned long long v[B][4];
        unsigned char *dst[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int u = min(u0 + b * NT, units - 1), g = fast_div_any(u, cq, mg_cq), c4 = (u - g * cq) * 4;
            int n, lin;
            window_slot(w, g * 8, &n, &lin);
            dst[b] = place(g * 8, c4);
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
            put_4x8(v[b], dst[b], pitch);
        }
    }
}
template <int NT, int B, bool RUNS>
__device__ __forceinline__ void window_from_nchw(const WindowSource &t, const WindowRange &w, int cq, unsigned mg_cq, unsigned char *win, int pitch, int tid)
{
    window_from_nchw_to<NT, B, RUNS, false>(t, w, cq, mg_cq, [&](int slot, int c4) { return win + slot * pitch + c4; }, pitch, tid);
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

// Blocked source [n][block][pixel][16 << g16_log2 channels] -> records: 16-byte pieces in the order they lie in, so that a wave's loads are whole
// lines.  u16: pieces of a record.
template <int NT, int B>
__device__ __forceinline__ void window_from_blocks(const WindowSource &t, const WindowRange &w, int u16, int g16_log2, unsigned char *win, int pitch, int tid)
{
    const int per = w.slots << g16_log2, blocks = (u16 + (1 << g16_log2) - 1) >> g16_log2, units = per * blocks;
    const unsigned mg_per = magic_for_device(max(per, 1));
    const int8_t *const src = t.src + (long long)w.n0 * t.img_bytes;
    const int block_bytes = t.HW * t.pstride;
    for (int u0 = tid; u0 < units; u0 += NT * B) {
        v4i v[B];
        int dst[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int u = min(u0 + b * NT, units - 1), blk = fast_div_any(u, per, mg_per), rest = u - blk * per;
            const int s = rest >> g16_log2, j = rest & ((1 << g16_log2) - 1), piece = (blk << g16_log2) + j;
            int n, lin;
            window_slot(w, s, &n, &lin);
            dst[b] = piece < u16 && u0 + b * NT < units ? s * pitch + piece * 16 : -1;
            v[b] = *reinterpret_cast<const v4i *>(src + (long long)(n - w.n0) * t.img_bytes + (blk * block_bytes + min(lin, t.HW - 1) * t.pstride + j * 16));
        }
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (dst[b] >= 0) *reinterpret_cast<v4i *>(win + dst[b]) = v[b];
    }
}

}  // namespace c2i8
