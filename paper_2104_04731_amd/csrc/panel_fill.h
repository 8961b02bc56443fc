// Windows of the panel kernel: slots of a virtual image, filled from the network's own tensors.
//
// The virtual image holds all images one below the other with `pad` rows of zeros above each and `pad` zeros in front of
// every row: rows of Wv = W + pad slots, Hv = H + pad rows per image.  What a tap reads right of a row are the next row's zeros, what
// it reads below an image the next one's.  So a tap is a fixed distance from the pixel's first one, nothing is masked, and the window of
// consecutive output pixels is one run of slots, over any number of images.
#pragma once
#include "window_fill.h"

namespace c2i8 {

struct VirtualImage {
    int Wv, Hv, N, C, H, W, HW, pad;
    int chunks;                       // of 64 channels
    int pstride;                      // NHWC: bytes from pixel to pixel
    long long img_bytes, src_bytes;
    unsigned mg_Wv, mg_Hv;
};

// What the above asks of a problem: eight slots meet a row's border at most once, and the window of an image's last pixels ends in the next
// image's border (its first taps follow the previous image's).  And slots and images that 32 bits count.
static inline bool virtual_image_fits(int R, int S, int dil, long long H, long long W, int pad, long long N, long long img_bytes)
{
    return (pad ? W + pad >= 8 : H * W >= 8) && pad <= (R - 1) * dil && pad <= (S - 1) * dil && (N + 1) * (H + pad) * (W + pad) <= 0x3FFFFFFFLL &&
           img_bytes <= 0x7FFFFFFFLL && N * img_bytes >= 16;
}
// Slots, in eights, of the largest window of `mper` pixels: from pixel to pixel `stride`, more where a row and where an image ends.
static inline long long window_slots(int mper, int PQ, int Q, int stride, long long Wv, long long Hv, long long span)
{
    const long long row = stride * (Wv - Q), img = (Hv - (long long)PQ / Q * stride) * Wv, steps = mper - 1;
    const long long rows = (steps + Q - 1) / Q, imgs = (steps + PQ - 1) / PQ;
    return (steps * stride + rows * (row > 0 ? row : 0) + imgs * (img > 0 ? img : 0) + span + 8) / 8 * 8;
}

// Where the window's slots lie in memory, once per workgroup and for all chunks.
//   NCHW: an entry per eight slots.  x: offset of the first real one from the window's first image; y, z: selectors that make the eight
//         slots of the eight bytes there -- zeros where the border is, which they meet at most once; w: 0, or (no border between them) where
//         in the eight the next image begins and, from bit 4 on, how many images on.
//   NHWC: an entry per slot, its pixel's offset or PANEL_BORDER.
typedef unsigned panel_v4u __attribute__((ext_vector_type(4)));
constexpr unsigned PANEL_ZERO = 0x0c0c0c0cu, PANEL_BORDER = 0xFFFFFFFFu;
__device__ __forceinline__ panel_v4u oct_entry(const VirtualImage &v, int n0, int slot)
{
    const int vr = fast_div_any(slot, v.Wv, v.mg_Wv), vc = slot - vr * v.Wv;
    const int n = fast_div_any(vr, v.Hv, v.mg_Hv), rr = vr - n * v.Hv;
    const int row = max(rr - v.pad, 0), col = rr < v.pad ? 0 : max(vc - v.pad, 0), lin = row * v.W + col;
    // bytes [lead, end) of the eight follow one another from pixel lin on, [next, 8) behind them (the next row's)
    const int lead = n >= v.N ? 8 : min(rr < v.pad ? (v.pad - rr) * v.Wv - vc + v.pad : max(v.pad - vc, 0), 8);
    const int end = min(lead + (v.pad ? v.W - col : v.HW - lin), 8);   // (without a border the rows of an image are one run)
    const bool cross = v.pad == 0 && end < 8 && n + 1 < v.N;
    const int next = cross ? end : v.pad && row + 1 < v.H ? min(end + v.pad, 8) : 8;
    panel_v4u e = {lead < 8 ? (unsigned)(n - n0) * (unsigned)v.img_bytes + (unsigned)lin : 0u, 0, 0, cross ? (unsigned)(end | (n + 1 - n0) << 4) : 0u};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const unsigned pick = i < lead ? 0x0cu : i < end ? (unsigned)(i - lead) : i < next ? 0x0cu : (unsigned)(i - lead - (next - end));
        e[1 + (i >> 2)] |= pick << (8 * (i & 3));
    }
    return e;
}
__device__ __forceinline__ unsigned slot_entry(const VirtualImage &v, int n0, int slot)
{
    const int vr = fast_div_any(slot, v.Wv, v.mg_Wv), col = slot - vr * v.Wv - v.pad;
    const int n = fast_div_any(vr, v.Hv, v.mg_Hv), row = vr - n * v.Hv - v.pad;
    return row < 0 || col < 0 || n >= v.N ? PANEL_BORDER : (unsigned)(n - n0) * (unsigned)v.img_bytes + (unsigned)((row * v.W + col) * v.pstride);
}

// base + off, the base uniform: one instruction's scalar base and 32-bit lane offset.  (Where the offset is made 64 bits wide in another block
// than the load's the compiler adds the two in vector registers instead.)
__device__ __forceinline__ const int8_t *panel_local(const int8_t *base, unsigned off)
{
#ifdef __HIP_DEVICE_COMPILE__
    asm("" : "+v"(off));
#endif
    return base + off;
}

// What a window is filled from: its slots [0, 8 * octs) in the images from img0 on; left: bytes from there to the tensor's end.
struct PanelWindow {
    const int8_t *img0;
    long long left;
    int octs;
    unsigned mg_octs;
    bool last;      // the tensor ends within 128 bytes of the last image filled from: a load that goes beyond what it is for could pass the end
};
__device__ __forceinline__ PanelWindow panel_window(const VirtualImage &v, const int8_t *src, int n0, int lo, int last_slot)
{
    // (the last slot that is filled, not the last one a tap reads: without a border up to seven more are the next image's pixels)
    const int n1 = fast_div_any(fast_div_any(lo + ((last_slot - lo + 8) & ~7) - 1, v.Wv, v.mg_Wv), v.Hv, v.mg_Hv);
    PanelWindow w;
    w.img0 = src + (long long)n0 * v.img_bytes;
    w.left = v.src_bytes - (long long)n0 * v.img_bytes;
    w.octs = (last_slot - lo + 8) >> 3;
    w.mg_octs = magic_for_device(w.octs);
    w.last = (long long)(n1 - n0 + 1) * v.img_bytes + 128 > w.left;
    return w;
}

// A round of a fill: 16 pieces (eight slots of a chunk) -- or 64 of slots, NHWC -- of those of `chunks` chunks from `first` on, by 256 threads.
// take() asks for the pixels, put() stores them to `buf`, a chunk's buffer `pitch * slots` bytes behind the one before.
template <bool PIXEL_MAJOR>
struct PanelFill;

// NCHW: a thread takes 8 slots of 4 channels; four neighbouring lanes are 32 slots of a channel quad, a wave's lanes all sixteen quads: the LDS stores
// of four lanes meet in the same banks.  (With 64 slots of eight quads eight do: 1.015 of the time; with one lane per quad the loads name more lines: 1.02.)
template <>
struct PanelFill<false> {
    static constexpr int ENTRY = 16;   // bytes of table per eight slots
    unsigned long long x[4];
    // the thread's piece of a round; false: none
    static __device__ __forceinline__ bool piece(const PanelWindow &w, int chunks, int round, int t, int *chunk, int *oct)
    {
        const int item = round * 16 + ((t >> 4) & 12) + (t & 3);
        *chunk = fast_div_any(item, w.octs, w.mg_octs);
        *oct = item - *chunk * w.octs;
        return *chunk < chunks;
    }

    static __device__ __forceinline__ int rounds(const PanelWindow &w, int chunks) { return (w.octs * chunks + 15) >> 4; }
    static __device__ __forceinline__ void table(const VirtualImage &v, const PanelWindow &w, int n0, int lo, unsigned char *tab, int t, int threads)
    {
        for (int o = t; o < w.octs; o += threads) reinterpret_cast<panel_v4u *>(tab)[o] = oct_entry(v, n0, lo + 8 * o);
    }
    template <bool LAST>   // PanelWindow::last
    __device__ __forceinline__ void take(const VirtualImage &v, const PanelWindow &w, const unsigned char *tab, int first, int chunks, int round, int t)
    {
        int chunk, oct;
        if (!piece(w, chunks, round, t, &chunk, &oct)) return;
        const panel_v4u *const e = reinterpret_cast<const panel_v4u *>(tab) + oct;
        const unsigned at = (*e)[0], cross = v.pad ? 0u : (*e)[3];
        const int c = (first + chunk) * 64 + ((t >> 2) & 15) * 4;
        // (channels past the last one: weights there are zeros, any byte will do)
        unsigned off[4];
        if ((v.C & 3) == 0) {   // (uniform)
            off[0] = at + (unsigned)(min(c, v.C - 4) * v.HW);
#pragma unroll
            for (int i = 1; i < 4; ++i) off[i] = off[0] + (unsigned)(i * v.HW);
        } else
#pragma unroll
            for (int i = 0; i < 4; ++i) off[i] = at + (unsigned)(min(c + i, v.C - 1) * v.HW);
        // LAST: eight bytes that would pass the tensor's end begin earlier
        auto eight = [&](unsigned o) -> unsigned long long {
            if constexpr (!LAST) return *reinterpret_cast<const u64_a1 *>(panel_local(w.img0, o));
            const long long from = (long long)o < w.left - 8 ? (long long)o : w.left - 8;
            return *reinterpret_cast<const u64_a1 *>(w.img0 + from) >> (8 * (int)((long long)o - from));
        };
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = eight(off[i]);
        if (cross) {
            const int end = cross & 15;   // (1 ... 7)
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = (x[i] & ((1ull << (8 * end)) - 1)) | eight(off[i] - at + (cross >> 4) * (unsigned)v.img_bytes) << (8 * end);
        }
    }
    __device__ __forceinline__ void put(const PanelWindow &w, const unsigned char *tab, int chunks, int round, unsigned char *buf, int bytes, int pitch, int t) const
    {
        int chunk, oct;
        if (!piece(w, chunks, round, t, &chunk, &oct)) return;
        const panel_v4u *const e = reinterpret_cast<const panel_v4u *>(tab) + oct;
        unsigned char *const d = buf + chunk * bytes + oct * 8 * pitch + ((t >> 2) & 15) * 4;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const unsigned pick = (*e)[1 + h];
            unsigned y[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) y[i] = __builtin_amdgcn_perm((unsigned)(x[i] >> 32), (unsigned)x[i], pick);
            put_4x4(y[0], y[1], y[2], y[3], d + h * 4 * pitch, pitch);
        }
    }
};

// NHWC: a thread takes 16 of a chunk's channels of two slots; four neighbouring lanes are a slot.
template <>
struct PanelFill<true> {
    static constexpr int ENTRY = 32;
    v4i x[2];
    static __device__ __forceinline__ bool piece(const PanelWindow &w, int chunks, int round, int h, int t, int *chunk, int *slot)
    {
        const int item = round * 16 + h * 8 + (t >> 5);
        *chunk = fast_div_any(item, w.octs, w.mg_octs);
        *slot = (item - *chunk * w.octs) * 8 + ((t >> 2) & 7);
        return *chunk < chunks;
    }

    static __device__ __forceinline__ int rounds(const PanelWindow &w, int chunks) { return (w.octs * chunks + 15) >> 4; }
    static __device__ __forceinline__ void table(const VirtualImage &v, const PanelWindow &w, int n0, int lo, unsigned char *tab, int t, int threads)
    {
        for (int s = t; s < 8 * w.octs; s += threads) reinterpret_cast<unsigned *>(tab)[s] = slot_entry(v, n0, lo + s);
    }
    template <bool LAST>   // PanelWindow::last
    __device__ __forceinline__ void take(const VirtualImage &v, const PanelWindow &w, const unsigned char *tab, int first, int chunks, int round, int t)
    {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int chunk, slot;
            if (!piece(w, chunks, round, h, t, &chunk, &slot)) continue;
            const unsigned at = reinterpret_cast<const unsigned *>(tab)[slot];
            const int c = (first + chunk) * 64 + (t & 3) * 16;
            const unsigned off = (at == PANEL_BORDER ? 0u : at) + (unsigned)c;
            if constexpr (!LAST) {   // (the channels behind a pixel's last one are the next pixels')
                __builtin_memcpy(&x[h], panel_local(w.img0, off), 16);
            } else {
                const long long want = off, from = want < w.left - 16 ? want : w.left - 16;
                v4i y;
                __builtin_memcpy(&y, w.img0 + from, 16);
                const int over = (int)(want - from);   // (16 and more: channels that no weight belongs to)
                x[h] = over ? shift_piece(y, -min(over, 15)) : y;
            }
        }
    }
    __device__ __forceinline__ void put(const PanelWindow &w, const unsigned char *tab, int chunks, int round, unsigned char *buf, int bytes, int pitch, int t) const
    {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int chunk, slot;
            if (!piece(w, chunks, round, h, t, &chunk, &slot)) continue;
            const bool border = reinterpret_cast<const unsigned *>(tab)[slot] == PANEL_BORDER;
            *reinterpret_cast<v4i *>(buf + chunk * bytes + slot * pitch + (t & 3) * 16) = border ? v4i{0, 0, 0, 0} : x[h];
        }
    }
};

}  // namespace c2i8
