// GEMM stage that takes its activations from the network's own tensor: channel blocking happens on the way into LDS,
// nothing rewritten is stored.
//
// The two-stage path (pack_layout, then the GEMM stage of igemm_mfma.hip) writes the blocked image to memory, fetches it
// once per kernel tap (R*S times through L2 and the global->LDS path), needs a launch of its own for the first half, and
// its one workgroup per compute unit does not store while it multiplies.  Here a workgroup owns `mper` consecutive output
// pixels x TK output channels; the weights of its channels and the input pixels it touches -- a contiguous range of every
// channel plane, turned around to pixel-major records of all channels -- are brought into LDS once, then every wave takes
// blocks of 32 or 64 pixels through the whole depth and stores them, with no barrier in between: the stores of one
// block drain while the next multiplies.
//   * window: the range is kept as it is, without the zero border; a lane whose tap falls outside the image reads a
//     record of zeros instead (one bit per tap and pixel).  A tile may span images: one range per image.
//   * record pitch: an odd number of 16-byte units, so that the fragment reads of 16 neighbouring pixels (stride 1)
//     start in 16 different bank groups and a tap's offset is a plain addition.
//   * depth order: that of pack_weights (PACKED with any block, PAD_ONLY), or (tap, channel) for 3x3 weights that come
//     raw: 36 bytes of four channels x nine taps are nine dwords of the tile after 27 byte permutes.
//   * 1x1 weights that come raw are in that order already, in rows of C bytes: fetched in pieces of 16, zeros behind the
//     last channel, so that a step of depth may read past a record (whatever lies there is multiplied by zero).
//   * the blocked image of the layer before (a chain's): records come whole, the border is in the image, and the result leaves as the next layer's
//     blocked input.  The general kernel fetches every activation once per tap.
// Bound: the memory system (input once, result once) for the small and middle depths the kernel is for -- weights plus
// window must fit one compute unit's LDS, which rules out 3x3 layers of more than about 300 channels.  Measured in a
// graph, two-stage -> this kernel: 64 images 56x56, 64 -> 64, 3x3: 38 -> 19.6 us with rewritten weights (12.8 MB in, 51 MB
// out), 38 -> 19.7 from raw ones; 16 images 56x56, 72 -> 96, stride 2: 12.2 -> 10.6; 445 images 14x14, 32 -> 405: 46 -> 36;
// dilation 2, 64 images 28x28, 64 -> 64: 19.6 through sub-images -> 8.9.  From and to blocked images: 64 images 56x56, 64 -> 64: 24.0 -> 14.7 (12.8 MB
// in, 12.8 MB out: a fill, a chain of MFMAs and a store that follow one another in the one workgroup that a compute unit has).
#include "act_store.h"
#include "launch.h"
#include "window_fill.h"

namespace c2i8 {

namespace {

typedef int v16i __attribute__((ext_vector_type(16)));

struct ResidentArgs {
    const int8_t *src, *wq;
    int32_t *out;                  // [N][K][P][Q], or [N][P][Q][K] (out_nhwc)
    int out_nhwc;
    int K, M, PQ, Q;
    int C, C1, H, W, HW;           // C1 = C - 1
    int stride, pad, dil, R, S;
    int depth, steps;              // bytes per weight row, 64-byte steps
    int cb, nreal, C16;            // weights' channel block; 16-byte chunks of depth that hold weights; bytes of a record
    int pitch, full8;              // record pitch; slots of a whole image (its range rounded up to 8 pixels)
    int pstride;                   // pixel-major source: bytes from pixel to pixel
    long long img_bytes, src_bytes;
    int zero_off, win_off, tab_off;  // LDS byte offsets (the weight tile is at 0)
    int tiles_k, tiles_m, mper;    // mper: output pixels of a workgroup
    int nblk, parts;               // blocks of pixels that a wave multiplies at a time; waves that share the depth of each (1: none do)
    int stream_out;                // NKPQ result with non-temporal stores
    unsigned mg_nblk, mg_parts, mg_PQ, mg_Q, mg_tiles_k, mg_c16q, mg_cq, mg_full8, mg_g16, mg_S, mg_R, mg_u16;
    int cq, u16;                   // channel quads / 16-byte units of a record that are loaded
};
struct ResidentBlockedArgs : ResidentArgs {
    ActOut act;
    int g16_log2;                  // 16-byte pieces of a block of the source
};

__device__ __forceinline__ void res_dma16(const int8_t *src, unsigned lds_base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_base), "v"(src) : "memory");
}
template <int N>
__device__ __forceinline__ void res_wait_dma()
{
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
__device__ __forceinline__ void res_barrier()
{
    asm volatile("" : : : "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" : : : "memory");
}

// RES_BLOCKED: the blocked image of the layer before, its border there already; the result goes on as the next one's (ActOut).
enum ResSource : int { RES_NCHW = 0, RES_PIXELS = 1, RES_BLOCKED = 2 };
enum ResWeights : int { RES_PACKED = 0, RES_RAW9 = 1, RES_RAW1 = 2 };   // in depth order; KCRS of 3 x 3 and of 1 x 1 kernels


// D block (i, f): column = lane%32 (pixel), row = 8*(v/4) + 4*(lane/32) + v%4 (channel).  kw, mw: the wave's first channel
// and pixel; pixels from m1 on are another workgroup's.  Whatever does not depend on the block is made from a value
// the compiler cannot see through: hoisted out of the loop over blocks it would take every scalar register there is.
template <int FK, int FM>
__device__ __forceinline__ void res_store(const ResidentArgs &a, const v16i (&acc)[FK][FM], int kw, int mw, int m1, int n0, int lane)
{
    int K = a.K, PQ = a.PQ;
    asm volatile("" : "+s"(K), "+s"(PQ));
    const int half4 = 4 * (lane >> 5);
    if (a.out_nhwc) {
        const bool wide = (K & 3) == 0 && (reinterpret_cast<uintptr_t>(a.out) & 15) == 0;
#pragma unroll
        for (int f = 0; f < FM; ++f) {
            const int m = mw + f * 32 + (lane & 31);
            int32_t *px = a.out + (size_t)m * K + kw + half4;
            if (m < m1)
#pragma unroll
                for (int i = 0; i < FK; ++i)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int left = K - (kw + half4 + i * 32 + 8 * g);
                        const v4i t = {acc[i][f][4 * g], acc[i][f][4 * g + 1], acc[i][f][4 * g + 2], acc[i][f][4 * g + 3]};
                        if (wide) {
                            if (left > 0) *reinterpret_cast<v4i *>(px + i * 32 + 8 * g) = t;
                        } else if (left >= 4) *reinterpret_cast<v4i_a4 *>(px + i * 32 + 8 * g) = t;   // (rows of K values begin on any dword)
                        else
                            for (int v = 0; v < 3; ++v)
                                if (v < left) px[i * 32 + 8 * g + v] = t[v];
                    }
        }
    } else {
        // a wave-uniform row base (advanced by whole rows) + one 32-bit byte offset per lane and pixel block
        const size_t row = (size_t)PQ * sizeof(int32_t);
        const bool whole = kw + FK * 32 <= K;
#pragma unroll
        for (int f = 0; f < FM; ++f) {
            const int m = mw + f * 32 + (lane & 31);
            const int n = fast_div_any(m, PQ, a.mg_PQ), pq = m - n * PQ;
            const unsigned off = ((unsigned)(n - n0) * (unsigned)K * (unsigned)PQ + (unsigned)(half4 * PQ + pq)) * 4u;
            char *r0 = reinterpret_cast<char *>(a.out) + ((size_t)n0 * K + kw) * row;
            if (m < m1) {
                if (whole && a.stream_out) {
#pragma unroll
                    for (int i = 0; i < FK; ++i)
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            __builtin_nontemporal_store(acc[i][f][v], reinterpret_cast<int32_t *>(r0 + off));
                            r0 += (v & 3) == 3 ? 5 * row : row;
                        }
                } else if (whole) {
#pragma unroll
                    for (int i = 0; i < FK; ++i)
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            *reinterpret_cast<int32_t *>(r0 + off) = acc[i][f][v];
                            r0 += (v & 3) == 3 ? 5 * row : row;
                        }
                } else {
                    const int left = K - kw - half4;
#pragma unroll
                    for (int i = 0; i < FK; ++i)
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            if (i * 32 + 8 * (v >> 2) + (v & 3) < left) *reinterpret_cast<int32_t *>(r0 + off) = acc[i][f][v];
                            r0 += (v & 3) == 3 ? 5 * row : row;
                        }
                }
            }
        }
    }
}

// The same activated, into the next layer's blocked input.
template <int FK, int FM>
__device__ __forceinline__ void res_store_act(const ResidentBlockedArgs &a, const v16i (&acc)[FK][FM], int kw, int mw, int m1, int lane)
{
    int K = a.K, PQ = a.PQ, cbl = a.act.cb_log2;
    asm volatile("" : "+s"(K), "+s"(PQ), "+s"(cbl));
    const int half = lane >> 5;
#pragma unroll
    for (int f = 0; f < FM; ++f) {
        const int m = mw + f * 32 + (lane & 31);
        const int n = fast_div_any(m, PQ, a.mg_PQ), pq = m - n * PQ;
        const int p = fast_div_any(pq, a.Q, a.mg_Q), q = pq - p * a.Q;
        const long long plane = (long long)a.act.Hp * a.act.Wp, pix = (long long)n * a.act.Cb * plane + (long long)(p + a.act.pad) * a.act.Wp + (q + a.act.pad);
#pragma unroll
        for (int i = 0; i < FK; ++i) {
            const int kb = kw + i * 32, k = kb + 16 * half;
            const v4i y = act_block16(acc[i][f], K - kb, lane, a.act.shift, a.act.relu);
            int8_t *dst = a.act.out + (((pix + (k >> cbl) * plane) << cbl) + (k & ((1 << cbl) - 1)));
            if (m < m1 && k < a.act.Cb << cbl) {
                *reinterpret_cast<v4i *>(dst) = y;
                if (FK == 1 && act_half_left(kb, K, cbl)) *reinterpret_cast<v4i *>(dst + 32) = v4i{0, 0, 0, 0};
            }
        }
    }
}

// One piece of a block (rows 8g + 4*(lane/32) + 0..3), summed up from the depth parts: row k of the result onwards, pixel m.
__device__ __forceinline__ void res_store_piece(const ResidentArgs &a, const v4i &t, int k, int m, int m1, int n0)
{
    const int left = a.K - k;
    if (m >= m1 || left <= 0) return;
    if (a.out_nhwc) {
        int32_t *px = a.out + (size_t)m * a.K + k;
        if ((a.K & 3) == 0 && (reinterpret_cast<uintptr_t>(a.out) & 15) == 0) *reinterpret_cast<v4i *>(px) = t;
        else if (left >= 4) *reinterpret_cast<v4i_a4 *>(px) = t;
        else
            for (int v = 0; v < 3; ++v)
                if (v < left) px[v] = t[v];
    } else {
        const int n = fast_div_any(m, a.PQ, a.mg_PQ), pq = m - n * a.PQ;
        int32_t *px = a.out + ((size_t)n * a.K + k) * a.PQ + pq;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (v < left) px[(size_t)v * a.PQ] = t[v];
    }
}

// TK: output channels of a workgroup, NW: waves (each multiplies all of the channels), FM: 32-pixel blocks a wave
// multiplies at a time; SRC: ResSource; UNI: a 64-byte step of depth lies within one tap (and channel block);
// SPLIT: a workgroup has fewer blocks of pixels than waves, and several waves share the depth of each (a form of its own: in the
// other one's code the smallest launches took half a microsecond longer).
// WTS: ResWeights.  RES_RAW9: turned into depth order (tap, channel padded to 16) on their way into LDS; RES_RAW1: in that order already, a step
// of depth always within the one tap (always UNI).
// RUNS: NCHW windows may be filled in 64-byte runs (a form of its own: that code, jumped over, cost calls of 4 to 6 us 1.0 to 1.6 % on given weights;
// on raw ones it is there for every plane of 64 pixels and more: 33 layers that jump over it took 1.5 % longer without it).
// The 64-channel tile of 8 waves keeps two output blocks' sums and the addresses of a whole tap in registers: at two of its
// workgroups per compute unit it spilled, at one it does not, and its LDS rarely leaves room for two (64 images 56 x 56,
// 64 -> 64, kept weights: 18.0 -> 17.4 us; 151 images 28 x 28, 128 -> 458: 116 -> 105).
template <int TK, int NW, int FM, int SRC, bool UNI, int WTS, bool SPLIT, bool RUNS>
__global__ void __launch_bounds__(NW * 64, TK == 64 && NW == 8 ? 2 : NW / 2)
    conv_resident_kernel(const std::conditional_t<SRC == RES_BLOCKED, ResidentBlockedArgs, ResidentArgs> a)
{
    constexpr int NT = NW * 64, FK = TK / 32;
    constexpr int STEP = TK * 64;   // LDS bytes of one 64-byte step of the weight tile
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const unsigned lds0 = (unsigned)(size_t)((__attribute__((address_space(3))) unsigned char *)smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // channel tiles fastest: the workgroups of one pixel range share its input behind one L2
    const int lid = xcd_contiguous(blockIdx.x, gridDim.x);
    const int tm = fast_div_any(lid, a.tiles_k, a.mg_tiles_k), tk = lid - tm * a.tiles_k;
    const int k0 = tk * TK, m0 = tm * a.mper, m1 = min(m0 + a.mper, a.M);

    int n1;
    const WindowRange range = tile_window(a, m0, m1, &n1);
    const int n0 = range.n0, lo0 = range.lo0, len0 = range.len0;

    // ---- weights ------------------------------------------------------------------------------------------------
    // RES_RAW1: the same pieces through registers, at any alignment.  The first two per thread are on their way while the window is asked for; four
    // were no faster in the deepest layers and 0.3 to 0.6 us slower in all others: a lone wave's instructions decide (2 images 120 x 56 x 56 -> 143,
    // the weights rewritten by a launch of their own: 8.5 us; four pieces per thread: 5.9, two: 5.3, what a whole piece does not need jumped over: 5.0).
    constexpr int G = TK / 16;
    const int lrow = lane >> 2, x = (lane & 3) ^ ((lane >> 4) & 3);
    constexpr int U1 = 2;
    v4i raw1[U1];
    auto raw1_batch = [&](int t0) {
#pragma unroll
        for (int b = 0; b < U1; ++b) {
            const int t = t0 + b * NW, st = t / G, g = t - st * G;
            if (t < a.steps * G) raw1[b] = raw1_load(a.wq, a.K, a.C, k0 + g * 16 + lrow, st * 64 + x * 16);
        }
    };
    if constexpr (WTS == RES_RAW1) raw1_batch(wave);
    if constexpr (WTS == RES_PACKED) {
        // a transfer moves 16 rows x 64 bytes of one step; a lane fetches the 16-byte chunk that belongs at its place
        // after the swizzle (chunk position XOR (row / 4) % 4)
        for (int t = wave; t < a.steps * G; t += NW) {
            const int st = t / G, g = t - st * G;
            const int8_t *src = a.wq + (size_t)min(k0 + g * 16 + lrow, a.K - 1) * a.depth + st * 64 + x * 16;
            res_dma16(src, lds0 + (unsigned)(st * STEP + g * 1024));
        }
    }
    // ---- window ---------------------------------------------------------------------------------------------------
    const WindowSource from{a.src, a.img_bytes, a.src_bytes, a.C1, a.HW, a.pstride};
    if constexpr (SRC == RES_NCHW) window_from_nchw<NT, 4, RUNS>(from, range, a.cq, a.mg_cq, smem + a.win_off, a.pitch, tid);
    else if constexpr (SRC == RES_BLOCKED) window_from_blocks<NT, 4>(from, range, a.u16, a.g16_log2, smem + a.win_off, a.pitch, tid);
    else window_from_pixels<NT, 4>(from, range, a.u16, a.mg_u16, smem + a.win_off, a.pitch, tid);
    if constexpr (WTS == RES_RAW1) {
        for (int t0 = wave; t0 < a.steps * G; t0 += NW * U1) {
            if (t0 != wave) raw1_batch(t0);
#pragma unroll
            for (int b = 0; b < U1; ++b)
                if (t0 + b * NW < a.steps * G) *reinterpret_cast<v4i *>(smem + (t0 + b * NW) * 1024 + lane * 16) = raw1[b];
        }
    }
    if constexpr (WTS == RES_RAW9) {
        // unit: one row, 4 channels; four units' loads in flight (15 images 256 x 7 x 7 -> 26, 4 units per thread: 7.9 us one by
        // one, 7.5 four at a time)
        constexpr int U = 4;
        const int cq = a.C16 >> 2, units = TK * cq;
        for (int u0 = tid; u0 < units; u0 += NT * U) {
            unsigned d[U][9];
            int row[U], c[U];
#pragma unroll
            for (int b = 0; b < U; ++b) {
                const int u = u0 + b * NT;
                row[b] = fast_div_any(u, cq, a.mg_c16q), c[b] = u - row[b] * cq;
                if (u < units) raw9_load(a.wq, a.K, a.C, k0 + row[b], c[b], d[b]);
            }
#pragma unroll
            for (int b = 0; b < U; ++b) {
                if (u0 + b * NT >= units) break;
                raw9_mask(a.C, c[b], d[b]);
                const int at0 = row[b] * 64 + (c[b] & 3) * 4, rsw = (row[b] >> 2) & 3;
                auto put = [&](int tap, unsigned v) {
                    if constexpr (UNI) {   // a tap is C16 / 64 whole steps
                        unsigned char *const at = smem + (c[b] >> 4) * STEP + at0 + ((((c[b] >> 2) & 3) ^ rsw) << 4);
                        *reinterpret_cast<unsigned *>(at + tap * (a.C16 >> 6) * STEP) = v;
                    } else {
                        const int j = tap * a.C16 + c[b] * 4;
                        *reinterpret_cast<unsigned *>(smem + (j >> 6) * STEP + at0 + ((((j >> 4) & 3) ^ rsw) << 4)) = v;
                    }
                };
                put(0, raw9_tap<0>(d[b])), put(1, raw9_tap<1>(d[b])), put(2, raw9_tap<2>(d[b]));
                put(3, raw9_tap<3>(d[b])), put(4, raw9_tap<4>(d[b])), put(5, raw9_tap<5>(d[b]));
                put(6, raw9_tap<6>(d[b])), put(7, raw9_tap<7>(d[b])), put(8, raw9_tap<8>(d[b]));
            }
        }
    }
    // A load whose value no unit of the last round needed may still be outstanding: without this wait the compiler puts
    // one before the first reuse of its register -- inside the main loop, where it waits for the weights just asked for.
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    if (tid < 16) *reinterpret_cast<unsigned *>(smem + a.zero_off + tid * 4) = 0;
    // ---- depth table: chunk -> record offset of its tap's chunk, bit of the tap in the lanes' masks (0: zeros) -----
    // UNI: a 64-byte step lies within one tap (and channel block): one entry per step
    typedef int v2i __attribute__((ext_vector_type(2)));
    v2i *const tab = reinterpret_cast<v2i *>(smem + a.tab_off);
    constexpr int EPS = UNI ? 1 : 4;    // entries per 64-byte step
    {
        const int g16 = a.cb >> 4;
        for (int i = tid; i < a.steps * EPS; i += NT) {
            const int t = UNI ? i * 4 : i;
            v2i e = {0, 0};
            if (t < a.nreal) {
                const int tap = fast_div_any(t, g16, a.mg_g16), sub = t - tap * g16;
                const int rb = fast_div_any(tap, a.S, a.mg_S), s = tap - rb * a.S;
                const int b = fast_div_any(rb, a.R, a.mg_R), r = rb - b * a.R;
                const int ch = b * a.cb + sub * 16;
                if (ch < a.C16) e = v2i{(r * a.W + s) * a.dil * a.pitch + ch, 1 << (r * a.S + s)};
            }
            tab[i] = e;
        }
    }

    res_wait_dma<0>();
    res_barrier();   // weights, window, table

    // ---- every wave on its own from here: blocks of FM x 32 pixels, all of the depth, straight to the result -------
    // (no barrier: the stores of one wave run beside the MFMAs of the others)
    const int rswz = (lane >> 2) & 3, half = lane >> 5;
    const int a0 = (lane & 31) * 64 + ((half ^ rswz) << 4), a1 = (lane & 31) * 64 + (((2 + half) ^ rswz) << 4);
    constexpr int NE = UNI ? 1 : 2;          // table entries of a step that a lane looks at
    constexpr int NQ = 2 * FK * FM, NI = 2 * (FK + FM);
    int blk = wave, j0 = 0, j1 = a.steps, part = 0;
    if constexpr (SPLIT) {
        part = fast_div(wave, a.mg_nblk);
        blk = part < a.parts ? wave - part * a.nblk : 1 << 20;
        const int per = fast_div(a.steps + a.parts - 1, a.mg_parts);
        j0 = min(part * per, a.steps), j1 = min(j0 + per, a.steps);
    }
    v16i acc[FK][FM];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < FK; ++i)
#pragma unroll
            for (int j = 0; j < FM; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;
    };
    if constexpr (SPLIT) clear();
    for (; m0 + blk * FM * 32 < m1; blk += NW) {
        const int mw = m0 + blk * FM * 32;
        // the lane's pixels: their records (tap (0, 0), first chunk) and which taps are in the image
        int base[FM];
        unsigned mask[FM];
#pragma unroll
        for (int f = 0; f < FM; ++f) {
            const int m = min(mw + f * 32 + (lane & 31), m1 - 1);
            const int n = fast_div_any(m, a.PQ, a.mg_PQ), pq = m - n * a.PQ;
            const int p = fast_div_any(pq, a.Q, a.mg_Q), q = pq - p * a.Q;
            const int row = p * a.stride - a.pad, col = q * a.stride - a.pad;
            const int seg = n == n0 ? -lo0 : len0 + (n - n0 - 1) * a.full8;
            base[f] = a.win_off + (seg + row * a.W + col) * a.pitch + (UNI ? half * 16 : 0);   // (else the table has the chunk)
            unsigned cm = 0, mk = 0;
            for (int s = 0; s < a.S; ++s) cm |= (unsigned)((unsigned)(col + s * a.dil) < (unsigned)a.W) << s;
            for (int r = 0; r < a.R; ++r) mk |= ((unsigned)(row + r * a.dil) < (unsigned)a.H ? cm : 0u) << (r * a.S);
            mask[f] = mk;
        }
        if constexpr (!SPLIT) clear();
        // The fragments of step j+1 are read into a second register set while step j multiplies, a few behind every
        // MFMA: a wave issues in order, so a block of reads and addresses would stand between the MFMAs of two steps.
        v4i af[2][2][FK], bf[2][2][FM];
        v2i te[NE];
        int bad[FM];                          // where the block's fragment of the current entry is
        auto read_item = [&](int t, const unsigned char *st, v4i(&ar)[2][FK], v4i(&br)[2][FM]) {
            const int h = t / (FK + FM), u = t % (FK + FM);
            if (u < FM) {
                if (!UNI || h == 0) {
                    const v2i e = te[UNI ? 0 : h];
                    bad[u] = (mask[u] & (unsigned)e[1]) ? base[u] + e[0] : a.zero_off;
                }
                br[h][u] = *reinterpret_cast<const v4i *>(__builtin_assume_aligned(smem + bad[u] + (UNI ? h * 32 : 0), 16));
            } else ar[h][u - FM] = *reinterpret_cast<const v4i *>(__builtin_assume_aligned(st + (h ? a1 : a0) + (u - FM) * 2048, 16));
        };
        auto read_table = [&](int j) {
            const v2i *e = tab + min(j, a.steps - 1) * EPS + (UNI ? 0 : half);
#pragma unroll
            for (int h = 0; h < NE; ++h) te[h] = e[2 * h];
        };
        read_table(j0);
#pragma unroll
        for (int t = 0; t < NI; ++t) read_item(t, smem + j0 * STEP, af[0], bf[0]);
        read_table(j0 + 1);
        const unsigned char *nxt = smem + (j0 + 1) * STEP;
        for (int j = j0; j < j1; j += 2) {
#pragma unroll
            for (int par = 0; par < 2; ++par) {
                if (j + par < j1) {
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        const int h = q / (FK * FM), i = q / FM % FK, f = q % FM;
                        acc[i][f] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[par][h][i], bf[par][h][f], acc[i][f], 0, 0, 0);
                        // (behind the last step this reads whatever lies after the weights; the values are never used)
#pragma unroll
                        for (int t = 0; t < NI; ++t)
                            if (t * (NQ > 2 ? NQ - 2 : 1) / NI == q) read_item(t, nxt, af[par ^ 1], bf[par ^ 1]);
                        if (q == NQ - 1) read_table(j + par + 2);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    nxt += STEP;
                }
            }
        }
        if constexpr (SPLIT) break;
        else if constexpr (SRC == RES_BLOCKED) res_store_act<FK, FM>(a, acc, k0, mw, m1, lane);
        else res_store<FK, FM>(a, acc, k0, mw, m1, n0, lane);
    }
    if constexpr (!SPLIT) return;

    // ---- the parts of a block meet in LDS (nothing there is read any more): part p adds up and stores every parts-th piece ----
    constexpr int NP = FK * FM * 4;
    res_barrier();
    v4i *const xch = reinterpret_cast<v4i *>(smem) + lane;
    const int b = wave - part * a.nblk, mw = m0 + b * FM * 32;
    if (part < a.parts)
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int i = p / (4 * FM), f = p / 4 % FM, g = p % 4;
            xch[((b * NP + p) * a.parts + part) * 64] = v4i{acc[i][f][4 * g], acc[i][f][4 * g + 1], acc[i][f][4 * g + 2], acc[i][f][4 * g + 3]};
        }
    res_barrier();
    if (part >= a.parts || mw >= m1) return;
    for (int p = part; p < NP; p += a.parts) {
        const v4i *at = xch + (b * NP + p) * a.parts * 64;
        v4i t = at[0];
        for (int d = 1; d < a.parts; ++d) t += at[d * 64];
        const int i = p / (4 * FM), f = p / 4 % FM, g = p % 4;
        const int k = k0 + i * 32 + g * 8 + 4 * half, m = mw + f * 32 + (lane & 31);
        if constexpr (SRC == RES_BLOCKED) {
            const int n = fast_div_any(m, a.PQ, a.mg_PQ), pq = m - n * a.PQ, row = fast_div_any(pq, a.Q, a.mg_Q);
            if (m < m1) act_store4(a.act, n, row, pq - row * a.Q, k, a.K, t[0], t[1], t[2], t[3]);
        } else res_store_piece(a, t, k, m, m1, n0);
    }
}

// TK, NW, FM, and how many of its workgroups fit a compute unit by their registers
#define C2I8_RES_LIST(X) \
    X(64, 8, 1, 1) \
    X(64, 4, 1, 3) \
    X(32, 4, 1, 5) \
    X(32, 4, 2, 3) \
    X(32, 8, 1, 2)

struct ResTile {
    int tk, nw, fm;
    int fit;   // workgroups whose registers fit a compute unit
};
constexpr ResTile kResTiles[] = {
#define C2I8_ROW(...) {__VA_ARGS__},
    C2I8_RES_LIST(C2I8_ROW)
#undef C2I8_ROW
};
constexpr int kNumResTiles = sizeof(kResTiles) / sizeof(kResTiles[0]);

template <int TK, int NW, int FM>
hipError_t launch_res_tile(const ResidentArgs &a, bool pixels, bool uni, int wts, bool runs, size_t lds, hipStream_t st)
{
    typedef void (*Kernel)(ResidentArgs);
    constexpr bool CAN_SPLIT = TK == 32 && FM == 1;
#define C2I8_FORMS(WTS, SPLIT, SRC, RUNS) \
    conv_resident_kernel<TK, NW, FM, SRC, WTS == RES_RAW1, WTS, SPLIT, RUNS>, conv_resident_kernel<TK, NW, FM, SRC, true, WTS, SPLIT, RUNS>
#define C2I8_SOURCES(WTS, SPLIT) C2I8_FORMS(WTS, SPLIT, RES_NCHW, false), C2I8_FORMS(WTS, SPLIT, RES_NCHW, true), C2I8_FORMS(WTS, SPLIT, RES_PIXELS, false)
    static constexpr Kernel kernels[] = {C2I8_SOURCES(RES_PACKED, false), C2I8_SOURCES(RES_RAW9, false), C2I8_SOURCES(RES_RAW1, false),
                                         C2I8_SOURCES(RES_PACKED, CAN_SPLIT), C2I8_SOURCES(RES_RAW9, CAN_SPLIT), C2I8_SOURCES(RES_RAW1, CAN_SPLIT)};
#undef C2I8_SOURCES
#undef C2I8_FORMS
    static bool raised[sizeof(kernels) / sizeof(kernels[0])];
    const int which = (((a.parts > 1) * 3 + wts) * 3 + (pixels ? 2 : runs)) * 2 + uni;
    const Kernel kern = kernels[which];
    if (lds > 64 * 1024 && !raised[which]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        raised[which] = true;
    }
    return launch(kern, dim3((unsigned)(a.tiles_k * a.tiles_m)), dim3(NW * 64), lds, st, a);
}

template <int TK, int NW, int FM>
hipError_t launch_res_blocked(const ResidentBlockedArgs &a, bool uni, size_t lds, hipStream_t st)
{
    typedef void (*Kernel)(ResidentBlockedArgs);
    constexpr bool CAN_SPLIT = TK == 32 && FM == 1;
#define C2I8_FORMS(SPLIT) \
    conv_resident_kernel<TK, NW, FM, RES_BLOCKED, false, RES_PACKED, SPLIT, false>, conv_resident_kernel<TK, NW, FM, RES_BLOCKED, true, RES_PACKED, SPLIT, false>
    static constexpr Kernel kernels[] = {C2I8_FORMS(false), C2I8_FORMS(CAN_SPLIT)};
#undef C2I8_FORMS
    static bool raised[sizeof(kernels) / sizeof(kernels[0])];
    const int which = (a.parts > 1) * 2 + uni;
    if (lds > 64 * 1024 && !raised[which]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernels[which]), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        raised[which] = true;
    }
    return launch(kernels[which], dim3((unsigned)(a.tiles_k * a.tiles_m)), dim3(NW * 64), lds, st, a);
}

struct ResidentPlan {
    ResidentBlockedArgs a;   // (what is behind its base: a blocked source's)
    int tile, wts;   // wts: ResWeights
    bool uni, runs;
    size_t lds;
};

// LDS of a workgroup: the weight tile and one step more (read behind the last step, never used), a record of zeros, the
// window and a chunk more, the depth table.
long long resident_lds(const ResTile &d, int steps, bool uni, long long slots, int pitch, int parts)
{
    const long long all = ((long long)steps + 1) * d.tk * 64 + 64 + slots * pitch + 64 + ((long long)steps * (uni ? 8 : 32) + 15) / 16 * 16;
    const long long meeting = parts > 1 ? (long long)d.nw * d.tk * d.fm * 128 : 0;   // (the parts' sums, in place of all that)
    return all > meeting ? all : meeting;
}
// Waves that share the depth of a block where a workgroup has fewer blocks than waves: from 16 steps of depth on (at 9 the
// meeting costs what the shorter chains save: 64 images 49 x 9 x 9 -> 256, stride 2: 5.4 -> 6.0 us; at 36, 3 images 256 x 14 x
// 14 -> 147: 7.4 -> 6.3).
int resident_parts(const ResTile &d, int mper, int steps)
{
    const int nblk = (mper + 32 * d.fm - 1) / (32 * d.fm);
    int parts = 1;
    if (d.tk == 32 && d.fm == 1 && steps >= 16)
        while (parts * 2 * nblk <= d.nw) parts *= 2;
    return parts;
}
constexpr long long RES_LDS_LIMIT = 160 * 1024;

// What does not depend on the tile.
struct ResidentShape {
    int C16, pitch, cb, nreal, steps;
    bool uni;
};
bool resident_shape(const ResidentProblem &r, ResidentShape *o)
{
    const GemmProblem &g = r.g;
    if (g.mode != ACT_BLOCKED || g.R * g.S > 31 || g.il_d || (g.act_out != nullptr) != (r.blocked != 0) || g.Q <= 0 || g.PQ % g.Q || g.M <= 0) return false;
    if (r.raw_weights ? g.R != g.S || (g.R == 1 ? (long long)g.K * r.C < 16 : g.R != 3) : g.cb < 16 || g.cb % 16) return false;
    // 32-bit offsets inside an image and of its pixels; 8- and 16-byte loads clamped to the tensor
    if (r.img_bytes > 0x7FFFFFFFLL || (long long)r.H * r.W > (1LL << 28) || (long long)r.N * r.img_bytes < 64) return false;
    if ((long long)g.Q * g.stride > (1LL << 28) || (long long)(g.PQ / g.Q) * g.stride > (1LL << 28)) return false;
    // (whole aligned pieces, none across two blocks; 32-bit offsets in a window's pieces)
    if (r.blocked && ((g.cb & (g.cb - 1)) || r.raw_weights || (reinterpret_cast<uintptr_t>(r.src) & 15) || (reinterpret_cast<uintptr_t>(g.act_out) & 15)))
        return false;
    o->C16 = (r.C + 15) / 16 * 16;
    o->pitch = (o->C16 / 16 | 1) * 16;
    o->cb = r.raw_weights ? o->C16 : g.cb;
    o->nreal = r.raw_weights ? g.R * g.S * o->C16 / 16 : g.Cb * g.R * g.S * (g.cb / 16);
    o->steps = r.raw_weights ? (o->nreal + 3) / 4 : g.depth / 64;
    o->uni = o->cb % 64 == 0;
    return true;
}

bool resident_plan(const ResidentProblem &r, int tile, int mper, ResidentPlan *out)
{
    const GemmProblem &g = r.g;
    const ResTile &d = kResTiles[tile];
    const int dil = g.dil > 0 ? g.dil : 1;
    ResidentShape sh;
    if (!resident_shape(r, &sh)) return false;
    const long long HW = (long long)r.H * r.W, img = r.img_bytes;
    ResidentBlockedArgs &a = out->a;
    a = ResidentBlockedArgs{};
    auto magic = [](long long v) { return v <= 1 ? 0u : magic_for(v); };
    a.out = g.out;
    a.out_nhwc = g.out_nhwc;
    a.K = g.K;
    a.M = g.M;
    a.PQ = g.PQ;
    a.Q = g.Q;
    a.mg_PQ = magic(g.PQ);
    a.mg_Q = magic(g.Q);
    a.src = r.src;
    a.wq = g.wq;
    a.C = r.C;
    a.C1 = r.C - 1;
    a.H = r.H;
    a.W = r.W;
    a.HW = (int)HW;
    a.stride = g.stride;
    a.pad = r.pad;
    a.dil = dil;
    a.R = g.R;
    a.S = g.S;
    a.depth = g.depth;
    a.steps = sh.steps;
    a.C16 = sh.C16;
    a.cb = sh.cb;
    a.nreal = sh.nreal;
    a.pitch = sh.pitch;
    a.pstride = r.pixel_bytes;
    a.img_bytes = img;
    a.src_bytes = img * r.N;
    a.cq = a.C16 / 4;
    a.mper = mper;
    a.u16 = a.C16 / 16;
    if (r.blocked) {
        auto log2_of = [](int v) {
            int l = 0;
            while ((1 << l) < v) ++l;
            return l;
        };
        a.g16_log2 = log2_of(g.cb / 16);
        a.act = ActOut{g.act_out, g.act_shift, g.act_relu, log2_of(g.o_cb), g.o_pad, (int)(g.PQ / g.Q) + 2 * g.o_pad, g.Q + 2 * g.o_pad,
                       (g.K + g.o_cb - 1) / g.o_cb};
    }
    const long long Q = g.Q, PQ = g.PQ;
    {
        const long long row = (PQ / Q - 1) * g.stride - r.pad + (g.R - 1) * dil, col = (Q - 1) * g.stride - r.pad + (g.S - 1) * dil;
        const long long end = row >= r.H ? HW : row * r.W + (col > r.W - 1 ? r.W - 1 : col < -1 ? -1 : col) + 1;
        if (end <= 0) return false;   // no pixel of the image is read at all
        a.full8 = (int)((end + 7) & ~7LL);
    }
    out->uni = sh.uni;
    // (raw 1x1 weights run the UNI kernel whatever C16 is; resident_lds still reckons with the other form's table, a few hundred bytes more)
    out->wts = !r.raw_weights ? RES_PACKED : g.R == 1 ? RES_RAW1 : RES_RAW9;
    if (!r.blocked && (mper / PQ + 2) * PQ * g.K * 4 >= (1LL << 32)) return false;   // 32-bit byte offsets from the workgroup's first image
    a.nblk = (mper + 32 * d.fm - 1) / (32 * d.fm);
    a.parts = resident_parts(d, mper, a.steps);
    a.mg_nblk = magic(a.nblk);
    a.mg_parts = magic(a.parts);
    const long long slots = window_walk(r).most(mper);
    // (what the largest window takes, on planes that take runs at all; raw weights: see the kernel's RUNS)
    out->runs = window_wide_units(HW) && (r.raw_weights || (slots < (1 << 20) && window_takes_runs((int)slots, a.cq, window_wide_units(HW), d.nw * 64)));
    const long long wts = ((long long)a.steps + 1) * d.tk * 64, lds = resident_lds(d, a.steps, sh.uni, slots, a.pitch, a.parts);
    if (lds > RES_LDS_LIMIT || (long long)((g.R - 1) * r.W + g.S - 1) * dil * a.pitch + a.C16 > (1LL << 30)) return false;
    // whole 64-byte sectors per store instruction: kept out of the caches on the way (64 images 56 x 56, 64 -> 64: 20.3 ->
    // 18.8 us; planes that start anywhere else come out up to twice as slow that way)
    a.stream_out = PQ % 16 == 0 && (reinterpret_cast<uintptr_t>(g.out) & 63) == 0;
    a.zero_off = (int)wts;
    a.win_off = (int)wts + 64;
    a.tab_off = (int)(wts + 64 + slots * a.pitch + 64);
    const long long tk = (g.K + d.tk - 1) / d.tk, tm = ((long long)g.M + mper - 1) / mper;
    if (tk * tm > 0x7FFFFFFFLL) return false;
    a.tiles_k = (int)tk;
    a.tiles_m = (int)tm;
    a.mg_tiles_k = magic(a.tiles_k);
    a.mg_cq = magic(a.cq);
    a.mg_c16q = magic(a.C16 / 4);
    a.mg_full8 = magic(a.full8);
    a.mg_g16 = magic(a.cb / 16);
    a.mg_S = magic(a.S);
    a.mg_R = magic(a.R);
    a.mg_u16 = magic(a.u16);
    out->tile = tile;
    out->lds = (size_t)lds;
    return true;
}


// Launch time in microseconds where the call brings its weights raw, turned around here or rewritten within the call: what the choice
// between stored rewrites and this kernel was fitted with, from 37900 measured launches of 4900 layers (every tile, 2 to 5 pixel counts each; a third
// of the layers held back).  A launch; per round of workgroups that fit the chip the chain of MFMAs of one wave and the
// rounds of window loads; for the busiest compute unit its MFMAs and the bytes in and out; for the whole chip all
// workgroups' bytes, which share the memory system (per: workgroups per compute unit -- without it a layer of 200 channels and
// more came out right on half a chip and 8 % low on a full one); from the second round on window and weights once more, because a
// round's loads queue behind the results that all workgroups of the round before store at its end; raw weights go through
// the registers in rounds of loads of their own, more than twice as long where the rows of 9 C bytes do not start on dwords.
// It was fitted before the wide fill, the depth parts and the raw weights' units in flight, and knows none of them.  What that means now, over 10000
// one-shot, NHWC and dilated calls: near each layer's best launch 12 % mean error on raw weights (11 % high in the median), 9 % on
// rewritten ones (6 % high), 18 % from NHWC (while results of K no multiple of four went value by value, in no term) -- but what it chooses, tile, pixels and this
// kernel or the stored path, loses 1.0 % against the best of what was measured, and 0.9 % if the chosen launch's time were known
// exactly.  Fits per tile with an error of 6 % chose worse (1.4 %: 1x1 layers, and candidates unlike the fitted ones), as did scaling this one's level (1.0 %).
__attribute__((always_inline)) inline double resident_cost_given(const ResidentProblem &r, const ResidentShape &sh, const ResTile &d, int mper, int tiles_m, int slots)
{
    const GemmProblem &g = r.g;
    const long long lds = resident_lds(d, sh.steps, sh.uni, slots, sh.pitch, 1);
    if (lds > RES_LDS_LIMIT) return 1e300;
    const long long wgs = (long long)((g.K + d.tk - 1) / d.tk) * tiles_m;
    int fit = (int)RES_LDS_LIMIT / (int)lds;              // workgroups sharing a compute unit
    if (fit > d.fit) fit = d.fit;
    const double per = wgs / 256.0;
    const double ncu = per <= (double)fit ? (double)((wgs + 255) / 256) : per + 0.4;
    const double rounds = (double)((wgs + 256 * fit - 1) / (256 * fit));
    const int blocks = (mper + 32 * d.fm - 1) / (32 * d.fm);
    const double chain = (double)((blocks + d.nw - 1) / d.nw) * d.fm * (d.tk / 32) * 2 * sh.steps;
    const double units = (double)((slots / 8 * (sh.C16 / 4) + d.nw * 256 - 1) / (d.nw * 256));
    const double mfma = d.tk / 32 * d.fm * blocks * 2.0 * sh.steps / 4, window = (double)slots * sh.C16, weights = (double)sh.steps * d.tk * 64;
    const double result = 4.0 * d.tk * mper;
    double t = 4.11 + rounds * (0.0258 * chain + 0.386 * units) + ncu * (8.14e-3 * mfma + 3.41e-5 * window + 1.43e-6 * weights + 5.66e-6 * result) +
               per * (1.41e-5 * window + 6.7e-6 * weights + (g.PQ % 16 == 0 ? 1.55e-5 : 2.47e-5) * result) +
               (rounds - 1) * (1.43e-5 * window + 8.08e-6 * weights);
    if (r.raw_weights && g.R == 3) {
        const int loads = (d.tk * (sh.C16 / 4) + d.nw * 64 - 1) / (d.nw * 64);
        t += rounds * (0.706 + (r.C % 4 ? 0.638 : 0.272) * loads);
    }
    // (raw 1x1 weights: batches of two pieces per thread.  Between 0.2 and 0.3 of a microsecond for each: at 0 the workgroups of 33 images 388 x 24 x 24
    // -> 256 fetch them twice as often as they have to, 21.7 us instead of 16.4, and 22 images 373 x 44 x 44 -> 128 stride 2 leave the stored path, 15.8 -> 16.6)
    else if (r.raw_weights) t += rounds * 0.25 * ((d.tk / 16 * sh.steps + 2 * d.nw - 1) / (2 * d.nw));
    return t;
}

// The same for kept weights, fitted per tile to 60000 measured launches of 13400 layers (two pixel counts each; a third of the
// layers held back: mean error 5 to 6 %, 8 with the formula above).  A launch; per round of workgroups that
// fit the chip its fixed part, the chain of MFMAs of one wave and the trips of window loads, in either form of the fill; for the
// busiest compute unit its MFMAs; for the whole chip the bytes of all windows, weight tiles and results (planes of whole 64-byte
// sectors, others), which share the memory system; the meeting of depth parts; from the second round on window and weights once
// more, because a round's loads queue behind the results of the round before. 
struct ResidentFit {
    double launch, round, chain, narrow, wide, mfma, window, weights, aligned, other, parts, window2, weights2;
};
constexpr ResidentFit kResFit[] = {
    {4.48, 0, 0.0237, 0, 0.379, 0.0139, 2.95e-05, 1.8e-06, 1.93e-05, 2.8e-05, 0, 7.09e-06, 1.41e-05},
    {3.64, 0.459, 0.0254, 0.47, 0.829, 0.00978, 1.94e-05, 4.04e-06, 2.46e-05, 3.65e-05, 0, 0, 1.05e-05},
    {3.42, 0.26, 0.0364, 0.682, 1.02, 0.0118, 1.3e-05, 9.74e-06, 2.79e-05, 4.16e-05, 0.78, 0, 8.3e-06},
    {4.39, 0, 0.0268, 0.299, 0.8, 0.0111, 1.77e-05, 5.95e-06, 2.72e-05, 3.91e-05, 0, 9.25e-06, 1.52e-05},
    {3.26, 0.891, 0.0197, 0.502, 0.756, 0.021, 1.9e-05, 9.3e-06, 1.82e-05, 3.14e-05, 0.699, 0, 7.95e-06},
};
__attribute__((always_inline)) inline double resident_cost(const ResidentProblem &r, const ResidentShape &sh, const ResTile &d, const ResidentFit &f, int mper, int tiles_m, int slots)
{
    const GemmProblem &g = r.g;
    const int parts = resident_parts(d, mper, sh.steps);
    const long long lds = resident_lds(d, sh.steps, sh.uni, slots, sh.pitch, parts);
    if (lds > RES_LDS_LIMIT) return 1e300;
    const long long wgs = (long long)((g.K + d.tk - 1) / d.tk) * tiles_m;
    int fit = (int)RES_LDS_LIMIT / (int)lds;              // workgroups sharing a compute unit
    if (fit > d.fit) fit = d.fit;
    const double per = wgs / 256.0;
    const double ncu = per <= (double)fit ? (double)((wgs + 255) / 256) : per + 0.4;
    const double rounds = (double)((wgs + 256 * fit - 1) / (256 * fit));
    const int blocks = (mper + 32 * d.fm - 1) / (32 * d.fm), runs = (slots + 63) / 64;
    const double chain = (double)((blocks + d.nw - 1) / d.nw) * d.fm * (d.tk / 32) * 2 * sh.steps / parts;
    const bool wide = (slots >= 128 || slots * 5 >= runs * 256) && runs * sh.C16 >= d.nw * 64;   // (window_from_nchw)
    const double trips = wide ? (double)((runs * sh.C16 + d.nw * 128 - 1) / (d.nw * 128)) : (double)((slots / 8 * (sh.C16 / 4) + d.nw * 256 - 1) / (d.nw * 256));
    const double mfma = d.tk / 32 * d.fm * blocks * 2.0 * sh.steps / 4, window = (double)slots * sh.C16, weights = (double)sh.steps * d.tk * 64;
    const double result = 4.0 * d.tk * mper;
    return f.launch + rounds * (f.round + f.chain * chain + (wide ? f.wide : f.narrow) * trips + (parts > 1 ? f.parts : 0)) + f.mfma * ncu * mfma +
           per * (f.window * window + f.weights * weights + (g.PQ % 16 == 0 ? f.aligned : f.other) * result) +
           (rounds - 1) * (f.window2 * window + f.weights2 * weights);
}

// From blocked images into the next layer's: the same kind of fit, to two thirds of 70000 launches of 2540 layers (mean error on the rest 7.5 to 9 % per
// tile).  Trips of 16-byte pieces; result bytes are a quarter; in the 64-channel tile of 8 waves the rounds of weight transfers, which nothing hides there.
struct ResidentActFit {
    double launch, round, chain, trips, mfma, window, weights, result, parts, window2, weights2, transfers;
};
constexpr ResidentActFit kResActFit[] = {
    {3.48, 0, 0.0158, 0.727, 0.0152, 7.69e-06, 0, 4.8e-05, 0, 2.82e-06, 9.05e-06, 0.274},
    {3.38, 0.32, 0.0252, 0.778, 0.0103, 0, 4.23e-06, 7.76e-05, 0, 3.69e-06, 9.73e-06, 0},
    {3.12, 0.516, 0.039, 0.763, 0.0124, 2.15e-06, 1.06e-05, 0.000111, 0.654, 0, 0, 0},
    {3.88, 0.213, 0.0239, 0.712, 0.0156, 4.36e-06, 8.02e-06, 9.71e-05, 0, 9.31e-06, 8.89e-06, 0},
    {3.25, 0.572, 0.0128, 0.764, 0.0239, 6.22e-06, 8.33e-06, 7.93e-05, 0.84, 4.51e-06, 2.72e-06, 0},
};
inline double resident_cost_act(const ResidentProblem &r, const ResidentShape &sh, const ResTile &d, const ResidentActFit &f, int mper, int tiles_m, int slots)
{
    const int parts = resident_parts(d, mper, sh.steps);
    const long long lds = resident_lds(d, sh.steps, sh.uni, slots, sh.pitch, parts);
    if (lds > RES_LDS_LIMIT) return 1e300;
    const long long wgs = (long long)((r.g.K + d.tk - 1) / d.tk) * tiles_m;
    int fit = (int)RES_LDS_LIMIT / (int)lds;
    if (fit > d.fit) fit = d.fit;
    const double per = wgs / 256.0;
    const double ncu = per <= (double)fit ? (double)((wgs + 255) / 256) : per + 0.4;
    const double rounds = (double)((wgs + 256 * fit - 1) / (256 * fit));
    const int blocks = (mper + 32 * d.fm - 1) / (32 * d.fm);
    const double chain = (double)((blocks + d.nw - 1) / d.nw) * d.fm * (d.tk / 32) * 2 * sh.steps / parts;
    const double trips = (double)((slots * (sh.C16 / 16) + d.nw * 256 - 1) / (d.nw * 256));
    const double mfma = d.tk / 32 * d.fm * blocks * 2.0 * sh.steps / 4, window = (double)slots * sh.C16, weights = (double)sh.steps * d.tk * 64;
    const double transfers = (double)((sh.steps * d.tk * 64 + d.nw * 8192 - 1) / (d.nw * 8192));
    return f.launch + rounds * (f.round + f.chain * chain + f.trips * trips + f.transfers * transfers + (parts > 1 ? f.parts : 0)) + f.mfma * ncu * mfma +
           per * (f.window * window + f.weights * weights + f.result * d.tk * mper) + (rounds - 1) * (f.window2 * window + f.weights2 * weights);
}

// With the choice: one layer on the same depth order may come with kept weights and with raw ones, whose estimates differ.
struct ResidentKey {
    GemmKey g;
    int v[12];
};
ResidentKey resident_key(const ResidentProblem &r, const ResidentChoice &c)
{
    const int out64 = (reinterpret_cast<uintptr_t>(r.g.out) & 63) == 0;
    return ResidentKey{gemm_key(r.g), {r.N, r.C, r.H, r.W, r.pad, r.pixel_major, r.pixel_bytes, r.raw_weights, r.blocked, out64, c.tile, c.mper}};
}

}  // namespace

bool resident_pick(const ResidentProblem &r, WindowWalk &walk, ResidentChoice *c)
{
    ResidentShape sh;
    if (!resident_shape(r, &sh)) return false;
    struct Cand {
        double cost;
        int tile, mper;
    } best[3] = {{1e300, 0, 0}, {1e300, 0, 0}, {1e300, 0, 0}};
    static const int sizes[] = {32, 64, 128, 192, 256, 384, 512, 768};
    int slots_of[12], mpers[12], n = 0;
    auto add = [&](long long mper) {
        if (mper < 32 || mper > 1024 || (mper >= (long long)r.g.M + 32 && mper > 32)) return;
        for (int i = 0; i < n; ++i)
            if (mpers[i] == (int)mper) return;
        mpers[n] = (int)mper;
        slots_of[n++] = walk.sampled((int)mper);
    };
    for (int w = 1; w <= 4; ++w) add((((long long)r.g.M + 256 * w - 1) / (256 * w) + 31) / 32 * 32);
    for (int m : sizes) add(m);
    int tiles_m[12];
    for (int i = 0; i < n; ++i) tiles_m[i] = (int)(((long long)r.g.M + mpers[i] - 1) / mpers[i]);
    // Kept weights: the middle of the two estimates, a twelfth lower (the first one's level is too high).  Their errors differ: of 700 drawn 3x3 and 5x5
    // layers 17 % were more than 2 % slower with the second one alone than with the first, 7 % with both, 0.987 of the time in the mean.  Kernels
    // of fewer taps than the second one was fitted on: the first alone (260 1x1 layers 0.956 in the mean; with the second up to 1.6 of it).
    const bool both = r.kept && !r.blocked && r.g.R * r.g.S >= 9;
    auto consider = [&](const ResTile &d, int t) __attribute__((always_inline)) {   // (a tile known to the compiler: its divisions are shifts)
        for (int i = 0; i < n; ++i) {
            Cand x{r.blocked ? resident_cost_act(r, sh, d, kResActFit[t], mpers[i], tiles_m[i], slots_of[i])
                             : resident_cost_given(r, sh, d, mpers[i], tiles_m[i], slots_of[i]), t, mpers[i]};
            if (both) x.cost = 0.46 * (x.cost + resident_cost(r, sh, d, kResFit[t], mpers[i], tiles_m[i], slots_of[i]));
            for (int k = 0; k < 3; ++k)
                if (x.cost < best[k].cost) {
                    for (int j = 2; j > k; --j) best[j] = best[j - 1];
                    best[k] = x;
                    break;
                }
        }
    };
    int index = 0;
#define C2I8_CASE(tk, nw, fm, fit) consider(ResTile{tk, nw, fm, fit}, index++);
    C2I8_RES_LIST(C2I8_CASE)
#undef C2I8_CASE
    for (const Cand &x : best) {   // (the window was sampled: the plan knows whether it fits)
        ResidentPlan p;
        if (x.cost < 1e300 && resident_plan(r, x.tile, x.mper, &p)) {
            *c = ResidentChoice{x.tile, x.mper, x.cost};
            return true;
        }
    }
    return false;
}

static hipError_t launch_plan(const ResidentProblem &r, const ResidentPlan &p, hipStream_t st)
{
    ResidentBlockedArgs a = p.a;
    a.src = r.src;
    a.wq = r.g.wq;
    a.out = r.g.out;
    a.act.out = r.g.act_out;
    int index = 0;
#define C2I8_CASE(tk, nw, fm, fit) \
    if (p.tile == index++) \
        return r.blocked ? launch_res_blocked<tk, nw, fm>(a, p.uni, p.lds, st) : launch_res_tile<tk, nw, fm>(a, r.pixel_major, p.uni, p.wts, p.runs, p.lds, st);
    C2I8_RES_LIST(C2I8_CASE)
#undef C2I8_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_resident(const ResidentProblem &r, const ResidentChoice &c, hipStream_t st)
{
    static thread_local PlanTable<ResidentKey, ResidentPlan, 64> plans;
    const ResidentPlan *kept = plans.get(resident_key(r, c), [&](ResidentPlan *p) { return resident_plan(r, c.tile, c.mper, p); });
    return kept ? launch_plan(r, *kept, st) : hipErrorInvalidValue;
}

int resident_num_tiles() { return kNumResTiles; }
TileInfo resident_tile_info(int tile) { return TileInfo{kResTiles[tile].tk, kResTiles[tile].fm * 32, kResTiles[tile].nw * 64, 0}; }

bool resident_applies(const ResidentProblem &r, int tile, int mper)
{
    ResidentPlan p;
    return resident_plan(r, tile, mper, &p);
}

hipError_t launch_resident_forced(const ResidentProblem &r, int tile, int mper, hipStream_t st)
{
    ResidentPlan p;   // (not kept: the table holds the library's own choices)
    return resident_plan(r, tile, mper, &p) ? launch_plan(r, p, st) : hipErrorInvalidValue;
}

}  // namespace c2i8
