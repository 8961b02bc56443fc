// Stencil unrolling in the GEMM stage for layers with a large result: tiles of consecutive pixels of the flattened output image.
// Same operands, depth order and result as the window kernel (window_mfma.hip): depth index (c*R + r)*S4 + s with
// S4 = ceil(S, 4), a kernel row padded to whole dwords.
//
// What bounds it is how memory takes the result.  Stores alone, no convolution around them, 334 MB as 128 images x 64 planes of
// 10200 pixels: workgroups of 128 pixels, two or three per compute unit, 5.2 TB/s; eight per compute unit 4.6; 512 pixels 4.0; workgroups
// that stay and take one tile after another 3.5, whatever the tile.  A plane that does not begin on a cache line shares the lines at a
// tile's ends with the neighbouring tiles, and a line that leaves the XCD's 4 MB L2 before its other half has come costs a second,
// partial write: what the workgroups of an XCD have written since must be less than the L2.  Planes of whole lines (112 x 112) take
// 5.7 to 6 TB/s from every tile up to 1024 pixels.  Results within the last-level cache do not depend on it.
//
//   * A tile is `mper` consecutive pixels of an image whatever the output's width: the window kernel's tiles of 32, 64 or 128 columns of
//     a row leave up to half their MFMA lanes outside (68 of 128 columns: 185 images 3 x 190 x 136, 5 x 5 / 2 -> 64, 100 -> 81 us).
//   * A window row is a margin of zeros, the image row, zeros; image rows come in 16-byte pieces, a thread per column of pieces, and one
//     thread per row makes what is left over.
//   * A lane's pixel moves on by a constant number of pixels from block to block: additions and one comparison, no division.
#include "kernels.h"
#include "launch.h"
#include "rewrite_bodies.h"

#include <algorithm>

namespace c2i8 {

namespace {

typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int STENCIL_THREADS = 256;
constexpr long long STENCIL_WINDOW = 40 * 1024;   // bytes of LDS a window may take

struct StencilArgs {
    const int8_t *in;
    const int8_t *wt;
    int32_t *out;
    int C, H, W, K, PQ, Q, R, stride, pad;
    int mper, tiles;           // pixels of a tile; tiles per image
    int RW, pitch, margin;     // window rows per channel; bytes per window row; zeros before an image row (a multiple of 16)
    int whole, full, rpp;      // whole 16-byte pieces of an image row (full: at least 1); window rows per pass of the threads (0: none whole)
    int step_byte, step_col, wrap_byte;   // from a lane's pixel to its next: window bytes and columns; more bytes where it wraps
    int win_bytes;             // one window buffer
    int CR, nd;                // C*R; dwords per kernel row
    int w_S, w_row, w_pitch;   // weight operand: bytes per kernel row and per channel; bytes per channel in LDS
    int wt16;                  // rewritten rows of the padded depth at a 16-byte aligned address
    long long in_bytes;
    unsigned m_Q, m_tiles, m_full, m_RW, m_nd, m_R;
};

__device__ __forceinline__ unsigned load_u32(const void *p)  // any alignment
{
    unsigned x;
    __builtin_memcpy(&x, p, 4);
    return x;
}

// Four waves, each 32 pixels x 32 * NKB channels at a time, 32 * NKK bytes of depth
template <int NKK, int NKB>
__global__ void __launch_bounds__(STENCIL_THREADS, NKK * NKB > 12 ? 3 : 4) conv_stencil_kernel(const StencilArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int ND = NKK * 8, KB = 32 * NKB, NT = STENCIL_THREADS;
    unsigned char *win = smem, *wl = smem + a.win_bytes;
    int *tab = reinterpret_cast<int *>(wl + KB * a.w_pitch);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l31 = lane & 31, half = lane >> 5;
    const int k0 = blockIdx.y * KB;
    const int t = xcd_contiguous(blockIdx.x, gridDim.x);
    const int n = fast_div_any(t, a.tiles, a.m_tiles), m0 = (t - n * a.tiles) * a.mper;
    const int cnt = min(a.mper, a.PQ - m0);
    const int p_first = fast_div_any(m0, a.Q, a.m_Q);

    // Every global load first, nothing that needs their data in between: one memory round trip for both operands.
    // weight rows k0 .. k0+KB-1 (those below K) in the padded depth order
    const int rows = min(KB, a.K - k0);
    const int8_t *wsrc = a.wt + (size_t)k0 * a.w_row;
    constexpr int PPR = ND / 4, WP16 = (KB * PPR + NT - 1) / NT;
    constexpr int RPP = NT / ND, WMAX = (KB + RPP - 1) / RPP;
    const int last = rows * a.w_row - 4;   // offset of the last whole dword of these rows
    const int r0 = tid / ND, d = tid - r0 * ND;
    const int wcr = fast_div(d, a.m_nd), ws0 = 4 * (d - wcr * a.nd);
    const int left = a.w_S - ws0;
    const bool real = wcr < a.CR && left > 0;
    const unsigned mask = !real ? 0u : left >= 4 ? 0xFFFFFFFFu : (1u << (8 * (left & 3))) - 1u;
    const int coff = wcr * a.w_S + ws0;
    v4i wp16[WP16];
    unsigned wv[WMAX];
    if (a.wt16) {
#pragma unroll
        for (int u = 0; u < WP16; ++u) wp16[u] = *reinterpret_cast<const v4i *>(wsrc + 16 * (unsigned)min(tid + u * NT, rows * PPR - 1));
    } else if (r0 < RPP && last >= 0) {
#pragma unroll
        for (int u = 0; u < WMAX; ++u) {
            const int off = real ? min(r0 + u * RPP, rows - 1) * a.w_row + coff : 0;
            wv[u] = load_u32(wsrc + (unsigned)min(off, last));   // a dword that would run past the rows is fetched lower
        }
    }
    // Window rows: a margin of zeros, the image row, zeros.  The whole 16-byte pieces of the rows: a thread keeps its column and walks
    // down the rows.  Then a thread per row for what is left: the row's last bytes and the zeros.
    {
        const int h_lo = p_first * a.stride - a.pad, rows_all = a.C * a.RW;
        const long long img = (long long)n * a.C * a.H * a.W;
        const int8_t *src = a.in + img;
        constexpr int NP = 4;
        const int wr = fast_div(tid, a.m_full), wj = tid - wr * a.full;   // (full >= 1; none whole: rpp = 0)
        auto row_off = [&](int row, bool *outside) {
            const int c = fast_div(row, a.m_RW), h = h_lo + row - c * a.RW, hc = min(max(h, 0), a.H - 1);
            *outside = h != hc;
            return (unsigned)((c * a.H + hc) * a.W);   // an image is below 2^31 bytes (host check)
        };
        v4i x[NP], tail{0, 0, 0, 0};
        bool out[NP], tail_out = false;
        int over = 0;
        auto load = [&](int base) {
#pragma unroll
            for (int u = 0; u < NP; ++u) {
                const unsigned off = row_off(min(base + wr + u * a.rpp, rows_all - 1), &out[u]) + 16 * wj;
                __builtin_memcpy(&x[u], src + off, 16);
            }
        };
        auto store = [&](int base) {
#pragma unroll
            for (int u = 0; u < NP; ++u) {
                const int row = base + wr + u * a.rpp;
                if (wr < a.rpp && row < rows_all)
                    *reinterpret_cast<v4i *>(win + row * a.pitch + a.margin + 16 * wj) = out[u] ? v4i{0, 0, 0, 0} : x[u];
            }
        };
        auto load_tail = [&](int row) {
            // (a piece that would run past the tensor's end is fetched lower, from a tensor of 16 bytes and more)
            const long long room = a.in_bytes - img - 16, off = row_off(min(row, rows_all - 1), &tail_out) + (unsigned)min(16 * a.whole, a.W - 1);
            over = room < off ? (int)(off - room) : 0;
            __builtin_memcpy(&tail, src + (off - over), 16);
        };
        auto store_tail = [&](int row) {
            if (row >= rows_all) return;
            unsigned char *to = win + row * a.pitch;
            for (int z = 0; z < a.margin; z += 16) *reinterpret_cast<v4i *>(to + z) = v4i{0, 0, 0, 0};
            unsigned __int128 v;
            __builtin_memcpy(&v, &tail, 16);
            v >>= 8 * over;
            const int left = tail_out ? 0 : a.W - 16 * a.whole;   // 0 .. 15
            v &= ((unsigned __int128)1 << (8 * left)) - 1;
            __builtin_memcpy(&tail, &v, 16);
            for (int z = a.margin + 16 * a.whole; z < a.pitch; z += 16) {
                *reinterpret_cast<v4i *>(to + z) = tail;
                tail = v4i{0, 0, 0, 0};
            }
        };
        if (a.rpp) load(0);
        load_tail(tid);
        if (a.rpp) store(0);
        store_tail(tid);
        // (the usual window in straight-line code: a loop header would wait for the weights)
        if (rows_all > NT)
            for (int row = tid + NT; row < rows_all; row += NT) {
                load_tail(row);
                store_tail(row);
            }
        if (a.rpp && rows_all > NP * a.rpp)
            for (int base = NP * a.rpp; base < rows_all; base += NP * a.rpp) {
                load(base);
                store(base);
            }
    }
    if (a.wt16) {
#pragma unroll
        for (int u = 0; u < WP16; ++u) {
            const int i = tid + u * NT, row = i / PPR, col = i - row * PPR;
            if (i < rows * PPR) *reinterpret_cast<v4i *>(wl + row * a.w_pitch + col * 16) = wp16[u];
        }
    } else if (r0 < RPP) {
        if (last >= 0) {
#pragma unroll
            for (int u = 0; u < WMAX; ++u) {
                const int row = r0 + u * RPP;
                if (row < rows)
                    *reinterpret_cast<unsigned *>(wl + row * a.w_pitch + 4 * d) = (wv[u] >> (8 * (unsigned)max(row * a.w_row + coff - last, 0))) & mask;
            }
        } else {   // fewer than four weight bytes in all
            for (int row = r0; row < rows; row += RPP) {
                unsigned x = 0;
                const int off = row * a.w_row + coff;
                if (real)
                    for (int b = 0; off + b < rows * a.w_row; ++b) x |= (unsigned)(unsigned char)wsrc[off + b] << (8 * b);
                *reinterpret_cast<unsigned *>(wl + row * a.w_pitch + 4 * d) = x & mask;
            }
        }
    }
    // where depth dword d starts in the window, relative to a pixel's first byte
    if (tid < ND) {
        const int cr = fast_div(tid, a.m_nd), s0 = 4 * (tid - cr * a.nd);
        const int c = fast_div(cr, a.m_R), r = cr - c * a.R;
        tab[tid] = cr < a.CR ? (c * a.RW + r) * a.pitch + s0 : 0;
    }
    __syncthreads();

    constexpr bool WREG = NKK * NKB <= 8, TREG = NKK * NKB <= 12;   // weights, table in registers
    v4i wf[NKK][NKB], ta[NKK];
    const unsigned char *wbase = wl + l31 * a.w_pitch + half * 16;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
        if (TREG) ta[kk] = *reinterpret_cast<const v4i *>(tab + kk * 8 + half * 4);
        if (WREG)
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) wf[kk][kb] = *reinterpret_cast<const v4i *>(wbase + kb * 32 * a.w_pitch + kk * 32);
    }
    const bool full = k0 + KB <= a.K;
    const unsigned PQ4 = 4u * (unsigned)a.PQ;
    char *ob = reinterpret_cast<char *>(a.out + ((size_t)n * a.K + k0) * a.PQ);
    // the lane's pixels: the first by division, the following ones a constant number of pixels on
    const int m_first = m0 + wave * 32 + l31, pl = fast_div_any(m_first, a.Q, a.m_Q);
    int col = m_first - pl * a.Q;
    int byte = (pl - p_first) * a.stride * a.pitch + a.margin - a.pad + col * a.stride;
    const int p_last = fast_div_any(m0 + cnt - 1, a.Q, a.m_Q);
    const int byte_max = (p_last - p_first) * a.stride * a.pitch + a.margin - a.pad + (a.Q - 1) * a.stride;
    for (int b0 = wave * 32; b0 < cnt; b0 += NT / 2) {
        const int bt = min(byte, byte_max);   // (a lane past the tile reads within the window)
        const unsigned ash = (unsigned)bt & 3u;   // (window rows are a multiple of 16 apart)
        const unsigned char *a4 = win + (bt & ~3);
        byte += a.step_byte;
        col += a.step_col;
        if (col >= a.Q) {
            col -= a.Q;
            byte += a.wrap_byte;
        }
        v16i acc[NKB];
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[kb][v] = 0;
        unsigned plo[2][4], phi[2][4];
        auto fetch_pairs = [&](int kk) {
            const v4i t4 = TREG ? ta[kk] : *reinterpret_cast<const v4i *>(tab + kk * 8 + half * 4);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned *pp = reinterpret_cast<const unsigned *>(a4 + t4[i]);
                plo[kk & 1][i] = pp[0];
                phi[kk & 1][i] = pp[1];
            }
        };
        fetch_pairs(0);
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) {
            if (kk + 1 < NKK) fetch_pairs(kk + 1);
            v4i af;
#pragma unroll
            for (int i = 0; i < 4; ++i) af[i] = (int)__builtin_amdgcn_alignbyte(phi[kk & 1][i], plo[kk & 1][i], ash);
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
                acc[kb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(
                    WREG ? wf[kk][kb] : *reinterpret_cast<const v4i *>(wbase + kb * 32 * a.w_pitch + kk * 32), af, acc[kb], 0, 0, 0);
        }
        // column = lane%32 = pixel, row = 8*(v/4) + 4*(lane/32) + v%4 = channel: 128-byte runs
        const unsigned o = (unsigned)(4 * half) * PQ4 + 4u * (unsigned)(m0 + b0 + l31);
        auto put = [&](int kb, int g, int v) {
            *reinterpret_cast<int32_t *>(ob + (size_t)(kb * 32 + 8 * g + v) * PQ4 + o) = acc[kb][4 * g + v];
        };
        if (full && b0 + 32 <= cnt) {
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int v = 0; v < 4; ++v) put(kb, g, v);
        } else if (b0 + l31 < cnt) {
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int kg = k0 + kb * 32 + 8 * g;
                    if (kg + 8 <= a.K) {   // (wave-uniform: groups of eight channels)
#pragma unroll
                        for (int v = 0; v < 4; ++v) put(kb, g, v);
                    } else if (kg < a.K) {
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (kg + 4 * half + v < a.K) put(kb, g, v);
                    }
                }
        }
    }
}

}  // namespace

// Pixels of a tile, 0 where the window kernel stays; `few`: three workgroups per compute unit at most.  From 190 stem, speech and small 3 x 3
// layers, each timed with tiles of 128 to 1024 pixels on three sets of buffers in turn, and from another 900 with results of 30 to 560 MB, this
// kernel and the window kernel on two sets, the best of three processes (figures: of the window kernel's time).
//   Results past the last-level cache (240 MB here: less than its 256 MB is free for a result that is written again).  Planes of whole lines:
//   512 pixels, up to 16 channels 1024 (4 - 16 channels, 320 MB: 0.82 of 512's time).  Others, from 190 MB on: what the workgroups of an XCD hold
//   written in parts must be less than its L2.  Where one writes 36 KB and more, three per compute unit (128 images 5 x 5 / 2 -> 32, 326 MB:
//   0.64, and 0.72 with as many as fit), 512 pixels, 256 above 32 channels (512: up to 1.2 of that).  Of less as many as fit, with 1024
//   pixels up to 8 channels: three were up to 1.95 (15352 images 3 x 62 x 62, 3 x 3 -> 2: 725 us, the window kernel 371, as many as fit 352).
//   (240 layers of 190 to 245 MB and more than 32 channels: 0.965 of the time of 512 pixels and as many as fit.)  1024 pixels whose window is too
//   large: 512 (2087 images 8 x 91 x 260, 3 x 3 / 2 -> 6, 300 MB: 177 us, the window kernel 535).
//   Smaller results, up to 32 channels: the most pixels of 256, 512, 1024 that leave 640 workgroups: the window's rows overlap and the weights come in
//   once per tile (112 images 20 x 5 / 2 -> 32, 140 MB: 256 pixels 0.89, 512 0.70, 1024 0.64).  Below 160 000 pixels, 240 000 for depths up to 128,
//   the window kernel's many small workgroups win (1.0 - 1.2), and so they do up to 125 MB for a depth of 64 and 25 - 32 channels (1.0 - 1.1).
//   Smaller results, more channels: from 120 MB on (0.65 - 0.95; 3 x 3 kernels in one depth of 64 from 200 MB, 1.0 - 1.2 below), deep stems from 36 MB
//   (0.61 - 1.0).  Many channels on narrow images make windows of many short rows: the window kernel's (up to 1.3).
//   And where the window kernel's blocks of 32 pixels suit the rows (stencil_pays).  906 layers drawn once that was settled, three inputs and two
//   results in turn, mean and worst, results from 190 MB on: up to 32 channels 0.75 and 1.17 on planes of partial lines, 0.72 and 1.03 on others; above
//   0.90 and 1.16, 0.84 and 1.03.  Smaller ones: 0.86 and 1.08, 0.90 and 1.05; above 32 channels 0.96 and 1.17, 0.96 and 1.05.
static bool stencil_pays(const WindowProblem &g, int depth, double out, bool lines)
{
    // how full its tiles of 128 pixels are
    const int QT = g.Q > 64 ? 128 : g.Q > 32 ? 64 : 32, PT = 128 / QT;
    const long long tiles = (long long)((g.Q + QT - 1) / QT) * ((g.P + PT - 1) / PT);
    const double fill = (double)g.P * g.Q / (128.0 * tiles);
    if (lines) {
        // its blocks are whole lines as well, and few channels' depth of 64 is multiplied in no time: 1.0 - 1.36, else 0.38 - 1.06
        return g.Q % 32 != 0 || g.K <= 8 || out < 150e6 || fill <= 0.65 || (g.K <= 16 && depth >= 128 && fill < 0.95);
    }
    if (g.K <= 32) return true;
    if (tiles == 1) return false;   // (an image to a workgroup on both sides: 0.8 - 1.5)
    if (out < 45e6) return fill <= 0.70;   // (deep stems of 36 MB and more: 0.85 - 0.91; better filled 0.91 - 1.17, 1.04 in the mean)
    // more than 64 channels: 0.57 - 1.23 and 0.98 in the mean, better filled 0.95 - 1.38 and 1.08
    return out < 190e6 || g.K <= 64 || fill < 0.80;
}

static int stencil_tile(const WindowProblem &g, int depth, bool *few)
{
    const double out = 4.0 * g.N * g.K * g.P * g.Q;
    const long long pixels = (long long)g.N * g.P * g.Q;
    const bool lines = (long long)g.P * g.Q % 32 == 0 && (reinterpret_cast<uintptr_t>(g.out) & 127) == 0;
    *few = false;
    if (g.C > 4 && g.K > 32 && g.stride > 1 && g.W <= 64) return 0;
    if (!stencil_pays(g, depth, out, lines)) return 0;
    const int partial = g.K <= 8 ? 1024 : g.K <= 32 ? 512 : 256;
    const double written = 4.0 * std::min<long long>(partial, (long long)g.P * g.Q) * std::min(g.K, 64);   // by a workgroup
    if (out >= (lines || g.K <= 32 ? 240e6 : 190e6)) {
        if (lines) return g.K <= 16 ? 1024 : 512;
        *few = written >= 36e3;
        return partial;
    }
    if (out < 120e6 ? g.C > 4 : g.C > 4 && g.W < 56) return 0;
    if (g.K > 32) return out >= (depth == 64 && g.R == 3 ? 200e6 : depth >= 128 && g.C <= 4 && g.W >= 56 ? 36e6 : 120e6) ? 512 : 0;
    if (depth == 64 && g.K > 24 && out < 125e6) return 0;
    if (out >= 190e6 && !lines) {
        *few = written >= 36e3;
        return partial;
    }
    if (pixels < (depth <= 128 ? 240000 : 160000)) return 0;
    return pixels >= 640 * 1024 ? 1024 : pixels >= 640 * 512 ? 512 : 256;
}

static bool stencil_plan(const WindowProblem &g, StencilArgs *out, dim3 *grid, size_t *lds)
{
    if (g.nhwc || g.act.out) return false;
    const int depth = window_depth(g.C, g.R, g.S);
    const long long PQ = (long long)g.P * g.Q;
    // (32-bit offsets within an image and within 128 planes; a piece fetched lower at the tensor's end needs 16 bytes)
    if (depth == 0 || (long long)g.C * g.H * g.W > 0x7FFFFFFFLL || (long long)g.N * g.C * g.H * g.W < 16 || PQ >= (1 << 23)) return false;
    bool few;
    const int target = stencil_tile(g, depth, &few);
    if (target == 0) return false;
    StencilArgs a{};
    a.in = g.in; a.wt = g.wt; a.out = g.out;
    a.C = g.C; a.H = g.H; a.W = g.W; a.K = g.K; a.PQ = (int)PQ; a.Q = g.Q; a.R = g.R; a.stride = g.stride; a.pad = g.pad;
    a.whole = g.W / 16;
    a.full = std::max(1, a.whole);
    if (a.full > STENCIL_THREADS) return false;
    a.rpp = a.whole ? STENCIL_THREADS / a.full : 0;
    const int S4 = (g.S + 3) / 4 * 4;
    const long long margin = ((long long)g.pad + 15) / 16 * 16;
    // a row holds the whole image row and what the last pixel's last dword pair reaches
    const long long reach = margin - g.pad + (long long)(g.Q - 1) * g.stride + S4 + 4;
    const long long pitch = (std::max(margin + ((long long)g.W + 15) / 16 * 16, reach) + 15) / 16 * 16;
    // the image's blocks of 32 pixels spread evenly over its tiles; 512 pixels where the window of 1024 is too large
    const int blocks = (int)((PQ + 31) / 32);
    long long RW, win;
    for (int pixels = target;; pixels = 512) {
        a.tiles = (blocks + pixels / 32 - 1) / (pixels / 32);
        a.mper = (blocks + a.tiles - 1) / a.tiles * 32;
        const long long rows_out = a.tiles == 1 ? g.P : std::min<long long>((a.mper + g.Q - 2) / g.Q + 1, g.P);   // that consecutive pixels touch at most
        RW = (rows_out - 1) * g.stride + g.R, win = g.C * RW * pitch;
        if (win <= STENCIL_WINDOW || pixels <= 512) break;
    }
    if (pitch > STENCIL_WINDOW || RW > STENCIL_WINDOW || win > STENCIL_WINDOW || (long long)g.N * a.tiles > 0x7FFFFFFFLL || (g.K + 63) / 64 > 65535) return false;
    a.RW = (int)RW;
    a.pitch = (int)pitch;
    a.margin = (int)margin;
    a.win_bytes = (int)win;
    constexpr int STEP = STENCIL_THREADS / 2;   // pixels from a lane's block to its next
    if ((long long)(STEP / g.Q + 1) * g.stride * pitch > (1 << 24)) return false;   // (a lane past its tile keeps counting)
    a.step_col = STEP % g.Q;
    a.step_byte = STEP / g.Q * g.stride * a.pitch + a.step_col * g.stride;
    a.wrap_byte = g.stride * a.pitch - g.Q * g.stride;
    a.CR = g.C * g.R;
    a.nd = S4 / 4;
    a.w_S = g.wt_rewritten ? S4 : g.S;
    a.w_row = g.wt_rewritten ? depth : g.C * g.R * g.S;
    a.w_pitch = depth + 16;
    a.wt16 = g.wt_rewritten && (reinterpret_cast<uintptr_t>(g.wt) & 15) == 0;
    a.in_bytes = (long long)g.N * g.C * g.H * g.W;
    a.m_Q = magic_for(g.Q);
    a.m_tiles = magic_for(a.tiles);
    a.m_full = magic_for(a.full);
    a.m_RW = magic_for(a.RW);
    a.m_nd = magic_for(a.nd);
    a.m_R = magic_for(g.R);
    const int kb = g.K > 32 ? 64 : 32;
    *lds = (size_t)a.win_bytes + (size_t)kb * a.w_pitch + depth;
    if (few) *lds = std::max(*lds, (size_t)(160 * 1024 / 4 + 1024));   // a fourth workgroup does not fit
    *grid = dim3((unsigned)(g.N * a.tiles), (unsigned)((g.K + kb - 1) / kb));
    *out = a;
    return true;
}

template <int NKK>
static hipError_t launch_stencil_nkk(const StencilArgs &a, dim3 grid, size_t lds, hipStream_t st)
{
    return a.K > 32 ? launch((conv_stencil_kernel<NKK, 2>), grid, dim3(STENCIL_THREADS), lds, st, a)
                    : launch((conv_stencil_kernel<NKK, 1>), grid, dim3(STENCIL_THREADS), lds, st, a);
}

bool launch_stencil_conv(const WindowProblem &g, hipStream_t st, hipError_t *e)
{
    StencilArgs a;
    dim3 grid;
    size_t lds;
    if (!stencil_plan(g, &a, &grid, &lds)) return false;
    switch ((a.w_pitch - 16) / 32) {
        case 2: *e = launch_stencil_nkk<2>(a, grid, lds, st); return true;
        case 4: *e = launch_stencil_nkk<4>(a, grid, lds, st); return true;
        case 6: *e = launch_stencil_nkk<6>(a, grid, lds, st); return true;
        case 8: *e = launch_stencil_nkk<8>(a, grid, lds, st); return true;
    }
    return false;
}

}  // namespace c2i8
