// GEMM stage for large layers: the input window of a tile lies in LDS and the weights go from the L2s straight into the registers of the wave
// that multiplies them, in panels laid out in the order in which its lanes ask for them.
//
// The general kernel passes both operands through LDS and fetches an activation once per tap; its waves wait for lines that miss the
// L2s, and its input is a tensor that a launch of its own wrote.  Here an activation is read once, from the network's own tensor, and
// between the window's fill and the result there is no barrier, no transfer and no test:
//   * a wave multiplies FM x FK blocks of 32 pixels x 32 channels (128 x 64: 128 registers of sums).  Its pixels come from LDS one step ahead, its
//     weights from L2 two steps ahead, 4 KB a step.  Rows of weights as pack_weights leaves them would name 32 cache lines per load instead
//     of 8: with two workgroups per compute unit 472 us where panels take 314 (2048 images 256 x 14 x 14 -> 512, main loop alone).
//   * the window is that of a virtual image with its border in it (panel_fill.h), so that a tap is one addition: masks instead cost 7 % of that
//     loop.  It holds as many chunks of 64 channels as LDS has room for, filled all at once.  (Filled chunk by chunk beside the MFMAs the same
//     layer took 1.09 times as long: a wave's loads return in order, so its next weights wait behind pixels that come from memory.)
//   * two workgroups (of the smaller tiles three, four) share a compute unit: one fills or stores while the other multiplies.
// The main loop alone keeps the matrix pipe busy all the time, and the power management lowers the clock to 1.4 - 1.5 GHz: 2.6 POP/s there where the
// register-resident probe has 3.2.  Calls with kept weights, both launches: the layer above 549 -> 474 us in turn, 462 images 256 x 28 x 28 -> 128 179 -> 113,
// 205 x 512 x 22 x 22 -> 128 90 -> 68, 675 x 512 x 14 x 14 -> 17 63 -> 42; all 2048 x 256 x 14 x 14 -> 512 needs at the probe's rate is 300.
#include "panel_fill.h"
#include "kernels.h"
#include "launch.h"
#include "store_past.h"

#include <type_traits>

namespace c2i8 {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int PN_PITCH = 80;                  // bytes of a 64-channel record
constexpr long long PN_LDS = 160 * 1024, PN_LDS_LIMIT = PN_LDS / 2;   // of a compute unit; of a workgroup
constexpr int panel_occupancy(int fm, int fk) { return fm * fk > 4 ? 2 : fm * fk > 2 ? 3 : 4; }   // workgroups per compute unit that the registers are for
constexpr int PN_AHEAD = 3;                   // steps of weights in registers, the one being multiplied among them
constexpr int PN_STEP = 4096;                 // bytes of a panel's step: 64 channels x 64 bytes of depth

enum PanelSource : int { PN_NCHW = 0, PN_NHWC = 1 };

struct PanelArgs {
    const int8_t *src, *wp;
    int32_t *out;                   // [N][K][P][Q], or from an NHWC source [N][P][Q][K]
    VirtualImage v;
    int past;                       // Past
    int K, M, PQ, Q;
    int stride, dil, S, RS;
    int steps, groups;              // 64-byte steps of the depth, 64-channel groups of the weights
    int span;                       // slots from a pixel's first tap to its last
    int buf_bytes, at_once;         // bytes of a chunk's window; chunks that are in LDS at a time
    int fill_off, tab_off;          // the window's places in memory, the steps' in the window
    int quads;                      // no four pixels from a multiple of four on belong to two images
    int tiles_k, mper;
    unsigned mg_PQ, mg_Q, mg_tiles_k, mg_RS, mg_S, mg_at_once;
};

// LDS reads and writes before it are done; loads of weights and pixels stay in flight.
__device__ __forceinline__ void panel_barrier()
{
    asm volatile("" : : : "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" : : : "memory");
}

// Slot, in the virtual image, of an output pixel's first tap.
__device__ __forceinline__ int first_tap(const PanelArgs &a, int m)
{
    const int n = fast_div_any(m, a.PQ, a.mg_PQ), pq = m - n * a.PQ;
    const int p = fast_div_any(pq, a.Q, a.mg_Q), q = pq - p * a.Q;
    return (n * a.v.Hv + p * a.stride) * a.v.Wv + q * a.stride;
}

// FM, FK: blocks of 32 pixels and of 32 output channels of a wave; WK x WM waves cover the tile.
template <int FM, int FK, int WK, int WM, int SRC>
__global__ void __launch_bounds__(256, panel_occupancy(FM, FK)) conv_panel_kernel(const PanelArgs a)
{
    static_assert(WK * WM == 4, "four waves");
    constexpr int U = PN_AHEAD, CH = FK * 32, TK = WK * CH, PX = FM * 32;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % WK, wm = wave / WK;
    const int lid = xcd_contiguous(blockIdx.x, gridDim.x), tm = fast_div_any(lid, a.tiles_k, a.mg_tiles_k), tk = lid - tm * a.tiles_k;
    const int k0 = tk * TK + wk * CH, m0 = tm * a.mper, m1 = min(m0 + a.mper, a.M);

    // ---- weights: panels of two blocks of 32 channels, step after step ---------------------------------------------------------
    const int first = min(k0 >> 5, a.groups * 2 - FK);   // (past the last channels the last blocks again: no result of theirs is stored)
    const int8_t *const weights = a.wp + (size_t)(first >> 1) * a.steps * PN_STEP + (first & 1) * (PN_STEP / 2), *const wend = weights + (size_t)(a.steps - 1) * PN_STEP;
    const int8_t *wb = weights;
    const unsigned wl = lane * 16;   // (a lane's part of a transfer)
    v4i b[U][FK * 2];                // (block of channels, half of the step)
    auto load_weights = [&](v4i(&x)[FK * 2]) {
#pragma unroll
        for (int i = 0; i < FK * 2; ++i) x[i] = *reinterpret_cast<const v4i *>(panel_local(wb, wl) + i * 1024);
        wb = wb < wend ? wb + PN_STEP : wend;   // (past the end the last one again; no step multiplies it)
    };

    // ---- the window: its slots' places, the steps' places in it, the first chunks ---------------------------------------------
    typedef PanelFill<SRC == PN_NHWC> Fill;
    const int lo = first_tap(a, m0), n0 = fast_div_any(m0, a.PQ, a.mg_PQ);
    const PanelWindow win = panel_window(a.v, a.src, n0, lo, first_tap(a, m1 - 1) + a.span);
    unsigned char *const ftab = smem + a.fill_off;
    Fill::table(a.v, win, n0, lo, ftab, tid, 256);
    int *const tab = reinterpret_cast<int *>(smem + a.tab_off);
    for (int i = tid; i <= a.steps; i += 256) {   // (the reads are a step ahead)
        const int st = min(i, a.steps - 1), c = fast_div_any(st, a.RS, a.mg_RS), tap = st - c * a.RS, r = fast_div_any(tap, a.S, a.mg_S), s = tap - r * a.S;
        tab[i] = (r * a.v.Wv + s) * a.dil * PN_PITCH + (c - fast_div_any(c, a.at_once, a.mg_at_once) * a.at_once) * a.buf_bytes;
    }
    panel_barrier();
    const int mw = m0 + wm * PX;
    int base[FM];
#pragma unroll
    for (int f = 0; f < FM; ++f) base[f] = (first_tap(a, min(mw + f * 32 + (lane & 31), m1 - 1)) - lo) * PN_PITCH + (lane >> 5) * 16;
    v16i acc[FM][FK];
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int i = 0; i < FK; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[f][i][v] = 0;

    v4i af[FM][2];
    auto read_pixels = [&](int f, int h, int at) { af[f][h] = *reinterpret_cast<const v4i *>(__builtin_assume_aligned(smem + base[f] + at + h * 32, 16)); };
    // A step: the blocks multiply the pixels and weights at hand; behind each its pixels of the next step, `at` bytes from the first tap's
    // record, are asked for, before all of them the weights of the step U - 1 ahead.
    auto step = [&](v4i(&now)[FK * 2], v4i(&later)[FK * 2], int at) {
        load_weights(later);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int f = 0; f < FM; ++f) {
#pragma unroll
                for (int i = 0; i < FK; ++i)
                    acc[f][i] = SRC == PN_NHWC ? __builtin_amdgcn_mfma_i32_32x32x32_i8(now[i * 2 + h], af[f][h], acc[f][i], 0, 0, 0)
                                               : __builtin_amdgcn_mfma_i32_32x32x32_i8(af[f][h], now[i * 2 + h], acc[f][i], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);   // (into the registers they came from)
                read_pixels(f, h, at);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    // Parts of the depth, as many chunks as LDS holds: the window, then its steps.
    for (int from = 0; from < a.v.chunks; from += a.at_once) {
        const int chunks = min(a.at_once, a.v.chunks - from), steps = chunks * a.RS;
        wb = weights + (size_t)(from * a.RS) * PN_STEP;   // (what the last part's last steps asked for comes again)
#pragma unroll
        for (int u = 0; u < U - 1; ++u) load_weights(b[u]);
        if (from) panel_barrier();   // (the part before it is read)
        const int rounds = Fill::rounds(win, chunks);
        if (!win.last)
            for (int r0 = 0; r0 < rounds; r0 += 2) {   // (with the loads of four on their way together the registers spill: 1.07 of the time)
                int r = r0;
                asm("" : "+s"(r));   // (as if from elsewhere: else what follows from it becomes registers that each turn adds to)
                Fill x[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    x[i].template take<false>(a.v, win, ftab, from, chunks, r + i, tid);
                    __builtin_amdgcn_sched_barrier(0);   // (one round's addresses at a time)
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    x[i].put(win, ftab, chunks, r + i, smem, a.buf_bytes, PN_PITCH, tid);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        else
            for (int r = 0; r < rounds; ++r) {
                Fill x;
                x.template take<true>(a.v, win, ftab, from, chunks, r, tid);
                x.put(win, ftab, chunks, r, smem, a.buf_bytes, PN_PITCH, tid);
            }
        panel_barrier();
        const int *const places = tab + from * a.RS;
        int at = places[0], next = places[1];
#pragma unroll
        for (int f = 0; f < FM; ++f) read_pixels(f, 0, at), read_pixels(f, 1, at);
        // While it multiplies a wave goes before the other workgroups', which fill their window or write their result beside: 0.975 of the time
        // (2048 images 256 x 14 x 14 -> 512; the other way round it takes what it takes without).
        __builtin_amdgcn_s_setprio(1);
        for (int j = 0; j < steps; j += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u > 0 && j + u >= steps) break;
                at = next;
                next = places[min(j + u + 2, steps)];
                step(b[u], b[(u + U - 1) % U], at);
            }
        }
        __builtin_amdgcn_s_setprio(0);
    }

    // ---- result: through a corner of LDS that is the wave's own, out in whole rows -------------------------------------------
    panel_barrier();
    if (k0 >= a.K || mw >= m1) return;
    if constexpr (SRC == PN_NCHW) {
        // 32 rows of QUADS pieces, a block of channels at a time: RPI rows per instruction, so that a lane has one place in all of them
        constexpr int ROW = PX * 4 + 16, QUADS = PX / 4, RPI = 64 / QUADS, NS = 32 / RPI;
        const int quad = lane % QUADS, row = lane / QUADS, m = mw + quad * 4;
        const int nw = fast_div_any(mw, a.PQ, a.mg_PQ), at = mw - nw * a.PQ + quad * 4, n = fast_div_any(at, a.PQ, a.mg_PQ);
        const unsigned plane = (unsigned)a.PQ * 4u;
        char *const to = reinterpret_cast<char *>(a.out + ((size_t)nw * a.K + k0) * a.PQ);
        unsigned char *const mine = smem + wave * 32 * ROW, *const from = mine + row * ROW + quad * 16;
        v4i t4[NS];
        auto turn = [&](int i) {
#pragma unroll
            for (int f = 0; f < FM; ++f)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<v4i *>(mine + (lane & 31) * ROW + f * 128 + g * 32 + (lane >> 5) * 16) =
                        v4i{acc[f][i][4 * g], acc[f][i][4 * g + 1], acc[f][i][4 * g + 2], acc[f][i][4 * g + 3]};
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int t = 0; t < NS; ++t) t4[t] = *reinterpret_cast<const v4i *>(__builtin_assume_aligned(from + t * RPI * ROW, 16));
            __builtin_amdgcn_wave_barrier();
        };
        if (a.quads && k0 + CH <= a.K) {
            const unsigned off = ((unsigned)n * (unsigned)a.K + (unsigned)row) * plane + (unsigned)(at - n * a.PQ) * 4u;
            const bool mine_there = m < m1;   // (m1 is a multiple of four, as is m)
            const auto out = past_base(to);
            auto passes = [&](auto past) {
#pragma unroll
                for (int i = 0; i < FK; ++i) {
                    turn(i);
                    if (mine_there)
#pragma unroll
                        for (int t = 0; t < NS; ++t) store_row16<decltype(past)::value>(out, off, (unsigned)(i * 32 + t * RPI) * plane, t4[t]);
                }
            };
            if (a.past == PAST_THROUGH) passes(PastHow<PAST_THROUGH>{});
            else if (a.past == PAST_STREAM) passes(PastHow<PAST_STREAM>{});
            else passes(PastHow<PAST_NONE>{});
        } else {   // the last channels, or two images meet in four pixels
            int32_t *px[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int x = min(m + e, m1 - 1), nx = fast_div_any(x, a.PQ, a.mg_PQ);
                px[e] = a.out + ((size_t)nx * a.K + k0 + row) * a.PQ + (x - nx * a.PQ);
            }
            const bool whole = m + 3 < m1 && at - n * a.PQ + 3 < a.PQ;
#pragma unroll
            for (int i = 0; i < FK; ++i) {
                turn(i);
#pragma unroll
                for (int t = 0; t < NS; ++t) {
                    const int k = i * 32 + t * RPI;
                    if (k0 + k + row >= a.K) continue;
                    if (whole) *reinterpret_cast<v4i_a4 *>(px[0] + (size_t)k * a.PQ) = t4[t];
                    else
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (m + e < m1) px[e][(size_t)k * a.PQ] = t4[t][e];
                }
            }
        }
    } else {
        constexpr int ROW = CH * 4 + 16, LPP = CH / 4, PPI = 64 / LPP, NS = 32 / PPI;   // a pixel's channels, LPP lanes; PPI pixels per instruction
        unsigned char *const mine = smem + wave * 32 * ROW;
        const int k = k0 + lane % LPP * 4;
        const bool whole = k + 3 < a.K;
        int32_t *const to = a.out + (size_t)mw * a.K + k;
#pragma unroll
        for (int f = 0; f < FM; ++f) {
#pragma unroll
            for (int i = 0; i < FK; ++i)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<v4i *>(mine + (lane & 31) * ROW + i * 128 + g * 32 + (lane >> 5) * 16) =
                        v4i{acc[f][i][4 * g], acc[f][i][4 * g + 1], acc[f][i][4 * g + 2], acc[f][i][4 * g + 3]};
            __builtin_amdgcn_wave_barrier();
            v4i t4[NS];
#pragma unroll
            for (int t = 0; t < NS; ++t) t4[t] = *reinterpret_cast<const v4i *>(__builtin_assume_aligned(mine + (t * PPI + lane / LPP) * ROW + lane % LPP * 16, 16));
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int t = 0; t < NS; ++t) {
                const int m = f * 32 + t * PPI + lane / LPP;
                if (mw + m >= m1) continue;
                int32_t *const px = to + (size_t)m * a.K;
                if (whole) *reinterpret_cast<v4i_a4 *>(px) = t4[t];
                else
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        if (k + e < a.K) px[e] = t4[t][e];
            }
        }
    }
}

// ---- weights into panels: [64-channel group][step][32 channels][half of the step][lane][16 bytes of depth] -------------------------------------
// Lane l of a block holds output channel l % 32, channels 16 (l / 32) ... of the half's 32.  Channels that are not there are zeros.
struct PanelWeights {
    const int8_t *src;
    int8_t *dst;
    int K, C, RS, steps, cb, depth, groups;
    unsigned mg_steps, mg_RS, mg_cb;
};
// From rows of channel blocks of cb.
__global__ void __launch_bounds__(256) panel_from_rows_kernel(const PanelWeights a)
{
    const int u = blockIdx.x * 256 + threadIdx.x, lane = u & 63, i = (u >> 6) & 3, gs = u >> 8;
    const int g = fast_div_any(gs, a.steps, a.mg_steps), st = gs - g * a.steps;
    if (g >= a.groups) return;
    const int chunk = fast_div_any(st, a.RS, a.mg_RS), tap = st - chunk * a.RS;
    const int k = g * 64 + (i >> 1) * 32 + (lane & 31), c = chunk * 64 + (i & 1) * 32 + (lane >> 5) * 16;
    v4i x = {0, 0, 0, 0};
    const int blk = fast_div_any(c, a.cb, a.mg_cb), at = (blk * a.RS + tap) * a.cb + c - blk * a.cb;
    if (k < a.K && c < a.C && at + 16 <= a.depth) x = *reinterpret_cast<const v4i *>(a.src + (size_t)k * a.depth + at);
    *reinterpret_cast<v4i *>(a.dst + (size_t)u * 16) = x;
}
// From KCRS: 16 output channels x 64 channels with all taps per workgroup, turned around in LDS.
__global__ void __launch_bounds__(256) panel_from_raw_kernel(const PanelWeights a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, chunks = gridDim.y, chunk = blockIdx.y, kb = blockIdx.x;   // kb: block of 16 output channels
    const int row = 64 * a.RS, pitch = row + 4, have = min(64, a.C - chunk * 64) * a.RS;
    const int8_t *const from = a.src + (size_t)kb * 16 * a.C * a.RS + (size_t)chunk * row;
    for (int r = tid >> 4; r < 16; r += 16) {
        const int8_t *const p = from + (size_t)r * a.C * a.RS;
        const bool there = kb * 16 + r < a.K;
        for (int x = (tid & 15) * 4; x < row; x += 64) {
            unsigned w = 0;
            if (there && x + 4 <= have) __builtin_memcpy(&w, p + x, 4);
            else if (there)
                for (int e = 0; e < 4; ++e)
                    if (x + e < have) w |= (unsigned)(unsigned char)p[x + e] << (8 * e);
            *reinterpret_cast<unsigned *>(smem + r * pitch + x) = w;
        }
    }
    __syncthreads();
    // (this block's 16 output channels are half of a block's lanes)
    int8_t *const to = a.dst + ((size_t)(kb >> 2) * chunks + chunk) * a.RS * PN_STEP + (kb & 2) * 1024 + (kb & 1) * 256;
    for (int u = tid; u < a.RS * 64; u += 256) {
        const int tap = u >> 6, lane = u & 63;
        const int quarter = lane >> 4;   // of the step's 64 channels
        const unsigned char *const p = smem + (lane & 15) * pitch + quarter * 16 * a.RS + tap;
        v4i x;
#pragma unroll
        for (int d = 0; d < 4; ++d)
            x[d] = (int)(p[(4 * d) * a.RS] | (unsigned)p[(4 * d + 1) * a.RS] << 8 | (unsigned)p[(4 * d + 2) * a.RS] << 16 | (unsigned)p[(4 * d + 3) * a.RS] << 24);
        *reinterpret_cast<v4i *>(to + (size_t)tap * PN_STEP + (quarter >> 1) * 1024 + (quarter & 1) * 512 + (lane & 15) * 16) = x;
    }
}

// FM, FK, WK, WM
#define C2I8_PANEL_LIST(X) \
    X(4, 2, 4, 1) /* 256 x 128 */ \
    X(4, 2, 2, 2) /* 128 x 256 */ \
    X(4, 2, 1, 4) /*  64 x 512 */ \
    X(2, 2, 4, 1) /* 256 x  64 */ \
    X(2, 2, 2, 2) /* 128 x 128 */ \
    X(2, 2, 1, 4) /*  64 x 256 */ \
    X(4, 1, 1, 4) /*  32 x 512 */ \
    X(2, 1, 1, 4) /*  32 x 256 */

struct PanelTile {
    int fm, fk, wk, wm;
    int tk() const { return wk * fk * 32; }
    int tm() const { return fm * wm * 32; }
    int stage(int source) const { return 4 * 32 * (source == PN_NHWC ? fk * 128 + 16 : fm * 128 + 16); }   // the result's way out
};
constexpr PanelTile kPanelTiles[] = {
#define C2I8_ROW(...) {__VA_ARGS__},
    C2I8_PANEL_LIST(C2I8_ROW)
#undef C2I8_ROW
};
constexpr int kNumPanelTiles = sizeof(kPanelTiles) / sizeof(kPanelTiles[0]);

template <int FM, int FK, int WK, int WM>
hipError_t launch_panel_tile(const PanelArgs &a, int source, unsigned grid, size_t lds, hipStream_t st)
{
    void (*const kern)(PanelArgs) = source == PN_NHWC ? conv_panel_kernel<FM, FK, WK, WM, PN_NHWC> : conv_panel_kernel<FM, FK, WK, WM, PN_NCHW>;
    static bool raised[2];
    if (!raised[source]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)PN_LDS_LIMIT);
        if (e != hipSuccess) return e;
        raised[source] = true;
    }
    return launch(kern, dim3(grid), dim3(256), lds, st, a);
}

// What the estimate and the plan share: window slots, chunks at a time, LDS.
struct PanelRoom {
    long long slots, tables, at_once, lds;
};
PanelRoom panel_room(const PanelTile &d, int source, long long slots, int chunks, int steps)
{
    PanelRoom m{slots, slots / 8 * (source == PN_NHWC ? PanelFill<true>::ENTRY : PanelFill<false>::ENTRY) + 4 * (steps + 1), 0, 0};
    const long long buf = slots * PN_PITCH;
    m.at_once = (PN_LDS / panel_occupancy(d.fm, d.fk) / 1024 * 1024 - m.tables) / buf;
    if (m.at_once < 1) m.at_once = (PN_LDS_LIMIT - m.tables) / buf;
    if (m.at_once < 1) return m;
    if (m.at_once >= chunks) m.at_once = chunks;
    else {   // parts of a size
        const long long parts = (chunks + m.at_once - 1) / m.at_once;
        m.at_once = (chunks + parts - 1) / parts;
    }
    m.lds = m.at_once * buf + m.tables;
    if (m.lds < d.stage(source)) m.lds = d.stage(source);
    return m;
}

struct PanelPlan {
    PanelArgs a;
    int tile, source;
    unsigned grid;
    size_t lds;
};

bool panel_plan(const ResidentProblem &r, int tile, int mper, PanelPlan *out)
{
    const GemmProblem &g = r.g;
    const PanelTile &d = kPanelTiles[tile];
    const int RS = g.R * g.S, dil = g.dil > 0 ? g.dil : 1;
    if (mper < 1 || mper > d.tm() || g.mode != ACT_BLOCKED || RS > 49 || g.il_d || g.act_out || r.pixel_major != g.out_nhwc || g.Q <= 0 || g.PQ % g.Q || g.M <= 0)
        return false;
    if (!virtual_image_fits(g.R, g.S, dil, r.H, r.W, r.pad, r.N, r.img_bytes)) return false;
    const long long HW = (long long)r.H * r.W, Wv = r.W + r.pad, Hv = r.H + r.pad;
    PanelArgs &a = out->a;
    a = PanelArgs{};
    auto magic = [](long long v) { return v <= 1 ? 0u : magic_for(v); };
    a.K = g.K, a.M = g.M, a.PQ = g.PQ, a.Q = g.Q;
    a.stride = g.stride, a.dil = dil, a.S = g.S, a.RS = RS;
    a.v = VirtualImage{(int)Wv, (int)Hv, r.N, r.C, r.H, r.W, (int)HW, r.pad, (r.C + 63) / 64, r.pixel_bytes, r.img_bytes, r.img_bytes * r.N, magic(Wv), magic(Hv)};
    a.steps = a.v.chunks * RS;
    a.groups = (g.K + 63) / 64;
    a.span = (int)(((g.R - 1) * Wv + g.S - 1) * dil);
    a.mper = mper;
    const long long slots = window_slots(mper, g.PQ, g.Q, g.stride, Wv, Hv, a.span), imgs = (mper + g.PQ - 2) / g.PQ;
    if ((imgs + 1) * r.img_bytes + 64 * HW > 0x7FFFFFFFLL || (imgs + 1) * g.K * (long long)g.PQ * 4 > 0x7FFFFFFFLL) return false;   // 32-bit offsets from the tile's first image
    a.buf_bytes = (int)(slots * PN_PITCH);
    const int source = r.pixel_major ? PN_NHWC : PN_NCHW;
    const PanelRoom room = panel_room(d, source, slots, a.v.chunks, a.steps);
    if (room.at_once < 1 || room.lds > PN_LDS_LIMIT) return false;
    a.at_once = (int)room.at_once;
    a.fill_off = a.at_once * a.buf_bytes;
    a.tab_off = a.fill_off + (int)room.tables - 4 * (a.steps + 1);
    a.quads = g.PQ % 4 == 0 && mper % 4 == 0;
    // Past the caches: non-temporal from 28 MB on (planes of whole sectors, 28 to 256 MB: 462 images 256 x 28 x 28 -> 128 124 -> 119.7 us), below
    // through the L2s.
    const double bytes = 4.0 * g.M * g.K;
    a.past = a.quads ? past_caches(bytes) : PAST_NONE;
    if (a.quads && g.PQ % 16 == 0 && mper % 16 == 0 && a.past == PAST_NONE) a.past = PAST_STREAM;
    a.tiles_k = (g.K + d.tk() - 1) / d.tk();
    const long long wgs = ((long long)g.M + mper - 1) / mper * a.tiles_k;
    if (wgs > 0x7FFFFFFFLL) return false;
    a.mg_PQ = magic(g.PQ), a.mg_Q = magic(g.Q), a.mg_tiles_k = magic(a.tiles_k), a.mg_RS = magic(RS), a.mg_S = magic(g.S), a.mg_at_once = magic(a.at_once);
    out->tile = tile;
    out->source = source;
    out->grid = (unsigned)wgs;
    out->lds = (size_t)room.lds;
    return true;
}

// Launch time in microseconds, both launches, fitted per tile to 59000 (NCHW) and 12000 (NHWC) measured pairs of 9400 layers (a third held back: mean
// error 5 to 7 %, NHWC 3 to 4 %; the tile it picks takes 1.011 of the best one's time in the mean).  A launch; the weights' bytes; what the
// busiest compute unit's workgroups take, one by one and as many at a time as fit, per workgroup, step, 64-byte record of the window and part of
// the depth; the same for all of them; the result's megabytes on planes of whole 64-byte sectors (NHWC: all), of 16-byte pieces, others, and
// of NHWC rows that are none; KCRS weights.  None is below zero and many are 0, as a fit that is bounded there
// leaves them: no measure of that term alone.
struct PanelFit {
    double launch, weights, one, one_step, one_fill, one_part, round, round_step, round_fill, all_step, all_fill, sectors, pieces, odd, odd_rows, all, raw;
};
constexpr PanelFit kPanelFit[2][kNumPanelTiles] = {
    {   // NCHW
        {6.448, 1.514, 0.2418, 0.2154, 7.12e-05, 0.4044, 1.663, 0.08706, 0.003625, 0.03559, 0.0003866, 0.0701, 0.09312, 0.1827, 0, 0, 1.269},
        {6.657, 0.8733, 0.6231, 0.178, 0.0007767, 0.2864, 1.143, 0.1227, 0.003169, 0.0454, 5.744e-05, 0.06481, 0.08257, 0.1787, 0, 0, 1.282},
        {6.32, 0.1445, 1.338, 0.1321, 0, 0.252, 0.7671, 0.1653, 0.004286, 0.05669, 0.0002436, 0.04901, 0.06347, 0.1614, 0, 0, 1.334},
        {6.858, 1.417, 0, 0.1059, 0.0006539, 0.4325, 0.482, 0.08906, 0.002907, 0.02103, 0.0002701, 0.08939, 0.1235, 0.1873, 0, 0, 1.145},
        {6.519, 0.8854, 0.1144, 0.09441, 0.0003723, 0.5138, 0.7446, 0.09955, 0.003489, 0.0223, 0.0001263, 0.06884, 0.1009, 0.1725, 0, 0, 1.199},
        {6.282, 0.5068, 0.5286, 0.07612, 0, 0.4895, 0.4981, 0.1146, 0.004025, 0.02406, 0.0003315, 0.05555, 0.07897, 0.1588, 0, 0, 1.169},
        {5.235, 0.1788, 0.461, 0.05201, 0, 0.3217, 1.482, 0.1324, 0.004234, 0.0316, 7.063e-05, 0.03382, 0.05973, 0.1721, 0, 0, 1.445},
        {5.646, 0.9771, 0.2852, 0.04492, 0.0005434, 0.1808, 0.3485, 0.1036, 0.003703, 0.01148, 3.404e-05, 0.04033, 0.06858, 0.154, 0, 0, 1.494},
    },
    {   // NHWC
        {9.057, 1.127, 1.049, 0.1889, 0, 0.07091, 0.06036, 0.002962, 0.007466, 0.09481, 0, 0.08082, 0, 0, 0.04712, 0, 0},
        {9.003, 0.7218, 1.278, 0.1227, 0, 0.3716, 0.07477, 0.06155, 0.005874, 0.08795, 0.0007506, 0.06592, 0, 0, 0.06205, 0.1448, 0},
        {8.673, 0, 2.37, 0.01484, 0, 0, 0, 0.1827, 0.005267, 0.03462, 0.002417, 0.01548, 0, 0, 0.05181, 0.6831, 0},
        {8.308, 0.9548, 0, 0.1035, 0, 0.6215, 0.1165, 0.05878, 0.00434, 0.05045, 0, 0.09644, 0, 0, 0.03993, 0.1356, 0},
        {8.088, 0.7721, 0, 0.09943, 0, 0.546, 0.3732, 0.05797, 0.004653, 0.04125, 5.542e-05, 0.07824, 0, 0, 0.04044, 0.4404, 0},
        {8.079, 0, 0.04147, 0.07934, 0, 0.3995, 0.4244, 0.003719, 0.006977, 0.02767, 0.0007237, 0.05014, 0, 0, 0.03665, 0.9583, 0},
        {7.752, 0, 0.8655, 0.0206, 0, 0, 0.129, 0.1024, 0.005006, 0.05417, 0.001016, 0.0813, 0, 0, 0.05264, 0, 0},
        {7.51, 0.4245, 0, 0.02278, 0, 0.2248, 0, 0.02998, 0.006575, 0.03488, 0, 0.09489, 0, 0, 0.04797, 0.2006, 0},
    },
};

double panel_us(const ResidentProblem &r, int tile, int mper)
{
    const GemmProblem &g = r.g;
    const PanelTile &d = kPanelTiles[tile];
    const int source = r.pixel_major ? PN_NHWC : PN_NCHW, RS = g.R * g.S, dil = g.dil > 0 ? g.dil : 1, chunks = (r.C + 63) / 64, steps = chunks * RS;
    const long long Wv = r.W + r.pad, Hv = r.H + r.pad, span = ((g.R - 1) * Wv + g.S - 1) * dil;
    const PanelRoom room = panel_room(d, source, window_slots(mper, g.PQ, g.Q, g.stride, Wv, Hv, span), chunks, steps);
    if (room.at_once < 1 || room.lds > PN_LDS_LIMIT) return 1e300;
    const long long wgs = (((long long)g.M + mper - 1) / mper) * ((g.K + d.tk() - 1) / d.tk());
    const long long fit = PN_LDS / room.lds, occ = panel_occupancy(d.fm, d.fk) < fit ? panel_occupancy(d.fm, d.fk) : fit;
    const double one = (double)((wgs + 255) / 256), round = (double)((wgs + 256 * occ - 1) / (256 * occ)), per = (double)wgs / 256;
    const double row = (double)g.stride * (Wv - g.Q), img = (double)(Hv - g.PQ / g.Q * g.stride) * Wv, n = mper - 1;
    const double fill = chunks * (n * g.stride + n / g.Q * (row > 0 ? row : 0) + n / g.PQ * img + span + 8), result = 4e-6 * g.M * g.K;
    const PanelFit &f = kPanelFit[source][tile];
    double us = f.launch + f.weights * 1e-6 * (double)panel_weight_bytes(g.K, r.C, RS) + one * (f.one + f.one_step * steps + f.one_fill * fill + f.one_part * (double)((chunks + room.at_once - 1) / room.at_once)) +
                round * (f.round + f.round_step * steps + f.round_fill * fill) + per * (f.all + f.all_step * steps + f.all_fill * fill) + (r.raw_weights ? f.raw : 0);
    if (r.pixel_major) us += result * (f.sectors + (g.K % 4 ? f.odd_rows : 0));
    else us += result * (g.PQ % 16 == 0 && mper % 16 == 0 ? f.sectors : g.PQ % 4 == 0 && mper % 4 == 0 ? f.pieces : f.odd);
    return us;
}

}  // namespace

int panel_num_tiles() { return kNumPanelTiles; }
TileInfo panel_tile_info(int tile) { return TileInfo{kPanelTiles[tile].tk(), kPanelTiles[tile].tm(), 256, PN_AHEAD}; }

size_t panel_weight_bytes(int K, int C, int RS) { return (size_t)((K + 63) / 64) * ((C + 63) / 64) * RS * PN_STEP; }

hipError_t launch_panel_weights(const ResidentProblem &r, int8_t *dst, hipStream_t st)
{
    const GemmProblem &g = r.g;
    const int RS = g.R * g.S, chunks = (r.C + 63) / 64, steps = chunks * RS, groups = (g.K + 63) / 64;
    auto magic = [](long long v) { return v <= 1 ? 0u : magic_for(v); };
    const PanelWeights a{g.wq, dst, g.K, r.C, RS, steps, g.cb, g.depth, groups, magic(steps), magic(RS), magic(g.cb)};
    if (r.raw_weights) return launch(panel_from_raw_kernel, dim3((unsigned)groups * 4, (unsigned)chunks), dim3(256), (size_t)16 * (64 * RS + 4), st, a);
    return launch(panel_from_rows_kernel, dim3((unsigned)((long long)groups * steps)), dim3(256), 0, st, a);
}

bool panel_applies(const ResidentProblem &r, int tile, int mper)
{
    PanelPlan p;
    return panel_plan(r, tile, mper, &p);
}

bool panel_pick(const ResidentProblem &r, double limit, ResidentChoice *c)
{
    PanelPlan p;
    ResidentChoice best[3] = {{0, 0, limit}, {0, 0, limit}, {0, 0, limit}};
    for (int t = 0; t < kNumPanelTiles; ++t) {
        const PanelTile &d = kPanelTiles[t];
        const int tiles_k = (r.g.K + d.tk() - 1) / d.tk();
        if (t > 0 && d.tk() >= 2 * r.g.K && d.tk() > 64) continue;   // (half of the waves for nothing)
        auto consider = [&](long long mper) {
            if (mper < 1 || mper > d.tm()) return;
            const ResidentChoice x{t, (int)mper, panel_us(r, t, (int)mper)};
            for (int k = 0; k < 3; ++k)
                if (x.us < best[k].us) {
                    for (int j = 2; j > k; --j) best[j] = best[j - 1];
                    best[k] = x;
                    break;
                }
        };
        consider(d.tm());
        for (int k = 1; k <= 4; ++k) {   // whole rounds of workgroups
            const long long m = (((long long)r.g.M * tiles_k + 256 * k - 1) / (256 * k) + 15) / 16 * 16;
            if (m > d.tm() / 2 && m < d.tm()) consider(m);
        }
        if (r.g.PQ < d.tm()) consider(d.tm() / r.g.PQ * r.g.PQ);   // whole images
    }
    for (const ResidentChoice &x : best)
        if (x.mper > 0 && panel_plan(r, x.tile, x.mper, &p)) {
            *c = x;
            return true;
        }
    return false;
}

struct PanelKey {
    GemmKey g;
    int v[12];
};

hipError_t launch_panel(const ResidentProblem &r, const int8_t *panels, int tile, int mper, hipStream_t st)
{
    static thread_local PlanTable<PanelKey, PanelPlan, 64> plans;
    const PanelKey key{gemm_key(r.g), {r.N, r.C, r.H, r.W, r.pad, r.pixel_major, r.pixel_bytes, 0, 0, tile, mper, (int)r.img_bytes}};
    const PanelPlan *kept = plans.get(key, [&](PanelPlan *p) { return panel_plan(r, tile, mper, p); });
    if (!kept) return hipErrorInvalidValue;
    PanelArgs a = kept->a;
    a.src = r.src;
    a.wp = panels;
    a.out = r.g.out;
    int index = 0;
#define C2I8_CASE(fm, fk, wk, wm) \
    if (kept->tile == index++) return launch_panel_tile<fm, fk, wk, wm>(a, kept->source, kept->grid, kept->lds, st);
    C2I8_PANEL_LIST(C2I8_CASE)
#undef C2I8_CASE
    return hipErrorInvalidValue;
}

}  // namespace c2i8
