// GEMM stage for deep layers that reads the activations once: the input window of a tile lies in LDS, 64 channels at a time,
// and serves every kernel tap; the weights stream past it through a ring of stages.
//
// The general kernel (igemm_mfma.hip) fetches an activation once per tap -- nine times through L2 and the global->LDS path
// for a 3x3 layer, and its ring covers less than an L2 miss; the resident kernel (resident_mfma.hip) fetches it once but
// needs all weights of its channels in LDS beside the window, which ends at about 300 channels.  Here only the weights pass
// through the ring and the window is kept in chunks of 64 channels, as many as fit: while chunk c is multiplied with its
// R*S taps, chunk c+1 is turned around from the network's own tensor into another buffer.
//   * eight waves, all of them multiply.  Waves 0-3 also transfer the weights (global -> LDS, counted waits), waves 4-7 also
//     fill the window (loads into registers, byte permutes, LDS stores).  A wave's loads return in order, so a wave that did
//     both would wait for its newest weights whenever it needs its oldest pixels; one of each kind shares every SIMD.
//   * a ring stage is 16 KB whatever the tile: 256/TK depth steps of 64 bytes x TK rows.  The DS depth groups of a
//     workgroup take its steps in turn; their sums meet in LDS at the end, each group finishing 1/DS of the tile.
//   * records of 64 channels at a pitch of 80 bytes: any 16 neighbouring pixels start in 16 different bank groups, whatever
//     tap offset is added.  Taps outside the image read a record of zeros (resident_mfma.hip has the same window).
#include "window_fill.h"
#include "kernels.h"
#include "launch.h"
#include "store_past.h"

#include <type_traits>

namespace c2i8 {
namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int ST_PITCH = 80;            // bytes of a 64-channel record
constexpr long long ST_LDS_LIMIT = 160 * 1024;

enum StreamSource : int { ST_NCHW = 0, ST_NHWC = 1 };

struct StreamArgs {
    const int8_t *src, *wq;
    int32_t *out;                  // [N][K][P][Q], or from an NHWC source [N][P][Q][K]
    int past;                      // NKPQ result past the caches: Past
    int K, M, PQ, Q;
    int C1, H, W, HW;              // C1: last channel
    int stride, pad, dil, R, S, RS;
    int depth, steps, stages;      // bytes per weight row, 64-byte steps, ring stages that hold them
    int cb, g16, nreal;            // channel block of the weights; 16-byte chunks of depth that hold weights
    int chunks, nbuf, buf_bytes;   // 64-channel chunks, window buffers, bytes of one
    int full8;                     // slots of a whole image (its range rounded up to 8 pixels)
    int pstride;                   // bytes from pixel to pixel (NHWC)
    int wide;                      // WindowSource::wide
    long long img_bytes, src_bytes;
    int zero_off, win_off, tab_off;
    int tiles_k, tiles_m, tiles_fast, m_fastest, mper;
    unsigned mg_PQ, mg_Q, mg_tiles_fast, mg_full8, mg_g16, mg_S, mg_R, mg_RS;
    int sub;                       // 64-channel chunks of a weight block (blocks of 64 and more), else 0
};

// 16 bytes per lane from base + off to LDS lds + 16*lane.
__device__ __forceinline__ void st_dma16(const int8_t *base, unsigned off, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds), "v"(off), "s"(base) : "memory");
}
template <int N>
__device__ __forceinline__ void st_wait_dma()
{
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
__device__ __forceinline__ void st_barrier()
{
    asm volatile("" : : : "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" : : : "memory");
}

// One round of the window fill beside the MFMAs: of chunk `c`, the records from slot ROUND*round on, by four waves.  take()
// asks for the pixels, put() stores them; between the two the loads are in flight, in 8 * G registers.
template <int SRC, int G>
struct Filler {
    static constexpr int FT = 256, ROUND = 128 * G;
    static constexpr int B = 2 * G;   // NHWC: 16-byte pieces of a thread
    v4i q[B];
    int at;                           // NCHW: the unit's first slot
    unsigned char *dst;

    __device__ __forceinline__ void take(const StreamArgs &a, const WindowRange &w, int n1, int c, int round, int t, unsigned char *buf)
    {
        const int8_t *const img0 = a.src + (long long)w.n0 * a.img_bytes;
        const bool whole = (long long)(n1 + 1) * a.img_bytes + 64 <= a.src_bytes;   // (uniform) no load can pass the tensor's end
        if constexpr (SRC == ST_NCHW) {
            // 4 channels x 16 pixels (G = 2) or 8 (G = 1): neighbouring lanes are neighbours within 64 bytes of a channel row
            constexpr int PX = 8 * G, LR = 64 / PX;
            const int lane = t & 63, wv = t >> 6;
            const int quad = G == 2 ? lane >> 2 : (lane >> 3) + 8 * (wv & 1), run = G == 2 ? wv + 4 * round : (wv >> 1) + 2 * round;
            at = run * 64 + (lane & (LR - 1)) * PX;
            dst = buf + at * ST_PITCH + quad * 4;
            if (at >= w.slots) return;
            const int ch = c * 64 + quad * 4;
            const bool fast = c * 64 + 79 <= a.C1 || (whole && c * 64 + 63 <= a.C1);   // every channel is there, and 16 bytes behind it
            int n, lin;
            window_slot(w, at, &n, &lin);
            const int ahead = at < w.len0 ? w.len0 - at : w.full8 - lin;
            if (fast) {
                const int8_t *const b0 = img0 + (long long)c * 64 * a.HW;
                const unsigned off = (unsigned)((n - w.n0) * (int)a.img_bytes + quad * 4 * a.HW + lin);
                if constexpr (G == 1) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const unsigned long long x = *reinterpret_cast<const u64_a1 *>(b0 + (long long)i * a.HW + off);
                        q[i >> 1][2 * (i & 1)] = (int)(unsigned)x;
                        q[i >> 1][2 * (i & 1) + 1] = (int)(unsigned)(x >> 32);
                    }
                } else if (ahead >= 16 || at + 8 >= w.slots) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) __builtin_memcpy(&q[i], b0 + (long long)i * a.HW + off, 16);
                } else {   // the other eight pixels begin the next image
                    const unsigned off2 = (unsigned)((n + 1 - w.n0) * (int)a.img_bytes + quad * 4 * a.HW);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        unsigned long long x[2];
                        x[0] = *reinterpret_cast<const u64_a1 *>(b0 + (long long)i * a.HW + off);
                        x[1] = *reinterpret_cast<const u64_a1 *>(b0 + (long long)i * a.HW + off2);
                        __builtin_memcpy(&q[i], x, 16);
                    }
                }
            } else {
                const long long left = a.src_bytes - 8 - (long long)w.n0 * a.img_bytes;
#pragma unroll
                for (int h = 0; h < G; ++h) {
                    if (h) window_slot(w, min(at + 8, w.slots - 8), &n, &lin);
                    const long long img = (long long)(n - w.n0) * a.img_bytes + lin;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const long long want = img + (long long)min(ch + i, a.C1) * a.HW, from = want < left ? want : left;
                        const unsigned long long x = *reinterpret_cast<const u64_a1 *>(img0 + from) >> (8 * (int)(want - from));
                        if constexpr (G == 1) q[i >> 1][2 * (i & 1)] = (int)(unsigned)x, q[i >> 1][2 * (i & 1) + 1] = (int)(unsigned)(x >> 32);
                        else q[i][2 * h] = (int)(unsigned)x, q[i][2 * h + 1] = (int)(unsigned)(x >> 32);
                    }
                }
            }
        } else {
            const int j = t & 3, s0 = (t >> 2) + round * ROUND;
            dst = buf + s0 * ST_PITCH + j * 16;
            const int ch = c * 64 + j * 16;
            const bool fast = c * 64 + 63 <= a.C1 || whole;
#pragma unroll
            for (int b = 0; b < B; ++b) {
                if (s0 + b * (FT / 4) >= w.slots) break;
                int n, lin;
                window_slot(w, s0 + b * (FT / 4), &n, &lin);
                lin = min(lin, a.HW - 1);
                const long long want = (long long)(n - w.n0) * a.img_bytes + ch + (long long)lin * a.pstride;
                if (fast) __builtin_memcpy(&q[b], img0 + want, 16);
                else {
                    const long long left = a.src_bytes - 16 - (long long)w.n0 * a.img_bytes, from = want < left ? want : left;
                    v4i x;
                    __builtin_memcpy(&x, img0 + from, 16);
                    const int over = (int)(want - from);   // (16 and more: channels that no weight belongs to)
                    q[b] = over ? shift_piece(x, -min(over, 15)) : x;
                }
            }
        }
    }
    __device__ __forceinline__ void put(const WindowRange &w, int round, int t) const
    {
        if constexpr (SRC == ST_NCHW) {
            if (at >= w.slots) return;
            if constexpr (G == 2) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e < 2 || at + 8 < w.slots)
                        put_4x4((unsigned)q[0][e], (unsigned)q[1][e], (unsigned)q[2][e], (unsigned)q[3][e], dst + 4 * e * ST_PITCH, ST_PITCH);
            } else {
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    put_4x4((unsigned)q[0][e], (unsigned)q[0][2 + e], (unsigned)q[1][e], (unsigned)q[1][2 + e], dst + 4 * e * ST_PITCH, ST_PITCH);
            }
        } else {
            const int s0 = (t >> 2) + round * ROUND;
#pragma unroll
            for (int b = 0; b < B; ++b)
                if (s0 + b * (FT / 4) < w.slots) *reinterpret_cast<v4i *>(dst + b * (FT / 4) * ST_PITCH) = q[b];
        }
    }
};

// FK, FM: 32x32 blocks of a wave (channels, pixels); WK x WM waves cover the tile, DS groups of them split the depth.
// NST: stages of the ring.
template <int FK, int FM, int WK, int WM, int DS, int NST, int SRC, bool UNI>
__global__ void __launch_bounds__(WK * WM * DS * 64, 2) conv_stream_kernel(const StreamArgs a)
{
    constexpr int TK = FK * WK * 32, NWM = WK * WM, NW = NWM * DS, NT = NW * 64;
    constexpr int DW = NW / 2, FT = NT / 2;          // waves that transfer, threads that fill
    constexpr int SPS = NW * 32 / TK, QS = SPS / DS;   // steps of a stage, of a wave in it
    constexpr int ST_STAGE = TK * SPS * 64;          // bytes of a stage: 2 KB per wave
    static_assert(NW == 8, "four waves transfer, four fill");
    static_assert(QS >= 1 && SPS % DS == 0, "every depth group has steps in a stage");
    constexpr int NM = FK * FM, NR = FK + FM, NH = 2 * QS, L = 4;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const unsigned lds0 = (unsigned)(size_t)((__attribute__((address_space(3))) unsigned char *)smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave / NWM, wi = wave % NWM, wk = wi % WK, wm = wi / WK;

    // the tiles of an XCD share the input of their pixels or the weights of their channels behind its L2
    const int lid = xcd_contiguous(blockIdx.x, gridDim.x), slow = fast_div_any(lid, a.tiles_fast, a.mg_tiles_fast), fast = lid - slow * a.tiles_fast;
    const int tm = a.m_fastest ? fast : slow, tk = a.m_fastest ? slow : fast;
    const int k0 = tk * TK, m0 = tm * a.mper, m1 = min(m0 + a.mper, a.M);
    int n1;
    const WindowRange w = tile_window(a, m0, m1, &n1);

    // ---- weights: transfer i = DW*u + wave of a stage moves rows 16 (i % G) ... of its step i / G ---------------------------
    constexpr int G = TK / 16, NROW = G > DW ? G / DW : 1;
    static_assert(G % DW == 0 || DW % G == 0, "a transfer's rows repeat");
    unsigned woff[NROW];
    {
        const int x = (lane & 3) ^ ((lane >> 4) & 3);
#pragma unroll
        for (int u = 0; u < NROW; ++u) {
            const int row = k0 + ((u * DW + (wave & (DW - 1))) % G) * 16 + (lane >> 2);
            woff[u] = (unsigned)min(row, a.K - 1) * (unsigned)a.depth + (unsigned)x * 16u;
        }
    }
    // where the next stage's steps are in a weight row: chunk c's taps follow one another in blocks of up to 64 channels; in a
    // larger block a tap's channels do.  (Steps past the last one fetch it again; the table has zeros for them.)
    int w_at = 0, w_tap = 0, w_sub = 0;
    const int w_last = (!UNI || a.sub <= 1) ? (a.steps - 1) * 64 : 0x7FFFFFFF;
    auto next_step = [&]() {
        if (!UNI || a.sub <= 1) w_at = min(w_at + 64, w_last);
        else if (++w_tap < a.RS) w_at += a.cb;
        else {
            w_tap = 0;
            if (++w_sub == a.sub) w_sub = 0, w_at += 64;                       // the next block begins behind this one's last tap
            else w_at -= (a.RS - 1) * a.cb - 64;                               // the block's next 64 channels, first tap
            if (w_at + 64 > a.depth) w_at = 0;                                 // (past the end)
        }
    };
    auto dma_stage_part = [&](int u, unsigned slot) {   // transfer u of the stage the counters stand at (waves below DW)
        constexpr int UPS = G > DW ? G / DW : 1;        // transfers of a wave per step
        const int i = u * DW + wave;
        if constexpr (DW <= G) {
            st_dma16(a.wq + w_at, woff[u % NROW], slot + (unsigned)i * 1024u);
            if ((u + 1) % UPS == 0) next_step();
        } else {   // several waves share the rows of several steps
            constexpr int SPU = DW / G;                 // steps that one transfer of every wave covers
            const int mine = wave / G;
            int at = w_at;
#pragma unroll
            for (int k = 0; k < SPU; ++k) {
                if (k == mine) at = w_at;
                next_step();
            }
            st_dma16(a.wq + at, woff[0], slot + (unsigned)i * 1024u);
        }
    };
    if (wave < DW) {
#pragma unroll
        for (int s = 0; s < NST - 1; ++s)
            if (s < a.stages) {
#pragma unroll
                for (int u = 0; u < L; ++u) dma_stage_part(u, lds0 + (unsigned)(s * ST_STAGE));
            }
    }
    // ---- the first chunks of the window, all waves; the record of zeros; the depth table --------------------------------
    typedef Filler<SRC, NM == 8 ? 1 : 2> Fill;   // (the largest wave tile has registers for one unit)
    const int rounds = (w.slots + Fill::ROUND - 1) / Fill::ROUND, ft = tid & (FT - 1);
    constexpr int BATCH = 4;
    const unsigned mg_rounds = rounds > 1 ? magic_for_device(rounds) : 0u;
    // (every buffer there is: the loads of many rounds share one trip to memory)
    const int first_chunks = min(a.nbuf, a.chunks);
    if constexpr (SRC == ST_NCHW) {
        const WindowSource from{a.src, a.img_bytes, a.src_bytes, a.C1, a.HW, 0, a.wide};
        const int cq = min(first_chunks * 16, (a.C1 + 4) >> 2);
        window_from_nchw_to<NT, 4, true, true>(from, w, cq, magic_for_device(cq), [&](int slot, int c4) { return smem + a.win_off + (c4 >> 6) * a.buf_bytes + slot * ST_PITCH + (c4 & 63); },
                                   ST_PITCH, tid);
    } else
        for (int i0 = tid / FT; i0 < first_chunks * rounds; i0 += 2 * BATCH) {
            Fill some[BATCH];
            int c = fast_div_any(i0, rounds, mg_rounds), r = i0 - c * rounds, rs[BATCH];
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                rs[b] = c < first_chunks ? r : -1;
                if (c < first_chunks) some[b].take(a, w, n1, c, r, ft, smem + a.win_off + c * a.buf_bytes);
                for (r += 2; r >= rounds; r -= rounds) ++c;
            }
#pragma unroll
            for (int b = 0; b < BATCH; ++b)
                if (rs[b] >= 0) some[b].put(w, rs[b], ft);
        }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): what no store waited for must not hold back the main loop
    Fill fill;
    if (tid < 16) *reinterpret_cast<unsigned *>(smem + a.zero_off + tid * 4) = 0;
    // step (UNI: it lies in one tap) or 16-byte chunk -> record offset of its tap's channels, bit of the tap in the lanes' masks
    v2i *const tab = reinterpret_cast<v2i *>(smem + a.tab_off);
    constexpr int EPS = UNI ? 1 : 4;
    for (int i = tid; i < a.stages * SPS * EPS; i += NT) {
        v2i e = {0, 0};   // (past the last weight: zeros)
        if constexpr (UNI) {
            if (i < a.steps) {
                const int c = fast_div_any(i, a.RS, a.mg_RS), tap = i - c * a.RS, r = fast_div_any(tap, a.S, a.mg_S), s = tap - r * a.S;
                e = v2i{(c % a.nbuf) * a.buf_bytes + (r * a.W + s) * a.dil * ST_PITCH, 1 << tap};
            }
        } else if (i < a.nreal) {
            const int tb = fast_div_any(i, a.g16, a.mg_g16), sub = i - tb * a.g16;
            const int rb = fast_div_any(tb, a.S, a.mg_S), s = tb - rb * a.S;
            const int b = fast_div_any(rb, a.R, a.mg_R), r = rb - b * a.R;
            const int ch = b * a.cb + sub * 16;
            e = v2i{((ch >> 6) % a.nbuf) * a.buf_bytes + (r * a.W + s) * a.dil * ST_PITCH + (ch & 63), 1 << (r * a.S + s)};
        }
        tab[i] = e;
    }

    // ---- the lane's pixels: their records (tap (0, 0), first channels) and which taps are in the image -------------------
    const int rswz = (lane >> 2) & 3, half = lane >> 5;
    const int mw = m0 + wm * FM * 32;
    int base[FM];
    unsigned mask[FM];
#pragma unroll
    for (int f = 0; f < FM; ++f) {
        const int m = min(mw + f * 32 + (lane & 31), m1 - 1);
        const int n = fast_div_any(m, a.PQ, a.mg_PQ), pq = m - n * a.PQ;
        const int p = fast_div_any(pq, a.Q, a.mg_Q), q = pq - p * a.Q;
        const int row = p * a.stride - a.pad, col = q * a.stride - a.pad;
        const int seg = n == w.n0 ? -w.lo0 : w.len0 + (n - w.n0 - 1) * a.full8;
        base[f] = a.win_off + (seg + row * a.W + col) * ST_PITCH + (UNI ? half * 16 : 0);
        unsigned cm = 0, mk = 0;
        for (int s = 0; s < a.S; ++s) cm |= (unsigned)((unsigned)(col + s * a.dil) < (unsigned)a.W) << s;
        for (int r = 0; r < a.R; ++r) mk |= ((unsigned)(row + r * a.dil) < (unsigned)a.H ? cm : 0u) << (r * a.S);
        mask[f] = mk;
    }
    const int wrow = (wk * FK * 32 + (lane & 31)) * 64;
    const int wa[2] = {wrow + ((half ^ rswz) << 4), wrow + (((2 + half) ^ rswz) << 4)};

    v16i acc[FK][FM];
#pragma unroll
    for (int i = 0; i < FK; ++i)
#pragma unroll
        for (int f = 0; f < FM; ++f)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][f][v] = 0;

    // Fragment sets alternate per 32-deep half: half h multiplies set h % 2 while the reads of half h+1 fill the other one.
    v4i wf[2][FK], af[2][FM];
    v2i te[UNI ? 1 : 2];
    int bad[UNI ? 1 : 2][FM];
    auto read_table = [&](int step) {
        const v2i *e = tab + (size_t)step * EPS + (UNI ? 0 : half);
        te[0] = e[0];
        if constexpr (!UNI) te[1] = e[2];
    };
    auto find = [&]() {   // the blocks' records for the step of the table entry at hand
#pragma unroll
        for (int x = 0; x < (UNI ? 1 : 2); ++x)
#pragma unroll
            for (int f = 0; f < FM; ++f) bad[x][f] = (mask[f] & (unsigned)te[x][1]) ? base[f] + te[x][0] : a.zero_off;
    };
    // item t of a half: weight block 0, every pixel block, the other weight blocks
    auto read_item = [&](int t, int h, const unsigned char *st, v4i(&wr)[FK], v4i(&ar)[FM]) {
        if (t >= 1 && t <= FM)
            ar[t - 1] = *reinterpret_cast<const v4i *>(__builtin_assume_aligned(smem + (UNI ? bad[0][t - 1] + h * 32 : bad[UNI ? 0 : h][t - 1]), 16));
        else {
            const int i = t == 0 ? 0 : t - FM;
            wr[i] = *reinterpret_cast<const v4i *>(__builtin_assume_aligned(st + wa[h] + i * 2048, 16));
        }
    };
    // read t of the next half goes behind MFMA read_slot(t) of this one
    auto read_slot = [](int t) constexpr { return NR > NM ? (t > NR - NM ? t - (NR - NM) : 0) : t; };
    auto group_step = [&](int j, int q) { return j * SPS + q * DS + grp; };
    const int last_stage = a.stages - 1;

    if (wave < DW) {
        if (NST - 1 <= a.stages) st_wait_dma<(NST - 2) * L>();
        else st_wait_dma<0>();
    }
    st_barrier();
    read_table(group_step(0, 0));
    find();
#pragma unroll
    for (int t = 0; t < NR; ++t) read_item(t, 0, smem + grp * TK * 64, wf[0], af[0]);

    // The loop twice, once for the waves that transfer and once for those that fill: the compiler's waits for the
    // pixels would otherwise stand in the transferring waves' way too.
    auto main_loop = [&](auto fills) {
        constexpr bool FILLS = decltype(fills)::value;
        // fill state: the round that is asked for next, the one that is on its way, and the chunks that are stored whole
        const int fill_chunks = w.slots > 0 ? a.chunks : 0;   // (a tile may see nothing but the border)
        int fc = first_chunks, fr = 0, stored = w.slots > 0 ? first_chunks : a.chunks, coming = -1;
        // stages that a round's loads may take: as many as let all rounds of a chunk go by in the time of a chunk
        const int delay = max(1, min(3, a.RS / (SPS * (rounds + 1))));
        int put_at = 0;
        unsigned char *const win = smem + a.win_off;
        for (int j = 0; j < a.stages; ++j) {
            const unsigned char *cur = smem + (j % NST) * ST_STAGE + grp * TK * 64;
            const unsigned char *nxt = smem + ((j + 1) % NST) * ST_STAGE + grp * TK * 64;
            const int jn = j + NST - 1;
            const unsigned slot = lds0 + (unsigned)((jn % NST) * ST_STAGE);
            if constexpr (FILLS) {
                if (coming >= 0 && j >= put_at) {
                    fill.put(w, coming, ft);
                    if (coming + 1 >= rounds) ++stored;
                    coming = -1;
                }
                // a buffer is free once the chunk it held lies behind the first step of this stage
                if (coming < 0 && fc < fill_chunks && fc < fast_div_any(j * SPS, a.RS, a.mg_RS) + a.nbuf) {
                    fill.take(a, w, n1, fc, fr, ft, win + (fc % a.nbuf) * a.buf_bytes);
                    coming = fr;
                    put_at = j + delay;
                    if (++fr >= rounds) fr = 0, ++fc;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                const int par = h & 1, qs = h >> 1;
                const bool last = h == NH - 1;
                const unsigned char *nst = last ? nxt : cur + ((h + 1) >> 1) * DS * TK * 64;
                if (par == 0) read_table(qs + 1 < QS ? group_step(j, qs + 1) : group_step(min(j + 1, last_stage), 0));
#pragma unroll
                for (int g = 0; g < NM; ++g) {
                    acc[g / FM][g % FM] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[par][g / FM], af[par][g % FM], acc[g / FM][g % FM], 0, 0, 0);
                    if (last && g == 0) {
                        // stage j+1 has landed, its chunks are stored, and everyone holds the rest of stage j in registers
                        if constexpr (!FILLS) {
                            if (jn < a.stages) st_wait_dma<(NST - 2) * L>();
                            else st_wait_dma<0>();
                        } else if (j < last_stage) {
                            const int need = min(fast_div_any((j + 2) * SPS - 1, a.RS, a.mg_RS), a.chunks - 1);
                            if (stored <= need) {   // (few steps per chunk: the rounds do not all fit behind the stages)
                                if (coming >= 0) {
                                    fill.put(w, coming, ft);
                                    if (coming + 1 >= rounds) ++stored;
                                    coming = -1;
                                }
                                while (stored <= need) {
                                    Fill now;
                                    now.take(a, w, n1, fc, fr, ft, win + (fc % a.nbuf) * a.buf_bytes);
                                    now.put(w, fr, ft);
                                    if (++fr >= rounds) fr = 0, ++fc, ++stored;
                                }
                                __builtin_amdgcn_s_waitcnt(0x0F70);   // (what no put() waited for must not hold back the stages behind)
                            }
                        }
                        st_barrier();
                    }
                    if (par == 1 && g == 0) find();
                    if constexpr (!FILLS) {
                        // this stage's transfers, all before its barrier
                        constexpr int SLOTS = (NH - 1) * NM;
                        if (!last && jn < a.stages)
#pragma unroll
                            for (int u = 0; u < L; ++u)
                                if (u * SLOTS / L == h * NM + g) dma_stage_part(u, slot);
                    }
                    // (after the last stage the reads hit a stale slot; the values are never used)
#pragma unroll
                    for (int t = 0; t < NR; ++t)
                        if (read_slot(t) == g) read_item(t, par ^ 1, nst, wf[par ^ 1], af[par ^ 1]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    };
    if (wave < DW) main_loop(std::false_type{});
    else main_loop(std::true_type{});

    // ---- result [N][K][P][Q]: through LDS, so that every store instruction writes whole rows of the tile ----------------------
    // (Straight from the blocks it is sixteen 4-byte stores per lane, two 128-byte runs each, and a compute unit takes twelve
    // cycles for a store instruction whatever its width: 5.8 us for a 256 x 256 tile on an idle chip, 1.3 us in 16-byte
    // stores.)  A pass takes one row block of every wave, all depth groups side by side; passes alternate between two buffers.
    if constexpr (SRC == ST_NCHW) {
        constexpr int PITCH = FM * WM * 128 + 32;                  // bytes of a row; four rows on are 32 banks on
        constexpr int ROWS = WK * 32, GROUP = ROWS * PITCH, BUF = DS * GROUP;
        constexpr int LPR = FM * WM * 8;                           // lanes of a row, four pixels each
        constexpr int RPI = 64 / LPR < 1 ? 1 : 64 / LPR;           // rows of a store instruction
        static_assert(LPR <= 64, "a wave stores a row of the tile");
        constexpr int NS = ROWS / (NW * RPI);                      // store instructions of a wave in a pass
        static_assert(ROWS % (NW * RPI) == 0 && 32 % (NS * RPI) == 0, "a wave's rows belong to one row of waves");
        const int quad = lane % LPR, mq = m0 + quad * 4;
        const int n = fast_div_any(min(mq, a.M - 1), a.PQ, a.mg_PQ), pq = mq - n * a.PQ;
        const unsigned row = (unsigned)a.PQ * 4u;
        const unsigned off = ((unsigned)(n - w.n0) * (unsigned)a.K * (unsigned)a.PQ + (unsigned)pq) * 4u + (unsigned)(lane / LPR) * row;
        const int ok = min(max(m1 - mq, 0), 4);
        const bool whole = ok == 4 && pq + 3 < a.PQ;
        // a wave's rows follow one another: their places are scalar, and which of them exist is asked for the tile as a whole
        const int r0 = wave * NS * RPI, kw = k0 + (r0 >> 5) * FK * 32 + (r0 & 31);
        char *const to0 = reinterpret_cast<char *>(a.out) + ((size_t)w.n0 * a.K + (size_t)kw) * row;
        const auto base = past_base(to0);
        const unsigned char *const from = smem + (r0 + lane / LPR) * PITCH + quad * 16;
        st_barrier();
        auto passes = [&](auto inside, auto past) {
#pragma unroll
            for (int i = 0; i < FK; ++i) {
                unsigned char *const mine = smem + (i & 1) * BUF + grp * GROUP + (wk * 32 + 4 * half) * PITCH + (wm * FM * 32 + (lane & 31)) * 4;
#pragma unroll
                for (int f = 0; f < FM; ++f)
#pragma unroll
                    for (int v = 0; v < 16; ++v) *reinterpret_cast<int *>(mine + (8 * (v >> 2) + (v & 3)) * PITCH + f * 128) = acc[i][f][v];
                st_barrier();
                v4i t[NS];
#pragma unroll
                for (int r = 0; r < NS; ++r) {
                    const unsigned char *const at = from + (i & 1) * BUF + r * RPI * PITCH;
                    t[r] = *reinterpret_cast<const v4i *>(__builtin_assume_aligned(at, 16));
#pragma unroll
                    for (int d = 1; d < DS; ++d) t[r] += *reinterpret_cast<const v4i *>(__builtin_assume_aligned(at + d * GROUP, 16));
                }
                auto there = [&](int r) { return decltype(inside)::value || kw + i * 32 + r * RPI + lane / LPR < a.K; };
                if (whole) {
#pragma unroll
                    for (int r = 0; r < NS; ++r) {
                        if (!there(r)) continue;
                        if constexpr (decltype(past)::value != PAST_NONE) store_past16<decltype(past)::value>(base, off, (unsigned)(i * 32 + r * RPI) * row, t[r]);
                        else *reinterpret_cast<v4i_a4 *>(to0 + (size_t)(i * 32 + r * RPI) * row + off) = t[r];
                    }
                } else if (ok) {   // (two images meet in the four pixels -- or more, of fewer than four -- or the tile ends)
#pragma unroll
                    for (int r = 0; r < NS; ++r) {
                        char *const to = to0 + (size_t)(i * 32 + r * RPI) * row;
                        if (!there(r)) continue;
                        unsigned o = off;
                        int q = pq;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (e < ok) *reinterpret_cast<int32_t *>(to + o) = t[r][e];
                            o += 4;
                            if (++q == a.PQ) q = 0, o += (unsigned)(a.K - 1) * row;
                        }
                    }
                }
            }
        };
        if (k0 + TK > a.K) passes(std::false_type{}, PastHow<PAST_NONE>{});
        else if (a.past == PAST_THROUGH) passes(std::true_type{}, PastHow<PAST_THROUGH>{});
        else if (a.past == PAST_STREAM) passes(std::true_type{}, PastHow<PAST_STREAM>{});
        else passes(std::true_type{}, PastHow<PAST_NONE>{});
        return;
    }

    // ---- result [N][P][Q][K]: a lane's four values of a piece are four channels of a pixel ----------------------------------
    // D block (i, f): column = lane%32 (pixel), row = 8*(v/4) + 4*(lane/32) + v%4 (channel); piece = four rows of a block
    constexpr int NP = NM * 4, OWN = NP / DS;
    static_assert(NP % DS == 0, "every depth group finishes the same number of pieces");
    auto store_piece = [&](int x, const v4i &t) {
        const int m = mw + x / 4 % FM * 32 + (lane & 31), k = k0 + wk * FK * 32 + x / (4 * FM) * 32 + x % 4 * 8 + 4 * half, left = a.K - k;
        if (m >= m1 || left <= 0) return;
        int32_t *px = a.out + (size_t)m * a.K + k;
        if ((a.K & 3) == 0 || left >= 4) *reinterpret_cast<v4i_a4 *>(px) = t;   // (rows of K values begin on any dword)
        else
            for (int v = 0; v < 3; ++v)
                if (v < left) px[v] = t[v];
    };
    auto piece = [&](int x) {
        const v16i &b = acc[x / (4 * FM)][x / 4 % FM];
        const int g = x % 4;
        return v4i{b[4 * g], b[4 * g + 1], b[4 * g + 2], b[4 * g + 3]};
    };
    if constexpr (DS == 1) {
#pragma unroll
        for (int x = 0; x < NP; ++x) store_piece(x, piece(x));
    } else {
        // every group leaves the pieces it does not own in LDS (nothing there is read any more) and adds up its own
        st_barrier();
        v4i *const xch = reinterpret_cast<v4i *>(smem);
        auto at = [&](int owner, int from, int p) { return xch + (((owner * (DS - 1) + (from < owner ? from : from - 1)) * NWM + wi) * OWN + p) * 64 + lane; };
        v4i own[OWN];
#pragma unroll
        for (int o = 0; o < DS; ++o) {
#pragma unroll
            for (int p = 0; p < OWN; ++p) {
                if (o == grp) own[p] = piece(o * OWN + p);
                else *at(o, grp, p) = piece(o * OWN + p);
            }
        }
        st_barrier();
#pragma unroll
        for (int s = 0; s < DS - 1; ++s) {
            const int from = s < grp ? s : s + 1;
#pragma unroll
            for (int p = 0; p < OWN; ++p) own[p] += *at(grp, from, p);
        }
#pragma unroll
        for (int p = 0; p < OWN; ++p) store_piece(grp * OWN + p, own[p]);
    }
}

// FK, FM, WK, WM, DS, NST
#define C2I8_STREAM_LIST(X) \
    X(4, 2, 2, 4, 1, 4) /* 256 x 256 */ \
    X(4, 2, 1, 4, 2, 4) /* 128 x 256 */ \
    X(2, 2, 2, 2, 2, 4) /* 128 x 128 */ \
    X(2, 2, 1, 4, 2, 4) /*  64 x 256 */ \
    X(2, 2, 1, 2, 4, 4) /*  64 x 128 */ \
    X(1, 2, 1, 2, 4, 4) /*  32 x 128 */ \
    X(1, 2, 1, 1, 8, 4) /*  32 x  64 */

struct StreamTile {
    int fk, fm, wk, wm, ds, nst;
    int tk() const { return fk * wk * 32; }
    int tm() const { return fm * wm * 32; }
    int waves() const { return wk * wm * ds; }
    int sps() const { return waves() * 32 / tk(); }
    int ring() const { return nst * waves() * 2048; }
    int exchange() const   // bytes that the result takes on its way out: the depth groups' meeting, or a pass (or two) of rows
    {
        const int pieces = (ds - 1) * wk * wm * fk * fm * 4 * 1024, pass = ds * wk * 32 * (fm * wm * 128 + 32);
        const int rows = (fk > 1 ? 2 : 1) * pass;
        return pieces > rows ? pieces : rows;
    }
};
constexpr StreamTile kStreamTiles[] = {
#define C2I8_ROW(...) {__VA_ARGS__},
    C2I8_STREAM_LIST(C2I8_ROW)
#undef C2I8_ROW
};
constexpr int kNumStreamTiles = sizeof(kStreamTiles) / sizeof(kStreamTiles[0]);

template <int FK, int FM, int WK, int WM, int DS, int NST>
hipError_t launch_stream_tile(const StreamArgs &a, int source, bool uni, size_t lds, hipStream_t st)
{
    void (*kern)(StreamArgs);
    switch (source * 2 + uni) {
        case 0: kern = conv_stream_kernel<FK, FM, WK, WM, DS, NST, ST_NCHW, false>; break;
        case 1: kern = conv_stream_kernel<FK, FM, WK, WM, DS, NST, ST_NCHW, true>; break;
        case 2: kern = conv_stream_kernel<FK, FM, WK, WM, DS, NST, ST_NHWC, false>; break;
        default: kern = conv_stream_kernel<FK, FM, WK, WM, DS, NST, ST_NHWC, true>; break;
    }
    static bool raised[4];
    if (!raised[source * 2 + uni]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)ST_LDS_LIMIT);
        if (e != hipSuccess) return e;
        raised[source * 2 + uni] = true;
    }
    return launch(kern, dim3((unsigned)(a.tiles_k * a.tiles_m)), dim3(WK * WM * DS * 64), lds, st, a);
}

struct StreamPlan {
    StreamArgs a;
    int tile, source;
    bool uni;
    size_t lds;
};

// What does not depend on the tile.
struct StreamShape {
    int source, RS, steps, chunks, nreal, sub;
    bool uni;
};
bool stream_shape(const ResidentProblem &r, StreamShape *o)
{
    const GemmProblem &g = r.g;
    if (g.mode != ACT_BLOCKED || g.R * g.S > 31 || g.il_d || g.act_out || r.raw_weights || r.pixel_major != g.out_nhwc || g.Q <= 0 || g.PQ % g.Q || g.M <= 0) return false;
    if (g.cb != 16 && g.cb != 32 && (g.cb < 64 || g.cb % 64)) return false;
    o->source = r.pixel_major ? ST_NHWC : ST_NCHW;
    o->RS = g.R * g.S;
    o->uni = g.cb % 64 == 0;
    o->sub = g.cb / 64;
    o->chunks = (r.C + 63) / 64;   // (what a block has beyond them is zeros on both sides)
    o->nreal = g.Cb * o->RS * (g.cb / 16);
    o->steps = o->uni ? o->chunks * o->RS : (o->nreal + 3) / 4;
    if (r.img_bytes > 0x7FFFFFFFLL || (long long)r.H * r.W > (1LL << 28) || (long long)r.N * r.img_bytes < 64) return false;
    if ((long long)g.Q * g.stride > (1LL << 28) || (long long)(g.PQ / g.Q) * g.stride > (1LL << 28)) return false;
    return (long long)g.K * g.depth <= 0x7FFFFFFFLL;
}

// Buffers without which a stage could need a chunk whose buffer is still read: the chunks that two stages can touch.
int least_buffers(const StreamShape &sh, int sps)
{
    const int touched = (2 * sps + sh.RS - 2) / sh.RS + 1;   // (at least what stage 0 alone needs)
    return touched < sh.chunks ? touched : sh.chunks;
}
long long stream_lds(const StreamTile &d, const StreamShape &sh, int nbuf, long long slots)
{
    const long long stages = (sh.steps + d.sps() - 1) / d.sps();
    const long long main = (long long)d.ring() + 64 + nbuf * slots * ST_PITCH + stages * d.sps() * (sh.uni ? 8 : 32);
    return main > d.exchange() ? main : d.exchange();
}

bool stream_plan(const ResidentProblem &r, int tile, int mper, StreamPlan *out)
{
    const GemmProblem &g = r.g;
    const StreamTile &d = kStreamTiles[tile];
    StreamShape sh;
    if (mper < 1 || mper > d.tm() || !stream_shape(r, &sh)) return false;
    const int dil = g.dil > 0 ? g.dil : 1;
    const long long HW = (long long)r.H * r.W, PQ = g.PQ;
    StreamArgs &a = out->a;
    a = StreamArgs{};
    auto magic = [](long long v) { return v <= 1 ? 0u : magic_for(v); };
    a.out = g.out;
    a.K = g.K, a.M = g.M, a.PQ = g.PQ, a.Q = g.Q;
    a.C1 = r.C - 1;
    a.H = r.H, a.W = r.W, a.HW = (int)HW;
    a.stride = g.stride, a.pad = r.pad, a.dil = dil;
    a.R = g.R, a.S = g.S, a.RS = sh.RS;
    a.depth = g.depth;
    a.steps = sh.steps;
    a.stages = (sh.steps + d.sps() - 1) / d.sps();
    a.cb = g.cb, a.g16 = g.cb / 16, a.nreal = sh.nreal, a.sub = sh.sub;
    a.chunks = sh.chunks;
    a.img_bytes = r.img_bytes;
    a.src_bytes = r.img_bytes * r.N;
    a.pstride = r.pixel_bytes;
    a.mper = mper;
    {
        const long long row = (PQ / g.Q - 1) * g.stride - r.pad + (g.R - 1) * dil, col = (long long)(g.Q - 1) * g.stride - r.pad + (g.S - 1) * dil;
        const long long end = row >= r.H ? HW : row * r.W + (col > r.W - 1 ? r.W - 1 : col < -1 ? -1 : col) + 1;
        if (end <= 0) return false;   // no pixel of the image is read at all
        a.full8 = (int)((end + 7) & ~7LL);
    }
    const long long images = mper / PQ + 2;
    if (images * PQ * g.K * 4 >= (1LL << 32) || images * r.img_bytes > 0x7FFFFFFFLL) return false;   // 32-bit offsets from the tile's first image
    const long long slots = window_walk(r).most(mper);
    a.wide = window_wide_units(HW);
    const int least = least_buffers(sh, d.sps());
    int nbuf = sh.chunks;
    while (nbuf > least && stream_lds(d, sh, nbuf, slots) > ST_LDS_LIMIT) --nbuf;
    const long long lds = stream_lds(d, sh, nbuf, slots);
    if (lds > ST_LDS_LIMIT || (long long)((g.R - 1) * r.W + g.S - 1) * dil * ST_PITCH > (1LL << 30)) return false;
    a.nbuf = nbuf;
    a.buf_bytes = (int)(slots * ST_PITCH);
    a.zero_off = d.ring();
    a.win_off = a.zero_off + 64;
    a.tab_off = a.win_off + nbuf * a.buf_bytes;
    // Past the caches: whole 64-byte sectors per store instruction, of planes and tiles that hold whole ones (37 drawn layers 0.97 of the
    // time, the worst 1.03); other planes of whole 16-byte pieces from 8 to 28 MB (0.98, 1.03) and above 256 (0.95, 0.97).  (From there to
    // 256 MB they take up to 1.28, below 8 up to 1.04, planes of other sizes up to 1.13.)  All that non-temporal; up to 28 MB they are
    // written through, which is level or faster (5 layers of whole sectors 0.99 - 1.00, 4 of quads 0.99 - 1.00) and better for their reader.
    const double bytes = 4.0 * g.M * g.K;
    const bool sectors = PQ % 16 == 0 && mper % 16 == 0 && (reinterpret_cast<uintptr_t>(g.out) & 63) == 0;
    const bool quads = PQ % 4 == 0 && mper % 4 == 0 && bytes > 8e6;
    a.past = sectors || quads ? past_caches(bytes) : PAST_NONE;
    if (sectors && a.past == PAST_NONE) a.past = PAST_STREAM;
    const long long tk = (g.K + d.tk() - 1) / d.tk(), tm = ((long long)g.M + mper - 1) / mper;
    if (tk * tm > 0x7FFFFFFFLL) return false;
    a.tiles_k = (int)tk;
    a.tiles_m = (int)tm;
    {   // what an XCD's L2 has to bring in: its share of the tile list in either order
        const double per = (double)(tk * tm) / 8, weights = (double)g.K * g.depth, input = (double)a.src_bytes;
        auto share = [&](double fast, double slow, double fast_bytes, double slow_bytes) {
            const double across = per < fast ? per : fast, down = per / fast < 1 ? 1 : per / fast;
            return across / fast * fast_bytes + (down < slow ? down : slow) / slow * slow_bytes;
        };
        a.m_fastest = share((double)tm, (double)tk, input, weights) < share((double)tk, (double)tm, weights, input);
        a.tiles_fast = a.m_fastest ? a.tiles_m : a.tiles_k;
    }
    a.mg_PQ = magic(g.PQ), a.mg_Q = magic(g.Q), a.mg_tiles_fast = magic(a.tiles_fast), a.mg_full8 = magic(a.full8);
    a.mg_g16 = magic(a.g16), a.mg_S = magic(g.S), a.mg_R = magic(g.R), a.mg_RS = magic(sh.RS);
    out->tile = tile;
    out->source = sh.source;
    out->uni = sh.uni;
    out->lds = (size_t)lds;
    return true;
}

// Launch time in microseconds, fitted per tile to 128000 measured launches of 13400 layers (kept weights, NCHW; a third of the
// layers held back: mean error 4 %, 7 % for the largest tile, which leaves 208 images 256 x 28 x 28 -> 219 on the stored path: 134 us, here 118).
// It serves NHWC and dilated calls too, from which nothing was fitted: 606 of them that it sends here take 0.64 (dilated) and 0.86
// (NHWC) of the best other launch in the mean, 0.94 where K is not a multiple of four (while those results went value by value, in no term; one in six lost
// more than 5 % there, of the others one in fifty; a term for them sent 200 calls elsewhere, at 0.999 in the mean).  A launch; per
// round of workgroups (one per compute unit) its fixed part, its ring stages, the window bytes it begins with and those that come
// later; the result's bytes on planes of whole 64-byte sectors and on others; what the stages of all workgroups share.
struct StreamFit {
    double launch, round, stage, first, rest, aligned, other, shared;
};
constexpr StreamFit kStreamFit[] = {
    {3.35, 7.66, 0.549, 1.03e-05, 6.29e-05, 2.09e-05, 3.23e-05, 0.236},
    {2.69, 6.36, 0.653, 1.44e-05, 5.4e-05, 1.61e-05, 3.08e-05, 0.153},
    {2.72, 4.48, 0.434, 1.86e-05, 5.56e-05, 1.1e-05, 3.07e-05, 0.0795},
    {2.45, 4.55, 0.681, 1.98e-05, 4.7e-05, 7.57e-06, 2.79e-05, 0.178},
    {2.36, 4.22, 0.455, 2.1e-05, 4.93e-05, 1.06e-05, 3.65e-05, 0.0876},
    {2.12, 3.62, 0.647, 1.92e-05, 3.89e-05, 3.85e-06, 3.46e-05, 0.107},
    {2.15, 3.53, 0.475, 2.25e-05, 4.82e-05, 2.29e-05, 5.84e-05, 0.0652},
};
// The estimate without its window, which only adds to it.
__attribute__((always_inline)) inline double stream_cost_bare(const ResidentProblem &r, const StreamTile &d, const StreamFit &f, long long wgs, int stages, int mper)
{
    const double rounds = (double)((wgs + 255) / 256), per = wgs / 256.0, channels = r.g.K < d.tk() ? r.g.K : d.tk();
    const double result = 4.0 * channels * mper;
    return f.launch + rounds * (f.round + f.stage * stages) + per * ((r.g.PQ % 16 == 0 ? f.aligned : f.other) * result + f.shared * stages);
}
// What the window adds: chunks there are buffers for, and the others.  (1e300: too few buffers fit.)
__attribute__((always_inline)) inline double stream_cost_window(const ResidentProblem &r, const StreamShape &sh, const StreamTile &d, const StreamFit &f, long long wgs, int slots)
{
    int nbuf = sh.chunks;
    while (nbuf > 1 && stream_lds(d, sh, nbuf, slots) > ST_LDS_LIMIT) --nbuf;
    if (nbuf < least_buffers(sh, d.sps()) || stream_lds(d, sh, nbuf, slots) > ST_LDS_LIMIT) return 1e300;
    const double first = 64.0 * slots * nbuf, rest = 64.0 * slots * (sh.chunks - nbuf);
    return (double)((wgs + 255) / 256) * (f.first * first + f.rest * rest);
}

hipError_t launch_plan(const ResidentProblem &r, const StreamPlan &p, hipStream_t st)
{
    StreamArgs a = p.a;
    a.src = r.src;
    a.wq = r.g.wq;
    a.out = r.g.out;
    int index = 0;
#define C2I8_CASE(fk, fm, wk, wm, ds, nst) \
    if (p.tile == index++) return launch_stream_tile<fk, fm, wk, wm, ds, nst>(a, p.source, p.uni, p.lds, st);
    C2I8_STREAM_LIST(C2I8_CASE)
#undef C2I8_CASE
    return hipErrorInvalidValue;
}

}  // namespace

bool stream_pick(const ResidentProblem &r, WindowWalk &walk, double limit, double smallest, ResidentChoice *c)
{
    StreamShape sh;
    // (fewer taps: a chunk of the window serves too few stages, and the estimate was fitted on 3x3 and 5x5 kernels)
    if (!stream_shape(r, &sh) || sh.RS < 9) return false;
    ResidentChoice best[3] = {{0, 0, limit}, {0, 0, limit}, {0, 0, limit}};
    bool larger = false;   // a larger tile is below the limit
    auto pick_in = [&](const StreamTile &d, const StreamFit &f, int t) __attribute__((always_inline)) {   // (a tile known to the compiler: its divisions are shifts)
        const long long M = r.g.M;
        const int tk = (r.g.K + d.tk() - 1) / d.tk(), stages = (sh.steps + d.sps() - 1) / d.sps();
        int tried[10], n = 0;
        auto consider = [&](long long mper) {   // whole rounds of workgroups, whole images, the tile
            if (mper > d.tm()) mper = d.tm();
            if (mper < 1) return;
            for (int i = 0; i < n; ++i)
                if (tried[i] == (int)mper) return;
            tried[n++] = (int)mper;
            const long long wgs = (long long)tk * (((unsigned)M + (unsigned)mper - 1) / (unsigned)mper);
            ResidentChoice x{t, (int)mper, stream_cost_bare(r, d, f, wgs, stages, (int)mper)};
            if (x.us >= best[2].us) return;   // (most counts end here, before their windows are walked)
            x.us += stream_cost_window(r, sh, d, f, wgs, walk.sampled(x.mper));
            larger = larger || (t != kNumStreamTiles - 1 && x.us < limit);
            for (int k = 0; k < 3; ++k)
                if (x.us < best[k].us) {
                    for (int j = 2; j > k; --j) best[j] = best[j - 1];
                    best[k] = x;
                    break;
                }
        };
        for (int rounds = 1; rounds <= 3; ++rounds) {
            const int wide = 256 * rounds / tk;
            const long long m = wide > 0 ? ((unsigned)M + (unsigned)wide - 1) / (unsigned)wide : d.tm();
            consider(m);
            consider((m + 31) / 32 * 32);
        }
        consider(d.tm());
        consider(r.g.PQ);
    };
    int index = 0;
#define C2I8_CASE(fk, fm, wk, wm, ds, nst) pick_in(StreamTile{fk, fm, wk, wm, ds, nst}, kStreamFit[index], index), ++index;
    C2I8_STREAM_LIST(C2I8_CASE)
#undef C2I8_CASE
    if (!larger && best[0].us >= smallest * limit) return false;
    for (const ResidentChoice &x : best) {   // (the window was sampled: the plan knows whether it fits)
        StreamPlan p, whole;
        if (x.mper > 0 && stream_plan(r, x.tile, x.mper, &p)) {
            *c = x;
            // Tiles that begin inside a 64-byte sector write it in two parts: on planes of whole sectors the count goes up to whole ones,
            // where that is at most an eighth more, cuts no image that was divided evenly, and leaves the window as many buffers.  41
            // layers, mean 1.033 (72 images 500 x 55 x 55 -> 64 stride 2: 111 -> 112 pixels, 63.8 -> 55.5 us), the worst 0.974; up to
            // 0.89 without the conditions.
            const int up = (x.mper + 15) / 16 * 16;
            if (r.g.PQ % 16 == 0 && !r.pixel_major && up != x.mper && r.g.PQ % x.mper && up * 8 <= x.mper * 9 && up <= kStreamTiles[x.tile].tm() &&
                stream_plan(r, x.tile, up, &whole) && whole.a.nbuf == p.a.nbuf)
                c->mper = up;
            return true;
        }
    }
    return false;
}

int stream_num_tiles() { return kNumStreamTiles; }
TileInfo stream_tile_info(int tile) { return TileInfo{kStreamTiles[tile].tk(), kStreamTiles[tile].tm(), kStreamTiles[tile].waves() * 64, kStreamTiles[tile].sps()}; }

struct StreamKey {
    GemmKey g;
    int v[12];
};

bool stream_applies(const ResidentProblem &r, int tile, int mper)
{
    StreamPlan p;
    return stream_plan(r, tile, mper, &p);
}

hipError_t launch_stream(const ResidentProblem &r, int tile, int mper, hipStream_t st)
{
    static thread_local PlanTable<StreamKey, StreamPlan, 64> plans;
    const int out64 = (reinterpret_cast<uintptr_t>(r.g.out) & 63) == 0;
    const StreamKey key{gemm_key(r.g), {r.N, r.C, r.H, r.W, r.pad, r.pixel_major, r.pixel_bytes, 0, out64, tile, mper, (int)r.img_bytes}};
    const StreamPlan *kept = plans.get(key, [&](StreamPlan *p) { return stream_plan(r, tile, mper, p); });
    return kept ? launch_plan(r, *kept, st) : hipErrorInvalidValue;
}

hipError_t launch_stream_forced(const ResidentProblem &r, int tile, int mper, hipStream_t st)
{
    StreamPlan p;
    return stream_plan(r, tile, mper, &p) ? launch_plan(r, p, st) : hipErrorInvalidValue;
}

}  // namespace c2i8
