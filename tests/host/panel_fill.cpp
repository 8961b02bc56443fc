// Host run of the panel kernel's window (panel_fill.h): the slots of a workgroup's output pixels, filled by its threads one after the
// other, from tensors that start behind and end before a page without access.  Checked: nothing is read outside the tensor or written
// outside the window, and every tap of every pixel finds its input, or the border's zero, at its distance from the pixel's first one.
#include <algorithm>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <vector>

// (plain C++: the device's own names as ordinary functions)
using std::max;
using std::min;
static inline unsigned host_perm(unsigned hi, unsigned lo, unsigned sel)
{
    const unsigned long long v = ((unsigned long long)hi << 32) | lo;
    unsigned r = 0;
    for (int i = 0; i < 4; ++i) {
        const unsigned s = (sel >> (8 * i)) & 255;
        r |= (s < 8 ? (unsigned)((v >> (8 * s)) & 255) : 0u) << (8 * i);
    }
    return r;
}
static inline unsigned __umulhi(unsigned a, unsigned b) { return (unsigned)(((unsigned long long)a * b) >> 32); }
static struct { unsigned x; } threadIdx;
#define __builtin_amdgcn_perm host_perm
#define __builtin_amdgcn_wave_barrier() ((void)0)
#include "../../paper_2104_04731_amd/csrc/panel_fill.h"

using namespace c2i8;

static unsigned rnd_state = 54321;
static int rnd(int lo, int hi)
{
    rnd_state = rnd_state * 1664525u + 1013904223u;
    return lo + (int)((rnd_state >> 8) % (unsigned)(hi - lo + 1));
}
static unsigned magic(int d) { return d <= 1 ? 0u : magic_for(d); }

template <typename Fill>
static void fill_window(const VirtualImage &v, const int8_t *src, int lo, int last, int octs, int first, int chunks, unsigned char *win)
{
    const int n0 = lo / v.Wv / v.Hv;
    std::vector<unsigned char> tab((size_t)octs * Fill::ENTRY, 0xEE);
    const PanelWindow w = panel_window(v, src, n0, lo, last);
    if (w.octs != octs) exit(3);
    for (int t = 0; t < 256; ++t) Fill::table(v, w, n0, lo, tab.data(), t, 256);
    for (int r = 0; r < Fill::rounds(w, chunks); ++r)
        for (int t = 0; t < 256; ++t) {
            Fill f;
            if (w.last) f.template take<true>(v, w, tab.data(), first, chunks, r, t);
            else f.template take<false>(v, w, tab.data(), first, chunks, r, t);
            f.put(w, tab.data(), chunks, r, win, octs * 8 * 80, 80, t);
        }
}

int main()
{
    const size_t page = 4096, room = 1 << 20;
    unsigned char *const map = (unsigned char *)mmap(nullptr, room + 2 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (map == MAP_FAILED || mprotect(map, page, PROT_NONE) || mprotect(map + page + room, page, PROT_NONE)) return 2;
    std::vector<unsigned char> win;
    int tiles = 0, problems = 0;
    for (int it = 0; it < 9000; ++it) {
        const int C = it % 3 ? rnd(1, 40) : rnd(60, 150), H = rnd(1, it % 5 ? 14 : 2), W = rnd(1, it % 5 ? 19 : 9), N = rnd(1, 9), R = rnd(1, 5), S = rnd(1, 5), st = rnd(1, 3), pad = rnd(0, 4), dil = rnd(1, 3);
        if (H + 2 * pad < dil * (R - 1) + 1 || W + 2 * pad < dil * (S - 1) + 1) continue;
        const int P = (H + 2 * pad - dil * (R - 1) - 1) / st + 1, Q = (W + 2 * pad - dil * (S - 1) - 1) / st + 1;
        const long long bytes = (long long)N * C * H * W;
        const int HW = H * W, PQ = P * Q, M = N * PQ, mper = it & 8 ? rnd(1, 448) : 16 * rnd(1, 28);
        if (bytes < 16 || bytes > (long long)room || !virtual_image_fits(R, S, dil, H, W, pad, N, (long long)C * HW)) continue;
        ++problems;
        unsigned char *const src = it & 1 ? map + page : map + page + room - bytes;
        for (long long i = 0; i < bytes; ++i) src[i] = (unsigned char)(i * 31 + i / 253 + it + 1);
        const VirtualImage v{W + pad, H + pad, N, C, H, W, HW, pad, (C + 63) / 64, C, (long long)C * HW, bytes, magic(W + pad), magic(H + pad)};
        auto first = [&](int m) { return (m / PQ * v.Hv + m % PQ / Q * st) * v.Wv + m % PQ % Q * st; };
        const int span = ((R - 1) * v.Wv + S - 1) * dil;
        const long long most = window_slots(mper, PQ, Q, st, v.Wv, v.Hv, span);
        for (int m0 = 0; m0 < M; m0 += mper) {
            const int m1 = min(m0 + mper, M), lo = first(m0), octs = (first(m1 - 1) + span - lo + 8) >> 3;
            if (8 * octs > most) return printf("%d slots, %lld planned: N %d H %d W %d %dx%d stride %d pad %d dil %d mper %d tile %d\n", 8 * octs, most, N, H, W, R, S, st, pad, dil, mper, m0), 1;
            const int at_once = rnd(1, v.chunks);
            for (int part = 0; part < v.chunks; part += at_once)
                for (int nhwc = 0; nhwc < 2; ++nhwc) {
                    const int chunks = min(at_once, v.chunks - part);
                    const size_t bytes_of = (size_t)octs * 8 * 80;
                    win.assign(bytes_of * chunks + 256, 0xEE);
                    if (nhwc) fill_window<PanelFill<true>>(v, (const int8_t *)src, lo, first(m1 - 1) + span, octs, part, chunks, win.data());
                    else fill_window<PanelFill<false>>(v, (const int8_t *)src, lo, first(m1 - 1) + span, octs, part, chunks, win.data());
                    for (size_t i = bytes_of * chunks; i < win.size(); ++i)
                        if (win[i] != 0xEE) return printf("written past the window: C %d H %d W %d\n", C, H, W), 1;
                    for (int m = m0; m < m1; ++m)
                        for (int r = 0; r < R; ++r)
                            for (int s = 0; s < S; ++s) {
                                const int n = m / PQ, row = m % PQ / Q * st + r * dil - pad, col = m % PQ % Q * st + s * dil - pad;
                                for (int c = part * 64; c < min(C, (part + chunks) * 64); ++c) {
                                    const unsigned char *const rec = win.data() + bytes_of * (c / 64 - part) + (size_t)(first(m) - lo + (r * v.Wv + s) * dil) * 80;
                                    const bool there = row >= 0 && row < H && col >= 0 && col < W;
                                    const unsigned char want = !there ? 0 : src[nhwc ? ((long long)n * HW + row * W + col) * C + c : ((long long)n * C + c) * HW + row * W + col];
                                    if (rec[c % 64] != want)
                                        return printf("N %d C %d H %d W %d %dx%d stride %d pad %d dil %d mper %d tile %d nhwc %d: pixel %d tap %d %d channel %d\n", N, C, H, W, R, S, st,
                                                      pad, dil, mper, m0, nhwc, m, r, s, c), 1;
                                }
                            }
                }
            ++tiles;
        }
    }
    if (problems < 1500 || tiles < 5000) return printf("%d problems, %d tiles only\n", problems, tiles), 1;
    puts("ok");
    return 0;
}
