// Host run of the window fills (window_fill.h): a workgroup's input ranges as the resident kernel makes them, its threads one
// after the other, from tensors that start behind and end before a page without access.  Checked: nothing is read outside
// the tensor or written outside the window, and every pixel of a range has its channels in its record.
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
#include "../../paper_2104_04731_amd/csrc/window_fill.h"

using namespace c2i8;

static unsigned rnd_state = 12345;
static int rnd(int lo, int hi)
{
    rnd_state = rnd_state * 1664525u + 1013904223u;
    return lo + (int)((rnd_state >> 8) % (unsigned)(hi - lo + 1));
}
static unsigned magic(int d) { return d <= 1 ? 0u : magic_for(d); }

int main()
{
    const size_t page = 4096, room = 1 << 20;
    unsigned char *const map = (unsigned char *)mmap(nullptr, room + 2 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (map == MAP_FAILED || mprotect(map, page, PROT_NONE) || mprotect(map + page + room, page, PROT_NONE)) return 2;
    std::vector<unsigned char> win;
    int tiles = 0;
    for (int it = 0; it < 6000; ++it) {
        const int C = it % 3 ? rnd(1, 40) : rnd(1, 150), H = rnd(1, 12), W = rnd(1, 14), N = rnd(1, 9), R = rnd(1, 5), S = rnd(1, 5), st = rnd(1, 3), pad = rnd(0, 4), dil = rnd(1, 3);
        const int P = (H + 2 * pad - dil * (R - 1) - 1) / st + 1, Q = (W + 2 * pad - dil * (S - 1) - 1) / st + 1;
        if (H + 2 * pad < dil * (R - 1) + 1 || W + 2 * pad < dil * (S - 1) + 1) continue;
        const long long bytes = (long long)N * C * H * W;
        if (bytes < 64 || bytes > (long long)room) continue;
        const int HW = H * W, PQ = P * Q, M = N * PQ, mper = 32 * rnd(1, 8), C16 = (C + 15) / 16 * 16, pitch = (C16 / 16 | 1) * 16;
        // against the end of the room, or against its start
        unsigned char *const src = it & 1 ? map + page : map + page + room - bytes;
        for (long long i = 0; i < bytes; ++i) src[i] = (unsigned char)(i * 31 + i / 253 + it + 1);
        auto first = [&](int pq) {
            const int row = pq / Q * st - pad, col = pq % Q * st - pad;
            return row < 0 ? 0 : (row * W + min(max(col, 0), W - 1)) & ~7;
        };
        auto end = [&](int pq) {
            const int row = pq / Q * st - pad + (R - 1) * dil, col = pq % Q * st - pad + (S - 1) * dil;
            return row >= H ? HW : row * W + max(min(W - 1, col), -1) + 1;
        };
        const int full8 = (end(PQ - 1) + 7) & ~7;
        if (end(PQ - 1) <= 0) continue;
        for (int m0 = 0; m0 < M; m0 += mper) {
            const int m1 = min(m0 + mper, M), n0 = m0 / PQ, n1 = (m1 - 1) / PQ, lo0 = first(m0 - n0 * PQ);
            const int len0 = max(((n1 > n0 ? end(PQ - 1) : end(m1 - 1 - n0 * PQ)) - lo0 + 7) & ~7, 0);
            const int last = n1 > n0 ? max((end(m1 - 1 - n1 * PQ) + 7) & ~7, 0) : 0, slots = len0 + (n1 > n0 ? (n1 - n0 - 1) * full8 + last : 0);
            const WindowRange range{n0, lo0, len0, full8, slots, magic(full8)};
            const WindowSource from{(const int8_t *)src, (long long)C * HW, bytes, C - 1, HW, C};
            for (int form = 0; form < 3; ++form) {
                const int nhwc = form == 2;
                win.assign((size_t)slots * pitch + 256, 0xEE);
                for (int tid = 0; tid < 256; ++tid) {
                    if (nhwc) window_from_pixels<256, 4>(from, range, C16 / 16, magic(C16 / 16), win.data(), pitch, tid);
                    else if (form) window_from_nchw<256, 4, true>(from, range, C16 / 4, magic(C16 / 4), win.data(), pitch, tid);
                    else window_from_nchw<256, 4, false>(from, range, C16 / 4, magic(C16 / 4), win.data(), pitch, tid);
                }
                for (size_t i = (size_t)slots * pitch; i < win.size(); ++i)
                    if (win[i] != 0xEE) return printf("written past the window: C %d H %d W %d\n", C, H, W), 1;
                for (int n = n0; n <= n1; ++n) {
                    const int base = n == n0 ? 0 : len0 + (n - n0 - 1) * full8, a = n == n0 ? lo0 : 0;
                    const int b = n < n1 ? end(PQ - 1) : end(m1 - 1 - n1 * PQ);
                    for (int lin = a; lin < b; ++lin)
                        for (int c = 0; c < (nhwc ? C : C16); ++c) {
                            const unsigned char want = c >= C ? 0 : src[nhwc ? ((long long)n * HW + lin) * C + c : ((long long)n * C + c) * HW + lin];
                            if (win[(size_t)(base + lin - a) * pitch + c] != want)
                                return printf("N %d C %d H %d W %d %dx%d stride %d pad %d dil %d mper %d tile %d nhwc %d: image %d pixel %d channel %d\n", N, C, H, W, R, S, st, pad,
                                              dil, mper, m0, nhwc, n, lin, c), 1;
                        }
                }
                ++tiles;
            }
        }
    }
    if (tiles < 5000) return printf("%d tiles only\n", tiles), 1;
    puts("ok");
    return 0;
}
