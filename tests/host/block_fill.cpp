// Host run of the fill from a blocked image (window_fill.h): a workgroup's ranges as the resident kernel makes them, its threads one after the other, from
// images that start behind and end before a page without access.  Checked: nothing is read outside the image or written outside the window, and every
// pixel of a range has all its channels in its record.
#include <algorithm>
#include <stdio.h>
#include <string.h>
#include <sys/mman.h>
#include <vector>

using std::max;
using std::min;
static inline unsigned __umulhi(unsigned a, unsigned b) { return (unsigned)(((unsigned long long)a * b) >> 32); }
static inline unsigned host_perm(unsigned, unsigned, unsigned) { return 0; }   // (not on this path)
static struct { unsigned x; } threadIdx;
#define __builtin_amdgcn_perm host_perm
#define __builtin_amdgcn_wave_barrier() ((void)0)
#include "../../paper_2104_04731_amd/csrc/window_fill.h"

using namespace c2i8;

static unsigned rnd_state = 4321;
static int rnd(int lo, int hi)
{
    rnd_state = rnd_state * 1664525u + 1013904223u;
    return lo + (int)((rnd_state >> 8) % (unsigned)(hi - lo + 1));
}
static unsigned magic(int d) { return d <= 1 ? 0u : magic_for(d); }

struct Layer {
    int PQ, Q, stride, pad, W, H, HW, R, S, dil, full8;
    unsigned mg_PQ, mg_Q, mg_full8;
};

int main()
{
    const size_t page = 4096, room = 1 << 20;
    unsigned char *const map = (unsigned char *)mmap(nullptr, room + 2 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (map == MAP_FAILED || mprotect(map, page, PROT_NONE) || mprotect(map + page + room, page, PROT_NONE)) return 2;
    std::vector<unsigned char> win;
    int tiles = 0;
    for (int it = 0; it < 6000; ++it) {
        const int g16l = rnd(0, 2), cb = 16 << g16l, C = rnd(1, 150), H = rnd(1, 12), W = rnd(1, 14), N = rnd(1, 9), R = rnd(1, 5), S = rnd(1, 5), st = rnd(1, 3);
        const int Cb = (C + cb - 1) / cb;
        if (H < R || W < S) continue;
        const int P = (H - R) / st + 1, Q = (W - S) / st + 1, HW = H * W, PQ = P * Q, M = N * PQ, mper = 32 * rnd(1, 8), u16 = (C + 15) / 16, pitch = (u16 | 1) * 16;
        const long long img = (long long)Cb * HW * cb, bytes = N * img;
        if (bytes > (long long)room) continue;
        unsigned char *const src = it & 1 ? map + page : map + page + room - bytes;
        for (long long i = 0; i < bytes; ++i) src[i] = (unsigned char)(i * 31 + i / 253 + it + 1);
        const int last = (P - 1) * st + R - 1, col = (Q - 1) * st + S - 1, full8 = (last * W + col + 1 + 7) & ~7;
        const Layer a{PQ, Q, st, 0, W, H, HW, R, S, 1, full8, magic(PQ), magic(Q), magic(full8)};
        for (int m0 = 0; m0 < M; m0 += mper, ++tiles) {
            int n1;
            const WindowRange w = tile_window(a, m0, min(m0 + mper, M), &n1);
            win.assign((size_t)w.slots * pitch + 64, 0xEE);
            const WindowSource t{(const int8_t *)src, img, bytes, C - 1, HW, cb};
            const int NT = 256;
            for (int tid = 0; tid < NT; ++tid) window_from_blocks<NT, 4>(t, w, u16, g16l, win.data(), pitch, tid);
            for (int s = 0; s < w.slots; ++s) {
                int n, lin;
                window_slot(w, s, &n, &lin);
                if (n >= N) return printf("image %d of %d\n", n, N), 1;
                for (int c = 0; c < u16 * 16; ++c) {
                    const unsigned char want = src[n * img + (long long)(c / cb) * HW * cb + (long long)min(lin, HW - 1) * cb + c % cb];
                    if (win[(size_t)s * pitch + c] != want) return printf("layer %d tile %d slot %d channel %d\n", it, m0 / mper, s, c), 1;
                }
                for (int c = u16 * 16; c < pitch; ++c)
                    if (win[(size_t)s * pitch + c] != 0xEE) return printf("layer %d: written behind a record\n", it), 1;
            }
            for (size_t i = (size_t)w.slots * pitch; i < win.size(); ++i)
                if (win[i] != 0xEE) return printf("layer %d: written behind the window\n", it), 1;
        }
    }
    if (tiles < 5000) return printf("%d tiles\n", tiles), 1;
    printf("ok\n");
    return 0;
}
