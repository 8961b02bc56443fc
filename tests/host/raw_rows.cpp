// Host run of the raw 1x1 weight loads (window_fill.h): the tensor ends where a page without access begins, every row and
// 16-channel piece that a tile may ask for is loaded, and what comes back is compared with the bytes.
#include "../../paper_2104_04731_amd/csrc/window_fill.h"

#include <stdio.h>
#include <string.h>
#include <sys/mman.h>

int main()
{
    const size_t room = 1 << 20;
    unsigned char *const base = (unsigned char *)mmap(nullptr, room + 4096, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (base == MAP_FAILED || mprotect(base + room, 4096, PROT_NONE)) return 2;
    for (int C = 1; C <= 130; ++C)
        for (int K : {1, 2, 3, 5, 16, 31, 33, 64, 512}) {
            const size_t bytes = (size_t)K * C;
            if (bytes < 16) continue;   // (such layers take another path)
            unsigned char *const wt = base + room - bytes;
            for (size_t i = 0; i < bytes; ++i) wt[i] = (unsigned char)(i * 37 + i / 251 + 1);
            for (int k = 0; k < (K + 63) / 64 * 64; ++k)
                for (int c0 = 0; c0 < (C + 63) / 64 * 64; c0 += 16) {
                    const c2i8::v4i d = c2i8::raw1_load((const int8_t *)wt, K, C, k, c0);
                    for (int b = 0; b < 16; ++b) {
                        const unsigned char want = c0 + b < C ? wt[(size_t)(k < K ? k : K - 1) * C + c0 + b] : 0;
                        if ((unsigned char)((unsigned)d[b >> 2] >> (8 * (b & 3))) != want) {
                            printf("K %d C %d row %d channel %d\n", K, C, k, c0 + b);
                            return 1;
                        }
                    }
                }
        }
    puts("ok");
    return 0;
}
