// Host run of the raw 3x3 weight loads (window_fill.h): the tensor ends where a page without access begins, every row and
// channel quad that a tile may ask for is loaded, and what comes back is compared with the bytes.
#include "../../paper_2104_04731_amd/csrc/window_fill.h"

#include <stdio.h>
#include <string.h>
#include <sys/mman.h>

int main()
{
    const size_t room = 1 << 20;
    unsigned char *const base = (unsigned char *)mmap(nullptr, room + 4096, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (base == MAP_FAILED || mprotect(base + room, 4096, PROT_NONE)) return 2;
    for (int C = 1; C <= 70; ++C)
        for (int K : {1, 2, 3, 4, 5, 31, 33, 64, 512}) {
            const size_t bytes = (size_t)K * C * 9;
            unsigned char *const wt = base + room - bytes;
            for (size_t i = 0; i < bytes; ++i) wt[i] = (unsigned char)(i * 37 + i / 251 + 1);
            for (int k = 0; k < (K + 63) / 64 * 64; ++k)
                for (int quad = 0; quad < (C + 15) / 16 * 4; ++quad) {
                    unsigned d[9];
                    c2i8::raw9_load((const int8_t *)wt, K, C, k, quad, d);
                    c2i8::raw9_mask(C, quad, d);
                    for (int b = 0; b < 36; ++b) {
                        const int c = quad * 4 + b / 9;
                        const unsigned char want = k < K && c < C ? wt[((size_t)k * C + c) * 9 + b % 9] : 0;
                        if ((unsigned char)(d[b >> 2] >> (8 * (b & 3))) != want) {
                            printf("K %d C %d row %d quad %d byte %d\n", K, C, k, quad, b);
                            return 1;
                        }
                    }
                }
        }
    puts("ok");
    return 0;
}
