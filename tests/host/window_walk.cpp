// Host run of the window walk (window_walk.h): the sizes it finds, against the ranges' definition with plain divisions.
#include "../../paper_2104_04731_amd/csrc/window_walk.h"

#include <algorithm>
#include <math.h>
#include <stdio.h>
#include <stdlib.h>

static unsigned long long state = 99;
static int rnd(int lo, int hi)
{
    state = state * 6364136223846793005ULL + 1442695040888963407ULL;
    return lo + (int)((state >> 33) % (unsigned long long)(hi - lo + 1));
}
static int spread(int hi) { return std::max(1, (int)exp(log((double)hi) * rnd(0, 1000) / 1000.0)); }

int main()
{
    for (int i = 0; i < 20000; ++i) {
        const int stride = rnd(1, 3), pad = rnd(0, 4), down = rnd(0, 8), across = rnd(0, 8);
        const long long P = spread(16000), Q = spread(16000);
        const long long H = std::max(1LL, (P - 1) * stride + down + 1 - 2 * pad + rnd(0, 2)), W = std::max(1LL, (Q - 1) * stride + across + 1 - 2 * pad + rnd(0, 2));
        if (H * W > 1 << 28) continue;
        const long long PQ = P * Q, N = std::min((long long)spread(400), (1LL << 30) / PQ), M = N * PQ;
        const int mper = rnd(0, 2) ? spread(1024) : (int)std::min(PQ, 1024LL);
        auto row_of = [&](long long pq) { return pq / Q * stride - pad; };
        auto col_of = [&](long long pq) { return pq % Q * stride - pad; };
        auto first = [&](long long pq) { return row_of(pq) < 0 ? 0 : (row_of(pq) * W + std::min(std::max(col_of(pq), 0LL), W - 1)) / 8 * 8; };
        auto end = [&](long long pq) { return row_of(pq) + down >= H ? H * W : (row_of(pq) + down) * W + std::max(std::min(col_of(pq) + across, W - 1), -1LL) + 1; };
        auto up8 = [](long long v) { return v <= 0 ? 0 : (v + 7) / 8 * 8; };
        long long want8 = 0, want = 0, tiles = 0;
        const long long limit = 3000;   // (enough for every start of most images; the others are compared over the first eight)
        for (long long m0 = 0; m0 < M && tiles < limit; m0 += mper, ++tiles) {
            const long long m1 = std::min(m0 + mper, M), n0 = m0 / PQ, n1 = (m1 - 1) / PQ;
            long long s = up8((n1 > n0 ? end(PQ - 1) : end(m1 - 1 - n0 * PQ)) - first(m0 - n0 * PQ));
            if (n1 > n0) s += (n1 - n0 - 1) * up8(end(PQ - 1)) + up8(end(m1 - 1 - n1 * PQ));
            want = std::max(want, s);
            if (tiles < 8 && (m0 == 0 || m0 % PQ != 0) && want8 >= 0) want8 = std::max(want8, s);
            if (m0 > 0 && m0 % PQ == 0) break;   // the starts repeat
        }
        c2i8::WindowWalk w((int)M, (int)PQ, (int)Q, (int)H, (int)W, stride, pad, down, across);
        const bool all = tiles < limit;
        if (w.sampled(mper) != want8 || w.sampled(mper) != want8 || w.most(mper, 8) != want8 || (all && w.most(mper) != want)) {
            printf("M %lld PQ %lld Q %lld mper %d: %d, not %lld\n", M, PQ, Q, mper, w.sampled(mper), want8);
            return 1;
        }
    }
    puts("ok");
    return 0;
}
