// The same windows (panel_fill.cpp) on small planes without a border, the tensor always against the page behind it: the eights of slots that a
// window is filled in end in the next image, and the pieces of one of its first pixels can pass the end of a tensor whose last image it is.
// Without a border the slots are the pixels of all images one behind the other, so every slot up to the last tap's is compared.
#define main panel_fill_main
#include "panel_fill.cpp"
#undef main

int main()
{
    const size_t page = 4096, room = 1 << 16;
    unsigned char *const map = (unsigned char *)mmap(nullptr, room + page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (map == MAP_FAILED || mprotect(map + room, page, PROT_NONE)) return 2;
    std::vector<unsigned char> win;
    int tiles = 0;
    for (int HW = 8; HW <= 27; ++HW)
        for (int H = 1; H <= HW; ++H)
            for (int C = 1; C <= 70; ++C)
                for (int N = 2; N <= 4; ++N) {
                    const int W = HW / H, R = rnd(1, H < 5 ? H : 5), S = rnd(1, W < 5 ? W : 5), st = rnd(1, 2);
                    const long long img = (long long)C * HW, bytes = N * img;
                    if (HW % H || bytes < 16 || bytes > (long long)room || !virtual_image_fits(R, S, 1, H, W, 0, N, img)) continue;
                    const int P = (H - R) / st + 1, Q = (W - S) / st + 1, PQ = P * Q, M = N * PQ, span = (R - 1) * W + S - 1;
                    unsigned char *const src = map + room - bytes;
                    for (long long i = 0; i < bytes; ++i) src[i] = (unsigned char)(i * 31 + i / 253 + C);
                    const VirtualImage v{W, H, N, C, H, W, HW, 0, (C + 63) / 64, C, img, bytes, magic(W), magic(H)};
                    auto first = [&](int m) { return (m / PQ * H + m % PQ / Q * st) * W + m % PQ % Q * st; };
                    const int pixels[] = {1, rnd(2, 17), rnd(18, 40)};
                    for (int mper : pixels)
                        for (int m0 = 0; m0 < M; m0 += mper, ++tiles)
                            for (int nhwc = 0; nhwc < 2; ++nhwc) {
                                const int lo = first(m0), last = first(min(m0 + mper, M) - 1) + span, octs = (last - lo + 8) >> 3;
                                win.assign((size_t)octs * 8 * 80 * v.chunks, 0xEE);
                                if (nhwc) fill_window<PanelFill<true>>(v, (const int8_t *)src, lo, last, octs, 0, v.chunks, win.data());
                                else fill_window<PanelFill<false>>(v, (const int8_t *)src, lo, last, octs, 0, v.chunks, win.data());
                                for (int s = lo; s <= last; ++s)
                                    for (int c = 0; c < C; ++c)
                                        if (win[((size_t)(c / 64) * octs * 8 + s - lo) * 80 + c % 64] != src[s / HW * img + (nhwc ? s % HW * C + c : c * HW + s % HW)])
                                            return printf("N %d C %d H %d W %d %dx%d stride %d mper %d tile %d nhwc %d: slot %d channel %d\n", N, C, H, W, R, S, st, mper, m0, nhwc, s, c), 1;
                            }
                }
    if (tiles < 100000) return printf("%d tiles only\n", tiles), 1;
    puts("ok");
    return 0;
}
