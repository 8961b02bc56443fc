// How many input pixels the workgroups of a problem keep (window_fill.h: WindowRange), walked tile by tile on the host.
#pragma once

namespace c2i8 {

// One of these serves every estimate of a call: the kernels look at the same pixel counts, and the walks are most of what
// choosing a kernel costs.  The divisions are by doubles' reciprocals, exact for what an int holds.
class WindowWalk {
public:
    // M output pixels in images of PQ in rows of Q, from H x W; down, across: from a pixel's first tap to its last.
    WindowWalk(int M, int PQ, int Q, int H, int W, int stride, int pad, int down, int across)
        : M_(M), PQ_(PQ), Q_(Q), W_(W), H_(H), HW_((int)((long long)H * W)), stride_(stride), pad_(pad), down_(down), across_(across),
          per_PQ_(1.0 / PQ), per_Q_(1.0 / Q)
    {
        image_end_ = end(PQ_ - 1);
        full8_ = (image_end_ + 7) & ~7;
    }

    // Slots of the largest window of `mper` output pixels over the first `tiles` tiles (0: all of them; tile starts repeat within
    // an image after PQ / gcd(mper, PQ) tiles).
    int most(int mper, int tiles = 0) const
    {
        const int step = mper - whole(mper, per_PQ_) * PQ_;   // from tile to tile, within an image
        int most = 0, a = 0, count = 0;
        for (long long m0 = 0; m0 < M_ && (m0 == 0 || a != 0) && (tiles == 0 || count < tiles); m0 += mper, ++count) {
            const int m1 = m0 + mper < M_ ? a + mper : a + (int)(M_ - m0);   // local end (may pass the image)
            const int n1 = whole(m1 - 1, per_PQ_);
            int s = ((n1 > 0 ? image_end_ : end(m1 - 1)) - first(a) + 7) & ~7;
            if (s < 0) s = 0;
            if (n1 > 0) {
                const int t = (end(m1 - 1 - n1 * PQ_) + 7) & ~7;
                s += (n1 - 1) * full8_ + (t > 0 ? t : 0);
            }
            if (s > most) most = s;
            a += step;
            if (a >= PQ_) a -= PQ_;
        }
        return most;
    }
    // The same over the first eight, kept.
    int sampled(int mper)
    {
        for (int i = 0; i < seen_; ++i)
            if (mper_[i] == mper) return slots_[i];
        const int s = most(mper, 8);
        if (seen_ < MOST_SEEN) mper_[seen_] = mper, slots_[seen_++] = s;
        return s;
    }

private:
    static constexpr int MOST_SEEN = 96;
    int M_, PQ_, Q_, W_, H_, HW_, stride_, pad_, down_, across_, image_end_, full8_;
    double per_PQ_, per_Q_;
    int seen_ = 0, mper_[MOST_SEEN], slots_[MOST_SEEN];

    static int whole(int n, double per) { return (int)((n + 0.5) * per); }   // (n >= 0: half a unit is far more than the rounding)
    int first(int pq) const
    {
        const int p = whole(pq, per_Q_), row = p * stride_ - pad_, col = (pq - p * Q_) * stride_ - pad_;
        return row < 0 ? 0 : (int)((long long)row * W_ + (col < 0 ? 0 : col > W_ - 1 ? W_ - 1 : col)) & ~7;
    }
    int end(int pq) const
    {
        const int p = whole(pq, per_Q_), row = p * stride_ - pad_ + down_, col = (pq - p * Q_) * stride_ - pad_ + across_;
        return row >= H_ ? HW_ : (int)((long long)row * W_ + (col > W_ - 1 ? W_ - 1 : col < -1 ? -1 : col)) + 1;
    }
};

}  // namespace c2i8
