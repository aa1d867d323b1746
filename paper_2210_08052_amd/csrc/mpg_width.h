// Strip width of a call that is not tuned: host arithmetic only (a CPU test
// compiles this header by itself).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace mpg {

// Strips of a pair of m residues (columns 0..m) at K = 1, 2 or 4 columns per
// lane.  (K >> 1 is K's logarithm: a call plans up to 10^5 pairs, and a division
// by a variable costs more than the rest.)
inline int pair_strips(int m, int K) { return (m + 64 * K) >> (6 + (K >> 1)); }

// Steps every strip of a pair runs (a multiple of 64).  Lane L reaches row
// n at step n + L: a pair of one strip stops once the lane of column m has,
// the strips of a wider pair run all 64 lanes to row n.
inline int pair_nsteps(int n, int m, int K) {
    const int lanes = pair_strips(m, K) == 1 ? (m >> (K >> 1)) + 1 : 64;
    return (n + lanes + 63) & ~63;
}

// Width 1 or 2 for a call, from what bounds it: its work (strips x steps)
// spread over the device's SIMDs, and the longest pair's own chain, its steps
// one after another with each strip kStripLag steps behind the one on its left.
// (A strip waits for three chunks of its left neighbour before its first, and
// a chunk is announced one chunk late: 256 steps, and the time of the polls.)
// Width 2 does a column's work in fewer instructions, width 1 makes a step
// shorter but doubles the strips.  Neither bound is reached while the other is
// near: a call takes about the kNorm-norm of the two.  The costs are fitted to
// 1,190 calls, each timed at both widths: 1 to 4,000 pairs of 100 to 8,000
// residues on 1.2 to 40 bases per residue, and the batch recipe, score-only,
// traced, without introns and in 16-bit lanes.  The widths picked take 0.3 to
// 0.4% longer than the faster ones (geometric mean); the worst calls, 1,000
// pairs of three narrow strips, 16% longer than at width 2.  Times at widths 2
// and 1, ms: one traced gene 0.56 and 0.39; score-only, 60 pairs of 2,000
// residues on 3,000 bases 0.92 and 1.15, 30 of 8,000 on 9,600 3.82 and 6.51,
// one of 2,000 on 8,000 1.47 and 1.32; batch recipe 1,200 pairs 3.34 and 2.43,
// 3,000 3.54 and 4.54.
struct WidthWork {
    static constexpr int kStripLag = 290;
    static constexpr double kNorm = 1.3;
    // width 1 only where it is this much faster: in doubt the wider strips,
    // whose time hangs less on where the wavefronts land
    static constexpr double kMargin = 0.97;
    // Cycles (at 2.4 GHz) of a strip's step at width K, step + column * K: on a
    // SIMD shared by four wavefronts, and alone.
    struct Cost { double step, column; };
    enum Kind { kPlain, kIntrons, kTracedPlain, kTraced, kInt16, kKinds };
    static constexpr Cost kShared[kKinds] = {{49, 29}, {66, 45}, {56, 53}, {83, 77}, {38, 88}};
    static constexpr Cost kAlone[kKinds] = {{94, 70}, {96, 99}, {96, 106}, {98, 174}, {74, 118}};
    // per kind, [0]: width 1, [1]: width 2: strips x steps, and the steps of the
    // longest chain
    int64_t work[kKinds][2] = {}, chain[kKinds][2] = {};
    void add(int n, int m, Kind kind) {
        for (int K = 1; K <= 2; ++K) {
            const int64_t steps = pair_nsteps(n, m, K), strips = pair_strips(m, K);
            work[kind][K - 1] += steps * strips;
            chain[kind][K - 1] = std::max(chain[kind][K - 1], steps + kStripLag * (strips - 1));
        }
    }
    // 32-bit lanes
    void add(int n, int m, bool tb, bool introns) { add(n, m, (Kind)(2 * tb + introns)); }
    // 16-bit lanes: a step advances two pairs
    void add16(int n, int m) { add(n, m, kInt16); }
    double time(int K, int ncu) const {
        double w = 0, c = 0;
        for (int k = 0; k < kKinds; ++k) {
            w += (kShared[k].step + kShared[k].column * K) * work[k][K - 1];
            c = std::max(c, (kAlone[k].step + kAlone[k].column * K) * chain[k][K - 1]);
        }
        return std::pow(std::pow(w / (4.0 * ncu), kNorm) + std::pow(c, kNorm), 1 / kNorm);
    }
    int width(int ncu) const { return time(1, ncu) < kMargin * time(2, ncu) ? 1 : 2; }
};

}  // namespace mpg
