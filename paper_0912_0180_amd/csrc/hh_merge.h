// hh_merge.h -- where the merged legs of a 2D batch pay (host code only).
#pragma once
#include <algorithm>

namespace hh {

// What the rule looks at, per problem of a batch.
struct BatchShape {
    int on;             // its last levels can be merged
    int levels, tail;   // levels of its grid; first level of its tail kernel on the tiled route
    int split;          // k_coarse solves its coarsest grid on the tiled route
    int kdown, kup;     // levels of its merged down- and up-leg
    long down, up;      // its workgroups there
};

// Whether the batch's cycle is faster with the merged legs of the problems
// marked `on` than with tiled legs and tail kernels: what its launches cost
// against what the merged legs' workgroups cost, in us per cycle.  Launches
// follow the deepest problem, so a problem beside the merged ones can keep the
// launches of all levels.  A merged workgroup takes a CU (LDS), so more of them
// than CUs run in rounds.  Measured, FP64 cycles, us without and with them, and
// the estimate of the difference (square problems, side/levels):
//   2 of 416/5          338 down-workgroups   90.5 -> 93.6    -3.0
//   3 of 288/5          243                   82.5 -> 71.0     9.5
//   3 of 432/5          588                  109.1 -> 124.1   -15.5
//   2 of 864/6          392                  160.9 -> 157.8    2.5
//   10 of 192/5         360                   99.4 -> 96.6     2.6
//   400/5, 3 of 256/5   361                  108.0 -> 94.4    13.6
//   512/5 and 512/7     272                  115.2 -> 119.1   -3.2
//   2 of 400/5, 64/2    338                   97.8 -> 100.1   -3.0
//   2 of 256/4          512                   74.1 -> 70.1     5.6
//   3 of 144/4, 96/3    243                   66.0 -> 68.2    -3.6
// FP32 cycles take fewer and cheaper workgroups: 2 of 416/5 7.0 -> 6.2 ms per
// 64 matvecs, 3 of 144/4 beside 96/3 9.0 -> 9.2.
inline bool batch_merge_pays(const BatchShape *p, int n, bool fp32)
{
    constexpr int CUS = 256;
    constexpr double LAUNCH = 5.5;    // a launch of few workgroups
    constexpr double TAIL = 2.8;      // more for one of the tail kernel
    constexpr double WHOLE = 8.0;     // more where it holds the coarsest solve and both legs
    const double deep = fp32 ? 3.0 : 6.25, shallow = fp32 ? 1.0 : 1.8;   // a round of merged legs over three, two levels
    double cost[2];
    long down = 0, up = 0;
    bool three = false;
    for (int m = 0; m < 2; ++m) {
        int dn = 0, u = 0;
        bool tail_down = false, tail_up = false, coarse = false, merged = false, whole = false;
        for (int q = 0; q < n; ++q) {
            const BatchShape &s = p[q];
            const int c = s.levels - 1;
            if (m && s.on) {
                dn = std::max(dn, c - s.kdown);
                u = std::max(u, c - s.kup);
                coarse = merged = true;
                three = three || s.kdown > 2;
                down += s.down;
                up += s.up;
            } else {
                dn = std::max(dn, s.tail);
                u = std::max(u, s.tail);
                tail_down = tail_down || !s.split || s.tail < c;
                tail_up = tail_up || (s.split && s.tail < c);
                coarse = coarse || s.split;
                whole = whole || !s.split;
            }
        }
        cost[m] = LAUNCH * (dn + u + tail_down + tail_up + coarse + 2 * merged) + TAIL * (tail_down + tail_up) + (whole ? WHOLE : 0.0);
    }
    const long rounds = (down + CUS - 1) / CUS + (up + CUS - 1) / CUS;
    return cost[0] - cost[1] > (three ? deep : shallow) * (double)rounds;
}

} // namespace hh
