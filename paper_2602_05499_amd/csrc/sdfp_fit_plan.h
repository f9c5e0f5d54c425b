// How the Gram matrices of Stage A are cut over the workgroups of k_fit_gram (host arithmetic only).
#pragma once
#include <algorithm>

namespace sdfp {

constexpr int FIT_GRAM_SLICES = 32;   // most stretches the columns of the matrices are cut into
constexpr int FIT_GRAM_PARTS = 3;     // matrices whose Gram matrices are added in one launch

struct FitGramSlices {
    int k_per;                        // columns per slice, a multiple of 16 (a matrix's last slice may be shorter)
    int slice0[FIT_GRAM_PARTS + 1];   // first slice of each matrix; the last entry is their number
};
// T positions, n matrices of w[i] columns each (a multiple of 16), n_cu compute units.
// Slices: at most FIT_GRAM_SLICES and 128 columns long at least, and of those the largest number whose workgroups (one per
// slice and 128 x 128 block of the upper triangle) make whole rounds of the compute units; where one slice alone is more
// than a round there is no whole number of rounds to make.  512 positions, 4096 columns, 256 compute units: 24 slices x 10
// blocks, one round, where 32 slices were 1.25.
inline FitGramSlices fit_gram_slices(int T, const int* w, int n, int n_cu) {
    const int tb = (T + 127) / 128, blocks = tb * (tb + 1) / 2;
    int w_all = 0;
    for (int i = 0; i < n; ++i) w_all += w[i];
    int ks = std::max(1, std::min(FIT_GRAM_SLICES, w_all / 128));
    const int rounds = ks * blocks / n_cu;
    if (rounds > 0) ks = std::max(1, rounds * n_cu / blocks);
    FitGramSlices s = {};
    s.k_per = ((w_all + ks - 1) / ks + 15) / 16 * 16;
    for (;; s.k_per += 16) {   // (a matrix's last slice may be short: longer slices until their number fits)
        for (int i = 0; i < n; ++i) s.slice0[i + 1] = s.slice0[i] + (w[i] + s.k_per - 1) / s.k_per;
        if (s.slice0[n] <= std::max(ks, n)) return s;
    }
}

}  // namespace sdfp
