// How the Gram matrices of Stage A are cut over the workgroups of k_fit_gram (host arithmetic only).
#pragma once
#include <algorithm>

namespace sdfp {

constexpr int FIT_GRAM_SLICES = 32;   // most stretches the columns of a matrix are cut into
constexpr int FIT_GRAM_PARTS = 3;     // matrices of one launch

struct FitGramSlices {
    int k_per[FIT_GRAM_PARTS];        // columns per slice of each matrix, a multiple of 16 (the last slice may be shorter)
    int slice0[FIT_GRAM_PARTS + 1];   // first slice of each matrix; entry n is the number of all
};
// n matrices of w[i] columns each (a multiple of 16): at most FIT_GRAM_SLICES slices per matrix, 128 columns long at least.
// (Fewer, longer ones that make whole rounds of the compute units -- 24 of 176 columns at 512 positions and 4096 columns --
// were tried: the error of the scores against float64 grows with a slice's length.)
inline FitGramSlices fit_gram_slices(const int* w, int n) {
    FitGramSlices s = {};
    for (int i = 0; i < n; ++i) {
        const int ks = std::max(1, std::min(FIT_GRAM_SLICES, w[i] / 128));
        s.k_per[i] = ((w[i] + ks - 1) / ks + 15) / 16 * 16;
        s.slice0[i + 1] = s.slice0[i] + (w[i] + s.k_per[i] - 1) / s.k_per[i];
    }
    return s;
}

}  // namespace sdfp
