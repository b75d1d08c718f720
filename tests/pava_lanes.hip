// Host harness of the monotone repair's wave pass (the template the kernels
// instantiate) that counts the windows it commits, for the CPU tests.
#include <vector>

#include "pr_coarse_dev.hpp"

namespace {
int windows = 0;
struct CountingLanes : pr::PavaHostLanes {
    static double value(const Value &x, int l) {
        windows += l == 0 ? 1 : 0;  // a window reads its first lane's value once, besides the sum at its end
        return PavaHostLanes::value(x, l);
    }
};
}  // namespace

// v[0..L) in place; returns the number of reads of a window's first lane.
extern "C" int pv_pava_windows(double *v, int L) {
    windows = 0;
    std::vector<int> vio;
    for (int j = 0; j + 1 < L; ++j)
        if (v[j] > v[j + 1]) vio.push_back(j);
    if (vio.empty()) return 0;
    std::vector<double> S(L);
    std::vector<int> SC(L);
    double fm, lm;
    const int np =
        pr::pava_range<CountingLanes>(v, 0, L, vio.data(), (int)vio.size(), S.data(), SC.data(), &fm, &lm);
    for (int b = 0; b < np; ++b) {
        const int c = SC[b] & 0xFFFF, st = SC[b] >> 16;
        const double mean = S[b] / (double)c;
        for (int t = 0; t < c; ++t) v[st + t] = mean;
    }
    return windows;
}
