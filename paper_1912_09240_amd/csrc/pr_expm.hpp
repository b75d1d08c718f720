// Dense exponentials E(tau) = exp(A tau) of tridiagonal generators, shared by
// every coarse model (one instance or a batch of them).
#pragma once

#include <vector>

#include "pr_internal.hpp"

namespace pr {

// Generator A: lo[i] = A[i][i-1], di[i] = A[i][i], up[i] = A[i][i+1];
// columns sum to zero (mass is conserved).
struct Tridiag {
    std::vector<double> lo, di, up;
};

struct ExpmReq {
    int gen;     // index of the generator
    double tau;  // time, >= 0
};

// out[e] (device, [reqs][n][n] row-major) = exp(gens[reqs[e].gen] reqs[e].tau).
// Waits for the stream.
int build_expms(const std::vector<Tridiag> &gens, const std::vector<ExpmReq> &reqs, int n, double *out,
                hipStream_t st);

}  // namespace pr
