// The filter of the paper's Eq. 4-7 (Section 3.3) as a convolution kernel along the tokens: Eq. 4, 5 and 7 together are a
// circular convolution of length N with the even kernel
//     p[j] = 1/N sum_{|f| <= sigma} M[f] e^{2 pi i f j / N},      M[f] = 0.54 + 0.46 cos(2 pi f / (N - 1)) or 1.
// The window is a sum of three exponentials in f, so p is a sum of three Dirichlet kernels and needs no sum over f:
//     N p[j] = 0.54 D(u) + 0.23 D(u + d) + 0.23 D(u - d),   u = j / N,  d = 1 / (N - 1),  D(v) = sin((2 sigma + 1) pi v) / sin(pi v),
// less M[sigma] (-1)^j where 2 sigma = N: the bins sigma and -sigma are then one bin, which D counts twice.
#pragma once
#include "common.hpp"

namespace luvc {

namespace {

struct SpuTaps {
    int N, sigma;
    bool hamming;
    double sd, cd, sKd, cKd;         // sin, cos of pi d and of (2 sigma + 1) pi d

    __device__ __forceinline__ SpuTaps(int N_, int sigma_, int use_hamming) : N(N_), sigma(sigma_), hamming(use_hamming && N_ > 2)
    {
        // N <= 2: the window is 1 at every bin
        sd = sKd = 0.0;
        cd = cKd = 1.0;
        if (hamming) {
            sincospi(1.0 / (double)(N - 1), &sd, &cd);
            sincospi((double)(2 * sigma + 1) / (double)(N - 1), &sKd, &cKd);
        }
    }
    // p[j], 0 <= j <= N / 2
    __device__ __forceinline__ double operator()(int j) const
    {
        const int K = 2 * sigma + 1;
        double s1, c1, sK, cK;
        sincospi((double)j / (double)N, &s1, &c1);
        sincospi((double)(((int64_t)K * j) % (2 * N)) / (double)N, &sK, &cK);
        const double D0 = j == 0 ? (double)K : sK / s1;
        double p = D0;
        if (hamming) {
            double np = sK * cKd + cK * sKd, dp = s1 * cd + c1 * sd, nm = sK * cKd - cK * sKd, dm = s1 * cd - c1 * sd;
            if (j == 1) {                // u - d = -1 / (N (N - 1)): the difference of the two angles has no digits left
                const double v = 1.0 / ((double)N * (double)(N - 1));
                nm = sinpi((double)K * v);
                dm = sinpi(v);
            }
            p = 0.54 * D0 + 0.23 * (np / dp + nm / dm);
        }
        if (2 * sigma == N) {
            const double w = hamming ? 0.54 + 0.46 * cospi(2.0 * (double)sigma / (double)(N - 1)) : 1.0;
            p -= (j & 1) ? -w : w;
        }
        return p / (double)N;
    }
};

}  // namespace

}  // namespace luvc
