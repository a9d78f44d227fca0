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

// for 1 <= N <= 4096, built and called by whole wavefronts
struct SpuTaps {
    int N, sigma;
    bool hamming;
    double sd, cd, sKd, cKd;         // sin, cos of pi d and of (2 sigma + 1) pi d
    double sv, sKv;                  // sin of pi v and of (2 sigma + 1) pi v, v = d - 1 / N = 1 / (N (N - 1))
    double inv;                      // 1 / N

    // Four angles, one evaluation: a lane takes one of them.
    __device__ __forceinline__ SpuTaps(int N_, int sigma_, int use_hamming) : N(N_), sigma(sigma_), hamming(use_hamming && N_ > 2)
    {
        // N <= 2: the window is 1 at every bin
        sd = sKd = sv = sKv = 0.0;
        cd = cKd = 1.0;
        inv = 1.0 / (double)N;
        if (hamming) {
            const int lane = threadIdx.x & 63;
            double s, c, a = 1.0 / (double)(N - 1);
            if (lane & 1) a *= inv;
            if (lane & 2) a *= (double)(2 * sigma + 1);
            sincospi(a, &s, &c);
            sd = of_lane(s, 0); cd = of_lane(c, 0); sv = of_lane(s, 1);
            sKd = of_lane(s, 2); cKd = of_lane(c, 2); sKv = of_lane(s, 3);
        }
    }
    // p[j], 0 <= j <= N / 2
    __device__ __forceinline__ double operator()(int j) const
    {
        const int K = 2 * sigma + 1, turn = 2 * N;
        // K j mod 2 N: below 2^24, the quotient is off by one at most
        int r = K * j - (int)((float)(K * j) * (0.5f * (float)inv)) * turn;
        r += r < 0 ? turn : 0;
        r -= r >= turn ? turn : 0;
        double s1, c1, sK, cK;
        sincospi((double)j * inv, &s1, &c1);
        sincospi((double)r * inv, &sK, &cK);
        const double num = j == 0 ? (double)K : sK, den = j == 0 ? 1.0 : s1;        // D(u)
        double p;
        if (hamming) {
            const double np = sK * cKd + cK * sKd, dp = s1 * cd + c1 * sd;
            // j = 1: u - d = -v, the difference of the two angles has no digits left
            const double nm = j == 1 ? -sKv : sK * cKd - cK * sKd, dm = j == 1 ? -sv : s1 * cd - c1 * sd;
            p = (0.54 * num * (dp * dm) + 0.23 * den * (np * dm + nm * dp)) / (den * (dp * dm));
        } else p = num / den;
        if (2 * sigma == N) {
            const double w = hamming ? 0.54 + 0.46 * cospi(2.0 * (double)sigma / (double)(N - 1)) : 1.0;
            p -= (j & 1) ? -w : w;
        }
        return p * inv;
    }

private:
    __device__ static __forceinline__ double of_lane(double v, int lane)
    {
        const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane), hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
        return __hiloint2double(hi, lo);
    }
};

}  // namespace

}  // namespace luvc
