// The filter of the paper's Eq. 4-7 (Section 3.3) as a convolution kernel along the tokens: Eq. 4, 5 and 7 together are a
// circular convolution of length N with the even kernel
//     p[j] = 1/N sum_{|f| <= sigma} M[f] e^{2 pi i f j / N},      M[f] = 0.54 + 0.46 cos(2 pi f / (N - 1)) or 1.
// The window is a sum of three exponentials in f, so p is a sum of three Dirichlet kernels and needs no sum over f:
//     N p[j] = 0.54 D(u) + 0.23 D(u + d) + 0.23 D(u - d),   u = j / N,  d = 1 / (N - 1),  D(v) = sin((2 sigma + 1) pi v) / sin(pi v),
// less M[sigma] (-1)^j where 2 sigma = N: the bins sigma and -sigma are then one bin, which D counts twice.
//
// The angles of j = 16 a + b are put together from those of 16 a and of b: some hundred angles, one evaluation per thread of
// a workgroup, and a few products per p[j].  With two evaluations per p[j], one after the other, and one more for the
// constants, the taps were ready .6 us later.  The sums of angles are good to a few 2^-53, taps are used to 24 bits.
#pragma once
#include "common.hpp"

namespace luvc {

namespace {

// for 1 <= N <= 4096
struct SpuTaps {
    int N, sigma;
    bool hamming;
    double sd, cd, sKd, cKd;         // sin, cos of pi d and of K pi d, K = 2 sigma + 1
    double sv, sKv;                  // sin of pi v and of K pi v, v = d - 1 / N = 1 / (N (N - 1))
    double inv;                      // 1 / N

    // (sin, cos) of pi times: d, v, K d, K v; then j / N and K j / N in turn for j = 0 .. 15, then for j = 0, 16, ..., N / 2
    static constexpr int kHead = 4;
    static __host__ __device__ constexpr int angles_count(int N) { return kHead + 32 + 2 * (N / 32 + 1); }
    template <int THREADS>
    static __device__ __forceinline__ void fill_angles(double2* angles, int N, int sigma)
    {
        const int K = 2 * sigma + 1, turn = 2 * N;
        for (int i = threadIdx.x; i < angles_count(N); i += THREADS) {
            double a;
            if (i < kHead) {
                a = (double)((i & 2) ? K : 1) / (N > 1 ? (double)((i & 1) ? N * (N - 1) : N - 1) : 1.0);
            } else {
                const int q = i - kHead, j = q < 32 ? q >> 1 : 16 * ((q - 32) >> 1);
                int r = j;
                if (q & 1) {                     // K j mod 2 N: K j is below 2^24, the quotient off by one at most
                    r = K * j - (int)((float)(K * j) / (float)turn) * turn;
                    r += r < 0 ? turn : 0;
                    r -= r >= turn ? turn : 0;
                }
                a = (double)r / (double)N;
            }
            double s, c;
            sincospi(a, &s, &c);
            angles[i] = make_double2(s, c);
        }
    }

    // angles: filled, and a barrier passed
    __device__ __forceinline__ SpuTaps(int N_, int sigma_, int use_hamming, const double2* angles) : N(N_), sigma(sigma_), hamming(use_hamming && N_ > 2)
    {
        // N <= 2: the window is 1 at every bin
        sd = sKd = sv = sKv = 0.0;
        cd = cKd = 1.0;
        inv = 1.0 / (double)N;
        if (hamming) {
            const double2 d1 = angles[0], v1 = angles[1], dK = angles[2], vK = angles[3];
            sd = d1.x; cd = d1.y; sv = v1.x;
            sKd = dK.x; cKd = dK.y; sKv = vK.x;
        }
    }
    // p[j], 0 <= j <= N / 2
    __device__ __forceinline__ double operator()(int j, const double2* angles) const
    {
        const double2* t = angles + kHead;
        const double2 b1 = t[2 * (j & 15)], bK = t[2 * (j & 15) + 1], a1 = t[32 + 2 * (j >> 4)], aK = t[32 + 2 * (j >> 4) + 1];
        const double s1 = a1.x * b1.y + a1.y * b1.x, c1 = a1.y * b1.y - a1.x * b1.x;
        const double sK = aK.x * bK.y + aK.y * bK.x, cK = aK.y * bK.y - aK.x * bK.x;
        const double num = j == 0 ? (double)(2 * sigma + 1) : sK, den = j == 0 ? 1.0 : s1;        // D(u)
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
};

}  // namespace

}  // namespace luvc
