// Register-level pieces shared by the transform kernels of the SPU score (paper Section 3.3): complex arithmetic, the
// radix-4 butterfly, the 8- and the 16-point DFT.
#pragma once
#include "common.hpp"

namespace luvc {

struct cf { float x, y; };
__device__ __forceinline__ cf operator+(cf a, cf b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cf operator-(cf a, cf b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ cf cmul(cf a, cf w) { return {fmaf(a.x, w.x, -a.y * w.y), fmaf(a.x, w.y, a.y * w.x)}; }
__device__ __forceinline__ cf cmulc(cf a, cf w) { return {fmaf(a.x, w.x, a.y * w.y), fmaf(a.y, w.x, -a.x * w.y)}; }   // a * conj(w)

// radix-4 butterfly, INV = false: e^{-i...}; true: e^{+i...}
template <bool INV>
__device__ __forceinline__ void bf4(cf& a0, cf& a1, cf& a2, cf& a3)
{
    const cf t0 = a0 + a2, t1 = a0 - a2, t2 = a1 + a3, d = a1 - a3;
    const cf t3 = INV ? cf{-d.y, d.x} : cf{d.y, -d.x};          // d * (+i) or d * (-i)
    a0 = t0 + t2; a1 = t1 + t3; a2 = t0 - t2; a3 = t1 - t3;
}

// the same with a2 = a3 = 0 (not read)
template <bool INV>
__device__ __forceinline__ void bf4_half(cf& a0, cf& a1, cf& a2, cf& a3)
{
    const cf t3 = INV ? cf{-a1.y, a1.x} : cf{a1.y, -a1.x}, a = a0, b = a1;
    a0 = a + b; a1 = a + t3; a2 = a - b; a3 = a - t3;
}

// acc + a w (INV) or acc + a conj(w)
template <bool INV>
__device__ __forceinline__ cf cmac(cf acc, cf a, cf w)
{
    return INV ? cf{fmaf(a.x, w.x, fmaf(-a.y, w.y, acc.x)), fmaf(a.x, w.y, fmaf(a.y, w.x, acc.y))}
               : cf{fmaf(a.x, w.x, fmaf(a.y, w.y, acc.x)), fmaf(a.y, w.x, fmaf(-a.x, w.y, acc.y))};
}

// Radix-4 butterfly of a0, a1 w1, a2 w2, a3 w3 (INV = false: of the conjugate factors).  Every factor goes into the additions
// that follow it: a0 - a2 w2 is 2 a0 - (a0 + a2 w2), likewise for the other pair, 24 instructions for 28.
template <bool INV>
__device__ __forceinline__ void bf4_tw(cf& a0, cf& a1, cf& a2, cf& a3, cf w1, cf w2, cf w3)
{
    const cf t0 = cmac<INV>(a0, a2, w2), t1{fmaf(2.f, a0.x, -t0.x), fmaf(2.f, a0.y, -t0.y)};
    const cf p = INV ? cmul(a1, w1) : cmulc(a1, w1);
    const cf t2 = cmac<INV>(p, a3, w3), d{fmaf(2.f, p.x, -t2.x), fmaf(2.f, p.y, -t2.y)};
    const cf t3 = INV ? cf{-d.y, d.x} : cf{d.y, -d.x};
    a0 = t0 + t2; a1 = t1 + t3; a2 = t0 - t2; a3 = t1 - t3;
}

// a + k u, a - k u
__device__ __forceinline__ cf axpy(float k, cf u, cf a) { return {fmaf(k, u.x, a.x), fmaf(k, u.y, a.y)}; }
// u = a (1 + i t) or its conjugate form, the direction of a twiddle whose real part is left to the caller; u = a (t + i) likewise
template <bool INV> __device__ __forceinline__ cf rot(cf a, float t) { return INV ? cf{fmaf(-t, a.y, a.x), fmaf(t, a.x, a.y)} : cf{fmaf(t, a.y, a.x), fmaf(-t, a.x, a.y)}; }
template <bool INV> __device__ __forceinline__ cf rotq(cf a, float t) { return INV ? cf{fmaf(t, a.x, -a.y), fmaf(t, a.y, a.x)} : cf{fmaf(t, a.x, a.y), fmaf(t, a.y, -a.x)}; }

__device__ __forceinline__ void transpose4x4(cf (&v)[16])
{
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int p = q + 1; p < 4; ++p) { const cf s = v[4 * q + p]; v[4 * q + p] = v[4 * p + q]; v[4 * p + q] = s; }
}

// 16-point DFT in registers: X[k] = sum_j v[j] e^{-+ 2 pi i jk/16}; natural order in, natural order out
// HALF: v[8..15] are taken to be zero and not read.  The constant twiddles between the two radix-4 levels are split into
// a direction and a length; the lengths go into the additions of the second level: 144 instructions for 160.
template <bool INV, bool HALF = false>
__device__ __forceinline__ void fft16(cf (&v)[16])
{
    constexpr float c1 = 0.9238795325112867f, s1 = 0.3826834323650898f, r = 0.7071067811865476f, tn = 0.41421356237309503f;   // tn = s1 / c1
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (HALF) bf4_half<INV>(v[i], v[i + 4], v[i + 8], v[i + 12]);
        else bf4<INV>(v[i], v[i + 4], v[i + 8], v[i + 12]);
    }
    // v[i + 4q] now holds the q-th output of column i; its twiddle is W16^{i q}, q = 0: none
    bf4<INV>(v[0], v[1], v[2], v[3]);
    auto quarter = [](cf d) { return INV ? cf{-d.y, d.x} : cf{d.y, -d.x}; };
    // the second level with a1 = l1 u1, a3 = l1 u3, l1 and u1 +- u3 given: outputs t0 +- l1 (u1 + u3), t1 +- quarter(l1 (u1 - u3))
    auto finish = [&](int q, cf t0, cf t1, float l1, cf s, cf d) {
        const cf e = quarter(d);
        v[4 * q] = axpy(l1, s, t0); v[4 * q + 1] = axpy(l1, e, t1); v[4 * q + 2] = axpy(-l1, s, t0); v[4 * q + 3] = axpy(-l1, e, t1);
    };
    {                                            // q = 1: W^1 = c1 (1, tn), W^2 = r (1, 1), W^3 = c1 (tn, 1)
        const cf u1 = rot<INV>(v[5], tn), u2 = rot<INV>(v[6], 1.f), u3 = rotq<INV>(v[7], tn);
        finish(1, axpy(r, u2, v[4]), axpy(-r, u2, v[4]), c1, u1 + u3, u1 - u3);
    }
    {                                            // q = 2: W^2 = r (1, 1), W^4 = -+ i, W^6 = r (-1, 1)
        const cf u1 = rot<INV>(v[9], 1.f), u2 = quarter(v[10]), u3 = rotq<INV>(v[11], -1.f);
        finish(2, v[8] + u2, v[8] - u2, r, u1 + u3, u1 - u3);
    }
    {                                            // q = 3: W^3 = c1 (tn, 1), W^6 = r (-1, 1), W^9 = c1 (-1, -tn)
        const cf u1 = rotq<INV>(v[13], tn), u2 = rotq<INV>(v[14], -1.f), u3 = rot<INV>(v[15], tn);
        finish(3, axpy(r, u2, v[12]), axpy(-r, u2, v[12]), c1, u1 - u3, u1 + u3);
    }
    // v[4q + p] holds X[q + 4p]: transpose the 4x4 index back to natural order
    transpose4x4(v);
}

// the same of v[j] h^j (INV = false: conjugate), h^j = lo[j / 4 - 1] hi[0][j mod 4 - 1], with hi[q][i - 1] = h^i e^{2 pi i q i / 16}
template <bool INV>
__device__ __forceinline__ void fft16_tw(cf (&v)[16], const cf (&lo)[3], const cf (&hi)[4][3])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) bf4_tw<INV>(v[i], v[i + 4], v[i + 8], v[i + 12], lo[0], lo[1], lo[2]);
#pragma unroll
    for (int q = 0; q < 4; ++q) bf4_tw<INV>(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3], hi[q][0], hi[q][1], hi[q][2]);
    transpose4x4(v);
}

// 8-point DFT of v[0], v[1], ... in registers, natural order in, natural order out
template <bool INV>
__device__ __forceinline__ void fft8(cf* v)
{
    constexpr float r = 0.7071067811865476f;
    cf e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    bf4<INV>(e[0], e[1], e[2], e[3]);
    bf4<INV>(o[0], o[1], o[2], o[3]);
    auto tw = [](cf a, cf w) { return INV ? cmulc(a, w) : cmul(a, w); };
    o[1] = tw(o[1], cf{r, -r});
    o[2] = INV ? cf{-o[2].y, o[2].x} : cf{o[2].y, -o[2].x};        // W8^2 = -i
    o[3] = tw(o[3], cf{-r, -r});
#pragma unroll
    for (int k = 0; k < 4; ++k) { v[k] = e[k] + o[k]; v[k + 4] = e[k] - o[k]; }
}

// 3-point DFT (INV: conjugate twiddles)
template <bool INV>
__device__ __forceinline__ void dft3(cf& a, cf& b, cf& c)
{
    constexpr float s3 = 0.8660254037844386f;
    const cf t = b + c, m{a.x - 0.5f * t.x, a.y - 0.5f * t.y};
    const cf d = b - c, r = INV ? cf{-d.y, d.x} : cf{d.y, -d.x};       // d * (+i) or d * (-i)
    a = a + t; b = axpy(s3, r, m); c = axpy(-s3, r, m);
}

// DFT of 3 C points, C = 2, 4 or 8 (no twiddles: C and 3 are coprime), natural order in, natural order out
template <int C, bool INV>
__device__ __forceinline__ void dft3c(cf (&v)[3 * C])
{
    constexpr int N = 3 * C, K1 = C * (C % 3), K2 = 3 * (C == 2 ? 1 : 3);       // C (1 / C mod 3), 3 (1 / 3 mod C)
    cf u[3][C];
#pragma unroll
    for (int n2 = 0; n2 < C; ++n2) {
        cf a = v[(3 * n2) % N], b = v[(C + 3 * n2) % N], c = v[(2 * C + 3 * n2) % N];
        dft3<INV>(a, b, c);
        u[0][n2] = a; u[1][n2] = b; u[2][n2] = c;
    }
#pragma unroll
    for (int k1 = 0; k1 < 3; ++k1) {
        if constexpr (C == 8) fft8<INV>(u[k1]);
        else if constexpr (C == 4) bf4<INV>(u[k1][0], u[k1][1], u[k1][2], u[k1][3]);
        else { const cf t = u[k1][0]; u[k1][0] = t + u[k1][1]; u[k1][1] = t - u[k1][1]; }
#pragma unroll
        for (int k2 = 0; k2 < C; ++k2) v[(K1 * k1 + K2 * k2) % N] = u[k1][k2];
    }
}

// cos(2 pi i / 48)
constexpr float kCos48[48] = {
    1.0f, 0.991444861f, 0.965925826f, 0.923879533f, 0.866025404f, 0.79335334f, 0.707106781f, 0.608761429f,
    0.5f, 0.382683432f, 0.258819045f, 0.130526192f, 0.0f, -0.130526192f, -0.258819045f, -0.382683432f,
    -0.5f, -0.608761429f, -0.707106781f, -0.79335334f, -0.866025404f, -0.923879533f, -0.965925826f, -0.991444861f,
    -1.0f, -0.991444861f, -0.965925826f, -0.923879533f, -0.866025404f, -0.79335334f, -0.707106781f, -0.608761429f,
    -0.5f, -0.382683432f, -0.258819045f, -0.130526192f, 0.0f, 0.130526192f, 0.258819045f, 0.382683432f,
    0.5f, 0.608761429f, 0.707106781f, 0.79335334f, 0.866025404f, 0.923879533f, 0.965925826f, 0.991444861f};
// e^{-2 pi i e / 48}
__device__ __forceinline__ constexpr cf w48(int e) { return {kCos48[e % 48], -kCos48[(e + 36) % 48]}; }

// cos(2 pi i / 64)
constexpr float kCos64[64] = {
    1.0f, 0.995184727f, 0.98078528f, 0.956940336f, 0.923879533f, 0.881921264f, 0.831469612f, 0.773010453f,
    0.707106781f, 0.634393284f, 0.555570233f, 0.471396737f, 0.382683432f, 0.290284677f, 0.195090322f, 0.0980171403f,
    0.0f, -0.0980171403f, -0.195090322f, -0.290284677f, -0.382683432f, -0.471396737f, -0.555570233f, -0.634393284f,
    -0.707106781f, -0.773010453f, -0.831469612f, -0.881921264f, -0.923879533f, -0.956940336f, -0.98078528f, -0.995184727f,
    -1.0f, -0.995184727f, -0.98078528f, -0.956940336f, -0.923879533f, -0.881921264f, -0.831469612f, -0.773010453f,
    -0.707106781f, -0.634393284f, -0.555570233f, -0.471396737f, -0.382683432f, -0.290284677f, -0.195090322f, -0.0980171403f,
    0.0f, 0.0980171403f, 0.195090322f, 0.290284677f, 0.382683432f, 0.471396737f, 0.555570233f, 0.634393284f,
    0.707106781f, 0.773010453f, 0.831469612f, 0.881921264f, 0.923879533f, 0.956940336f, 0.98078528f, 0.995184727f};
// e^{-2 pi i e / 64}
__device__ __forceinline__ constexpr cf w64(int e) { return {kCos64[e & 63], -kCos64[(e + 48) & 63]}; }

}  // namespace luvc
