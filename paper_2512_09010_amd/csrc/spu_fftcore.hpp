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

// 16-point DFT in registers: X[k] = sum_j v[j] e^{-+ 2 pi i jk/16}; natural order in, natural order out
// HALF: v[8..15] are taken to be zero and not read
template <bool INV, bool HALF = false>
__device__ __forceinline__ void fft16(cf (&v)[16])
{
    constexpr float c1 = 0.9238795325112867f, s1 = 0.3826834323650898f, r = 0.7071067811865476f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (HALF) bf4_half<INV>(v[i], v[i + 4], v[i + 8], v[i + 12]);
        else bf4<INV>(v[i], v[i + 4], v[i + 8], v[i + 12]);
    }
    // v[i + 4q] now holds the q-th output of column i; twiddle by W16^{i q}
    const cf w1{c1, -s1}, w2{r, -r}, w3{s1, -c1}, w6{-r, -r}, w9{-c1, s1};
    auto tw = [](cf a, cf w) { return INV ? cmulc(a, w) : cmul(a, w); };
    v[1 + 4] = tw(v[1 + 4], w1);  v[1 + 8] = tw(v[1 + 8], w2);  v[1 + 12] = tw(v[1 + 12], w3);
    v[2 + 4] = tw(v[2 + 4], w2);
    v[2 + 8] = INV ? cf{-v[2 + 8].y, v[2 + 8].x} : cf{v[2 + 8].y, -v[2 + 8].x};     // W16^4 = -i
    v[2 + 12] = tw(v[2 + 12], w6);
    v[3 + 4] = tw(v[3 + 4], w3);  v[3 + 8] = tw(v[3 + 8], w6);  v[3 + 12] = tw(v[3 + 12], w9);
#pragma unroll
    for (int q = 0; q < 4; ++q) bf4<INV>(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    // v[4q + p] holds X[q + 4p]: transpose the 4x4 index back to natural order
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int p = q + 1; p < 4; ++p) { const cf s = v[4 * q + p]; v[4 * q + p] = v[4 * p + q]; v[4 * p + q] = s; }
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
