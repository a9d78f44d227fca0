// The matrix products of spu_mat.hip and spu_fold.hip: operands, values as sums of two fp16 values, circle points, loads to LDS.
#pragma once
#include <type_traits>

#include "common.hpp"
#include "spu.hpp"
#include "spu_tiles.hpp"

namespace luvc {

namespace {

typedef unsigned int mat_u32x4 __attribute__((__vector_size__(16)));
typedef float mat_f32x4 __attribute__((ext_vector_type(4)));
typedef float mat_f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 mat_f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 mat_f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 mat_bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 mat_bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ mat_f32x4 mac_f16(mat_f32x4 acc, const mat_u32x4& a, const mat_u32x4& b)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(mat_f16x8, a), __builtin_bit_cast(mat_f16x8, b), acc, 0, 0, 0);
}
__device__ __forceinline__ mat_f32x4 mac_bf16(mat_f32x4 acc, const mat_u32x4& a, const mat_u32x4& b)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(mat_bf16x8, a), __builtin_bit_cast(mat_bf16x8, b), acc, 0, 0, 0);
}

// a, b = hi + lo, two fp16 values each (nearest): 2^-24 of the value, or 2^-25 for small ones
__device__ __forceinline__ void split16(float a, float b, uint32_t& hi, uint32_t& lo)
{
    const mat_f16x2 h = __builtin_convertvector(mat_f32x2{a, b}, mat_f16x2);
    hi = __builtin_bit_cast(uint32_t, h);
    float one = 1.f;
    asm("" : "+s"(one));                         // a factor that stays: with it the difference is one instruction, taking the half as it lies
    const float ra = fmaf(-(float)h[0], one, a), rb = fmaf(-(float)h[1], one, b);
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(mat_f32x2{ra, rb}, mat_f16x2));
}
__device__ __forceinline__ uint32_t pk_bf16x2(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(mat_f32x2{a, b}, mat_bf16x2));
}
// a, b as three bf16 values each
__device__ __forceinline__ void split_bf16(double a, double b, uint32_t& t0, uint32_t& t1, uint32_t& t2)
{
    t0 = pk_bf16x2((float)a, (float)b);
    a -= (double)__uint_as_float(t0 << 16);
    b -= (double)__uint_as_float(t0 & 0xffff0000u);
    t1 = pk_bf16x2((float)a, (float)b);
    a -= (double)__uint_as_float(t1 << 16);
    b -= (double)__uint_as_float(t1 & 0xffff0000u);
    t2 = pk_bf16x2((float)a, (float)b);
}

typedef volatile __attribute__((address_space(3))) uint32_t lds_word;      // volatile: as one access for four pairs, it takes a move per word

// the largest of the 64 lanes' values (none below zero), in every lane
__device__ __forceinline__ float wave_max(float v)
{
    auto step = [&](auto ctrl, auto rows) { v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), decltype(ctrl)::value, decltype(rows)::value, 0xf, false))); };
    using all = std::integral_constant<int, 0xf>;
    step(std::integral_constant<int, 0xB1>{}, all{});            // quad_perm [1,0,3,2]
    step(std::integral_constant<int, 0x4E>{}, all{});            // quad_perm [2,3,0,1]
    step(std::integral_constant<int, 0x141>{}, all{});           // row_half_mirror
    step(std::integral_constant<int, 0x140>{}, all{});           // row_mirror
    step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});      // row_bcast:15 -> rows 1, 3
    step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});      // row_bcast:31 -> rows 2, 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// 16 (4) bytes per lane from memory to consecutive places in LDS, from the wavefront's first lane on; the caller waits for
// vmcnt.  Written out, because behind the builtin every read of LDS waits for all such loads; the scalar write of m0 has to lie
// a wait state before its use, one of the base by a vector instruction five.
__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p; }
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds(const void* base /* the same in all lanes */, uint32_t offset, uint32_t to)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(to), "v"(offset), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void load_word_to_lds(const void* from, uint32_t to)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dword %1, off sc1" :: "s"(to), "v"(from) : "memory", "m0");
}
#pragma clang diagnostic pop
// cos and sin of 2 pi num / den, 0 <= num <= den, inv = 1 / den: the eighth of the circle it falls in, then the series of either
// up to terms below 1e-15 of it.  (A third of the code of sincospi, which the first wavefronts of a compute unit fetch from
// afar: 3 us of a launch.)
__device__ __forceinline__ void circle(int num, int den, double inv, double* cosine, double* sine)
{
    int o = (int)(((float)(8 * num) + 0.5f) * (float)inv);       // exact: num <= 32768
    int rem = 8 * num - o * den;
    if (o & 1) rem = den - rem;
    const double a = 0.78539816339744830962 * ((double)rem * inv), q = a * a;
    double c = -1.0 / 87178291200.0, s = -1.0 / 1307674368000.0;             // 14!, 15!
    c = fma(c, q, 1.0 / 479001600.0);    s = fma(s, q, 1.0 / 6227020800.0);
    c = fma(c, q, -1.0 / 3628800.0);     s = fma(s, q, -1.0 / 39916800.0);
    c = fma(c, q, 1.0 / 40320.0);        s = fma(s, q, 1.0 / 362880.0);
    c = fma(c, q, -1.0 / 720.0);         s = fma(s, q, -1.0 / 5040.0);
    c = fma(c, q, 1.0 / 24.0);           s = fma(s, q, 1.0 / 120.0);
    c = fma(c, q, -0.5);                 s = fma(s, q, -1.0 / 6.0);
    c = fma(c, q, 1.0);                  s = fma(s * q, a, a);
    const bool swap = ((o + 1) & 2) != 0;
    const double x = swap ? s : c, y = swap ? c : s;
    *cosine = ((o + 2) & 4) ? -x : x;
    *sine = (o & 4) ? -y : y;
}
__device__ __forceinline__ float pow2(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }     // -126 .. 127
// e with 2^e <= m < 2^(e + 1)
__device__ __forceinline__ int exponent(float m) { return (int)((__float_as_uint(m) >> 23) & 255u) - 127; }
__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : v > hi ? hi : v; }

// The power of two that brings a wavefront's values into the range of fp16
struct MatScale {
    int e = 0;
    float f = 1.f;                               // 2^e
    bool unset = true;
};
// Places -> bins c of N1, and the twiddle, times `scale`: subsequences 4 g + v of a tile, P channel pairs.  The largest value of the lane.
template <int P>
__device__ __forceinline__ float places_to_bins(mat_f32x4 (&T)[P][2], const lds_word* buf, const mat_u32x4 (&f1)[2][3], const float2* twiddles, float scale)
{
    float wc[4], ws[4], m = 0.f;
    const float4* twr = reinterpret_cast<const float4*>(twiddles);
    const float4 w01 = twr[0], w23 = twr[1];
    wc[0] = w01.x; ws[0] = w01.y; wc[1] = w01.z; ws[1] = w01.w; wc[2] = w23.x; ws[2] = w23.y; wc[3] = w23.z; ws[3] = w23.w;
#pragma unroll
    for (int v = 0; v < 4; ++v) { wc[v] *= scale; ws[v] *= scale; }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        mat_u32x4 xa;
#pragma unroll
        for (int i = 0; i < 4; ++i) xa[i] = buf[i * 16 * 32 + p];
        mat_f32x4 y[2];
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            y[o] = mac_bf16(mat_f32x4{0.f, 0.f, 0.f, 0.f}, xa, f1[o][2]);
            y[o] = mac_bf16(y[o], xa, f1[o][1]);
            y[o] = mac_bf16(y[o], xa, f1[o][0]);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            T[p][0][v] = fmaf(y[0][v], wc[v], y[1][v] * ws[v]);
            T[p][1][v] = fmaf(y[1][v], wc[v], -y[0][v] * ws[v]);
            m = fmaxf(fmaxf(m, fabsf(T[p][0][v])), fabsf(T[p][1][v]));
        }
    }
    return m;
}
// The range of fp16: the first values that are not zero set the scale, 64 times larger ones change it; what was added up so far follows
// by the factor returned.  The scale they are met with may take them beyond fp32 (2^120 behind values of 1e-34): then they are formed
// again without it.
template <int P>
__device__ __forceinline__ float into_range(mat_f32x4 (&T)[P][2], float m, const lds_word* buf, const mat_u32x4 (&f1)[2][3], const float2* twiddles, MatScale& scale)
{
    float top = wave_max(m);
    int e = scale.e;
    if (top > 3.4028234663852886e38f) {
        top = wave_max(places_to_bins(T, buf, f1, twiddles, 1.f));
        e = 0;
    }
    const int to = clampi(e + 9 - exponent(top), -120, 120);
    const float f = pow2(clampi(to - e, -126, 126)), sums = pow2(clampi(to - scale.e, -126, 126));
#pragma unroll
    for (int p = 0; p < P; ++p) { T[p][0] *= f; T[p][1] *= f; }
    scale.e = to;
    scale.f = pow2(to);
    scale.unset = false;
    return sums;
}

}  // namespace

struct MatShape {
    double inv_N, inv_N_1, inv_N1;               // 1 / N, 1 / (N - 1), 1 / N1
    double length;                               // what the weights give back (mat_length)
    int N, N1, N2, NT /* tiles of 16 subsequences */, sigma, dn /* lowest multiple of N1 in the band, negated */, nb /* multiples */;
};
double mat_length(const MatShape& sh, double sums);

}  // namespace luvc
