// The matrix products of spu_mat.hip and spu_fold.hip: operands, values as sums of fp16 values, circle points, tokens on their way to LDS.
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

// a, b = hi + lo, two fp16 values each (nearest): off by at most 2^-23 of the value (a quarter of all fp32 values have a last bit that
// is lost), or by 2^-25 for small ones
__device__ __forceinline__ void split16(float a, float b, uint32_t& hi, uint32_t& lo)
{
    const mat_f16x2 h = __builtin_convertvector(mat_f32x2{a, b}, mat_f16x2);
    hi = __builtin_bit_cast(uint32_t, h);
    float one = 1.f;
    asm("" : "+s"(one));                         // a factor that stays: with it the difference is one instruction, taking the half as it lies
    const float ra = fmaf(-(float)h[0], one, a), rb = fmaf(-(float)h[1], one, b);
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(mat_f32x2{ra, rb}, mat_f16x2));
}
// and a third one, of what the two leave: 2^-33 of the value
__device__ __forceinline__ void split16x3(double a, double b, uint32_t& hi, uint32_t& lo, uint32_t& least)
{
    split16((float)a, (float)b, hi, lo);
    const mat_f16x2 h = __builtin_bit_cast(mat_f16x2, hi), l = __builtin_bit_cast(mat_f16x2, lo);
    const float ra = (float)(a - (double)(float)h[0] - (double)(float)l[0]), rb = (float)(b - (double)(float)h[1] - (double)(float)l[1]);
    least = __builtin_bit_cast(uint32_t, __builtin_convertvector(mat_f32x2{ra, rb}, mat_f16x2));
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

// Constants of the band stand 2^10 above their values, so that their low and third fp16 terms are no subnormal ones; the twiddles
// stand as much below theirs.
constexpr int kMatBoost = 10;
// Twiddles [row][16 columns] without a pad: the pieces of 16 bytes of a row in an order that puts those of 16 rows in different banks
__device__ __forceinline__ int tw_place(int row, int col) { return row * 16 + (((col >> 1) ^ (row >> 1 & 7)) << 1 | (col & 1)); }

// Tokens on their way to LDS, 16 subsequences (32 KB) at a time.  The older half of the wavefronts fetches: they come first where two
// share a SIMD, and would wait for the younger ones.  A thread fetches eight pieces of a chunk, the same piece of the rows of one
// subsequence s0 of a tile; places a >= N1, subsequences >= N2 and channels >= D are not used, but have to be numbers: others of
// the same sample.  Row 16 a + s holds its pieces in an order that depends on s, so that the 16 subsequences' words of a channel pair
// lie in 16 banks.
constexpr int kMatWaves = 8, kMatPairs = 4;      // wavefronts of a workgroup, channel pairs of a wavefront
constexpr int kMatThreads = 64 * kMatWaves, kMatWidth = 2 * kMatWaves * kMatPairs;
constexpr int kMatBuf = 256 * 8;                 // 16-byte pieces of a buffer: 256 rows of 8, which are 64 channels
struct MatTokens {
    const char* base;                            // the sample's first token
    uint32_t lds0, row_bytes, off, over;
    int D, N1, N2, NT, piece, wave;
    __device__ __forceinline__ MatTokens(const bf16_t* x, int64_t row_stride, int D_, int N1_, int N2_, int NT_, const void* data, int wave_)
        : base(reinterpret_cast<const char*>(x)), lds0(lds_address(data)), row_bytes((uint32_t)row_stride * 2u), D(D_), N1(N1_), N2(N2_), NT(NT_), wave(wave_)
    {
        const int s0 = (int)threadIdx.x / 8 & 15;
        piece = ((int)threadIdx.x & 7) ^ (s0 >> 1);
        off = (uint32_t)s0 * row_bytes + 16u * (uint32_t)piece;
        over = 16 * NT - 16 + s0 < N2 ? 0u : (uint32_t)(16 * NT - 15 + s0 - N2) * row_bytes;       // in the last tile
    }
    // chunk i: tile t of the channels from d on
    __device__ __forceinline__ void issue(int i, int t, int d) const
    {
        const char* from = base + (int64_t)(16 * t) * row_bytes + 2 * d;
        uint32_t less = t == NT - 1 ? over : 0u;
        if (d + 8 * piece >= D) less += 16u * (uint32_t)piece;
#pragma unroll
        for (int u = 0; u < 2 * kMatPairs; ++u) {
            int a = 2 * u + wave / 2;
            a = a < N1 ? a : N1 - 1;
            load_to_lds(from + (int64_t)(N2 * a) * row_bytes, off - less, lds0 + (uint32_t)((i % 3) * kMatBuf + u * (kMatThreads / 2) + wave * 64) * 16u);
        }
    }
    // wait for all but the newest chunk asked for
    __device__ __forceinline__ static void landed(bool newer)
    {
        if (newer) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * kMatPairs) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
};
__device__ __forceinline__ int mat_rest(int v, int n, float inv) { return v - n * (int)(((float)v + 0.5f) * inv); }      // v mod n, 0 <= v < 2^20, inv = 1 / n

// The operands on the side of the N1 places, [re, im of the result][terms][64][4]: f1t of the way there, i2t of the way back, whose
// circle has the radius `scale` (mat_place_scale).  root: e^(2 pi i k / N1).
__device__ __forceinline__ void place_operands(const double2* root, int N1, float inv_n1, double scale, uint32_t* f1t, uint32_t* i2t)
{
#pragma clang loop unroll(disable)
    for (int j = threadIdx.x; j < 512; j += kMatThreads) {
        const int w = j & 3, l = j >> 2 & 63, o = j >> 8, u = l & 15, a = 4 * (l >> 4) + w;
        double2 q = root[mat_rest(a < N1 && u < N1 ? a * u : 0, N1, inv_n1)];
        if (a >= N1 || u >= N1) q = make_double2(0.0, 0.0);
        uint32_t t0, t1, t2;
        split_bf16(o ? -q.y : q.x, o ? q.x : q.y, t0, t1, t2);
        uint32_t* to = f1t + o * 768 + l * 4 + w;
        to[0] = t0; to[256] = t1; to[512] = t2;
        const int c0 = 4 * (l >> 4) + 2 * (w & 1);           // u is a place here, c0 and c0 + 1 are bins
        const double2 q0 = root[mat_rest(c0 < N1 && u < N1 ? c0 * u : 0, N1, inv_n1)], q1 = root[mat_rest(c0 + 1 < N1 && u < N1 ? (c0 + 1) * u : 0, N1, inv_n1)];
        const bool sine = (w >> 1) != o;
        const double by = sine && !o ? -scale : scale;
        const float v0 = c0 < N1 && u < N1 ? (float)(by * (sine ? q0.y : q0.x)) : 0.f, v1 = c0 + 1 < N1 && u < N1 ? (float)(by * (sine ? q1.y : q1.x)) : 0.f;
        split16(v0, v1, t0, t1);
        to = i2t + o * 512 + l * 4 + w;
        to[0] = t0; to[256] = t1;
    }
}

// The power of two that brings a wavefront's values into the range of fp16
struct MatScale {
    int e = 0;
    float f = 1.f;                               // 2^e
    bool unset = true;
};
// Places -> bins c of N1, and the twiddle (two pieces of its row: subsequences 4 g, 4 g + 1 and 4 g + 2, 4 g + 3), times `scale`:
// subsequences 4 g + v of a tile, P channel pairs.  The largest value of the lane.
struct MatTwiddles { const float2 *w01, *w23; };
template <int P>
__device__ __forceinline__ float places_to_bins(mat_f32x4 (&T)[P][2], const lds_word* buf, const mat_u32x4 (&f1)[2][3], const MatTwiddles& twiddles, float scale)
{
    float wc[4], ws[4], m = 0.f;
    const float4 w01 = *reinterpret_cast<const float4*>(twiddles.w01), w23 = *reinterpret_cast<const float4*>(twiddles.w23);
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
__device__ __forceinline__ float into_range(mat_f32x4 (&T)[P][2], float m, const lds_word* buf, const mat_u32x4 (&f1)[2][3], const MatTwiddles& twiddles, MatScale& scale)
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
// The twiddle (wc, ws) and bins c -> places, of a tile on the way back: energies of its subsequence c at places 4 g + v, added up over P pairs
template <int P>
__device__ __forceinline__ void bins_to_energies(float (&sum)[4], const mat_f32x4 (&z)[P][2], const float (&wc)[4], const float (&ws)[4], const mat_u32x4 (&i2)[2][2])
{
#pragma unroll
    for (int p = 0; p < P; ++p) {
        float u[2][4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            u[0][v] = fmaf(z[p][0][v], wc[v], -z[p][1][v] * ws[v]);
            u[1][v] = fmaf(z[p][1][v], wc[v], z[p][0][v] * ws[v]);
        }
        mat_u32x4 uh, ul;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            uint32_t h, l;
            split16(u[w >> 1][2 * (w & 1)], u[w >> 1][2 * (w & 1) + 1], h, l);
            uh[w] = h; ul[w] = l;
        }
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            mat_f32x4 y = mac_f16(mat_f32x4{0.f, 0.f, 0.f, 0.f}, i2[o][0], ul);
            y = mac_f16(y, i2[o][1], uh);
            y = mac_f16(y, i2[o][0], uh);
#pragma unroll
            for (int v = 0; v < 4; ++v) sum[v] = fmaf(y[v], y[v], sum[v]);
        }
    }
}

}  // namespace

struct MatShape {
    double inv_N, inv_N_1, inv_N1;               // 1 / N, 1 / (N - 1), 1 / N1
    double place_scale, energy;                  // mat_scales
    int N, N1, N2, NT /* tiles of 16 subsequences */, sigma, dn /* lowest multiple of N1 in the band, negated */, nb /* multiples */;
    int down;                                    // the power of two next to N place_scale, which energies in fp32 are without: half to twice what they are
};
void mat_scales(MatShape* sh, int ways);

}  // namespace luvc
