// SPU score (paper Section 3.3, Eq. 4-8) for any number of tokens and any pass band: one transform of M = 1536 to 16384
// points forward, one back, all of it in the registers and the LDS of a workgroup.
//
// Eq. 4-7 together are a circular convolution of length N with the even kernel
//     p[j] = 1/N sum_{|f| <= sigma} M[f] e^{2 pi i f j / N}.
// N = M: the spectrum of the kernel is the mask itself, M[f] / N.  Any other N <= M / 2: the tokens are followed by M - N
// zeros and the kernel is laid out over the lags -(N - 1) .. N - 1, so that the M-point circular convolution equals the
// N-point one on the N tokens; its spectrum (real and even, like the kernel's) is
//     P[k] = 1/(N M) sum_{|f| <= sigma} M[f] sin((2 N - 1) pi u) / sin(pi u),   u = f / N - k / M,
// evaluated in fp64 by spu_conv_spectrum.  Nothing about N has to factor.
//
// Two channels of a token are one complex value (the filter is real).  A workgroup holds P channel pairs at a time:
//   A    thread (pair c, column n2 of C = 256, or 128 for M <= 2048): tokens n2, n2 + C, ... straight from memory, R-point DFT
//        (M = R C) in registers over them, twiddle W_M^{k1 n2}, row k1 of the exchange grid [R][C][P] gets the result;
//   B,C  the points of a row = 16 x 16 (16 x 8): both passes, the spectrum and the two inverse passes run inside one wavefront, in
//        place, so nothing but the order of one wavefront's LDS accesses stands between them;
//   A'   thread (c, n2) again: twiddle, R-point inverse DFT, |.|^2 added to the thread's R (R/2) token energies.
// Two barriers per P pairs; the next pairs' tokens are fetched while B and C run.  A workgroup walks the pairs in steps of
// the number of workgroups of its sample, so that at any time neighbouring workgroups (same XCD) read neighbouring
// 4 P-byte pieces of the same cache lines, and keeps the energies in registers until its last pairs are done.
// An access of a wavefront touches up to 64 / P cache lines and takes the memory path as many cycles and more, so that
// the next tokens, asked for all at once, fill its queue and the wavefronts stand still before the barrier until it has
// taken them.  They are asked for a few at a time between the transforms of B and C.  And where N = M, workgroups that read
// nothing but one cache line in eight, bytes 384 .. 511 of every 1024, end later than the others (4x4096x3584 bf16, seven steps: 81 us
// after the start of the first step, the others 71 to 72; the same with rows 8 KB apart; with the four steps of 2048 channels all end
// together), so a workgroup moves on by kConvTurn places with every step.  us of a call on tokens that no cache holds, asked for all at
// once, in parts, and in parts with the turn: bf16 8x700x3584 57, 54, 54; 8x1000x3584 74, 67, 67; 8x1200x3584 107, 98, 98; 2x3000x3584 96,
// 82, 79; 1x5245x3328 157, 130, 130; 1x8000x2048 164, 140, 135; 8x2048x3584 91, 75, 73; 4x4096x3584 108, 96, 84; 2x8192x2048 110, 98, 88;
// fp32 8x1200x3584 125, 102, 102; 2x3000x3584 112, 88, 82; 8x2048x3584 122, 101, 94; 4x4096x3584 155, 159, 141.
// With half of the inputs zero and half of the outputs unwanted (N <= M / 2) passes A and A' take half the loads and skip a
// butterfly level each.
// M is the smallest that fits, a power of two or three times one: the longer transform costs its zeros (measured before the tokens
// were asked for in parts: 8x1000x3584 bf16: 152 us on 4096 points, 77 on 2048; 8x2048x3584: 208 and 88; 8x700x3584: 76 on
// 2048, 62 on 1536; 8x1200x3584: 138 on 4096, 110 on 3072; 1x5245x3328: 190 on 16384, 160 on 12288).
//
// Bound: fp32 vector arithmetic (about 5 M log2 M flops per direction and pair) and the LDS traffic beside it (64 bytes per
// point and pair).
#include <type_traits>

#include "common.hpp"
#include "spu.hpp"
#include "spu_fftcore.hpp"
#include "spu_tiles.hpp"

namespace luvc {

namespace {

// R-point DFT across the registers of a thread, natural order in and out; HALF: inputs j >= R/2 are zero and not read
// (forward), outputs j >= R/2 are not formed (inverse)
template <int R, bool HALF> struct dft_cols_pow2;
template <bool HALF> struct dft_cols_pow2<16, HALF> {
    __device__ static __forceinline__ void fwd(cf (&v)[16]) { fft16<false, HALF>(v); }
    __device__ static __forceinline__ void inv(cf (&v)[16]) { fft16<true>(v); }
};
template <bool HALF> struct dft_cols_pow2<32, HALF> {
    __device__ static __forceinline__ void fwd(cf (&v)[32])
    {
        cf e[16], o[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const cf a = v[j], s = HALF ? a : a + v[j + 16], d = HALF ? a : a - v[j + 16];
            e[j] = s;
            o[j] = j ? cmul(d, w64(2 * j)) : d;
        }
        fft16<false>(e);
        fft16<false>(o);
#pragma unroll
        for (int q = 0; q < 16; ++q) { v[2 * q] = e[q]; v[2 * q + 1] = o[q]; }
    }
    __device__ static __forceinline__ void inv(cf (&v)[32])
    {
        cf e[16], o[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) { e[q] = v[2 * q]; o[q] = v[2 * q + 1]; }
        fft16<true>(e);
        fft16<true>(o);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const cf t = j ? cmulc(o[j], w64(2 * j)) : o[j];
            v[j] = e[j] + t;
            if (!HALF) v[j + 16] = e[j] - t;
        }
    }
};
template <bool HALF> struct dft_cols_pow2<64, HALF> {
    __device__ static __forceinline__ void fwd(cf (&v)[64])
    {
        cf u[4][16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            cf a0 = v[j], a1 = v[j + 16], a2 = HALF ? cf{0.f, 0.f} : v[j + 32], a3 = HALF ? cf{0.f, 0.f} : v[j + 48];
            if (HALF) bf4_half<false>(a0, a1, a2, a3);
            else bf4<false>(a0, a1, a2, a3);
            u[0][j] = a0;
            u[1][j] = j ? cmul(a1, w64(j)) : a1;
            u[2][j] = j ? cmul(a2, w64(2 * j)) : a2;
            u[3][j] = j ? cmul(a3, w64(3 * j)) : a3;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            fft16<false>(u[s]);
#pragma unroll
            for (int q = 0; q < 16; ++q) v[4 * q + s] = u[s][q];
        }
    }
    __device__ static __forceinline__ void inv(cf (&v)[64])
    {
        cf u[4][16];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int q = 0; q < 16; ++q) u[s][q] = v[4 * q + s];
            fft16<true>(u[s]);
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            cf a0 = u[0][j];
            cf a1 = j ? cmulc(u[1][j], w64(j)) : u[1][j];
            cf a2 = j ? cmulc(u[2][j], w64(2 * j)) : u[2][j];
            cf a3 = j ? cmulc(u[3][j], w64(3 * j)) : u[3][j];
            bf4<true>(a0, a1, a2, a3);
            v[j] = a0;
            v[j + 16] = a1;
            if (!HALF) { v[j + 32] = a2; v[j + 48] = a3; }
        }
    }
};

// R = 12, 24, 48, zeros in the upper half
template <int R> struct dft_cols_three {
    static_assert(R % 12 == 0 && 48 % R == 0, "");
    static constexpr int S = 48 / R;
    __device__ static __forceinline__ void fwd(cf (&v)[R])
    {
        cf e[R / 2], o[R / 2];
#pragma unroll
        for (int j = 0; j < R / 2; ++j) { e[j] = v[j]; o[j] = j ? cmul(v[j], w48(S * j)) : v[j]; }
        dft3c<R / 6, false>(e);
        dft3c<R / 6, false>(o);
#pragma unroll
        for (int q = 0; q < R / 2; ++q) { v[2 * q] = e[q]; v[2 * q + 1] = o[q]; }
    }
    __device__ static __forceinline__ void inv(cf (&v)[R])
    {
        cf e[R / 2], o[R / 2];
#pragma unroll
        for (int q = 0; q < R / 2; ++q) { e[q] = v[2 * q]; o[q] = v[2 * q + 1]; }
        dft3c<R / 6, true>(e);
        dft3c<R / 6, true>(o);
#pragma unroll
        for (int j = 0; j < R / 2; ++j) v[j] = e[j] + (j ? cmulc(o[j], w48(S * j)) : o[j]);
    }
};

template <int R, bool HALF> using dft_cols = std::conditional_t<R % 3 == 0, dft_cols_three<R % 3 == 0 ? R : 12>, dft_cols_pow2<R % 3 == 0 ? 16 : R, HALF>>;

// one channel pair as it lies in memory: by buffer access (one instruction, bounds by the descriptor) or element by element
template <typename T> struct raw_pair;
template <> struct raw_pair<bf16_t> {
    uint32_t v;
    __device__ static __forceinline__ raw_pair load(__amdgpu_buffer_rsrc_t r, uint32_t off) { return {__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0)}; }
    __device__ static __forceinline__ raw_pair load(const bf16_t* p, bool second)
    {
        const uint32_t lo = p[0].bits, hi = second ? p[1].bits : 0u;
        return {lo | (hi << 16)};
    }
    __device__ __forceinline__ cf widen() const { return {__uint_as_float(v << 16), __uint_as_float(v & 0xffff0000u)}; }
};
typedef unsigned int u32x2 __attribute__((__vector_size__(8)));
template <> struct raw_pair<float> {
    u32x2 v;
    __device__ static __forceinline__ raw_pair load(__amdgpu_buffer_rsrc_t r, uint32_t off) { return {__builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0)}; }
    __device__ static __forceinline__ raw_pair load(const float* p, bool second)
    {
        raw_pair o;
        o.v[0] = __float_as_uint(p[0]);
        o.v[1] = second ? __float_as_uint(p[1]) : 0u;
        return o;
    }
    __device__ __forceinline__ cf widen() const { return {__uint_as_float(v[0]), __uint_as_float(v[1])}; }
};

// Sixteen values times W^{exponent(i)}, exponent(0) = 0, out of the table twb, forward or inverse, handed to `put` one by
// one.  The twiddles come from LDS in groups: read one at a time, each would wait for the write before it (the compiler
// cannot tell the table from the exchange grid), all at once they would not fit beside the values.
template <bool INV, int GROUP, typename E, typename F>
__device__ __forceinline__ void twiddled(const cf (&v)[16], const float2* twb, E exponent, F put)
{
#pragma unroll
    for (int i0 = 0; i0 < 16; i0 += GROUP) {
        __builtin_amdgcn_sched_barrier(0);
        float2 w[GROUP];
#pragma unroll
        for (int i = 0; i < GROUP; ++i) w[i] = twb[exponent(i0 + i)];
#pragma unroll
        for (int i = 0; i < GROUP; ++i) {
            const cf t{w[i].x, w[i].y};
            put(i0 + i, i0 + i == 0 ? v[0] : INV ? cmul(v[i0 + i], t) : cmulc(v[i0 + i], t));
        }
    }
}

// The lane, formed anew in every step of the kernel: the places derived from it are worked out where they are used instead of being
// kept.  (The step is an operand for the sake of the compiler, which would form the lane once; ID tells the uses of a step apart.)
template <int ID>
__device__ __forceinline__ int fresh_lane(int step)
{
    int l;
    asm("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(l) : "s"(step), "n"(ID));
    return l;
}

// LDS accesses of one wavefront are served in order: this only keeps the compiler from moving them
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

}  // namespace

// The constants of the transforms as fp32 values are short: cos(pi / 8) by 2.9e-8, 1 / sqrt 2 by 1.7e-8, and a token passes four
// to six transforms there and back.  All scores came out too small by this share (mean over the tokens against fp64,
// white and smooth tokens of 700 to 16384: 6.7e-8 .. 8.2e-8 up to 4096 points, 7.6e-8 .. 9.8e-8 beyond, beside 3e-8 of noise);
// the weights, which are worked out in fp64, give it back.
__host__ __device__ constexpr double conv_length(int M) { return M <= 4096 ? 1.0 + 7.4e-8 : 1.0 + 8.9e-8; }

// P[k], k = 0 .. M/2.  A workgroup owns kSpecBins bins; its threads split the frequencies f >= 1 of each bin.  With
// a = pi f / N and b = pi k / M the terms of +f and -f add to
//     -sin(2 pi N k / M) sin 2b / (sin(a - b) sin(a + b)) - 2 cos(2 pi N k / M),
// and to 2 N - 2 where f / N = k / M (4 N - 2 where both are 1/2: then -f / N and k / M differ by 1).
constexpr int kSpecBins = 8, kSpecLanes = 256 / kSpecBins;
__global__ void __launch_bounds__(256)
spu_conv_spectrum(int N, int M, int sigma, int use_hamming, float* __restrict__ spec /* [M/2 + 1] */)
{
    __shared__ double sn[256], cs[256], wt[256];
    __shared__ double part[kSpecBins][kSpecLanes];
    const int tid = threadIdx.x, g = tid / kSpecLanes, l = tid % kSpecLanes;
    const int k = blockIdx.x * kSpecBins + g;
    double sb, cb, s2, c2, sk, ck;
    sincospi((double)k / (double)M, &sb, &cb);
    sincospi(2.0 * (double)k / (double)M, &s2, &c2);
    sincospi(2.0 * (double)((N * k) % M) / (double)M, &sk, &ck);       // all products stay below 2^28
    double acc = 0.0;
    for (int f0 = 1; f0 <= sigma; f0 += 256) {
        const int f = f0 + tid;
        __syncthreads();
        if (f <= sigma) {
            double s, c;
            sincospi((double)f / (double)N, &s, &c);
            sn[tid] = s;
            cs[tid] = c;
            // 2 sigma = N: the bins f = N/2 and f = -N/2 are the same one
            wt[tid] = (2 * f == N ? 0.5 : 1.0) * (use_hamming ? 0.54 + 0.46 * cospi(2.0 * (double)f / (double)(N - 1)) : 1.0);
        }
        __syncthreads();
        const int cnt = sigma - f0 + 1 < 256 ? sigma - f0 + 1 : 256;
        for (int i = l; i < cnt; i += kSpecLanes) {
            const double d = sn[i] * cb - cs[i] * sb, s = sn[i] * cb + cs[i] * sb;
            const bool same = (f0 + i) * M == k * N;
            // 1 / (d s): the hardware's estimate and two Newton steps
            const double q = d * s;
            double inv = __builtin_amdgcn_rcp(q);
            inv = fma(fma(-q, inv, 1.0), inv, inv);
            inv = fma(fma(-q, inv, 1.0), inv, inv);
            const double t = same ? (2 * k == M ? 4.0 : 2.0) * (double)N - 2.0 : fma(-sk * s2, inv, -2.0 * ck);
            acc += wt[i] * t;
        }
    }
    part[g][l] = acc;
    __syncthreads();
    if (l == 0 && k <= M / 2) {
        double tot = k == 0 ? 2.0 * (double)N - 1.0 : sk * cb / sb - ck;            // f = 0, weight 1
        for (int i = 0; i < kSpecLanes; ++i) tot += part[g][i];
        spec[k] = (float)(tot / ((double)N * (double)M) * conv_length(M));
    }
}

// Tokens of the next group, of JN, that have been asked for behind a point of a step.  fp32, N = M: from the second point on, there are
// no registers for them before.
template <typename T, bool HALF>
constexpr int conv_part(int point, int points, int JN)
{
    if (point == points - 1) return JN;
    return HALF || sizeof(T) == 2 ? (point + 1) * JN / (points - 1) : point * JN / (points - 1);
}
// Places a workgroup moves on by with every step: for bf16 and P = 4 (4096 points) a cache line of them; with fp32 tokens or another P it
// is another part of a line or several, and was not chosen for those.  Where N = M it gains 2 to 13 %, behind zeros up to 7 % on 6144 and
// 16384 points, nothing on up to 4096 or where a sample has 8 workgroups (nothing turns); fp32 1x5245x3328 loses, 140 us against 136.
constexpr int kConvTurn = 8;

template <typename T, int R, int LB, int P, bool HALF /* N <= M/2: zeros behind the tokens; else N = M */, bool PAIRED /* every pair is one aligned access */>
__global__ void __launch_bounds__(16 * LB * P)
spu_conv(const T* __restrict__ x, int N, int D, int64_t row_stride, int sigma, int use_hamming,
         const float* __restrict__ spec /* HALF: [M/2 + 1] */, int n_groups /* of P pairs, per sample */,
         int ld, float* __restrict__ partial /* [B, n_tiles, ld] */, float* __restrict__ gpartial, const TileSync sy,
         float* __restrict__ scores /* [B, N] */)
{
    constexpr int COLS = 16 * LB, M = COLS * R, THREADS = COLS * P, JN = HALF ? R / 2 : R;
    constexpr int LROW = (COLS + LB) * P;        // complex values per row of the exchange grid: a pad of P after every 16 columns
    constexpr int ROWS = 64 / (LB * P), NIT = (R + 15) / 16;       // rows a wavefront takes at a time, and how often
    constexpr bool SPEC_LDS = R <= 16;           // the spectrum in LDS (registers are short at 1024 threads) or in registers
    extern __shared__ float2 sm[];               // [R][LROW]; the M-entry table while the twiddles are picked
    float2* twb = sm + R * LROW;                 // [COLS] (cos, sin)(2 pi i / COLS)
    float* sp = reinterpret_cast<float*>(twb + COLS);              // SPEC_LDS: [R k1][16 i][LB lw]
    __shared__ int flag;
    const int tid = threadIdx.x, c = tid % P, n2 = tid / P, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_tiles = gridDim.x;
    const unsigned item = xcd_contiguous(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
    const int tile = item % n_tiles, b = item / n_tiles;

    const T* xs = x + (int64_t)b * N * row_stride;
    using raw_t = raw_pair<T>;
    raw_t raw[JN];
    // FRESH: the registers of 1024 threads do not hold the places of a thread in memory and in the grid beside R points.  A place that
    // is spilled and read back behind a fetch is a wait for the tokens.
    constexpr bool FRESH = R <= 16 && (!PAIRED || (R == 16 && (LB == 16 || !HALF)));
    // PAIRED: the descriptor ends with the sample's last token (a lane past it, or past D, reads zeros)
    const uint32_t row_bytes = (uint32_t)row_stride * (uint32_t)sizeof(T);
    const uint32_t lane_off = (uint32_t)n2 * row_bytes + (uint32_t)c * 2u * (uint32_t)sizeof(T);
    auto fetch = [&](auto id, int g, int from, int to) {           // tokens from .. to - 1 of this thread
        const int l = FRESH ? fresh_lane<decltype(id)::value>(g) : 0, fc = FRESH ? l % P : c, fn2 = FRESH ? wave * (64 / P) + l / P : n2, d0 = (g * P + fc) * 2;
        if constexpr (PAIRED) {
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<T*>(xs) + 2 * P * g, 0, (int)((uint32_t)(N - 1) * row_bytes + (uint32_t)((D - 2 * P * g) * (int)sizeof(T))), 0x00020000);
            const uint32_t own = FRESH ? (uint32_t)fn2 * row_bytes + (uint32_t)fc * 2u * (uint32_t)sizeof(T) : lane_off, off = d0 < D ? own : 0x80000000u;
#pragma unroll
            for (int j = 0; j < JN; ++j)
                if (j >= from && j < to) raw[j] = raw_t::load(r, off + (uint32_t)(j * COLS) * row_bytes);
        } else {
            const bool live = d0 < D, second = d0 + 1 < D;
            const T* p = xs + (live ? d0 : 0);
#pragma unroll
            for (int j = 0; j < JN; ++j) {
                const int n = COLS * j + fn2;
                const bool there = live && (!HALF || n < N);
                if (j >= from && j < to) raw[j] = there ? raw_t::load(p + (int64_t)n * row_stride, second) : raw_t{};
            }
        }
    };
    // The next group's tokens are asked for in parts, point by point of a step: 0 after A, three in every iteration of B and C, the
    // last behind them.
    constexpr int POINTS = 3 * NIT + 2;
    auto upto = [&](int point) { return conv_part<T, HALF>(point, POINTS, JN); };
    fetch(std::integral_constant<int, 10>{}, tile, 0, JN);

    // ---- tables: one octant of the circle in fp64, rounded once, the rest by symmetry
    for (int i = tid; i <= M / 8; i += THREADS) {
        double sd, cd;
        sincospi(2.0 * (double)i / (double)M, &sd, &cd);
        const float cs = (float)cd, sn = (float)sd;
        constexpr int n4 = M / 4, nh = M / 2, n34 = nh + n4;
        sm[i] = make_float2(cs, sn);
        sm[n4 - i] = make_float2(sn, cs);
        sm[n4 + i] = make_float2(-sn, cs);
        sm[nh - i] = make_float2(-cs, sn);
        sm[nh + i] = make_float2(-cs, -sn);
        sm[n34 - i] = make_float2(-sn, -cs);
        sm[n34 + i] = make_float2(sn, -cs);
        if (i) sm[M - i] = make_float2(cs, -sn);
    }
    auto weight = [&](int k) {                   // P[k] / mask
        const int f = k <= M / 2 ? k : M - k;
        if (HALF) return spec[f];
        float w = 0.f;
        if (f <= sigma) {
            double v = 1.0;
            if (use_hamming) v = 0.54 + 0.46 * cospi(2.0 * (double)f / (double)(N - 1));
            w = (float)(v / (double)N * conv_length(M));
        }
        return w;
    };
    const int lw = lane / P % LB;                // b of pass B; in pass C, a lane holds ka = lw (LB = 16) or ka = 2 lw and 2 lw + 1 (LB = 8)
    const int wrow = (tid >> 6) * ROWS + lane / (LB * P);          // row within an iteration's 16
    auto bin = [&](int k1, int i, int l) { return k1 + R * (LB == 16 ? l + 16 * i : 2 * l + (i >> 3) + 16 * (i & 7)); };      // of pass C's value i
    float wr[SPEC_LDS ? 1 : NIT][16];
    if (SPEC_LDS) {
        for (int i = tid; i < M; i += THREADS) sp[i] = weight(bin(i / COLS, i / LB % 16, i % LB));
    } else {
#pragma unroll
        for (int it = 0; it < NIT; ++it)
#pragma unroll
            for (int kb = 0; kb < 16; ++kb) wr[it % (SPEC_LDS ? 1 : NIT)][kb] = weight(bin(it * 16 + wrow < R ? it * 16 + wrow : 0, kb, lw));
    }
    __syncthreads();
    // W_M^{k1 n2} (conjugated on use).  N = M, where a thread holds R tokens and R sums, or fp32 tokens, or eight pairs: the
    // upper half as W_C^{n2} conj(W_M^{(R - k1) n2}), so that the rest stays in registers - what spills goes through L2, and
    // the cache lines of the tokens, which neighbouring workgroups share, have left it when the next one asks (4x4096x3584
    // bf16 out of HBM with all of them kept and spilled: 313 MB fetched for 117, 172 us against 109).
    constexpr bool FOLD = !HALF || sizeof(T) == 4 || LB == 8;
    constexpr int KEPT = FOLD ? R / 2 + 1 : R;
    cf wa[KEPT], wtop{0.f, 0.f};
#pragma unroll
    for (int k1 = 1; k1 < KEPT; ++k1) { const float2 w = sm[k1 * n2]; wa[k1] = {w.x, w.y}; }
    if (FOLD) { const float2 w = sm[R * n2]; wtop = {w.x, w.y}; }
    auto tw_a = [&](int k1) { return k1 < KEPT ? wa[k1 < KEPT ? k1 : 0] : cmulc(wtop, wa[k1 < KEPT ? 0 : R - k1]); };
    if (tid < COLS) twb[tid] = sm[tid * R];
    float acc[JN];
#pragma unroll
    for (int j = 0; j < JN; ++j) acc[j] = 0.f;
    __syncthreads();

    float2* kept_col = sm + (n2 + n2 / 16) * P + c;
    auto column = [&](auto id, int step) {       // this thread's column of the grid
        if (!FRESH) return kept_col;
        const int l = fresh_lane<decltype(id)::value>(step), n2 = wave * (64 / P) + l / P;
        return sm + (n2 + n2 / 16) * P + l % P;
    };
    tile_tag_t seen = 0;
    for (int g = tile, round = 0, turned = tile; g < n_groups;) {
        round += n_tiles;
        turned = (turned + kConvTurn) % n_tiles;
        const int next = round + turned;
        const bool fetches = next < n_groups;
        auto fetch_part = [&](auto id, int point) { if (fetches) fetch(id, next, point ? upto(point - 1) : 0, upto(point)); };
        // ---- A
        if (FOLD) asm("" : "+v"(wtop.x), "+v"(wtop.y) : "s"(g), "n"(5));         // the products with it are formed where they are used, not kept
        {
            float2* col = column(std::integral_constant<int, 1>{}, g);
            cf v[R];
#pragma unroll
            for (int j = 0; j < JN; ++j) v[j] = raw[j].widen();
            dft_cols<R, HALF>::fwd(v);
            col[0] = make_float2(v[0].x, v[0].y);
#pragma unroll
            for (int k1 = 1; k1 < R; ++k1) {
                const cf r = cmulc(v[k1], tw_a(k1));
                col[k1 * LROW] = make_float2(r.x, r.y);
            }
        }
        if (!fetches) seen = tiles_look(sy, b, tile, n_tiles);
        fetch_part(std::integral_constant<int, 11>{}, 0);
        __syncthreads();
        // ---- B, C, spectrum, C', B'
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            if (R % 16 != 0 && (it * 16 + wave * ROWS >= R)) {                     // a whole wavefront: R is a multiple of ROWS
                if (fetches) fetch(std::integral_constant<int, 12>{}, next, upto(3 * it), upto(POINTS - 2));
                break;
            }
            const int l = FRESH ? fresh_lane<3>(g + it) : lane, k1 = FRESH ? it * 16 + wave * ROWS + l / (LB * P) : it * 16 + wrow;
            int lt = FRESH ? l / P % LB : lw;
            if (!FRESH) asm volatile("" : "+v"(lt));                     // the places of the twiddles are formed here, not kept
            const int rl = FRESH ? lt : lw;
            float2* row = sm + k1 * LROW + (FRESH ? l % P : c);
            cf v[16];
#pragma unroll
            for (int a = 0; a < 16; ++a) { const float2 q = row[(a * LB + a * LB / 16 + rl) * P]; v[a] = {q.x, q.y}; }
            fft16<false>(v);
            twiddled<false, R <= 16 ? 4 : 8>(v, twb, [&](int ka) { return ka * lt; }, [&](int ka, cf r) { row[(ka * LB + ka * LB / 16 + rl) * P] = make_float2(r.x, r.y); });
            wave_lds_fence();
            fetch_part(std::integral_constant<int, 13>{}, 3 * it + 1);
#pragma unroll
            for (int i = 0; i < 16; ++i) { const float2 q = row[(17 * rl + i) * P]; v[i] = {q.x, q.y}; }
            if constexpr (LB == 16) fft16<false>(v);
            else { fft8<false>(v); fft8<false>(v + 8); }
#pragma unroll
            for (int kb = 0; kb < 16; ++kb) {
                const float w = SPEC_LDS ? sp[(k1 * 16 + kb) * LB + rl] : wr[it % (SPEC_LDS ? 1 : NIT)][kb];
                v[kb] = {v[kb].x * w, v[kb].y * w};
            }
            fetch_part(std::integral_constant<int, 14>{}, 3 * it + 2);
            if constexpr (LB == 16) fft16<true>(v);
            else { fft8<true>(v); fft8<true>(v + 8); }
            twiddled<true, R <= 16 ? 4 : 8>(v, twb, [&](int i) { return LB == 16 ? i * lt : (i & 7) * (2 * lt + (i >> 3)); }, [&](int i, cf r) { row[(17 * rl + i) * P] = make_float2(r.x, r.y); });
            wave_lds_fence();
            fetch_part(std::integral_constant<int, 15>{}, 3 * it + 3);
#pragma unroll
            for (int ka = 0; ka < 16; ++ka) { const float2 q = row[(ka * LB + ka * LB / 16 + rl) * P]; v[ka] = {q.x, q.y}; }
            fft16<true>(v);
#pragma unroll
            for (int a = 0; a < 16; ++a) row[(a * LB + a * LB / 16 + rl) * P] = make_float2(v[a].x, v[a].y);
        }
        __syncthreads();
        fetch_part(std::integral_constant<int, 16>{}, POINTS - 1);
        // ---- A'
        if (FOLD) asm("" : "+v"(wtop.x), "+v"(wtop.y) : "s"(g), "n"(6));
        {
            cf v[R];
            const float2* col = column(std::integral_constant<int, 2>{}, g);
            { const float2 q = col[0]; v[0] = {q.x, q.y}; }
#pragma unroll
            for (int k1 = 1; k1 < R; ++k1) { const float2 q = col[k1 * LROW]; v[k1] = cmul(cf{q.x, q.y}, tw_a(k1)); }
            dft_cols<R, HALF>::inv(v);
#pragma unroll
            for (int j = 0; j < JN; ++j) acc[j] = fmaf(v[j].x, v[j].x, fmaf(v[j].y, v[j].y, acc[j]));
        }
        g = next;
    }
    tiles_claim(sy, b, tile, n_tiles, seen);
    // ---- Eq. 8: over the P pairs of a thread group, then across the workgroups of the sample
    float* pout = partial + ((int64_t)b * n_tiles + tile) * ld;
#pragma unroll
    for (int j = 0; j < JN; ++j) {
        float e = acc[j];
        if (P >= 2) e += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(e), 0xB1, 0xf, 0xf, false));    // quad_perm [1,0,3,2]
        if (P >= 4) e += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(e), 0x4E, 0xf, 0xf, false));    // quad_perm [2,3,0,1]
        if (P >= 8) e += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(e), 0x141, 0xf, 0xf, false));   // row_half_mirror
        const int n = COLS * j + n2;
        if (c == 0 && n < ld) tile_store(pout + n, n < N ? e : 0.f);
    }
    tiles_to_scores<THREADS>(partial, gpartial, sy, scores, b, tile, n_tiles, N, ld, &flag);
}

// ------------------------------------------------------------------ host side
// Points M of the transform for N tokens; *half: zeros behind the tokens (N <= M / 2), else N = M.  0: too long.
int spu_conv_points(int N, bool* half)
{
    for (int M : {1536, 2048, 3072, 4096, 6144, 8192, 12288, 16384})
        if (2 * N <= M || (N == M && (M & (M - 1)) == 0)) { *half = N != M; return M; }
    return 0;
}

static int conv_pairs(int M) { return M <= 2048 ? 8 : M <= 4096 ? 4 : M <= 8192 ? 2 : 1; }

// Workgroups per sample.  One workgroup fills a compute unit; a workgroup's time is its pair groups plus about one more
// for tables and hand-over, and the launch takes as many rounds of that as there are multiples of 256 workgroups.  At most
// `most` of them.
int spu_conv_tiles(int B, int N, int D, int most)
{
    bool half;
    const int P = conv_pairs(spu_conv_points(N, &half)), ng = (D + 2 * P - 1) / (2 * P);
    int best = ng < most ? ng : most;
    int64_t best_cost = INT64_MAX;
    for (int g = 1; g <= ng && g <= 64; ++g) {
        const int t = (ng + g - 1) / g;
        if (t > most) continue;
        const int64_t cost = (((int64_t)B * t + 255) / 256) * (g + 1);
        if (cost < best_cost) { best_cost = cost; best = t; }
    }
    return best;
}

// us of one call as the paths are weighed with: a launch for the spectrum where one is needed, then what a workgroup starts with and its
// pair groups one after the other.  Fitted to a form of the kernel that asked for all tokens at once; most calls now take less.  Measured,
// the estimates: 8x700x3584 bf16 54 (63), 8x1000x3584 67 (79), 8x1200x3584 98 (110), 2x3000x3584 79 (95), 4x4096x3584 84 (101; fp32 141,
// 131), 8x2048x3584 73 (88; fp32 94, 113).  They keep calls of 2048 and 4096 tokens with a short pass band on spu_fft16q
// (2x2048x3584, sigma 102: 34.8 us, here 31.3; 4x4096x3584, sigma 100: 110, here 84), whose scores are closer to exact on white
// tokens (rms 3.3e-8 against 3.6e-8, 2.9e-8 against 3.0e-8).  Up to 1024 tokens they are compared with spu_circ's, which are an
// earlier form's too.
double spu_conv_us(int B, int N, int D, luvc_dtype dt)
{
    bool half;
    const int M = spu_conv_points(N, &half), P = conv_pairs(M), ng = (D + 2 * P - 1) / (2 * P), t = spu_conv_tiles(B, N, D);
    const double rounds = (double)(((int64_t)B * t + 255) / 256) * ((ng + t - 1) / t);
    const bool three = M % 3 == 0;
    if (half) return 15.0 + rounds * (M <= 4096 ? (three ? 6.8 : 9.1) : M <= 8192 ? (three ? 11.4 : 14.0) : (three ? 20.7 : 25.0));
    return 14.0 + rounds * (M == 2048 ? 10.5 : 12.4) * (dt == LUVC_F32 && M <= 4096 ? 1.35 : 1.0);
}

// bf16, as measured since tokens are asked for in parts: 158 shapes of 49 to 7549 tokens, 0.92 to 1.09 of it
double spu_conv_measured_us(int B, int N, int D)
{
    bool half;
    const int M = spu_conv_points(N, &half), P = conv_pairs(M), ng = (D + 2 * P - 1) / (2 * P), t = spu_conv_tiles(B, N, D);
    const double rounds = (double)(((int64_t)B * t + 255) / 256) * ((ng + t - 1) / t);
    if (!half) return M == 2048 ? 16.0 + 8.1 * rounds : M == 4096 ? 19.0 + 9.6 * rounds : 20.0 + 17.0 * rounds;
    switch (M) {
    case 1536: return 12.5 + 6.1 * rounds;
    case 2048: return 14.0 + 7.9 * rounds;
    case 3072: return 16.0 + 6.1 * rounds;
    case 4096: return 18.0 + 8.3 * rounds;
    case 6144: return 24.0 + 7.05 * rounds;
    case 8192: return 20.0 + 10.0 * rounds;
    case 12288: return 50.0 + 10.5 * rounds;
    default: return 30.0 + 25.0 * rounds;
    }
}

size_t spu_conv_spec_bytes(int N)
{
    bool half;
    const int M = spu_conv_points(N, &half);
    return half ? sizeof(float) * (size_t)(M / 2 + 1) : 0;
}

template <typename T, int R, int LB, int P>
static void conv_launch(const T* x, int B, int N, int D, int64_t row_stride, int sigma, int use_hamming, bool half, bool aligned,
                        const float* spec, float* partial, float* gpartial, const TileSync& sy, int n_tiles, float* scores, hipStream_t st)
{
    const int ng = (D + 2 * P - 1) / (2 * P), ld = spu_conv_ld(N);
    const size_t lds = sizeof(float2) * (size_t)(R * 17 * LB * P + 16 * LB) + (R <= 16 ? sizeof(float) * 16 * LB * R : 0);
    const dim3 grid((unsigned)n_tiles, (unsigned)B), block(16 * LB * P);
#define LUVC_CONV(HF, AL) LUVC_LAUNCH("spu_conv", (spu_conv<T, R, LB, P, HF, AL>), grid, block, lds, st, x, N, D, row_stride, sigma, use_hamming, spec, ng, ld, partial, gpartial, sy, scores)
    if (half) { if (aligned) LUVC_CONV(true, true); else LUVC_CONV(true, false); }
    else if constexpr (R % 3 != 0) { if (aligned) LUVC_CONV(false, true); else LUVC_CONV(false, false); }
#undef LUVC_CONV
}

luvc_status spu_score_conv(const void* x, int B, int N, int D, int64_t row_stride, luvc_dtype dt, int sigma, int use_hamming,
                           float* spec, float* partial, float* gpartial, const TileSync& sy, int n_tiles, float* scores, hipStream_t st)
{
    bool half;
    const int M = spu_conv_points(N, &half);
    const size_t es = dt == LUVC_F32 ? 4 : 2;
    // a sample, rounded up to M tokens, has to stay below the offset that marks a lane without channels
    const bool aligned = (row_stride % 2 == 0) && ((uintptr_t)x % (2 * es) == 0) && (D % 2 == 0) && (int64_t)M * row_stride * (int64_t)es < ((int64_t)1 << 31);
    if (half) {
        LUVC_LAUNCH("spu_conv_spectrum", spu_conv_spectrum, dim3((unsigned)(M / 2 / kSpecBins + 1)), dim3(256), 0, st, N, M, sigma, use_hamming, spec);
    }
#define LUVC_CONV_S(TT, R, LB, P) conv_launch<TT, R, LB, P>((const TT*)x, B, N, D, row_stride, sigma, use_hamming, half, aligned, spec, partial, gpartial, sy, n_tiles, scores, st)
#define LUVC_CONV_R(TT) do { \
        if (M == 1536)       LUVC_CONV_S(TT, 12, 8, 8); \
        else if (M == 2048)  LUVC_CONV_S(TT, 16, 8, 8); \
        else if (M == 3072)  LUVC_CONV_S(TT, 12, 16, 4); \
        else if (M == 4096)  LUVC_CONV_S(TT, 16, 16, 4); \
        else if (M == 6144)  LUVC_CONV_S(TT, 24, 16, 2); \
        else if (M == 8192)  LUVC_CONV_S(TT, 32, 16, 2); \
        else if (M == 12288) LUVC_CONV_S(TT, 48, 16, 1); \
        else                 LUVC_CONV_S(TT, 64, 16, 1); \
    } while (0)
    if (dt == LUVC_F32) LUVC_CONV_R(float); else LUVC_CONV_R(bf16_t);
#undef LUVC_CONV_R
#undef LUVC_CONV_S
    return check_launch("spu score (convolution)");
}

}  // namespace luvc
