// SPU score (paper Section 3.3, Eq. 4-8): fast path for N = N1 * N2 with N1 = 16 * Q, Q in {16, 15, 9},
// and 2*sigma + 1 <= N1 (N = 1024, 2048, 720, 144 ... of the benchmark workloads).
//
// Two real channels (d, d+1) are packed as one complex signal z = x_d + i x_{d+1}.  The mask of
// Eq. 5 is real and symmetric in k, so the filter is a real linear operator and Re / Im of the
// filtered z are the two filtered channels: no unpacking is ever needed.
//
// Transform decomposition along the token index, n = N2 (16 j + t) + n2 (n2 < N2, j < Q, t < 16), bins k1 = a + Q b of an
// N1-point transform (a < Q, b < 16):
//   Eq. 4 on the pass band:  A[a] = Q-point DFT over j of the tokens of residue t, subsequence n2;
//                            Y[a + Q b] = 16-point DFT over t of A_t[a] W_N1^{t a};
//                            F <- F W_N^k + Y, n2 falling (Horner), k = a + Q b, for b >= 8 less N1: |k| <= sigma;
//   Eq. 6:                   F *= M[|k|] / N;
//   Eq. 7:                   16-point DFT over b of F W_N^{-(k - a) n2}, then Q-point DFT over a of its outputs t times
//                            W_N^{-a (n2 + N2 t)}: the filtered tokens of residue t, subsequence n2;
//   Eq. 8:                   |.|^2 summed over the channel pairs of the tile.
// A workgroup owns 16 channel pairs (32 channels, 64-byte row segments for bf16).  Thread (c, r) = (pair, 0 .. 15) is residue
// t = r on the token side, Q points, and (if r < Q) output a = r on the bin side, 16 points; one exchange through LDS in
// between.  The twiddles of a 16-point transform (and of a 16-point Q) are geometric in its index, so they split into
// those of its two radix-4 levels and go into the additions there (fft16_tw); those over b depend on n2 only.
// The pass-band accumulators F stay in registers across the N2 subsequences, so x is read exactly once and nothing but
// N floats per tile is written.
// Bound: fp32 vector arithmetic, about 900 instructions per wavefront and subsequence.  With the twiddles between the sides
// as multiplications of their own, and the accumulation's looked up per subsequence, it was 1160: 8x1024x3584 bf16 49 us
// (40 now), 16x720x4096 72 (57), 4x2048x3584 47 (43), 8x1440x3584 fp32 76 (65), on tokens whose norms vary by region.
//
// What it gave up: an inverse on every second or fourth subsequence, with the energies between interpolated from the band
// limit.  On tokens of even energy, merged tokens through a random projection, it took 42.8 us for 8x1024x3584 bf16
// (this kernel: 39.8), 67.7 for 16x720x4096 (57.2), but 39.1 for 4x2048x3584 (44.4): eight subsequences, of which six were
// interpolated.  On tokens whose norms vary by region it ran in full after all, nearly always: 52 us for 8x1024x3584 against
// 46 for this kernel of then.  Interpolated scores were only known to 3e-6 of their value (the taps' stop band); these
// are fp32 transforms throughout, 3e-8 off (rms).
#include <type_traits>

#include "common.hpp"
#include "spu.hpp"
#include "spu_fftcore.hpp"
#include "spu_tiles.hpp"

namespace luvc {

namespace {

// 5-point DFT
template <bool INV>
__device__ __forceinline__ void dft5(cf& x0, cf& x1, cf& x2, cf& x3, cf& x4)
{
    constexpr float c1 = 0.30901699437494745f, c2 = -0.8090169943749475f, s1 = 0.9510565162951535f, s2 = 0.5877852522924731f;
    const cf t1 = x1 + x4, t2 = x2 + x3, t3 = x1 - x4, t4 = x2 - x3;
    const cf m1{fmaf(c2, t2.x, fmaf(c1, t1.x, x0.x)), fmaf(c2, t2.y, fmaf(c1, t1.y, x0.y))};
    const cf m2{fmaf(c1, t2.x, fmaf(c2, t1.x, x0.x)), fmaf(c1, t2.y, fmaf(c2, t1.y, x0.y))};
    const cf u1{fmaf(s2, t4.x, s1 * t3.x), fmaf(s2, t4.y, s1 * t3.y)};
    const cf u2{fmaf(-s1, t4.x, s2 * t3.x), fmaf(-s1, t4.y, s2 * t3.y)};
    const cf r1 = INV ? cf{-u1.y, u1.x} : cf{u1.y, -u1.x};
    const cf r2 = INV ? cf{-u2.y, u2.x} : cf{u2.y, -u2.x};
    x0 = x0 + t1 + t2;
    x1 = m1 + r1; x4 = m1 - r1;
    x2 = m2 + r2; x3 = m2 - r2;
}

// Q-point DFT in registers, natural order in and out
template <int Q, bool INV> struct dftq;
template <bool INV> struct dftq<16, INV> {
    __device__ static __forceinline__ void run(cf (&v)[16]) { fft16<INV>(v); }
};
template <bool INV> struct dftq<15, INV> {
    // prime-factor map (no twiddles): n = (5 n1 + 3 n2) mod 15, k = (10 k1 + 6 k2) mod 15
    __device__ static __forceinline__ void run(cf (&v)[15])
    {
        cf u[3][5];
#pragma unroll
        for (int n2 = 0; n2 < 5; ++n2) {
            cf a = v[(3 * n2) % 15], b = v[(5 + 3 * n2) % 15], c = v[(10 + 3 * n2) % 15];
            dft3<INV>(a, b, c);
            u[0][n2] = a; u[1][n2] = b; u[2][n2] = c;
        }
#pragma unroll
        for (int k1 = 0; k1 < 3; ++k1) {
            dft5<INV>(u[k1][0], u[k1][1], u[k1][2], u[k1][3], u[k1][4]);
#pragma unroll
            for (int k2 = 0; k2 < 5; ++k2) v[(10 * k1 + 6 * k2) % 15] = u[k1][k2];
        }
    }
};
template <bool INV> struct dftq<9, INV> {
    // 3 x 3: n = 3 n1 + n2, k = k1 + 3 k2, twiddle W_9^{n2 k1}
    __device__ static __forceinline__ void run(cf (&v)[9])
    {
        constexpr float c1 = 0.766044443118978f, s1 = 0.6427876096865393f;      // W_9^1
        constexpr float c2 = 0.17364817766693036f, s2 = 0.984807753012208f;     // W_9^2
        constexpr float c4 = -0.9396926207859084f, s4 = 0.3420201433256687f;    // W_9^4
        cf u[3][3];
#pragma unroll
        for (int n2 = 0; n2 < 3; ++n2) {
            cf a = v[n2], b = v[3 + n2], c = v[6 + n2];
            dft3<INV>(a, b, c);
            u[0][n2] = a; u[1][n2] = b; u[2][n2] = c;
        }
        auto tw = [](cf a, cf w) { return INV ? cmulc(a, w) : cmul(a, w); };
        u[1][1] = tw(u[1][1], cf{c1, -s1}); u[1][2] = tw(u[1][2], cf{c2, -s2});
        u[2][1] = tw(u[2][1], cf{c2, -s2}); u[2][2] = tw(u[2][2], cf{c4, -s4});
#pragma unroll
        for (int k1 = 0; k1 < 3; ++k1) {
            dft3<INV>(u[k1][0], u[k1][1], u[k1][2]);
#pragma unroll
            for (int k2 = 0; k2 < 3; ++k2) v[k1 + 3 * k2] = u[k1][k2];
        }
    }
};

typedef unsigned int u32x2 __attribute__((__vector_size__(8)));

// One channel pair of one token.  Rows are addressed through a buffer resource that spans the whole
// sample; a lane whose pair lies past D is given an offset beyond the resource and reads zeros, so
// the loads need no branch.
template <typename T> struct pair_io;
template <> struct pair_io<bf16_t> {
    using raw_t = uint32_t;
    __device__ static __forceinline__ raw_t load(__amdgpu_buffer_rsrc_t r, uint32_t off, bool second, bool aligned)
    {
        if (aligned) return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
        const uint32_t lo = __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
        const uint32_t hi = second ? (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, off + 2, 0, 0) : 0u;
        return (lo & 0xffffu) | (hi << 16);
    }
    __device__ static __forceinline__ cf widen(raw_t r) { return {__uint_as_float(r << 16), __uint_as_float(r & 0xffff0000u)}; }
};
template <> struct pair_io<float> {
    using raw_t = u32x2;
    __device__ static __forceinline__ raw_t load(__amdgpu_buffer_rsrc_t r, uint32_t off, bool second, bool aligned)
    {
        if (aligned) return __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
        raw_t v;
        v[0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
        v[1] = second ? __builtin_amdgcn_raw_buffer_load_b32(r, off + 4, 0, 0) : 0u;
        return v;
    }
    __device__ static __forceinline__ cf widen(raw_t r) { return {__uint_as_float(r[0]), __uint_as_float(r[1])}; }
};

constexpr int kPairs = 16;                       // channel pairs per workgroup
constexpr int kRowPad = 16 * kPairs + kPairs;    // float2 per exchange row: 16 x 16 pairs + one pad group

// Lane c of a DPP row of 16 gets the sum of e[c] over the 16 lanes, fixed order: halves, then quarters of the list go with
// the halves and quarters of the row, so that 16 sums take 45 instructions (64 one by one, into every lane).
__device__ __forceinline__ float row16_scatter(const float (&e)[16], bool odd, bool upper /* bits 0 and 1 of the lane */)
{
    auto dpp = [](float v, auto ctrl) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, false)); };
    auto banks = [](float lo, float hi, auto mask) { return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(lo), __float_as_int(hi), 0xE4, 0xf, decltype(mask)::value, false)); };
    using mirror = std::integral_constant<int, 0x140>;
    using half_mirror = std::integral_constant<int, 0x141>;
    using swap1 = std::integral_constant<int, 0xB1>;             // quad_perm [1,0,3,2]
    using swap2 = std::integral_constant<int, 0x4E>;             // quad_perm [2,3,0,1]
    float r[8], q[4];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = banks(e[i] + dpp(e[i], mirror{}), e[i + 8] + dpp(e[i + 8], mirror{}), std::integral_constant<int, 0xc>{});
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = banks(r[i] + dpp(r[i], half_mirror{}), r[i + 4] + dpp(r[i + 4], half_mirror{}), std::integral_constant<int, 0xa>{});
    const float a = (odd ? q[1] : q[0]) + dpp(odd ? q[0] : q[1], swap1{}), b = (odd ? q[3] : q[2]) + dpp(odd ? q[2] : q[3], swap1{});
    return (upper ? b : a) + dpp(upper ? a : b, swap2{});
}

}  // namespace

template <typename T, int Q, bool ALIGNED>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((Q == 9 || (Q == 15 && sizeof(T) == 2)) ? 3 : 2)))
spu_fft16q(const T* __restrict__ x, int N, int D, int64_t row_stride, int sigma, int use_hamming,
           float* __restrict__ partial /* [B, n_tiles, N] */, float* __restrict__ gpartial /* [B, n_groups, N] */,
           const TileSync sy, float* __restrict__ scores /* [B, N] */)
{
    using pio = pair_io<T>;
    constexpr int N1 = 16 * Q;
    // the constants of a 16-point transform as fp32 values are short (see spu_conv.hip): with Q = 16 scores came out
    // 4.6e-8 .. 5.1e-8 too small on the mean, 256 to 1024 tokens, white and smooth; with Q = 15 0.3e-8
    constexpr double kLength = Q == 16 ? 1.0 + 4.8e-8 : 1.0;
    extern __shared__ float2 smem[];
    float2* xbuf = smem;                         // [16][kRowPad]  exchange between the two sides
    float2* tw = smem + 16 * kRowPad;            // [N]    (cos, sin)(2 pi i / N)
    float* eperm = reinterpret_cast<float*>(tw + N);        // [N2][16 t][16 j] energies of this tile
    float* gm = eperm + N / Q * 16;              // [sigma + 1]  M[f] / N  (Eq. 5 with the 1/N of Eq. 7)
    __shared__ int is_last;
    const int tid = threadIdx.x, c = tid & 15, r = tid >> 4;
    // neighbouring channel tiles share 128-byte lines of every token row: keep them on one XCD
    const int n_tiles = gridDim.x;
    const unsigned item = xcd_contiguous(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
    const int tile = item % n_tiles, b = item / n_tiles;
    const int N2 = N / N1, n16 = N / 16;

    const int d0 = tile * 32 + 2 * c;
    const bool bins = Q == 16 || r < Q;          // this thread takes part on the bin side
    const bool live = d0 < D, second = d0 + 1 < D;
    const uint32_t es = (uint32_t)sizeof(T);
    const uint32_t row_bytes = (uint32_t)row_stride * es;
    // resource over sample b (N rows); lanes without a channel pair point past its end
    const uint64_t span = (uint64_t)(N - 1) * row_bytes + (uint64_t)D * es;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(x) + (int64_t)b * N * row_stride, 0, (int)(span > 0x7fffffffull ? 0x7fffffffull : span), 0x00020000);
    const uint32_t lane_off = live ? (uint32_t)d0 * es : 0x80000000u;

    typename pio::raw_t raw[Q];
    auto load_sub = [&](int n2) {
#pragma unroll
        for (int j = 0; j < Q; ++j)
            raw[j] = pio::load(rsrc, lane_off + (uint32_t)(N2 * (16 * j + r) + n2) * row_bytes, second, ALIGNED);
    };
    load_sub(N2 - 1);
    // Tables, built while the first loads are in flight.  One octant of the circle is evaluated in fp64
    // and rounded once; the other seven follow by symmetry (8 divides N).
    {
        const int n8 = N >> 3, n4 = N >> 2, nh = N >> 1, n34 = nh + n4;
        for (int i = tid; i <= n8; i += 256) {
            double sd, cd;
            sincospi(2.0 * (double)i / (double)N, &sd, &cd);
            const float cs = (float)cd, sn = (float)sd;
            tw[i] = make_float2(cs, sn);
            tw[n4 - i] = make_float2(sn, cs);
            tw[n4 + i] = make_float2(-sn, cs);
            tw[nh - i] = make_float2(-cs, sn);
            tw[nh + i] = make_float2(-cs, -sn);
            tw[n34 - i] = make_float2(-sn, -cs);
            tw[n34 + i] = make_float2(sn, -cs);
            if (i) tw[N - i] = make_float2(cs, -sn);
        }
        // the window weights on the upper half of the workgroup: for N <= 1024 the octant above keeps the lower one busy
        if (tid >= 128 && tid - 128 <= sigma) {
            const int f = tid - 128;
            double w = 1.0;
            if (use_hamming) w = 0.54 + 0.46 * cospi(2.0 * (double)f / (double)(N - 1));
            gm[f] = (float)(w / (double)N * kLength);
        }
    }
    __syncthreads();
    auto table = [&](int i) { const float2 q = tw[i]; return cf{q.x, q.y}; };
    // h^j = W_N^{j p}, j < 16, as fft16_tw takes them; p < N / Q: none of the places reaches N
    auto powers = [&](int p, cf (&lo)[3], cf (&hi)[4][3]) {
#pragma unroll
        for (int i = 1; i < 4; ++i) lo[i - 1] = table(4 * i * p);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 1; i < 4; ++i) hi[q][i - 1] = table(i * (p + q * n16));
    };

    // ------------------------------------------------------------------ forward (Eq. 4 on the pass band)
    cf F[16];
    {
        // W_N1^{t a}, and W_N^k of this thread's bins: in registers for Q = 16, from the table in every pass where that
        // keeps a third wavefront per SIMD
        constexpr bool kHold = Q == 16;
        cf lo[3], hi[4][3], wk[16];
        const int a = bins ? r : 0;
        powers(N2 * a, lo, hi);
        auto bin_turn = [&](int kb) { return table(a + Q * kb + (kb < 8 ? 0 : N - N1)); };
        if (kHold) {
#pragma unroll
            for (int kb = 0; kb < 16; ++kb) wk[kb] = bin_turn(kb);
        }
        // The next subsequence is in flight while the bin side works on this one.  Asked for before the token side's transform, its
        // Q requests stood in the way of that side's start: 32x1152x1152 bf16 59.5 us (58.5 here), 4x2048x3584 43.8 (42.7),
        // 2x2880x2048 52.4 (51.6), 8x1440x3584 55.7 (55.2), 8x1024x3584 39.7 (39.6); and with fp32 tokens and Q = 15 it took the
        // registers of the third wavefront per SIMD: 8x1440x3584 69.1 (64.5), 16x720x4096 74.0 (68.0).  The other fp32 kernels,
        // whose tokens take twice the time, want them early: late, 32x1152x1152 took 68.0 (66.7), 8x1024x3584 49.0 (47.2).
        constexpr bool kEarly = sizeof(T) == 4 && Q != 15;
        // The last subsequence comes first and starts the sums: its pass is a copy of the loop body without them.
        auto forward = [&](int n2, auto first) {
            cf u[Q];
#pragma unroll
            for (int j = 0; j < Q; ++j) u[j] = pio::widen(raw[j]);
            if (kEarly && n2 > 0) load_sub(n2 - 1);
            dftq<Q, false>::run(u);              // over j -> a
#pragma unroll
            for (int i = 0; i < Q; ++i) xbuf[i * kRowPad + r * kPairs + c] = make_float2(u[i].x, u[i].y);
            if (!kEarly && n2 > 0) load_sub(n2 - 1);
            __syncthreads();
            cf v[16];
            if (bins) {
#pragma unroll
                for (int t = 0; t < 16; ++t) { const float2 q = xbuf[r * kRowPad + t * kPairs + c]; v[t] = {q.x, q.y}; }
            }
            __syncthreads();
            if (bins) {
                fft16_tw<false>(v, lo, hi);      // over t -> b
#pragma unroll
                for (int kb = 0; kb < 16; ++kb) F[kb] = decltype(first)::value ? v[kb] : cmac<false>(v[kb], F[kb], kHold ? wk[kb] : bin_turn(kb));
            }
        };
        forward(N2 - 1, std::true_type{});
        for (int n2 = N2 - 2; n2 >= 0; --n2) forward(n2, std::false_type{});
    }
    const tile_tag_t seen = tiles_look(sy, b, tile, n_tiles);     // no loads follow: nothing waits behind this one
    // ------------------------------------------------------------------ mask (Eq. 5-6) with the 1/N of Eq. 7
#pragma unroll
    for (int kb = 0; kb < 16; ++kb) {
        const int f = kb < 8 ? r + Q * kb : N1 - (r + Q * kb);       // |k|
        const float g = bins && f <= sigma ? gm[f] : 0.f;
        F[kb] = {F[kb].x * g, F[kb].y * g};
    }
    // ------------------------------------------------------------------ inverse (Eq. 7) and energy (Eq. 8)
    const bool odd = (tid & 1) != 0, upper = (tid & 2) != 0;
    auto inverse = [&](int n2, auto first) {
        if (bins) {
            cf v[16];
#pragma unroll
            for (int kb = 0; kb < 16; ++kb) v[kb] = F[kb];
            if constexpr (decltype(first)::value) fft16<true>(v);    // over b -> t
            else {
                // W_N^{-Q b n2}, b >= 8: W_N^{-Q (b - 16) n2}
                const int p = Q * n2;
                const cf w1 = table(4 * p), w2 = table(8 * p);
                const cf lo[3] = {w1, {w2.x, -w2.y}, {w1.x, -w1.y}};
                cf hi[4][3];
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 1; i < 4; ++i) hi[q][i - 1] = table(i * (p + q * n16));
                fft16_tw<true>(v, lo, hi);
            }
#pragma unroll
            for (int t = 0; t < 16; ++t) xbuf[t * kRowPad + r * kPairs + c] = make_float2(v[t].x, v[t].y);
        }
        const int p = n2 + N2 * r;
        cf lo[3], hi[4][3], wa[Q];
        if constexpr (Q == 16) powers(p, lo, hi);
        else {
#pragma unroll
            for (int i = 1; i < Q; ++i) wa[i] = table(i * p);
        }
        __syncthreads();
        cf u[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) { const float2 q = xbuf[r * kRowPad + i * kPairs + c]; u[i] = {q.x, q.y}; }
        if constexpr (Q == 16) fft16_tw<true>(u, lo, hi);            // over a -> j ; u[j] = z'[N2 (16 j + t) + n2]
        else {
#pragma unroll
            for (int i = 1; i < Q; ++i) u[i] = cmul(u[i], wa[i]);
            dftq<Q, true>::run(u);
        }
        float e[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) e[j] = j < Q ? fmaf(u[j < Q ? j : 0].x, u[j < Q ? j : 0].x, u[j < Q ? j : 0].y * u[j < Q ? j : 0].y) : 0.f;
        eperm[(n2 * 16 + r) * 16 + c] = row16_scatter(e, odd, upper);                    // over the 16 pairs
        __syncthreads();
    };
    inverse(0, std::true_type{});
    tiles_claim(sy, b, tile, n_tiles, seen);
    for (int n2 = 1; n2 < N2; ++n2) inverse(n2, std::false_type{});
    float* pout = partial + ((int64_t)b * n_tiles + tile) * N;
    const float inv_n2 = 1.f / (float)N2;
    for (int n = tid; n < N; n += 256) {         // n = N2 (16 j + t) + n2
        const int q = (int)(((float)n + 0.5f) * inv_n2), n2 = n - q * N2;                // exact: n < 4097
        tile_store(pout + n, eperm[(n2 * 16 + (q & 15)) * 16 + (q >> 4)]);
    }
    // ------------------------------------------------------------------ Eq. 8 across the channel tiles
    tiles_to_scores<256>(partial, gpartial, sy, scores, b, tile, n_tiles, N, N, &is_last);
}

static size_t fft_lds_bytes(int N, int Q, int sigma)
{
    return sizeof(float2) * (size_t)(16 * kRowPad + N) + sizeof(float) * (size_t)(N / Q * 16 + sigma + 1);
}

// the residue-side length Q of the 16 x Q transform that serves (N, sigma); 0 if none does
static int fft_pick_q(int N, int sigma)
{
    if (N > 4096) return 0;
    for (int Q : {16, 15, 9}) {
        const int N1 = 16 * Q;
        if (N % N1 == 0 && 2 * sigma + 1 <= N1) return Q;
    }
    return 0;
}

bool spu_fft_supported(int N, int sigma) { return fft_pick_q(N, sigma) != 0; }

// us of one call, from measurements: a workgroup's share of a subsequence, both ways, and the rounds the workgroups take on
// the chip (two per compute unit for Q = 16, three otherwise; a last round that is half empty costs less than a full one).
// 8x1024x3584 bf16: 42, 4x2048x3584: 42, 16x720x4096: 60, 8x1440x3584: 61, 32x1152x2048: 105, fp32 1x576x4096: 18.
double spu_fft_us(int B, int N, int D, int sigma)
{
    const int Q = fft_pick_q(N, sigma);
    const int64_t wgs = (int64_t)B * ((D + 31) / 32), slots = Q == 16 ? 512 : 768;
    const double n2 = N / (16 * Q);
    if (wgs <= slots) return 7.0 + n2 * (wgs <= 256 ? 2.9 : 4.4);
    const double rounds = 0.5 * ((double)((wgs + slots - 1) / slots) + (double)wgs / (double)slots);
    return 5.0 + rounds * n2 * (Q == 16 ? 5.0 : Q == 15 ? 6.2 : 4.35);
}

// As measured on 18 shapes: short samples pay for the start of a workgroup too (19x256x4864: 51, the above 34; 11x240x4480: 28, 20.5;
// 7x512x2432: 22.6, 20.2; from 3 or 4 subsequences on, 0.94 to 1.17 of it but for 4x4096x3584, sigma = 100: 110, 77)
double spu_fft_measured_us(int B, int N, int D, int sigma)
{
    const int Q = fft_pick_q(N, sigma);
    return spu_fft_us(B, N, D, sigma) + (N <= 2 * 16 * Q ? 3.0 * (double)((int64_t)B * ((D + 31) / 32)) / (Q == 16 ? 512.0 : 768.0) : 0.0);
}

luvc_status spu_score_fft(const void* x, int B, int N, int D, int64_t row_stride, luvc_dtype dt, int sigma, int use_hamming,
                          float* partial, float* gpartial, const TileSync& sy, int n_tiles, float* scores, hipStream_t st)
{
    const int Q = fft_pick_q(N, sigma);
    const size_t lds = fft_lds_bytes(N, Q, sigma);
    // channel pairs are fetched with one access when every pair is naturally aligned
    const size_t es = dt == LUVC_F32 ? 4 : 2;
    const bool aligned = (row_stride % 2 == 0) && ((uintptr_t)x % (2 * es) == 0) && (D % 2 == 0);
    if (n_tiles > 65535) { set_error("D=%d exceeds the supported width of the fft path", D); return LUVC_ERR_UNSUPPORTED; }
    const dim3 grid((unsigned)n_tiles, (unsigned)B);
#define LUVC_FFT(TT, QQ, AL) LUVC_LAUNCH("spu_fft16q", (spu_fft16q<TT, QQ, AL>), grid, dim3(256), lds, st, (const TT*)x, N, D, row_stride, sigma, use_hamming, partial, gpartial, sy, scores)
#define LUVC_FFT_A(TT, QQ) do { if (aligned) LUVC_FFT(TT, QQ, true); else LUVC_FFT(TT, QQ, false); } while (0)
#define LUVC_FFT_T(TT) do { if (Q == 16) LUVC_FFT_A(TT, 16); else if (Q == 15) LUVC_FFT_A(TT, 15); else LUVC_FFT_A(TT, 9); } while (0)
    if (dt == LUVC_F32) LUVC_FFT_T(float); else LUVC_FFT_T(bf16_t);
#undef LUVC_FFT_T
#undef LUVC_FFT_A
#undef LUVC_FFT
    return check_launch("spu score (fft)");
}

}  // namespace luvc
