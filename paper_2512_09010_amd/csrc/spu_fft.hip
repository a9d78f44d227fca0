// SPU score (paper Section 3.3, Eq. 4-8): fast path for N = N1 * N2 with N1 = 16 * Q, Q in {16, 15, 9},
// and 2*sigma + 1 <= N1 (N = 1024, 2048, 720, 144 ... of the benchmark workloads).
//
// Two real channels (d, d+1) are packed as one complex signal z = x_d + i x_{d+1}.  The mask of
// Eq. 5 is real and symmetric in k, so the filter is a real linear operator and Re / Im of the
// filtered z are the two filtered channels: no unpacking is ever needed.
//
// Transform decomposition along the token index, n = N2 * n1 + n2 (n1 < N1, n2 < N2):
//   Eq. 4 on the pass band:  F[k] = sum_{n2} W_N^{k n2} Y_{n2}[k mod N1],  |k| <= sigma,
//                            Y_{n2} = N1-point DFT of the stride-N2 subsequence n2;
//   Eq. 6:                   F[k] *= M[|k|] / N;
//   Eq. 7:                   z'[N2 n1 + n2] = N1-point inverse DFT over k1 of F[k] W_N^{-k n2};
//   Eq. 8:                   |z'|^2 summed over the channel pairs of the tile.
// Each N1-point transform is 16 x Q (n1 = Q j + t, k1 = ka + 16 kb): a radix-16 butterfly over j held
// in registers, the twiddle W_N1^{t ka}, one exchange through LDS, and a Q-point transform over t
// (radix-16 again, or 3 x 5 by the prime-factor map, or 3 x 3).  A workgroup owns 16 channel pairs
// (32 channels, 64-byte row segments for bf16); thread (c, t) = (pair, residue): Q of the 16 residue
// threads hold 16 points each for the radix-16 side, all 16 hold Q points each for the other side.
// The pass-band accumulators F stay in registers across the N2 subsequences, so x is read exactly
// once and nothing but N floats per tile is written.
//
// (An inverse on every second or fourth subsequence, with the energies between interpolated from the band limit, needs
// tokens of even energy to stay within fp32 error and otherwise has to run in full after all: on tokens whose norms
// vary by region it did so nearly always, at 52 us for 8 x 1024 x 3584 bf16 against 46 for this kernel.)
#include <type_traits>

#include "common.hpp"
#include "spu.hpp"
#include "spu_fftcore.hpp"
#include "spu_tiles.hpp"

namespace luvc {

namespace {

// 3-point DFT (INV: conjugate twiddles)
template <bool INV>
__device__ __forceinline__ void dft3(cf& a, cf& b, cf& c)
{
    constexpr float s3 = 0.8660254037844386f;
    const cf t = b + c, m{a.x - 0.5f * t.x, a.y - 0.5f * t.y};
    const cf d{(b.x - c.x) * s3, (b.y - c.y) * s3};
    const cf r = INV ? cf{-d.y, d.x} : cf{d.y, -d.x};          // d * (+i) or d * (-i)
    a = a + t; b = m + r; c = m - r;
}

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

// sum over the 16 lanes of a DPP row; every lane of the row ends up with the total, fixed order
__device__ __forceinline__ float row16_sum(float v)
{
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, false));    // quad_perm [1,0,3,2]
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xf, 0xf, false));    // quad_perm [2,3,0,1]
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xf, 0xf, false));   // row_half_mirror
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xf, 0xf, false));   // row_mirror
    return v;
}

}  // namespace

template <typename T, int Q, bool POW2, bool ALIGNED>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((Q == 9 || (Q == 15 && sizeof(T) == 2)) ? 3 : 2)))
spu_fft16q(const T* __restrict__ x, int N, int D, int64_t row_stride, int sigma, int use_hamming,
           float* __restrict__ partial /* [B, n_tiles, N] */, float* __restrict__ gpartial /* [B, n_groups, N] */,
           const TileSync sy, float* __restrict__ scores /* [B, N] */)
{
    using pio = pair_io<T>;
    constexpr int N1 = 16 * Q;
    extern __shared__ float2 smem[];
    float2* xbuf = smem;                         // [16][kRowPad]  exchange between the two passes
    float2* tw = smem + 16 * kRowPad;            // [N]    (cos, sin)(2 pi i / N)
    float2* tw1 = tw + N;                        // [N1]   (cos, sin)(2 pi i / N1)
    float* eperm = reinterpret_cast<float*>(tw1 + N1);      // [N2][Q t][16 j] energies of this tile
    float* gm = eperm + N;                       // [sigma + 1]  M[f] / N  (Eq. 5 with the 1/N of Eq. 7)
    __shared__ int is_last;
    const int tid = threadIdx.x, c = tid & 15, t = tid >> 4;
    // neighbouring channel tiles share 128-byte lines of every token row: keep them on one XCD
    const int n_tiles = gridDim.x;
    const unsigned item = xcd_contiguous(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
    const int tile = item % n_tiles, b = item / n_tiles;
    const int N2 = N / N1;

    const int d0 = tile * 32 + 2 * c;
    const bool rdx = Q == 16 || t < Q;           // this thread takes part in the radix-16 side
    const bool live = d0 < D && rdx, second = d0 + 1 < D;
    const uint32_t es = (uint32_t)sizeof(T);
    const uint32_t row_bytes = (uint32_t)row_stride * es;
    // resource over sample b (N rows); lanes without a channel pair point past its end
    const uint64_t span = (uint64_t)(N - 1) * row_bytes + (uint64_t)D * es;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(x) + (int64_t)b * N * row_stride, 0, (int)(span > 0x7fffffffull ? 0x7fffffffull : span), 0x00020000);
    const uint32_t lane_off = live ? (uint32_t)d0 * es : 0x80000000u;

    // this thread's output bins of every N1-point transform: k1 = t + 16 kb (t doubles as ka)
    int kpos[Q], ph[Q];
    cf F[Q];
#pragma unroll
    for (int kb = 0; kb < Q; ++kb) {
        const int k1 = t + 16 * kb;
        kpos[kb] = 8 * (k1 <= sigma ? k1 : N - N1 + k1);  // k mod N (bins outside the band are masked later), as a byte offset into tw
        ph[kb] = 0;                                        // (k * n2) mod N, likewise
        F[kb] = {0.f, 0.f};
    }
    // W_N^{+-k n2} for bin kb of this thread: a power-of-two N takes the product modulo N directly, any other N
    // keeps a running sum
    auto tw_k = [&](int kb, int n2) {
        int off;
        if (POW2) off = (int)__umul24((unsigned)kpos[kb], (unsigned)n2) & (8 * N - 1);
        else {
            off = ph[kb];
            ph[kb] += kpos[kb];
            if (ph[kb] >= 8 * N) ph[kb] -= 8 * N;
        }
        return *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(tw) + off);
    };

    typename pio::raw_t raw[16];
    auto load_sub = [&](int n2) {
#pragma unroll
        for (int j = 0; j < 16; ++j)
            raw[j] = pio::load(rsrc, lane_off + (uint32_t)(N2 * (Q * j + t) + n2) * row_bytes, second, ALIGNED);
    };
    load_sub(0);
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
            gm[f] = (float)(w / (double)N);
        }
    }
    __syncthreads();
    // W_N1^{t i}, i < 16: the twiddles between the two passes of every N1-point transform, both directions
    constexpr bool kHoist = Q == 16;
    cf w1[16];
    if (kHoist) {
        int e1 = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float2 w = tw[e1 * N2];
            w1[i] = {w.x, w.y};
            e1 += t;
            if (e1 >= N1) e1 -= N1;
        }
    }
    else {
        if (tid < N1) tw1[tid] = tw[tid * N2];
        __syncthreads();
    }
    // v[i] times W_N1^{-+ t i} to its place in the exchange buffer.  Without the register copy the twiddles come out of
    // the N1 table eight at a time: the compiler has to assume that a table read and a write into the buffer meet, so
    // read one by one each of them would wait for its own trip to LDS (8x1440x3584 fp32: 83 us, 75 in eights).  With bf16
    // tokens the three wavefronts per SIMD hide that, and have no registers for eight more (16x720x4096: 72 and 78 us).
    auto to_exchange = [&](auto& v, auto count, auto inv) {
        constexpr int n = decltype(count)::value, G = kHoist ? n : sizeof(T) == 4 ? 8 : 1;
        int o1 = 0;                                              // t i mod N1
#pragma unroll
        for (int i0 = 0; i0 < n; i0 += G) {
            cf w[G];
#pragma unroll
            for (int i = 0; i < G && i0 + i < n; ++i) {
                if (kHoist) w[i] = w1[i0 + i];
                else {
                    const float2 q = tw1[o1];
                    w[i] = {q.x, q.y};
                    o1 += t;
                    if (o1 >= N1) o1 -= N1;
                }
            }
            if (!kHoist && G > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < G && i0 + i < n; ++i) {
                const cf r = decltype(inv)::value ? cmul(v[i0 + i], w[i]) : cmulc(v[i0 + i], w[i]);
                xbuf[(i0 + i) * kRowPad + t * kPairs + c] = make_float2(r.x, r.y);
            }
        }
    };

    // ------------------------------------------------------------------ forward (Eq. 4 on the pass band)
    // The subsequence n2 = 0 carries the twiddle W_N^0 = 1: its pass is a copy of the loop body without the
    // pass-band multiplications (the same holds for the inverse below).
    auto forward = [&](int n2, auto first) {
        cf v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = pio::widen(raw[j]);
        if (n2 + 1 < N2) load_sub(n2 + 1);       // next subsequence in flight while this one is transformed
        if (rdx) {
            fft16<false>(v);                     // over j -> ka
            to_exchange(v, std::integral_constant<int, 16>{}, std::false_type{});      // * W_N1^{t ka}
        }
        __syncthreads();
        cf u[Q];
#pragma unroll
        for (int s = 0; s < Q; ++s) { const float2 q = xbuf[t * kRowPad + s * kPairs + c]; u[s] = {q.x, q.y}; }
        __syncthreads();
        dftq<Q, false>::run(u);                  // over the residue -> kb ; u[kb] = Y[t + 16 kb]
#pragma unroll
        for (int kb = 0; kb < Q; ++kb) {
            if constexpr (decltype(first)::value) {
                F[kb] = u[kb];
                ph[kb] = kpos[kb];               // (k * 1) mod N for the next subsequence
            }
            else {
                const float2 w = tw_k(kb, n2);
                F[kb] = F[kb] + cmulc(u[kb], cf{w.x, w.y});    // * W_N^{k n2}
            }
        }
    };
    forward(0, std::true_type{});
    for (int n2 = 1; n2 < N2; ++n2) forward(n2, std::false_type{});
    const tile_tag_t seen = tiles_look<4>(sy, b, tile, n_tiles);     // no loads follow: nothing waits behind this one
    // ------------------------------------------------------------------ mask (Eq. 5-6) with the 1/N of Eq. 7
#pragma unroll
    for (int kb = 0; kb < Q; ++kb) {
        const int k1 = t + 16 * kb;
        const bool lo = k1 <= sigma, hi = k1 >= N1 - sigma;
        const float g = (lo || hi) ? gm[lo ? k1 : N1 - k1] : 0.f;
        F[kb] = {F[kb].x * g, F[kb].y * g};
        ph[kb] = 0;
    }
    // ------------------------------------------------------------------ inverse (Eq. 7) and energy (Eq. 8)
    auto inverse = [&](int n2, auto first) {
        cf u[Q];
#pragma unroll
        for (int kb = 0; kb < Q; ++kb) {
            if constexpr (decltype(first)::value) {
                u[kb] = F[kb];
                ph[kb] = kpos[kb];
            }
            else {
                const float2 w = tw_k(kb, n2);
                u[kb] = cmul(F[kb], cf{w.x, w.y});   // F[k] W_N^{-k n2}
            }
        }
        dftq<Q, true>::run(u);                   // over kb -> residue s
        to_exchange(u, std::integral_constant<int, Q>{}, std::true_type{});            // * W_N1^{-s ka}
        __syncthreads();
        if (rdx) {
            cf v[16];
#pragma unroll
            for (int ka = 0; ka < 16; ++ka) { const float2 q = xbuf[t * kRowPad + ka * kPairs + c]; v[ka] = {q.x, q.y}; }
            fft16<true>(v);                      // over ka -> j ; v[j] = z'[N2 (Q j + t) + n2]
            float e[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) e[j] = row16_sum(fmaf(v[j].x, v[j].x, v[j].y * v[j].y));   // over the 16 pairs
            if (c == 0) {
                float4* dst = reinterpret_cast<float4*>(eperm + (n2 * Q + t) * 16);
#pragma unroll
                for (int q = 0; q < 4; ++q) dst[q] = make_float4(e[4 * q], e[4 * q + 1], e[4 * q + 2], e[4 * q + 3]);
            }
        }
        __syncthreads();
    };
    inverse(0, std::true_type{});
    tiles_claim<4>(sy, b, tile, n_tiles, seen);
    for (int n2 = 1; n2 < N2; ++n2) inverse(n2, std::false_type{});
    float* pout = partial + ((int64_t)b * n_tiles + tile) * N;
    for (int n = tid; n < N; n += 256) {         // n = N2 (Q j + t') + n2
        const int n2 = POW2 ? (n & (N2 - 1)) : n % N2;
        const int q = (n - n2) / N2;
        const int tq = Q == 16 ? (q & 15) : q % Q, j = Q == 16 ? (q >> 4) : q / Q;
        tile_store(pout + n, eperm[(n2 * Q + tq) * 16 + j]);
    }
    // ------------------------------------------------------------------ Eq. 8 across the channel tiles
    tiles_to_scores<256, 4>(partial, gpartial, sy, scores, b, tile, n_tiles, N, N, &is_last);
}

static size_t fft_lds_bytes(int N, int Q, int sigma)
{
    return sizeof(float2) * (size_t)(16 * kRowPad + N + 16 * Q) + sizeof(float) * (size_t)(N + sigma + 1);
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
// the chip (two per compute unit for Q = 16, three otherwise).  8x1024x3584 bf16: 46, 2x4096x1792: 74, 16x720x4096: 69.
double spu_fft_us(int B, int N, int D, int sigma)
{
    const int Q = fft_pick_q(N, sigma);
    const int64_t wgs = (int64_t)B * ((D + 31) / 32), slots = Q == 16 ? 512 : 768;
    return 5.0 + (double)((wgs + slots - 1) / slots) * (N / (16 * Q)) * (wgs <= slots ? 4.4 : Q == 16 ? 5.1 : 7.1);
}

luvc_status spu_score_fft(const void* x, int B, int N, int D, int64_t row_stride, luvc_dtype dt, int sigma, int use_hamming,
                          float* partial, float* gpartial, const TileSync& sy, int n_tiles, float* scores, hipStream_t st)
{
    const int Q = fft_pick_q(N, sigma);
    const size_t lds = fft_lds_bytes(N, Q, sigma);
    const bool pow2 = (N & (N - 1)) == 0;
    // channel pairs are fetched with one access when every pair is naturally aligned
    const size_t es = dt == LUVC_F32 ? 4 : 2;
    const bool aligned = (row_stride % 2 == 0) && ((uintptr_t)x % (2 * es) == 0) && (D % 2 == 0);
    if (n_tiles > 65535) { set_error("D=%d exceeds the supported width of the fft path", D); return LUVC_ERR_UNSUPPORTED; }
    const dim3 grid((unsigned)n_tiles, (unsigned)B);
#define LUVC_FFT(TT, QQ, P2, AL) LUVC_LAUNCH("spu_fft16q", (spu_fft16q<TT, QQ, P2, AL>), grid, dim3(256), lds, st, (const TT*)x, N, D, row_stride, sigma, use_hamming, partial, gpartial, sy, scores)
#define LUVC_FFT_A(TT, QQ, P2) do { if (aligned) LUVC_FFT(TT, QQ, P2, true); else LUVC_FFT(TT, QQ, P2, false); } while (0)
#define LUVC_FFT_T(TT) do { if (Q == 16) { if (pow2) LUVC_FFT_A(TT, 16, true); else LUVC_FFT_A(TT, 16, false); } \
                            else if (Q == 15) LUVC_FFT_A(TT, 15, false); else LUVC_FFT_A(TT, 9, false); } while (0)
    if (dt == LUVC_F32) LUVC_FFT_T(float); else LUVC_FFT_T(bf16_t);
#undef LUVC_FFT_T
#undef LUVC_FFT_A
#undef LUVC_FFT
    return check_launch("spu score (fft)");
}

}  // namespace luvc
