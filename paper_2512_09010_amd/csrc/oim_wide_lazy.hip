// OIM (paper Section 3.2, Algorithm 1) with candidates beyond the adjacent destinations, for schedules that take few
// tokens out of a line per pass (the paper's appendix runs a merge number of 2): one launch per pass, and the
// tokens are moved once, at the end of the call.
//
// Between the passes a grid is not a tensor of tokens but a tensor of ROW IDS: id < n0 names a token of the call's
// input, id >= n0 a row of the "overlay", the buffer that receives every token a merge produces.  A pass reads the
// ids of its grid, fetches the tokens behind them, and writes the ids of the next grid (compacted: survivors move
// up on their line), the sizes, the anchors and the pass map; only the merged destinations - at most m per line -
// are written as tokens, into overlay rows of their own.  After the last pass oim_lazy_finish copies the rows behind
// the final ids to the output.  A pass that rewrote its whole grid would move 97 % of the tokens unchanged when two
// of 64 leave a line.
//
// oim_wide_line, one workgroup per line (lines of at most 128 tokens).  The decisions are the fp64 decisions of the
// method, reached in two steps:
//   1. SCREENING.  The source x destination dot products of the line on the matrix cores in the storage precision
//      (v_mfma_f32_16x16x32_bf16, or four v_mfma_f32_16x16x4_f32 for fp32 tokens): a 32 x 32 tile at a time, eight
//      wavefronts split the channels, every token byte is fetched once per tile.  The squared norms are summed in fp32
//      on the way (in fp64, they took as long as everything else of the screening).  A screened cosine is taken to be
//      within eps = (5 D / 32 + 53) 2^-23 of the fp64 cosine.  In units of 2^-23, for a wavefront that contracts c channels:
//      the products are at most c accumulation steps of one unit each, relative to the sum of the magnitudes of the products,
//      which is at most the product of the norms (the products of bf16 values are exact in fp32) - tests/test_gpu_oim_wide.py
//      pins the contraction at that rate against fp64 on adversarial rows - and 3.5 for adding the eight parts.  A squared
//      norm is c / 4 roundings of half a unit in a lane, which has a quarter of the channels, and 9 behind it, halved by the
//      root, twice: c / 8 + 4.5.  Two roots, two reciprocals and the two products of a cosine are 3.  That is 9 c / 8 + 11
//      together, and with c <= D / 8 + 28 at most 9 D / 64 + 42.5 (tests/test_abi.py holds the longest run of channels against eps
//      for every width).  The roundings count along the longest chain of additions, an eighth of the channels, not over all
//      of them.  With (D + 24) 2^-22, ten times as much at 1280 channels, more sources and destinations had to be repeated in fp64,
//      a memory trip behind the screening (8 x 64 x 64 x 1280 bf16, six passes of merge number 2: 185.7 us, 173.0 with this bound).
//      Sums of squares beyond 2^100 end the screening of their line: everything is repeated then.  Small values need no such
//      care: what flushed products lose is below 2^-116, far below a norm of 1e-12, which is where the method clamps.
//   2. EXACT.  A source may be among the m best of the line only if fewer than m screened best cosines exceed its own by
//      more than 2 eps; for each such contender, the destinations within 2 eps of its best screened cosine may be its
//      best destination, no other can.  Their dot products are repeated in fp64 (a wavefront per contender, two
//      destinations at a time), and the rules of the method - higher cosine wins, ties go to the lower position - are
//      applied to the fp64 values.  Nothing is repeated for a contender with one candidate where there are no more
//      than m contenders.
//   3. Layout of the next grid from two 64-bit masks, sources gone and destinations taking sources in, which every
//      wavefront works out for itself; ids / sizes / anchors / maps of the next grid.
//   4. Size-weighted mean of every destination that takes sources in: a wavefront per destination, or, where a line has one or two
//      rows to merge, the wavefronts share the channels of each.
// All lines of a grid start together, so what follows the screening is serial time of the launch: no lists or
// flags are handed through LDS where a ballot does, and each step after the screening is one barrier.
// Bound: the screening, by the rate at which the tokens arrive (8 x 64 x 64 x 1280 bf16: 84 MB a pass), then latency.
// Of a pass of that grid (20.4 us) the tokens of the last lines are there after 13.9 us, their screened cosines 1.5 us later, and the fp64
// repeats (0 .. 4), the layout (1) and the merged rows (1.5) follow; six passes of merge number 2 and the last copy take 144 us.  What the
// parts give, us with and without: contenders from the m-th highest cosine instead of a comparison with every source 144.1, 149.5, and
// 8 x 48 x 48 x 768, six passes 84.7, 89.0; lines of up to 64 tokens as one tile, with the registers for a fifth step in flight 144.1, 177.7;
// lines of up to 32 with half the loads of such a tile 12 x 32 x 32 x 1024, six passes 75.9, 83.5, 1 x 16 x 16 x 768, six 44.6, 50.0,
// 8 x 24 x 24 x 1024 fp32, radius 2, four 54.6, 61.0.  fp32 on lines of 64 and 100 tokens: 4 x 64 x 64 x 1024, six passes 138.1,
// 2 x 100 x 100 x 1024, two 107.8.
#include <type_traits>

#include "common.hpp"
#include "oim.hpp"
#include "oim_lazy.hpp"
#include "oim_sum64.hpp"
#include "oim_wide_tok.hpp"

namespace luvc {

namespace {

// floats between the rows (a destination each) of the screened matrix: whole tiles of sources, and 4 mod 32
__host__ __device__ inline int lazy_row_stride(int n_src) { return 32 * ((n_src + 31) / 32) + 4; }

}  // namespace

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_lz __attribute__((ext_vector_type(2)));
typedef float f32x4_lz __attribute__((ext_vector_type(4)));

// What a lane feeds to the matrix cores per step of the screening contraction: 16 bytes of a token.  Lane l belongs
// to row l % 16 of a 16 x 16 product (a source for the A side, a destination for the B side) and to quarter l / 16 of the
// step's channels: 64 bytes of 16 rows to a load.
template <typename T> struct screen;
template <> struct screen<bf16_t> {
    static constexpr int KS = 32, KL = 8;      // channels per step, per lane
    __device__ static __forceinline__ f32x4_lz mac(f32x4_lz acc, const u32x4& a, const u32x4& c)
    {
        bf16x8_t va, vc;
        __builtin_memcpy(&va, &a, 16);
        __builtin_memcpy(&vc, &c, 16);
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, vc, acc, 0, 0, 0);
    }
    __device__ static __forceinline__ float sq(const u32x4& a, float acc)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            bf16x2_lz w;
            const uint32_t bits = a[i];
            __builtin_memcpy(&w, &bits, 4);
            acc = __builtin_amdgcn_fdot2_f32_bf16(w, w, acc, false);
        }
        return acc;
    }
    __device__ static __forceinline__ double dot(const u32x4& a, const u32x4& c, double acc)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc = fma((double)__uint_as_float(a[i] << 16), (double)__uint_as_float(c[i] << 16), acc);
            acc = fma((double)__uint_as_float(a[i] & 0xffff0000u), (double)__uint_as_float(c[i] & 0xffff0000u), acc);
        }
        return acc;
    }
};
template <> struct screen<float> {
    static constexpr int KS = 16, KL = 4;
    // instruction e contracts channels {e, 4 + e, 8 + e, 12 + e} of the step: the same grouping on both sides
    __device__ static __forceinline__ f32x4_lz mac(f32x4_lz acc, const u32x4& a, const u32x4& c)
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[e]), __uint_as_float(c[e]), acc, 0, 0, 0);
        return acc;
    }
    __device__ static __forceinline__ float sq(const u32x4& a, float acc)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc = fmaf(__uint_as_float(a[i]), __uint_as_float(a[i]), acc);
        return acc;
    }
    __device__ static __forceinline__ double dot(const u32x4& a, const u32x4& c, double acc)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc = fma((double)__uint_as_float(a[i]), (double)__uint_as_float(c[i]), acc);
        return acc;
    }
};

constexpr int kScreenWaves = 8;                  // wavefronts that split the channels of a tile

// A wavefront's run of steps of KS channels, and the channels behind the last whole step, which go to the last wavefront: its run is never
// the longest, so no wavefront contracts more than D / 8 + 28 channels.
struct ScreenRun { int step0, steps, rest; };
template <int KS> __host__ __device__ inline ScreenRun screen_run(int D, int wave)
{
    const unsigned all = (unsigned)D / KS, upto = wave * all + kScreenWaves - 1, step0 = upto / kScreenWaves;
    return {(int)step0, (int)((upto + all) / kScreenWaves - step0), wave == kScreenWaves - 1 ? (int)(D - all * KS) : 0};
}
// what a screened cosine may be off by
__host__ __device__ inline float screen_eps(int D) { return (0.15625f * (float)D + 53.f) * 1.1920929e-7f; }

// 16 bytes of a token at channel d, zeros past its end or for a token that is not there (rows are multiples of 16 bytes)
template <typename T>
__device__ __forceinline__ u32x4 piece(const T* tok, int D, int d, bool present)
{
    u32x4 v = {0u, 0u, 0u, 0u};
    if (present && d < D) v = *reinterpret_cast<const u32x4*>(tok + d);
    return v;
}

// fp64 cosines of a with c1 and c2 by one wavefront, all fetches in flight together
template <typename T>
__device__ __forceinline__ void cos64_wave2(const T* a, const T* c1, const T* c2, int D, int lane, double& s1, double& s2)
{
    constexpr int V = 16 / (int)sizeof(T);
    double v[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};            // aa, c1 c1, c2 c2, a c1, a c2
    const __amdgpu_buffer_rsrc_t ba = lz_row(a, D, true), b1 = lz_row(c1, D, true), b2 = lz_row(c2, D, true);
    for (int d0 = 0; d0 < D; d0 += 64 * V * 3) {
        u32x4 ra[3], r1[3], r2[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const int off = (d0 + (u * 64 + lane) * V) * (int)sizeof(T);
            ra[u] = lz_load(ba, off);
            r1[u] = lz_load(b1, off);
            r2[u] = lz_load(b2, off);
        }
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            v[0] = screen<T>::dot(ra[u], ra[u], v[0]);
            v[1] = screen<T>::dot(r1[u], r1[u], v[1]);
            v[2] = screen<T>::dot(r2[u], r2[u], v[2]);
            v[3] = screen<T>::dot(ra[u], r1[u], v[3]);
            v[4] = screen<T>::dot(ra[u], r2[u], v[4]);
        }
    }
    wave_total64x8(v, lane);
    auto norm = [](double n2) { const double n = sqrt(n2); return n < 1e-12 ? 1e-12 : n; };
    const double na = norm(v[0]);
    s1 = v[3] / (na * norm(v[1]));
    s2 = v[4] / (na * norm(v[2]));
}

// sum over the four quarters of the wavefront, in every lane
__device__ __forceinline__ float quarters_total(float v)
{
    auto swapped = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(swapped[0]) + __uint_as_float(swapped[1]);
    swapped = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(swapped[0]) + __uint_as_float(swapped[1]);
}

// largest value over the wavefront, in every lane
__device__ __forceinline__ float wave_max32(float v)
{
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, true)));    // lane ^ 1
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xf, 0xf, true)));    // lane ^ 2
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xf, 0xf, true)));   // row_half_mirror
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xf, 0xf, true)));   // row_mirror
    auto swapped = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(swapped[0]), __uint_as_float(swapped[1]));
    swapped = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(swapped[0]), __uint_as_float(swapped[1]));
}

// largest value over groups of eight lanes, in every lane
__device__ __forceinline__ float oct_max(float v)
{
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, true)));    // lane ^ 1
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xf, 0xf, true)));    // lane ^ 2
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xf, 0xf, true)));   // lane ^ 7
    return v;
}

__device__ __forceinline__ double lane_f64(double v, int i)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), i), __builtin_amdgcn_readlane(__double2loint(v), i));
}

}  // namespace

// the screening tile of one wavefront over all channels (a test hook: tests pin the contraction's error against fp64).
// a, c: [32, D] rows; out[i * 32 + j] = <a_i, c_j>.
template <typename T>
__global__ void __launch_bounds__(64)
selftest_screen_tile(const T* __restrict__ a, const T* __restrict__ c, int D, float* __restrict__ out)
{
    using sc = screen<T>;
    const int lane = threadIdx.x, r = lane & 15, kq = lane >> 4;
    f32x4_lz acc[2][2];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q >> 1][q & 1] = f32x4_lz{0.f, 0.f, 0.f, 0.f};
    for (int d = 0; d < D; d += sc::KS)         // the same trip count in every lane: the matrix instructions want the whole wavefront
#pragma unroll
        for (int q = 0; q < 4; ++q)
            acc[q >> 1][q & 1] = sc::mac(acc[q >> 1][q & 1], piece(a + (int64_t)(16 * (q >> 1) + r) * D, D, d + kq * sc::KL, true),
                                         piece(c + (int64_t)(16 * (q & 1) + r) * D, D, d + kq * sc::KL, true));
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) out[(16 * (q >> 1) + 4 * kq + v) * 32 + 16 * (q & 1) + r] = acc[q >> 1][q & 1][v];
}

template <typename T, int TILE /* 1, 2: lines of up to 32, 64 tokens, which are one tile; 0: any */, int LOADS /* steps in flight */>
__global__ void __launch_bounds__(1024)
oim_wide_line(const T* __restrict__ x, T* ov, const T* __restrict__ xk /* metric [.., Dk] the decisions are taken on, or null: x */,
              T* ovk /* its overlay */, int Dk, const int32_t* __restrict__ idx_in /* null: identity */,
              const int32_t* __restrict__ sizes_in /* null: ones */, const int32_t* __restrict__ kept_in /* null: identity */,
              LazyGeom g, int32_t* __restrict__ idx_out, int32_t* __restrict__ sizes_out, int32_t* __restrict__ kept_out /* or null */,
              int32_t* __restrict__ pass_map /* or null */)
{
    using sc = screen<T>;
    constexpr bool ONE = TILE > 0;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int len = g.axis ? g.w : g.h, nlines = g.axis ? g.h : g.w;
    const int n_src = (len + 1) / 2, n_dst = len / 2;
    const int Wo = g.axis ? g.w - g.m : g.w, Ho = g.axis ? g.h : g.h - g.m;
    double* escore = reinterpret_cast<double*>(smem_raw);              // [64] fp64 cosine of a contender with its best destination
    // [kScreenWaves][32 destinations][8] a tile, the part of each wavefront: pieces of four sources, in an order that depends on the
    // destination, so that 16-byte accesses of eight destinations fall into different banks
    float4* P = reinterpret_cast<float4*>(escore + 64);
    float* S = reinterpret_cast<float*>(P + kScreenWaves * 256);       // [n_dst][sd] screened dot products
    const int sd = lazy_row_stride(n_src);
    float* pn = S + n_dst * sd;                          // [kScreenWaves][len] squared norms, the part of each wavefront
    float* inv32 = pn + kScreenWaves * len;              // [len] 1 / norm
    float* b32 = inv32 + len;                            // [64] best screened cosine of a source
    int* rid = reinterpret_cast<int*>(b32 + 64);         // [len] row id of the token at position p
    int* sz = rid + len;                                 // [len] its size
    int* kept = sz + len;                                // [len] its anchor
    int* ebest = kept + len;                             // [64] best destination of a contender
    int* wild = ebest + 64;                              // [1] a norm that fp32 does not hold

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), NW = blockDim.x >> 6;
    const unsigned item = xcd_contiguous(blockIdx.x, gridDim.x);       // lines of one image meet in one L2
    const int64_t b = item / nlines;
    const int line = item % nlines;
    const int64_t img = b * g.h * g.w, img_out = b * Ho * Wo;
    auto in_flat = [&](int p) -> int { return g.axis ? line * g.w + p : p * g.w + line; };
    auto out_flat = [&](int q) -> int { return g.axis ? line * Wo + q : q * Wo + line; };
    // the tensor the decisions are taken on
    const T* dx = xk ? xk : x;
    const T* dov = xk ? ovk : ov;
    const int dD = xk ? Dk : g.D;
    float tau = 2.f * screen_eps(dD);

    // All asked for before any is waited for: six passes of 1 x 16 x 16 x 768 48.0 -> 44.8 us, of 8 x 64 x 64 x 1280 148.1 -> 145.8.
    if (tid < len) {
        const int f = in_flat(tid);
        int id = f, size = 1, anchor = f;
        if (idx_in) id = idx_in[img + f];
        if (sizes_in) size = sizes_in[img + f];
        if (kept_in) anchor = kept_in[img + f];
        rid[tid] = id;
        sz[tid] = size;
        kept[tid] = anchor;
    }
    if (tid == 0) *wild = 0;
    __syncthreads();

    // Lines that ask for their tokens come before those that decide, so that the memory path has work.  On keys, a tenth of the bytes,
    // the decisions are what lasts.  Six passes of 8 x 64 x 64 x 1280 bf16 145.8 -> 144.8 us, 12 x 32 x 32 x 1024 78.6 -> 77.1, two of 4 x 100 x
    // 100 x 1024 95.6 -> 94.7; on keys of 128 it would be 130.6 -> 132.0.  (Raised ahead
    // of the ids it gave 145.5 and cost the same.)
    if (!xk) __builtin_amdgcn_s_setprio(2);
    // ------------------------------------------------------------------ 1. screening: dot products and squared norms
    // Result layout of the 16 x 16 instructions: lane l, register v holds row 4 (l / 16) + v, column l % 16.
    {
        constexpr int SUB = TILE == 1 ? 1 : 2;                                // 16 x 16 products along each side of a tile
        // Steps in flight are a ring, of which one is asked for when another has been used, or, on bf16 lines of one tile of 64, blocks: all
        // used, then the next asked for.  A fifth step fits the registers in blocks only (as a ring 48 spill, 8 x 64 x 64 x 1280, six
        // passes 144.9 -> 166.5 us).  In blocks fp32 is slower, 4 x 64 x 64 x 1024 138.1 -> 142.4, 2 x 100 x 100 x 1024 107.8 -> 116.2; bf16 on
        // longer lines is not.
        constexpr bool BLOCKS = TILE == 2 && sizeof(T) == 2;
        const int tiles_s = ONE ? 1 : (n_src + 31) / 32, tiles_d = ONE ? n_dst > 0 : (n_dst + 31) / 32, tiles = tiles_s * tiles_d;
        const int r = lane & 15, kq = lane >> 4;
        const bool screens = wave < kScreenWaves;
        // A wavefront owns a run of steps of KS channels, a lane its quarter of each; the trip count is the same in every lane (the
        // matrix instructions want the whole wavefront).  Rows that are not there, and steps beyond the last, are read from where some
        // are, without a branch: the compiler waits for everything in flight at a join.  Channels that do not fill a step are the last
        // wavefront's, at the end (it has the shortest run, see screen_run()).
        // LOADS steps stay in flight, across the tiles of a long line too, asked for row by row: the two halves of a cache line one
        // after the other.  Reads of 8 x 64 x 64 x 1280 bf16 in this order, nothing done with them, 12.8 us from the shared cache
        // and 15.5 from memory; 32 bytes of 32 rows to a load and the halves of a line with different wavefronts 15.4 and 21.2; step
        // by step 13.7 and 18.7; in the order of memory 12.3 and 14.4.
        const ScreenRun run = screen_run<sc::KS>(dD, wave);
        const int first = run.step0, steps = run.steps, rest = run.rest;
        const T* tok[2 * SUB];                                                // sources r, 16 + r and destinations r, 16 + r of the tile
        u32x4 raw[LOADS][2 * SUB];
        auto fetch = [&](int u, int i, int step) { raw[u][i] = *reinterpret_cast<const u32x4*>(tok[i] + sc::KS * step); };
        auto begin_tile = [&](int t) {
            const int js = (ONE ? 0 : t / tiles_d * 32) + r, jd = (ONE ? 0 : t % tiles_d * 32) + r;
#pragma unroll
            for (int i = 0; i < SUB; ++i) {
                const int at = first * sc::KS + kq * sc::KL;
                tok[i] = row_of<T>(dx, dov, b, rid[js + 16 * i < n_src ? 2 * (js + 16 * i) : 0], g, dD) + at;
                tok[SUB + i] = row_of<T>(dx, dov, b, rid[jd + 16 * i < n_dst ? 2 * (jd + 16 * i) + 1 : 0], g, dD) + at;
            }
            auto fetch_steps = [&](auto n) {
#pragma unroll
                for (int i = 0; i < 2 * SUB; ++i)
#pragma unroll
                    for (int u = 0; u < decltype(n)::value; ++u) fetch(u, i, u);
            };
            if (steps >= LOADS) fetch_steps(std::integral_constant<int, LOADS>{});
            else if (!ONE) {                             // (few registers are left beside the next tile's)
#pragma unroll
                for (int u = 0; u < LOADS - 1; ++u)
                    if (u < steps) {
#pragma unroll
                        for (int i = 0; i < 2 * SUB; ++i) fetch(u, i, u);
                    }
            }
            else if (steps == 5) fetch_steps(std::integral_constant<int, LOADS < 5 ? 0 : 5>{});
            else if (steps == 4) fetch_steps(std::integral_constant<int, LOADS < 4 ? 0 : 4>{});
            else if (steps == 3) fetch_steps(std::integral_constant<int, 3>{});
            else if (steps == 2) fetch_steps(std::integral_constant<int, 2>{});
            else if (steps == 1) fetch_steps(std::integral_constant<int, 1>{});
        };
        if (screens && tiles > 0) begin_tile(0);
        for (int t = 0; t < tiles; ++t) {
            const int ts = ONE ? 0 : t / tiles_d, td = ONE ? 0 : t % tiles_d;
            if (screens) {
                f32x4_lz acc[SUB][SUB];
                float n2[2 * SUB];
#pragma unroll
                for (int i = 0; i < 2 * SUB; ++i) n2[i] = 0.f;
#pragma unroll
                for (int q = 0; q < SUB * SUB; ++q) acc[q / SUB][q % SUB] = f32x4_lz{0.f, 0.f, 0.f, 0.f};
                auto use = [&](const u32x4 (&v)[2 * SUB]) {
#pragma unroll
                    for (int i = 0; i < 2 * SUB; ++i) n2[i] = sc::sq(v[i], n2[i]);
#pragma unroll
                    for (int q = 0; q < SUB * SUB; ++q) acc[q / SUB][q % SUB] = sc::mac(acc[q / SUB][q % SUB], v[q / SUB], v[SUB + q % SUB]);
                };
                int left = steps;
                for (; left > LOADS; left -= LOADS) {
#pragma unroll
                    for (int u = 0; u < LOADS; ++u) {
                        use(raw[u]);
                        if (BLOCKS) continue;
                        const int step = min(u + LOADS, left - 1);
#pragma unroll
                        for (int i = 0; i < 2 * SUB; ++i) fetch(u, i, step);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < 2 * SUB; ++i) tok[i] += sc::KS * LOADS;
                    if (!BLOCKS) continue;
#pragma unroll
                    for (int i = 0; i < 2 * SUB; ++i)
#pragma unroll
                        for (int u = 0; u < LOADS; ++u) fetch(u, i, min(u, left - LOADS - 1));
                }
#pragma unroll
                for (int u = 0; u < LOADS; ++u)
                    if (u < left) use(raw[u]);
                if (rest) {
                    const bool there = kq * sc::KL < rest;
                    u32x4 v[2 * SUB];
#pragma unroll
                    for (int i = 0; i < 2 * SUB; ++i) {
                        v[i] = u32x4{0u, 0u, 0u, 0u};
                        if (there) v[i] = *reinterpret_cast<const u32x4*>(tok[i] + sc::KS * left);
                    }
                    use(v);
                }
                if (!ONE && t + 1 < tiles) begin_tile(t + 1);
#pragma unroll
                for (int q = 0; q < SUB * SUB; ++q) {
                    const int j = 16 * (q % SUB) + r, piece = 4 * (q / SUB) + kq;
                    const f32x4_lz& y = acc[q / SUB][q % SUB];
                    P[wave * 256 + j * 8 + (piece ^ (j & 7))] = make_float4(y[0], y[1], y[2], y[3]);
                }
#pragma unroll
                for (int i = 0; i < 2 * SUB; ++i) n2[i] = quarters_total(n2[i]);
                const int js = ts * 32 + r, jd = td * 32 + r;
                if (kq == 0) {
#pragma unroll
                    for (int i = 0; i < SUB; ++i) {
                        if (td == 0 && js + 16 * i < n_src) pn[wave * len + 2 * (js + 16 * i)] = n2[i];
                        if (ts == 0 && jd + 16 * i < n_dst) pn[wave * len + 2 * (jd + 16 * i) + 1] = n2[SUB + i];
                    }
                }
            }
            __syncthreads();
            // half of the wavefronts add up the products, the other half the squared norms
            if (tid < 256) {
                const int j = tid >> 3, col = td * 32 + j, row = ts * 32 + 4 * ((tid & 7) ^ (j & 7));
                float4 sum = P[tid];
#pragma unroll
                for (int w = 1; w < kScreenWaves; ++w) {
                    const float4 p = P[w * 256 + tid];
                    sum.x += p.x; sum.y += p.y; sum.z += p.z; sum.w += p.w;
                }
                if (col < n_dst) *reinterpret_cast<float4*>(S + col * sd + row) = sum;
            }
            if (t + 1 < tiles) __syncthreads();
        }
    }
    const int p = tid - 256;
    if (p >= 0 && p < len && n_dst > 0) {                // a line of one token has no products and no decisions
        float v = pn[p];
#pragma unroll
        for (int w = 1; w < kScreenWaves; ++w) v += pn[w * len + p];
        if (!(v <= 1.2676506e30f)) *wild = 1;
        v = sqrtf(v);
        inv32[p] = 1.0f / (v < 1e-12f ? 1e-12f : v);
    }
    __syncthreads();
    if (*wild) tau = INFINITY;
    // A screened cosine; outside the radius: never a candidate.  One that is no number counts as the lowest, so that exactly m sources
    // leave the line whatever the tokens hold.
    auto cosine = [&](int j, int k, float inv_src) {
        const int c = 2 * k + 1, dist = abs(c - 2 * j);
        float s = (S[k * sd + j] * inv_src) * inv32[c];
        s = s >= -2.f ? s : -2.f;
        return g.radius <= 0 || dist <= 2 * g.radius - 1 ? s : -INFINITY;
    };
    // the best of each source: eight lanes per source
    if (wave < 8) {
        const int j = tid >> 3, part = tid & 7;
        float mx = -INFINITY;
        if (j < n_src) {
            const float ia = inv32[2 * j];
            if (ONE) {                                   // all at once; destinations that are not there are others again
#pragma unroll
                for (int i = 0; i < 2 * TILE; ++i) mx = n_dst > 0 ? fmaxf(mx, cosine(j, min(part + 8 * i, n_dst - 1), ia)) : mx;
            } else {
                for (int k = part; k < n_dst; k += 8) mx = fmaxf(mx, cosine(j, k, ia));
            }
        }
        mx = oct_max(mx);
        if (j < n_src && part == 0) b32[j] = mx;
    }
    __syncthreads();

    __builtin_amdgcn_s_setprio(0);
    // ------------------------------------------------------------------ 2. exact: fp64 cosines where the screening cannot tell
    const bool is_src = lane < n_src;
    const float vbest = is_src ? b32[lane] : -INFINITY;
    bool contender = is_src && g.m > 0 && vbest > -INFINITY;
    if (g.m < n_src) {                                   // fewer than m above it: the m-th highest is not
        if (g.m <= 4) {
            float rest = vbest, top = -INFINITY;
            for (int i = 0; i < g.m; ++i) {
                top = wave_max32(rest);
                if (lane == (int)__builtin_ctzll(__ballot(rest == top))) rest = -INFINITY;
            }
            contender = contender && !(top > vbest + tau);
        } else {
            int above = 0;
            for (int i = 0; i < n_src; ++i) above += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(vbest), i)) > vbest + tau ? 1 : 0;
            contender = contender && above < g.m;
        }
    }
    const unsigned long long con = __ballot(contender), below = (1ull << lane) - 1ull;
    const int n_con = __popcll(con);
    const bool ranked = n_con > g.m;                     // some contender stays
    {
        unsigned long long left = con;
        for (int q = 0; q < n_con; ++q, left &= left - 1) {
            if (q % NW != wave) continue;
            const int j = (int)__builtin_ctzll(left), a = 2 * j;
            const float bj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(vbest), j));
            unsigned long long cand = __ballot(lane < n_dst && cosine(j, lane < n_dst ? lane : 0, inv32[a]) >= fmaxf(bj - tau, -3.f));
            double bs = -INFINITY;
            int bk = (int)__builtin_ctzll(cand);
            if (ranked || (cand & (cand - 1))) {
                const T* ta = row_of<T>(dx, dov, b, rid[a], g, dD);
                while (cand) {                           // ascending, two at a time
                    const int k1 = (int)__builtin_ctzll(cand);
                    cand &= cand - 1;
                    const int k2 = cand ? (int)__builtin_ctzll(cand) : k1;
                    cand &= cand - 1;
                    double c1, c2;
                    cos64_wave2<T>(ta, row_of<T>(dx, dov, b, rid[2 * k1 + 1], g, dD), row_of<T>(dx, dov, b, rid[2 * k2 + 1], g, dD), dD, lane, c1, c2);
                    if (c1 > bs) { bs = c1; bk = k1; }
                    if (c2 > bs) { bs = c2; bk = k2; }
                }
            }
            if (lane == 0) { escore[j] = bs; ebest[j] = bk; }
        }
    }
    __syncthreads();
    // the m best contenders (higher cosine, equal cosines: lower position), a source per lane, in every wavefront
    const double es = contender ? escore[lane] : 0.0;
    const int bk = contender ? ebest[lane] : -1;
    bool leaves = contender;
    if (ranked) {
        int rank = 0;
        for (unsigned long long left = con; left; left &= left - 1) {
            const int i = (int)__builtin_ctzll(left);
            const double t = lane_f64(es, i);
            rank += (t > es || (t == es && i < lane)) ? 1 : 0;
        }
        leaves = contender && rank < g.m;
    }
    LazyLine ln = {__ballot(leaves), 0ull};
    for (unsigned long long left = ln.gone; left; left &= left - 1)
        ln.takes |= 1ull << __builtin_amdgcn_readlane(bk, (int)__builtin_ctzll(left));

    // ------------------------------------------------------------------ 3. layout of the next grid
    auto slot = [&](int p) { return out_flat(lazy_slot(ln, p)); };
    if (wave == NW - 2 && is_src) {                      // sources
        const int p = 2 * lane, f = in_flat(p);
        if (!leaves) {
            const int of = slot(p);
            idx_out[img_out + of] = rid[p];
            sizes_out[img_out + of] = sz[p];
            if (kept_out) kept_out[img_out + of] = kept[p];
            if (pass_map) pass_map[img + f] = of;
        } else if (pass_map) {
            pass_map[img + f] = slot(2 * bk + 1);        // a merged source lands in its destination's slot
        }
    }
    if (wave == NW - 1) {                                // destinations
        const int ssz = is_src ? sz[2 * lane] : 0;
        int S1 = lane < n_dst ? sz[2 * lane + 1] : 0;
        for (unsigned long long left = ln.gone; left; left &= left - 1) {
            const int i = (int)__builtin_ctzll(left);
            S1 += __builtin_amdgcn_readlane(bk, i) == lane ? __builtin_amdgcn_readlane(ssz, i) : 0;
        }
        if (lane < n_dst) {
            const int p = 2 * lane + 1, f = in_flat(p), of = slot(p);
            idx_out[img_out + of] = ((ln.takes >> lane) & 1ull) ? g.n0 + g.ov_base + line * g.per_line + __popcll(ln.takes & below) : rid[p];
            sizes_out[img_out + of] = S1;
            if (kept_out) kept_out[img_out + of] = kept[p];
            if (pass_map) pass_map[img + f] = of;
        }
    }

    // ------------------------------------------------------------------ 4. the merged destinations
    // (features, and the metric too when the decisions were taken on one: it follows its own decisions)
    const int n_abs = __popcll(ln.takes);
    // One or two rows to merge: wavefronts without one of their own take a share of its channels (8x64x64x1280 bf16, merge
    // number 2, six passes: 173.0 us, 170.0; 12x32x32x1024: 99.9, 97.3; four rows in halves: 37.5, 39.2, so not those).
    // Tokens and metric differ in width: the parts of a row are counted on the wider of them, and a part's channels on the row itself
    // (of the narrower one, the last parts may have none).
    constexpr int kPiece = 64 * lz_io<T>::V;
    auto pieces = [](int width) { return (width + kPiece - 1) / kPiece; };
    const int n_merges = (xk ? 2 : 1) * n_abs, widest = pieces(xk && Dk > g.D ? Dk : g.D);
    const int parts = n_merges > 0 && 4 * n_merges <= NW ? min(NW / n_merges, widest) : 1;
    for (int kk = wave; kk < n_merges * parts; kk += NW) {
        const int merge = kk / parts;
        const bool on_metric = merge >= n_abs;
        const int at = on_metric ? merge - n_abs : merge;
        unsigned long long left = ln.takes;
        for (int i = 0; i < at; ++i) left &= left - 1;
        const int k = (int)__builtin_ctzll(left);
        T* mov = on_metric ? ovk : ov;
        const int mD = on_metric ? Dk : g.D, share = (pieces(mD) + parts - 1) / parts * kPiece, from = (kk - merge * parts) * share;
        lazy_merge<T>(on_metric ? xk : x, mov, g, mD, b, rid, sz, k, __ballot(leaves && bk == k),
                      mov + (b * g.cap + g.ov_base + line * g.per_line + at) * mD, lane, from, min(mD, from + share));
    }
}

// ------------------------------------------------------------------ the end of a call
typedef unsigned int lazy_u32x4 __attribute__((__vector_size__(16)));

struct FinishPart {
    const unsigned char *x, *ov;
    unsigned char* out;
    int row_bytes, lanes;        // lanes per row: 16 or 32 for rows of at most 256 or 512 bytes, else the wavefront
    int rows;                    // rows per wavefront where a row takes all of its lanes
    unsigned blocks;
};
struct FinishArgs {
    FinishPart part[2];          // tokens, metric (0 blocks: not wanted)
    const int32_t* idx;          // final ids, or null: the input grid as it is
    int n0, cap, n_out_per;
    int64_t n_rows, n_tok;       // output rows, input tokens of the whole call
    PassMaps maps;
    int32_t* merged_map;         // or null
    const int32_t* sizes_in;     // the rest only where idx is null
    int32_t *sizes_out, *kept_map;
};

// Three kinds of workgroup in one launch (none waits for another): rows of the tokens, rows of the metric, the composition
// of the pass maps, 256 entries each.  Rows are copied eight 16-byte pieces per lane at a time; short rows several to a
// wavefront, since a wavefront is three memory round trips long whatever it moves.
// Bound: HBM (8 x 64 x 64 x 1280 bf16: 20.4 us for 138 MB).
__global__ void __launch_bounds__(256)
oim_lazy_finish_k(FinishArgs a)
{
    unsigned blk = blockIdx.x;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const FinishPart& f = a.part[q];
        if (blk < f.blocks) {
            auto row_in = [&](int64_t b, int id) {
                id = id < 0 ? 0 : (id >= a.n0 + a.cap ? a.n0 + a.cap - 1 : id);        // ids come from the passes; stay in bounds regardless
                return id < a.n0 ? f.x + (b * a.n0 + id) * (int64_t)f.row_bytes : f.ov + (b * a.cap + (id - a.n0)) * (int64_t)f.row_bytes;
            };
            const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
            if (f.lanes < 64) {
                const int per_wave = 64 / f.lanes;
                const int64_t row = ((int64_t)blk * 4 + wave) * per_wave + lane / f.lanes;
                if (row >= a.n_rows) return;
                const int off = lane % f.lanes * 16;
                const uint32_t b = (uint32_t)row / (uint32_t)a.n_out_per;
                const unsigned char* in = row_in(b, a.idx ? a.idx[row] : (int)((uint32_t)row - b * (uint32_t)a.n_out_per));
                unsigned char* o = f.out + row * (int64_t)f.row_bytes;
                if (off < f.row_bytes) *reinterpret_cast<lazy_u32x4*>(o + off) = *reinterpret_cast<const lazy_u32x4*>(in + off);
                return;
            }
            // R rows of up to 8 / R pieces, all in flight together; the descriptors bound every piece, a row past the last has none
            auto copy = [&](auto rows) {
                constexpr int R = decltype(rows)::value, P = 8 / R;
                const int64_t row0 = ((int64_t)blk * 4 + wave) * R;
                if (row0 >= a.n_rows) return;
                // image and place of each row, and the ids, asked for together (there are fewer than 2^31 rows)
                uint32_t image[R];
                int id[R];
                uint32_t b = (uint32_t)row0 / (uint32_t)a.n_out_per, at = (uint32_t)row0 - b * (uint32_t)a.n_out_per;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    image[r] = b;
                    id[r] = (int)at;
                    if (++at == (uint32_t)a.n_out_per) { at = 0; ++b; }
                }
                if (a.idx)
#pragma unroll
                    for (int r = 0; r < R; ++r) id[r] = a.idx[row0 + r < a.n_rows ? row0 + r : row0];
                __amdgpu_buffer_rsrc_t ri[R], ro[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const bool there = row0 + r < a.n_rows;
                    const int64_t row = there ? row0 + r : row0;
                    ri[r] = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(row_in(there ? image[r] : image[0], id[r])), 0, there ? f.row_bytes : 0, 0x00020000);
                    ro[r] = __builtin_amdgcn_make_buffer_rsrc(f.out + row * (int64_t)f.row_bytes, 0, there ? f.row_bytes : 0, 0x00020000);
                }
                for (int base = 0; base < f.row_bytes; base += P * 1024) {
                    lazy_u32x4 v[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) v[k] = __builtin_amdgcn_raw_buffer_load_b128(ri[k / P], base + k % P * 1024 + lane * 16, 0, 0);
#pragma unroll
                    for (int k = 0; k < 8; ++k) __builtin_amdgcn_raw_buffer_store_b128(v[k], ro[k / P], base + k % P * 1024 + lane * 16, 0, 2);
                }
            };
            if (f.rows == 8) copy(std::integral_constant<int, 8>{});
            else if (f.rows == 4) copy(std::integral_constant<int, 4>{});
            else if (f.rows == 2) copy(std::integral_constant<int, 2>{});
            else copy(std::integral_constant<int, 1>{});
            return;
        }
        blk -= f.blocks;
    }
    const int64_t i = (int64_t)blk * 256 + threadIdx.x;
    if (i >= a.n_tok) return;
    const int64_t b = i / a.n0;
    int t = (int)(i - b * a.n0);
    if (!a.idx) {
        a.sizes_out[i] = a.sizes_in ? a.sizes_in[i] : 1;
        if (a.kept_map) a.kept_map[i] = t;
    }
    if (!a.merged_map) return;
    for (int k = 0; k < a.maps.n; ++k) t = a.maps.map[k][b * a.maps.n_in[k] + t];
    a.merged_map[i] = t;
}

// ------------------------------------------------------------------ host side
int oim_wide_lazy_rows(int h, int w, int axis, int m)
{
    const int len = axis ? w : h, nlines = axis ? h : w, n_dst = len / 2;
    return nlines * (m < n_dst ? m : n_dst);
}

// bf16 lines of 33 to 64 tokens are read in blocks of steps: of five where the wavefronts take fewer blocks of five than of four, else
// of four.  us of a call, merge number 2 out of both axes of 4 x 64 x 64, in blocks of four and of five: 1152 channels (4 and 5 steps of a
// wavefront) 42.1, 39.4; 1408 (5 and 6) 49.2, 47.8; 1536 (6) 50.4, 54.1; 1792 (7) 56.8, 60.5; 2048 (8) 60.3, 66.2; 2560 (10) 74.3, 71.2; 4096
// (16) 110.0, 119.0; up to 1024 the same.  (8 x 64 x 64 x 1280, 5 steps: 77.0, 66.2.  Six in flight do not fit the registers.)
static bool screen_by_fives(int D)
{
    int fours = 0, fives = 0;
    for (int wave = 0; wave < kScreenWaves; ++wave) {
        const int steps = screen_run<screen<bf16_t>::KS>(D, wave).steps;
        fours += (steps + 3) / 4;
        fives += (steps + 4) / 5;
    }
    return fives < fours;
}

template <typename T>
static luvc_status run_lazy_pass(const T* x, T* ov, const T* xk, T* ovk, int Dk, const int32_t* idx_in, const int32_t* sizes_in, const int32_t* kept_in,
                                 int B, int n0, int h, int w, int D, int axis, int m, int radius, int cap, int ov_base,
                                 int32_t* idx_out, int32_t* sizes_out, int32_t* kept_out, int32_t* pass_map, hipStream_t st)
{
    const int len = axis ? w : h, nlines = axis ? h : w, n_src = (len + 1) / 2, n_dst = len / 2;
    if (len > kLazyMaxLen) { set_error("wide matching (one launch per pass): line of %d tokens", len); return LUVC_ERR_UNSUPPORTED; }
    LazyGeom g;
    g.n0 = n0; g.h = h; g.w = w; g.D = D; g.axis = axis; g.m = m; g.radius = radius; g.cap = cap; g.ov_base = ov_base;
    g.per_line = m < n_dst ? m : n_dst;
    const int sd = lazy_row_stride(n_src);
    const size_t lds = sizeof(double) * 64 + sizeof(float) * ((size_t)kScreenWaves * (1024 + len) + (size_t)n_dst * sd + len + 64) + sizeof(int) * ((size_t)3 * len + 65);
    // eight wavefronts; sixteen where so many destinations are merged that eight would take several rounds and a compute
    // unit has no second line to work on
    const int waves = g.per_line * (xk ? 2 : 1) > 8 && B * nlines <= 256 ? 16 : 8;
    // Steps in flight: six on lines of up to 32 tokens, four on others, or five (above).  us with other numbers: 12 x 32 x 32 x 1024 bf16, six
    // passes 76.6 with four to six; 8 x 32 x 32 x 1408, four 49.9, 54.1 with four; x 2048 69.0, 62.1; fp32 8 x 24 x 24 x 1024, four 54.5, 49.6.
    // fp32 lines of 33 to 64 with three: 4 x 64 x 64 x 1024 138.1, 142.1; 8 x 48 x 48 x 768 101.1, 95.3.  Longer lines with three: bf16
    // 4 x 100 x 100 x 1024, two 94.2, 119.2, fp32 2 x 100 x 100 x 1024 107.8, 113.8; five do not fit the registers.
    constexpr int kMost = sizeof(T) == 2 ? 5 : 4;
#define LUVC_WIDE(TILE, LOADS) LUVC_LAUNCH("oim_wide_line", (oim_wide_line<T, TILE, LOADS>), dim3((unsigned)(B * nlines)), dim3(64 * waves), lds, st, x, ov, xk, ovk, Dk, \
                                   idx_in, sizes_in, kept_in, g, idx_out, sizes_out, kept_out, pass_map)
    if (len <= 32) LUVC_WIDE(1, 6);
    else if (len > 64) LUVC_WIDE(0, 4);
    else if (sizeof(T) == 2 && screen_by_fives(xk ? Dk : D)) LUVC_WIDE(2, kMost);
    else LUVC_WIDE(2, 4);
#undef LUVC_WIDE
    return check_launch("oim pass (wide matching, one launch)");
}

luvc_status oim_wide_lazy_pass(const void* x, void* ov, const void* metric, void* ov_metric, int Dm, const int32_t* idx_in, const int32_t* sizes_in, const int32_t* kept_in,
                               int B, int n0, int h, int w, int D, luvc_dtype dt, int axis, int m, int radius, int cap, int ov_base,
                               int32_t* idx_out, int32_t* sizes_out, int32_t* kept_out, int32_t* pass_map, hipStream_t st)
{
    if (dt == LUVC_F32)
        return run_lazy_pass<float>((const float*)x, (float*)ov, (const float*)metric, (float*)ov_metric, Dm, idx_in, sizes_in, kept_in, B, n0, h, w, D, axis, m, radius, cap, ov_base,
                                    idx_out, sizes_out, kept_out, pass_map, st);
    return run_lazy_pass<bf16_t>((const bf16_t*)x, (bf16_t*)ov, (const bf16_t*)metric, (bf16_t*)ov_metric, Dm, idx_in, sizes_in, kept_in, B, n0, h, w, D, axis, m, radius, cap, ov_base,
                                 idx_out, sizes_out, kept_out, pass_map, st);
}

luvc_status oim_lazy_finish(const LazyOutput* outs, int n_outs, const int32_t* idx, int B, int n0, int cap, int n_out_per, const PassMaps& maps,
                            int32_t* merged_map, const int32_t* sizes_in, int32_t* sizes_out, int32_t* kept_map, hipStream_t st)
{
    FinishArgs a{};
    a.idx = idx; a.n0 = n0; a.cap = cap; a.n_out_per = n_out_per;
    a.n_rows = (int64_t)B * n_out_per;
    a.n_tok = (int64_t)B * n0;
    a.maps = maps;
    a.merged_map = merged_map; a.sizes_in = sizes_in; a.sizes_out = sizes_out; a.kept_map = kept_map;
    unsigned grid = (merged_map || !idx) ? (unsigned)((a.n_tok + 255) / 256) : 0u;
    for (int q = 0; q < n_outs; ++q) {
        FinishPart& f = a.part[q];
        f.x = (const unsigned char*)outs[q].x; f.ov = (const unsigned char*)outs[q].ov; f.out = (unsigned char*)outs[q].out;
        f.row_bytes = outs[q].row_bytes;
        f.lanes = f.row_bytes <= 256 ? 16 : f.row_bytes <= 512 ? 32 : 64;
        // rows of a wavefront: as many as have eight pieces together, as long as there are 8192 wavefronts
        f.rows = 1;
        while (f.lanes == 64 && f.rows < 8 && 2 * f.rows * ((f.row_bytes + 1023) / 1024) <= 8 && a.n_rows >= (int64_t)8192 * 2 * f.rows) f.rows *= 2;
        const int64_t per_block = 4 * (64 / f.lanes) * f.rows;
        f.blocks = (unsigned)((a.n_rows + per_block - 1) / per_block);
        grid += f.blocks;
    }
    LUVC_LAUNCH("oim_lazy_finish", oim_lazy_finish_k, dim3(grid), dim3(256), 0, st, a);
    return check_launch("oim output rows and maps");
}

}  // namespace luvc

extern "C" luvc_status luvc_selftest_screen_tile(const void* a, const void* c, int D, luvc_dtype dtype, float* out, void* hip_stream)
{
    using namespace luvc;
    const int es = dtype == LUVC_F32 ? 4 : 2;
    if ((dtype != LUVC_F32 && dtype != LUVC_BF16) || !a || !c || !out || D < 1 || (D * es) % 16 != 0 ||
        ((uintptr_t)a | (uintptr_t)c) % 16 || (uintptr_t)out % 4) {
        set_error("luvc_selftest_screen_tile: unknown dtype, null or misaligned pointer, or rows that are not multiples of 16 bytes");
        return LUVC_ERR_INVALID_ARG;
    }
    hipStream_t st = (hipStream_t)hip_stream;
    if (dtype == LUVC_F32) LUVC_LAUNCH("selftest_screen_tile", (selftest_screen_tile<float>), dim3(1), dim3(64), 0, st, (const float*)a, (const float*)c, D, out);
    else                   LUVC_LAUNCH("selftest_screen_tile", (selftest_screen_tile<bf16_t>), dim3(1), dim3(64), 0, st, (const bf16_t*)a, (const bf16_t*)c, D, out);
    return check_launch("selftest screen tile");
}

extern "C" luvc_status luvc_selftest_screen_bound(int D, luvc_dtype dtype, int* channels, float* eps)
{
    using namespace luvc;
    if ((dtype != LUVC_F32 && dtype != LUVC_BF16) || !channels || !eps || D < 1) {
        set_error("luvc_selftest_screen_bound: unknown dtype, null pointer, or no channels");
        return LUVC_ERR_INVALID_ARG;
    }
    *channels = 0;
    for (int wave = 0; wave < kScreenWaves; ++wave) {
        const bool f32 = dtype == LUVC_F32;
        const ScreenRun run = f32 ? screen_run<screen<float>::KS>(D, wave) : screen_run<screen<bf16_t>::KS>(D, wave);
        const int c = run.steps * (f32 ? screen<float>::KS : screen<bf16_t>::KS) + run.rest;
        if (c > *channels) *channels = c;
    }
    *eps = screen_eps(D);
    return LUVC_OK;
}
