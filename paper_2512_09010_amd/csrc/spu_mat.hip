// SPU score (paper Section 3.3, Eq. 4-8) for N = N1 N2 tokens with N1 in 9 .. 16, N2 <= 128 and a pass band of up to 7 N1: the two
// transforms and the two back as products on the matrix cores, in fp32 accuracy, without a trip through LDS in between.
//
// Two real channels (d, d + 1) are one complex signal, as in spu_fft.hip; they lie side by side in memory, so a 32-bit word is a
// complex value of an operand.  Token n = N2 a + b (place a < N1, subsequence b < N2), bin k = c + N1 j, c < N1, and j over the
// multiples of N1 that the pass band meets:
//   products 1   Y[b][c] = sum_a z[N2 a + b] e^(-2 pi i a c / N1)           rows b, K = (a, re / im): tokens x constants
//   twiddle      T[b][c] = Y[b][c] e^(-2 pi i b c / N)
//   products 2   Z[j][c] = sum_b e^(-2 pi i b j / N2) T[b][c]               rows j, K = b: constants x T
//   mask         G = M[|c + N1 j|] Z
//   products 3   V[c][b] = sum_j G[j][c] e^(2 pi i b j / N2)                rows c, K = j: G x constants
//   twiddle      U[c][b] = V[c][b] e^(2 pi i b c / N)
//   products 4   z'[a][b] = sum_c e^(2 pi i a c / N1) U[c][b]               rows a, K = (c, re / im): constants x U
//   energy       |z'|^2 / N^2 over the channel pairs
// Up to eight multiples have two rows of products 2 and 3 each, real and imaginary part, and K = (b, re / im); of more, j and -j go
// together, rows (cosine, sine) of j >= 0 and the real and the imaginary part of T as two operands: see spu_fold.hip.  16 x 16 tiles with 32 values of K (v_mfma_f32_16x16x32): a lane's result holds four rows 4 g .. 4 g + 3
// of one column (g = lane / 16), an operand eight values of K of one row or column.  Each product contracts what were the rows of the
// one before it, and the order of K is free, so a result, turned into fp16, is the next operand as it lies in the registers.
//
// Accuracy.  Tokens are bf16 and enter as they are, the constants of products 1 are three bf16 terms.  From then on a value is the sum of
// two fp16 values, to nearest (2^-23 of it at most); a wavefront brings its values into the range of fp16 by powers of two.  That
// rounding differs from channel to channel and all but vanishes in the energy over them.  What is the same in all channels does not:
// the constants on the way back, which raise and lower every score with its place.  Those of products 3 are three fp16 terms (low
// times high, high times high: one product; high times low and third times high: the other), the circle of products 4 has a radius
// at which its points are all but exact (mat_scales), M is applied as it is (at most 1) and everything that scales all energies
// alike, 1 / N^2 among it, is one factor in fp64.  rms of the relative error against fp64, 2.0 .. 3.8e-8, of which the fp32 score's own
// rounding is 1.9 .. 3.4e-8.  Of the error of the kernel that takes the same call where rows do not lie in 16-byte pieces, on 125
// shapes: spu_conv 0.81, spu_fft16q 0.65, spu_circ 0.99 for tokens smooth over an image and 1.04 for white ones.  (Two terms in products 3,
// radius 1 and weights M / N as fp32 values: up to 7e-8, 1.0 to 1.5 of it.)
//
// A workgroup owns 64 channels (a cache line of every token row) at a time, a wavefront four pairs.  Tokens come into LDS by 16
// subsequences (32 KB) straight from memory, three chunks in turn, two on their way; every wavefront reads its own words.  On the way
// back nothing is fetched but constants, and the next group's first chunks come in meanwhile.
// Bound: instructions issued by two wavefronts per SIMD.  Per pair and 16 subsequences 20 products (one holds the vector unit
// up for 8 of its 16 cycles; a row per multiple and part: 19) and about 100 vector instructions of 4 cycles, 72 of which the method needs: twiddles 32, halves 32,
// energies 8.  us of a call, bf16 tokens that no cache holds, calls one after the other: 8x1024x3584, sigma = 102 33.0 (spu_fft16q 40.9),
// 16x720x4096, 54 44.1 (58.1), 8x1280x3584, 110 42.0 (49.5), 4x2048x3584, 102 34.8 (42.9), 32x390x3584, 58 54.2 (spu_circ 105),
// 32x576x896, 57 26.8 (spu_fft16q 32.6), 5x1352x3200, 91 31.6 (spu_conv 63.7).  Folded rows for all bands: 16x720x4096 45.8.
// Tried and not kept: two wavefronts that fetch for the other eight (40 us for 38 at that time); two pairs per wavefront and
// four wavefronts per SIMD (16x720x4096 71 for 51); products and vector instructions put in turns by hand; tokens through registers
// (one chunk on its way: 42); bands of up to 32 multiples with a row per multiple and part, as two-term constants (24 products for
// two blocks and more; farther off than the general kernels and little quicker).
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <numeric>

#include "spu_mat.hpp"

namespace luvc {

namespace {

constexpr int kMatTiles = 8;                     // most tiles of 16 subsequences
constexpr int kMatMultiples = 7;                 // highest multiple of N1
constexpr int kMatRows = 8;                      // most multiples of a band that has a row for each: 19 products for 20
constexpr int kMatDirect = 32;                   // tiles of a sample whose energies are added in one go

}  // namespace

// runs of equal samples that share a launch
struct MatLaunchRun {
    MatShape sh;
    int wg0, sample0;                            // first workgroup, first sample of the launch
    int64_t tok0;                                // first token
};
template <int RUNS> struct MatLaunch { int n; MatLaunchRun run[RUNS]; };

template <bool FOLD /* multiples j and -j together, or a row for each: up to 8 of them */, int RUNS>
__global__ void __launch_bounds__(kMatThreads, 2)
spu_mat(const bf16_t* __restrict__ x, const MatLaunch<RUNS> runs, int D, int64_t row_stride, int use_hamming, int gpw /* groups of channels per workgroup */,
        int n_tiles /* workgroups per sample */, float* __restrict__ partial /* [samples, n_tiles, ld] */, float* __restrict__ gpartial, const TileSync sy, int ld,
        float* __restrict__ scores)
{
    const int item = (int)xcd_contiguous(blockIdx.x, gridDim.x);
    int at_run = 0;
    if (RUNS > 1) at_run = run_of(runs.n, (unsigned)item, [&](int i) { return (unsigned)runs.run[i].wg0; });
    const MatLaunchRun& run = runs.run[at_run];
    const MatShape& sh = run.sh;
    constexpr int P = kMatPairs, WAVES = kMatWaves, THREADS = kMatThreads;
    constexpr int NA = FOLD ? 2 : 1;             // results of the way there per pair: of the two parts of T, or of both in one
    extern __shared__ __align__(16) unsigned char smem[];
    const int N = sh.N, N1 = sh.N1, N2 = sh.N2, NT = sh.NT, sigma = sh.sigma;
    mat_u32x4* f2 = reinterpret_cast<mat_u32x4*>(smem);                         // [NT][64] operands of the way there
    mat_u32x4* i1 = f2 + NT * 64;                                               // [NT][64] operands of the way back: low parts, high parts
    uint2* i1e = reinterpret_cast<uint2*>(i1 + NT * 64);                        // [NT][64] and their third terms
    float2* tw = reinterpret_cast<float2*>(i1e + NT * 64);                      // [NT][16 c][16]
    mat_u32x4* data = reinterpret_cast<mat_u32x4*>(tw + NT * 256);              // [3][256 rows][8]
    // what the tables are made of, where the third chunk comes
    double2* root = reinterpret_cast<double2*>(data + 2 * kMatBuf);             // [16]  e^(2 pi i / N1)
    double2* ring = root + 16;                                                  // [N2]  e^(2 pi i / N2)
    uint32_t* f1t = reinterpret_cast<uint32_t*>(ring + N2);                     // [2][3][64][4] first operand
    uint32_t* i2t = f1t + 2 * 3 * 256;                                          // [2][2][64][4] last operand
    float2* cs = reinterpret_cast<float2*>(i2t + 2 * 2 * 256);                  // [N]   (cos, sin)(2 pi i / N),
    float* gm = reinterpret_cast<float*>(cs + N);                               // [sigma + 1]  M[f]
    // energies of each wavefront [WAVES][NT][64]; one group leaves the tokens' place free by then
    float4* esum = reinterpret_cast<float4*>(gpw == 1 ? data : data + 3 * kMatBuf);
    __shared__ uint32_t look[2][64];
    __shared__ int is_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 15, g = lane >> 4;
    const int local = (item - run.wg0) / n_tiles, tile = item - run.wg0 - local * n_tiles, b = run.sample0 + local;
    const int64_t tok = run.tok0 + (int64_t)local * N;
    const int groups_all = (D + kMatWidth - 1) / kMatWidth, grp0 = tile * gpw, groups = groups_all - grp0 < gpw ? groups_all - grp0 : gpw;

    // ---- tokens
    const MatTokens tokens(x + tok * row_stride, row_stride, D, N1, N2, NT, data, wave);
    const int chunks = groups * NT;
    auto issue = [&](int i) {                    // chunk i: subsequences 16 t .. + 15 of group i / NT
        const int grp = i / NT;
        tokens.issue(i, i - grp * NT, (grp0 + grp) * kMatWidth);
    };
    if (wave < WAVES / 2) issue(0);

    // ---- tables
    {
        const int half = (N + 1) / 2, at_gm = half, at_ring = at_gm + sigma + 1, at_root = at_ring + N2, jobs = at_root + N1;
        for (int j = tid; j < jobs; j += THREADS) {
            int num = j, den = N;
            double inv = sh.inv_N, sd, cd;
            if (j >= at_root) { num = j - at_root; den = N1; inv = sh.inv_N1; }
            else if (j >= at_ring) { num = j - at_ring; den = N2; inv = sh.inv_N * (double)N1; }
            else if (j >= at_gm) { num = j - at_gm; den = N - 1; inv = sh.inv_N_1; }
            circle(num, den, inv, &cd, &sd);
            if (j >= at_root) root[num] = make_double2(cd, sd);
            else if (j >= at_ring) ring[num] = make_double2(cd, sd);
            else if (j >= at_gm) gm[num] = (float)(use_hamming ? 0.54 + 0.46 * cd : 1.0);
            else {
                cs[j] = make_float2((float)cd, (float)sd);
                if (j) cs[N - j] = make_float2((float)cd, -(float)sd);
                else if (N % 2 == 0) cs[half] = make_float2(-1.f, 0.f);
            }
        }
    }
    __syncthreads();
    if (wave < WAVES / 2 && chunks > 1) issue(1);
    const float inv_n2 = 1.f / (float)N2, inv_n1 = 1.f / (float)N1;
    // In loops that are not unrolled: the code runs once, and its size is what it costs.
    // way there, FOLD: row r of lane l is the cosine (r even) or sine of multiple r / 2, subsequences 4 (l / 16) .. + 3 of a tile; else rows 2 di,
    // 2 di + 1 are the real and the imaginary part of multiple di - dn, whose cosines and sines stand once.  Way back: cosine and sine of
    // multiples 2 (l / 16) and the next, subsequence l % 16
    constexpr double kBoost = (double)(1 << kMatBoost);
    if constexpr (!FOLD) {
#pragma clang loop unroll(disable)
        for (int j = tid; j < NT * 128; j += THREADS) {
            const int w = j & 3, i = j >> 2, di = i >> 2 & 7, s = 16 * (i >> 5) + 4 * (i & 3) + 2 * (w & 1), m = di - sh.dn + N2;
            const double2 q0 = ring[mat_rest(s * m, N2, inv_n2)], q1 = ring[mat_rest((s + 1) * m, N2, inv_n2)];
            const double on = di < sh.nb ? kBoost : 0.0;
            uint32_t h, l;
            split16((float)(on * (w & 2 ? q0.y : q0.x)), (float)(on * (w & 2 ? q1.y : q1.x)), h, l);
            uint32_t* to = reinterpret_cast<uint32_t*>(f2) + (i >> 5) * 256 + (j & 127);
            to[0] = h;
            to[128] = l;
        }
    }
#pragma clang loop unroll(disable)
    for (int i = tid; i < NT * 64; i += THREADS) {
        const int l = i & 63, r = l & 15, gg = l >> 4, t = i >> 6;
        uint32_t th[2], tl[2], bh[2], bl[2], be[2];
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            if constexpr (FOLD) {
                const int s = 16 * t + 4 * gg + 2 * w, m = r >> 1;
                const double2 q0 = ring[mat_rest(s * m, N2, inv_n2)], q1 = ring[mat_rest((s + 1) * m, N2, inv_n2)];
                split16((float)(kBoost * (r & 1 ? q0.y : q0.x)), (float)(kBoost * (r & 1 ? q1.y : q1.x)), th[w], tl[w]);
            }
            const int m = FOLD ? 2 * gg + w : 2 * gg + w - sh.dn + N2;
            const double2 q = ring[mat_rest((16 * t + r) * m, N2, inv_n2)];
            split16x3(kBoost * q.x, (FOLD ? kBoost : -kBoost) * q.y, bh[w], bl[w], be[w]);
        }
        if constexpr (FOLD) f2[i] = mat_u32x4{th[0], th[1], tl[0], tl[1]};
        i1[i] = mat_u32x4{bl[0], bl[1], bh[0], bh[1]};
        i1e[i] = make_uint2(be[0], be[1]);
    }
#pragma clang loop unroll(disable)
    for (int i = tid; i < NT * 256; i += THREADS) {
        const int s = 16 * (i >> 8) + (i & 15), cc = (i >> 4) & 15;
        constexpr float down = (float)(1.0 / kBoost);
        const float2 q = s < N2 && cc < N1 ? cs[s * cc] : make_float2(0.f, 0.f);
        tw[tw_place(i >> 4, i & 15)] = make_float2(q.x * down, q.y * down);
    }
    place_operands(root, N1, inv_n1, sh.place_scale, f1t, i2t);
    // of a lane's two multiples.  FOLD: M[j] + M[-j], M[j] - M[-j]
    float weight[NA][2];
    {
        auto at = [&](int k) {
            const int f = k < 0 ? -k : k;
            return c < N1 && f <= sigma && 2 * k != -N ? gm[f <= sigma ? f : 0] : 0.f;
        };
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int j = 2 * g + e;
            if constexpr (FOLD) {
                const float up = at(c + N1 * j), down = j ? at(c - N1 * j) : 0.f;
                weight[0][e] = up + down;
                weight[NA - 1][e] = j ? up - down : 0.f;
            } else {
                weight[0][e] = j < sh.nb ? at(c + N1 * (j - sh.dn)) : 0.f;
            }
        }
    }
    __syncthreads();
    mat_u32x4 f1[2][3], i2[2][2];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
#pragma unroll
        for (int k = 0; k < 3; ++k) f1[o][k] = *reinterpret_cast<const mat_u32x4*>(f1t + (o * 3 + k) * 256 + lane * 4);
#pragma unroll
        for (int k = 0; k < 2; ++k) i2[o][k] = *reinterpret_cast<const mat_u32x4*>(i2t + (o * 2 + k) * 256 + lane * 4);
    }
    MatTokens::landed(chunks > 1);
    __syncthreads();

    // this lane's words: places 4 g .. + 3 of subsequence c of a tile, channel pairs 4 wave .. + 3 of a group
    const lds_word* words = (const lds_word*)reinterpret_cast<const uint32_t*>(data) + ((4 * g) * 16 + c) * 32 + (wave ^ (c >> 1)) * 4;
    const int f2_at = ((c >> 1) * 4 + g) * 2, ro = c & 1;        // in 8-byte units: a row's cosines and sines, in either order
    const uint32_t f2_sign = ro ? 0x80008000u : 0u;
    const int tw_there = tw_place(c, 4 * g), tw_there2 = tw_place(c, 4 * g + 2);
    int tw_back[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) tw_back[v] = tw_place(4 * g + v, c);
    int ci = 0;
    for (int grp = 0; grp < groups; ++grp) {
        mat_f32x4 acc[P][NA];
#pragma unroll
        for (int p = 0; p < P; ++p) acc[p][0] = acc[p][NA - 1] = mat_f32x4{0.f, 0.f, 0.f, 0.f};
        MatScale scale;
        for (int t = 0; t < NT; ++t, ++ci) {
            const lds_word* buf = words + (ci % 3) * (kMatBuf * 4);
            mat_f32x4 T[P][2];                   // subsequence 4 g + v of the tile
            const MatTwiddles twiddles{tw + t * 256 + tw_there, tw + t * 256 + tw_there2};
            const float m = places_to_bins(T, buf, f1, twiddles, scale.f);
            if (wave < WAVES / 2 && ci + 2 < chunks) issue(ci + 2);
            if (__any(m > (scale.unset ? 0.f : 32768.f))) {
                const float f = into_range(T, m, buf, f1, twiddles, scale);
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int o = 0; o < NA; ++o) acc[p][o] *= f;
            }
            // subsequences -> rows of the band
            mat_u32x4 tv[P][2];
            if constexpr (FOLD) {
                // the real and the imaginary part; high and low parts of four subsequences are the eight values of K: one product with the
                // high parts of the constants twice, one with their low parts
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int o = 0; o < 2; ++o)
#pragma unroll
                        for (int w = 0; w < 2; ++w) {
                            uint32_t h, l;
                            split16(T[p][o][2 * w], T[p][o][2 * w + 1], h, l);
                            tv[p][o][w] = h; tv[p][o][2 + w] = l;
                        }
                const mat_u32x4 k = f2[t * 64 + lane], ah{k[0], k[1], k[0], k[1]}, al{k[2], k[3], k[2], k[3]};
#pragma unroll
                for (int o = 0; o < NA; ++o)
#pragma unroll
                    for (int p = 0; p < P; ++p) acc[p][o] = mac_f16(acc[p][o], al, tv[p][o]);
#pragma unroll
                for (int o = 0; o < NA; ++o)
#pragma unroll
                    for (int p = 0; p < P; ++p) acc[p][o] = mac_f16(acc[p][o], ah, tv[p][o]);
            } else {
                // high parts, low parts; real and imaginary parts of four subsequences are the eight values of K
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        uint32_t h, l;
                        split16(T[p][w >> 1][2 * (w & 1)], T[p][w >> 1][2 * (w & 1) + 1], h, l);
                        tv[p][0][w] = h; tv[p][1][w] = l;
                    }
                const uint2* at = reinterpret_cast<const uint2*>(f2 + t * 64) + f2_at;
                const uint2 h0 = at[ro], h1 = at[1 - ro], l0 = at[64 + ro], l1 = at[65 - ro];
                const mat_u32x4 ah{h0.x ^ f2_sign, h0.y ^ f2_sign, h1.x, h1.y}, al{l0.x ^ f2_sign, l0.y ^ f2_sign, l1.x, l1.y};
#pragma unroll
                for (int p = 0; p < P; ++p) acc[p][0] = mac_f16(acc[p][0], ah, tv[p][1]);
#pragma unroll
                for (int p = 0; p < P; ++p) acc[p][0] = mac_f16(acc[p][0], al, tv[p][0]);
#pragma unroll
                for (int p = 0; p < P; ++p) acc[p][0] = mac_f16(acc[p][0], ah, tv[p][0]);
            }
            MatTokens::landed(ci + 2 < chunks);
            __syncthreads();
        }
        // ---- mask, scaled for the way back: high parts twice, low and high parts; FOLD: of the real and of the imaginary part
        mat_u32x4 ghh[P][NA], glh[P][NA];
        float back;
        {
            const bool live = (grp0 + grp) * kMatWidth + 8 * wave < D;          // channels come in eights
            float m = 0.f;
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int o = 0; o < NA; ++o)
#pragma unroll
                    for (int v = 0; v < 4; ++v) m = fmaxf(m, fabsf(acc[p][o][v]));
            m = wave_max(m) * (FOLD ? 4.f : 1.f);           // no weight is larger than 1, folded values are of four
            const int by = clampi(9 - exponent(m), -120, 120);
            const float f = m > 0.f && live ? pow2(by) : 0.f;
            back = pow2(clampi(-(scale.e + by + sh.down), -126, 126));
            float wf[NA][2];
#pragma unroll
            for (int o = 0; o < NA; ++o) { wf[o][0] = weight[o][0] * f; wf[o][1] = weight[o][1] * f; }
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    const int e = 2 * w;
                    auto set = [&](int o, float a, float b) {
                        uint32_t h, l;
                        split16(a, b, h, l);
                        ghh[p][o][w] = ghh[p][o][2 + w] = glh[p][o][2 + w] = h; glh[p][o][w] = l;
                    };
                    if constexpr (FOLD) {
                        const mat_f32x4 &r = acc[p][0], &i = acc[p][NA - 1];
                        const float gp = wf[0][w], gn = wf[NA - 1][w];
                        set(0, fmaf(gp, r[e], gn * i[e + 1]), fmaf(gp, r[e + 1], -gn * i[e]));
                        set(NA - 1, fmaf(gp, i[e], -gn * r[e + 1]), fmaf(gn, r[e], gp * i[e + 1]));
                    } else {
                        set(0, acc[p][0][e] * wf[0][w], acc[p][0][e + 1] * wf[0][w]);
                    }
                }
        }
        // The look at the arrival words goes to LDS as well: a result in registers would be waited for in front of every
        // group's way back, with the tokens of the next one.  A word read in two halves that belong to different moments has
        // been claimed in between, and the claim then does nothing.
        if (wave == 0 && grp == groups - 1) {
            const tile_tag_t* w = tiles_word<kMatDirect>(sy, b, tile, n_tiles);
            if (w) {
                load_word_to_lds(w, lds_address(look[0]));
                load_word_to_lds((const uint32_t*)w + 1, lds_address(look[1]));
            }
        }
        // ---- back
#pragma clang loop unroll(disable)
        for (int t = 0; t < NT; ++t) {
            float wc[4], ws[4], sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int v = 0; v < 4; ++v) { const float2 q = tw[t * 256 + tw_back[v]]; wc[v] = q.x; ws[v] = q.y; }
            const mat_u32x4 klh = i1[t * 64 + lane];
            const uint2 ke = i1e[t * 64 + lane];
            mat_f32x4 z[P][2];
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                // else the operand of the imaginary part: (cos, -sin) -> (sin, cos)
                auto turn = [&](uint32_t k) { return FOLD || !o ? k : __builtin_amdgcn_alignbit(k, k, 16) ^ 0x8000u; };
                const mat_u32x4 klo{turn(klh[0]), turn(klh[1]), turn(klh[2]), turn(klh[3])}, kho{klo[2], klo[3], turn(ke.x), turn(ke.y)};
                const int go = FOLD ? o : 0;
#pragma unroll
                for (int p = 0; p < P; ++p) z[p][o] = mac_f16(mat_f32x4{0.f, 0.f, 0.f, 0.f}, glh[p][go], kho);
#pragma unroll
                for (int p = 0; p < P; ++p) z[p][o] = mac_f16(z[p][o], ghh[p][go], klo);
            }
            // The older wavefront of a SIMD would come first throughout and leave the other one alone at the end, where hardly anything
            // overlaps.  Whichever is in the second half of a tile, its vector instructions and short products, comes before one that
            // asks for the long products of the first.  us of score and prune with turns tile by tile, which had taken 32x390x3584 from 48.9
            // to 46.1 for the score alone, and so: 8x1024x3584 38.2, 37.2; 32x390x3584 54.5, 53.8; 16x720x4096 50.6, 49.9; 4x2048x3584 42.0, 41.0;
            // 5x1352x3200 38.5, 37.6.
            __builtin_amdgcn_s_setprio(1);
            bins_to_energies(sum, z, wc, ws, i2);
            __builtin_amdgcn_s_setprio(0);
            float4* at = esum + (wave * NT + t) * 64 + lane;
            float4 q = grp ? *at : make_float4(0.f, 0.f, 0.f, 0.f);
            q.x = fmaf(sum[0] * back, back, q.x);
            q.y = fmaf(sum[1] * back, back, q.y);
            q.z = fmaf(sum[2] * back, back, q.z);
            q.w = fmaf(sum[3] * back, back, q.w);
            *at = q;
        }
    }
    if (wave == 0) {
        MatTokens::landed(false);
        tiles_claim<kMatDirect>(sy, b, tile, n_tiles, (tile_tag_t)look[1][lane] << 32 | look[0][lane]);
    }
    // ---- sums over the wavefronts
    __syncthreads();
    const float* sums = reinterpret_cast<const float*>(esum);
    float* pout = partial + ((int64_t)b * n_tiles + tile) * ld;
    for (int n = tid; n < N; n += THREADS) {
        const int a = n / N2, s = n - a * N2;
        const float* at = sums + (s >> 4) * 256 + ((a >> 2) * 16 + (s & 15)) * 4 + (a & 3);
        double q = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) q += (double)at[w * NT * 256];
        tile_store(pout + n, (float)(q * sh.energy));
    }
    tiles_to_scores<THREADS, kMatDirect>(partial, gpartial, sy, scores + (tok - (int64_t)b * N), b, tile, n_tiles, N, ld, &is_last);
}

namespace {

constexpr size_t kMatLds = 160 * 1024 - 1024;

// How much shorter than 1 the (cos, sin) of multiples of 2 pi / n are as the sum of two fp16 values, on the mean
struct CircleLengths {
    double of[257];
    CircleLengths()
    {
        auto two_halves = [](double v) {
            auto half = [](double x) {
                int e;
                std::frexp(x, &e);
                const double unit = std::ldexp(1.0, (e < -13 ? -13 : e) - 11);
                return std::nearbyint(x / unit) * unit;
            };
            const double f = (double)(float)std::ldexp(v, kMatBoost), h = half(f);
            return std::ldexp(h + half(f - h), -kMatBoost);
        };
        of[0] = 0.0;
        for (int n = 1; n <= 256; ++n) {
            double sum = 0.0;
            for (int i = 0; i < n; ++i) {
                const double a = 6.283185307179586 * i / n, c = std::cos(a), s = std::sin(a);
                sum += c * two_halves(c) + s * two_halves(s) - 1.0;
            }
            of[n] = sum / n;
        }
    }
};
}  // namespace

// What the constants and the sums of the products make of the energies, given back in fp64 with the 1 / N of both transforms:
// - The circle of the N1 places, met by all channels alike in the last product, has a radius at which its points lie close to sums of
//   two fp16 values: found among 1 .. 2 in steps of 2^-20, rms distance 4e-10 (N1 = 10, 16) to 8e-9 of the radius, and 0 for N1 = 12,
//   for 1.8 to 4.7e-8 at radius 1.
// - Operands of the band as two fp16 terms are too short or too long by up to 5e-8, in a way that depends on N2 and the multiples: those
//   of the way there, and of the way back where there is no third term (`ways`).
// - The matrix cores' sums are cut off rather than rounded: 0.2e-8, the mean over 125 shapes of 240 to 4096 tokens, white and smooth.
void mat_scales(MatShape* sh, int ways)
{
    static const CircleLengths circle;
    static constexpr int kRadius[8] = {712158, 808423, 179569, 532094, 782212, 966972, 733288, 829792};         // N1 = 9 .. 16: 1 + this 2^-20
    double band = 0.0;
    for (int i = 0; i < sh->nb; ++i) band += circle.of[sh->N2 / std::gcd(sh->N2, std::abs(i - sh->dn))];
    sh->place_scale = 1.0 + std::ldexp((double)kRadius[sh->N1 - 9], -20);
    sh->down = (int)std::lround(std::log2(sh->N * sh->place_scale));
    const double one = std::ldexp(1.0 - ways * band / sh->nb + 0.2e-8, sh->down) / (sh->N * sh->place_scale);
    sh->energy = one * one;
}

namespace {

// fewest tiles, and the largest N1 with as many
bool mat_shape(int N, int sigma, MatShape* sh)
{
    int best = 0;
    for (int N1 = 16; N1 >= 9; --N1) {
        if (N % N1) continue;
        const int N2 = N / N1, NT = (N2 + 15) / 16, dn = (sigma + N1 - 1) / N1;
        if (NT > kMatTiles || dn > kMatMultiples || N2 < 2 || (best && NT >= best)) continue;
        best = NT;
        *sh = MatShape{1.0 / N, 1.0 / (N - 1), 1.0 / N1, 1.0, 1.0, N, N1, N2, NT, sigma, dn, dn + sigma / N1 + 1, 0};
    }
    return best != 0;
}
size_t mat_lds(const MatShape& sh, int gpw)
{
    return (size_t)3 * kMatBuf * 16 + (size_t)sh.NT * (64 * (16 + 16 + 8) + 256 * 8) + (gpw > 1 ? (size_t)kMatWaves * sh.NT * 1024 : 0);
}

}  // namespace

bool spu_mat_supported(int N, int sigma)
{
    MatShape sh;
    return mat_shape(N, sigma, &sh);
}

static int mat_groups(int D) { return (D + kMatWidth - 1) / kMatWidth; }

// How the samples of a launch are split: as few groups of channels to a workgroup as leave each compute unit one workgroup, or one
// group where the energies of several do not fit beside the tokens
MatPlan spu_mat_plan(const MatRun* runs, int n, int D)
{
    MatPlan p{};
    size_t lds_groups = 0;
    for (int i = 0; i < n; ++i) {
        MatShape sh;
        mat_shape(runs[i].N, runs[i].sigma, &sh);
        p.samples += runs[i].count;
        p.ld = std::max(p.ld, (runs[i].N + 3) / 4 * 4);
        p.lds = std::max(p.lds, mat_lds(sh, 1));
        lds_groups = std::max(lds_groups, mat_lds(sh, 2));
        p.fold = p.fold || sh.nb > kMatRows;
    }
    const int groups = mat_groups(D);
    p.gpw = (int)((p.samples * groups + 255) / 256);
    if (p.gpw > 1 && lds_groups > kMatLds) p.gpw = 1;
    if (p.gpw > 1) p.lds = lds_groups;
    p.n_tiles = (groups + p.gpw - 1) / p.gpw;
    return p;
}

// us of one call: the rounds that the workgroups take on the chip, one per compute unit, each with its tables and its hand-over.
// Fitted to 92 shapes of 56 to 2048 tokens, 0.91 to 1.15 of what was measured (two rounds of one tile 14.8
// for 16; five groups and more 42 for 48).  The kernel takes up to 6 % less since, and the line to the other kernels still lies well: with this
// estimate and that of spu_fold 5 % lower, 5 of 768 drawn calls change kernel, at 0.81, 0.98, 1.09, 1.11 and 1.14 of the time; 6 % higher 5, at 0.98
// to 1.34.
static double mat_group_us(const MatShape& sh) { return 0.4 + sh.NT * 2.95; }
double spu_mat_us(int B, int N, int D, int sigma)
{
    MatShape sh;
    mat_shape(N, sigma, &sh);
    const MatRun run{N, sigma, B, 0};
    const MatPlan p = spu_mat_plan(&run, 1, D);
    return 6.4 + (p.n_tiles > kMatDirect ? 1.4 : 0.0) + (double)(((int64_t)B * p.n_tiles + 255) / 256) * (2.1 + p.gpw * mat_group_us(sh));
}
// what a run adds to a launch that several share; 0: it does not go there
double spu_mat_work_us(int B, int N, int D, int sigma)
{
    MatShape sh;
    if (!mat_shape(N, sigma, &sh)) return 0.0;
    return (double)B * mat_groups(D) / 256.0 * mat_group_us(sh);
}

template <bool FOLD, int RUNS>
static void mat_launch(const void* x, const MatRun* runs, int n, const MatPlan& p, int D, int64_t row_stride, int use_hamming,
                       float* partial, float* gpartial, const TileSync& sy, float* scores, hipStream_t st)
{
    MatLaunch<RUNS> l;
    l.n = n;
    int64_t samples = 0;
    for (int i = 0; i < n; ++i) {
        mat_shape(runs[i].N, runs[i].sigma, &l.run[i].sh);
        mat_scales(&l.run[i].sh, 1);
        l.run[i].wg0 = (int)(samples * p.n_tiles);
        l.run[i].sample0 = (int)samples;
        l.run[i].tok0 = runs[i].tok0;
        samples += runs[i].count;
    }
    LUVC_LAUNCH("spu_mat", (spu_mat<FOLD, RUNS>), dim3((unsigned)(samples * p.n_tiles)), dim3(kMatThreads), p.lds, st, (const bf16_t*)x, l, D, row_stride, use_hamming,
                p.gpw, p.n_tiles, partial, gpartial, sy, p.ld, scores);
}

luvc_status spu_score_mat(const void* x, const MatRun* runs, int n, const MatPlan& p, int D, int64_t row_stride, int use_hamming,
                          float* partial, float* gpartial, const TileSync& sy, float* scores, hipStream_t st)
{
#define LUVC_MAT(FOLD, RUNS) mat_launch<FOLD, RUNS>(x, runs, n, p, D, row_stride, use_hamming, partial, gpartial, sy, scores, st)
    if (n > 1) { if (p.fold) LUVC_MAT(true, kMatMaxRuns); else LUVC_MAT(false, kMatMaxRuns); }
    else if (p.fold) LUVC_MAT(true, 1);
    else LUVC_MAT(false, 1);
#undef LUVC_MAT
    return check_launch("spu score (mat)");
}

}  // namespace luvc
