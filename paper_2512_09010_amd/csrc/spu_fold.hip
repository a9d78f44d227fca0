// SPU score (paper Section 3.3, Eq. 4-8) for N = N1 N2 tokens with N1 in 9 .. 16, N2 <= 256 and a pass band of up to 15 N1: the products of
// spu_mat.hip without a table of operands.
//
// The multiples j and -j of N1 are folded together.  With C_j = sum_b cos(2 pi b j / N2) T[b], S_j likewise, of the real and the imaginary parts of T (see spu_mat.hip), the bins
// c + N1 j and c - N1 j are
//   Z[j] = (C_j Tr + S_j Ti) + i (C_j Ti - S_j Tr),      Z[-j] = (C_j Tr - S_j Ti) + i (C_j Ti + S_j Tr)
// so products 2 have the rows (C_j, S_j), j >= 0, and Tr and Ti as two operands: half the products of one row per bin and part.  With
// g+ = M[j] + M[-j], g- = M[j] - M[-j] the way back takes
//   Vr = sum_j cos (g+ C_j Tr + g- S_j Ti) + sin (g+ S_j Tr - g- C_j Ti),      Vi = sum_j cos (g+ C_j Ti - g- S_j Tr) + sin (g- C_j Tr + g+ S_j Ti)
// and a lane has all eight values of a j in its own registers.
// The cosines and sines are those of N2 places on a circle.  A table of these places, each value two fp16 terms in a word (and a third
// beside them), is all there is in LDS (3 KB; operands as they enter the products would be 128 KB for 4096 tokens): a lane follows its own b j
// modulo N2 and puts its operand together from what it reads, for the eight products of a row block that use it.
// Accuracy: as in spu_mat.  The third term is taken by one block of rows, whose products have room for it; with two the way back is
// two terms, and what they take on the mean is given back.
// A workgroup owns 64 channels, a wavefront four pairs; tokens come as in spu_mat.hip.  Energies of four tiles at a time are added
// over the wavefronts.
// Bound: the instructions of two wavefronts per SIMD, whose products and vector instructions overlap little: 20 or 26 products
// and about 110 vector instructions per pair and 16 subsequences.  us of a call, bf16 tokens that no cache holds, calls one after the other:
// 4x4096x3584, sigma = 100 63.6 (spu_conv 90, spu_fft16q 110), sigma = 240 70.7 (spu_conv 85.9), 2x3328x5120, 133 57.8 (121), 2x3000x3584, 150 54.6 (76.6);
// where spu_mat takes the call too, it is the quicker one but for a few per cent: 4x2048x3584, 102 35.8 (34.8), 16x720x4096, 54 69.9 (45.8: several
// groups of channels per workgroup).
// Three and four blocks of rows (4x4096x3584, sigma = 409) are slower than spu_conv, 95 us for 84.  Tried and not kept: wavefronts
// of a SIMD half a tile apart, so that one has products while the other has vector instructions (no difference).
#include <algorithm>
#include <cstdlib>

#include "spu_mat.hpp"

namespace luvc {

namespace {

constexpr int kFoldTiles = 16;                   // most tiles of 16 subsequences
constexpr int kFoldRows = 2;                     // most blocks of 16 rows of the band, 8 multiples of N1 each
constexpr int kFoldDirect = 32;                  // tiles of a sample whose energies are added in one go
constexpr int kFoldPast = 3 * (8 * kFoldRows - 1);            // places behind the circle that repeat its first ones

// Where a place of the circle lies: steps of 4, 8, 16 or 32 places, which lengths with many factors of two take, fall in different banks
__device__ __forceinline__ uint32_t ring_place(uint32_t i) { return i ^ i >> 5; }
inline __host__ __device__ int ring_size(int N2) { return (N2 + kFoldPast + 15) / 16 * 16; }

}  // namespace

template <int RB /* blocks of 16 rows of the band */>
__global__ void __launch_bounds__(kMatThreads, 2)
spu_fold(const bf16_t* __restrict__ x, const MatShape sh, int D, int64_t row_stride, int use_hamming, int n_tiles /* workgroups per sample */,
         float* __restrict__ partial /* [B, n_tiles, ld] */, float* __restrict__ gpartial, const TileSync sy, int ld, float* __restrict__ scores)
{
    constexpr int P = kMatPairs, WAVES = kMatWaves, THREADS = kMatThreads;
    constexpr int KS = (RB + 1) / 2;             // steps of a product over the band
    extern __shared__ __align__(16) unsigned char smem[];
    const int N = sh.N, N1 = sh.N1, N2 = sh.N2, NT = sh.NT, sigma = sh.sigma;
    mat_u32x4* data = reinterpret_cast<mat_u32x4*>(smem);                       // [3][256 rows][8]
    uint32_t* i2t = reinterpret_cast<uint32_t*>(data + 3 * kMatBuf);            // [2][2][64][4] last operand
    float2* tw = reinterpret_cast<float2*>(i2t + 2 * 2 * 256);                  // [NT][16 c][16]
    uint2* ring = reinterpret_cast<uint2*>(tw + NT * 256);                      // [ring_size]  cos, sin of 2 pi i / N2, each high | low,
    uint32_t* ring3 = reinterpret_cast<uint32_t*>(ring + ring_size(N2));        // [ring_size]  and their third terms
    float* gm = reinterpret_cast<float*>(ring3 + ring_size(N2));                // [sigma + 1]  M[f]
    // where the third chunk comes
    double2* root = reinterpret_cast<double2*>(data + 2 * kMatBuf);             // [16]  e^(2 pi i / N1)
    uint32_t* f1t = reinterpret_cast<uint32_t*>(root + 16);                     // [2][3][64][4] first operand
    float4* esum = reinterpret_cast<float4*>(data);                             // [2][4 tiles][WAVES][64] energies, on the way back
    __shared__ uint32_t look[2][64];
    __shared__ int is_last;
    const int item = (int)xcd_contiguous(blockIdx.x, gridDim.x);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 15, g = lane >> 4;
    const int b = item / n_tiles, tile = item - b * n_tiles, d0 = tile * kMatWidth;

    // ---- tokens
    const MatTokens tokens(x + (int64_t)b * N * row_stride, row_stride, D, N1, N2, NT, data, wave);
    auto issue = [&](int t) { tokens.issue(t, t, d0); };         // chunk t: subsequences 16 t .. + 15
    if (wave < WAVES / 2) {
        issue(0);
        if (NT > 1) issue(1);
    }

    // ---- tables
    {
        const int ntw = NT * 256, at_ring = ntw, at_gm = at_ring + N2, at_root = at_gm + sigma + 1, jobs = at_root + N1;
        const double inv_N2 = sh.inv_N * (double)N1;
        constexpr double kBoost = (double)(1 << kMatBoost);
#pragma clang loop unroll(disable)
        for (int j = tid; j < jobs; j += THREADS) {
            const int s = 16 * (j >> 8) + (j & 15), cc = (j >> 4) & 15;
            int num = s < N2 && cc < N1 ? s * cc : 0, den = N;
            double inv = sh.inv_N, sd, cd;
            if (j >= at_root) { num = j - at_root; den = N1; inv = sh.inv_N1; }
            else if (j >= at_gm) { num = j - at_gm; den = N - 1; inv = sh.inv_N_1; }
            else if (j >= at_ring) { num = j - at_ring; den = N2; inv = inv_N2; }
            circle(num, den, inv, &cd, &sd);
            if (j >= at_root) root[num] = make_double2(cd, sd);
            else if (j >= at_gm) gm[num] = (float)(use_hamming ? 0.54 + 0.46 * cd : 1.0);
            else if (j >= at_ring) {
                uint32_t h, l, e;
                split16x3(kBoost * cd, kBoost * sd, h, l, e);
                const uint2 q = make_uint2((h & 0xffffu) | l << 16, h >> 16 | (l & 0xffff0000u));
                for (int i = num; i < N2 + kFoldPast; i += N2) { ring[ring_place(i)] = q; ring3[ring_place(i)] = e; }
            } else {
                constexpr float down = (float)(1.0 / kBoost);
                tw[tw_place(j >> 4, j & 15)] = s < N2 && cc < N1 ? make_float2((float)cd * down, (float)sd * down) : make_float2(0.f, 0.f);
            }
        }
    }
    __syncthreads();
    const float inv_n2 = 1.f / (float)N2, inv_n1 = 1.f / (float)N1;
    place_operands(root, N1, inv_n1, sh.place_scale, f1t, i2t);
    __syncthreads();
    mat_u32x4 f1[2][3];
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int k = 0; k < 3; ++k) f1[o][k] = *reinterpret_cast<const mat_u32x4*>(f1t + (o * 3 + k) * 256 + lane * 4);
    MatTokens::landed(NT > 1);
    __syncthreads();

    // ---- there
    // this lane's words: places 4 g .. + 3 of subsequence c of a tile, channel pairs 4 wave .. + 3
    const lds_word* words = (const lds_word*)reinterpret_cast<const uint32_t*>(data) + ((4 * g) * 16 + c) * 32 + (wave ^ (c >> 1)) * 4;
    auto onward = [&](uint32_t& at, uint32_t by) {           // places modulo N2
        const uint32_t n = at + by, less = n - (uint32_t)N2;
        at = n < less ? n : less;
    };
    mat_f32x4 acc[P][RB][2];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int rt = 0; rt < RB; ++rt) acc[p][rt][0] = acc[p][rt][1] = mat_f32x4{0.f, 0.f, 0.f, 0.f};
    MatScale scale;
    {
        // operand of block rt: row c, which is the cosine or the sine of multiple j, columns b = 16 t + 4 g .. + 3
        uint32_t at[RB], one[RB], tile_step[RB];
#pragma unroll
        for (int rt = 0; rt < RB; ++rt) {
            const int j = rt * 8 + (c >> 1);
            at[rt] = (uint32_t)mat_rest(4 * g * j, N2, inv_n2);
            one[rt] = (uint32_t)mat_rest(j, N2, inv_n2);
            tile_step[rt] = (uint32_t)mat_rest(16 * j, N2, inv_n2);
        }
        const uint32_t* mine = reinterpret_cast<const uint32_t*>(ring) + (c & 1);
        const int tw_there = tw_place(c, 4 * g), tw_there2 = tw_place(c, 4 * g + 2);
#pragma clang loop unroll(disable)
        for (int t = 0; t < NT; ++t) {
            const lds_word* buf = words + (t % 3) * (kMatBuf * 4);
            mat_f32x4 T[P][2];                   // subsequence 4 g + v of the tile
            const MatTwiddles twiddles{tw + t * 256 + tw_there, tw + t * 256 + tw_there2};
            const float m = places_to_bins(T, buf, f1, twiddles, scale.f);
            if (wave < WAVES / 2 && t + 2 < NT) issue(t + 2);
            if (__any(m > (scale.unset ? 0.f : 32768.f))) {
                const float f = into_range(T, m, buf, f1, twiddles, scale);
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int rt = 0; rt < RB; ++rt) { acc[p][rt][0] *= f; acc[p][rt][1] *= f; }
            }
            // high and low parts of four subsequences are the eight values of K: one product with the high parts of the constants
            // twice, one with their low parts
            mat_u32x4 tv[P][2];
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
            // subsequences -> rows of the band
#pragma unroll
            for (int rt = 0; rt < RB; ++rt) {
                uint32_t k[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) k[v] = mine[2 * ring_place(at[rt] + (uint32_t)v * one[rt])];
                onward(at[rt], tile_step[rt]);
                const uint32_t h0 = __builtin_amdgcn_perm(k[1], k[0], 0x05040100u), h1 = __builtin_amdgcn_perm(k[3], k[2], 0x05040100u);
                const uint32_t l0 = __builtin_amdgcn_perm(k[1], k[0], 0x07060302u), l1 = __builtin_amdgcn_perm(k[3], k[2], 0x07060302u);
                const mat_u32x4 ah{h0, h1, h0, h1}, al{l0, l1, l0, l1};
#pragma unroll
                for (int o = 0; o < 2; ++o)
#pragma unroll
                    for (int p = 0; p < P; ++p) acc[p][rt][o] = mac_f16(acc[p][rt][o], al, tv[p][o]);
#pragma unroll
                for (int o = 0; o < 2; ++o)
#pragma unroll
                    for (int p = 0; p < P; ++p) acc[p][rt][o] = mac_f16(acc[p][rt][o], ah, tv[p][o]);
            }
            MatTokens::landed(t + 2 < NT);
            __syncthreads();
        }
    }
    // ---- mask, scaled for the way back; row of the operands: bin c, K: (cosine, sine) of the multiples of a lane
    mat_u32x4 gh[P][2][KS], gl[P][2][KS];
    float back;
    {
        const bool live = d0 + 8 * wave < D;     // channels come in eights
        float m = 0.f;
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int rt = 0; rt < RB; ++rt)
#pragma unroll
                for (int o = 0; o < 2; ++o)
#pragma unroll
                    for (int v = 0; v < 4; ++v) m = fmaxf(m, fabsf(acc[p][rt][o][v]));
        m = 4.f * wave_max(m);                   // no weight is larger than 1, no value than four products with one
        const int by = clampi(9 - exponent(m), -120, 120);
        const float f = m > 0.f && live ? pow2(by) : 0.f;
        back = pow2(clampi(-(scale.e + by + sh.down), -126, 126));
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int rt = 2 * ks + (w >> 1), e = 2 * (w & 1), j = rt * 8 + 2 * g + (w & 1);
                if (rt >= RB) {
#pragma unroll
                    for (int p = 0; p < P; ++p)
#pragma unroll
                        for (int o = 0; o < 2; ++o) gh[p][o][ks][w] = gl[p][o][ks][w] = 0u;
                    continue;
                }
                auto weight = [&](int k) {
                    const int a = k < 0 ? -k : k;
                    return c < N1 && a <= sigma && 2 * k != -N ? gm[a <= sigma ? a : 0] * f : 0.f;
                };
                const float up = weight(c + N1 * j), down = j ? weight(c - N1 * j) : 0.f;
                const float gp = up + down, gn = j ? up - down : 0.f;
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const mat_f32x4 &r = acc[p][rt < RB ? rt : 0][0], &i = acc[p][rt < RB ? rt : 0][1];
                    uint32_t h, l;
                    split16(fmaf(gp, r[e], gn * i[e + 1]), fmaf(gp, r[e + 1], -gn * i[e]), h, l);
                    gh[p][0][ks][w] = h; gl[p][0][ks][w] = l;
                    split16(fmaf(gp, i[e], -gn * r[e + 1]), fmaf(gn, r[e], gp * i[e + 1]), h, l);
                    gh[p][1][ks][w] = h; gl[p][1][ks][w] = l;
                }
            }
        if constexpr (RB == 1) {                 // eight values are half the K of a product: high parts twice, low and high parts
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int o = 0; o < 2; ++o)
#pragma unroll
                    for (int w = 0; w < 2; ++w) gh[p][o][0][2 + w] = gl[p][o][0][2 + w] = gh[p][o][0][w];
        }
    }
    // the look at the arrival words, through LDS: see spu_mat
    if (wave == 0) {
        const tile_tag_t* w = tiles_word<kFoldDirect>(sy, b, tile, n_tiles);
        if (w) {
            load_word_to_lds(w, lds_address(look[0]));
            load_word_to_lds((const uint32_t*)w + 1, lds_address(look[1]));
        }
    }
    // ---- back
    {
        mat_u32x4 i2[2][2];
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int k = 0; k < 2; ++k) i2[o][k] = *reinterpret_cast<const mat_u32x4*>(i2t + (o * 2 + k) * 256 + lane * 4);
        float* pout = partial + ((int64_t)b * n_tiles + tile) * ld;
        // operand of block rt: column b = 16 t + c, multiples 8 rt + 2 g and the next
        uint32_t at[RB][2], tile_step[RB][2];
        int tw_back[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) tw_back[v] = tw_place(4 * g + v, c);
#pragma unroll
        for (int rt = 0; rt < RB; ++rt)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int j = rt * 8 + 2 * g + e;
                at[rt][e] = (uint32_t)mat_rest(c * j, N2, inv_n2);
                tile_step[rt][e] = (uint32_t)mat_rest(16 * j, N2, inv_n2);
            }
#pragma clang loop unroll(disable)
        for (int t = 0; t < NT; ++t) {
            float wc[4], ws[4], sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int v = 0; v < 4; ++v) { const float2 q = tw[t * 256 + tw_back[v]]; wc[v] = q.x; ws[v] = q.y; }
            mat_u32x4 kh[KS], kl[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const int rt = 2 * ks + (w >> 1);
                    if (rt >= RB) continue;
                    uint32_t& a = at[rt < RB ? rt : 0][w & 1];
                    const uint32_t place = ring_place(a);
                    const uint2 q = ring[place];
                    onward(a, tile_step[rt < RB ? rt : 0][w & 1]);
                    kh[ks][w] = __builtin_amdgcn_perm(q.y, q.x, 0x05040100u);
                    kl[ks][w] = __builtin_amdgcn_perm(q.y, q.x, 0x07060302u);
                    if (RB == 1) { kl[ks][2 + w] = kh[ks][w]; kh[ks][2 + w] = ring3[place]; }         // to go with gh, gl
                }
            mat_f32x4 z[P][2];
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int p = 0; p < P; ++p) z[p][o] = mat_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
                for (int o = 0; o < 2; ++o)
#pragma unroll
                    for (int p = 0; p < P; ++p) z[p][o] = mac_f16(z[p][o], gl[p][o][ks], kh[ks]);
#pragma unroll
                for (int o = 0; o < 2; ++o)
#pragma unroll
                    for (int p = 0; p < P; ++p) z[p][o] = mac_f16(z[p][o], gh[p][o][ks], kl[ks]);
                if (RB > 1)
#pragma unroll
                for (int o = 0; o < 2; ++o)
#pragma unroll
                    for (int p = 0; p < P; ++p) z[p][o] = mac_f16(z[p][o], gh[p][o][ks], kh[ks]);
            }
            // before the products of the other wavefront of the SIMD: see spu_mat.  Score and prune of 4x4096x3584, sigma = 102, 70.1 -> 69.4 us,
            // 2x3328x5120 67.2 -> 66.6, 2x3000x3584 57.2 -> 56.6.
            __builtin_amdgcn_s_setprio(1);
            bins_to_energies(sum, z, wc, ws, i2);
            __builtin_amdgcn_s_setprio(0);
            esum[((t & 7) * WAVES + wave) * 64 + lane] = make_float4(sum[0] * back * back, sum[1] * back * back, sum[2] * back * back, sum[3] * back * back);
            if ((t & 3) == 3 || t == NT - 1) {
                // four tiles: the sums over the wavefronts; the next four go to the other half meanwhile
                __syncthreads();
                const int t0 = t & ~3;
                for (int q = tid; q < (t - t0 + 1) * 256; q += THREADS) {
                    const int s = 16 * (t0 + (q >> 8)) + (q & 15), a = (q >> 4) & 15;
                    const float* e = reinterpret_cast<const float*>(esum + ((t0 & 7) + (q >> 8)) * WAVES * 64) + ((a >> 2) * 16 + (q & 15)) * 4 + (a & 3);
                    double all = 0.0;
#pragma unroll
                    for (int w = 0; w < WAVES; ++w) all += (double)e[w * 256];
                    if (a < N1 && s < N2) tile_store(pout + (N2 * a + s), (float)(all * sh.energy));
                }
            }
        }
    }
    if (wave == 0) {
        MatTokens::landed(false);
        tiles_claim<kFoldDirect>(sy, b, tile, n_tiles, (tile_tag_t)look[1][lane] << 32 | look[0][lane]);
    }
    tiles_to_scores<THREADS, kFoldDirect>(partial, gpartial, sy, scores, b, tile, n_tiles, N, ld, &is_last);
}

namespace {

size_t fold_lds(const MatShape& sh)
{
    return (size_t)3 * kMatBuf * 16 + 4096 + (size_t)sh.NT * 256 * 8 + (size_t)ring_size(sh.N2) * 12 + (size_t)(sh.sigma + 1) * 4;
}
// the largest N1: fewest tiles, fewest multiples
bool fold_shape(int N, int sigma, MatShape* sh, int* rb)
{
    for (int N1 = 16; N1 >= 9; --N1) {
        if (N % N1) continue;
        const int N2 = N / N1, NT = (N2 + 15) / 16, dn = (sigma + N1 - 1) / N1, RB = (dn + 8) / 8;       // multiples 0 .. dn
        if (NT > kFoldTiles || RB > kFoldRows || N2 < 2) continue;
        *sh = MatShape{1.0 / N, 1.0 / (N - 1), 1.0 / N1, 1.0, 1.0, N, N1, N2, NT, sigma, dn, dn + sigma / N1 + 1, 0};
        *rb = RB;
        return true;
    }
    return false;
}

}  // namespace

int spu_fold_blocks(int N, int sigma)
{
    MatShape sh;
    int rb;
    return fold_shape(N, sigma, &sh, &rb) ? rb : 0;
}
int spu_fold_tiles(int D) { return (D + kMatWidth - 1) / kMatWidth; }

// us of one call as that of spu_mat: rounds of workgroups, one per compute unit, each with its tables and its hand-over.  Fitted to 123
// shapes of 56 to 4096 tokens, 0.87 to 1.12 of what was measured; the kernel takes 1 % less since (spu_mat_us has what a lower estimate would change).
double spu_fold_us(int B, int N, int D, int sigma)
{
    MatShape sh;
    int rb;
    fold_shape(N, sigma, &sh, &rb);
    const int n_tiles = spu_fold_tiles(D);
    return 4.6 + (n_tiles > kFoldDirect ? 1.4 : 0.0) + (double)(((int64_t)B * n_tiles + 255) / 256) * (4.8 + sh.NT * (2.5 + 0.53 * rb));
}

luvc_status spu_score_fold(const void* x, int B, int N, int D, int64_t row_stride, int sigma, int use_hamming,
                           float* partial, float* gpartial, const TileSync& sy, float* scores, hipStream_t st)
{
    MatShape sh;
    int rb;
    if (!fold_shape(N, sigma, &sh, &rb)) { set_error("spu_fold: N = %d, sigma = %d", N, sigma); return LUVC_ERR_INVALID_ARG; }
    mat_scales(&sh, rb == 1 ? 1 : 2);
    const int n_tiles = spu_fold_tiles(D), ld = (N + 3) / 4 * 4;
#define LUVC_FOLD(RB) LUVC_LAUNCH("spu_fold", (spu_fold<RB>), dim3((unsigned)((int64_t)B * n_tiles)), dim3(kMatThreads), fold_lds(sh), st, (const bf16_t*)x, sh, D, \
                                  row_stride, use_hamming, n_tiles, partial, gpartial, sy, ld, scores)
    if (rb == 1) LUVC_FOLD(1);
    else LUVC_FOLD(2);
#undef LUVC_FOLD
    return check_launch("spu score (fold)");
}

}  // namespace luvc
