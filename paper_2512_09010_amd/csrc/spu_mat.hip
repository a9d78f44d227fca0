// SPU score (paper Section 3.3, Eq. 4-8) for N = N1 N2 tokens with N1 in 9 .. 16 and N2 <= 128: the two transforms and the two
// back as products on the matrix cores, in fp32 accuracy, without a trip through LDS in between.
//
// Two real channels (d, d + 1) are one complex signal, as in spu_fft.hip; they lie side by side in memory, so a 32-bit word is a
// complex value of an operand.  Token n = N2 a + b (place a < N1, subsequence b < N2), bin k = c + N1 j, c < N1, and j over the
// multiples of N1 that the pass band meets, nb of them:
//   products 1   Y[b][c] = sum_a z[N2 a + b] e^(-2 pi i a c / N1)           rows b, K = (a, re / im): tokens x constants
//   twiddle      T[b][c] = Y[b][c] e^(-2 pi i b c / N)
//   products 2   Z[j][c] = sum_b e^(-2 pi i b j / N2) T[b][c]               rows (j, re / im), K = (b, re / im): constants x T
//   mask         G = M[|c + N1 j|] / N  Z
//   products 3   V[c][b] = sum_j G[j][c] e^(2 pi i b j / N2)                rows c, K = (j, re / im): G x constants
//   twiddle      U[c][b] = V[c][b] e^(2 pi i b c / N)
//   products 4   z'[a][b] = sum_c e^(2 pi i a c / N1) U[c][b]               rows a, K = (c, re / im): constants x U
//   energy       |z'|^2 over the channel pairs
// 16 x 16 tiles with 32 values of K (v_mfma_f32_16x16x32): a lane's result holds four rows 4 g .. 4 g + 3 of one column (g = lane / 16),
// an operand eight values of K of one row or column.  Each product contracts what were the rows of the one before it, and the
// order of K is free, so a result, turned into fp16, is the next operand as it lies in the registers.
// Accuracy: tokens are bf16 and enter as they are, the constants of products 1 are three bf16 terms; from then on every value is
// the sum of two fp16 values, to nearest (2^-24 of it), constants too, in three products of the four.  A wavefront brings its
// values into the range of fp16 by powers of two.  What the rounding of the constants takes from every score the weights give back
// (mat_length).  Error against fp64 (rms of the relative error, 512 channels and more): 2.8 .. 3.8e-8, of which 2.4 .. 3.0e-8 are
// the score's own rounding; spu_fft16q stands at 3.6 .. 4.3e-8 on the same tokens.
//
// A workgroup owns 64 channels (a cache line of every token row) at a time, a wavefront four pairs.  Tokens come into LDS by 16
// subsequences (32 KB) straight from memory, three chunks in turn, two on their way; every wavefront reads its own words.  On the way
// back nothing is fetched but constants, and the next group's first chunks come in meanwhile.
// Bound: instructions issued by two wavefronts per SIMD.  Per pair and 16 subsequences 19, 20 or 24 products (one holds the vector unit
// up for 8 of its 16 cycles) and about 100 vector instructions of 4 cycles, 72 of which the method needs: twiddles 32, halves 32,
// energies 8.  bf16, tokens that no cache holds: 8x1024x3584 42 -> 36.4 us against spu_fft16q, 16x720x4096 65 -> 46,
// against spu_conv 16x390x1536 27 -> 19, against spu_circ 32x390x3584 102 -> 48.
// Bands of two blocks of rows whose multiples fit -7 .. 7 have their rows folded as in spu_fold.hip, 20 products for 24 and half the
// tables, which leaves room for several groups of channels per workgroup: 8x1024x3584 41.0 -> 36.4, 8x1280x3584, sigma = 110 54.7 ->
// 42.9, 8x1152x3584 53.7 -> 43.3, 16x1040x1536 51.3 -> 39.6; error 3.3 .. 3.8e-8 for 4.0 .. 4.5e-8 on the last.
// Tried and not kept: two wavefronts that fetch for the other eight (40 us for 38 at that time); two pairs per wavefront and
// four wavefronts per SIMD (16x720x4096 71 for 51); products and vector instructions put in turns by hand; tokens through registers
// (one chunk on its way: 42).
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <numeric>

#include "spu_mat.hpp"

namespace luvc {

namespace {

constexpr int kMatWaves = 8, kMatPairs = 4;      // wavefronts of a workgroup, channel pairs of a wavefront
constexpr int kMatWidth = 2 * kMatWaves * kMatPairs;
constexpr int kMatTiles = 8;                     // most tiles of 16 subsequences
constexpr int kMatDirect = 32;                   // tiles of a sample whose energies are added in one go
constexpr int kTwRow = 18;                       // float2 per row of the twiddles: 16 and a pad for the banks

}  // namespace

// runs of equal samples that share a launch
struct MatLaunchRun {
    MatShape sh;
    int wg0, sample0;                            // first workgroup, first sample of the launch
    int64_t tok0;                                // first token
};
template <int RUNS> struct MatLaunch { int n; MatLaunchRun run[RUNS]; };

template <int RB /* blocks of 16 rows of the band, 0: one of folded rows */, int RUNS>
__global__ void __launch_bounds__(64 * kMatWaves, 2)
spu_mat(const bf16_t* __restrict__ x, const MatLaunch<RUNS> runs, int D, int64_t row_stride, int use_hamming, int gpw /* groups of channels per workgroup */,
        int n_tiles /* workgroups per sample */, float* __restrict__ partial /* [samples, n_tiles, ld] */, float* __restrict__ gpartial, const TileSync sy, int ld,
        float* __restrict__ scores)
{
    const int item = (int)xcd_contiguous(blockIdx.x, gridDim.x);
    int at_run = 0;
    if (RUNS > 1)
        for (int i = 1; i < runs.n; ++i)
            if (item >= runs.run[i].wg0) at_run = i;
    const MatLaunchRun& run = runs.run[at_run];
    const MatShape& sh = run.sh;
    constexpr int P = kMatPairs, WAVES = kMatWaves, THREADS = 64 * WAVES;
    constexpr bool FOLD = RB == 0;
    constexpr int KS = FOLD ? 1 : (RB + 1) / 2;  // steps of a product over the band
    constexpr int NA = FOLD ? 2 : RB;            // results of the way there per pair: blocks, or the parts of the one
    constexpr int kF2 = FOLD ? 64 : RB * 2 * 32; // 16-byte pieces of a tile's operands on the way there
    constexpr int kBuf = 256 * 8;                // 16-byte pieces of a buffer: 256 rows of 8, which are 64 channels
    constexpr int kI1 = RB <= 1 ? 1 : 2 * KS;    // 1 KB blocks of an inverse operand
    extern __shared__ __align__(16) unsigned char smem[];
    const int N = sh.N, N1 = sh.N1, N2 = sh.N2, NT = sh.NT, sigma = sh.sigma;
    mat_u32x4* f2 = reinterpret_cast<mat_u32x4*>(smem);                         // [NT][RB][2][32] or [NT][64]
    mat_u32x4* i1 = f2 + NT * kF2;                                              // [NT][kI1][64]
    float2* tw = reinterpret_cast<float2*>(i1 + NT * kI1 * 64);                 // [NT][16 c][kTwRow]
    mat_u32x4* data = reinterpret_cast<mat_u32x4*>(tw + NT * 16 * kTwRow);      // [3][256 rows][8]
    // what the tables are made of, where the third chunk comes
    double2* root = reinterpret_cast<double2*>(data + 2 * kBuf);                // [16]  e^(2 pi i / N1)
    uint32_t* f1t = reinterpret_cast<uint32_t*>(root + 16);                     // [2][3][64][4] first operand
    uint32_t* i2t = f1t + 2 * 3 * 256;                                          // [2][2][64][4] last operand
    float2* cs = reinterpret_cast<float2*>(i2t + 2 * 2 * 256);                  // [N]   (cos, sin)(2 pi i / N),
    float* gm = reinterpret_cast<float*>(cs + N);                               // [sigma + 1]  M[f] / N
    // energies of each wavefront [WAVES][NT][64]; one group leaves the tokens' place free by then
    float4* esum = reinterpret_cast<float4*>(gpw == 1 ? data : data + 3 * kBuf);
    __shared__ uint32_t look[2][64];
    __shared__ int is_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 15, g = lane >> 4;
    const int local = (item - run.wg0) / n_tiles, tile = item - run.wg0 - local * n_tiles, b = run.sample0 + local;
    const int64_t tok = run.tok0 + (int64_t)local * N;
    const int groups_all = (D + kMatWidth - 1) / kMatWidth, grp0 = tile * gpw, groups = groups_all - grp0 < gpw ? groups_all - grp0 : gpw;
    const bf16_t* xb = x + tok * row_stride;

    // ---- tokens
    const uint32_t lds0 = lds_address(data);
    // The older half of the wavefronts fetches: they come first where two share a SIMD, and would wait for the younger ones.  A
    // thread fetches eight pieces of a chunk, the same piece of the rows of one subsequence s0 of a tile; places a >= N1,
    // subsequences >= N2 and channels >= D are not used, but have to be numbers: others of the same sample.  Row 16 a + s holds
    // its pieces in an order that depends on s, so that the 16 subsequences' words of a channel pair lie in 16 banks.
    const int s0 = tid / 8 & 15, piece = (tid & 7) ^ (s0 >> 1);
    const uint32_t row_bytes = (uint32_t)row_stride * 2u;
    const uint32_t off = (uint32_t)s0 * row_bytes + 16u * (uint32_t)piece;
    const uint32_t over = 16 * NT - 16 + s0 < N2 ? 0u : (uint32_t)(16 * NT - 15 + s0 - N2) * row_bytes;       // in the last tile
    auto issue = [&](int i) {                    // chunk i: subsequences 16 t .. + 15 of group i / NT
        const int grp = i / NT, t = i - grp * NT, d = (grp0 + grp) * kMatWidth;
        const char* base = reinterpret_cast<const char*>(xb) + (int64_t)(16 * t) * row_bytes + 2 * d;
        uint32_t less = t == NT - 1 ? over : 0u;
        if (d + 8 * piece >= D) less += 16u * (uint32_t)piece;
#pragma unroll
        for (int u = 0; u < 2 * P; ++u) {
            int a = 2 * u + wave / 2;
            a = a < N1 ? a : N1 - 1;
            load_to_lds(base + (int64_t)(N2 * a) * row_bytes, off - less, lds0 + (uint32_t)((i % 3) * kBuf + u * (THREADS / 2) + wave * 64) * 16u);
        }
    };
    auto landed = [&](bool newer) {              // all but the newest chunk asked for
        if (newer) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * P) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    const int chunks = groups * NT;
    if (wave < WAVES / 2) issue(0);

    // ---- tables
    {
        const int half = (N + 1) / 2, jobs = half + sigma + 1 + N1;
        for (int j = tid; j < jobs; j += THREADS) {
            const int f = j - half, r = f - (sigma + 1);
            double sd, cd;
            circle(r >= 0 ? r : f >= 0 ? f : j, r >= 0 ? N1 : f >= 0 ? N - 1 : N, r >= 0 ? sh.inv_N1 : f >= 0 ? sh.inv_N_1 : sh.inv_N, &cd, &sd);
            if (r >= 0) root[r] = make_double2(cd, sd);
            else if (f >= 0) gm[f] = (float)((use_hamming ? 0.54 + 0.46 * cd : 1.0) * sh.inv_N * sh.length);
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
    auto rest = [](int v, int n, float inv) { return v - n * (int)(((float)v + 0.5f) * inv); };      // v mod n, 0 <= v < 2^20
    // Word by word, in loops that are not unrolled: the code runs once, and its size is what it costs.  Rows of the band:
    // 2 di, 2 di + 1 are the real and the imaginary part of multiple di - dn of N1.
    if constexpr (FOLD) {
        // way there: row r of lane l is the cosine (r even) or sine of multiple r / 2, subsequences 4 (l / 16) .. + 3 of a tile; way back: cosine
        // and sine of multiples 2 (l / 16) and the next, subsequence l % 16; high parts, low parts
#pragma clang loop unroll(disable)
        for (int i = tid; i < NT * 64; i += THREADS) {
            const int l = i & 63, r = l & 15, gg = l >> 4, t = i >> 6;
            uint32_t th[2], tl[2], bh[2], bl[2];
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const int s = 16 * t + 4 * gg + 2 * w, m = r >> 1;
                const float2 q0 = cs[rest(s * m, N2, inv_n2) * N1], q1 = cs[rest((s + 1) * m, N2, inv_n2) * N1];
                split16(r & 1 ? q0.y : q0.x, r & 1 ? q1.y : q1.x, th[w], tl[w]);
                const float2 q = cs[rest((16 * t + r) * (2 * gg + w), N2, inv_n2) * N1];
                split16(q.x, q.y, bh[w], bl[w]);
            }
            f2[i] = mat_u32x4{th[0], th[1], tl[0], tl[1]};
            i1[i] = mat_u32x4{bh[0], bh[1], bl[0], bl[1]};
        }
    }
#pragma clang loop unroll(disable)
    for (int j = tid; j < NT * RB * 128; j += THREADS) {
        const int w = j & 3, i = j >> 2, gg = i & 3, di = (i >> 5) % (RB ? RB : 1) * 8 + (i >> 2 & 7), s = 16 * ((i >> 5) / (RB ? RB : 1)) + 4 * gg + 2 * (w & 1), m = di - sh.dn + N2;
        const float2 q0 = cs[rest(s * m, N2, inv_n2) * N1], q1 = cs[rest((s + 1) * m, N2, inv_n2) * N1];
        uint32_t h, l;
        split16(di < sh.nb && s < N2 ? (w & 2 ? q0.y : q0.x) : 0.f, di < sh.nb && s + 1 < N2 ? (w & 2 ? q1.y : q1.x) : 0.f, h, l);
        uint32_t* to = reinterpret_cast<uint32_t*>(f2) + (i >> 5) * 256 + (j & 127);
        to[0] = h;
        to[128] = l;
    }
#pragma clang loop unroll(disable)
    for (int j = tid; j < (FOLD ? 0 : NT * KS * 256); j += THREADS) {
        const int w = j & 3, l = j >> 2 & 63, ks = (j >> 8) % KS, t = (j >> 8) / KS, s = 16 * t + (l & 15), gg = l >> 4;
        const int di = (32 * ks + 16 * (w >> 1) + 4 * gg + 2 * (w & 1)) >> 1;        // rows 2 di, 2 di + 1
        const float2 q = cs[rest(s * (di - sh.dn + N2), N2, inv_n2) * N1];
        const bool on = di < sh.nb && s < N2;
        uint32_t h, lo;
        split16(on ? q.x : 0.f, on ? -q.y : 0.f, h, lo);
        uint32_t* to = reinterpret_cast<uint32_t*>(i1);
        if constexpr (RB == 1) {                 // high and low parts of two words
            if (w < 2) { to[t * 256 + l * 4 + w] = h; to[t * 256 + l * 4 + 2 + w] = lo; }
        } else {
            to[(t * KS + ks) * 512 + l * 4 + w] = h;
            to[(t * KS + ks) * 512 + 256 + l * 4 + w] = lo;
        }
    }
#pragma clang loop unroll(disable)
    for (int i = tid; i < NT * 256; i += THREADS) {
        const int s = 16 * (i >> 8) + (i & 15), cc = (i >> 4) & 15;
        tw[(i >> 4) * kTwRow + (i & 15)] = s < N2 && cc < N1 ? cs[s * cc] : make_float2(0.f, 0.f);
    }
    // the operands on the side of the N1 places: [re, im of the result][terms]
#pragma clang loop unroll(disable)
    for (int j = tid; j < 512; j += THREADS) {
        const int w = j & 3, l = j >> 2 & 63, o = j >> 8, u = l & 15, a = 4 * (l >> 4) + w;
        double2 q = root[rest(a < N1 && u < N1 ? a * u : 0, N1, inv_n1)];
        if (a >= N1 || u >= N1) q = make_double2(0.0, 0.0);
        uint32_t t0, t1, t2;
        split_bf16(o ? -q.y : q.x, o ? q.x : q.y, t0, t1, t2);
        uint32_t* to = f1t + o * 768 + l * 4 + w;
        to[0] = t0; to[256] = t1; to[512] = t2;
        const int c0 = 4 * (l >> 4) + 2 * (w & 1);           // u is a place here, c0 and c0 + 1 are bins
        const double2 q0 = root[rest(c0 < N1 && u < N1 ? c0 * u : 0, N1, inv_n1)], q1 = root[rest(c0 + 1 < N1 && u < N1 ? (c0 + 1) * u : 0, N1, inv_n1)];
        const bool sine = (w >> 1) != o;
        const float sign = sine && !o ? -1.f : 1.f;
        const float v0 = c0 < N1 && u < N1 ? sign * (float)(sine ? q0.y : q0.x) : 0.f, v1 = c0 + 1 < N1 && u < N1 ? sign * (float)(sine ? q1.y : q1.x) : 0.f;
        split16(v0, v1, t0, t1);
        to = i2t + o * 512 + l * 4 + w;
        to[0] = t0; to[256] = t1;
    }
    float weight[NA][2];                         // FOLD: M[j] + M[-j], M[j] - M[-j] of a lane's two multiples
    if constexpr (FOLD) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int j = 2 * g + e;
            auto at = [&](int k) {
                const int f = k < 0 ? -k : k;
                return c < N1 && f <= sigma && 2 * k != -N ? gm[f <= sigma ? f : 0] : 0.f;
            };
            const float up = at(c + N1 * j), down = j ? at(c - N1 * j) : 0.f;
            weight[0][e] = up + down;
            weight[NA - 1][e] = j ? up - down : 0.f;
        }
    }
#pragma unroll
    for (int rt = 0; rt < RB; ++rt)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int di = (rt * 16 + 4 * g + 2 * e) >> 1, k = c + N1 * (di - sh.dn), f = k < 0 ? -k : k;
            weight[rt][e] = c < N1 && di < sh.nb && f <= sigma && 2 * k != -N ? gm[f] : 0.f;
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
    landed(chunks > 1);
    __syncthreads();

    // this lane's words: places 4 g .. + 3 of subsequence c of a tile, channel pairs 4 wave .. + 3 of a group
    const lds_word* words = (const lds_word*)reinterpret_cast<const uint32_t*>(data) + ((4 * g) * 16 + c) * 32 + (wave ^ (c >> 1)) * 4;
    const int f2_at = ((c >> 1) * 4 + g) * 2, ro = c & 1;        // in 8-byte units: a row's cosines and sines, in either order
    const uint32_t f2_sign = ro ? 0x80008000u : 0u;
    int ci = 0;
    for (int grp = 0; grp < groups; ++grp) {
        mat_f32x4 acc[P][NA];
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int rt = 0; rt < NA; ++rt) acc[p][rt] = mat_f32x4{0.f, 0.f, 0.f, 0.f};
        MatScale scale;
        for (int t = 0; t < NT; ++t, ++ci) {
            const lds_word* buf = words + (ci % 3) * (kBuf * 4);
            mat_f32x4 T[P][2];                   // subsequence 4 g + v of the tile
            const float2* twiddles = tw + (t * 16 + c) * kTwRow + 4 * g;
            const float m = places_to_bins(T, buf, f1, twiddles, scale.f);
            if (wave < WAVES / 2 && ci + 2 < chunks) issue(ci + 2);
            if (__any(m > (scale.unset ? 0.f : 32768.f))) {
                const float f = into_range(T, m, buf, f1, twiddles, scale);
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int rt = 0; rt < NA; ++rt) acc[p][rt] *= f;
            }
            if constexpr (FOLD) {
                // as in spu_fold: high and low parts of four subsequences are the eight values of K
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
                const mat_u32x4 k = f2[t * 64 + lane], ah{k[0], k[1], k[0], k[1]}, al{k[2], k[3], k[2], k[3]};
#pragma unroll
                for (int o = 0; o < 2; ++o)
#pragma unroll
                    for (int p = 0; p < P; ++p) acc[p][o] = mac_f16(acc[p][o], al, tv[p][o]);
#pragma unroll
                for (int o = 0; o < 2; ++o)
#pragma unroll
                    for (int p = 0; p < P; ++p) acc[p][o] = mac_f16(acc[p][o], ah, tv[p][o]);
                landed(ci + 2 < chunks);
                __syncthreads();
                continue;
            }
            mat_u32x4 th[P], tl[P];
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    uint32_t h, l;
                    split16(T[p][w >> 1][2 * (w & 1)], T[p][w >> 1][2 * (w & 1) + 1], h, l);
                    th[p][w] = h; tl[p][w] = l;
                }
            // subsequences -> rows of the band
#pragma unroll
            for (int rt = 0; rt < RB; ++rt) {
                mat_u32x4 ah, al;
                {
                    const uint2* at = reinterpret_cast<const uint2*>(f2 + (t * RB + rt) * 64) + f2_at;
                    const uint2 h0 = at[ro], h1 = at[1 - ro], l0 = at[64 + ro], l1 = at[65 - ro];
                    ah = mat_u32x4{h0.x ^ f2_sign, h0.y ^ f2_sign, h1.x, h1.y};
                    al = mat_u32x4{l0.x ^ f2_sign, l0.y ^ f2_sign, l1.x, l1.y};
                }
#pragma unroll
                for (int p = 0; p < P; ++p) acc[p][rt] = mac_f16(acc[p][rt], ah, tl[p]);
#pragma unroll
                for (int p = 0; p < P; ++p) acc[p][rt] = mac_f16(acc[p][rt], al, th[p]);
#pragma unroll
                for (int p = 0; p < P; ++p) acc[p][rt] = mac_f16(acc[p][rt], ah, th[p]);
            }
            landed(ci + 2 < chunks);
            __syncthreads();
        }
        // ---- mask, scaled for the way back
        mat_u32x4 gh[P][KS], gl[P][KS];          // FOLD: the real and the imaginary part's, high and low parts in one
        float back;
        {
            const bool live = (grp0 + grp) * kMatWidth + 8 * wave < D;          // channels come in eights
            float m = 0.f;
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int rt = 0; rt < NA; ++rt)
#pragma unroll
                    for (int e = 0; e < 2; ++e) m = fmaxf(fmaxf(m, fabsf(acc[p][rt][2 * e])), fabsf(acc[p][rt][2 * e + 1]));
            m = wave_max(m) * (FOLD ? 4.f : 1.f) * (float)sh.inv_N;         // no weight is larger than 1 / N; folded values are of four
            const int by = clampi(9 - exponent(m), -120, 120);
            const float f = m > 0.f && live ? pow2(by) : 0.f;
            back = pow2(clampi(-(scale.e + by), -126, 126));
            float wf[NA][2];
#pragma unroll
            for (int rt = 0; rt < NA; ++rt) { wf[rt][0] = weight[rt][0] * f; wf[rt][1] = weight[rt][1] * f; }
            if constexpr (FOLD) {
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        const mat_f32x4 &r = acc[p][0], &i = acc[p][NA - 1];
                        const int e = 2 * w;
                        const float gp = wf[0][w], gn = wf[NA - 1][w];
                        uint32_t h, l;
                        split16(fmaf(gp, r[e], gn * i[e + 1]), fmaf(gp, r[e + 1], -gn * i[e]), h, l);
                        gh[p][0][w] = h; gh[p][0][2 + w] = l;
                        split16(fmaf(gp, i[e], -gn * r[e + 1]), fmaf(gn, r[e], gp * i[e + 1]), h, l);
                        gl[p][0][w] = h; gl[p][0][2 + w] = l;
                    }
            }
#pragma unroll
            for (int p = 0; p < (FOLD ? 0 : P); ++p)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const int rt = 2 * ks + (w >> 1), v = 2 * (w & 1);
                        uint32_t h = 0, l = 0;
                        if (rt < RB) split16(acc[p][rt < NA ? rt : 0][v] * wf[rt < NA ? rt : 0][w & 1], acc[p][rt < NA ? rt : 0][v + 1] * wf[rt < NA ? rt : 0][w & 1], h, l);
                        gh[p][ks][w] = h; gl[p][ks][w] = l;
                    }
            if constexpr (RB == 1) {
#pragma unroll
                for (int p = 0; p < P; ++p) { gh[p][0][2] = gl[p][0][0]; gh[p][0][3] = gl[p][0][1]; }
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
            for (int v = 0; v < 4; ++v) { const float2 q = tw[(t * 16 + 4 * g + v) * kTwRow + c]; wc[v] = q.x; ws[v] = q.y; }
            mat_f32x4 z[P][2];
#pragma unroll
            for (int o = 0; o < 2; ++o) {
#pragma unroll
                for (int p = 0; p < P; ++p) z[p][o] = mat_f32x4{0.f, 0.f, 0.f, 0.f};
                // the operand of the imaginary part: (cos, -sin) -> (sin, cos)
                auto turn = [&](const mat_u32x4& k) {
                    mat_u32x4 r;
#pragma unroll
                    for (int w = 0; w < 4; ++w) r[w] = o ? __builtin_amdgcn_alignbit(k[w], k[w], 16) ^ 0x8000u : k[w];
                    return r;
                };
                if constexpr (FOLD) {
                    const mat_u32x4 k = i1[t * 64 + lane], kh{k[0], k[1], k[0], k[1]}, kl{k[2], k[3], k[2], k[3]};
#pragma unroll
                    for (int p = 0; p < P; ++p) z[p][o] = mac_f16(z[p][o], o ? gl[p][0] : gh[p][0], kl);
#pragma unroll
                    for (int p = 0; p < P; ++p) z[p][o] = mac_f16(z[p][o], o ? gl[p][0] : gh[p][0], kh);
                } else if constexpr (RB == 1) {
                    const mat_u32x4 k = turn(i1[t * 64 + lane]);
                    const mat_u32x4 kh{k[0], k[1], k[0], k[1]}, kl{k[2], k[3], 0u, 0u};
#pragma unroll
                    for (int p = 0; p < P; ++p) z[p][o] = mac_f16(z[p][o], gh[p][0], kl);
#pragma unroll
                    for (int p = 0; p < P; ++p) z[p][o] = mac_f16(z[p][o], gh[p][0], kh);
                } else {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        const mat_u32x4 kh = turn(i1[((t * KS + ks) * 2 + 0) * 64 + lane]), kl = turn(i1[((t * KS + ks) * 2 + 1) * 64 + lane]);
#pragma unroll
                        for (int p = 0; p < P; ++p) z[p][o] = mac_f16(z[p][o], gl[p][ks], kh);
#pragma unroll
                        for (int p = 0; p < P; ++p) z[p][o] = mac_f16(z[p][o], gh[p][ks], kl);
#pragma unroll
                        for (int p = 0; p < P; ++p) z[p][o] = mac_f16(z[p][o], gh[p][ks], kh);
                    }
                }
            }
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
        landed(false);
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
        tile_store(pout + n, (float)q);
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
            const double f = (double)(float)v, h = half(f);
            return h + half(f - h);
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

// The rounded constants make every score too small or too large by up to 5e-8, in a way that depends on N1 and N2 alone: the
// rows of the band on the way there and back, and the N1 places.  The matrix cores' sums, which are cut off rather than
// rounded, take another `sums`.
double mat_length(const MatShape& sh, double sums)
{
    static const CircleLengths circle;
    double band = 0.0, places = 0.0;
    for (int i = 0; i < sh.nb; ++i) band += circle.of[sh.N2 / std::gcd(sh.N2, std::abs(i - sh.dn))];
    for (int i = 0; i < sh.N1; ++i) places += circle.of[sh.N1 / std::gcd(sh.N1, i)];
    return 1.0 - 2.0 * band / sh.nb - places / sh.N1 + sums;
}

namespace {

bool mat_shape(int N, int sigma, MatShape* sh, int* rb)
{
    int best = 0;
    double best_cost = 0.0;
    for (int N1 = 16; N1 >= 9; --N1) {
        if (N % N1) continue;
        const int N2 = N / N1, NT = (N2 + 15) / 16, dn = (sigma + N1 - 1) / N1, nb = dn + sigma / N1 + 1, RB = (nb + 7) / 8;
        if (NT > kMatTiles || RB > 4 || N2 < 2) continue;
        const double cost = NT * (12.0 + 3 * RB + (RB == 1 ? 4 : 6 * ((RB + 1) / 2)));
        if (best && cost >= best_cost) continue;
        best = N1;
        best_cost = cost;
        *sh = MatShape{1.0 / N, 1.0 / (N - 1), 1.0 / N1, 1.0, N, N1, N2, NT, sigma, dn, nb};
        *rb = RB;
    }
    return best != 0;
}
size_t mat_lds(const MatShape& sh, int RB, int gpw)
{
    const int KS = (RB + 1) / 2, kI1 = RB <= 1 ? 1 : 2 * KS;
    return (size_t)3 * 256 * (kMatWidth * 2) + (size_t)sh.NT * ((RB ? RB : 1) + kI1) * 1024 + (size_t)sh.NT * 16 * kTwRow * 8 + (gpw > 1 ? (size_t)kMatWaves * sh.NT * 1024 : 0);
}

}  // namespace

bool spu_mat_supported(int N, int sigma)
{
    MatShape sh;
    int rb;
    return mat_shape(N, sigma, &sh, &rb) && mat_lds(sh, rb, 1) <= kMatLds;
}

static int mat_groups(int D) { return (D + kMatWidth - 1) / kMatWidth; }

// How the samples of a launch are split: as few groups of channels to a workgroup as leave each compute unit one workgroup, or one
// group where the energies of several do not fit beside the tokens
MatPlan spu_mat_plan(const MatRun* runs, int n, int D)
{
    MatPlan p{};
    int lds_groups = 0;
    bool folds = true;                           // one block of folded rows holds the bands
    for (int i = 0; i < n; ++i) {
        MatShape sh;
        int rb;
        mat_shape(runs[i].N, runs[i].sigma, &sh, &rb);
        p.rb = std::max(p.rb, rb);
        folds = folds && sh.dn <= 7;
        p.samples += runs[i].count;
        p.ld = std::max(p.ld, (runs[i].N + 3) / 4 * 4);
    }
    if (p.rb == 2 && folds) p.rb = 0;            // 20 products for 24
    for (int i = 0; i < n; ++i) {
        MatShape sh;
        int rb;
        mat_shape(runs[i].N, runs[i].sigma, &sh, &rb);
        p.lds = std::max(p.lds, mat_lds(sh, p.rb, 1));
        lds_groups = std::max(lds_groups, (int)mat_lds(sh, p.rb, 2));
    }
    const int groups = mat_groups(D);
    p.gpw = (int)((p.samples * groups + 255) / 256);
    if (p.gpw > 1 && (size_t)lds_groups > kMatLds) p.gpw = 1;
    if (p.gpw > 1) p.lds = (size_t)lds_groups;
    p.n_tiles = (groups + p.gpw - 1) / p.gpw;
    return p;
}

// us of one call, from measurements: the rounds that the workgroups take on the chip, one per compute unit, each with its tables
// and its hand-over.  bf16 8x1024x3584, sigma = 102: 36.4, 32x390x3584, 58: 48, 32x576x896, 57: 24, 16x1536x1536, 153: 61,
// 4x234x1536, 17: 13, 1x1280x896, 32: 21.
static double mat_tile_us(const MatShape& sh, int rb) { return sh.NT * (2.5 + 0.5 * rb); }
double spu_mat_us(int B, int N, int D, int sigma)
{
    MatShape sh;
    int rb;
    mat_shape(N, sigma, &sh, &rb);
    const MatRun run{N, sigma, B, 0};
    const MatPlan p = spu_mat_plan(&run, 1, D);
    return 3.0 + (p.n_tiles > kMatDirect ? 2.0 : 0.0) + (double)(((int64_t)B * p.n_tiles + 255) / 256) * (4.5 + p.gpw * mat_tile_us(sh, rb));
}
// what a run adds to a launch that several share; 0: it does not go there
double spu_mat_work_us(int B, int N, int D, int sigma)
{
    MatShape sh;
    int rb;
    if (!mat_shape(N, sigma, &sh, &rb) || rb > 2 || mat_lds(sh, 2, 1) > kMatLds) return 0.0;
    return (double)B * mat_groups(D) / 256.0 * mat_tile_us(sh, 2);
}

template <int RB, int RUNS>
static void mat_launch(const void* x, const MatRun* runs, int n, const MatPlan& p, int D, int64_t row_stride, int use_hamming,
                       float* partial, float* gpartial, const TileSync& sy, float* scores, hipStream_t st)
{
    MatLaunch<RUNS> l;
    l.n = n;
    int64_t samples = 0;
    for (int i = 0; i < n; ++i) {
        int rb;
        mat_shape(runs[i].N, runs[i].sigma, &l.run[i].sh, &rb);
        l.run[i].sh.length = mat_length(l.run[i].sh, RB ? 2.4e-8 : 0.5e-8);         // measured, 576 to 2048 tokens, white and smooth
        l.run[i].wg0 = (int)(samples * p.n_tiles);
        l.run[i].sample0 = (int)samples;
        l.run[i].tok0 = runs[i].tok0;
        samples += runs[i].count;
    }
    LUVC_LAUNCH("spu_mat", (spu_mat<RB, RUNS>), dim3((unsigned)(samples * p.n_tiles)), dim3(64 * kMatWaves), p.lds, st, (const bf16_t*)x, l, D, row_stride, use_hamming,
                p.gpw, p.n_tiles, partial, gpartial, sy, p.ld, scores);
}

luvc_status spu_score_mat(const void* x, const MatRun* runs, int n, const MatPlan& p, int D, int64_t row_stride, int use_hamming,
                          float* partial, float* gpartial, const TileSync& sy, float* scores, hipStream_t st)
{
#define LUVC_MAT(RB, RUNS) mat_launch<RB, RUNS>(x, runs, n, p, D, row_stride, use_hamming, partial, gpartial, sy, scores, st)
    if (n > 1) {
        if (p.rb == 0) LUVC_MAT(0, kMatMaxRuns);
        else if (p.rb == 1) LUVC_MAT(1, kMatMaxRuns);
        else LUVC_MAT(2, kMatMaxRuns);
    }
    else if (p.rb == 0) LUVC_MAT(0, 1);
    else if (p.rb == 1) LUVC_MAT(1, 1);
    else if (p.rb == 2) LUVC_MAT(2, 1);
    else if (p.rb == 3) LUVC_MAT(3, 1);
    else LUVC_MAT(4, 1);
#undef LUVC_MAT
    return check_launch("spu score (mat)");
}

}  // namespace luvc
