// SPU score (paper Section 3.3, Eq. 4-8): direct pass-band DFT path, valid for any N.
//
// The mask of Eq. 5 is real and symmetric in k, so for a real signal x[n] the filtered signal is
//     x'[n] = sum_{k=0..sigma} g_k ( C_k cos(2 pi k n / N) + S_k sin(2 pi k n / N) ),
//     C_k = sum_n x[n] cos(2 pi k n / N),  S_k = sum_n x[n] sin(2 pi k n / N),
//     g_0 = M[0]/N,  g_k = 2 M[k]/N  (g_k = M[k]/N when 2k = N, the self-mirrored bin),
// i.e. Eq. 4 evaluated on the pass-band bins only (all other bins are multiplied by zero in Eq. 6)
// and Eq. 7 with the +k / -k terms paired.  Lanes of a wavefront are channels, so twiddles are
// wave-uniform and come through the scalar path; token rows are read coalesced.
//
//   spu_tables      twiddles (fp64 sincospi rounded to fp32) and the weights g_k
//   spu_fwd_dense   C_k, S_k for a tile of 64 channels and a group of bins
//   spu_inv_dense   x'[n] for a tile of 64 channels and a chunk of tokens, squared and summed over the tile
//   spu_finish      fixed-order sum over channel tiles, square root (Eq. 8)
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <random>

#include "common.hpp"
#include "spu.hpp"
#include "spu_tiles.hpp"

namespace luvc {

__global__ void __launch_bounds__(256)
spu_tables(int N, int sigma, int use_hamming, float2* __restrict__ tw, float* __restrict__ gk, float* __restrict__ gm)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) {
        double s, c;
        sincospi(2.0 * (double)i / (double)N, &s, &c);
        tw[i] = make_float2((float)c, (float)s);
    }
    if (i <= sigma) {
        double w = 1.0;
        if (use_hamming && N > 1) w = 0.54 + 0.46 * cospi(2.0 * (double)i / (double)(N - 1));
        const double pair = (i == 0 || 2 * i == N) ? 1.0 : 2.0;
        gk[i] = (float)(pair * w / (double)N);     // +k and -k paired (real-signal form)
        gm[i] = (float)(w / (double)N);            // per bin (complex form)
    }
}

constexpr int kKPW = 8;    // bins per wavefront in the forward kernel
constexpr int kNB = 8;     // tokens per register block in the inverse kernel
constexpr int kNChunk = 128;  // tokens per workgroup in the inverse kernel (4 waves x 4 blocks x kNB)

template <typename T>
__global__ void __launch_bounds__(256)
spu_fwd_dense(const T* __restrict__ x, int N, int D, int64_t row_stride, int sigma,
              const float2* __restrict__ tw, float* __restrict__ Fc, float* __restrict__ Fs)
{
    using tr = io_traits<T>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int d = blockIdx.x * 64 + lane;
    const int b = blockIdx.z;
    const int k0 = (blockIdx.y * 4 + wave) * kKPW;
    if (k0 > sigma) return;
    const bool live = d < D;
    const T* xb = x + (int64_t)b * N * row_stride + (live ? d : 0);
    float ac[kKPW], as[kKPW];
    int idx[kKPW], kstep[kKPW];
#pragma unroll
    for (int j = 0; j < kKPW; ++j) { ac[j] = 0.f; as[j] = 0.f; idx[j] = 0; kstep[j] = (k0 + j <= sigma) ? k0 + j : 0; }
    for (int n = 0; n < N; ++n) {
        const float xv = live ? tr::load(xb + (int64_t)n * row_stride) : 0.f;
#pragma unroll
        for (int j = 0; j < kKPW; ++j) {
            const float2 t = tw[idx[j]];
            ac[j] = fmaf(xv, t.x, ac[j]);
            as[j] = fmaf(xv, t.y, as[j]);
            idx[j] += kstep[j];                    // (k * n) mod N, kept incrementally (k <= sigma < N)
            if (idx[j] >= N) idx[j] -= N;
        }
    }
    if (!live) return;
#pragma unroll
    for (int j = 0; j < kKPW; ++j) {
        const int k = k0 + j;
        if (k <= sigma) {
            Fc[((int64_t)b * (sigma + 1) + k) * D + d] = ac[j];
            Fs[((int64_t)b * (sigma + 1) + k) * D + d] = as[j];
        }
    }
}

__global__ void __launch_bounds__(256)
spu_inv_dense(const float* __restrict__ Fc, const float* __restrict__ Fs, int N, int D, int sigma,
              const float2* __restrict__ tw, const float* __restrict__ gk,
              float* __restrict__ partial /* [B, n_tiles, N] */)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = blockIdx.x, n_tiles = gridDim.x;
    const int d = tile * 64 + lane;
    const int b = blockIdx.z;
    const bool live = d < D;
    const float* fc = Fc + (int64_t)b * (sigma + 1) * D + (live ? d : 0);
    const float* fs = Fs + (int64_t)b * (sigma + 1) * D + (live ? d : 0);
    for (int blk = 0; blk < kNChunk / (4 * kNB); ++blk) {
        const int n0 = blockIdx.y * kNChunk + (blk * 4 + wave) * kNB;
        if (n0 >= N) break;
        float acc[kNB];
        int idx[kNB], stepn[kNB];
#pragma unroll
        for (int j = 0; j < kNB; ++j) { acc[j] = 0.f; idx[j] = 0; stepn[j] = (n0 + j) % N; }
        for (int k = 0; k <= sigma; ++k) {
            const float g = gk[k];
            const float c = live ? g * fc[(int64_t)k * D] : 0.f;
            const float s = live ? g * fs[(int64_t)k * D] : 0.f;
#pragma unroll
            for (int j = 0; j < kNB; ++j) {
                const float2 t = tw[idx[j]];
                acc[j] = fmaf(c, t.x, acc[j]);
                acc[j] = fmaf(s, t.y, acc[j]);
                idx[j] += stepn[j];                // (k * n) mod N
                if (idx[j] >= N) idx[j] -= N;
            }
        }
#pragma unroll
        for (int j = 0; j < kNB; ++j) {
            const float e = wave_sum(acc[j] * acc[j]);
            if (lane == 0 && n0 + j < N) partial[((int64_t)b * n_tiles + tile) * N + n0 + j] = e;
        }
    }
}

// Eq. 8: fixed-order sum of the per-tile energies, then the square root.  A workgroup owns 64
// consecutive tokens; its 8 waves split the channel tiles, partial sums meet in LDS in wave order.
constexpr int kFinParts = 8;
__global__ void __launch_bounds__(64 * kFinParts)
spu_finish(const float* __restrict__ partial, int N, int n_tiles, int64_t total, float* __restrict__ scores)
{
    __shared__ double part_sum[kFinParts][64];
    const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    double e = 0.0;
    if (i < total) {
        const int64_t b = i / N;
        const int n = (int)(i - b * N);
        for (int t = part; t < n_tiles; t += kFinParts) e += (double)partial[(b * n_tiles + t) * N + n];
    }
    part_sum[part][lane] = e;
    __syncthreads();
    if (part == 0 && i < total) {
        double tot = 0.0;
#pragma unroll
        for (int p = 0; p < kFinParts; ++p) tot += part_sum[p][lane];
        scores[i] = (float)sqrt(tot);
    }
}

// Tags of the arrival words (spu_tiles.hpp): one per launch, from a process-wide sequence that starts at a random
// 48-bit value, so that whatever a workspace held before cannot pass for a word of this launch.  Never zero.
tile_tag_t spu_next_tag()
{
    static std::atomic<unsigned long long> next{[] {
        unsigned long long r = 0;
        try {
            std::random_device rd;
            r = ((unsigned long long)rd() << 32) ^ (unsigned long long)rd();
        } catch (...) {                                    // no entropy source: the clock and an address will have to do
            r = (unsigned long long)(uintptr_t)&r;
        }
        const unsigned long long t = (unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count();
        return r ^ (t * 0x9E3779B97F4A7C15ull);
    }()};
    for (;;) {
        const tile_tag_t tag = next.fetch_add(1, std::memory_order_relaxed) & 0xffffffffffffull;
        if (tag) return tag;
    }
}

// ------------------------------------------------------------------ host side
// Which kernel serves a call, from times (us, one call) as functions of the sizes.  spu_circ: its products at 1.1e15 flop/s, and a
// chain of steps that grows with N, which overlap in part (fitted to bf16 8x205x3584: 14, 1x729x3584: 20, 1x1000x1024: 16,
// 4x861x1408: 34; fp32 1x300x2048: 13, 1x1000x1024: 29; channel by channel 8x205x3585: 16, 1x729x3585: 27; since its taps are ready
// earlier it takes .5 to 2 us less); the others beside their launchers.
double spu_circ_work_us(int64_t B, int N, int D, luvc_dtype dt) { return (dt == LUVC_F32 ? 12.0 : 6.0) * N * N * (double)D * (double)B / 1.1e9; }
static double circ_us(int64_t B, int N, int D, luvc_dtype dt, CircRows rows)
{
    const double work = 1.15 * spu_circ_work_us(B, N, D, dt), chain = (dt == LUVC_F32 ? 0.0218 : 0.0105) * N;
    return (dt == LUVC_F32 ? 6.3 : 5.5) + (rows == CircRows::Single ? 1.35 : 1.0) * std::sqrt(work * work + chain * chain);
}
// bf16, as measured since (101 shapes of 56 to 1024 tokens, 0.74 to 1.15 of it): large calls take three quarters of the above
static double circ_measured_us(int64_t B, int N, int D)
{
    const double work = 0.94 * spu_circ_work_us(B, N, D, LUVC_BF16), chain = 0.01 * N;
    return 6.5 + std::sqrt(work * work + chain * chain);
}
// The kernels for rows of any kind are weighed against each other with estimates that are those of their first forms; which of them
// a call goes to has stayed as it was, its error with it.
struct SpuChoice { SpuPath path; double us; };
static SpuChoice long_path(int B, int N, int D, int sigma, luvc_dtype dt)
{
    bool half;
    SpuChoice p{SpuPath::Dense, 0.0};
    if (spu_fft_supported(N, sigma)) p = {SpuPath::Fft, spu_fft_us(B, N, D, sigma)};
    if (spu_conv_points(N, &half) != 0) {
        const double us = spu_conv_us(B, N, D, dt);
        if (p.path == SpuPath::Dense || us < p.us) p = {SpuPath::Conv, us};
    }
    return p;
}
static SpuChoice or_circ(const SpuChoice& p, int B, int N, int D, luvc_dtype dt, CircRows rows)
{
    if (rows == CircRows::None || N > kCircMaxN) return p;
    const double us = circ_us(B, N, D, dt, rows);
    return us <= p.us ? SpuChoice{SpuPath::Circ, us} : p;
}
// spu_mat and spu_fold take a call from the kernel that it would go to where they are quicker than that one measures.  On 158 shapes
// of bf16 tokens with every kernel that takes them, drawn over 1 to 32 samples of 49 to 7549 tokens, they take 104 calls in 0.69 of
// the time (one is slower: 4x637x1536, sigma = 35 20.2 for 19.3) and leave two that they would take in 0.95 of it; on 90 more with the two
// sides within a quarter of each other, 42 in 0.85 of the time, none slower, and leave five at 0.91 to 0.97.  spu_fold with two
// blocks of rows takes none from spu_circ, whose scores are the closer ones (rms error 2.9e-8 for 3.1e-8).
static SpuChoice or_products(SpuChoice p, int B, int N, int D, int sigma)
{
    const int blocks = spu_fold_blocks(N, sigma);
    const bool mat = spu_mat_supported(N, sigma), fold = blocks == 1 || (blocks == 2 && p.path != SpuPath::Circ);
    if (p.path == SpuPath::Dense || !(mat || fold)) return p;
    double limit = p.path == SpuPath::Fft ? spu_fft_measured_us(B, N, D, sigma) : p.path == SpuPath::Conv ? spu_conv_measured_us(B, N, D) : circ_measured_us(B, N, D);
    auto offer = [&](SpuPath path, double us) {
        if (us < limit) { p = {path, us}; limit = us; }
    };
    if (mat) offer(SpuPath::Mat, spu_mat_us(B, N, D, sigma));
    if (fold) offer(SpuPath::Fold, spu_fold_us(B, N, D, sigma));
    return p;
}
static SpuChoice spu_choice(int B, int N, int D, int sigma, luvc_dtype dt, SpuRows rows)
{
    const SpuChoice p = or_circ(long_path(B, N, D, sigma, dt), B, N, D, dt, rows.circ);
    return rows.pieces ? or_products(p, B, N, D, sigma) : p;
}
SpuRows spu_rows(const void* x, int D, int64_t row_stride, luvc_dtype dt)
{
    return SpuRows{spu_circ_rows(x, D, row_stride, dt), dt == LUVC_BF16 && D % 8 == 0 && row_stride % 8 == 0 && row_stride < (1 << 19) && (uintptr_t)x % 16 == 0};
}
double spu_alone_us(int B, int N, int D, int sigma, luvc_dtype dt, bool pieces)
{
    return spu_choice(B, N, D, sigma, dt, SpuRows{CircRows::None, pieces}).us;
}

// Energies per tile and group of tiles, arrival words.  Up to kTileGroup tiles have no group level.
static size_t tile_bytes(int B, int n_tiles, size_t ld, SpuLayout* L, size_t off)
{
    const int groups = spu_tile_groups(n_tiles);
    L->partial = off;  off += align_up(sizeof(float) * (size_t)B * n_tiles * ld);
    L->gpartial = off; off += groups > 1 ? align_up(sizeof(float) * (size_t)B * groups * ld) : 0;
    L->arrive = off;   off += align_up(sizeof(tile_tag_t) * (size_t)B * (groups + 1));
    return off;
}

// Of a path.  spu_conv takes fewer workgroups per sample where `most` bytes of scratch ask for it, down to one per 64 channels,
// which is what the direct path's energies take (1 x 8192 x 2048: 256 of them want 8.9 MB, 205 want 7.2).
static SpuLayout layout_of(SpuPath path, int B, int N, int D, int sigma, size_t most)
{
    SpuLayout L{};
    L.path = path;
    if (L.path == SpuPath::Circ) {
        L.n_tiles = 1;
        L.bytes = align_up(spu_circ_bytes(B, N, D));
        return L;
    }
    if (L.path == SpuPath::Mat || L.path == SpuPath::Fold) {
        const MatRun run{N, sigma, B, 0};
        L.n_tiles = L.path == SpuPath::Fold ? spu_fold_tiles(D) : spu_mat_plan(&run, 1, D).n_tiles;
        L.bytes = tile_bytes(B, L.n_tiles, (N + 3) / 4 * 4, &L, 0);
        return L;
    }
    L.n_tiles = L.path == SpuPath::Fft ? (D + 31) / 32 : (D + 63) / 64;
    const bool dense = L.path == SpuPath::Dense;                     // the one path whose tables and spectra do not stay in LDS
    const size_t spec = dense ? (size_t)B * (sigma + 1) * D : 0;     // pass-band spectra
    size_t off = 0;
    L.tw = off;      off += dense ? align_up(sizeof(float2) * (size_t)N) : 0;
    L.gk = off;      off += dense ? align_up(sizeof(float) * (size_t)(sigma + 1)) : 0;
    L.gm = off;      off += dense ? align_up(sizeof(float) * (size_t)(sigma + 1)) : 0;
    L.Fc = off;      off += align_up(sizeof(float) * spec);
    L.Fs = off;      off += align_up(sizeof(float) * spec);
    L.spec = off;
    if (L.path != SpuPath::Conv) {
        L.bytes = tile_bytes(B, L.n_tiles, N, &L, off);
        return L;
    }
    off += align_up(spu_conv_spec_bytes(N));
    const int fewest = L.n_tiles;
    for (int limit = INT32_MAX;;) {
        L.n_tiles = spu_conv_tiles(B, N, D, limit);
        L.bytes = tile_bytes(B, L.n_tiles, spu_conv_ld(N), &L, off);
        if (L.bytes <= most || L.n_tiles <= fewest) return L;
        limit = L.n_tiles - 1;
    }
}

// most: scratch the call has to do with; a layout that needs more is returned where nothing smaller serves the call.  Short samples then
// go to the kernels of long ones, and what spu_mat or spu_fold would take to the others.
SpuLayout spu_layout(int B, int N, int D, int sigma, luvc_dtype dt, SpuRows rows, size_t most)
{
    const SpuLayout L = layout_of(spu_choice(B, N, D, sigma, dt, rows).path, B, N, D, sigma, most);
    if (L.bytes <= most) return L;
    if (L.path == SpuPath::Circ) return spu_layout(B, N, D, sigma, dt, SpuRows{CircRows::None, rows.pieces}, most);
    if (L.path == SpuPath::Mat || L.path == SpuPath::Fold) return spu_layout(B, N, D, sigma, dt, SpuRows{rows.circ, false}, most);
    return L;
}

// What a call needs whichever way its rows lie: the most of all paths that it may take (for single rows spu_circ is taken where it is
// for pairs, or less)
size_t spu_workspace(int B, int N, int D, int sigma, luvc_dtype dt, size_t most)
{
    const SpuChoice base = long_path(B, N, D, sigma, dt), circ = or_circ(base, B, N, D, dt, CircRows::Paired);
    size_t need = layout_of(base.path, B, N, D, sigma, most).bytes;
    SpuPath seen = base.path;
    auto add = [&](SpuPath path) {
        if (path == base.path || path == seen) return;
        seen = path;
        const size_t bytes = layout_of(path, B, N, D, sigma, most).bytes;
        if (bytes <= most) need = std::max(need, bytes);
    };
    add(circ.path);
    if (dt == LUVC_BF16) {
        add(or_products(base, B, N, D, sigma).path);
        if (circ.path != base.path) add(or_products(circ, B, N, D, sigma).path);
    }
    return need;
}

size_t spu_mat_bytes(const MatRun* runs, int n, int D)
{
    const MatPlan p = spu_mat_plan(runs, n, D);
    SpuLayout L{};
    return tile_bytes((int)p.samples, p.n_tiles, p.ld, &L, 0);
}
luvc_status spu_score_mat_runs(const void* x, const MatRun* runs, int n, int D, int64_t row_stride, int use_hamming, float* scores, void* workspace, hipStream_t st)
{
    const MatPlan p = spu_mat_plan(runs, n, D);
    SpuLayout L{};
    tile_bytes((int)p.samples, p.n_tiles, p.ld, &L, 0);
    char* ws = (char*)workspace;
    TileSync sy;
    sy.arrive = (tile_tag_t*)(ws + L.arrive);
    sy.tag = spu_next_tag();
    return spu_score_mat(x, runs, n, p, D, row_stride, use_hamming, (float*)(ws + L.partial), (float*)(ws + L.gpartial), sy, scores, st);
}

luvc_status spu_score_dense(const void* x, int B, int N, int D, int64_t row_stride, luvc_dtype dt, int sigma,
                            int use_hamming, float* scores, void* workspace, size_t most, hipStream_t st)
{
    const SpuLayout L = spu_layout(B, N, D, sigma, dt, spu_rows(x, D, row_stride, dt), most);
    char* ws = (char*)workspace;
    if (L.path == SpuPath::Circ) {
        CircRuns runs;
        runs.n = 1;
        runs.run[0] = CircRun{0, N, sigma, B, 0};
        return spu_score_circ(x, row_stride, D, dt, use_hamming, runs, workspace, scores, st);
    }
    float2* tw = (float2*)(ws + L.tw);
    float* gk = (float*)(ws + L.gk);
    float* gm = (float*)(ws + L.gm);
    float* Fc = (float*)(ws + L.Fc);
    float* Fs = (float*)(ws + L.Fs);
    float* partial = (float*)(ws + L.partial);
    float* gpartial = (float*)(ws + L.gpartial);
    if (L.n_tiles > 65535) { set_error("D=%d exceeds the supported width", D); return LUVC_ERR_UNSUPPORTED; }
    TileSync sy;
    sy.arrive = (tile_tag_t*)(ws + L.arrive);
    sy.tag = spu_next_tag();
    if (L.path == SpuPath::Fft) return spu_score_fft(x, B, N, D, row_stride, dt, sigma, use_hamming, partial, gpartial, sy, L.n_tiles, scores, st);
    if (L.path == SpuPath::Mat) {
        const MatRun run{N, sigma, B, 0};
        return spu_score_mat(x, &run, 1, spu_mat_plan(&run, 1, D), D, row_stride, use_hamming, partial, gpartial, sy, scores, st);
    }
    if (L.path == SpuPath::Fold) return spu_score_fold(x, B, N, D, row_stride, sigma, use_hamming, partial, gpartial, sy, scores, st);
    if (L.path == SpuPath::Conv)
        return spu_score_conv(x, B, N, D, row_stride, dt, sigma, use_hamming, (float*)(ws + L.spec), partial, gpartial, sy, L.n_tiles, scores, st);
    LUVC_LAUNCH("spu_tables", spu_tables, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, N, sigma, use_hamming, tw, gk, gm);
    const int64_t total = (int64_t)B * N;
    const dim3 gf((unsigned)L.n_tiles, (unsigned)((sigma + 1 + 4 * kKPW - 1) / (4 * kKPW)), (unsigned)B);
    if (dt == LUVC_F32)
        LUVC_LAUNCH("spu_fwd_dense", (spu_fwd_dense<float>), gf, dim3(256), 0, st, (const float*)x, N, D, row_stride, sigma, tw, Fc, Fs);
    else
        LUVC_LAUNCH("spu_fwd_dense", (spu_fwd_dense<bf16_t>), gf, dim3(256), 0, st, (const bf16_t*)x, N, D, row_stride, sigma, tw, Fc, Fs);
    const dim3 gi((unsigned)L.n_tiles, (unsigned)((N + kNChunk - 1) / kNChunk), (unsigned)B);
    LUVC_LAUNCH("spu_inv_dense", spu_inv_dense, gi, dim3(256), 0, st, Fc, Fs, N, D, sigma, tw, gk, partial);
    LUVC_LAUNCH("spu_finish", spu_finish, dim3((unsigned)((total + 63) / 64)), dim3(64 * kFinParts), 0, st, partial, N, L.n_tiles, total, scores);
    return check_launch("spu score");
}

}  // namespace luvc
