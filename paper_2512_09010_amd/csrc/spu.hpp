// Internal interface between the C-ABI layer and the SPU kernels.
#pragma once
#include "common.hpp"

namespace luvc {

constexpr int kSpuMaxN = 32768;     // tokens per sample (twiddle index arithmetic stays in int32)

// Which kernels serve a score call (chosen from the sizes and the alignment of the rows)
enum class SpuPath {
    Circ,       // spu_circ: the filter as a circulant matrix on the matrix cores, short samples
    Fft,        // spu_fft16q: transform decomposition, N = 16 Q N2
    Mat,        // spu_mat: two transforms on the matrix cores, N = N1 N2 with a factor N1 in 9 .. 16
    Fold,       // spu_fold: the same for wide pass bands and up to 4096 tokens
    Conv,       // spu_conv: M-point transforms in one workgroup, any N up to 8192
    Dense       // direct pass-band DFT through the workspace, any N
};

// How spu_circ reads the rows of a call: channel pairs in one access, channel by channel, or not at all (strides too large)
enum class CircRows { None, Single, Paired };
// What the rows of a call allow: the kernels that need more than single elements
struct SpuRows {
    CircRows circ;
    bool pieces;                     // bf16 rows in aligned 16-byte pieces
};
SpuRows spu_rows(const void* x, int D, int64_t row_stride, luvc_dtype dt);

// Offsets (bytes) of the score kernels' scratch inside the caller's workspace.
struct SpuLayout {
    size_t tw, gk, gm, Fc, Fs, spec, partial, gpartial, arrive, bytes;
    int n_tiles;
    SpuPath path;
};
SpuLayout spu_layout(int B, int N, int D, int sigma, luvc_dtype dt, SpuRows rows, size_t most);
size_t spu_workspace(int B, int N, int D, int sigma, luvc_dtype dt, size_t most = SIZE_MAX);
// us of a run: on its own, and what its products add to a spu_circ launch that several share
double spu_alone_us(int B, int N, int D, int sigma, luvc_dtype dt, bool pieces);
double spu_circ_work_us(int64_t B, int N, int D, luvc_dtype dt);

luvc_status spu_score_dense(const void* x, int B, int N, int D, int64_t row_stride, luvc_dtype dt, int sigma,
                            int use_hamming, float* scores, void* workspace, size_t most, hipStream_t st);
// luvc_spu_score behind its entry points; most: the layout has to fit so much scratch (SIZE_MAX: the quickest one)
luvc_status spu_score_call(const void* x, int B, int N, int D, int64_t row_stride, luvc_dtype dtype, int sigma, int use_hamming,
                           float* scores, void* workspace, size_t workspace_bytes, size_t most, void* hip_stream);

// Fast path (spu_fft.hip): N = 16 * Q * N2 with Q in {16, 15, 9}, 2 * sigma + 1 <= 16 * Q, N <= 4096.
bool spu_fft_supported(int N, int sigma);
double spu_fft_us(int B, int N, int D, int sigma);
double spu_fft_measured_us(int B, int N, int D, int sigma);
struct TileSync;
luvc_status spu_score_fft(const void* x, int B, int N, int D, int64_t row_stride, luvc_dtype dt, int sigma, int use_hamming,
                          float* partial, float* gpartial, const TileSync& sy, int n_tiles, float* scores, hipStream_t st);

// Samples of N = N1 N2 tokens on the matrix cores (spu_mat.hip), runs of equal samples in one launch
constexpr int kMatMaxRuns = 16;
struct MatRun {
    int N, sigma, count;
    int64_t tok0;                    // first token of the first sample
};
struct MatPlan {
    int gpw, n_tiles, ld;
    bool fold;
    int64_t samples;
    size_t lds;
};
bool spu_mat_supported(int N, int sigma);
MatPlan spu_mat_plan(const MatRun* runs, int n, int D);
double spu_mat_us(int B, int N, int D, int sigma);
double spu_mat_work_us(int B, int N, int D, int sigma);
luvc_status spu_score_mat(const void* x, const MatRun* runs, int n, const MatPlan& p, int D, int64_t row_stride, int use_hamming,
                          float* partial, float* gpartial, const TileSync& sy, float* scores, hipStream_t st);
// a launch that several runs share: scratch, and the launch on it
size_t spu_mat_bytes(const MatRun* runs, int n, int D);
luvc_status spu_score_mat_runs(const void* x, const MatRun* runs, int n, int D, int64_t row_stride, int use_hamming, float* scores, void* workspace, hipStream_t st);

// One launch of equal samples, up to 4096 tokens (spu_fold.hip); the workspace is that of spu_fold_tiles(D) tiles
int spu_fold_blocks(int N, int sigma);          // of 16 rows of the band; 0: not here
int spu_fold_tiles(int D);
double spu_fold_us(int B, int N, int D, int sigma);
luvc_status spu_score_fold(const void* x, int B, int N, int D, int64_t row_stride, int sigma, int use_hamming,
                           float* partial, float* gpartial, const TileSync& sy, float* scores, hipStream_t st);

// Short samples on the matrix cores (spu_circ.hip), runs of equal samples in one launch
constexpr int kCircMaxN = 1024, kCircMaxRuns = 64;
struct CircRun {
    int group0, N, sigma, count;     // first group of output tokens (filled in by the launcher)
    int64_t tok0;                    // first token of the first sample
};
struct CircRuns { int n; CircRun run[kCircMaxRuns]; };
CircRows spu_circ_rows(const void* x, int D, int64_t row_stride, luvc_dtype dt);
size_t spu_circ_bytes(int64_t samples, int N, int D);
luvc_status spu_score_circ(const void* x, int64_t row_stride, int D, luvc_dtype dt, int use_hamming, CircRuns& runs, void* words, float* scores, hipStream_t st);

// Any N (spu_conv.hip): N <= 8192, or N = 16384
int spu_conv_points(int N, bool* half);
int spu_conv_tiles(int B, int N, int D, int most = INT32_MAX);
double spu_conv_us(int B, int N, int D, luvc_dtype dt);
double spu_conv_measured_us(int B, int N, int D);
size_t spu_conv_spec_bytes(int N);
inline int spu_conv_ld(int N) { return (N + 3) / 4 * 4; }
luvc_status spu_score_conv(const void* x, int B, int N, int D, int64_t row_stride, luvc_dtype dt, int sigma, int use_hamming,
                           float* spec, float* partial, float* gpartial, const TileSync& sy, int n_tiles, float* scores, hipStream_t st);

// Runs of equal samples, packed one after the other, pruned together
constexpr int kPruneMaxRuns = 64;
struct PruneRun {
    int wg0, N, n_keep, count;       // first workgroup (filled in by the launcher)
    int64_t tok_in, tok_out;         // first token of the first sample, in and out
};
struct PruneRuns { int n; PruneRun run[kPruneMaxRuns]; };
luvc_status spu_prune_run(const void* x, const float* scores, int D, int64_t row_stride, luvc_dtype dt, PruneRuns& runs,
                          int32_t* kept_idx, void* x_out, const int32_t* origin_in, int32_t* origin_out, hipStream_t st);

}  // namespace luvc
