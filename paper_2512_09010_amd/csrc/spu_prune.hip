// SPU prune (paper Algorithm 2, last two steps): order-preserving top-k keep and gather.
//
//   spu_select   samples of more than 8192 tokens, one workgroup each.  Scores are mapped to unsigned keys whose integer order
//                is the float order; a most-significant-digit radix select (4 passes of 8 bits,
//                histogram in LDS) finds the key T of the n_keep-th largest score and how many
//                tokens with key == T still belong to the keep set; a stable block-wide compaction
//                then emits, in ascending index order, every token with key > T and the first of
//                those with key == T (equal scores: the lower index wins).
//   spu_gather   one wavefront per kept token copies the ORIGINAL row.
#include <type_traits>

#include "common.hpp"
#include "spu.hpp"

namespace luvc {

__device__ __forceinline__ uint32_t score_key(float s)
{
    uint32_t u = __float_as_uint(s);
    if (u == 0x80000000u) u = 0;                      // -0 and +0 compare equal
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// inclusive prefix sum over the 64 lanes without the LDS crossbar: shifts inside each row of 16 lanes, then the
// last lane of rows 0 / 2 into rows 1 / 3, then lane 31 into the upper half (lanes without a source add zero)
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);     // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);     // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);     // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);     // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);     // row_bcast:15 -> rows 1, 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);     // row_bcast:31 -> rows 2, 3
    return v;
}

// largest value of the wavefront in every lane's hands: DPP row steps, then the four row results through readlane
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    auto mx = [](uint32_t a, int b) { return a > (uint32_t)b ? a : (uint32_t)b; };
    v = mx(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xf, 0xf, false));     // quad_perm [1,0,3,2]
    v = mx(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xf, 0xf, false));     // quad_perm [2,3,0,1]
    v = mx(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xf, 0xf, false));    // row_half_mirror
    v = mx(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xf, 0xf, false));    // row_mirror
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), r1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 16),
                   r2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), r3 = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
    const uint32_t a = r0 > r1 ? r0 : r1, c = r2 > r3 ? r2 : r3;
    return a > c ? a : c;
}

constexpr int kSelThreads = 1024;

// inclusive block scan of one int per thread; returns the inclusive prefix, *total gets the block sum
__device__ __forceinline__ int block_scan_incl(int v, int* wave_tot /*[16]*/, int* total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int s = (int)wave_scan_incl((uint32_t)v);
    __syncthreads();                                   // wave_tot may still be read from a previous scan
    if (lane == 63) wave_tot[wave] = s;
    __syncthreads();
    int base = 0, tot = 0;
    const int nw = blockDim.x >> 6;
    for (int w = 0; w < nw; ++w) {
        const int t = wave_tot[w];
        if (w < wave) base += t;
        tot += t;
    }
    *total = tot;
    return s + base;
}

__global__ void __launch_bounds__(kSelThreads)
spu_select(const float* __restrict__ scores, int N, int n_keep, int32_t* __restrict__ kept_idx,
           const int32_t* __restrict__ origin_in /* [B,N] or null: identity */, int32_t* __restrict__ origin_out /* [B,n_keep] or null */)
{
    __shared__ int hist[256];
    __shared__ int wave_tot[16];
    __shared__ uint32_t sh_prefix;
    __shared__ int sh_remaining;
    const int b = blockIdx.x, tid = threadIdx.x;
    const float* s = scores + (int64_t)b * N;
    int32_t* out = kept_idx + (int64_t)b * n_keep;

    uint32_t prefix = 0, mask = 0;
    int remaining = n_keep;                            // still to pick among keys matching the prefix
    for (int shift = 24; shift >= 0; shift -= 8) {
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        for (int n = tid; n < N; n += kSelThreads) {
            const uint32_t k = score_key(s[n]);
            if ((k & mask) == prefix) atomicAdd(&hist[(k >> shift) & 255u], 1);
        }
        __syncthreads();
        // digit d is the one where (tokens with a larger digit) < remaining <= (those plus hist[d]);
        // thread i looks at digit 255 - i so that an inclusive scan counts "this digit and larger"
        int h = 0, incl = 0, tot;
        if (tid < 256) h = hist[255 - tid];
        incl = block_scan_incl(tid < 256 ? h : 0, wave_tot, &tot);
        if (tid < 256 && incl - h < remaining && remaining <= incl) {
            sh_prefix = prefix | ((uint32_t)(255 - tid) << shift);
            sh_remaining = remaining - (incl - h);
        }
        __syncthreads();
        prefix = sh_prefix;
        remaining = sh_remaining;
        mask |= 255u << shift;
    }
    const uint32_t T = prefix;                         // key of the n_keep-th largest score
    const int take_eq = remaining;                     // tokens with key == T that are kept (lowest indices)

    int eq_before = 0, sel_before = 0;
    for (int n0 = 0, i = 0; n0 < N; n0 += kSelThreads, ++i) {
        const int n = n0 + tid;
        uint32_t k = 0;
        bool eq = false, gt = false;
        if (n < N) {
            k = score_key(s[n]);
            eq = (k == T);
            gt = (k > T);
        }
        int tot_eq, tot_sel;
        const int eq_incl = block_scan_incl(eq ? 1 : 0, wave_tot, &tot_eq);
        const bool sel = gt || (eq && (eq_before + eq_incl - 1) < take_eq);
        const int sel_incl = block_scan_incl(sel ? 1 : 0, wave_tot, &tot_sel);
        if (sel) {
            const int q = sel_before + sel_incl - 1;
            if (q < n_keep) {
                out[q] = n;
                if (origin_out) origin_out[(int64_t)b * n_keep + q] = origin_in ? origin_in[(int64_t)b * N + n] : n;
            }
        }
        eq_before += tot_eq;
        sel_before += tot_sel;
    }
}

template <int BYTES>   // 16: vector rows, 4 / 2: element rows
__global__ void __launch_bounds__(256)
spu_gather(const unsigned char* __restrict__ x, const int32_t* __restrict__ kept_idx, int N, int n_keep,
           int64_t row_bytes_in, int64_t row_bytes_out, int64_t n_rows, unsigned char* __restrict__ x_out)
{
    const int64_t row = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (row >= n_rows) return;
    const int64_t b = row / n_keep;
    int src = kept_idx[row];
    src = src < 0 ? 0 : (src >= N ? N - 1 : src);      // indices come from spu_select; stay in bounds regardless
    const unsigned char* in = x + (b * N + src) * row_bytes_in;
    unsigned char* o = x_out + row * row_bytes_out;
    if (BYTES == 16) {
        for (int64_t i = (int64_t)lane * 16; i < row_bytes_out; i += 64 * 16)
            *reinterpret_cast<uint4*>(o + i) = *reinterpret_cast<const uint4*>(in + i);
    } else if (BYTES == 4) {
        for (int64_t i = (int64_t)lane * 4; i < row_bytes_out; i += 64 * 4)
            *reinterpret_cast<uint32_t*>(o + i) = *reinterpret_cast<const uint32_t*>(in + i);
    } else {
        for (int64_t i = (int64_t)lane * 2; i < row_bytes_out; i += 64 * 2)
            *reinterpret_cast<uint16_t*>(o + i) = *reinterpret_cast<const uint16_t*>(in + i);
    }
}

// ------------------------------------------------------------------ select + gather in one launch (N <= kFusedMaxN)
// Workgroup g of sample b repeats the selection of the sample on its own (the scores of a sample
// are a few KB, and the groups run side by side; samples of different lengths share a launch, the argument lists
// runs of equal ones), keeps the list of kept tokens in LDS, and then copies
// its share of the kept rows: row q goes to wavefront q mod (4 G) of the sample.  The last group, which may have
// fewer rows, also writes kept_idx.  Compared with a selection launch followed by a gather launch this saves a dispatch and the
// wait between the two, which is most of the time at these sizes.
// Bound: latency of the selection, then HBM.  us of a call with scores asked for one by one, an argument list for 64 runs, descriptors
// made of vector registers and the indices ahead of the rows, and as it is: 8 x 1024 x 3584 bf16, 205 kept, 6.98, 6.77; 32 x 500 x 3584,
// 100, 10.0, 9.6; 1 x 4096 x 1024, 1433, 7.87, 7.45; fp32 16 x 512 x 896, 150, 6.20, 5.87.  One by one, three stages of 8 x 1024 x 3584
// with their scores, 67.0: 68.4 without the kernel for one run, 67.7 with vector descriptors, 67.2 with scores one by one, 67.2 with the indices first.
// cache policy of the row copies (buffer aux bits): the copied rows are not read again by this kernel, so the stores
// carry the non-temporal hint (2) and leave less dirty data in L2 for the end of the kernel (measured: -0.3 us)
constexpr int kPruneLoadAux = 0, kPruneStoreAux = 2;
typedef unsigned int prune_u32x4 __attribute__((__vector_size__(16)));
// Threads: 256 for samples of up to 1024 tokens, four keys each; longer ones take 1024, so that the selection stays four
// keys per thread and fewer workgroups repeat it (4 x 4096 tokens, 819 kept, 3584 channels bf16:
// 19 us with 256 threads, 12 with 1024).
// Above 4096 tokens it is eight keys per thread: 1 x 5245 tokens, 545 kept, 21 us as a selection and a
// gather launch, 8.6 like this.
constexpr int kFusedMaxN = 8192;

// workgroups of a sample: one kept row per wavefront, up to 256 of them
__host__ __device__ inline int prune_groups(int n_keep, int waves, bool gather)
{
    const int G = gather ? (n_keep + waves - 1) / waves : 1;
    return G > 256 ? 256 : G;
}

// One run, the common case, has a kernel of its own: an argument list for 64 of them is 2 KB, and its run is fetched a trip later.
template <int RUNS> struct PruneTable { int n; PruneRun run[RUNS]; };

template <int BYTES, int kFusedThreads, int kFusedKeys, int RUNS>
__global__ void __launch_bounds__(kFusedThreads)
spu_prune_fused(const unsigned char* __restrict__ x, const float* __restrict__ scores, const PruneTable<RUNS> runs,
                int64_t row_bytes_in, int64_t row_bytes_out, int32_t* __restrict__ kept_idx, unsigned char* __restrict__ x_out,
                const int32_t* __restrict__ origin_in /* per token or null: identity */, int32_t* __restrict__ origin_out /* per kept token or null */)
{
    __shared__ int32_t kept[kFusedThreads * kFusedKeys];
    __shared__ __align__(16) int hist[4][256];         // one histogram per digit pass: none has to be cleared in between
    constexpr int WAVES = kFusedThreads / 64;
    __shared__ uint32_t wave_tot[WAVES], wave_hi[WAVES], wave_lo[WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    PruneRun run = runs.run[0];
    if constexpr (RUNS > 1) {
        run = runs.run[run_of(runs.n, blockIdx.x, [&](int i) { return (unsigned)runs.run[i].wg0; })];
    }
    const int N = run.N, n_keep = run.n_keep, G = prune_groups(n_keep, WAVES, x_out != nullptr);
    const int b = ((int)blockIdx.x - run.wg0) / G, g = (int)blockIdx.x - run.wg0 - b * G;
    const int64_t tok_in = run.tok_in + (int64_t)b * N, tok_out = run.tok_out + (int64_t)b * n_keep;
    const float* s = scores + tok_in;
    // thread tid owns the K consecutive tokens tid * K .. tid * K + K - 1 and reads them straight from memory
    // (a wavefront covers 64 K consecutive scores; a few KB per sample, served by the caches)
    const int K = (N + kFusedThreads - 1) / kFusedThreads, n0 = tid * K;
    // All asked for together: the descriptor keeps them in bounds, where a branch around each made one trip of every load.
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(s), 0, N * (int)sizeof(float), 0x00020000);
    uint32_t key[kFusedKeys];
#pragma unroll
    for (int i = 0; i < kFusedKeys; ++i) key[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, (n0 + i) * (int)sizeof(float), 0, 0);
    if (tid < 256) *reinterpret_cast<int4*>(&hist[0][0] + 4 * tid) = make_int4(0, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < kFusedKeys; ++i) key[i] = score_key(__uint_as_float(key[i]));
    // Largest and smallest key of the sample: the bits above the highest one in which they differ are common to all
    // keys and need no digit pass (scores of one sample share sign and most of the exponent, so the first of four
    // 8-bit passes would pile every key onto one or two counters - same-address LDS atomics, one after the other).
    uint32_t hi = 0u, lo = 0xffffffffu;
#pragma unroll
    for (int i = 0; i < kFusedKeys; ++i)
        if (i < K && n0 + i < N) { hi = key[i] > hi ? key[i] : hi; lo = key[i] < lo ? key[i] : lo; }
    hi = wave_max_u32(hi);
    lo = ~wave_max_u32(~lo);
    if (lane == 0) { wave_hi[wave] = hi; wave_lo[wave] = lo; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; ++w) { hi = wave_hi[w] > hi ? wave_hi[w] : hi; lo = wave_lo[w] < lo ? wave_lo[w] : lo; }
    const int nb = 32 - __clz((int)(hi ^ lo));         // the keys differ in their low nb bits only (0: all equal)

    // MSD radix select on those bits, 8 at a time (the last pass takes what is left).  Every wavefront scans the
    // histogram of a pass on its own - same counters, same result - so a pass costs one barrier and nothing is
    // handed from wavefront to wavefront.
    uint32_t prefix = nb >= 32 ? 0u : (hi >> nb) << nb, mask = nb >= 32 ? 0u : ~((1u << nb) - 1u);
    int remaining = n_keep;                            // still to pick among keys matching the prefix
    bool whole = false;                                // ... which is all of them: no further digit matters
    for (int top = nb, pass = 0; top > 0 && !whole; top -= 8, ++pass) {
        const int shift = top > 8 ? top - 8 : 0, width = top - shift;
        const uint32_t dmask = (1u << width) - 1u;
        int* h_pass = hist[pass];
#pragma unroll
        for (int i = 0; i < kFusedKeys; ++i)
            if (i < K && n0 + i < N && (key[i] & mask) == prefix) atomicAdd(&h_pass[(key[i] >> shift) & dmask], 1);
        __syncthreads();
        // lane l looks at digits 255 - 4 l .. 252 - 4 l, largest first
        int h[4], sum = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) { h[j] = h_pass[255 - 4 * lane - j]; sum += h[j]; }
        const int incl = (int)wave_scan_incl((uint32_t)sum);
        int above = incl - sum;                        // tokens with a larger digit
        int digit = 0, left = 0, in_digit = 0;
        bool found = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (above < remaining && remaining <= above + h[j]) { digit = 255 - 4 * lane - j; left = remaining - above; in_digit = h[j]; found = true; }
            above += h[j];
        }
        const unsigned long long who = __ballot(found);
        if (who) {                                     // one lane at most (none only when nothing is kept)
            const int src = (int)__builtin_ctzll(who);
            digit = __builtin_amdgcn_readlane(digit, src);
            remaining = __builtin_amdgcn_readlane(left, src);
            whole = remaining == __builtin_amdgcn_readlane(in_digit, src);
        }
        prefix |= (uint32_t)digit << shift;
        mask |= dmask << shift;
    }
    // Kept: the keys whose bits under the mask exceed the prefix, and the first `remaining` of those that equal it - once every
    // bit is under the mask, the n_keep-th largest key and the lowest indices among its equals.
    const uint32_t T = prefix;
    const int take_eq = remaining;

    // one scan for both counts: tokens above T in the low half, tokens equal to T in the high half
    uint32_t cnt = 0;
#pragma unroll
    for (int i = 0; i < kFusedKeys; ++i)
        if (i < K && n0 + i < N) cnt += ((key[i] & mask) > T ? 1u : 0u) + ((key[i] & mask) == T ? 0x10000u : 0u);
    const uint32_t incl = wave_scan_incl(cnt);
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    uint32_t before = incl - cnt;
    for (int w = 0; w < wave; ++w) before += wave_tot[w];
    int eq_rank = (int)(before >> 16);
    int pos = (int)(before & 0xffffu) + (eq_rank < take_eq ? eq_rank : take_eq);
#pragma unroll
    for (int i = 0; i < kFusedKeys; ++i) {
        if (i < K && n0 + i < N) {
            const bool eq = (key[i] & mask) == T;
            if ((key[i] & mask) > T || (eq && eq_rank < take_eq)) {
                if (pos < n_keep) kept[pos] = n0 + i;
                ++pos;
            }
            eq_rank += eq ? 1 : 0;
        }
    }
    __syncthreads();
    for (int q = x_out ? g * WAVES + wave : n_keep; q < n_keep; q += G * WAVES) {
        int src = __builtin_amdgcn_readfirstlane(kept[q]);         // scalars: descriptors made of vectors are a loop around every access
        src = src < 0 ? 0 : (src >= N ? N - 1 : src);  // in bounds whatever the scores held
        const unsigned char* in = x + (tok_in + src) * row_bytes_in;
        unsigned char* o = x_out + (tok_out + q) * row_bytes_out;
        if (BYTES == 16) {
            // eight 16-byte pieces per lane in flight before the first store (bounds by the buffer descriptors: pieces
            // past the end of the row read zeros and write nothing), so a row costs one trip to memory, not seven
            const int rb = (int)(row_bytes_out > 0x7fffffff ? 0x7fffffff : row_bytes_out);
            const __amdgpu_buffer_rsrc_t ri = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(in), 0, rb, 0x00020000);
            const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(o, 0, rb, 0x00020000);
            for (int base = 0; base < rb; base += 8 * 1024) {
                prune_u32x4 v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = __builtin_amdgcn_raw_buffer_load_b128(ri, base + k * 1024 + lane * 16, 0, kPruneLoadAux);
#pragma unroll
                for (int k = 0; k < 8; ++k) __builtin_amdgcn_raw_buffer_store_b128(v[k], ro, base + k * 1024 + lane * 16, 0, kPruneStoreAux);
            }
        } else if (BYTES == 4) {
            for (int64_t i = (int64_t)lane * 4; i < row_bytes_out; i += 64 * 4)
                *reinterpret_cast<uint32_t*>(o + i) = *reinterpret_cast<const uint32_t*>(in + i);
        } else {
            for (int64_t i = (int64_t)lane * 2; i < row_bytes_out; i += 64 * 2)
                *reinterpret_cast<uint16_t*>(o + i) = *reinterpret_cast<const uint16_t*>(in + i);
        }
    }
    if (g == G - 1)                                    // the last group, which may have fewer rows
        for (int q = tid; q < n_keep; q += kFusedThreads) {
            const int src = kept[q];
            kept_idx[tok_out + q] = src;
            // position before the first stage of a cascade
            if (origin_out) {
                int from = src;
                if (origin_in) from = origin_in[tok_in + src];
                origin_out[tok_out + q] = from;
            }
        }
}

static luvc_status prune_two_launches(const void* x, const float* scores, int B, int N, int D, int64_t row_stride, luvc_dtype dt,
                                      int n_keep, int32_t* kept_idx, void* x_out, const int32_t* origin_in, int32_t* origin_out, bool v16, hipStream_t st)
{
    const int es = dt == LUVC_F32 ? 4 : 2;
    const int64_t rin = row_stride * es, rout = (int64_t)D * es, rows = (int64_t)B * n_keep;
    LUVC_LAUNCH("spu_select", spu_select, dim3((unsigned)B), dim3(kSelThreads), 0, st, scores, N, n_keep, kept_idx, origin_in, origin_out);
    if (x_out) {
        const unsigned g = (unsigned)((rows * 64 + 255) / 256);
        if (v16)
            LUVC_LAUNCH("spu_gather", (spu_gather<16>), dim3(g), dim3(256), 0, st, (const unsigned char*)x, kept_idx, N, n_keep, rin, rout, rows, (unsigned char*)x_out);
        else if (es == 4)
            LUVC_LAUNCH("spu_gather", (spu_gather<4>), dim3(g), dim3(256), 0, st, (const unsigned char*)x, kept_idx, N, n_keep, rin, rout, rows, (unsigned char*)x_out);
        else
            LUVC_LAUNCH("spu_gather", (spu_gather<2>), dim3(g), dim3(256), 0, st, (const unsigned char*)x, kept_idx, N, n_keep, rin, rout, rows, (unsigned char*)x_out);
    }
    return check_launch("spu prune");
}

luvc_status spu_prune_run(const void* x, const float* scores, int D, int64_t row_stride, luvc_dtype dt, PruneRuns& runs,
                          int32_t* kept_idx, void* x_out, const int32_t* origin_in, int32_t* origin_out, hipStream_t st)
{
    const int es = dt == LUVC_F32 ? 4 : 2;
    const int64_t rin = row_stride * es, rout = (int64_t)D * es;
    const bool v16 = x_out && rin % 16 == 0 && rout % 16 == 0 && ((uintptr_t)x % 16 == 0) && ((uintptr_t)x_out % 16 == 0);
    int64_t wgs = 0;
    int fused = 0;
    int longest = 0;                                       // of the samples of the shared launch
    for (int i = 0; i < runs.n; ++i)
        if (runs.run[i].N <= kFusedMaxN && runs.run[i].N > longest) longest = runs.run[i].N;
    const bool wide = longest > 1024;
    for (int i = 0; i < runs.n; ++i) {
        const PruneRun r = runs.run[i];
        if (r.N > kFusedMaxN) {                            // the list of kept tokens does not fit in LDS
            const luvc_status rc = prune_two_launches((const char*)x + r.tok_in * rin, scores + r.tok_in, r.count, r.N, D, row_stride, dt, r.n_keep, kept_idx + r.tok_out,
                                                      x_out ? (char*)x_out + r.tok_out * rout : nullptr, origin_in ? origin_in + r.tok_in : nullptr,
                                                      origin_out ? origin_out + r.tok_out : nullptr, v16, st);
            if (rc != LUVC_OK) return rc;
            continue;
        }
        runs.run[fused] = r;
        runs.run[fused].wg0 = (int)wgs;
        wgs += (int64_t)r.count * prune_groups(r.n_keep, wide ? 16 : 4, x_out != nullptr);
        ++fused;
    }
    if (fused == 0) return LUVC_OK;
    if (wgs >= ((int64_t)1 << 31)) { set_error("too many kept tokens in one call"); return LUVC_ERR_UNSUPPORTED; }
    runs.n = fused;
    auto table = [&](auto runs_of) {
        PruneTable<decltype(runs_of)::value> t;
        t.n = runs.n;
        for (int i = 0; i < runs.n; ++i) t.run[i] = runs.run[i];
        return t;
    };
#define LUVC_PRUNE_R(BYTES, THREADS, KEYS, RUNS) LUVC_LAUNCH("spu_prune_fused", (spu_prune_fused<BYTES, THREADS, KEYS, RUNS>), dim3((unsigned)wgs), dim3(THREADS), 0, st, \
                                                 (const unsigned char*)x, scores, table(std::integral_constant<int, RUNS>{}), rin, rout, kept_idx, (unsigned char*)x_out, origin_in, origin_out)
#define LUVC_PRUNE_T(BYTES, THREADS, KEYS) do { if (runs.n == 1) LUVC_PRUNE_R(BYTES, THREADS, KEYS, 1); else LUVC_PRUNE_R(BYTES, THREADS, KEYS, kPruneMaxRuns); } while (0)
#define LUVC_PRUNE(BYTES) do { if (longest > 4096) LUVC_PRUNE_T(BYTES, 1024, 8); else if (wide) LUVC_PRUNE_T(BYTES, 1024, 4); else LUVC_PRUNE_T(BYTES, 256, 4); } while (0)
    if (v16 || !x_out) LUVC_PRUNE(16);
    else if (es == 4)  LUVC_PRUNE(4);
    else               LUVC_PRUNE(2);
#undef LUVC_PRUNE
#undef LUVC_PRUNE_T
#undef LUVC_PRUNE_R
    return check_launch("spu prune");
}

}  // namespace luvc
