// SPU score (paper Section 3.3, Eq. 4-8) for samples of up to kCircMaxN tokens: the filter as a circulant matrix on the
// matrix cores.  x'[n, d] = sum_m p[n - m] x[m, d] with the kernel p of spu_taps.hpp, in fp32 accuracy: p is the sum of three
// bf16 terms (24 bits), bf16 tokens enter as they are (the products are exact), fp32 tokens as three bf16 terms of their
// own with the six products that matter (the rest is below 2^-24 of |x| |p|).
//
// A workgroup owns 32 RT output tokens and 256 channels of a sample, a wavefront 64 of them.  Per step of 16 tokens a lane
// fetches 8 tokens of a pair of neighbouring channels, straight from memory (half a wavefront: one 128-byte row piece), and
// two byte permutations per pair of tokens turn that into the operands of two 32-channel tiles (the even and the odd
// channels; their order does not matter, the energies are summed over channels).  The channels are the rows of the
// product, the output tokens its columns: squares are added in a lane's own registers.  The columns of p are shifts of one
// another, so the other operand is read from LDS at a shift: a lane's 8 taps start anywhere, therefore the taps lie there
// eight times, displaced by one to seven places, and every read is one aligned 16-byte access (copies 32 bytes apart
// modulo 256, for the sake of the banks; the counters still show about 3 cycles of bank conflicts per LDS instruction).
//
// Samples of different lengths share a launch: the argument lists runs of equal samples, and workgroups find theirs.
//
// Hand-over between the workgroups of 32 RT tokens: each writes its sums as 64-bit words (value, launch tag), waits for its
// stores, then reads the words of all of them.  Whoever finds every tag adds the sums in channel order in fp64, writes the
// scores and clears the tags; the last to write always does, and if another does too it writes the same values.  One
// trip to memory each way, no atomics; nothing has to be set up, and a captured launch replayed with its tag starts over.
// A tag has 32 bits and depends on the token's row (circ_tag), so memory that another call left behind passes for the
// words of a workgroup only if it holds 32 RT different right values in a row: a constant fill never does.
//
// Bound: matrix cores for N near kCircMaxN (6 N^2 D flops per bf16 sample, 12 for fp32), latency for short samples.
// 1x729x3584 bf16: 18.1 us (2048-point transform: 22), 8x205x3584: 12.8, 4x144x4096: 8.4, 4x861x1408: 31.3.  Rows of odd width,
// stride or start, channel by channel: 16x64x3585 bf16 11.6 us (1536-point transform: 102), 8x205x3585 15.8 (62), fp32 24
// (64), 1x64x65 5.0 (14.8), but 1x729x3585 26.7 (22.3).  Laying out the
// taps costs about 1 us less than with a division per angle and a copy at a time: 1x512x3584 13.9 -> 12.6; and another .5 to 1 us
// less with the angles put together (spu_taps.hpp), every tap written straight to its places in the line instead of by way
// of a list of p, and the first fetches spread over these phases: 1x729x3584 19.1 -> 18.1, 1x1000x1024 14.8 -> 13.8,
// 4x144x4096 9.0 -> 8.4, fp32 1x144x4096 9.6 -> 9.1.  The start, until the first product, is 3 us of those.
#include "common.hpp"
#include "spu.hpp"
#include "spu_taps.hpp"
#include "spu_tiles.hpp"

namespace luvc {

namespace {

typedef __bf16 circ_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 circ_bf16x2 __attribute__((ext_vector_type(2)));
typedef float circ_f32x2 __attribute__((ext_vector_type(2)));
typedef float circ_f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int circ_u32x4 __attribute__((__vector_size__(16)));
typedef unsigned int circ_u32x2 __attribute__((__vector_size__(8)));

// two values rounded to bf16, packed (first one low)
__device__ __forceinline__ uint32_t pk_bf16(float a, float b)
{
    const circ_bf16x2 v = __builtin_convertvector(circ_f32x2{a, b}, circ_bf16x2);
    uint32_t u;
    __builtin_memcpy(&u, &v, 4);
    return u;
}

__device__ __forceinline__ circ_f32x16 circ_mac(circ_f32x16 acc, const circ_u32x4& a, const circ_u32x4& b)
{
    circ_bf16x8 va, vb;
    __builtin_memcpy(&va, &a, 16);
    __builtin_memcpy(&vb, &b, 16);
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, vb, acc, 0, 0, 0);
}

// 8 tokens of two channels as they lie in memory, and the operands of the two channel tiles made of them.  PAIRED: neighbouring
// channels, one access; else the channels are 32 apart and fetched one by one (at `off` and `off1`), wherever they start.
template <typename T, bool PAIRED> struct circ_raw;
template <> struct circ_raw<bf16_t, true> {
    static constexpr int TERMS = 1;
    uint32_t w[8];
    __device__ __forceinline__ void fetch(int j, __amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t) { w[j] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0); }
    __device__ __forceinline__ void operands(circ_u32x4 (&even)[1], circ_u32x4 (&odd)[1]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            even[0][i] = __builtin_amdgcn_perm(w[2 * i + 1], w[2 * i], 0x05040100u);
            odd[0][i] = __builtin_amdgcn_perm(w[2 * i + 1], w[2 * i], 0x07060302u);
        }
    }
};
template <> struct circ_raw<bf16_t, false> {
    static constexpr int TERMS = 1;
    uint32_t w[8], w1[8];
    __device__ __forceinline__ void fetch(int j, __amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t off1)
    {
        w[j] = __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
        w1[j] = __builtin_amdgcn_raw_buffer_load_b16(r, off1, 0, 0);
    }
    __device__ __forceinline__ void operands(circ_u32x4 (&even)[1], circ_u32x4 (&odd)[1]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            even[0][i] = __builtin_amdgcn_perm(w[2 * i + 1], w[2 * i], 0x05040100u);
            odd[0][i] = __builtin_amdgcn_perm(w1[2 * i + 1], w1[2 * i], 0x05040100u);
        }
    }
};
template <bool PAIRED> struct circ_raw<float, PAIRED> {
    static constexpr int TERMS = 3;
    circ_u32x2 w[8];
    __device__ __forceinline__ void fetch(int j, __amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t off1)
    {
        if constexpr (PAIRED) w[j] = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
        else {
            w[j][0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
            w[j][1] = __builtin_amdgcn_raw_buffer_load_b32(r, off1, 0, 0);
        }
    }
    __device__ static __forceinline__ void split(float a, float b, uint32_t& t0, uint32_t& t1, uint32_t& t2)
    {
        t0 = pk_bf16(a, b);
        a -= __uint_as_float(t0 << 16);
        b -= __uint_as_float(t0 & 0xffff0000u);
        t1 = pk_bf16(a, b);
        a -= __uint_as_float(t1 << 16);
        b -= __uint_as_float(t1 & 0xffff0000u);
        t2 = pk_bf16(a, b);
    }
    __device__ __forceinline__ void operands(circ_u32x4 (&even)[3], circ_u32x4 (&odd)[3]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t t0, t1, t2;
            split(__uint_as_float(w[2 * i][0]), __uint_as_float(w[2 * i + 1][0]), t0, t1, t2);
            even[0][i] = t0; even[1][i] = t1; even[2][i] = t2;
            split(__uint_as_float(w[2 * i][1]), __uint_as_float(w[2 * i + 1][1]), t0, t1, t2);
            odd[0][i] = t0; odd[1][i] = t1; odd[2][i] = t2;
        }
    }
};

// the tag of the words of a group's token `row`
__device__ __forceinline__ uint32_t circ_tag(uint32_t tag, int row) { return tag + (uint32_t)row * 0x9E3779B1u; }

// LDS: taps [3 terms][8 displacements] of circ_stride bytes, 32 mod 256; the taps once more, undisplaced
__host__ __device__ inline int circ_taps(int N, int RT) { return (N + 15) / 16 * 16 + 32 * RT + 8; }
__host__ __device__ inline int circ_stride(int N, int RT) { return ((circ_taps(N, RT) + 8) * 2 + 223) / 256 * 256 + 32; }
__host__ __device__ inline int circ_lds(int N, int RT) { return 24 * circ_stride(N, RT) + 3 * 2 * (circ_taps(N, RT) + 16); }

}  // namespace

// KS: wavefronts that share the steps of a product, each an equal run of them (RT = 1)
// RUNS: one run, the common case, has a kernel of its own, without an argument list for 64 (1.5 KB)
template <int RUNS> struct CircTable { int n; CircRun run[RUNS]; };
template <typename T, int RT, int KS, bool PAIRED /* every channel pair is one aligned access */, int RUNS>
__global__ void __launch_bounds__(256 * KS, KS == 1 || sizeof(T) == 4 ? 2 : 4)
spu_circ(const T* __restrict__ x, int64_t row_stride, int D, int n_quads /* workgroups across the channels */, int use_hamming, const CircTable<RUNS> runs,
         unsigned long long* __restrict__ words /* [groups of 32 RT tokens][n_quads][32 RT] */, uint32_t tag, float* __restrict__ scores)
{
    using raw_t = circ_raw<T, PAIRED>;
    constexpr int ROWS = 32 * RT, TERMS = raw_t::TERMS, THREADS = 256 * KS;
    static_assert(KS == 1 || RT == 1, "");
    // steps of 16 tokens in flight; a bf16 channel fetched by itself takes a register, as a pair does
    constexpr int PF = TERMS == 3 ? (RT == 4 ? 2 : RT == 2 ? 3 : 4) : PAIRED ? (RT == 4 ? 3 : RT == 2 ? 4 : 6) : (RT == 4 || KS == 2 ? 2 : 3);
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double part[THREADS];
    __shared__ float red[4 * ROWS];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int item = (int)xcd_contiguous(blockIdx.x, gridDim.x);
    CircRun run = runs.run[0];
    if constexpr (RUNS > 1) run = runs.run[run_of(runs.n, (unsigned)item, [&](int i) { return (unsigned)(runs.run[i].group0 * n_quads); })];
    const int N = run.N, sigma = run.sigma, group0 = run.group0;
    const int n_groups = (N + ROWS - 1) / ROWS, local = item - group0 * n_quads;
    const int s = local / (n_quads * n_groups), rem = local - s * (n_quads * n_groups), quad = rem / n_groups, grp = rem - quad * n_groups;
    const int64_t tok = run.tok0 + (int64_t)s * N;
    const int n0 = grp * ROWS, all_steps = (N + 15) / 16, share = (all_steps + KS - 1) / KS;
    const int k0 = (wave >> 2) * share, steps = k0 + share < all_steps ? k0 + share : all_steps;      // this wavefront's: k0 .. steps - 1

    // ---- tokens: lane l fetches channels 2 (l % 32), + 1 (or l % 32, + 32) of the wavefront's 64 and the tokens of half l / 32 of a step
    const int d0 = (quad * 4 + (wave & 3)) * 64, h = lane >> 5, c31 = lane & 31;
    const bool live = d0 < D;
    const uint32_t row_bytes = (uint32_t)row_stride * (uint32_t)sizeof(T);
    // the descriptor ends with the last token of the sample: tokens past it read zeros; so do channels past D (an offset beyond any descriptor)
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(x) + tok * row_stride + (live ? d0 : 0), 0,
        live ? (int)((uint32_t)(N - 1) * row_bytes + (uint32_t)((D - d0 < 64 ? D - d0 : 64) * (int)sizeof(T))) : 0, 0x00020000);
    const int c0 = PAIRED ? 2 * c31 : c31, c1 = c31 + 32;
    const uint32_t half_off = (uint32_t)(8 * h) * row_bytes;
    const uint32_t lane_off = d0 + c0 < D ? half_off + (uint32_t)(c0 * (int)sizeof(T)) : 0x80000000u;
    const uint32_t lane_off1 = d0 + c1 < D ? half_off + (uint32_t)(c1 * (int)sizeof(T)) : 0x80000000u;         // not PAIRED
    raw_t raw[PF];
    auto fetch = [&](raw_t& r, int k) {
        const uint32_t at = (uint32_t)(16 * k) * row_bytes;
#pragma unroll
        for (int j = 0; j < 8; ++j) r.fetch(j, rx, lane_off + at + (uint32_t)j * row_bytes, lane_off1 + at + (uint32_t)j * row_bytes);
    };
    // asked for in three parts, between the phases of the taps: all at once they are .6 us in which nothing else starts
    constexpr int PF1 = (PF + 2) / 3, PF2 = (2 * PF + 2) / 3;
#pragma unroll
    for (int u = 0; u < PF1; ++u) fetch(raw[u], k0 + u);

    // ---- taps: p[0 .. N/2] in fp64, split into three bf16 terms, to every place of the line of taps where they belong: entry o of
    // the line is p[o - n0 - ROWS].  p is even and repeats after N, so also after `turn`, N or a multiple of it that is 64 at least
    // and leaves a thread few places.
    const int taps = circ_taps(N, RT), stride = circ_stride(N, RT);
    uint16_t* line = reinterpret_cast<uint16_t*>(smem + 24 * stride);          // [3][taps + 16]
    double2* angles = reinterpret_cast<double2*>(smem);                        // where the displaced taps will lie
    SpuTaps::fill_angles<THREADS>(angles, N, sigma);
#pragma unroll
    for (int u = PF1; u < PF2; ++u) fetch(raw[u], k0 + u);
    __syncthreads();
    {
        const SpuTaps p(N, sigma, use_hamming, angles);
        const int turn = N >= 64 ? N : N * (63 / N + 1), zero = (n0 + ROWS) % turn;
        for (int jj = tid; jj <= turn / 2; jj += THREADS) {
            int j = jj;
            if (N < 64) {
                j = jj % N;
                j = 2 * j > N ? N - j : j;
            }
            double v = p(j, angles);
            uint16_t b[3];
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                b[t] = f64_to_bf16(v);
                v -= (double)bf16_to_f32(b[t]);
            }
            const int up = zero + jj, down = zero - jj;
            auto put = [&](int at) {
                for (; at < taps + 16; at += turn)
#pragma unroll
                    for (int t = 0; t < 3; ++t) line[t * (taps + 16) + at] = b[t];
            };
            put(up >= turn ? up - turn : up);
            put(down < 0 ? down + turn : down);
        }
    }
#pragma unroll
    for (int u = PF2; u < PF; ++u) fetch(raw[u], k0 + u);
    __syncthreads();
    // a thread: 16 taps of a term, out of which 8 of every displaced copy
    const int eights = taps / 8;
    for (int at = tid; at < 3 * eights; at += THREADS) {
        const int t = at / eights, i = at - t * eights;
        const circ_u32x4* from = reinterpret_cast<const circ_u32x4*>(line + t * (taps + 16)) + i;
        const circ_u32x4 lo = from[0], hi = from[1];
        const uint32_t v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            circ_u32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (c & 1) ? __builtin_amdgcn_alignbit(v[c / 2 + e + 1], v[c / 2 + e], 16) : v[c / 2 + e];
            *reinterpret_cast<circ_u32x4*>(smem + (8 * t + c) * stride + i * 16) = o;
        }
    }
    __syncthreads();

    // ---- the product
    circ_f32x16 acc[RT][2];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][o][v] = 0.f;
    if (live) {
        const int cp = (8 - (c31 & 7)) & 7;
        const unsigned char* tap = smem + cp * stride + (8 * h + ROWS - c31 - cp) * 2;
        // the taps of the next tile (of this step, or the first of the next) are read ahead of a tile's products
        circ_u32x4 next[3];
        auto read_taps = [&](int k, int t) {
#pragma unroll
            for (int e = 0; e < 3; ++e) next[e] = *reinterpret_cast<const circ_u32x4*>(tap + e * 8 * stride + k * 32 - t * 64);
        };
        read_taps(k0, 0);
        auto step = [&](const raw_t& r, int k) {
            circ_u32x4 xe[TERMS], xo[TERMS];
            r.operands(xe, xo);
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                const circ_u32x4 pt[3] = {next[0], next[1], next[2]};
                read_taps(t + 1 < RT ? k : k + 1, t + 1 < RT ? t + 1 : 0);
                __builtin_amdgcn_sched_barrier(0);
                // smallest products first
#pragma unroll
                for (int sum = 2; sum >= 0; --sum)
#pragma unroll
                    for (int e = 2; e >= 0; --e) {
                        const int f = TERMS == 1 ? 0 : sum - e;
                        if (TERMS == 1 ? e != sum : (f < 0 || f >= TERMS)) continue;
                        acc[t][0] = circ_mac(acc[t][0], xe[f < 0 ? 0 : f], pt[e]);
                        acc[t][1] = circ_mac(acc[t][1], xo[f < 0 ? 0 : f], pt[e]);
                    }
            }
        };
        // whole rounds of PF steps without a branch inside: at a join the compiler waits for everything in flight
        int k = k0;
        for (; k + PF <= steps; k += PF) {
#pragma unroll
            for (int u = 0; u < PF; ++u) {
                step(raw[u], k + u);
                fetch(raw[u], k + u + PF);
                __builtin_amdgcn_sched_barrier(0);       // fetches, and the permutations that wait for them, stay in this order
            }
        }
#pragma unroll
        for (int u = 0; u < PF - 1; ++u)
            if (k + u < steps) step(raw[u], k + u);
    }
    // ---- the shares of a product, the first one's wavefronts add the others' in order
    if constexpr (KS > 1) {
        float4* grid = reinterpret_cast<float4*>(smem);          // [KS - 1][4 wavefronts][8][64 lanes], where the taps were
        __syncthreads();
        if (wave >= 4) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const circ_f32x16& a = acc[0][q >> 2];
                grid[((wave - 4) * 8 + q) * 64 + lane] = make_float4(a[4 * (q & 3)], a[4 * (q & 3) + 1], a[4 * (q & 3) + 2], a[4 * (q & 3) + 3]);
            }
        }
        __syncthreads();
        if (wave < 4) {
#pragma unroll
            for (int u = 0; u < KS - 1; ++u)
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    circ_f32x16& a = acc[0][q >> 2];
                    const float4 o = grid[((4 * u + wave) * 8 + q) * 64 + lane];
                    a[4 * (q & 3)] += o.x; a[4 * (q & 3) + 1] += o.y; a[4 * (q & 3) + 2] += o.z; a[4 * (q & 3) + 3] += o.w;
                }
        }
    }
    // ---- Eq. 8: over the wavefront's channels (16 rows per lane and tile, two halves of the wavefront), then the four wavefronts
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        // in four parts: fewer roundings on the way to a sum, and a shorter chain
        float p[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) p[v] = acc[t][v & 1][v >> 1] * acc[t][v & 1][v >> 1];
#pragma unroll
        for (int v = 4; v < 32; ++v) p[v & 3] = fmaf(acc[t][v & 1][v >> 1], acc[t][v & 1][v >> 1], p[v & 3]);
        float e = (p[0] + p[1]) + (p[2] + p[3]);
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(e), __float_as_uint(e), false, false);
        e = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        if (h == 0 && wave < 4) red[wave * ROWS + t * 32 + c31] = e;
    }
    __syncthreads();
    double sum4 = 0.0;
    if (tid < ROWS) sum4 = (((double)red[tid] + (double)red[ROWS + tid]) + (double)red[2 * ROWS + tid]) + (double)red[3 * ROWS + tid];
    float* out = scores + tok + n0;
    if (n_quads == 1) {
        if (tid < ROWS && n0 + tid < N) out[tid] = (float)sqrt(sum4);
        return;
    }
    const float own = (float)sum4;
    const int row = tid % ROWS;
    const uint32_t row_tag = circ_tag(tag, row);
    unsigned long long* w = words + (int64_t)(group0 + s * n_groups + grp) * n_quads * ROWS;
    if (tid < ROWS)
        __hip_atomic_store(w + quad * ROWS + tid, ((unsigned long long)row_tag << 32) | __float_as_uint(own), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // ---- all of them there?  Thread: a token, every PARTS-th workgroup
    constexpr int PARTS = THREADS / ROWS;
    const int pt0 = tid / ROWS;
    bool all = true;
    double e = 0.0;
    for (int i0 = pt0; i0 < n_quads; i0 += 8 * PARTS) {
        unsigned long long v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int at = i0 + i * PARTS < n_quads ? i0 + i * PARTS : i0;
            v[i] = __hip_atomic_load(w + at * ROWS + row, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            all = all && (uint32_t)(v[i] >> 32) == row_tag;
            e += i0 + i * PARTS < n_quads ? (double)__uint_as_float((uint32_t)v[i]) : 0.0;
        }
    }
    part[tid] = e;
    if (!__syncthreads_and(all)) return;
    for (int i = pt0; i < n_quads; i += PARTS) __hip_atomic_store(w + i * ROWS + row, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid < ROWS && n0 + tid < N) {
        double sum = 0.0;
#pragma unroll
        for (int i = 0; i < PARTS; ++i) sum += part[i * ROWS + tid];
        out[tid] = (float)sqrt(sum);
    }
}

// ------------------------------------------------------------------ host side
static int circ_quads(int D) { return (D + 255) / 256; }

// Output tokens per workgroup / 32.  More of them share a fetch and a set of operands (a row of output costs 1.25 with
// RT = 1, 1.05 with 2, 1 with 4), fewer pad less and make more workgroups, of which every compute unit should have one.
static int circ_rt(const CircRuns& runs, int D)
{
    int best = 1;
    double best_cost = 0.0;
    for (int RT = 1; RT <= 4; RT *= 2) {
        int64_t wg = 0;
        double cost = 0.0;
        for (int i = 0; i < runs.n; ++i) {
            const int64_t groups = (int64_t)runs.run[i].count * ((runs.run[i].N + 32 * RT - 1) / (32 * RT));
            wg += groups * circ_quads(D);
            cost += (double)groups * RT * ((runs.run[i].N + 15) / 16) * (RT == 1 ? 1.25 : RT == 2 ? 1.05 : 1.0);
        }
        if (RT == 1 || (wg >= 256 && cost < best_cost)) { best = RT; best_cost = cost; }
    }
    return best;
}

CircRows spu_circ_rows(const void* x, int D, int64_t row_stride, luvc_dtype dt)
{
    const int64_t es = dt == LUVC_F32 ? 4 : 2;
    // a sample inside one descriptor, below the offset that marks a lane without channels
    if ((int64_t)(kCircMaxN + 256) * row_stride * es >= ((int64_t)1 << 31)) return CircRows::None;
    return D % 2 == 0 && row_stride % 2 == 0 && (uintptr_t)x % (uintptr_t)(2 * es) == 0 ? CircRows::Paired : CircRows::Single;
}

// one word per output token (rounded up to a workgroup's share) and 256 channels
size_t spu_circ_bytes(int64_t samples, int N, int D)
{
    return circ_quads(D) == 1 ? 0 : sizeof(unsigned long long) * (size_t)samples * circ_quads(D) * ((size_t)(N + 127) / 128 * 128);
}

// Wavefronts per product.  Its steps come one after the other; where the workgroups do not fill the chip and the samples are
// long enough to pay for a last addition, two wavefronts take half of them each (1x1000x1024 bf16 17.3 -> 16.1 us, fp32
// 32.5 -> 28.6, 1x300x2048 fp32 13.4 -> 12.9; 1x144x4096 bf16 would go from 7.2 to 7.6, and four wavefronts gain nothing more).
static int circ_shares(const CircRuns& runs, int D, luvc_dtype dt)
{
    int64_t wg = 0;
    int longest = 0;
    for (int i = 0; i < runs.n; ++i) {
        wg += (int64_t)runs.run[i].count * ((runs.run[i].N + 31) / 32) * circ_quads(D);
        longest = runs.run[i].N > longest ? runs.run[i].N : longest;
    }
    return wg <= 256 && longest >= (dt == LUVC_F32 ? 256 : 512) ? 2 : 1;
}

template <typename T, int RT, int KS, bool PAIRED, int RUNS>
static void circ_launch(const T* x, int64_t row_stride, int D, int use_hamming, CircRuns& runs, void* words, float* scores, hipStream_t st)
{
    int64_t groups = 0;
    int lds = (KS - 1) * 32768;
    for (int i = 0; i < runs.n; ++i) {
        runs.run[i].group0 = (int)groups;
        groups += (int64_t)runs.run[i].count * ((runs.run[i].N + 32 * RT - 1) / (32 * RT));
        const int b = circ_lds(runs.run[i].N, RT);
        lds = b > lds ? b : lds;
    }
    CircTable<RUNS> table;
    table.n = runs.n;
    for (int i = 0; i < runs.n; ++i) table.run[i] = runs.run[i];
    LUVC_LAUNCH("spu_circ", (spu_circ<T, RT, KS, PAIRED, RUNS>), dim3((unsigned)(groups * circ_quads(D))), dim3(256 * KS), (size_t)lds, st, x, row_stride, D, circ_quads(D), use_hamming,
                table, (unsigned long long*)words, (uint32_t)(spu_next_tag() % 0xffffffffull) + 1u, scores);
}

luvc_status spu_score_circ(const void* x, int64_t row_stride, int D, luvc_dtype dt, int use_hamming, CircRuns& runs, void* words, float* scores, hipStream_t st)
{
    const int RT = circ_rt(runs, D), KS = RT == 1 ? circ_shares(runs, D, dt) : 1;
    const bool paired = spu_circ_rows(x, D, row_stride, dt) == CircRows::Paired;
#define LUVC_CIRC_N(TT, R, K, PAIRED) do { \
        if (runs.n == 1) circ_launch<TT, R, K, PAIRED, 1>((const TT*)x, row_stride, D, use_hamming, runs, words, scores, st); \
        else circ_launch<TT, R, K, PAIRED, kCircMaxRuns>((const TT*)x, row_stride, D, use_hamming, runs, words, scores, st); \
    } while (0)
#define LUVC_CIRC(TT, R, K) do { if (paired) LUVC_CIRC_N(TT, R, K, true); else LUVC_CIRC_N(TT, R, K, false); } while (0)
#define LUVC_CIRC_T(TT) do { if (RT == 4) LUVC_CIRC(TT, 4, 1); else if (RT == 2) LUVC_CIRC(TT, 2, 1); else if (KS == 2) LUVC_CIRC(TT, 1, 2); else LUVC_CIRC(TT, 1, 1); } while (0)
    if (dt == LUVC_F32) LUVC_CIRC_T(float); else LUVC_CIRC_T(bf16_t);
#undef LUVC_CIRC_T
#undef LUVC_CIRC
#undef LUVC_CIRC_N
    return check_launch("spu score (circulant)");
}

}  // namespace luvc
