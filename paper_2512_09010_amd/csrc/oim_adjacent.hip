// OIM (paper Section 3.2, Algorithm 1) with the adjacent destinations as candidates, for schedules that take few tokens
// out of a line per pass (merge number 2): one launch per pass on grids of row ids (see oim_wide_lazy.hip: the tokens
// are moved once, after the last pass).
//
// One workgroup per line of at most 128 tokens.  A wavefront fetches four consecutive tokens and the one after them, all
// in flight together, and forms their squared norms and neighbour products in fp64 at once: with two candidates per
// source there is little to save by screening, and a pass needs no second look at the tokens.  Then the cosines of the
// sources (one wavefront, a source per lane), the m best of them (a source per ballot), the layout of the next grid and
// the size-weighted means of the destinations that take sources in, written to overlay rows.
//
// Bound: latency.  A pass reads its tokens once, but a line is a chain of memory trips - ids, tokens, merged rows - with
// the decisions between them; as many wavefronts as a line has groups of four tokens share it, so that each trip is made once.
// 12 x 32 x 32 x 1024 bf16, three operations of (W,2),(H,2): 157 us as three launches per pass (norms and products,
// decisions, a merge that rewrote the whole grid), {ADJ_US} us as one.
#include "common.hpp"
#include "oim.hpp"
#include "oim_lazy.hpp"
#include "oim_sum64.hpp"

namespace luvc {

namespace {

typedef unsigned int adj_u32x4 __attribute__((__vector_size__(16)));

template <typename T> struct adj_io;
template <> struct adj_io<bf16_t> {
    static constexpr int V = 8;
    __device__ static __forceinline__ double at(const adj_u32x4& v, int e) { return (double)__uint_as_float((e & 1) ? v[e >> 1] & 0xffff0000u : v[e >> 1] << 16); }
};
template <> struct adj_io<float> {
    static constexpr int V = 4;
    __device__ static __forceinline__ double at(const adj_u32x4& v, int e) { return (double)__uint_as_float(v[e]); }
};

// 16 bytes per lane of a row of `bytes` bytes; zeros past its end
__device__ __forceinline__ adj_u32x4 adj_load(__amdgpu_buffer_rsrc_t r, int off) { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0); }
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t adj_row(const T* p, int D, bool present)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), 0, present ? D * (int)sizeof(T) : 0, 0x00020000);
}

}  // namespace

constexpr int kAdjTok = 4;                       // consecutive tokens of a wavefront
constexpr int kAdjPieces = 3;                    // 16-byte pieces of a token per lane in flight (bf16: 1536 channels)

template <typename T>
__global__ void __launch_bounds__(1024)
oim_adjacent_line(const T* __restrict__ x, T* ov, const T* __restrict__ xk /* metric [.., Dk] the decisions are taken on, or null: x */,
                  T* ovk /* its overlay */, int Dk, const int32_t* __restrict__ idx_in /* null: identity */,
                  const int32_t* __restrict__ sizes_in /* null: ones */, const int32_t* __restrict__ kept_in /* null: identity */,
                  LazyGeom g, int32_t* __restrict__ idx_out, int32_t* __restrict__ sizes_out, int32_t* __restrict__ kept_out /* or null */,
                  int32_t* __restrict__ pass_map /* or null */)
{
    using io = adj_io<T>;
    constexpr int V = io::V;
    __shared__ double nrm2[kLazyMaxLen + 4], dnx[kLazyMaxLen + 4];     // squared norm; product with the next token of the line
    __shared__ double score[64];
    __shared__ int rid[kLazyMaxLen], sz[kLazyMaxLen];
    __shared__ int side[64];                     // best destination of a source: 0 the one before it, 1 the one after it, -1 none
    __shared__ int gone[64];                     // the source is merged
    const int len = g.axis ? g.w : g.h, nlines = g.axis ? g.h : g.w;
    const int n_src = (len + 1) / 2, n_dst = len / 2;
    const int Wo = g.axis ? g.w - g.m : g.w, Ho = g.axis ? g.h : g.h - g.m;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), NW = blockDim.x >> 6;
    const unsigned item = xcd_contiguous(blockIdx.x, gridDim.x);       // lines of one image meet in one L2
    const int64_t b = item / nlines;
    const int line = item % nlines;
    const int64_t img = b * g.h * g.w, img_out = b * Ho * Wo;
    auto in_flat = [&](int p) -> int { return g.axis ? line * g.w + p : p * g.w + line; };
    auto out_flat = [&](int q) -> int { return g.axis ? line * Wo + q : q * Wo + line; };
    const T* dx = xk ? xk : x;
    const T* dov = xk ? ovk : ov;
    const int dD = xk ? Dk : g.D;

    for (int p = tid; p < len; p += blockDim.x) {
        const int f = in_flat(p);
        rid[p] = idx_in ? idx_in[img + f] : f;
        sz[p] = sizes_in ? sizes_in[img + f] : 1;
    }
    // ---- squared norms and neighbour products
    for (int p0 = wave * kAdjTok; p0 < len; p0 += NW * kAdjTok) {
        __amdgpu_buffer_rsrc_t r[kAdjTok + 1];
#pragma unroll
        for (int i = 0; i <= kAdjTok; ++i) {
            const int p = p0 + i < len ? p0 + i : len - 1, f = in_flat(p);
            r[i] = adj_row(row_of<T>(dx, dov, b, idx_in ? idx_in[img + f] : f, g, dD), dD, p0 + i < len);
        }
        double s[2 * kAdjTok];
#pragma unroll
        for (int i = 0; i < 2 * kAdjTok; ++i) s[i] = 0.0;
        for (int d0 = 0; d0 < dD; d0 += 64 * V * kAdjPieces) {
            adj_u32x4 t[kAdjTok + 1][kAdjPieces];
#pragma unroll
            for (int i = 0; i <= kAdjTok; ++i)
#pragma unroll
                for (int u = 0; u < kAdjPieces; ++u) t[i][u] = adj_load(r[i], (d0 + (u * 64 + lane) * V) * (int)sizeof(T));
#pragma unroll
            for (int u = 0; u < kAdjPieces; ++u)
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    double a = io::at(t[0][u], e);
#pragma unroll
                    for (int i = 0; i < kAdjTok; ++i) {
                        const double c = io::at(t[i + 1][u], e);
                        s[i] = fma(a, a, s[i]);
                        s[kAdjTok + i] = fma(a, c, s[kAdjTok + i]);
                        a = c;
                    }
                }
        }
        wave_total64x8(s, lane);
        if (lane == 0) {
#pragma unroll
            for (int i = 0; i < kAdjTok; ++i) { nrm2[p0 + i] = s[i]; dnx[p0 + i] = s[kAdjTok + i]; }
        }
    }
    __syncthreads();
    // ---- cosine of every source with its two neighbours (equal: the lower position)
    if (wave == 0 && lane < n_src) {
        const int a = 2 * lane;
        const bool hl = a >= 1, hr = a + 1 < len;
        auto norm = [&](int p) { const double n = sqrt(nrm2[p]); return n < 1e-12 ? 1e-12 : n; };
        const double na = norm(a);
        const double sl = hl ? dnx[a - 1] / (na * norm(a - 1)) : 0.0, sr = hr ? dnx[a] / (na * norm(a + 1)) : 0.0;
        const bool left = hl && (!hr || !(sr > sl));
        const double best = left ? sl : sr;
        score[lane] = best == best ? best : -INFINITY;       // NaN: last, so that exactly m sources leave the line whatever the tokens hold
        side[lane] = hl || hr ? (left ? 0 : 1) : -1;
    }
    __syncthreads();
    // ---- the m best (equal: the lower position): a source per ballot of those that beat it
    {
        const double mine = lane < n_src ? score[lane] : 0.0;
        for (int j = wave; j < n_src; j += NW) {
            const double s = score[j];
            const int rank = __popcll(__ballot(lane < n_src && (mine > s || (mine == s && lane < j))));
            if (lane == 0) gone[j] = g.m == n_src || rank < g.m;
        }
    }
    __syncthreads();
    // ---- layout of the next grid: lane k of every wavefront looks at source 2 k and destination 2 k + 1
    const unsigned long long below = (1ull << lane) - 1ull;
    const bool sgone = lane < n_src && gone[lane];
    const int sside = lane < n_src ? side[lane] : -1;
    const unsigned long long m_gone = __ballot(sgone), m_right = __ballot(sgone && sside == 1), m_left = __ballot(sgone && sside == 0);
    const unsigned long long from_prev = m_right, from_next = m_left >> 1;       // destinations that take in source 2 k, source 2 k + 2
    const unsigned long long takes = from_prev | from_next;
    auto slot = [&](int p) {                     // output slot of the surviving position p: the survivors before it
        const int k = p >> 1;                    // sources before p: k (+ 1 when p is odd), destinations before p: k
        const unsigned long long before = (p & 1) ? (2ull << k) - 1ull : (1ull << k) - 1ull;
        return out_flat(p - __popcll(m_gone & before));
    };
    auto taken = [&](int k) {                    // size of destination 2 k + 1 after the pass
        int S = sz[2 * k + 1];
        if ((from_prev >> k) & 1ull) S += sz[2 * k];
        if ((from_next >> k) & 1ull) S += sz[2 * k + 2];
        return S;
    };
    if (wave == 0 && lane < n_src) {             // sources
        const int p = 2 * lane, f = in_flat(p);
        if (!sgone) {
            const int of = slot(p);
            idx_out[img_out + of] = rid[p];
            sizes_out[img_out + of] = sz[p];
            if (kept_out) kept_out[img_out + of] = kept_in ? kept_in[img + f] : f;
            if (pass_map) pass_map[img + f] = of;
        } else if (pass_map && sside >= 0) {
            pass_map[img + f] = slot(sside ? p + 1 : p - 1);
        }
    }
    if (wave == NW - 1 && lane < n_dst) {        // destinations
        const int p = 2 * lane + 1, f = in_flat(p), of = slot(p);
        idx_out[img_out + of] = ((takes >> lane) & 1ull) ? g.n0 + g.ov_base + line * g.per_line + __popcll(takes & below) : rid[p];
        sizes_out[img_out + of] = taken(lane);
        if (kept_out) kept_out[img_out + of] = kept_in ? kept_in[img + f] : f;
        if (pass_map) pass_map[img + f] = of;
    }
    // ---- the destinations that take sources in: size-weighted mean in fp64 (destination first, then the sources in
    // ascending position), rounded once; a wavefront per destination and tensor
    const int n_abs = __popcll(takes);
    for (int kk = wave; kk < (xk ? 2 : 1) * n_abs; kk += NW) {
        const bool on_metric = kk >= n_abs;
        const int at = on_metric ? kk - n_abs : kk;
        unsigned long long left = takes;
        for (int i = 0; i < at; ++i) left &= left - 1;
        const int k = (int)__builtin_ctzll(left), p = 2 * k + 1;
        const T* mx = on_metric ? xk : x;
        T* mov = on_metric ? ovk : ov;
        const int mD = on_metric ? Dk : g.D;
        const bool fa = (from_prev >> k) & 1ull, fc = (from_next >> k) & 1ull;
        const __amdgpu_buffer_rsrc_t rp = adj_row(row_of<T>(mx, mov, b, rid[p], g, mD), mD, true),
                                     ra = adj_row(row_of<T>(mx, mov, b, rid[p - 1], g, mD), mD, fa),
                                     rc = adj_row(row_of<T>(mx, mov, b, rid[fc ? p + 1 : p], g, mD), mD, fc);
        T* o = mov + (b * g.cap + g.ov_base + line * g.per_line + at) * mD;
        const double sp = sz[p], sa = fa ? sz[p - 1] : 0, s2 = fc ? sz[p + 1] : 0, S = (sp + sa) + s2, inv = 1.0 / S;
        for (int d0 = 0; d0 < mD; d0 += 64 * V * kAdjPieces) {
            adj_u32x4 vp[kAdjPieces], va[kAdjPieces], vc[kAdjPieces];
#pragma unroll
            for (int u = 0; u < kAdjPieces; ++u) {
                const int off = (d0 + (u * 64 + lane) * V) * (int)sizeof(T);
                vp[u] = adj_load(rp, off);
                va[u] = adj_load(ra, off);
                vc[u] = adj_load(rc, off);
            }
#pragma unroll
            for (int u = 0; u < kAdjPieces; ++u) {
                const int d = d0 + (u * 64 + lane) * V;
                if (d >= mD) continue;
                T q[V];
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    double acc = sp * io::at(vp[u], e);
                    if (fa) acc += sa * io::at(va[u], e);
                    if (fc) acc += s2 * io::at(vc[u], e);
                    // acc / S, correctly rounded: the reciprocal is, and one step on the exact remainder corrects the product
                    const double h = acc * inv, rem = fma(-h, S, acc);
                    io_traits<T>::store(&q[e], rem == 0.0 ? h : fma(rem, inv, h));       // (a zero keeps its sign)
                }
                *reinterpret_cast<adj_u32x4*>(o + d) = *reinterpret_cast<const adj_u32x4*>(q);
            }
        }
    }
}

// ------------------------------------------------------------------ host side
template <typename T>
static luvc_status run_adjacent(const T* x, T* ov, const T* xk, T* ovk, int Dk, const int32_t* idx_in, const int32_t* sizes_in, const int32_t* kept_in,
                                int B, const LazyGeom& g, int32_t* idx_out, int32_t* sizes_out, int32_t* kept_out, int32_t* pass_map, hipStream_t st)
{
    const int len = g.axis ? g.w : g.h, nlines = g.axis ? g.h : g.w;
    int waves = (len + kAdjTok - 1) / kAdjTok;
    waves = waves > 16 ? 16 : waves;
    LUVC_LAUNCH("oim_adjacent_line", (oim_adjacent_line<T>), dim3((unsigned)(B * nlines)), dim3(64 * waves), 0, st, x, ov, xk, ovk, Dk,
                idx_in, sizes_in, kept_in, g, idx_out, sizes_out, kept_out, pass_map);
    return check_launch("oim pass (adjacent matching, one launch)");
}

luvc_status oim_adjacent_pass(const void* x, void* ov, const void* metric, void* ov_metric, int Dm, const int32_t* idx_in, const int32_t* sizes_in, const int32_t* kept_in,
                              int B, int n0, int h, int w, int D, luvc_dtype dt, int axis, int m, int cap, int ov_base,
                              int32_t* idx_out, int32_t* sizes_out, int32_t* kept_out, int32_t* pass_map, hipStream_t st)
{
    const int len = axis ? w : h, n_dst = len / 2;
    if (len > kLazyMaxLen) { set_error("adjacent matching (one launch per pass): line of %d tokens", len); return LUVC_ERR_UNSUPPORTED; }
    LazyGeom g;
    g.n0 = n0; g.h = h; g.w = w; g.D = D; g.axis = axis; g.m = m; g.radius = 1; g.cap = cap; g.ov_base = ov_base;
    g.per_line = m < n_dst ? m : n_dst;
    if (dt == LUVC_F32)
        return run_adjacent<float>((const float*)x, (float*)ov, (const float*)metric, (float*)ov_metric, Dm, idx_in, sizes_in, kept_in, B, g,
                                   idx_out, sizes_out, kept_out, pass_map, st);
    return run_adjacent<bf16_t>((const bf16_t*)x, (bf16_t*)ov, (const bf16_t*)metric, (bf16_t*)ov_metric, Dm, idx_in, sizes_in, kept_in, B, g,
                                idx_out, sizes_out, kept_out, pass_map, st);
}

}  // namespace luvc
