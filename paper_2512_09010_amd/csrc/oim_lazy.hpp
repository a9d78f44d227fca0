// Grids of row ids (paper Section 3.2, Algorithm 1, with few tokens leaving a line per pass): shared by the kernels
// that run a pass without moving the tokens (oim_wide_lazy.hip, oim_adjacent.hip).
#pragma once
#include "common.hpp"

namespace luvc {

namespace {

struct LazyGeom {
    int n0;         // tokens per image of the call's input grid: ids below it are rows of x
    int h, w;       // grid before this pass
    int D, axis, m, radius;
    int cap;        // overlay rows per image over the whole call
    int ov_base;    // first overlay row of this pass
    int per_line;   // overlay rows a line of this pass may write: min(m, destinations of the line)
};

template <typename T>
__device__ __forceinline__ const T* row_of(const T* x, const T* ov, int64_t b, int id, const LazyGeom& g, int D)
{
    return id < g.n0 ? x + (b * g.n0 + id) * D : ov + (b * g.cap + (id - g.n0)) * D;
}


// ------------------------------------------------------------------ rows in 16-byte pieces
typedef unsigned int lz_u32x4 __attribute__((__vector_size__(16)));

template <typename T> struct lz_io;
template <> struct lz_io<bf16_t> {
    static constexpr int V = 8;
    __device__ static __forceinline__ double at(const lz_u32x4& v, int e) { return (double)__uint_as_float((e & 1) ? v[e >> 1] & 0xffff0000u : v[e >> 1] << 16); }
};
template <> struct lz_io<float> {
    static constexpr int V = 4;
    __device__ static __forceinline__ double at(const lz_u32x4& v, int e) { return (double)__uint_as_float(v[e]); }
};

// a row as a buffer: pieces past its end read zeros; a row that is not there reads zeros throughout
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t lz_row(const T* p, int D, bool present)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), 0, present ? D * (int)sizeof(T) : 0, 0x00020000);
}
__device__ __forceinline__ lz_u32x4 lz_load(__amdgpu_buffer_rsrc_t r, int off) { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0); }

constexpr int kLzPieces = 3;                     // 16-byte pieces of a row per lane in flight (bf16: 1536 channels)

// ------------------------------------------------------------------ what a pass writes, once the decisions are known
// Lane k of the wavefront holds source 2 k and destination 2 k + 1 of a line of at most 128 tokens.
struct LazyLine {
    unsigned long long gone, takes;              // sources that leave the line, destinations that take sources in
};

// survivors before position p
__device__ __forceinline__ int lazy_slot(const LazyLine& l, int p)
{
    const int k = p >> 1;                        // sources before p: k (+ 1 when p is odd)
    return p - __popcll(l.gone & ((p & 1) ? (2ull << k) - 1ull : (1ull << k) - 1ull));
}

// acc / S, correctly rounded, once to the storage type: the reciprocal is, and one step on the exact remainder corrects the
// product (a zero keeps its sign, an infinity, whose remainder is no number, stays one)
template <typename T>
__device__ __forceinline__ void lazy_round_store(const double (&acc)[lz_io<T>::V], double S, double inv, T* to)
{
    T q[lz_io<T>::V];
#pragma unroll
    for (int e = 0; e < lz_io<T>::V; ++e) {
        const double w = acc[e] * inv, rem = fma(-w, S, acc[e]);
        io_traits<T>::store(&q[e], __builtin_islessgreater(rem, 0.0) ? fma(rem, inv, w) : w);
    }
    *reinterpret_cast<lz_u32x4*>(to) = *reinterpret_cast<const lz_u32x4*>(q);
}

// Size-weighted mean of destination k and the sources `hits` (bit j: source 2 j) of the line, to row o: fp64, destination
// first, then the sources in ascending position, rounded once.  The destination and two sources are fetched together, P pieces
// of each at a time.  The wavefront's share of the row: channels `from` .. `to` - 1.
template <typename T, int P = kLzPieces>
__device__ __forceinline__ void lazy_merge(const T* x, const T* ov, const LazyGeom& g, int D, int64_t b, const int* rid, const int* sz, int k,
                                           unsigned long long hits, T* o, int lane, int from, int to)
{
    using io = lz_io<T>;
    constexpr int V = io::V;
    const __amdgpu_buffer_rsrc_t rp = lz_row(row_of<T>(x, ov, b, rid[2 * k + 1], g, D), D, true);
    const double sp = (double)sz[2 * k + 1];
    for (int d0 = from; d0 < to; d0 += 64 * V * P) {
        double acc[P][V], S = sp;
        const int pieces = (to - d0 + 64 * V - 1) / (64 * V);           // of this block that hold anything, the same in every lane
        unsigned long long h = hits;
        bool first = true;
        do {
            const int j1 = h ? (int)__builtin_ctzll(h) : -1;
            h &= h - 1;
            const int j2 = h ? (int)__builtin_ctzll(h) : -1;
            h &= h - 1;
            const __amdgpu_buffer_rsrc_t r1 = lz_row(row_of<T>(x, ov, b, rid[j1 < 0 ? 0 : 2 * j1], g, D), D, j1 >= 0),
                                         r2 = lz_row(row_of<T>(x, ov, b, rid[j2 < 0 ? 0 : 2 * j2], g, D), D, j2 >= 0);
            lz_u32x4 vp[P], v1[P], v2[P];
#pragma unroll
            for (int u = 0; u < P; ++u) {
                if (u >= pieces) continue;
                const int off = (d0 + (u * 64 + lane) * V) * (int)sizeof(T);
                if (first) vp[u] = lz_load(rp, off);
                v1[u] = lz_load(r1, off);
                if (j2 >= 0) v2[u] = lz_load(r2, off);
            }
            const double s1 = j1 >= 0 ? (double)sz[2 * j1] : 0.0, s2 = j2 >= 0 ? (double)sz[2 * j2] : 0.0;
#pragma unroll
            for (int u = 0; u < P; ++u) {
                if (u >= pieces) continue;
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    if (first) acc[u][e] = sp * io::at(vp[u], e);
                    if (j1 >= 0) acc[u][e] += s1 * io::at(v1[u], e);
                    if (j2 >= 0) acc[u][e] += s2 * io::at(v2[u], e);
                }
            }
            S = (S + s1) + s2;
            first = false;
        } while (h);
        const double inv = 1.0 / S;
#pragma unroll
        for (int u = 0; u < P; ++u) {
            const int d = d0 + (u * 64 + lane) * V;
            if (d >= to) continue;
            lazy_round_store<T>(acc[u], S, inv, o + d);
        }
    }
}

}  // namespace

}  // namespace luvc
