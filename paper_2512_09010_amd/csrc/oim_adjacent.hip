// OIM (paper Section 3.2, Algorithm 1) with the adjacent destinations as candidates, for schedules that take few tokens
// out of a line per pass (merge number 2): one launch per pass on grids of row ids (see oim_wide_lazy.hip: the tokens
// are moved once, after the last pass).
//
// One workgroup per line of at most 128 tokens.  A wavefront fetches four consecutive tokens and the one after them, all
// in flight together, and forms their squared norms and neighbour products in fp64 at once: with two candidates per
// source there is little to save by screening, and a pass needs no second look at the tokens (screened in fp32, a line in a
// hundred had to be repeated in fp64, which is a line in nearly every launch: no quicker).  Then the cosines of the
// sources (one wavefront, a source per lane), the m best of them (few: picked one by one by that wavefront; else a source
// per ballot), the layout of the next grid and the size-weighted means of the destinations that take sources in, written
// to overlay rows.
//
// Bound: latency.  A pass reads its tokens once, but a line is a chain of memory trips - ids, tokens, merged rows - with
// the decisions between them; as many wavefronts as a line has groups of four tokens share it, so that each trip is made once.
// 12 x 32 x 32 x 1024 bf16, three operations of (W,2),(H,2): 160 us as three launches per pass (norms and products,
// decisions, a merge that rewrites the whole grid), 62 as one with two pieces of a row per lane where a row has no more, the ids of a
// wavefront's tokens asked for together (one behind the other, each a branch and a wait, they were most of the 1.2 us before its first
// token), a root per token (63.0 with one in every cosine) and a merged row shared by two wavefronts (66.4 without).
// Narrow rows were slower than the three launches while every row took three pieces: 32 x 64 x 64 x 384 bf16, (W,2): 92 us by
// pass, 130, 78 then, of which the copy of the output rows went from 63 to 31.
#include "common.hpp"
#include "oim.hpp"
#include "oim_lazy.hpp"
#include "oim_sum64.hpp"

namespace luvc {

constexpr int kAdjTok = 4;                       // consecutive tokens of a wavefront

// P, PM: 16-byte pieces of a row per lane at a time, for the decisions and for the merged rows.  A piece past the row's end
// costs its products all the same, and the registers of fewer pieces leave room for a second line on a compute unit.
// HOLD: a line has at most four tokens per wavefront, a row at most P pieces, and the decisions are taken on the tokens:
// they stay in registers until the end of the pass, and a wavefront merges the two destinations among its own.  Taken where
// the lines come in several rounds: 8 x 64 x 64 x 1280 bf16, merge number 2 three times, 158.1 us a call without, 153.3 with;
// 32 x 64 x 64 x 384, once, 117.8, 112.8.  A launch that is one round long is no quicker for the trip it saves: 12 x 32 x 32 x 1024
// three times 62.3, 67.8; 1 x 100 x 24 x 1408 64.9, 67.6.
template <typename T, int P, int PM, bool HOLD>
__global__ void __launch_bounds__(1024)
oim_adjacent_line(const T* __restrict__ x, T* ov, const T* __restrict__ xk /* metric [.., Dk] the decisions are taken on, or null: x */,
                  T* ovk /* its overlay */, int Dk, const int32_t* __restrict__ idx_in /* null: identity */,
                  const int32_t* __restrict__ sizes_in /* null: ones */, const int32_t* __restrict__ kept_in /* null: identity */,
                  LazyGeom g, int32_t* __restrict__ idx_out, int32_t* __restrict__ sizes_out, int32_t* __restrict__ kept_out /* or null */,
                  int32_t* __restrict__ pass_map /* or null */)
{
    using io = lz_io<T>;
    constexpr int V = io::V;
    __shared__ double nrm2[kLazyMaxLen + 4], dnx[kLazyMaxLen + 4];     // squared norm, then norm; product with the next token of the line
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

    // Lines in several rounds: those that ask for their tokens come before those that decide and merge (8 x 64 x 64 x 1280 bf16, merge number 2
    // three times, 154.6 -> 152.9 us; in one round 12 x 32 x 32 x 1024 would go from 62.5 to 62.7).
    if constexpr (HOLD) __builtin_amdgcn_s_setprio(2);
    // What the line shares comes beside the tokens, one to a thread (there are 16 per token, or 1024), and is written to LDS behind the
    // sums.  (The ids of a wavefront's tokens one to a lane as well, instead of by scalar loads: 12 x 32 x 32 x 1024 67.6 us for 65.5.)
    int line_id = 0, line_size = 1;
    if (tid < len) {
        line_id = in_flat(tid);
        if (sizes_in) line_size = sizes_in[img + line_id];
        if (idx_in) line_id = idx_in[img + line_id];
    }
    // ---- squared norms and neighbour products
    lz_u32x4 tok[kAdjTok + 1][P];                // tokens p0 .. p0 + 4 of the line, P pieces of each
    for (int p0 = wave * kAdjTok; p0 < len; p0 += NW * kAdjTok) {
        int id[kAdjTok + 1];                     // asked for together
#pragma unroll
        for (int i = 0; i <= kAdjTok; ++i) id[i] = in_flat(p0 + i < len ? p0 + i : len - 1);
        if (idx_in)
#pragma unroll
            for (int i = 0; i <= kAdjTok; ++i) id[i] = idx_in[img + id[i]];
        __amdgpu_buffer_rsrc_t r[kAdjTok + 1];
#pragma unroll
        for (int i = 0; i <= kAdjTok; ++i) r[i] = lz_row(row_of<T>(dx, dov, b, id[i], g, dD), dD, p0 + i < len);
        double s[2 * kAdjTok];
#pragma unroll
        for (int i = 0; i < 2 * kAdjTok; ++i) s[i] = 0.0;
        for (int d0 = 0; d0 < (HOLD ? 1 : dD); d0 += 64 * V * P) {
#pragma unroll
            for (int i = 0; i <= kAdjTok; ++i)
#pragma unroll
                for (int u = 0; u < P; ++u) tok[i][u] = lz_load(r[i], (d0 + (u * 64 + lane) * V) * (int)sizeof(T));
#pragma unroll
            for (int u = 0; u < P; ++u)
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    double a = io::at(tok[0][u], e);
#pragma unroll
                    for (int i = 0; i < kAdjTok; ++i) {
                        const double c = io::at(tok[i + 1][u], e);
                        s[i] = fma(a, a, s[i]);
                        s[kAdjTok + i] = fma(a, c, s[kAdjTok + i]);
                        a = c;
                    }
                }
        }
        static_assert(kAdjTok == 4, "eight sums, one to a lane");
        const double sum = wave_totals64(s, lane);
        if (lane < 2 * kAdjTok) (lane < kAdjTok ? nrm2 : dnx)[p0 + (lane & (kAdjTok - 1))] = sum;
    }
    if constexpr (HOLD) __builtin_amdgcn_s_setprio(0);
    if (tid < len) {
        rid[tid] = line_id;
        sz[tid] = line_size;
    }
    __syncthreads();
    // ---- cosine of every source with its two neighbours (equal: the lower position)
    // Up to three sources are picked one by one by this wavefront; more are ranked by all, since every pick is a step behind the last:
    // 32 x 64 x 64 x 384 bf16, m out of both axes, picked and ranked, when the two were compared: m = 2 116.6 us, 119; 3 120.2, 122.0; 4 123.3,
    // 122.8; 10 135.0, 122.5 (as it is taken, now 113, 116, 119, 119).
    const bool few = g.m <= 3;
    if (wave == 0) {
        const bool is_src = lane < n_src;
        const int a = is_src ? 2 * lane : 0;
        const bool hl = a >= 1, hr = a + 1 < len;
        for (int p = lane; p < len; p += 64) {               // a root per token: each is in the cosines of up to three sources
            const double n = sqrt(nrm2[p]);
            nrm2[p] = n < 1e-12 ? 1e-12 : n;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const double na = nrm2[a];
        const double sl = hl ? dnx[a - 1] / (na * nrm2[a - 1]) : 0.0, sr = hr ? dnx[a] / (na * nrm2[a + 1]) : 0.0;
        const bool left = hl && (!hr || !(sr > sl));
        double best = left ? sl : sr;
        best = best == best ? best : -INFINITY;              // NaN: last, so that exactly m sources leave the line whatever the tokens hold
        if (few) {
            // m times the highest of those left (equal: the lower position)
            unsigned long long out = 0ull;
            for (int i = 0; i < g.m; ++i) {
                const bool in = is_src && !((out >> lane) & 1ull);
                const double top = wave_max64(in ? best : -INFINITY);
                out |= 1ull << __builtin_ctzll(__ballot(in && best == top));
            }
            if (is_src) gone[lane] = (int)((out >> lane) & 1ull);
        } else if (is_src) score[lane] = best;
        if (is_src) side[lane] = hl || hr ? (left ? 0 : 1) : -1;
    }
    __syncthreads();
    if (!few) {                                  // the m best (equal: the lower position): a source per ballot of those that beat it
        const double mine = lane < n_src ? score[lane] : 0.0;
        for (int j = wave; j < n_src; j += NW) {
            const double s = score[j];
            const int rank = __popcll(__ballot(lane < n_src && (mine > s || (mine == s && lane < j))));
            if (lane == 0) gone[j] = g.m == n_src || rank < g.m;
        }
        __syncthreads();
    }
    // ---- layout of the next grid: lane k of every wavefront looks at source 2 k and destination 2 k + 1
    const unsigned long long below = (1ull << lane) - 1ull;
    const bool sgone = lane < n_src && gone[lane];
    const int sside = lane < n_src ? side[lane] : -1;
    const unsigned long long m_gone = __ballot(sgone), m_right = __ballot(sgone && sside == 1), m_left = __ballot(sgone && sside == 0);
    const unsigned long long from_prev = m_right, from_next = m_left >> 1;       // destinations that take in source 2 k, source 2 k + 2
    const LazyLine ln = {m_gone, from_prev | from_next};
    auto slot = [&](int p) { return out_flat(lazy_slot(ln, p)); };
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
        idx_out[img_out + of] = ((ln.takes >> lane) & 1ull) ? g.n0 + g.ov_base + line * g.per_line + __popcll(ln.takes & below) : rid[p];
        sizes_out[img_out + of] = taken(lane);
        if (kept_out) kept_out[img_out + of] = kept_in ? kept_in[img + f] : f;
        if (pass_map) pass_map[img + f] = of;
    }
    if constexpr (HOLD) {
        // ---- the destinations that take sources in: size-weighted mean in fp64, destination first, rounded once
        // (the widened tokens of the sums are not kept for it: fp64 copies of whole tokens do not fit)
#pragma unroll
        for (int i = 0; i <= kAdjTok; ++i)
#pragma unroll
            for (int u = 0; u < P; ++u) asm volatile("" : "+v"(tok[i][u]));
#pragma unroll
        for (int o = 0; o < kAdjTok / 2; ++o) {
            const int p = wave * kAdjTok + 2 * o + 1, k = p >> 1;
            if (p >= len || !((ln.takes >> k) & 1ull)) continue;
            const bool prev = (from_prev >> k) & 1ull, next = (from_next >> k) & 1ull;
            const double sp = (double)sz[p], s1 = prev ? (double)sz[p - 1] : 0.0, s2 = next ? (double)sz[p + 1] : 0.0;
            T* to = ov + (b * g.cap + g.ov_base + line * g.per_line + __popcll(ln.takes & ((1ull << k) - 1ull))) * g.D;
            const double S = (sp + s1) + s2, inv = 1.0 / S;
#pragma unroll
            for (int u = 0; u < P; ++u) {
                const int d = (u * 64 + lane) * V;
                if (d >= g.D) continue;
                double acc[V];
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    acc[e] = sp * io::at(tok[2 * o + 1][u], e);
                    if (prev) acc[e] += s1 * io::at(tok[2 * o][u], e);
                    if (next) acc[e] += s2 * io::at(tok[2 * o + 2][u], e);
                }
                lazy_round_store<T>(acc, S, inv, to + d);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    } else {
        // ---- the same, a wavefront per destination and tensor; one or two destinations: up to four per row, of a piece and more each.
        // (us of a call without and with it, merge number 2: 12 x 32 x 32 x 1024 bf16 three times 66.4, 62.2; 2 x 64 x 64 x 1280 twice 49.1,
        // 47.7.  When it came in, of three and more rows the shares stand in each other's way: m = 3 52.1, 53.4; 4 53.1, 53.5; 6 57.1, 57.8.)
        const int n_abs = __popcll(ln.takes), n_rows = (xk ? 2 : 1) * n_abs;
        int split = 0;                           // 2^split wavefronts
        while ((64 * V << split) < g.D && (n_abs << (split + 1)) <= 4 && (n_rows << (split + 1)) <= NW) ++split;
        for (int kp = wave; kp < n_rows << split; kp += NW) {
            const int kk = kp >> split, part = kp - (kk << split);
            const bool on_metric = kk >= n_abs;
            const int at = on_metric ? kk - n_abs : kk;
            unsigned long long left = ln.takes;
            for (int i = 0; i < at; ++i) left &= left - 1;
            const int k = (int)__builtin_ctzll(left);
            const unsigned long long hits = ((from_prev >> k) & 1ull) << k | (((from_next >> k) & 1ull) << k) << 1;
            T* mov = on_metric ? ovk : ov;
            const int mD = on_metric ? Dk : g.D;
            const int share = ((mD - 1) / (64 * V) >> split) + 1, from = part * share * 64 * V, to = from + share * 64 * V < mD ? from + share * 64 * V : mD;
            if (from < to)
                lazy_merge<T, PM>(on_metric ? xk : x, mov, g, mD, b, rid, sz, k, hits, mov + (b * g.cap + g.ov_base + line * g.per_line + at) * mD, lane, from, to);
        }
    }
}

// ------------------------------------------------------------------ host side
static int adjacent_waves(int len)
{
    const int waves = (len + kAdjTok - 1) / kAdjTok;
    return waves > 16 ? 16 : waves;
}

// Is a schedule of adjacent matching quicker on grids of row ids than pass by pass (halving kernels, or norms, decisions and a
// merge that moves the whole grid)?  us of either way, fitted to 190 schedules on twelve grids of 2 to 430 MB, one to six
// passes of m = 2 up to every source (off by 15 %, rms).  What counts is bytes (MB of a grid) and, where the lines leave
// compute units idle, the rounds in which the wavefronts of a line sum its tokens and merge its destinations.  Both ways
// measured: 8x64x64x1280 bf16 (W,2),(H,2) three times 341 us pass by pass, 153 on ids; (W,31) 60, 59; 32x64x64x384 (W,2) 90, 72;
// (W,32),(H,16) 114, 105; 2x30x120x1152 (W,2) 23, 20; (W,59) 25, 37; (W,60),(H,7) 37, 46; 1x12x100x640 (W,50),(H,3) 26, 30.
// The fit is older than the kernels, which take up to 9 % less on ids since.  The line has not moved with them, since the fit's own
// error is larger: with by_ids 5 % lower, 3 of 816 drawn schedules go to ids, at 0.82, 0.86 and 1.08 of the time; 10 % lower 7, at 0.82 to 1.08;
// 6 % higher 21 leave them, at 0.81 to 1.28, most above 1.07.
// Decided on keys, pass by pass is two more launches and ids always win: (W,31) 65 and 63, (W,32),(H,16) 109 and 80.
bool oim_adjacent_pays(const int* h, const int* w, const luvc_oim_pass* passes, int n, int B, int D, luvc_dtype dt)
{
    const double mb = (double)B * D * (dt == LUVC_F32 ? 4 : 2) * 1e-6;
    auto halves = [&](int i) { return passes[i].m == ((passes[i].axis ? w[i] : h[i]) + 1) / 2; };
    auto size = [&](int i) { return mb * h[i] * w[i]; };                        // MB before pass i
    double by_pass = 0.0, by_ids = 2.5 + 0.30 * size(n);
    int steps = 0, last_axis = -1;                                              // axis of a halving that may still find a partner
    for (int i = 0; i < n; ++i) {
        const int axis = passes[i].axis, m = passes[i].m, len = axis ? w[i] : h[i], n_src = (len + 1) / 2, n_dst = len / 2;
        if (m == 0) continue;
        const int64_t lines = (int64_t)B * (axis ? h[i] : w[i]);
        const int waves = adjacent_waves(len), sums = (len + kAdjTok * waves - 1) / (kAdjTok * waves);
        const int rounds = ((m < n_dst ? m : n_dst) + waves - 1) / waves;
        by_ids += 3.9 + 0.18 * size(i) + 0.24 * size(i) * m / n_src + 2.8 * sums + (lines <= 192 ? 3.6 * (rounds - 1) : 0.0);
        if (halves(i) && last_axis >= 0 && last_axis != axis) {                 // the second of a pair: one launch for both
            by_pass += 0.20 * (size(i + 1) - size(i));
            last_axis = -1;
            continue;
        }
        by_pass += halves(i) ? 6.3 + 0.20 * (size(i) + size(i + 1)) : 15.7 + 0.54 * size(i);
        last_axis = halves(i) ? axis : -1;
        ++steps;
    }
    return by_ids <= by_pass + (steps > 1 ? 3.9 : 0.0);
}

template <typename T>
static luvc_status run_adjacent(const T* x, T* ov, const T* xk, T* ovk, int Dk, const int32_t* idx_in, const int32_t* sizes_in, const int32_t* kept_in,
                                int B, const LazyGeom& g, int32_t* idx_out, int32_t* sizes_out, int32_t* kept_out, int32_t* pass_map, hipStream_t st)
{
    const int len = g.axis ? g.w : g.h, nlines = g.axis ? g.h : g.w;
    const int waves = adjacent_waves(len);
    auto pieces = [](int D) { return (D + 64 * lz_io<T>::V - 1) / (64 * lz_io<T>::V); };
    const int p = pieces(xk ? Dk : g.D), pm = pieces(xk && Dk > g.D ? Dk : g.D);
#define LUVC_ADJ(P, PM, HOLD) LUVC_LAUNCH("oim_adjacent_line", (oim_adjacent_line<T, P, PM, HOLD>), dim3((unsigned)(B * nlines)), dim3(64 * waves), 0, st, x, ov, xk, ovk, Dk, \
                                      idx_in, sizes_in, kept_in, g, idx_out, sizes_out, kept_out, pass_map)
    // More wavefronts than 16 per compute unit: several rounds of lines.  bf16 rows of two or three pieces on lines of many wavefronts
    // only where a line merges one or two: the merges of a wavefront wait for one another there (64 tokens of 1280, m = 4 out of
    // both axes of 8 x 64 x 64: 73.1 us held, 71.6 not; 640, 5 x 62 x 63, m = 8: 46.7, 45.0; but 48 of 1024, 15 x 48 x 48, m = 8: 63.2, 68.0).
    const bool merges_wait = sizeof(T) == 2 && p * waves > 24 && g.m > 2;
    if (!xk && len <= kAdjTok * waves && p <= 3 && (int64_t)B * nlines * waves > 4096 && !merges_wait) {
        if (p == 1) LUVC_ADJ(1, 1, true);
        else if (p == 2) LUVC_ADJ(2, 2, true);
        else LUVC_ADJ(3, 3, true);
    }
    else if (p == 1 && pm == 1) LUVC_ADJ(1, 1, false);
    else if (p == 1) LUVC_ADJ(1, kLzPieces, false);
    else if (p == 2 && pm == 2) LUVC_ADJ(2, 2, false);
    else if (p == 2) LUVC_ADJ(2, kLzPieces, false);
    else LUVC_ADJ(kLzPieces, kLzPieces, false);
#undef LUVC_ADJ
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
