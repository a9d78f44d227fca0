// OIM (paper Section 3.2, Algorithm 1) - one launch for a PAIR of halving passes on orthogonal
// axes (row merge then column merge, or the other way round): H x W -> H/2 x W/2 without the
// intermediate grid ever leaving the chip.
//
// Work split.  A workgroup owns one line position j of the first pass (output column j for a
// row-then-column pair) and a run of output slots of the second pass.  Each wavefront owns four (on small
// grids two) consecutive lines of the first pass: for each of them it loads destination b = 2j+1, its two
// sources a = 2j, c = 2j+2 and the two destinations beyond them (l = 2j-1, r = 2j+3, needed only
// to decide where a and c go), forms the first-pass token, rounds it to the storage type - the
// second pass must read what a separate launch would have read from memory - and keeps it packed
// in registers.  The four intermediate tokens of a wavefront are two destinations of the second
// pass with the sources between them (two: one destination and the source above it); the one token a wavefront needs from its neighbour (the
// first token of the next wavefront) goes through LDS, as do the norms and neighbour dot
// products every wavefront needs from the tokens around its own.  A workgroup that owns only
// part of a long line recomputes the three intermediate tokens just outside its run.
//
// A token in registers is NQ 16-byte pieces per lane plus a 4- or 8-byte tail piece, so that a
// token of 1280 bf16 values costs 10 registers per lane, not 12; buffer resources bound every
// piece, so lanes past the end of a token read zeros and write nothing.
//
// Decisions are fp64 decisions reached in two steps, as in the single-pass kernel: a screening
// sweep in fp32 with a rigorous error bound, and a repeat in fp64 of whatever is closer than the
// bound.  In the first pass the repeat is local to a wavefront; in the second pass the sums of a
// decision may live in two wavefronts, which then both put theirs in LDS.  A source shared by
// two workgroups is decided from the same bits by the same expressions in both.
//
// Bound: instructions.  Loads alone, in this order, take 14 us for 8 x 64 x 64 x 1280 bf16 (84 MB); a row of a wavefront is about 300
// vector instructions beside its 15 loads (90 the products, 60 the totals and the verdicts, the rest the merge), and without the
// products of the first pass a call takes 24 us of 29.  So all decisions of a row are worked out side by side, a sum per lane
// (`wave_totals32`), rather than one after the other on values all lanes hold: 32 x 64 x 64 x 384 54.2 -> 49.4 us, 8 x 64 x 64 x 1280
// 30.5 -> 29.2, 80 x 24 x 24 x 1024 35.0 -> 33.7, fp32 40 x 24 x 24 x 768 23.2 -> 22.4.  (The same totals by the matrix cores, nine
// 16 x 16 x 4 products against unit columns, are fewer instructions and slower, 58: they take the vector unit's time.  The next
// row's tokens asked for before a row is merged: 57, 31.3 and, for want of registers, 49.)
// The older wavefronts of a workgroup get their tokens first, the youngest as they come to 20 us.  A wavefront therefore
// waits only for its two neighbours (`stage`), not at barriers for all: the merges and stores of the older ones run
// while the younger ones' tokens are on their way: a call of 34.5 us took 30.5 (32 x 64 x 64 x 384 61.5 -> 54.8; 80 x 24 x 24 x
// 1024, workgroups of 6 wavefronts, 35.9 -> 34.7; 128 x 16 x 16 x 1152, of 4, the same).  Tokens of a few hundred bytes, which come in
// together, pay for the words: 16 x 17 x 15 x 128 bf16 6.9 -> 7.4, 80 x 24 x 24 x 256 19.5 -> 20.1.
//
// The merge is the size-weighted mean evaluated in fp64 in position order and rounded once.  One
// case needs no fp64: bf16 storage, one absorbed source, equal sizes.  Then the mean is (b + x) / 2
// and the fp32 sum, halved and rounded to bf16 by the hardware conversion, is the correctly rounded
// result: either the sum is exact in fp32 (exponents at most 15 apart), or the smaller term is below
// 2^-15 of the larger, whose half lies on the bf16 grid at least 2^-10 (relative) away from every
// rounding boundary - too far for the smaller term or the fp32 rounding to matter.
#include "oim_pair_tok.hpp"

namespace luvc {

// The items of a launch.  One item, the common case, has a kernel of its own: an argument list with room for all of them is
// 2 KB and costs a launch 0.3 .. 0.7 us (8 x 64 x 64 x 1280 bf16 34.7 -> 34.0, 2 x 112 x 112 x 1280 and its two smaller
// grids 59.8 -> 58.3).
template <int MOST>
struct PairTable : StepMore<MOST> {
    int n;
    struct { PairGeom g; StepAt at; } it[MOST];
};

// Tokens of at most 8 words per lane (1 KB in bf16) are compiled for six wavefronts per SIMD (80 registers, a few spilled
// in the fp64 repeat): on batches of small grids a workgroup is 6 wavefronts, and four workgroups per compute unit instead
// of three put 80 x 24 x 24 grids (960 workgroups) on the chip in one round - measured 36.8 -> 33.9 us.  The same
// hint on wider tokens (96 instead of 103 registers) measured slower on every workload and is not given.
template <typename T, int NQ, int TW, int NW, int R /* first-pass lines of a wavefront */, int MOST>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu((4 * NQ + TW <= 8 && NW == 16) ? 6 : 1)))
oim_halve_pair(const T* __restrict__ x, const int32_t* __restrict__ sizes_in, const int32_t* __restrict__ kept_prev, const StepOutOf<MOST> out, const PairTable<MOST> tab)
{
    using TokT = Tok<NQ, TW>;
    constexpr int N = TokT::N;
    constexpr int kRows = R * NW + 8;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    uint32_t* lds_tok = reinterpret_cast<uint32_t*>(lds_raw);     // [live waves][N][64]: first token of each wave
    __shared__ float inv32[kRows], dt32[kRows];                   // 1/|T[r]|, <T[r], T[r+1]> of the intermediate tokens
    __shared__ double inv64[kRows], dt64[kRows];
    __shared__ int szl[kRows];
    // What a wavefront has written: 1 its first token, 2 inv32, dt32 and szl, 3 (kSums) inv64 and dt64; or, where it needs no fp64,
    // kSettled and its verdicts (kFirstUp: of its first source, kNextUp: of the one after its last row).  Every wavefront with rows gets
    // to 3 or beyond and waits for no more than a 2 before, so every wait ends, whatever the verdicts.
    __shared__ int stage[NW];
    constexpr int kSums = 3, kSettled = 16, kFirstUp = 4, kNextUp = 8;
    // Of the wavefronts of a SIMD the oldest comes first, with merges of the second pass before younger ones that have tokens to ask for.
    // The merges, which nobody waits for, come last instead; the exchange, which neighbours wait for, first.  us of the cases with the oldest
    // first and so, with the score: 2 x 112 x 112 x 1280 three times 61.6, 58.9; 128 x 16 x 16 x 1152 69.1, 68.2; 8 x 64 x 64 x 1280 68.0, 67.0;
    // 80 x 24 x 24 x 1024 81.0, 80.0.
    // Of the first pass the earlier rows come first where a token has more than 8 words, which was never slower.  us of a merge without and
    // with it: 8 x 64 x 64 x 1152 25.5, 24.9; x 1280 23.6, 23.4; x 1408 34.3, 34.2; 128 x 16 x 16 x 1152 24.8, 24.3; 80 x 24 x 24 x 1280 45.0,
    // 44.5; 32 x 32 x 32 x 640 fp32 26.1, 25.5; 2 x 112 x 112 x 1280, 4 x 48 x 48 x 1408 fp32 the same.  Narrower tokens gain on some grids
    // (128 x 16 x 16 x 384 13.8, 12.9; x 1024 22.6, 22.1; 8 x 64 x 64 x 384 13.9, 13.4) and lose on others (80 x 24 x 24 x 768 26.4, 26.9; x 1024
    // 30.2, 30.8; 8 x 64 x 64 x 512 fp32 21.5, 21.8); what decides there is not known, and they go without.
    constexpr bool kRowsTakeTurns = N > 8;
    __builtin_amdgcn_s_setprio(1);

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned item = xcd_contiguous(blockIdx.x, gridDim.x);
    PairGeom g = tab.it[0].g;
    StepAt at = tab.it[0].at;
    if constexpr (MOST > 1) {
        const int ent = run_of(tab.n, item, [&](int i) { return tab.it[i].at.wg0; });
        g = tab.it[ent].g;
        at = tab.it[ent].at;
        if (at.src) {
            const StepIn& from = tab.from[at.src - 1];
            x = (const T*)from.x;
            sizes_in = from.sizes;
            kept_prev = from.kept;
        }
    }
    item -= at.wg0;
    const int j = item % g.nd1;
    const int seg = (item / g.nd1) % g.segs;
    const int b = item / (g.nd1 * g.segs);
    const int u0 = seg * g.seg_out;
    const int nseg = min(g.seg_out, g.nd2 - u0);                  // second-pass outputs of this workgroup
    const int row_base = 2 * u0;
    const int row_lo = u0 > 0 ? row_base - 1 : row_base;          // one intermediate row above the run decides its first source
    const int row_end = min(g.L2 - 1, row_base + 2 * nseg + 1);   // two below decide its last source (or close an odd line)
    const int nwm = (row_end - row_base + R) / R;                 // wavefronts with rows of the run
    const bool is_main = w < nwm;
    const bool is_halo = u0 > 0 && w == nwm;                      // holds row_base - 1 as ITS LAST row
    const bool active = is_main || is_halo;
    const int r0 = is_halo ? row_base - R : row_base + R * w;
    const int rr0 = r0 - row_base + 1;                            // LDS index of row r0 (negative only for the halo wave's unused rows)
    // Error bound of the screening, in units of u = 2^-24.  A sum takes at most E = R + 6 roundings of
    // relative size u on partial sums bounded by the sum of the magnitudes of its terms (R per lane: two
    // per packed bf16 product pair, one per fp32 product; six reduction steps); against |a||b| that is E u
    // on a dot product and E u on each squared norm, i.e. (E + 4) u on the two reciprocal norms together
    // (hardware reciprocal square root: 1 ulp each), plus two products: 2 E + 6 per cosine, 4 E + 13 on
    // the difference of two.  tau is 1.5 times that.  Each step of the packed bf16 dot product is taken as one or two
    // roundings to nearest of the exact value (tests/test_gpu_oim.py pins the instruction's sums against fp64);
    // underflow and overflow are kept out by inv_norm32().
    constexpr int kE = N * (words<T>::per == 2 ? 2 : 1) + 6;
    const float tau = (float)(6 * kE + 20) * 5.9604645e-8f;
    const int tok_bytes = g.D * (int)sizeof(T);
    if (threadIdx.x < NW) stage[threadIdx.x] = 0;
    auto reached = [&](int v) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        if (lane == 0) __hip_atomic_store(stage + w, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // A wavefront that waits has a high priority, yet cannot keep the one it waits for from running: each look is a trip to LDS that it
    // stalls on, and the SIMD issues for the others meanwhile.
    auto wait_for = [&](int other, int v) {
        int word;
        do word = __builtin_amdgcn_readfirstlane(__hip_atomic_load(stage + other, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
        while (word < v);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        return word;
    };

    // ------------------------------------------------------------------ first pass: R intermediate tokens
    const int pa = 2 * j, pb = pa + 1, pc = pa + 2;
    const bool has_l = j > 0, has_c = pc < g.L1, has_r = pc + 1 < g.L1;
    const int64_t img_in = at.in_off + (int64_t)b * g.n_in;
    const scalar_words sizes = as_scalars(sizes_in);
    TokT Tk[R];
    int sk[R];
    unsigned took_a = 0, took_c = 0;                              // bit k: row k absorbed its a / its c
    // the rows unrolled: the compiler renames tokens instead of moving 10 registers per token and row
    // (measured: 35.3 -> 34.2 us on 8 x 64 x 64 x 1280 bf16)
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int r = r0 + k;
        TokT& Tn = Tk[k];
        if constexpr (kRowsTakeTurns) {
            if (k < R / 2) __builtin_amdgcn_s_setprio(2);
            else __builtin_amdgcn_s_setprio(1);
        }
        TokT A, Bt, C, Lt, Rt;
        int sn = 0, sa_in = 1, sb = 1, sc_in = 1;
        const bool there = active && r >= row_lo && r <= row_end;
        if (there) {
            const int64_t t0 = img_in + (int64_t)r * g.sB;        // token of position 0 on this line
            const int64_t ta = t0 + (int64_t)pa * g.sA, tb = t0 + (int64_t)pb * g.sA, tc = t0 + (int64_t)pc * g.sA;
            load_tok(A, x + ta * g.D, tok_bytes, lane);
            load_tok(Bt, x + tb * g.D, tok_bytes, lane);
            load_tok(C, x + (has_c ? tc : tb) * g.D, tok_bytes, lane, has_c);
            load_tok(Lt, x + (has_l ? ta - g.sA : tb) * g.D, tok_bytes, lane, has_l);
            load_tok(Rt, x + (has_r ? tc + g.sA : tb) * g.D, tok_bytes, lane, has_r);
            sb = sizes_in ? sizes[tb] : 1;
            sa_in = sizes_in ? sizes[ta] : 1;
            sc_in = (sizes_in && has_c) ? sizes[tc] : 1;
        }
        if (k == 0) {                                             // `stage` is cleared for everyone before it is used; the first tokens are on their way
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        }
        if (there) {
            // screening: every sum is formed lower position first, so the sum two workgroups share has the same bits
            // (tokens that are not there were loaded as zeros: their sums are zero and never looked at)
            const float sm[9] = {dot32_lane<T>(Lt, Lt), dot32_lane<T>(A, A), dot32_lane<T>(Bt, Bt), dot32_lane<T>(C, C), dot32_lane<T>(Rt, Rt),
                                 dot32_lane<T>(Lt, A), dot32_lane<T>(A, Bt), dot32_lane<T>(Bt, C), dot32_lane<T>(C, Rt)};
            // lanes 0 .. 4: the squared norms, lanes 5 .. 8: the products of neighbours; lane i < 4 then works on token i and the next,
            // of which the odd one is the source; lane 0 has the verdict on a, lane 2 the one on c
            const float tot = wave_totals32(sm, lane);
            const float inv = inv_norm32(tot), inv_next = from_lane_above<1>(inv);
            const bool odd = lane & 1;
            const float cosine = screen_cosine(from_lane_above<5>(tot), odd ? inv : inv_next, odd ? inv_next : inv);
            const Verdicts sure = screen_verdicts(cosine, from_lane_above<1>(cosine), tau);
            int va = -1, vc = -1;
            if (has_l) va = (int)(sure.left & 1u) - (int)(sure.right & 1u);
            if (has_c) vc = has_r ? (int)(sure.left >> 2 & 1u) - (int)(sure.right >> 2 & 1u) : 1;
            bool a_left = va > 0, c_left = vc > 0;
            if (va == 0 || vc == 0) {                             // too close for fp32: the fp64 cosines decide
                double n[5], d[4];
                chain_sums64<T>(Lt, A, Bt, C, Rt, n, d);
                const double jb = inv_norm64(n[2]);
                if (va == 0) a_left = source_goes_left(true, true, inv_norm64(n[1]), d[0], inv_norm64(n[0]), d[1], jb);
                if (vc == 0) c_left = source_goes_left(true, true, inv_norm64(n[3]), d[2], jb, d[3], inv_norm64(n[4]));
            }
            const bool take_a = !a_left, take_c = has_c && c_left;
            const int sa = take_a ? sa_in : 0, sc = take_c ? sc_in : 0;
            sn = sb + sa + sc;
            if (take_a) took_a |= 1u << k;
            if (take_c) took_c |= 1u << k;
            if (!take_a && !take_c) Tn = Bt;
            else merge_tok<T>(Tn, Bt, A, C, sb, sa, sc);
        } else {
            zero_tok(Tn);
        }
        sk[k] = sn;
    }

    if (!active) return;

    // ------------------------------------------------------------------ second pass: exchange
    __builtin_amdgcn_s_setprio(3);
    if (is_main) {
#pragma unroll
        for (int i = 0; i < N; ++i) lds_tok[(w * N + i) * 64 + lane] = Tk[0].w[i];
    }
    reached(1);
    const int above = is_halo ? -1 : w > 0 ? w - 1 : u0 > 0 ? nwm : -1, below = is_halo ? 0 : w + 1;
    TokT Tx;                                                      // the token after the last: first token of the next wavefront
    if (r0 + R <= row_end) {
        wait_for(below, 1);
#pragma unroll
        for (int i = 0; i < N; ++i) Tx.w[i] = lds_tok[(below * N + i) * 64 + lane];
    } else {
        zero_tok(Tx);
    }
    {
        float sm[8];                                              // squared norms (lanes 0 .. 3), products with the token below (lanes 4 .. 7)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            sm[k] = k < R ? dot32_lane<T>(Tk[k < R ? k : 0], Tk[k < R ? k : 0]) : 0.f;
            sm[4 + k] = k < R ? dot32_lane<T>(Tk[k < R ? k : 0], k + 1 < R ? Tk[k + 1 < R ? k + 1 : 0] : Tx) : 0.f;
        }
        const float n2 = wave_totals32(sm, lane), dn = from_lane_above<4>(n2);
        if (lane < R) {
            const int k = lane, r = r0 + k;
            if (r >= row_lo && r <= row_end) {
                int sz = sk[0];
#pragma unroll
                for (int i = 1; i < R; ++i)
                    if (k == i) sz = sk[i];
                inv32[rr0 + k] = inv_norm32(n2);
                dt32[rr0 + k] = dn;
                szl[rr0 + k] = sz;
            }
        }
    }
    reached(2);
    const bool e2 = R > 2 && is_main && r0 + 2 <= row_end, e4 = r0 + R <= row_end;
    if (above >= 0) wait_for(above, 2);
    if (e4) wait_for(below, 2);
    // a source at intermediate row r0 + lane (LDS index q) goes UP (to the lower position) unless the row below is strictly more similar
    const int q = rr0 + (lane < R ? lane : R), qc = q > 0 ? q : 0, qm = q > 0 ? q - 1 : 0;        // (of the halo only the row after its last)
    const float own = inv32[qc];
    const Verdicts sure = screen_verdicts(screen_cosine(dt32[qm], own, inv32[qm]), screen_cosine(dt32[qc], own, inv32[qc + 1]), tau);
    auto verdict = [&](int k) { return r0 + k < 1 ? -1 : r0 + k + 1 >= g.L2 ? 1 : (int)(sure.left >> k & 1u) - (int)(sure.right >> k & 1u); };
    const int v0 = is_main ? verdict(0) : -1, v2 = e2 ? verdict(2) : -1, v4 = e4 ? verdict(R) : -1;
    bool up0 = v0 > 0, up2 = v2 > 0, up4 = v4 > 0;
    if (v0 == 0 || v2 == 0 || v4 == 0) {                          // too close for fp32: fp64 decides
        double n[R], d[R];
#pragma unroll
        for (int k = 0; k < R; ++k) n[k] = norm64<T>(Tk[k]);
#pragma unroll
        for (int k = 0; k < R; ++k) d[k] = dot64<T>(Tk[k], k + 1 < R ? Tk[k + 1 < R ? k + 1 : 0] : Tx);
        if (lane < R) {
            const int k = lane, r = r0 + k;
            if (r >= row_lo && r <= row_end) {
                double n2 = n[0], dn = d[0];
#pragma unroll
                for (int i = 1; i < R; ++i)
                    if (k == i) { n2 = n[i]; dn = d[i]; }
                inv64[rr0 + k] = inv_norm64(n2);
                dt64[rr0 + k] = dn;
            }
        }
        reached(kSums);
        auto decide64 = [&](int q) { return source_goes_left(true, true, inv64[q], dt64[q - 1], inv64[q - 1], dt64[q], inv64[q + 1]); };
        // The wavefront that shares a source looks at the same bits and comes here as well; had it not, its verdict would be the one.
        const int wa = v0 == 0 ? wait_for(above, kSums) : 0, wb = v4 == 0 ? wait_for(below, kSums) : 0;
        if (v0 == 0) up0 = wa & kSettled ? (wa & kNextUp) != 0 : decide64(rr0);
        if (v2 == 0) up2 = decide64(rr0 + 2);
        if (v4 == 0) up4 = wb & kSettled ? (wb & kFirstUp) != 0 : decide64(rr0 + R);
    } else {
        reached(kSettled | (up0 ? kFirstUp : 0) | (up4 ? kNextUp : 0));
    }
    if (is_halo) return;

    // ------------------------------------------------------------------ second pass: merge, write, maps
    __builtin_amdgcn_s_setprio(0);
    const int own_end = row_base + 2 * nseg;                      // rows below it belong to the next run ...
    const bool tail = (g.L2 & 1) && own_end == g.L2 - 1;          // ... except the last source of an odd line
    const int64_t img_out = at.out_off + (int64_t)b * g.n_out;
    const int dst = MOST > 1 ? at.dst : 0;
    T* x_out = (T*)out.x[dst];
    int32_t *sizes_out = out.sizes[dst], *kept_out = out.kept[dst], *pair_map = out.map[MOST > 1 ? at.map_dst : 0];
    const int uo = r0 >> 1;                                       // output slot (second axis) of destination r0 + 1
#pragma unroll
    for (int o = 0; o < R / 2; ++o) {
        const int dest = r0 + 1 + 2 * o;
        if (dest >= own_end) break;
        constexpr int kLast = R / 2 - 1;
        const bool take_a = o == 0 ? !up0 : !up2;                 // the source above comes down
        const bool take_c = o < kLast ? (e2 && up2) : (e4 && up4);      // the source below goes up
        const TokT &Bt = Tk[2 * o + 1], &A = Tk[2 * o], &C = o < kLast ? Tk[o < kLast ? 2 * o + 2 : 0] : Tx;
        const int sb = sk[2 * o + 1];
        const int sa = take_a ? sk[2 * o] : 0;
        const int sc = take_c ? (o < kLast ? sk[o < kLast ? 2 * o + 2 : 0] : szl[rr0 + R]) : 0;
        const int slot = (uo + o) * g.oB + j * g.oA;
        T* op = x_out + (img_out + slot) * g.D;
        if (lane == 0) {
            sizes_out[img_out + slot] = sb + sa + sc;
            if (kept_out) {
                const int p_in = dest * g.sB + pb * g.sA;
                kept_out[img_out + slot] = kept_prev ? kept_prev[img_in + p_in] : p_in;
            }
        }
        if (!take_a && !take_c) {
            store_tok(op, tok_bytes, Bt, lane);
        } else {
            TokT merged;
            merge_tok<T>(merged, Bt, A, C, sb, sa, sc);
            store_tok(op, tok_bytes, merged, lane);
        }
    }
    if (pair_map && lane < R) {
        const int k = lane, r = r0 + k;
        if (r <= row_end && (r < own_end || (tail && r == own_end))) {
            // intermediate row r lands in output slot: odd rows are destinations; an even row goes up or down
            int u;
            if (r & 1) u = r >> 1;
            else u = (k == 0 ? up0 : up2) ? (r >> 1) - 1 : (r >> 1);
            const int slot = u * g.oB + j * g.oA;
            const int64_t t0 = at.map_off + (int64_t)b * at.map_stride + (int64_t)r * g.sB;
            pair_map[t0 + (int64_t)pb * g.sA] = slot;
            if ((took_a >> k) & 1u) pair_map[t0 + (int64_t)pa * g.sA] = slot;
            if ((took_c >> k) & 1u) pair_map[t0 + (int64_t)pc * g.sA] = slot;
        }
    }
}

// ------------------------------------------------------------------ host side
namespace {

constexpr int pair_waves(int words) { return words <= 10 ? 16 : 8; }      // 16 wavefronts leave 128 registers per lane, 8 leave 256

template <typename T, int NQ, int TW, int R, int MOST>
luvc_status launch_pair(const OimStepItem* items, int n, const StepIns& in, const StepOut& out, int D, int64_t lines, hipStream_t st)
{
    constexpr int N = 4 * NQ + TW, NW = pair_waves(N);
    PairTable<MOST> tab;
    tab.n = n;
    int64_t wgs = 0;
    int waves = 1;
    for (int i = 0; i < n; ++i) {
        const int H = items[i].H, W = items[i].W, axis = items[i].axis, Wo = W / 2;
        PairGeom& g = tab.it[i].g;
        g.L1 = axis ? W : H;
        g.L2 = axis ? H : W;
        g.nd1 = g.L1 / 2;
        g.nd2 = g.L2 / 2;
        g.sA = axis ? 1 : W;
        g.sB = axis ? W : 1;
        g.oA = axis ? 1 : Wo;
        g.oB = axis ? Wo : 1;
        g.n_in = H * W;
        g.n_out = (H / 2) * Wo;
        g.D = D;
        const PairPlan p = plan_pair(g.L2, NW, lines, R);
        g.segs = p.segs;
        g.seg_out = p.seg_out;
        waves = p.waves > waves ? p.waves : waves;     // a workgroup with fewer rows leaves the rest idle
        tab.it[i].at = items[i].at;
        tab.it[i].at.wg0 = (unsigned)wgs;
        wgs += (int64_t)items[i].count * g.segs * g.nd1;
    }
    const size_t lds = (size_t)waves * N * 64 * 4;             // at most 16 * 10 * 256 = 40 KiB
    if constexpr (MOST > 1) { tab.from[0] = in.set[1]; tab.from[1] = in.set[2]; }
    const StepIn& first = in.set[MOST > 1 ? 0 : items[0].at.src];
    LUVC_LAUNCH("oim_halve_pair", (oim_halve_pair<T, NQ, TW, NW, R, MOST>), dim3((unsigned)wgs), dim3(64 * waves), lds, st,
                (const T*)first.x, first.sizes, first.kept, step_out_of<MOST>(out, items[0].at), tab);
    return check_launch("oim halving pair");
}

// Two rows per wavefront instead of four where all those wavefronts fit the chip at once: a small grid takes the time of one
// wavefront's rows, one after the other.  us with four and with two rows, and the wavefronts of two: bf16 2x28x28x1280 10.8, 7.6 (630),
// 1x40x24x1024 10.0, 7.2, 5x21x16x896 10.0, 7.1, fp32 1x24x24x1024 10.1, 7.3, 1x64x64x1280 11.8, 9.9, 2x56x56x1280 13.0, 12.8 (2240),
// 11x24x38x1216 16.8, 14.7 (2508), 3x43x85x576 12.4, 10.7 (3528); beyond it 12x32x32x1024 15.5, 15.8 (3840), 2x67x107x896
// 18.4, 21.8 (5300), 2x112x112x1280 28, 38, 8x64x64x1280 29, 39.
constexpr int64_t kTwoRowWaves = 3600;
template <typename T, int NQ, int TW>
luvc_status launch_pair_rows(const OimStepItem* items, int n, const StepIns& in, const StepOut& out, int D, hipStream_t st)
{
    int64_t lines = 0, waves2 = 0;
    for (int i = 0; i < n; ++i) lines += (int64_t)items[i].count * ((items[i].axis ? items[i].W : items[i].H) / 2);
    for (int i = 0; i < n; ++i) {
        const PairPlan p = plan_pair(items[i].axis ? items[i].H : items[i].W, pair_waves(4 * NQ + TW), lines, 2);
        waves2 += (int64_t)items[i].count * ((items[i].axis ? items[i].W : items[i].H) / 2) * p.segs * p.waves;
    }
    const bool two = waves2 <= kTwoRowWaves;
#define LUVC_PAIR_ROWS(R) (n == 1 ? launch_pair<T, NQ, TW, R, 1>(items, n, in, out, D, lines, st) : launch_pair<T, NQ, TW, R, kOimMaxItems>(items, n, in, out, D, lines, st))
    return two ? LUVC_PAIR_ROWS(2) : LUVC_PAIR_ROWS(4);
#undef LUVC_PAIR_ROWS
}

template <typename T>
luvc_status dispatch_pair(const OimStepItem* items, int n, const StepIns& in, const StepOut& out, int D, hipStream_t st)
{
    // 16-byte pieces per lane, then a 4- or 8-byte tail piece if that covers what is left
    const int bytes = D * (int)sizeof(T);
    int nq = bytes / 1024, tw = 0;
    const int rem = bytes % 1024;
    if (rem > 512) ++nq;
    else if (rem > 256) tw = 2;
    else if (rem > 0) tw = 1;
#define LUVC_PAIR(Q, W_) if (nq == Q && tw == W_) return launch_pair_rows<T, Q, W_>(items, n, in, out, D, st)
    LUVC_PAIR(0, 1); LUVC_PAIR(0, 2);
    LUVC_PAIR(1, 0); LUVC_PAIR(1, 1); LUVC_PAIR(1, 2);
    LUVC_PAIR(2, 0); LUVC_PAIR(2, 1); LUVC_PAIR(2, 2);
    LUVC_PAIR(3, 0); LUVC_PAIR(3, 1); LUVC_PAIR(3, 2);
    LUVC_PAIR(4, 0);
#undef LUVC_PAIR
    set_error("oim pair: unsupported D");
    return LUVC_ERR_UNSUPPORTED;
}

}  // namespace

bool oim_pair_supported(int H, int W, int D, luvc_dtype dt, int axis0, int m0, int axis1, int m1, bool vec)
{
    if (!vec || axis0 == axis1) return false;
    const int len0 = axis0 ? W : H, len1 = axis1 ? W : H;           // the second pass runs on the untouched axis
    if (len0 < 2 || len1 < 2 || m0 != (len0 + 1) / 2 || m1 != (len1 + 1) / 2) return false;
    return (int64_t)D * (dt == LUVC_F32 ? 4 : 2) <= 4096;
}

luvc_status oim_pair_step(const OimStepItem* items, int n, const StepIns& in, const StepOut& out, int D, luvc_dtype dt, hipStream_t st)
{
    return dt == LUVC_F32 ? dispatch_pair<float>(items, n, in, out, D, st) : dispatch_pair<bf16_t>(items, n, in, out, D, st);
}

}  // namespace luvc
