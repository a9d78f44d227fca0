// Ragged batches (appendix "Iterative Strategy and Pseudocode of OIM": with any-resolution inputs every image has
// its own grid and its own number of merges): images / samples of different shapes packed back to back.  Host code
// only: consecutive items of equal shape and schedule form a run; every item is validated before the first launch.
//
// Runs share launches wherever a kernel takes several of them.  OIM: images whose schedules consist of halvings advance
// together, sharing launches of either kind of step (a pair of passes, a single pass) in the best of three orders, then one for the images
// that stay as they are and the maps of those with several steps.  SPU: the short samples are scored in one launch, all samples pruned
// in one.  What does not fit these (other merge numbers, long samples, unaligned rows) is a batched call of the entry points
// in api.hip per run.  A launch costs 4 to 12 us whatever it does: eight images of 24x24 to 56x56 tokens took
// 30 launches and 398 us run by run, 95 us like this.
#include <algorithm>
#include <vector>

#include "common.hpp"
#include "oim.hpp"
#include "spu.hpp"

namespace luvc {

namespace {

struct OimRun {
    int count;                   // consecutive images of this shape and schedule
    int H, W;
    const luvc_oim_pass* passes;
    int n_passes;
    int64_t tok_in, tok_out;     // packed token offsets of the first image
};

bool same_schedule(const luvc_oim_pass* a, int na, const luvc_oim_pass* b, int nb)
{
    if (na != nb) return false;
    for (int i = 0; i < na; ++i)
        if (a[i].axis != b[i].axis || a[i].m != b[i].m) return false;
    return true;
}

// Splits the images into runs; false (with an error message) when an argument is unusable.
bool oim_runs(int n_images, const int32_t* H, const int32_t* W, const luvc_oim_pass* passes, const int32_t* n_passes,
              std::vector<OimRun>* runs)
{
    if (n_images < 1 || !H || !W || !passes || !n_passes) { set_error("n_images, H, W, passes and n_passes must be given"); return false; }
    int64_t tin = 0, tout = 0;
    const luvc_oim_pass* p = passes;
    for (int i = 0; i < n_images; ++i) {
        if (H[i] < 1 || W[i] < 1) { set_error("image %d: H and W must be positive (got %d,%d)", i, H[i], W[i]); return false; }
        if (n_passes[i] < 1 || n_passes[i] > kMaxPasses) { set_error("image %d: need 1..%d passes", i, kMaxPasses); return false; }
        int h = H[i], w = W[i];
        for (int k = 0; k < n_passes[i]; ++k) {
            const int axis = p[k].axis, m = p[k].m;
            if (axis != 0 && axis != 1) { set_error("image %d pass %d: axis must be 0 (H) or 1 (W)", i, k); return false; }
            const int len = axis ? w : h;
            if (m < 0 || m > (len + 1) / 2 || len - m < 1) { set_error("image %d pass %d: m=%d does not fit a line of %d", i, k, m, len); return false; }
            if (axis) w -= m; else h -= m;
        }
        const bool extend = !runs->empty() && runs->back().H == H[i] && runs->back().W == W[i] &&
                            same_schedule(runs->back().passes, runs->back().n_passes, p, n_passes[i]);
        if (extend) ++runs->back().count;
        else runs->push_back(OimRun{1, H[i], W[i], p, n_passes[i], tin, tout});
        tin += (int64_t)H[i] * W[i];
        tout += (int64_t)h * w;
        if (tin >= ((int64_t)1 << 31)) { set_error("the packed batch must stay below 2^31 tokens"); return false; }
        p += n_passes[i];
    }
    return true;
}

// ---- runs that advance together
struct BatchStep { int h, w, axis, passes; };        // grid before the step; one pass or a fused pair
struct BatchRun {
    const OimRun* run;
    int n;
    BatchStep step[kMaxPasses];
    int64_t tokens, between;                          // of the run: entering, and the most any step but the last leaves
    int64_t map_off, between_off;                     // its place among the runs with several steps
};
struct BatchPlan {
    std::vector<BatchRun> runs;
    std::vector<const OimRun*> others;
    int levels = 0;
    int64_t map_level = 0, between = 0;               // tokens of the runs with several steps: map entries per step, scratch rows
    size_t x[2], sizes[2], kept[2], maps, bytes;
};

bool batch_run(const OimRun& r, int D, luvc_dtype dt, BatchRun* b)
{
    luvc_oim_pass ps[kMaxPasses];
    int n = 0, h = r.H, w = r.W;
    for (int i = 0; i < r.n_passes; ++i)
        if (r.passes[i].m != 0) ps[n++] = r.passes[i];
    b->run = &r;
    b->n = 0;
    b->tokens = (int64_t)r.count * h * w;
    b->between = 0;
    for (int i = 0; i < n;) {
        const bool pair = i + 1 < n && oim_pair_supported(h, w, D, dt, ps[i].axis, ps[i].m, ps[i + 1].axis, ps[i + 1].m, true);
        if (!pair && !oim_halve_supported(h, w, D, dt, ps[i].axis, ps[i].m, true)) return false;
        if (b->n) b->between = std::max(b->between, (int64_t)r.count * h * w);
        b->step[b->n++] = BatchStep{h, w, ps[i].axis, pair ? 2 : 1};
        for (int k = 0; k < (pair ? 2 : 1); ++k, ++i) (ps[i].axis ? w : h) -= ps[i].m;
    }
    return true;
}

// vec: rows are 16-byte aligned
void batch_plan(const std::vector<OimRun>& runs, int D, luvc_dtype dt, bool vec, BatchPlan* p)
{
    BatchRun b;
    for (const OimRun& r : runs) {
        if (runs.size() > 1 && vec && batch_run(r, D, dt, &b)) {
            b.map_off = p->map_level;
            b.between_off = p->between;
            if (b.n > 1) { p->map_level += b.tokens; p->between += b.between; }
            p->levels = std::max(p->levels, b.n);
            p->runs.push_back(b);
        } else {
            p->others.push_back(&r);
        }
    }
    size_t off = 0;
    for (int j = 0; j < 2; ++j) {
        p->x[j] = off;     off += align_up((size_t)p->between * D * (dt == LUVC_F32 ? 4 : 2));
        p->sizes[j] = off; off += align_up((size_t)p->between * sizeof(int32_t));
        p->kept[j] = off;  off += align_up((size_t)p->between * sizeof(int32_t));
    }
    p->maps = off;         off += p->levels > 1 ? align_up((size_t)p->levels * p->map_level * sizeof(int32_t)) : 0;
    p->bytes = off;
}

// The kinds (2: a pair of passes, 1: a single one) of the launches that take all runs through their steps.  A run joins the first
// launch of the kind it needs next.  Of three orders the one with the fewest launches: one kind as long as any run needs it, so that
// the others gather behind it (a schedule of one pass goes along with the third pass of another), with the pairs first or the single
// passes, and step by step, pairs before single passes.  The last is one of them because it can be the shortest - runs of steps 1 2 1 and
// 2 2 1 are four launches like that, five either other way; of random batches on the aspect-ratio schedule it saves one to three
// launches on a fifth.
std::vector<int> step_kinds(const std::vector<BatchRun>& runs)
{
    int levels = 0;
    for (const BatchRun& b : runs) levels = std::max(levels, b.n);
    std::vector<int> best, kinds, at;
    auto kind_of = [&](size_t i, int s) { return s < runs[i].n ? runs[i].step[s].passes : 0; };
    auto launch = [&](int kind) {
        bool any = false;
        for (size_t i = 0; i < runs.size(); ++i)
            if (kind_of(i, at[i]) == kind) { ++at[i]; any = true; }
        if (any) kinds.push_back(kind);
        return any;
    };
    for (int first = 2; first >= 0; --first) {
        kinds.clear();
        at.assign(runs.size(), 0);
        if (first > 0) {
            while (launch(first) || launch(3 - first)) {}
        } else {
            for (int s = 0; s < levels; ++s)
                for (int kind = 2; kind >= 1; --kind) {
                    bool wanted = false;
                    for (size_t i = 0; i < runs.size(); ++i) wanted |= kind_of(i, s) == kind;
                    if (wanted) launch(kind);
                }
        }
        if (first == 2 || kinds.size() < best.size()) best = kinds;
    }
    return best;
}

luvc_status batch_run_all(const BatchPlan& p, const void* x, const int32_t* sizes_in, int D, luvc_dtype dt, void* x_out, int32_t* sizes_out,
                          int32_t* merged_map, int32_t* kept_map, char* ws, hipStream_t st)
{
    int32_t* maps = (int32_t*)(ws + p.maps);
    StepIns in = {{{x, sizes_in, nullptr}}};
    StepOut out = {{x_out}, {sizes_out}, {kept_map}, {merged_map, merged_map ? maps : nullptr}};
    for (int j = 0; j < 2; ++j) {
        int32_t *sz = (int32_t*)(ws + p.sizes[j]), *kept = (int32_t*)(ws + p.kept[j]);
        in.set[1 + j] = StepIn{ws + p.x[j], sz, kept};
        out.x[1 + j] = ws + p.x[j];
        out.sizes[1 + j] = sz;
        out.kept[1 + j] = kept_map ? kept : nullptr;
    }
    OimStepItem items[kOimMaxItems];
    std::vector<int> done(p.runs.size(), 0);
    for (int passes : step_kinds(p.runs)) {
        int n = 0;
        for (size_t i = 0; i <= p.runs.size(); ++i) {
            if (n == kOimMaxItems || (i == p.runs.size() && n)) {
                const luvc_status rc = passes == 2 ? oim_pair_step(items, n, in, out, D, dt, st) : oim_halve_step(items, n, in, out, D, dt, st);
                if (rc != LUVC_OK) return rc;
                n = 0;
            }
            if (i == p.runs.size()) break;
            const BatchRun& b = p.runs[i];
            const int s = done[i];
            if (s >= b.n || b.step[s].passes != passes) continue;
            ++done[i];
            // step s leaves its tokens in number s & 1 of the two grids between steps
            const bool last = s + 1 == b.n, single = b.n == 1;
            items[n++] = OimStepItem{b.step[s].h, b.step[s].w, b.step[s].axis, b.run->count,
                                     StepAt{s == 0 ? b.run->tok_in : b.between_off, last ? b.run->tok_out : b.between_off,
                                            single ? b.run->tok_in : s * p.map_level + b.map_off, b.run->H * b.run->W, 0,
                                            s == 0 ? 0 : 1 + ((s + 1) & 1), last ? 0 : 1 + (s & 1), single ? 0 : 1}};
        }
    }
    OimTailItem tail[kOimMaxItems];
    int n = 0;
    for (size_t i = 0; i <= p.runs.size(); ++i) {
        if (n == kOimMaxItems || (i == p.runs.size() && n)) {
            const luvc_status rc = oim_batch_tail(tail, n, x, sizes_in, D * (dt == LUVC_F32 ? 4 : 2), x_out, sizes_out, merged_map, kept_map, maps, p.map_level, st);
            if (rc != LUVC_OK) return rc;
            n = 0;
        }
        if (i == p.runs.size()) break;
        const BatchRun& b = p.runs[i];
        if (b.n == 0 || (b.n > 1 && merged_map))
            tail[n++] = OimTailItem{b.n == 0, b.run->H * b.run->W, b.n, 0, b.tokens, b.run->tok_in, b.run->tok_out, b.map_off};
    }
    return LUVC_OK;
}

struct SpuRun {
    int count, N, sigma, keep;   // consecutive samples with these parameters
    int64_t tok_in, tok_out;
};

// n_keep NULL: the runs that are scored together, which keep counts do not split
bool spu_runs(int n_samples, const int32_t* N, const int32_t* sigma, const int32_t* n_keep, std::vector<SpuRun>* runs)
{
    if (n_samples < 1 || !N || !sigma) { set_error("n_samples, N and sigma must be given"); return false; }
    int64_t tin = 0, tout = 0;
    for (int i = 0; i < n_samples; ++i) {
        const int keep = n_keep ? n_keep[i] : 0;
        if (N[i] < 1 || N[i] > kSpuMaxN) { set_error("sample %d: N=%d must lie in 1..%d", i, N[i], kSpuMaxN); return false; }
        if (sigma[i] < 0 || sigma[i] > N[i] / 2) { set_error("sample %d: sigma=%d must lie in 0..N/2=%d", i, sigma[i], N[i] / 2); return false; }
        if (keep < 0 || keep > N[i]) { set_error("sample %d: n_keep=%d must lie in 0..N=%d", i, keep, N[i]); return false; }
        const bool extend = !runs->empty() && runs->back().N == N[i] && runs->back().sigma == sigma[i] && runs->back().keep == keep &&
                            runs->back().count < 65535;
        if (extend) ++runs->back().count;
        else runs->push_back(SpuRun{1, N[i], sigma[i], keep, tin, tout});
        tin += N[i];
        tout += keep;
        if (tin >= ((int64_t)1 << 31)) { set_error("the packed batch must stay below 2^31 tokens"); return false; }
    }
    return true;
}

size_t esz(luvc_dtype dt) { return dt == LUVC_F32 ? 4 : 2; }

// How the runs of a ragged batch are scored: on their own, or in a launch that several share, spu_circ's or spu_mat's.  In such a
// launch a run adds its products and nothing else.  spu_circ takes short samples of any length; a second kind of launch is made
// where it saves more than the 9 us it takes (eight samples of 312 to 576 tokens, 3584 channels: 45 -> 30 us with all in spu_mat,
// which has N log N work for lengths with a factor in 9 .. 16).
enum class SpuKind : char { Own, Circ, Mat };
std::vector<SpuKind> spu_kinds(const std::vector<SpuRun>& runs, int D, luvc_dtype dt, SpuRows rows)
{
    std::vector<SpuKind> kinds(runs.size(), SpuKind::Own), with_mat;
    double saved = 0.0;
    bool circ = false, circ_left = false;
    with_mat = kinds;
    for (size_t i = 0; i < runs.size(); ++i) {
        const SpuRun& r = runs[i];
        double us = spu_alone_us(r.count, r.N, D, r.sigma, dt, rows.pieces);
        const double c = spu_circ_work_us(r.count, r.N, D, dt), m = rows.pieces ? spu_mat_work_us(r.count, r.N, D, r.sigma) : 0.0;
        if (rows.circ != CircRows::None && r.N <= kCircMaxN && c <= us) {
            kinds[i] = with_mat[i] = SpuKind::Circ;
            us = c;
            circ = true;
        }
        if (m > 0.0 && m < us) {
            with_mat[i] = SpuKind::Mat;
            saved += us - m;
        }
        circ_left |= with_mat[i] == SpuKind::Circ;
    }
    return saved > (circ && !circ_left ? 1.0 : 9.0) ? with_mat : kinds;
}

std::vector<MatRun> mat_runs(const std::vector<SpuRun>& runs, const std::vector<SpuKind>& kinds)
{
    std::vector<MatRun> out;
    for (size_t i = 0; i < runs.size(); ++i)
        if (kinds[i] == SpuKind::Mat) out.push_back(MatRun{runs[i].N, runs[i].sigma, runs[i].count, runs[i].tok_in});
    return out;
}

// Workspace of the scores of a ragged batch: the largest need of a run that is a call of its own, or of a launch that several
// share.  0 (with an error message) when a run is not supported.
size_t spu_runs_workspace(const std::vector<SpuRun>& runs, int D, luvc_dtype dt, SpuRows rows)
{
    const std::vector<SpuKind> kinds = spu_kinds(runs, D, dt, rows);
    size_t need = 0, shared = 0;
    for (size_t i = 0; i < runs.size(); ++i) {
        const SpuRun& r = runs[i];
        const size_t b = luvc_spu_workspace_bytes(r.count, r.N, D, dt, r.sigma);
        if (b == 0) { set_error("run of %d samples with N=%d, sigma=%d is not supported", r.count, r.N, r.sigma); return 0; }
        need = std::max(need, b);
        if (kinds[i] == SpuKind::Circ) shared += spu_circ_bytes(r.count, r.N, D);
    }
    const std::vector<MatRun> mat = mat_runs(runs, kinds);
    for (size_t i = 0; i < mat.size(); i += kMatMaxRuns) need = std::max(need, spu_mat_bytes(&mat[i], (int)std::min<size_t>(kMatMaxRuns, mat.size() - i), D));
    return std::max(need, align_up(shared));
}

}  // namespace

}  // namespace luvc

using namespace luvc;

extern "C" {

luvc_status luvc_oim_plan_anyres(int H, int W, int64_t max_tokens, luvc_oim_pass* passes, int max_passes, int* n_passes)
{
    if (!passes || !n_passes || max_passes < 1) { set_error("passes / n_passes must be given"); return LUVC_ERR_INVALID_ARG; }
    if (H < 1 || W < 1 || max_tokens < 1) { set_error("H, W and max_tokens must be positive"); return LUVC_ERR_INVALID_ARG; }
    int h = H, w = W, n = 0;
    while ((int64_t)h * w > max_tokens) {
        if (n >= max_passes) { set_error("schedule needs more than %d passes", max_passes); return LUVC_ERR_INVALID_ARG; }
        const int axis = w >= h ? 1 : 0;                 // the longer side; a square grid starts with the row merge
        const int len = axis ? w : h;                    // > 1 here: h * w > max_tokens >= 1
        passes[n].axis = axis;
        passes[n].m = (len + 1) / 2;
        ++n;
        if (axis) w = len / 2; else h = len / 2;
    }
    if (n == 0) {                                        // nothing to merge: the pass that leaves every line as it is
        passes[0].axis = 1;
        passes[0].m = 0;
        n = 1;
    }
    *n_passes = n;
    return LUVC_OK;
}

size_t luvc_oim_ragged_workspace_bytes(int n_images, const int32_t* H, const int32_t* W, int D, luvc_dtype dtype,
                                       const luvc_oim_pass* passes, const int32_t* n_passes)
{
    std::vector<OimRun> runs;
    if (D < 1 || !oim_runs(n_images, H, W, passes, n_passes, &runs)) return 0;
    size_t need = 0;
    for (const OimRun& r : runs) {
        const size_t b = luvc_oim_workspace_bytes(r.count, r.H, r.W, D, dtype, r.passes, r.n_passes);
        if (b == 0) return 0;
        need = b > need ? b : need;
    }
    BatchPlan plan;
    batch_plan(runs, D, dtype, (size_t)D * esz(dtype) % 16 == 0, &plan);
    need = plan.bytes > need ? plan.bytes : need;
    return need;
}

luvc_status luvc_oim_merge_ragged(const void* x, const int32_t* sizes_in, int n_images, const int32_t* H, const int32_t* W,
                                  int D, luvc_dtype dtype, const luvc_oim_pass* passes, const int32_t* n_passes,
                                  void* x_out, int32_t* sizes_out, int32_t* merged_map, int32_t* kept_map,
                                  void* workspace, size_t workspace_bytes, void* hip_stream)
{
    if (dtype != LUVC_F32 && dtype != LUVC_BF16) { set_error("unknown dtype %d", (int)dtype); return LUVC_ERR_INVALID_ARG; }
    if (!x || !x_out || !sizes_out) { set_error("x, x_out and sizes_out must not be NULL"); return LUVC_ERR_INVALID_ARG; }
    if (D < 1) { set_error("D must be positive (got %d)", D); return LUVC_ERR_INVALID_ARG; }
    std::vector<OimRun> runs;
    if (!oim_runs(n_images, H, W, passes, n_passes, &runs)) return LUVC_ERR_INVALID_ARG;
    // all runs are checked (shape limits, workspace) before the first one is launched
    for (const OimRun& r : runs) {
        const size_t b = luvc_oim_workspace_bytes(r.count, r.H, r.W, D, dtype, r.passes, r.n_passes);
        if (b == 0) return LUVC_ERR_INVALID_ARG;         // message set by the query
        if (!workspace_ok(workspace, workspace_bytes, b)) return LUVC_ERR_WORKSPACE;
    }
    const size_t row = (size_t)D * esz(dtype);
    BatchPlan plan;
    batch_plan(runs, D, dtype, row % 16 == 0 && (uintptr_t)x % 16 == 0 && (uintptr_t)x_out % 16 == 0, &plan);
    if (!workspace_ok(workspace, workspace_bytes, plan.bytes)) return LUVC_ERR_WORKSPACE;
    const luvc_status rc = batch_run_all(plan, x, sizes_in, D, dtype, x_out, sizes_out, merged_map, kept_map, (char*)workspace, (hipStream_t)hip_stream);
    if (rc != LUVC_OK) return rc;
    for (const OimRun* q : plan.others) {
        const OimRun& r = *q;
        const luvc_status rc = luvc_oim_merge(
            (const char*)x + (size_t)r.tok_in * row, sizes_in ? sizes_in + r.tok_in : nullptr, r.count, r.H, r.W, D, dtype,
            r.passes, r.n_passes, 0, (char*)x_out + (size_t)r.tok_out * row, sizes_out + r.tok_out,
            merged_map ? merged_map + r.tok_in : nullptr, kept_map ? kept_map + r.tok_out : nullptr,
            workspace, workspace_bytes, hip_stream);
        if (rc != LUVC_OK) return rc;
    }
    return LUVC_OK;
}

size_t luvc_spu_ragged_workspace_bytes(int n_samples, const int32_t* N, int D, luvc_dtype dtype, const int32_t* sigma)
{
    std::vector<SpuRun> runs;
    if (D < 1 || !spu_runs(n_samples, N, sigma, nullptr, &runs)) return 0;
    // whichever way the rows will lie
    const size_t a = spu_runs_workspace(runs, D, dtype, SpuRows{CircRows::Paired, false}), b = spu_runs_workspace(runs, D, dtype, SpuRows{CircRows::Paired, dtype == LUVC_BF16 && D % 8 == 0});
    return a && b ? std::max(a, b) : 0;
}

luvc_status luvc_spu_stage_ragged(const void* x, int n_samples, const int32_t* N, int D, int64_t row_stride, luvc_dtype dtype,
                                  const int32_t* sigma, int use_hamming, const int32_t* n_keep, const int32_t* origin_in,
                                  float* scores, int32_t* kept_idx, int32_t* origin_out, void* x_out,
                                  void* workspace, size_t workspace_bytes, void* hip_stream)
{
    if (dtype != LUVC_F32 && dtype != LUVC_BF16) { set_error("unknown dtype %d", (int)dtype); return LUVC_ERR_INVALID_ARG; }
    if (!x || !scores) { set_error("x and scores must not be NULL"); return LUVC_ERR_INVALID_ARG; }
    if (D < 1 || row_stride < D) { set_error("need D >= 1 and row_stride >= D (got %d, %lld)", D, (long long)row_stride); return LUVC_ERR_INVALID_ARG; }
    if (n_keep && (!kept_idx || !origin_out)) { set_error("kept_idx and origin_out must be given with n_keep"); return LUVC_ERR_INVALID_ARG; }
    // What is scored together and what is pruned together are runs of their own: which kernel scores a sample, and with it the
    // workspace, follows from lengths and cut-offs alone, as in the query, which has no keep counts.
    std::vector<SpuRun> runs, kept;
    if (!spu_runs(n_samples, N, sigma, nullptr, &runs) || (n_keep && !spu_runs(n_samples, N, sigma, n_keep, &kept))) return LUVC_ERR_INVALID_ARG;
    const SpuRows rows = spu_rows(x, D, row_stride, dtype);
    const size_t need = spu_runs_workspace(runs, D, dtype, rows);
    if (need == 0) return LUVC_ERR_INVALID_ARG;
    if (!workspace_ok(workspace, workspace_bytes, need)) return LUVC_ERR_WORKSPACE;
    const size_t es = esz(dtype);
    hipStream_t st = (hipStream_t)hip_stream;
    // scores: the short samples share launches, every other run is a call of its own
    CircRuns cr;
    cr.n = 0;
    auto flush_scores = [&]() {
        const luvc_status rc = cr.n ? spu_score_circ(x, row_stride, D, dtype, use_hamming ? 1 : 0, cr, workspace, scores, st) : LUVC_OK;
        cr.n = 0;
        return rc;
    };
    const std::vector<SpuKind> kinds = spu_kinds(runs, D, dtype, rows);
    for (size_t i = 0; i < runs.size(); ++i) {
        const SpuRun& r = runs[i];
        luvc_status rc = LUVC_OK;
        if (kinds[i] == SpuKind::Circ) {
            cr.run[cr.n++] = CircRun{0, r.N, r.sigma, r.count, r.tok_in};
            if (cr.n == kCircMaxRuns) rc = flush_scores();
        } else if (kinds[i] == SpuKind::Own) {
            rc = luvc_spu_score((const char*)x + (size_t)r.tok_in * (size_t)row_stride * es, r.count, r.N, D, row_stride, dtype, r.sigma, use_hamming,
                                scores + r.tok_in, workspace, workspace_bytes, hip_stream);
        }
        if (rc != LUVC_OK) return rc;
    }
    const std::vector<MatRun> mat = mat_runs(runs, kinds);
    for (size_t i = 0; i < mat.size(); i += kMatMaxRuns) {
        const luvc_status rc = spu_score_mat_runs(x, &mat[i], (int)std::min<size_t>(kMatMaxRuns, mat.size() - i), D, row_stride, use_hamming ? 1 : 0, scores, workspace, st);
        if (rc != LUVC_OK) return rc;
    }
    luvc_status rc = flush_scores();
    if (rc != LUVC_OK || !n_keep) return rc;
    // keep and gather (a sample that is eliminated only gets its scores)
    PruneRuns pr;
    pr.n = 0;
    for (const SpuRun& r : kept) {
        if (r.keep == 0) continue;
        pr.run[pr.n++] = PruneRun{0, r.N, r.keep, r.count, r.tok_in, r.tok_out};
        if (pr.n < kPruneMaxRuns) continue;
        rc = spu_prune_run(x, scores, D, row_stride, dtype, pr, kept_idx, x_out, origin_in, origin_out, st);
        if (rc != LUVC_OK) return rc;
        pr.n = 0;
    }
    return pr.n ? spu_prune_run(x, scores, D, row_stride, dtype, pr, kept_idx, x_out, origin_in, origin_out, st) : LUVC_OK;
}

}  // extern "C"
