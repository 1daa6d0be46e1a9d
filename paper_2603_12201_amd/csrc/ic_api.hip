// C ABI of the library: argument validation, workspace planning, the Full/Shared layer loop
// (paper Fig. 2b) and optional per-kernel event timing.  All device work is enqueued on the
// caller's stream; nothing here allocates device memory or synchronises in the hot path.
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <algorithm>
#include <vector>

#include "ic_common.hpp"

// Scratch for ic_sparse_attn_static: part of the code object, one copy per GPU at its own address.
// In host code this name is only a handle for hipGetSymbolAddress; kernels get the address it returns.
static __device__ __align__(256) unsigned char scratch[IC_STATIC_SCRATCH_BYTES];

namespace {

thread_local char g_err[512] = "";

ic_status fail(ic_status s, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return s;
}

std::atomic<uint64_t> g_indexer_launches{0};

// ---- per-kernel event timing -------------------------------------------------------------
constexpr int kProfClasses = 4;
constexpr size_t kProfPool = 8192;
struct ProfRec {
    hipEvent_t e0, e1;
    int which;
};
std::mutex g_prof_mu;
bool g_prof_on = false;
std::vector<ProfRec> g_prof_recs;
int64_t g_prof_n[kProfClasses] = {0, 0, 0, 0};
double g_prof_ms[kProfClasses] = {0, 0, 0, 0};

struct ProfScope {
    hipStream_t st;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int which;
    bool live = false;
    ProfScope(int which_, hipStream_t st_) : st(st_), which(which_)
    {
        if (!g_prof_on) return;
        std::lock_guard<std::mutex> lk(g_prof_mu);
        if (g_prof_recs.size() >= kProfPool) return;
        if (hipEventCreate(&e0) != hipSuccess) return;
        if (hipEventCreate(&e1) != hipSuccess) {
            (void)hipEventDestroy(e0);
            return;
        }
        live = true;
        (void)hipEventRecord(e0, st);
    }
    ~ProfScope()
    {
        if (!live) return;
        (void)hipEventRecord(e1, st);
        std::lock_guard<std::mutex> lk(g_prof_mu);
        g_prof_recs.push_back(ProfRec{e0, e1, which});
    }
};

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Default strip budget when the caller asks how much workspace to bring.
constexpr size_t kStripBudget = (size_t)1 << 30;   // 1 GiB of score rows in flight
// Problems whose whole score matrix is below this keep it in one strip, and larger ones have strips of at least as much: every strip ends in
// rounds of a part of the CUs.  us, 32 heads of 128, with 64 / 128 / 256 MiB: 1000 rows before 20000 keys (76 MiB) 203 / 176 / 178, 2048
// before 12000 (94) 218 / 193 / 193, 300 before 80000 (91) 234 / 198 / 198, 4096 before 8000 (125) 237 / 215 / 214; larger than that:
// 1500 before 41700 (238) 546 / 495 / 466, 4096 before 16384 (256) 533 / 476 / 447, 4096 before 32768 (512) 1010 / 1009 / 952.  Not more, for the
// memory that a caller brings.
constexpr size_t kSmallStrip = (size_t)128 << 20;
constexpr int kMinStripRows = 16;

ic_status check_indexer(const ic_indexer_desc *d)
{
    if (!d) return fail(IC_ERR_NULL, "indexer descriptor is NULL");
    if (d->B <= 0 || d->Tq <= 0 || d->Lk <= 0 || d->H_I <= 0 || d->d_I <= 0 || d->k_sel <= 0)
        return fail(IC_ERR_SHAPE, "indexer sizes must be positive (B=%d Tq=%d Lk=%d H_I=%d d_I=%d k_sel=%d)",
                    d->B, d->Tq, d->Lk, d->H_I, d->d_I, d->k_sel);
    if (d->k_sel > IC_MAX_K) return fail(IC_ERR_UNSUPPORTED, "k_sel=%d exceeds IC_MAX_K=%d", d->k_sel, IC_MAX_K);
    if (d->flags != 0) return fail(IC_ERR_UNSUPPORTED, "indexer flags must be 0");
    if (d->dtype != IC_BF16 && d->dtype != IC_FP8_E4M3) return fail(IC_ERR_UNSUPPORTED, "unknown dtype %d", d->dtype);
    if (!ic::score_shape_supported(d->dtype, d->H_I, d->d_I))
        return fail(IC_ERR_UNSUPPORTED, "indexer shape not covered: dtype=%d H_I=%d d_I=%d (H_I<=64; bf16: d_I in {64,128}; fp8: d_I = 128)",
                    d->dtype, d->H_I, d->d_I);
    if ((int64_t)d->B * d->Tq > INT32_MAX / 2 || (int64_t)d->B * d->Tq * d->k_sel > ((int64_t)1 << 40))
        return fail(IC_ERR_SHAPE, "B*Tq too large");
    if (d->q_pos0 < -(int64_t)d->Tq || d->q_pos0 > ((int64_t)1 << 40))
        return fail(IC_ERR_SHAPE, "q_pos0 out of range");
    if (d->dtype == IC_FP8_E4M3 && (!d->q_scale || !d->k_scale))
        return fail(IC_ERR_NULL, "fp8 indexer needs q_scale and k_scale");
    return IC_OK;
}

size_t strip_ld(const ic_indexer_desc *d) { return ((size_t)d->Lk + 63) / 64 * 64; }

// Rows of the strip a workspace of `bytes` can hold.
int64_t strip_rows(const ic_indexer_desc *d, size_t bytes) { return (int64_t)(bytes / (strip_ld(d) * sizeof(float))); }

// Workspace for selecting all rows of the call in parts (few long rows): every row's scores, then the candidate lists;
// 0 when the call does not qualify.
size_t parts_ws(const ic_indexer_desc *d)
{
    const int64_t rows = (int64_t)d->B * d->Tq;
    const size_t lists = rows > INT32_MAX ? 0 : ic::select_parts_bytes((int)rows, d->Lk);
    const size_t strip = (size_t)rows * strip_ld(d) * sizeof(float);
    return lists == 0 || strip > kStripBudget ? 0 : align_up(strip) + align_up(lists);
}

ic_status check_attn(const ic_attn_desc *d)
{
    if (!d) return fail(IC_ERR_NULL, "attention descriptor is NULL");
    if (d->B <= 0 || d->Tq <= 0 || d->Lk <= 0 || d->H_q <= 0 || d->d_qk <= 0 || d->d_v <= 0 || d->k_sel <= 0 ||
        d->row_elems <= 0 || d->v_off < 0)
        return fail(IC_ERR_SHAPE, "attention sizes must be positive");
    if (d->H_q > IC_MAX_HEADS_Q) return fail(IC_ERR_UNSUPPORTED, "H_q=%d exceeds %d", d->H_q, IC_MAX_HEADS_Q);
    if (!ic::attn_shape_supported(d->d_qk, d->d_v))
        return fail(IC_ERR_UNSUPPORTED, "attention head dims not covered: d_qk=%d d_v=%d ((576,512) or (64,64))", d->d_qk, d->d_v);
    if (d->v_off % 8 != 0 || d->row_elems % 8 != 0)
        return fail(IC_ERR_SHAPE, "v_off and row_elems must be multiples of 8");
    const int staged = d->d_qk == 576 ? 576 : 128;   // features of a row the kernel stages
    if (d->v_off + d->d_v > staged || d->row_elems < staged)
        return fail(IC_ERR_UNSUPPORTED, "KV row layout not covered: need v_off+d_v <= %d <= row_elems", staged);
    if ((int64_t)d->B * d->Tq > INT32_MAX / 2) return fail(IC_ERR_SHAPE, "B*Tq too large");
    if (!(d->sm_scale > 0.f) || d->sm_scale > 1e6f) return fail(IC_ERR_SHAPE, "sm_scale must be positive and finite");
    return IC_OK;
}

// Workgroups one launch can have resident: MLA rows with the values in front run one workgroup per CU, the other
// layouts two.
int64_t attn_resident(const ic_attn_desc *d) { return (d->d_qk == 576 && d->v_off == 0) ? 256 : 512; }

// What is known about an index tensor: the causal top-k of this library for query rows at positions pos0 + t over the
// first lk keys (row t then holds the min(k_sel, pos0 + t + 1, lk) best of them and -1s behind); pos0 < 0: nothing.  lk
// is the Full layer's: a Shared layer's cache may be longer.
struct Causal {
    int64_t pos0;
    int32_t lk;
};
constexpr Causal kUnknown = {-1, 0};

// Entries that the longest row can hold, all of them in front.
int32_t held_entries(const ic_attn_desc *d, Causal c)
{
    if (c.pos0 < 0) return d->k_sel;
    return (int32_t)std::max<int64_t>(1, std::min<int64_t>(std::min(d->k_sel, c.lk), c.pos0 + d->Tq));
}

// The most key-slot splits per query a launch of n_layers layers uses, which sizes the workspace: one when the queries
// alone fill the chip, otherwise what brings their number up to that.
int64_t attn_max_splits(const ic_attn_desc *d, int n_layers)
{
    const int64_t nq = (int64_t)n_layers * d->B * d->Tq, wgs = attn_resident(d), tiles = (d->k_sel + 63) / 64;
    const int64_t want = nq >= wgs ? 1 : (wgs + nq - 1) / nq;
    const int64_t ns = want > tiles ? tiles : want;
    const int64_t per = (tiles + ns - 1) / ns;
    return (tiles + per - 1) / per;
}

// Partials of `parts` (query, split) pairs: outputs in bf16 or fp32 (wide), fp32 (max, sum).
size_t part_o_bytes(const ic_attn_desc *d, int64_t parts, bool wide) { return align_up((size_t)parts * d->H_q * d->d_v * (wide ? 4 : 2)); }
size_t split_bytes(const ic_attn_desc *d, int64_t parts, bool wide)
{
    return part_o_bytes(d, parts, wide) + align_up((size_t)parts * d->H_q * 2 * sizeof(float));
}

// Splits of a launch.  Workgroups run in rounds of attn_resident(), and a round takes as long as its longest workgroup:
// tiles plus what a workgroup pays once (launch, Q, first rows, output: about two tiles).  The merge launch costs about
// two tiles more.  One split too many can therefore double the time (40 queries x 7 splits of 5 tiles = 280 workgroups on
// 256 CUs took 36 us, 6 splits of 6 tiles take 30), so the number with the fewest tile times wins, the smaller at a tie.
// The rounding of bf16 partials weighs the more the fewer there are (relative distance from 64 bits: 32 of them 0.0022, 8
// 0.0023, 2 0.00244, no split or fp32 partials 0.0020).  A query in as many as one layer's launch may have, which is what
// the workspace is sized for, keeps them in bf16; in fewer they are fp32 (24 queries in 8 splits: 1.2 us more for the
// launch and its merge).
struct Splits {
    int n, len;
    bool wide;
    size_t bytes;
};
Splits attn_splits(const ic_attn_desc *d, int n_layers, size_t ws_bytes, int64_t narrow, Causal c = kUnknown)
{
    const int64_t nq = (int64_t)n_layers * d->B * d->Tq, wgs = attn_resident(d), tiles = (held_entries(d, c) + 63) / 64;
    int64_t best = 0;
    Splits r = {1, (int)tiles * 64, false, 0};
    for (int64_t ns = 1, most = std::min(tiles, attn_max_splits(d, n_layers)); ns <= most; ++ns) {
        const int64_t per = (tiles + ns - 1) / ns, n = (tiles + per - 1) / per;
        const bool wide = n > 1 && n < narrow;
        const size_t bytes = n > 1 ? split_bytes(d, nq * n, wide) : 0;
        if (bytes > ws_bytes) continue;
        const int64_t cost = (nq * n + wgs - 1) / wgs * (per + 2) + (n > 1 ? 2 : 0);
        if (best == 0 || cost < best) {
            best = cost;
            r = {(int)n, (int)per * 64, wide, bytes};
        }
    }
    return r;
}

// What one layer's launch has to have (0: it writes nothing into a workspace) and what serves it, or a run of layers, best.
size_t attn_ws_bytes(const ic_attn_desc *d)
{
    const size_t ns = (size_t)attn_max_splits(d, 1);
    if (ns <= 1) return 0;
    return split_bytes(d, (int64_t)d->B * d->Tq * (int64_t)ns, false);
}
size_t attn_best_bytes(const ic_attn_desc *d, int n_layers) { return attn_splits(d, n_layers, SIZE_MAX, attn_max_splits(d, 1)).bytes; }
size_t attn_query_bytes(const ic_attn_desc *d)
{
    const size_t least = attn_ws_bytes(d), best = attn_best_bytes(d, 1);
    return least > best ? least : best;
}

// Layers that one attention launch may take together: a Full layer and the Shared layers behind it read the same index
// tensor, so what is left is that their shapes agree and that no layer's output overlaps another one's inputs or output
// (called one after the other such layers would see each other's results).  Per layer, launches with few queries are
// mostly latency (a launch and its merge of one decode token: 13.5 us for 2.4 MB of rows) and a last round of a few
// workgroups.  576 / 512 rows: together up to twelve rounds of queries a layer, from where on the layers' caches in turn are
// worth as much as the launches saved.  Four layers of causal rows in the row forms, together / a launch each: 64 rows 11.9 / 36.5 us, 256 40 / 64, 700
// behind 1700 476 / 545, 2100 821 / 863, 3000 1430 / 1449, 4096 2195 / 2155.  Other rows: where an eighth of the tile
// times or more is saved.
struct Range {
    const char *p;
    size_t n;
    bool meets(const Range &o) const { return p < o.p + o.n && o.p < p + n; }
};
int attn_batch(const ic_layer *layers, int n, const ic_paged_cache *pc)
{
    const ic_attn_desc &d = layers[0].at;
    const size_t nq = (size_t)d.B * d.Tq;
    const size_t rows = pc && pc->page_table ? (size_t)d.B * pc->max_pages * pc->page_size : (size_t)d.B * d.Lk;
    auto q = [&](const ic_layer &l) { return Range{(const char *)l.Q, nq * d.H_q * d.d_qk * 2}; };
    auto kv = [&](const ic_layer &l) { return Range{(const char *)l.KV, rows * d.row_elems * 2}; };
    auto o = [&](const ic_layer &l) { return Range{(const char *)l.O, nq * d.H_q * d.d_v * 2}; };
    int m = 1;
    for (; m < n && m < ic::kMaxBatchLayers; ++m) {
        const ic_layer &l = layers[m];
        if (memcmp(&l.at, &d, sizeof d) != 0) break;
        bool apart = true;
        for (int j = 0; j < m && apart; ++j)
            apart = !o(l).meets(q(layers[j])) && !o(l).meets(kv(layers[j])) && !o(l).meets(o(layers[j])) &&
                    !o(layers[j]).meets(q(l)) && !o(layers[j]).meets(kv(l));
        if (!apart) break;
    }
    const int64_t wgs = attn_resident(&d), tiles = (d.k_sel + 63) / 64;
    if (wgs == 256) return (int64_t)nq < 12 * wgs ? m : 1;
    // in tile times, as in attn_splits(): rounds of (tiles + 2), 2 per launch
    const int64_t together = ((int64_t)(m * nq) + wgs - 1) / wgs * (tiles + 2) + 2, alone = m * (((int64_t)nq + wgs - 1) / wgs * (tiles + 2) + 2);
    return together * 8 <= alone * 7 ? m : 1;
}

// ragged / paged cache description -> the kernels' view (all-zero when pc is NULL)
ic::PagedView paged_view(const ic_paged_cache *pc)
{
    ic::PagedView v;
    memset(&v, 0, sizeof v);
    if (pc) {
        v.seq_lens = pc->seq_lens;
        v.page_table = pc->page_table;
        v.max_pages = pc->max_pages;
        int sh = 0;
        while ((1 << sh) < pc->page_size) ++sh;
        v.page_shift = sh;
    }
    return v;
}

ic_status check_paged(const ic_paged_cache *pc, int32_t Lk)
{
    if (!pc) return fail(IC_ERR_NULL, "paged cache descriptor is NULL");
    if (!pc->seq_lens && !pc->page_table) return fail(IC_ERR_NULL, "paged cache: seq_lens and page_table are both NULL");
    if (pc->page_table) {
        if (pc->page_size < 64 || (pc->page_size & (pc->page_size - 1)) != 0)
            return fail(IC_ERR_SHAPE, "page_size=%d must be a power of two >= 64", pc->page_size);
        if (pc->max_pages <= 0 || (int64_t)pc->max_pages * pc->page_size < Lk)
            return fail(IC_ERR_SHAPE, "page table rows of %d pages x %d positions do not cover Lk=%d", pc->max_pages, pc->page_size, Lk);
    }
    return IC_OK;
}

ic_status run_indexer(const ic_indexer_desc *d, const void *q, const void *k, const float *w, int32_t *idx,
                      float *sel, void *ws, size_t ws_bytes, hipStream_t st, const ic_paged_cache *pc = nullptr)
{
    const int64_t rows_cap = strip_rows(d, ws_bytes);
    const int Ri = (int)(d->Tq < rows_cap ? d->Tq : rows_cap);
    int64_t bc64 = rows_cap / Ri;
    const int Bc = (int)(bc64 < 1 ? 1 : (bc64 > d->B ? d->B : bc64));
    const size_t pw = parts_ws(d);
    void *const lists = pw != 0 && ws_bytes >= pw ? (char *)ws + align_up((size_t)d->B * d->Tq * strip_ld(d) * sizeof(float)) : nullptr;
    ic::ScoreArgs sa;
    memset(&sa, 0, sizeof sa);
    sa.q = q;
    sa.k = k;
    sa.w = w;
    sa.q_scale = d->q_scale;
    sa.k_scale = d->k_scale;
    sa.strip = (float *)ws;
    sa.ld = (int64_t)strip_ld(d);
    sa.q_pos0 = d->q_pos0;
    sa.Tq = d->Tq;
    sa.Lk = d->Lk;
    sa.H_I = d->H_I;
    sa.pv = paged_view(pc);
    ic::SelectArgs se;
    memset(&se, 0, sizeof se);
    se.strip = (const float *)ws;
    se.ld = sa.ld;
    se.q_pos0 = d->q_pos0;
    se.Tq = d->Tq;
    se.Lk = d->Lk;
    se.k_sel = d->k_sel;
    se.idx = idx;
    se.sel = sel;
    se.seq_lens = pc ? pc->seq_lens : nullptr;
    for (int b0 = 0; b0 < d->B; b0 += Bc) {
        const int bc = d->B - b0 < Bc ? d->B - b0 : Bc;
        for (int i0 = 0; i0 < d->Tq; i0 += Ri) {
            const int ri = d->Tq - i0 < Ri ? d->Tq - i0 : Ri;
            sa.b0 = b0;
            sa.i0 = i0;
            sa.Ri = ri;
            int64_t max_vis = d->q_pos0 + i0 + ri;
            max_vis = max_vis < 0 ? 0 : (max_vis > d->Lk ? d->Lk : max_vis);
            if (pc && pc->seq_lens) max_vis = d->Lk;   // ragged: lengths are device data, Lk bounds them
            if ((max_vis > d->k_sel || sel) && ic::topk_short(sa, d->dtype, d->d_I, bc * ri, max_vis)) {
                se.b0 = b0;
                se.i0 = i0;
                se.Ri = ri;
                ProfScope ps(0, st);
                hipError_t e = ic::launch_topk_short(sa, se, d->d_I, bc, st);
                if (e != hipSuccess) return fail(IC_ERR_HIP, "indexer launch failed: %s", hipGetErrorString(e));
                continue;
            }
            if (max_vis > d->k_sel || sel) {   // rows with <= k_sel visible keys need no scores
                ProfScope ps(0, st);
                hipError_t e = ic::launch_score(sa, d->dtype, d->d_I, bc, st);
                if (e != hipSuccess) return fail(IC_ERR_HIP, "indexer score launch failed: %s", hipGetErrorString(e));
            }
            se.b0 = b0;
            se.i0 = i0;
            se.Ri = ri;
            {
                ProfScope ps(1, st);
                const bool fit = se.seq_lens || ic::select_parts_fit(d->k_sel, (int)max_vis);   // (ragged: shorter than max_vis, maybe)
                hipError_t e = lists && fit && ic::select_parts(bc * ri, (int)max_vis) > 0
                                   ? ic::launch_select_parts(se, bc * ri, d->Lk, lists, st)
                                   : ic::launch_select(se, bc * ri, (int)max_vis, st);
                if (e != hipSuccess) return fail(IC_ERR_HIP, "top-k select launch failed: %s", hipGetErrorString(e));
            }
        }
    }
    g_indexer_launches.fetch_add(1);
    return IC_OK;
}

ic_status check_ws(void *ws, size_t have, size_t need)
{
    if (need == 0) return IC_OK;
    if (!ws) return fail(IC_ERR_WORKSPACE, "workspace is NULL but %zu bytes are needed", need);
    if (((uintptr_t)ws) % kAlign != 0) return fail(IC_ERR_WORKSPACE, "workspace must be %zu-byte aligned", kAlign);
    if (have < need) return fail(IC_ERR_WORKSPACE, "workspace too small: %zu < %zu bytes", have, need);
    return IC_OK;
}

size_t indexer_min_ws(const ic_indexer_desc *d)
{
    // at least kMinStripRows rows (or every row of one sequence when there are fewer)
    const int64_t rows = d->Tq < kMinStripRows ? d->Tq : kMinStripRows;
    return align_up((size_t)rows * strip_ld(d) * sizeof(float));
}

// Strip asked for when rows are not selected in parts.
size_t indexer_strip_ws(const ic_indexer_desc *d)
{
    const size_t row_bytes = strip_ld(d) * sizeof(float);
    const size_t all = (size_t)d->B * d->Tq * row_bytes;
    // small problems keep every row in flight; larger ones at most a quarter of their rows and at most the budget,
    // so that the scores of a long sequence are never all resident at once
    size_t want = all;
    if (all > kSmallStrip) {
        want = all / 4 > kSmallStrip ? all / 4 : kSmallStrip;
        if (want > kStripBudget) want = kStripBudget;
    }
    const size_t min_b = indexer_min_ws(d);
    if (want < min_b) want = min_b;
    return align_up(want / row_bytes * row_bytes);
}

// Leading query rows of every sequence that the dense form can take: the rows that select exactly the keys 0 .. pos0 + t, of
// which they see at most k_sel and all below lk.
int prefix_queries(const ic_attn_desc *d, Causal c)
{
    if (c.pos0 < 0 || attn_resident(d) != 256 || d->d_v != 512) return 0;
    const int32_t keys = c.lk < d->Lk ? c.lk : d->Lk;
    const int64_t n = (d->k_sel < keys ? d->k_sel : keys) - c.pos0;
    return (int)(n < 0 ? 0 : (n > d->Tq ? d->Tq : n));
}

// It stores 16 bytes of O at a time; the row form takes any address of a bf16.
bool dense_output(const void *O) { return (uintptr_t)O % 16 == 0; }

// The rules below weigh launches of 576 / 512 rows by their time in us, to about a tenth: fitted to 250 launches and runs of up to
// eight layers, 1 to 128 sequences of 1 to 2048 rows, of which the form taken is within 5 % of the fastest in all but eight (13 %).
constexpr double kLaunchUs = 9;                // an attention launch of the row forms until its workgroups are busy, and its end
constexpr double kGranuleUs = 0.61;            // 32 rows in the stream form; a query's Q is as many again
constexpr double kSplitTileUs = 3;             // 64 rows in the row-slab form with its queries split, merge included
constexpr double kDenseLaunchUs = 7;
constexpr double kDenseTileUs = 0.9;           // 32 keys of a block in the dense form
constexpr double kDenseBlockUs = 5;            // another block in a workgroup's chain
// Q and O of n queries at 5 TB/s
double query_us(const ic_attn_desc *d, int64_t n) { return (double)n * d->H_q * (d->d_qk + d->d_v) * 2 / 5e6; }

// Rows of one or more layers in the row forms: split, in short selections of resident queries, or in the stream form, in which the
// longest chain counts and which leaves the granules behind a causal row's last entry out.
double row_time(const ic_attn_desc *d, int n_layers, Causal c, size_t ws_bytes, int64_t narrow)
{
    const int64_t nq = (int64_t)n_layers * d->B * d->Tq, wgs = attn_resident(d), rounds = (nq + wgs - 1) / wgs;
    const Splits sp = attn_splits(d, n_layers, ws_bytes, narrow, c);
    if (sp.n > 1) return kLaunchUs + kSplitTileUs * (double)((nq * sp.n + wgs - 1) / wgs * (sp.len / 64));
    if (nq <= wgs && sp.len <= 128) return 6.5 + 2. * (sp.len / 64);
    const double longest = held_entries(d, c);
    double granules;
    if (rounds == 1) {
        granules = longest / 32 + 1;
    } else if (c.pos0 < 0 || c.pos0 >= d->k_sel) {
        granules = (double)rounds * (longest / 32 + 1);
    } else if (c.pos0 + d->Tq <= d->k_sel && (d->Tq % wgs == 0 || wgs % d->Tq == 0)) {
        // a chain takes the same places of every sequence and layer: the last one those at the end
        granules = (double)rounds * ((c.pos0 + 0.5 * (d->Tq + std::min<double>(d->Tq, (double)wgs))) / 32 + 1);
    } else {                                   // rows that hold fewer entries than k, and the others
        const double few = (double)std::min<int64_t>(d->Tq, d->k_sel - c.pos0);
        const double mean = (few * (c.pos0 + 0.5 * (few + 1)) + (d->Tq - few) * d->k_sel) / d->Tq;
        granules = (double)rounds * (mean / 32 + 1) + 0.5 * longest / 32 * (double)std::min<int64_t>(rounds, n_layers);
    }
    return kLaunchUs + std::max(kGranuleUs * granules + 0.3 * query_us(d, nq), query_us(d, nq));
}

// The first n rows of every sequence in the dense form: blocks of 64 (query, head) rows ranked by length, in chains there and back
// over the CUs, as long as the longest block or as a chain of those that all rounds of them have a block for.  Several layers
// take turns: their blocks of mean length, and half of what the longest has more.
double dense_time(const ic_attn_desc *d, int n, int64_t pos0, int n_layers = 1)
{
    const int64_t blocks = ((int64_t)n * d->H_q + 63) / 64 * d->B, rounds = (blocks * n_layers + 255) / 256;
    auto tiles = [&](double rank) { return (pos0 + std::max(0., n * (1 - rank / (double)blocks))) / 32 + 0.5; };
    // two rounds, there and back: twice the block at the turn
    const double pairs = (double)(rounds / 2), chain = 2 * pairs * tiles(256 * pairs) + (rounds % 2 ? tiles(256. * (double)(rounds - 1)) : 0.);
    double walk = std::max(kDenseTileUs * tiles(0), kDenseTileUs * chain + kDenseBlockUs * (double)(rounds - 1));
    if (n_layers > 1 && rounds > 1) {
        const double mean = tiles(0.5 * (double)blocks), all = (double)(blocks * n_layers) / 256 * mean + 0.5 * (tiles(0) - mean);
        walk = std::max(kDenseTileUs * tiles(0), kDenseTileUs * all + kDenseBlockUs * (double)(rounds - 1));
    }
    return kDenseLaunchUs + std::max(walk, query_us(d, (int64_t)n * d->B * n_layers));
}

ic_attn_desc rows_behind(const ic_attn_desc *d, int n)
{
    ic_attn_desc t = *d;
    t.Tq = d->Tq - n;
    return t;
}

// Layers whose dense rows share a launch: up to four rounds of blocks a layer, from where on a launch's start and end count
// nothing.  Four layers, together / a launch each, us a call: 256 rows 30 / 47, 512 62 / 101, 1000 169 / 196, 1024 173 / 200, 2048
// 575 / 580, 4 x 256 88 / 112, 16 x 32 36 / 43, 3 x 1021 514 / 520, 2 x 2048 1104 / 1105.
int dense_batch(const ic_attn_desc *d, int n) { return ((int64_t)n * d->H_q + 63) / 64 * d->B <= 4 * 256 ? ic::kMaxBatchLayers : 1; }

// How many of them it takes, for n_layers layers that the row forms would take together.  The rows behind (ws_bytes:
// workspace for their splits) are a launch of their own, with some 11 us for the two ends between them.  Measured, k = 2048, row forms / dense form (and
// what is left): 128 rows 12.5 / 12.6 us, 320 21.2 / 18.0, 1024 64 / 46, 4 x 64 11.8 / 11.9, 16 x 32 19.0 / 13.3, 256 rows behind 1792
// 48.5 / 54.7, 512 behind 1536 84 / 67; four layers: 128 rows 22 / 15.6, 512 82 / 53, 768 144 / 95, 16 x 32 39 / 32, 4 x 256
// 125 / 80; with rows left: 4 x 256 behind 1800 204 / 182, behind 1900 198 / 229, four layers 684 / 541 and 724 / 612.
int dense_queries(const ic_attn_desc *d, int n_layers, Causal c, size_t ws_bytes)
{
    const int n = prefix_queries(d, c);
    if (n == 0) return 0;
    const double whole = row_time(d, n_layers, c, ws_bytes, attn_max_splits(d, 1));
    const int m = std::min(n_layers, dense_batch(d, n));
    const double runs = (double)n_layers / m, dense = dense_time(d, n, c.pos0, m);
    if (n == d->Tq) return 0.97 * runs * dense <= whole ? n : 0;
    const ic_attn_desc t = rows_behind(d, n);
    return runs * (dense + 11 + row_time(&t, m, Causal{c.pos0 + n, c.lk}, ws_bytes, INT64_MAX)) <= whole ? n : 0;
}

// Workspace that serves the rows behind best.
size_t dense_tail_bytes(const ic_attn_desc *d, int n_layers, Causal c)
{
    const int n = dense_queries(d, n_layers, c, SIZE_MAX);
    if (n == 0 || n == d->Tq) return 0;
    const ic_attn_desc t = rows_behind(d, n);
    return attn_splits(&t, std::min(n_layers, dense_batch(d, n)), SIZE_MAX, INT64_MAX).bytes;
}

// Leading query rows of every sequence that may be whole prefixes when nothing is known about idx: in a causal selection
// for the last Tq of Lk positions, rows t < k_sel - (Lk - Tq).  Their number is then counted on the device (lead_kernel)
// and the dense form and what follows it read the counts.  Without the dense form a row costs k_sel / 32 granules
// however little of it is filled.  The rows behind the candidates go along with the candidates that the counts leave, or
// are split over the chip on their own.  Whichever of the two gains more on a causal selection than it loses on any other is
// taken if that difference is a seventh of what the candidates take in the row form; the scan and the launches that find nothing
// to do cost 8 us.  Measured, k = 2048, row form / this for causal rows / for other rows: 256 rows 43 / 21 / 49 us, 2048 rows
// 328 / 147 / 347, 4096 rows 667 / 490 / 696, 4 x 2060 rows 1354 / 601 / 1410; not taken: 700 rows behind 1700 keys 126 / 152
// / 131, 1000 behind 1500 161 / 184 / 176, 64 x 8 rows behind 2036 95 / 76 / 184.
struct LeadPlan {
    int n;
    bool along;
};
LeadPlan lead_plan(const ic_attn_desc *d)
{
    const int64_t pos0 = (int64_t)d->Lk - d->Tq;
    const int n = pos0 < 0 ? 0 : prefix_queries(d, Causal{pos0, d->Lk});
    const LeadPlan none = {0, false};
    if (n == 0) return none;
    auto unsplit = [&](int64_t rows) { return rows == 0 ? 0. : kLaunchUs + kGranuleUs * (double)((d->B * rows + 255) / 256) * (d->k_sel / 32. + 1); };
    const double whole = row_time(d, 1, kUnknown, SIZE_MAX, attn_max_splits(d, 1)), dense = dense_time(d, n, pos0) + 8;
    const ic_attn_desc t = rows_behind(d, n);
    // gain on causal rows minus loss on others
    const double along = whole - (dense + unsplit(t.Tq)) - (unsplit(d->Tq) + 8 - whole);
    double apart = 2 * whole;
    if (t.Tq > 0 && (int64_t)d->B * t.Tq < 256) {
        const double tail = row_time(&t, 1, kUnknown, SIZE_MAX, INT64_MAX);
        apart -= dense + tail + unsplit(n) + tail + 8;
    } else {
        apart = along;                         // (nothing to split)
    }
    if (std::max(along, apart) < 0.15 * (whole - unsplit(t.Tq))) return none;
    return {n, along >= apart};
}
int lead_queries(const ic_attn_desc *d) { return lead_plan(d).n; }

int lead_chunks(int n) { return (n + ic::kLeadChunk - 1) / ic::kLeadChunk; }

size_t lead_bytes(const ic_attn_desc *d, int n_tensors)
{
    const int n = lead_queries(d);
    return n ? align_up((size_t)n_tensors * d->B * lead_chunks(n) * sizeof(int32_t)) : 0;
}

// Partials of the rows behind the candidates where they are split over the chip on their own.
size_t lead_tail_bytes(const ic_attn_desc *d)
{
    const LeadPlan lp = lead_plan(d);
    if (lp.n == 0 || lp.n == d->Tq || lp.along) return 0;
    const ic_attn_desc t = rows_behind(d, lp.n);
    return attn_splits(&t, 1, SIZE_MAX, INT64_MAX).bytes;
}

// Counts of n_tensors index tensors into lead.
ic_status count_lead(const ic_attn_desc *d, const int32_t *const *idx, int n_tensors, int32_t *lead, hipStream_t st)
{
    ic::LeadArgs la;
    memset(&la, 0, sizeof la);
    for (int i = 0; i < n_tensors; ++i) la.idx[i] = idx[i];
    la.lead = lead;
    la.B = d->B;
    la.Tq = d->Tq;
    la.k_sel = d->k_sel;
    la.pos0 = d->Lk - d->Tq;
    la.n_rows = lead_queries(d);
    la.n_chunks = lead_chunks(la.n_rows);
    hipError_t e = ic::launch_lead(la, n_tensors, st);
    if (e != hipSuccess) return fail(IC_ERR_HIP, "index scan launch failed: %s", hipGetErrorString(e));
    return IC_OK;
}

ic::AttnArgs attn_args(const ic_layer *layers, int n_layers, const int32_t *idx, float *lse, const ic_paged_cache *pc,
                       Causal c)
{
    const ic_attn_desc *d = &layers[0].at;
    ic::AttnArgs a;
    memset(&a, 0, sizeof a);
    a.Q = layers[0].Q;
    a.KV = layers[0].KV;
    a.O = layers[0].O;
    for (int l = 0; l < n_layers; ++l) {
        a.Qs[l] = layers[l].Q;
        a.KVs[l] = layers[l].KV;
        a.Os[l] = layers[l].O;
    }
    a.n_layers = n_layers;
    a.idx = idx;
    a.lse = lse;
    a.B = d->B;
    a.Tq = d->Tq;
    a.Lk = d->Lk;
    a.H_q = d->H_q;
    a.v_off = d->v_off;
    a.row_elems = d->row_elems;
    a.k_sel = d->k_sel;
    a.scale_log2e = d->sm_scale * 1.4426950408889634f;
    a.pv = paged_view(pc);
    a.causal_pos0 = c.pos0;
    return a;
}

// skipped > 0: the last Tq rows of every sequence, behind `skipped` others that another launch has taken (Q, O, idx and lse
// point to sequence 0's first one).  Undivided they were not split, so their partials are fp32.
ic_status run_attn_layers(const ic_layer *layers, int n_layers, const int32_t *idx, float *lse, void *ws, size_t ws_bytes,
                          hipStream_t st, const ic_paged_cache *pc, Causal c, int skipped = 0);

// A layer with an index tensor whose leading rows are counted (lead); lead2: counts of a second tensor, only the rows that are
// leading in both are left out.
struct LeadJob {
    ic_layer L;
    const int32_t *idx, *lead, *lead2;
};

// The leading rows of layers of one shape whose counts follow one another.
ic_status run_lead_dense(const LeadJob *jobs, int n_jobs, float *lse, hipStream_t st)
{
    const ic_attn_desc *d = &jobs[0].L.at;
    const int n = lead_queries(d);
    ProfScope ps(2, st);
    const ic::DenseArgs da{n, d->Lk - d->Tq, jobs[0].lead, lead_chunks(n)};
    ic::AttnArgs a = attn_args(&jobs[0].L, 1, jobs[0].idx, lse, nullptr, kUnknown);
    a.n_layers = n_jobs;
    for (int i = 0; i < n_jobs; ++i) {
        a.Qs[i] = jobs[i].L.Q;
        a.KVs[i] = jobs[i].L.KV;
        a.Os[i] = jobs[i].L.O;
    }
    hipError_t e = ic::launch_attn_dense(a, da, st);
    if (e != hipSuccess) return fail(IC_ERR_HIP, "dense attention launch failed: %s", hipGetErrorString(e));
    return IC_OK;
}

// The other rows of up to kMaxBatchLayers layers of one shape.  (A launch takes up to kRestSeqs sequences; lse: one layer only.)
ic_status run_lead_rest(const LeadJob *jobs, int n_jobs, float *lse, void *ws, size_t ws_bytes, hipStream_t st)
{
    const ic_attn_desc *d = &jobs[0].L.at;
    const LeadPlan lp = lead_plan(d);
    const int n = lp.n, n_chunks = lead_chunks(n);
    const bool along = lp.along;
    const int most = std::max(1, ic::kRestSeqs / n_jobs);
    for (int b0 = 0; b0 < d->B; b0 += most) {
        ProfScope ps(2, st);
        ic::AttnArgs a = attn_args(&jobs[0].L, 1, jobs[0].idx, lse ? lse + (int64_t)b0 * d->Tq * d->H_q : nullptr, nullptr, kUnknown);
        a.n_splits = 1;
        a.split_len = (d->k_sel + 63) / 64 * 64;
        a.B = std::min(most, d->B - b0);
        ic::RestArgs ra;
        memset(&ra, 0, sizeof ra);
        ra.n_jobs = n_jobs;
        ra.n_chunks = n_chunks;
        ra.n_rows = along ? d->Tq : n;
        const int64_t r0 = (int64_t)b0 * d->Tq;
        for (int i = 0; i < n_jobs; ++i) {
            const LeadJob &j = jobs[i];
            a.Qs[i] = (const char *)j.L.Q + r0 * d->H_q * d->d_qk * 2;
            a.KVs[i] = (const char *)j.L.KV + (int64_t)b0 * d->Lk * d->row_elems * 2;
            a.Os[i] = (char *)j.L.O + r0 * d->H_q * d->d_v * 2;
            ra.idx[i] = j.idx + r0 * d->k_sel;
            ra.lead[i] = j.lead + (int64_t)b0 * n_chunks;
            ra.lead2[i] = j.lead2 + (int64_t)b0 * n_chunks;
        }
        a.Q = a.Qs[0];                         // (one sequence of one layer is read here)
        a.KV = a.KVs[0];
        a.O = a.Os[0];
        a.idx = ra.idx[0];
        hipError_t e = ic::launch_attn_rest(a, ra, st);
        if (e != hipSuccess) return fail(IC_ERR_HIP, "sparse attention launch failed: %s", hipGetErrorString(e));
    }
    if (along || n == d->Tq) return IC_OK;
    for (int i = 0; i < n_jobs; ++i) {
        ic_layer r = jobs[i].L;
        r.at = rows_behind(d, n);
        r.Q = (const char *)r.Q + (int64_t)n * d->H_q * d->d_qk * 2;
        r.O = (char *)r.O + (int64_t)n * d->H_q * d->d_v * 2;
        const ic_status s = run_attn_layers(&r, 1, jobs[i].idx + (int64_t)n * d->k_sel, lse ? lse + (int64_t)n * d->H_q : nullptr, ws,
                                            ws_bytes, st, nullptr, kUnknown, n);
        if (s != IC_OK) return s;
    }
    return IC_OK;
}

// c: idx is this library's own (rows that can hold fewer than k_sel entries end in -1s, and the kernels leave their empty
// tiles out) or the caller's (kUnknown)
ic_status run_attn_layers(const ic_layer *layers, int n_layers, const int32_t *idx, float *lse, void *ws, size_t ws_bytes,
                          hipStream_t st, const ic_paged_cache *pc, Causal c, int skipped)
{
    const ic_attn_desc *d = &layers[0].at;
    ic::AttnArgs a = attn_args(layers, n_layers, idx, lse, pc, c);
    if (d->B > 1) a.row_gap = skipped;
    const Splits sp = attn_splits(d, n_layers, ws_bytes, skipped > 0 ? INT64_MAX : attn_max_splits(d, 1), c);
    a.n_splits = sp.n;
    a.split_len = sp.len;
    if (sp.n > 1) {
        a.part_o = ws;
        a.part_wide = sp.wide;
        a.part_ml = (float *)((char *)ws + part_o_bytes(d, (int64_t)n_layers * d->B * d->Tq * sp.n, sp.wide));
    }
    {
        ProfScope ps(2, st);
        hipError_t e = ic::launch_attn(a, d->d_qk, d->d_v, st);
        if (e != hipSuccess) return fail(IC_ERR_HIP, "sparse attention launch failed: %s", hipGetErrorString(e));
    }
    if (a.n_splits > 1) {
        ProfScope ps(3, st);
        hipError_t e = ic::launch_attn_merge(a, d->d_v, st);
        if (e != hipSuccess) return fail(IC_ERR_HIP, "attention merge launch failed: %s", hipGetErrorString(e));
    }
    return IC_OK;
}

// Layers whose first nd rows of every sequence are whole prefixes: those in the dense form, then the others.
ic_status run_attn_dense(const ic_layer *L, int n_layers, int nd, const int32_t *idx, void *ws, size_t ws_bytes, hipStream_t st,
                         const ic_paged_cache *pc, Causal c)
{
    const ic_attn_desc *d = &L->at;
    {
        ProfScope ps(2, st);                   // (the rows behind them are timed by their own launch)
        const ic::DenseArgs da{nd, (int32_t)c.pos0, nullptr, 0};
        hipError_t e = ic::launch_attn_dense(attn_args(L, n_layers, idx, nullptr, pc, c), da, st);
        if (e != hipSuccess) return fail(IC_ERR_HIP, "dense attention launch failed: %s", hipGetErrorString(e));
    }
    if (nd == d->Tq) return IC_OK;
    ic_layer r[ic::kMaxBatchLayers];
    for (int l = 0; l < n_layers; ++l) {
        r[l] = L[l];
        r[l].at = rows_behind(d, nd);
        r[l].Q = (const char *)r[l].Q + (int64_t)nd * d->H_q * d->d_qk * 2;
        r[l].O = (char *)r[l].O + (int64_t)nd * d->H_q * d->d_v * 2;
    }
    return run_attn_layers(r, n_layers, idx + (int64_t)nd * d->k_sel, nullptr, ws, ws_bytes, st, pc, Causal{c.pos0 + nd, c.lk}, nd);
}

ic_layer attn_layer(const ic_attn_desc *d, const void *Q, const void *KV, void *O)
{
    ic_layer l;
    memset(&l, 0, sizeof l);
    l.at = *d;
    l.Q = Q;
    l.KV = KV;
    l.O = O;
    return l;
}

ic_status run_attn(const ic_attn_desc *d, const void *Q, const void *KV, const int32_t *idx, void *O, float *lse,
                   void *ws, size_t ws_bytes, hipStream_t st, const ic_paged_cache *pc = nullptr)
{
    const ic_layer l = attn_layer(d, Q, KV, O);
    return run_attn_layers(&l, 1, idx, lse, ws, ws_bytes, st, pc, kUnknown);
}

} // namespace

extern "C" {

const char *ic_last_error(void) { return g_err; }

size_t ic_indexer_topk_workspace(const ic_indexer_desc *d)
{
    if (check_indexer(d) != IC_OK) return 0;
    if (const size_t pw = parts_ws(d)) return pw;
    return indexer_strip_ws(d);
}

ic_status ic_indexer_topk(const ic_indexer_desc *d, const void *q, const void *k, const float *w, int32_t *idx,
                          float *sel_scores, void *workspace, size_t workspace_bytes, void *stream)
{
    ic_status s = check_indexer(d);
    if (s != IC_OK) return s;
    if (!q || !k || !w || !idx) return fail(IC_ERR_NULL, "q, k, w and idx must not be NULL");
    s = check_ws(workspace, workspace_bytes, indexer_min_ws(d));
    if (s != IC_OK) return s;
    return run_indexer(d, q, k, w, idx, sel_scores, workspace, workspace_bytes, (hipStream_t)stream);
}

size_t ic_sparse_attn_workspace(const ic_attn_desc *d)
{
    if (check_attn(d) != IC_OK) return 0;
    return attn_query_bytes(d);
}

size_t ic_sparse_attn_lead_workspace(const ic_attn_desc *d)
{
    if (check_attn(d) != IC_OK) return 0;
    const size_t lb = lead_bytes(d, 1);
    return lb ? lb + align_up(lead_tail_bytes(d)) : attn_query_bytes(d);
}

ic_status ic_sparse_attn_lead(const ic_attn_desc *d, const void *Q, const void *KV, const int32_t *idx, void *O,
                              float *lse, void *workspace, size_t workspace_bytes, void *stream)
{
    ic_status s = check_attn(d);
    if (s != IC_OK) return s;
    if (!Q || !KV || !idx || !O) return fail(IC_ERR_NULL, "Q, KV, idx and O must not be NULL");
    s = check_ws(workspace, workspace_bytes, ic_sparse_attn_lead_workspace(d));
    if (s != IC_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    const size_t lb = lead_bytes(d, 1);
    if (lb == 0 || !dense_output(O)) return run_attn(d, Q, KV, idx, O, lse, workspace, workspace_bytes, st);
    int32_t *const lead = (int32_t *)workspace;
    s = count_lead(d, &idx, 1, lead, st);
    if (s != IC_OK) return s;
    const LeadJob job = {attn_layer(d, Q, KV, O), idx, lead, lead};
    s = run_lead_dense(&job, 1, lse, st);
    return s != IC_OK ? s : run_lead_rest(&job, 1, lse, (char *)workspace + lb, workspace_bytes - lb, st);
}

ic_status ic_sparse_attn(const ic_attn_desc *d, const void *Q, const void *KV, const int32_t *idx, void *O,
                         float *lse, void *workspace, size_t workspace_bytes, void *stream)
{
    ic_status s = check_attn(d);
    if (s != IC_OK) return s;
    if (!Q || !KV || !idx || !O) return fail(IC_ERR_NULL, "Q, KV, idx and O must not be NULL");
    s = check_ws(workspace, workspace_bytes, attn_ws_bytes(d));
    if (s != IC_OK) return s;
    return run_attn(d, Q, KV, idx, O, lse, workspace, workspace_bytes, (hipStream_t)stream);
}

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of the current GPU's copy of `scratch`, looked up once per device.
ic_status static_scratch(void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(IC_ERR_HIP, "hipGetDevice failed: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(IC_ERR_UNSUPPORTED, "device ordinal %d outside [0, %d)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(IC_ERR_HIP, "address of the static scratch on device %d: %s", dev, hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return IC_OK;
}
} // namespace

ic_status ic_sparse_attn_static(const ic_attn_desc *d, const void *Q, const void *KV, const int32_t *idx, void *O,
                                float *lse, void *stream)
{
    ic_status s = check_attn(d);
    if (s != IC_OK) return s;
    if (!Q || !KV || !idx || !O) return fail(IC_ERR_NULL, "Q, KV, idx and O must not be NULL");
    const size_t need = attn_ws_bytes(d);
    if (need > (size_t)IC_STATIC_SCRATCH_BYTES)
        return fail(IC_ERR_WORKSPACE, "this shape needs %zu bytes of split-attention scratch, the static scratch holds %zu",
                    need, (size_t)IC_STATIC_SCRATCH_BYTES);
    void *ws = nullptr;
    if (need > 0) {
        s = static_scratch(&ws);
        if (s != IC_OK) return s;
    }
    return run_attn(d, Q, KV, idx, O, lse, ws, need > 0 ? (size_t)IC_STATIC_SCRATCH_BYTES : 0, (hipStream_t)stream);
}

static ic_status check_stack(const ic_layer *layers, int32_t n, const uint8_t *full_mask)
{
    if (!layers) return fail(IC_ERR_NULL, "layers is NULL");
    if (n <= 0) return fail(IC_ERR_SHAPE, "n_layers must be positive");
    if (full_mask) {
        if (!full_mask[0]) return fail(IC_ERR_PATTERN, "the first layer must be Full: there are no indices to reuse yet");
    }
    int32_t idx_lk = 0;                        // key range the cached indices were drawn from (the last Full layer's)
    for (int l = 0; l < n; ++l) {
        const ic_layer *L = &layers[l];
        const bool full = !full_mask || full_mask[l];
        ic_status s = check_attn(&L->at);
        if (s != IC_OK) return s;
        if (!L->Q || !L->KV || !L->O) return fail(IC_ERR_NULL, "layer %d: Q, KV and O must not be NULL", l);
        if (full) {
            s = check_indexer(&L->ix);
            if (s != IC_OK) return s;
            if (!L->q || !L->k || !L->w) return fail(IC_ERR_NULL, "Full layer %d: q, k and w must not be NULL", l);
            if (L->ix.B != L->at.B || L->ix.Tq != L->at.Tq || L->ix.k_sel != L->at.k_sel)
                return fail(IC_ERR_SHAPE, "layer %d: indexer and attention disagree on B, Tq or k_sel", l);
            if (L->ix.Lk != L->at.Lk)
                return fail(IC_ERR_SHAPE, "layer %d: indexer scores %d keys but the KV cache holds %d rows", l, L->ix.Lk, L->at.Lk);
            idx_lk = L->ix.Lk;
        } else if (L->at.Lk < idx_lk) {
            // a Shared layer reads positions selected among idx_lk keys: its own cache must hold them all
            return fail(IC_ERR_SHAPE, "Shared layer %d: its KV cache holds %d rows, the inherited indices cover %d", l, L->at.Lk, idx_lk);
        }
        if (L->at.B != layers[0].at.B || L->at.Tq != layers[0].at.Tq || L->at.k_sel != layers[0].at.k_sel)
            return fail(IC_ERR_SHAPE, "layer %d: all layers must share B, Tq and k_sel (one index buffer)", l);
    }
    return IC_OK;
}

size_t ic_forward_stack_workspace(const ic_layer *layers, int32_t n_layers)
{
    if (!layers || n_layers <= 0) return 0;
    size_t need = 0;
    for (int l = 0; l < n_layers; ++l) {
        size_t a = ic_sparse_attn_workspace(&layers[l].at);
        size_t b = layers[l].q ? ic_indexer_topk_workspace(&layers[l].ix) : 0;
        const bool ok = check_attn(&layers[l].at) == IC_OK;
        for (int m = 1; ok && layers[l].q && layers[l].ix.q_pos0 >= 0 && m <= std::min(n_layers - l, ic::kMaxBatchLayers); ++m)
            a = std::max(a, dense_tail_bytes(&layers[l].at, m, Causal{layers[l].ix.q_pos0, layers[l].ix.Lk}));
        // which layers are Full is not known here: room for any run of layers of this shape
        if (ok && attn_ws_bytes(&layers[l].at) > 0) {
            const int run = n_layers - l < ic::kMaxBatchLayers ? n_layers - l : ic::kMaxBatchLayers;
            for (int m = 2; m <= run && memcmp(&layers[l + m - 1].at, &layers[l].at, sizeof layers[l].at) == 0; ++m) {
                const size_t am = attn_best_bytes(&layers[l].at, m);
                if (am > a) a = am;
            }
        }
        if (a > need) need = a;
        if (b > need) need = b;
    }
    return need;
}

static ic_status forward_stack_impl(const ic_layer *layers, int32_t n_layers, const uint8_t *full_mask, const ic_paged_cache *pc,
                                    int32_t *idx_cache, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!full_mask) return fail(IC_ERR_NULL, "full_mask is NULL");
    if (!idx_cache) return fail(IC_ERR_NULL, "idx_cache is NULL");
    ic_status s = check_stack(layers, n_layers, full_mask);
    if (s != IC_OK) return s;
    if (pc) {
        for (int l = 0; l < n_layers; ++l) {
            s = check_paged(pc, layers[l].at.Lk);
            if (s != IC_OK) return s;
            if (full_mask[l] && pc->page_table && layers[l].ix.dtype != IC_BF16)
                return fail(IC_ERR_UNSUPPORTED, "layer %d: a paged index-key cache must be bf16", l);
        }
    }
    size_t need = 0;
    for (int l = 0; l < n_layers; ++l) {
        size_t a = attn_ws_bytes(&layers[l].at);
        size_t b = full_mask[l] ? indexer_min_ws(&layers[l].ix) : 0;
        if (a > need) need = a;
        if (b > need) need = b;
    }
    s = check_ws(workspace, workspace_bytes, need);
    if (s != IC_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    Causal known = kUnknown;                   // of the cached indices
    for (int l = 0; l < n_layers; ++l) {
        const ic_layer *L = &layers[l];
        if (full_mask[l]) {   // Full: fresh indices overwrite the cache; Shared: cache left as it is
            s = run_indexer(&L->ix, L->q, L->k, L->w, idx_cache, nullptr, workspace, workspace_bytes, st, pc);
            if (s != IC_OK) return s;
            known = (pc && pc->seq_lens) || L->ix.q_pos0 < 0 ? kUnknown : Causal{L->ix.q_pos0, L->ix.Lk};
        }
        int run = 1;                           // this layer and the Shared layers behind it
        while (l + run < n_layers && !full_mask[l + run]) ++run;
        int m = attn_batch(L, run, pc);
        while (m > 1 && attn_best_bytes(&L->at, m) > workspace_bytes) --m;
        int stored = 0;                        // the first of them, whose outputs the dense form can store
        while (stored < m && dense_output(L[stored].O)) ++stored;
        const int nd = stored ? dense_queries(&L->at, stored, known, workspace_bytes) : 0;
        if (nd) m = std::min(stored, dense_batch(&L->at, nd));
        s = nd ? run_attn_dense(L, m, nd, idx_cache, workspace, workspace_bytes, st, pc, known)
               : run_attn_layers(L, m, idx_cache, nullptr, workspace, workspace_bytes, st, pc, known);
        if (s != IC_OK) return s;
        l += m - 1;
    }
    return IC_OK;
}

ic_status ic_forward_stack(const ic_layer *layers, int32_t n_layers, const uint8_t *full_mask, int32_t *idx_cache,
                           void *workspace, size_t workspace_bytes, void *stream)
{
    return forward_stack_impl(layers, n_layers, full_mask, nullptr, idx_cache, workspace, workspace_bytes, stream);
}

ic_status ic_forward_stack_paged(const ic_layer *layers, int32_t n_layers, const uint8_t *full_mask, const ic_paged_cache *pc,
                                 int32_t *idx_cache, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!pc) return fail(IC_ERR_NULL, "paged cache descriptor is NULL");
    return forward_stack_impl(layers, n_layers, full_mask, pc, idx_cache, workspace, workspace_bytes, stream);
}

ic_status ic_indexer_topk_paged(const ic_indexer_desc *d, const ic_paged_cache *pc, const void *q, const void *k_pool,
                                const float *w, int32_t *idx, float *sel_scores, void *workspace, size_t workspace_bytes,
                                void *stream)
{
    ic_status s = check_indexer(d);
    if (s != IC_OK) return s;
    s = check_paged(pc, d->Lk);
    if (s != IC_OK) return s;
    if (pc->page_table && d->dtype != IC_BF16) return fail(IC_ERR_UNSUPPORTED, "a paged index-key cache must be bf16");
    if (!q || !k_pool || !w || !idx) return fail(IC_ERR_NULL, "q, k_pool, w and idx must not be NULL");
    s = check_ws(workspace, workspace_bytes, indexer_min_ws(d));
    if (s != IC_OK) return s;
    return run_indexer(d, q, k_pool, w, idx, sel_scores, workspace, workspace_bytes, (hipStream_t)stream, pc);
}

ic_status ic_sparse_attn_paged(const ic_attn_desc *d, const ic_paged_cache *pc, const void *Q, const void *KV_pool,
                               const int32_t *idx, void *O, float *lse, void *workspace, size_t workspace_bytes, void *stream)
{
    ic_status s = check_attn(d);
    if (s != IC_OK) return s;
    s = check_paged(pc, d->Lk);
    if (s != IC_OK) return s;
    if (!Q || !KV_pool || !idx || !O) return fail(IC_ERR_NULL, "Q, KV_pool, idx and O must not be NULL");
    s = check_ws(workspace, workspace_bytes, attn_ws_bytes(d));
    if (s != IC_OK) return s;
    return run_attn(d, Q, KV_pool, idx, O, lse, workspace, workspace_bytes, (hipStream_t)stream, pc);
}

ic_status ic_pattern_from_string(const char *fs, uint8_t *full_mask, int32_t n)
{
    if (!fs || !full_mask) return fail(IC_ERR_NULL, "pattern string and mask must not be NULL");
    if (n <= 0) return fail(IC_ERR_SHAPE, "n must be positive");
    if ((int64_t)strlen(fs) != n) return fail(IC_ERR_SHAPE, "pattern has %zu characters, expected %d", strlen(fs), n);
    for (int l = 0; l < n; ++l) {
        if (fs[l] == 'F')
            full_mask[l] = 1;
        else if (fs[l] == 'S')
            full_mask[l] = 0;
        else
            return fail(IC_ERR_PATTERN, "pattern character %d is '%c', expected F or S", l, fs[l]);
    }
    if (!full_mask[0]) return fail(IC_ERR_PATTERN, "the first layer must be Full");
    return IC_OK;
}

ic_status ic_pattern_uniform(int32_t n, int32_t r, uint8_t *full_mask)
{
    if (!full_mask) return fail(IC_ERR_NULL, "mask must not be NULL");
    if (n <= 0 || r <= 0) return fail(IC_ERR_SHAPE, "n and r must be positive");
    for (int l = 0; l < n; ++l) full_mask[l] = (l % r) == 0;
    return IC_OK;
}

size_t ic_cosine_rows_workspace(void) { return kAlign; }

ic_status ic_cosine_rows(const void *A, const void *B, int64_t n_rows, int64_t row_len, double *mean, float *per_row,
                         void *workspace, size_t workspace_bytes, void *stream)
{
    if (!A || !B || !mean) return fail(IC_ERR_NULL, "A, B and mean must not be NULL");
    if (n_rows <= 0 || row_len <= 0 || n_rows > INT32_MAX) return fail(IC_ERR_SHAPE, "n_rows and row_len must be positive");
    ic_status s = check_ws(workspace, workspace_bytes, ic_cosine_rows_workspace());
    if (s != IC_OK) return s;
    hipError_t e = ic::launch_cosine(A, B, n_rows, row_len, mean, per_row, (double *)workspace, (hipStream_t)stream);
    if (e != hipSuccess) return fail(IC_ERR_HIP, "cosine launch failed: %s", hipGetErrorString(e));
    return IC_OK;
}

namespace {

// layers of the similarity matrix share one attention shape (any layer's index tensor fits any layer)
ic_status check_sim_layers(const ic_layer *layers, int32_t n_layers)
{
    if (!layers) return fail(IC_ERR_NULL, "layers is NULL");
    if (n_layers <= 0 || n_layers > IC_MAX_OVERLAP_LAYERS)
        return fail(IC_ERR_SHAPE, "n_layers must be in [1, %d]", IC_MAX_OVERLAP_LAYERS);
    for (int l = 0; l < n_layers; ++l) {
        ic_status s = check_attn(&layers[l].at);
        if (s != IC_OK) return s;
        if (!layers[l].Q || !layers[l].KV || !layers[l].O) return fail(IC_ERR_NULL, "layer %d: Q, KV and O must not be NULL", l);
        const ic_attn_desc &a = layers[l].at, &b = layers[0].at;
        if (a.B != b.B || a.Tq != b.Tq || a.k_sel != b.k_sel || a.H_q != b.H_q || a.d_v != b.d_v)
            return fail(IC_ERR_SHAPE, "layer %d: attention shape differs from layer 0", l);
    }
    return IC_OK;
}

// counts of the layers' leading rows (layers of one cache length only: the counts depend on it)
size_t sim_lead_bytes(const ic_layer *layers, int n_layers)
{
    for (int l = 1; l < n_layers; ++l)
        if (layers[l].at.Lk != layers[0].at.Lk || lead_queries(&layers[l].at) != lead_queries(&layers[0].at)) return 0;
    return lead_bytes(&layers[0].at, n_layers);
}

size_t sim_o_bytes(const ic_attn_desc *a) { return align_up((size_t)a->B * a->Tq * a->H_q * a->d_v * 2); }

// What the rows that are the same in both outputs of a pair compare to, per layer.
size_t sim_self_bytes(const ic_attn_desc *a, int n_layers) { return align_up((size_t)n_layers * a->B * a->Tq * sizeof(double)); }

// Outputs under reused indices that are computed, and compared, together where leading rows are counted: few rows of a pair are
// left (a third of 3000), and every launch of them ends in a round of a part of the CUs (952 rows: 3.7 rounds in four).  Up to
// 1 GiB of them: a launch of more rows loses less.
constexpr size_t kSimOutputs = (size_t)1 << 30;
int sim_outputs(const ic_attn_desc *a, int n_layers)
{
    const int64_t pairs = (int64_t)n_layers * (n_layers - 1) / 2, fit = (int64_t)(kSimOutputs / sim_o_bytes(a));
    return (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(pairs, fit), ic::kMaxBatchLayers));
}

// The first layer whose rows are compared to themselves ahead of the pairs (n_layers: none): layer i is asked by i pairs.  Few rows are
// 16 us of latency a launch, 7 where all is known; many read an output at 4 TB/s.  us for all comparisons, ahead from layer 0 / 2 / none: 3 layers of
// 557 rows 23 / 34 / 18; 2 of 5000 rows 122 / 41 / 41; 6 of 3000 about 155 / 127 / 360.
int sim_self_from(const ic_attn_desc *a, int n_layers, int n_out)
{
    const double read = (double)sim_o_bytes(a) / 4e6;
    const int pairs = n_layers * (n_layers - 1) / 2, launches = (pairs + n_out - 1) / n_out;
    const double none = std::max(16. * launches, read * pairs);
    const double one = std::max(16., read * (n_layers - 1)) + 7 * launches;
    const double two = n_layers > 2 ? std::max(16., read * (n_layers - 2)) + std::max(16., read) + 7 * (launches - 1) : none;
    return none <= std::min(one, two) ? n_layers : (one < two ? 1 : 2);
}

// Whether no layer's output overlaps another one's output or inputs: only then may they all be written before the first pair
// is compared.
bool sim_apart(const ic_layer *layers, int n_layers)
{
    const ic_attn_desc *d = &layers[0].at;
    const size_t nq = (size_t)d->B * d->Tq, ob = nq * d->H_q * d->d_v * 2, qb = nq * d->H_q * d->d_qk * 2;
    for (int i = 0; i < n_layers; ++i) {
        const Range o{(const char *)layers[i].O, ob};
        for (int j = 0; j < n_layers; ++j) {
            if (j == i) continue;
            const ic_layer &l = layers[j];
            if (o.meets(Range{(const char *)l.O, ob}) || o.meets(Range{(const char *)l.Q, qb}) ||
                o.meets(Range{(const char *)l.KV, (size_t)d->B * l.at.Lk * l.at.row_elems * 2}))
                return false;
        }
    }
    return true;
}

// The layers whose leading rows are counted: outputs under their own indices, and for every pair those under reused ones.  Rows
// that are whole prefixes in both index tensors of a pair select the same keys in the same order, so their outputs are the
// layer's own and nothing is left to compute.  Layers that are not apart are finished one after the other.  (No containers: an
// allocation that fails would throw through the C entry.)
ic_status run_similarity(const ic_layer *layers, int n_layers, const int32_t *const *idx, double *S, int32_t *lead, double *self,   // (self: or nullptr)
                         char *o_reuse, int n_out, void *ws, size_t ws_bytes, hipStream_t st)
{
    const ic_attn_desc *d = &layers[0].at;
    const int64_t n_rows = (int64_t)d->B * d->Tq;
    const int n_chunks = lead_chunks(lead_queries(d));
    auto counts = [&](int l) { return lead + (int64_t)l * d->B * n_chunks; };
    const int self_from = self ? sim_self_from(d, n_layers, n_out) : n_layers;
    auto self_of = [&](int l) -> double * { return l >= self_from ? self + l * n_rows : nullptr; };
    ic::CosineArgs c0;
    memset(&c0, 0, sizeof c0);
    c0.n_rows = n_rows;
    c0.row_len = (int64_t)d->H_q * d->d_v;
    c0.n_chunks = n_chunks;
    c0.Tq = d->Tq;
    const int step = sim_apart(layers, n_layers) ? n_layers : 1;
    LeadJob jobs[ic::kMaxBatchLayers];         // of one shape, collected until a launch is full
    auto ends = [&](int i, int next) { return next >= n_layers || memcmp(&layers[i].at, &layers[next].at, sizeof layers[i].at) != 0; };
    for (int first = 0; first < n_layers; first += step) {
        const int end = first + step;
        int n = 0;
        for (int i = first; i < end; ++i) {
            jobs[n++] = LeadJob{layers[i], idx[i], counts(i), counts(i)};
            if (n < ic::kMaxBatchLayers && i + 1 < end && !ends(i, i + 1)) continue;
            ic_status r = run_lead_dense(jobs, n, nullptr, st);
            if (r == IC_OK) r = run_lead_rest(jobs, n, nullptr, ws, ws_bytes, st);
            if (r != IC_OK) return r;
            ic::CosineArgs c = c0;
            c.self_out = 1;
            int m = 0;
            for (int l = i + 1 - n; l <= i; ++l)
                if (self_of(l)) {
                    c.A[m] = c.B[m] = (const unsigned short *)layers[l].O;
                    c.lead[m] = c.lead2[m] = counts(l);
                    c.self[m++] = self_of(l);
                }
            if (m) {
                const hipError_t e = ic::launch_cosines(c, m, st);
                if (e != hipSuccess) return fail(IC_ERR_HIP, "cosine launch failed: %s", hipGetErrorString(e));
            }
            n = 0;
        }
        ic::CosineArgs c = c0;
        for (int i = first; i < end; ++i)
            for (int j = 0; j < i; ++j) {      // layer i as a Shared one reading j
                c.A[n] = (const unsigned short *)layers[i].O;
                c.B[n] = (const unsigned short *)(o_reuse + n * sim_o_bytes(d));
                c.acc[n] = S + (size_t)i * n_layers + j;
                c.lead[n] = counts(j);
                c.lead2[n] = counts(i);
                c.self[n] = self_of(i);
                jobs[n] = LeadJob{layers[i], idx[j], counts(j), counts(i)};
                jobs[n].L.O = o_reuse + n * sim_o_bytes(d);
                if (++n < n_out && (j + 1 < i || (i + 1 < end && !ends(i, i + 1)))) continue;
                const ic_status r = run_lead_rest(jobs, n, nullptr, ws, ws_bytes, st);
                if (r != IC_OK) return r;
                const hipError_t e = ic::launch_cosines(c, n, st);
                if (e != hipSuccess) return fail(IC_ERR_HIP, "cosine launch failed: %s", hipGetErrorString(e));
                n = 0;
            }
    }
    return IC_OK;
}

} // namespace

size_t ic_similarity_matrix_workspace(const ic_layer *layers, int32_t n_layers)
{
    if (!layers || n_layers <= 0 || n_layers > IC_MAX_OVERLAP_LAYERS) return 0;
    size_t at = 0;
    for (int l = 0; l < n_layers; ++l) {
        const size_t a = attn_query_bytes(&layers[l].at);
        if (a > at) at = a;
    }
    const ic_attn_desc *a0 = &layers[0].at;
    const size_t lb = sim_lead_bytes(layers, n_layers);
    if (!lb) return sim_o_bytes(a0) + align_up(at);
    at = std::max(at, lead_tail_bytes(a0));
    return sim_outputs(a0, n_layers) * sim_o_bytes(a0) + align_up(at) + lb + sim_self_bytes(a0, n_layers);
}

ic_status ic_similarity_matrix(const ic_layer *layers, int32_t n_layers, const int32_t *const *idx_layers, double *S,
                               void *workspace, size_t workspace_bytes, void *stream)
{
    ic_status s = check_sim_layers(layers, n_layers);
    if (s != IC_OK) return s;
    if (!idx_layers || !S) return fail(IC_ERR_NULL, "idx_layers and S must not be NULL");
    for (int l = 0; l < n_layers; ++l)
        if (!idx_layers[l]) return fail(IC_ERR_NULL, "idx_layers[%d] is NULL", l);
    // the counts of leading rows, wide partials and several outputs at a time are for more speed or precision: a workspace
    // without room for them will do
    const ic_attn_desc *a0 = &layers[0].at;
    const size_t ob = sim_o_bytes(a0);
    size_t lb = sim_lead_bytes(layers, n_layers), at = 0, best = lead_tail_bytes(a0);
    for (int l = 0; l < n_layers; ++l) {
        at = std::max(at, attn_ws_bytes(&layers[l].at));
        best = std::max(best, attn_query_bytes(&layers[l].at));
    }
    const size_t min_ws = ob + align_up(at);
    s = check_ws(workspace, workspace_bytes, min_ws);
    if (s != IC_OK) return s;
    if (workspace_bytes < min_ws + lb) lb = 0;
    for (int l = 0; l < n_layers; ++l)
        if (!dense_output(layers[l].O)) lb = 0;
    hipStream_t st = (hipStream_t)stream;
    char *ws = (char *)workspace;
    hipError_t e = ic::launch_sim_init(S, n_layers, st);
    if (e != hipSuccess) return fail(IC_ERR_HIP, "similarity init failed: %s", hipGetErrorString(e));
    const int64_t n_rows = (int64_t)a0->B * a0->Tq;
    if (lb) {
        const size_t one = ob + align_up(best) + lb, sb = workspace_bytes >= one + sim_self_bytes(a0, n_layers) ? sim_self_bytes(a0, n_layers) : 0;
        const size_t more = workspace_bytes > one + sb ? (workspace_bytes - one - sb) / ob : 0;
        const int n_out = (int)std::min<size_t>(1 + more, sim_outputs(a0, n_layers));
        int32_t *const lead = (int32_t *)(ws + n_out * ob);
        double *const self = sb ? (double *)((char *)lead + lb) : nullptr;
        lb += sb;
        s = count_lead(a0, idx_layers, n_layers, lead, st);
        if (s != IC_OK) return s;
        s = run_similarity(layers, n_layers, idx_layers, S, lead, self, ws, n_out, (char *)lead + lb, workspace_bytes - n_out * ob - lb, st);
        if (s != IC_OK) return s;
    } else {
        for (int i = 0; i < n_layers; ++i) {
            const ic_layer *L = &layers[i];
            s = run_attn(&L->at, L->Q, L->KV, idx_layers[i], L->O, nullptr, ws + ob, workspace_bytes - ob, st);      // own indices
            if (s != IC_OK) return s;
            for (int j = 0; j < i; ++j) {      // as a Shared layer reading j
                s = run_attn(&L->at, L->Q, L->KV, idx_layers[j], ws, nullptr, ws + ob, workspace_bytes - ob, st);
                if (s != IC_OK) return s;
                ic::CosineArgs c;
                memset(&c, 0, sizeof c);
                c.A[0] = (const unsigned short *)L->O;
                c.B[0] = (const unsigned short *)ws;
                c.acc[0] = S + (size_t)i * n_layers + j;
                c.n_rows = n_rows;
                c.row_len = (int64_t)a0->H_q * a0->d_v;
                e = ic::launch_cosines(c, 1, st);
                if (e != hipSuccess) return fail(IC_ERR_HIP, "cosine launch failed: %s", hipGetErrorString(e));
            }
        }
    }
    e = ic::launch_sim_finish(S, n_layers, n_rows, st);
    if (e != hipSuccess) return fail(IC_ERR_HIP, "similarity finish failed: %s", hipGetErrorString(e));
    return IC_OK;
}

ic_status ic_pattern_search_dp(const double *S, int32_t n_layers, int32_t n_full, uint8_t *full_mask, double *total)
{
    if (!S || !full_mask) return fail(IC_ERR_NULL, "S and full_mask must not be NULL");
    if (n_layers <= 0 || n_full <= 0 || n_full > n_layers)
        return fail(IC_ERR_SHAPE, "need 1 <= n_full <= n_layers (n_full=%d n_layers=%d)", n_full, n_layers);
    const int N = n_layers, M = n_full;
    // run[j][i] = sum of S[m][j] over j < m < i: what the Shared layers between Full layers j and i collect
    std::vector<double> run((size_t)N * (N + 1), 0.0);
    for (int j = 0; j < N; ++j)
        for (int i = j + 1; i <= N; ++i)
            run[(size_t)j * (N + 1) + i] = (i == j + 1) ? 0.0 : run[(size_t)j * (N + 1) + i - 1] + S[(size_t)(i - 1) * N + j];
    const double NEG = -1e300;
    std::vector<double> dp((size_t)N * (M + 1), NEG);       // dp[i][c]: layer i Full, c Full layers in 0..i
    std::vector<int> from((size_t)N * (M + 1), -1);
    dp[(size_t)0 * (M + 1) + 1] = 0.0;                         // the first layer is always Full
    for (int i = 1; i < N; ++i)
        for (int c = 2; c <= M && c <= i + 1; ++c)
            for (int j = c - 2; j < i; ++j) {
                const double prev = dp[(size_t)j * (M + 1) + c - 1];
                if (prev <= NEG) continue;
                const double v = prev + run[(size_t)j * (N + 1) + i];
                if (v > dp[(size_t)i * (M + 1) + c]) {
                    dp[(size_t)i * (M + 1) + c] = v;
                    from[(size_t)i * (M + 1) + c] = j;
                }
            }
    double best = NEG;
    int last = -1;
    for (int i = M - 1; i < N; ++i) {                          // the last Full layer; everything after it reads it
        const double prev = dp[(size_t)i * (M + 1) + M];
        if (prev <= NEG) continue;
        const double v = prev + run[(size_t)i * (N + 1) + N];
        if (v > best) {
            best = v;
            last = i;
        }
    }
    if (last < 0) return fail(IC_ERR_SHAPE, "no pattern with %d Full layers", M);
    for (int l = 0; l < N; ++l) full_mask[l] = 0;
    for (int i = last, c = M; i >= 0 && c >= 1; --c) {
        full_mask[i] = 1;
        i = from[(size_t)i * (M + 1) + c];
    }
    if (total) *total = best;
    return IC_OK;
}

// ---- greedy layer selection (paper Alg. 1) over a surrogate loss ---------------------------------

extern "C++" {
namespace {

// Alg. 1 with the blocked variant of Sec. 3.2: `eval` fills losses[i] with the loss of the current
// pattern with layer cands[i] flipped to Shared as well.  Ties go to the lowest layer.
template <typename Eval>
ic_status greedy_core(int N, int K, int P, uint8_t *mask, int32_t *order, double *curve, Eval eval)
{
    if (N <= 0 || K < 0 || K > N - 1 || P < 1 || P > N)
        return fail(IC_ERR_SHAPE, "need 0 <= n_shared <= n_layers-1 and 1 <= n_blocks <= n_layers (n_layers=%d n_shared=%d n_blocks=%d)", N, K, P);
    const int size = (N + P - 1) / P;
    int n_cand = 0;
    for (int b0 = 0; b0 < N; b0 += size) n_cand += (b0 + size < N ? size : N - b0) - 1;   // a block's first layer stays Full
    if (K > n_cand) return fail(IC_ERR_SHAPE, "n_shared=%d but only %d layers may become Shared with %d blocks", K, n_cand, P);
    for (int l = 0; l < N; ++l) mask[l] = 1;
    std::vector<int32_t> cands;
    std::vector<double> losses;
    int done = 0;
    while (done < K) {
        for (int b0 = 0; b0 < N && done < K; b0 += size) {
            const int b1 = b0 + size < N ? b0 + size : N;
            cands.clear();
            for (int l = b0 + 1; l < b1; ++l)
                if (mask[l]) cands.push_back(l);
            if (cands.empty()) continue;
            losses.assign(cands.size(), 0.0);
            ic_status s = eval(mask, cands, losses);
            if (s != IC_OK) return s;
            size_t arg = 0;
            for (size_t i = 1; i < cands.size(); ++i)
                if (losses[i] < losses[arg]) arg = i;
            mask[cands[arg]] = 0;
            if (order) order[done] = cands[arg];
            if (curve) curve[done] = losses[arg];
            ++done;
        }
    }
    return IC_OK;
}

// The layers' similarities and an accumulator; the stack's workspace follows them.
size_t loss_head_bytes(int32_t n_layers) { return align_up((size_t)n_layers * sizeof(double)) + kAlign; }

size_t pattern_loss_ws(const ic_layer *layers, int32_t n_layers)
{
    return loss_head_bytes(n_layers) + align_up(ic_forward_stack_workspace(layers, n_layers));
}

// What has to be there: a layer at a time.  Room for runs of layers and for rows in parts only makes the stack faster.
size_t pattern_loss_min_ws(const ic_layer *layers, int32_t n_layers)
{
    size_t fw = 0;
    for (int l = 0; l < n_layers; ++l) {
        const size_t a = attn_ws_bytes(&layers[l].at);
        const size_t b = layers[l].q && check_indexer(&layers[l].ix) == IC_OK ? indexer_strip_ws(&layers[l].ix) : 0;
        if (a > fw) fw = a;
        if (b > fw) fw = b;
    }
    return loss_head_bytes(n_layers) + align_up(fw);
}

ic_status run_pattern_loss(const ic_layer *layers, int32_t n_layers, const uint8_t *full_mask, const void *const *O_ref,
                           int32_t *idx_cache, double *loss, void *workspace, size_t workspace_bytes, hipStream_t st)
{
    char *ws = (char *)workspace;
    const size_t head = loss_head_bytes(n_layers), most = pattern_loss_ws(layers, n_layers);
    double *sims = (double *)ws;
    double *acc = (double *)(ws + head - kAlign);
    const size_t fw = (workspace_bytes < most ? workspace_bytes : most) - head;
    ic_status s = ic_forward_stack(layers, n_layers, full_mask, idx_cache, ws + head, fw, (void *)st);
    if (s != IC_OK) return s;
    const ic_attn_desc *a0 = &layers[0].at;
    const int64_t n_rows = (int64_t)a0->B * a0->Tq, row_len = (int64_t)a0->H_q * a0->d_v;
    for (int l = 0; l < n_layers; ++l) {
        hipError_t e = ic::launch_cosine(layers[l].O, O_ref[l], n_rows, row_len, sims + l, nullptr, acc, st);
        if (e != hipSuccess) return fail(IC_ERR_HIP, "cosine launch failed: %s", hipGetErrorString(e));
    }
    hipError_t e = ic::launch_loss_finish(sims, n_layers, loss, st);
    if (e != hipSuccess) return fail(IC_ERR_HIP, "loss reduction launch failed: %s", hipGetErrorString(e));
    return IC_OK;
}

ic_status check_loss_args(const ic_layer *layers, int32_t n_layers, const void *const *O_ref, const int32_t *idx_cache)
{
    ic_status s = check_sim_layers(layers, n_layers);
    if (s != IC_OK) return s;
    if (!O_ref || !idx_cache) return fail(IC_ERR_NULL, "O_ref and idx_cache must not be NULL");
    for (int l = 0; l < n_layers; ++l) {
        if (!O_ref[l]) return fail(IC_ERR_NULL, "O_ref[%d] is NULL", l);
        if (O_ref[l] == layers[l].O) return fail(IC_ERR_SHAPE, "O_ref[%d] is the layer's own output buffer", l);
    }
    return IC_OK;
}

} // namespace
} // extern "C++"

ic_status ic_pattern_search_greedy(const double *S, int32_t n_layers, int32_t n_shared, int32_t n_blocks,
                                   uint8_t *full_mask, int32_t *order, double *loss_curve)
{
    if (!S || !full_mask) return fail(IC_ERR_NULL, "S and full_mask must not be NULL");
    const int N = n_layers;
    auto loss_of = [&](const uint8_t *m) {
        double t = 0.0;
        int src = 0;
        for (int l = 0; l < N; ++l) {
            if (m[l]) src = l;
            else t += 1.0 - S[(size_t)l * N + src];
        }
        return t / N;
    };
    return greedy_core(N, n_shared, n_blocks, full_mask, order, loss_curve,
                       [&](uint8_t *m, const std::vector<int32_t> &cands, std::vector<double> &out) {
                           for (size_t i = 0; i < cands.size(); ++i) {
                               m[cands[i]] = 0;
                               out[i] = loss_of(m);
                               m[cands[i]] = 1;
                           }
                           return IC_OK;
                       });
}

size_t ic_pattern_loss_workspace(const ic_layer *layers, int32_t n_layers)
{
    if (!layers || n_layers <= 0 || n_layers > IC_MAX_OVERLAP_LAYERS) return 0;
    return pattern_loss_ws(layers, n_layers);
}

ic_status ic_pattern_loss(const ic_layer *layers, int32_t n_layers, const uint8_t *full_mask, const void *const *O_ref,
                          int32_t *idx_cache, double *loss, void *workspace, size_t workspace_bytes, void *stream)
{
    ic_status s = check_loss_args(layers, n_layers, O_ref, idx_cache);
    if (s != IC_OK) return s;
    if (!full_mask || !loss) return fail(IC_ERR_NULL, "full_mask and loss must not be NULL");
    s = check_ws(workspace, workspace_bytes, pattern_loss_min_ws(layers, n_layers));
    if (s != IC_OK) return s;
    return run_pattern_loss(layers, n_layers, full_mask, O_ref, idx_cache, loss, workspace, workspace_bytes, (hipStream_t)stream);
}

size_t ic_greedy_search_forward_workspace(const ic_layer *layers, int32_t n_layers)
{
    if (!layers || n_layers <= 0 || n_layers > IC_MAX_OVERLAP_LAYERS) return 0;
    return pattern_loss_ws(layers, n_layers) + align_up((size_t)n_layers * sizeof(double));
}

ic_status ic_greedy_search_forward(const ic_layer *layers, int32_t n_layers, int32_t n_shared, int32_t n_blocks,
                                   const void *const *O_ref, int32_t *idx_cache, uint8_t *full_mask, int32_t *order,
                                   double *loss_curve, void *workspace, size_t workspace_bytes, void *stream)
{
    ic_status s = check_loss_args(layers, n_layers, O_ref, idx_cache);
    if (s != IC_OK) return s;
    if (!full_mask) return fail(IC_ERR_NULL, "full_mask must not be NULL");
    const size_t cands_bytes = align_up((size_t)n_layers * sizeof(double));
    s = check_ws(workspace, workspace_bytes, cands_bytes + pattern_loss_min_ws(layers, n_layers));
    if (s != IC_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    double *dev_losses = (double *)workspace;
    void *const loss_ws = (char *)workspace + cands_bytes;
    const size_t loss_bytes = workspace_bytes - cands_bytes;
    return greedy_core(n_layers, n_shared, n_blocks, full_mask, order, loss_curve,
                       [&](uint8_t *m, const std::vector<int32_t> &cands, std::vector<double> &out) {
                           // one forward pass of the whole stack per candidate, all on the stream;
                           // then the host needs the losses to choose: one synchronisation per search step
                           for (size_t i = 0; i < cands.size(); ++i) {
                               m[cands[i]] = 0;
                               ic_status r = run_pattern_loss(layers, n_layers, m, O_ref, idx_cache, dev_losses + i, loss_ws, loss_bytes, st);
                               m[cands[i]] = 1;
                               if (r != IC_OK) return r;
                           }
                           hipError_t e = hipStreamSynchronize(st);
                           if (e == hipSuccess) e = hipMemcpy(out.data(), dev_losses, cands.size() * sizeof(double), hipMemcpyDeviceToHost);
                           if (e != hipSuccess) return fail(IC_ERR_HIP, "reading the candidate losses failed: %s", hipGetErrorString(e));
                           return IC_OK;
                       });
}

// ---- distillation loss forward (paper Sec. 3.3) ---------------------------------------------------

ic_status ic_attn_probs(const ic_attn_desc *d, const void *Q, const void *KV, const int32_t *idx, const float *lse,
                        float *probs, void *stream)
{
    ic_status s = check_attn(d);
    if (s != IC_OK) return s;
    if (!Q || !KV || !idx || !lse || !probs) return fail(IC_ERR_NULL, "Q, KV, idx, lse and probs must not be NULL");
    ic::ProbsArgs a;
    memset(&a, 0, sizeof a);
    a.Q = Q;
    a.KV = KV;
    a.idx = idx;
    a.lse = lse;
    a.probs = probs;
    a.B = d->B;
    a.Tq = d->Tq;
    a.Lk = d->Lk;
    a.H_q = d->H_q;
    a.row_elems = d->row_elems;
    a.k_sel = d->k_sel;
    a.scale_log2e = d->sm_scale * 1.4426950408889634f;
    hipError_t e = ic::launch_attn_probs(a, d->d_qk, (hipStream_t)stream);
    if (e != hipSuccess) return fail(IC_ERR_HIP, "attention-probability launch failed: %s", hipGetErrorString(e));
    return IC_OK;
}

size_t ic_distill_loss_workspace(int64_t nq)
{
    if (nq <= 0) return kAlign;
    return 2 * align_up((size_t)nq * sizeof(double));
}

ic_status ic_distill_loss(const float *const *probs, int32_t n_targets, const float *sel_scores, int64_t nq, int32_t k_sel,
                          double *loss_multi, double *loss_avg, float *grad, void *workspace, size_t workspace_bytes,
                          void *stream)
{
    if (!probs || !sel_scores) return fail(IC_ERR_NULL, "probs and sel_scores must not be NULL");
    if (n_targets < 1 || n_targets > IC_MAX_DISTILL_TARGETS)
        return fail(IC_ERR_SHAPE, "n_targets=%d must be in [1, %d]", n_targets, IC_MAX_DISTILL_TARGETS);
    if (nq < 0 || nq > INT32_MAX || k_sel <= 0) return fail(IC_ERR_SHAPE, "need 0 <= nq <= 2^31-1 and k_sel > 0");
    for (int j = 0; j < n_targets; ++j)
        if (!probs[j]) return fail(IC_ERR_NULL, "probs[%d] is NULL", j);
    if (!loss_multi && !loss_avg && !grad) return fail(IC_ERR_NULL, "at least one output must be given");
    ic_status s = check_ws(workspace, workspace_bytes, ic_distill_loss_workspace(nq));
    if (s != IC_OK) return s;
    ic::DistillArgs a;
    memset(&a, 0, sizeof a);
    for (int j = 0; j < n_targets; ++j) a.probs[j] = probs[j];
    a.n_targets = n_targets;
    a.k_sel = k_sel;
    a.scores = sel_scores;
    a.row_multi = (double *)workspace;
    a.row_avg = (double *)((char *)workspace + align_up((size_t)(nq > 0 ? nq : 1) * sizeof(double)));
    a.grad = grad;
    hipError_t e = ic::launch_distill(a, nq, loss_multi, loss_avg, (hipStream_t)stream);
    if (e != hipSuccess) return fail(IC_ERR_HIP, "distillation loss launch failed: %s", hipGetErrorString(e));
    return IC_OK;
}

size_t ic_topk_overlap_workspace(int32_t n_layers)
{
    if (n_layers <= 0 || n_layers > IC_MAX_OVERLAP_LAYERS) return 0;
    return align_up(ic::overlap_ws_bytes(n_layers));
}

ic_status ic_topk_overlap(const int32_t *const *idx_layers, int32_t n_layers, int64_t nq, int32_t k_sel, int32_t Lk,
                          double *overlap, uint64_t *inter, uint64_t *sizes, void *workspace, size_t workspace_bytes,
                          void *stream)
{
    if (!idx_layers) return fail(IC_ERR_NULL, "idx_layers must not be NULL");
    if (n_layers <= 0 || nq < 0 || k_sel <= 0 || Lk <= 0) return fail(IC_ERR_SHAPE, "overlap sizes must be positive");
    if (n_layers > IC_MAX_OVERLAP_LAYERS)
        return fail(IC_ERR_UNSUPPORTED, "n_layers=%d exceeds IC_MAX_OVERLAP_LAYERS=%d", n_layers, IC_MAX_OVERLAP_LAYERS);
    if (Lk > IC_MAX_OVERLAP_LK) return fail(IC_ERR_UNSUPPORTED, "Lk=%d exceeds IC_MAX_OVERLAP_LK=%d", Lk, IC_MAX_OVERLAP_LK);
    if ((nq + 15) / 16 * n_layers > (int64_t)INT32_MAX) return fail(IC_ERR_SHAPE, "nq * n_layers too large");
    for (int l = 0; l < n_layers; ++l)
        if (!idx_layers[l]) return fail(IC_ERR_NULL, "idx_layers[%d] is NULL", l);
    if (!overlap && !inter && !sizes) return fail(IC_ERR_NULL, "at least one output must be given");
    ic_status s = check_ws(workspace, workspace_bytes, ic_topk_overlap_workspace(n_layers));
    if (s != IC_OK) return s;
    hipError_t e = ic::launch_overlap(idx_layers, n_layers, nq, k_sel, Lk, overlap, (unsigned long long *)inter,
                                      (unsigned long long *)sizes, workspace, (hipStream_t)stream);
    if (e != hipSuccess) return fail(IC_ERR_HIP, "overlap launch failed: %s", hipGetErrorString(e));
    return IC_OK;
}

ic_status ic_debug_indexer_scores(const ic_indexer_desc *d, const void *q, const void *k, const float *w,
                                  int32_t row0, int32_t n_rows, float *out, void *stream)
{
    ic_status s = check_indexer(d);
    if (s != IC_OK) return s;
    if (!q || !k || !w || !out) return fail(IC_ERR_NULL, "q, k, w and out must not be NULL");
    if (row0 < 0 || n_rows <= 0 || (int64_t)row0 + n_rows > d->Tq)
        return fail(IC_ERR_SHAPE, "rows [%d, %d) outside [0, Tq=%d)", row0, row0 + n_rows, d->Tq);
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = ic::launch_fill(out, (int64_t)d->B * n_rows * d->Lk, -INFINITY, st);
    if (e != hipSuccess) return fail(IC_ERR_HIP, "fill launch failed: %s", hipGetErrorString(e));
    ic::ScoreArgs sa;
    memset(&sa, 0, sizeof sa);
    sa.q = q;
    sa.k = k;
    sa.w = w;
    sa.q_scale = d->q_scale;
    sa.k_scale = d->k_scale;
    sa.strip = out;
    sa.ld = d->Lk;
    sa.q_pos0 = d->q_pos0;
    sa.Tq = d->Tq;
    sa.Lk = d->Lk;
    sa.H_I = d->H_I;
    sa.b0 = 0;
    sa.i0 = row0;
    sa.Ri = n_rows;
    ProfScope ps(0, st);
    e = ic::launch_score(sa, d->dtype, d->d_I, d->B, st);
    if (e != hipSuccess) return fail(IC_ERR_HIP, "indexer score launch failed: %s", hipGetErrorString(e));
    return IC_OK;
}

uint64_t ic_debug_indexer_launch_count(void) { return g_indexer_launches.load(); }

ic_status ic_calibrate(int32_t kind, const void *src, void *dst, const int32_t *idx, int64_t n, int64_t table_rows,
                       int32_t row_bytes, int32_t wgs, void *stream)
{
    if (kind < IC_CALIB_READ || kind > IC_CALIB_LDS_TR8_ROWS1) return fail(IC_ERR_SHAPE, "unknown calibration kind %d", kind);
    if (!dst) return fail(IC_ERR_NULL, "dst must not be NULL");
    if (wgs < 1 || wgs > (1 << 20)) return fail(IC_ERR_SHAPE, "wgs=%d outside [1, 2^20]", wgs);
    if (n < 0) return fail(IC_ERR_SHAPE, "n must not be negative");
    if (kind == IC_CALIB_READ || kind == IC_CALIB_COPY) {
        if (!src) return fail(IC_ERR_NULL, "src must not be NULL");
        if (n % 16 != 0) return fail(IC_ERR_SHAPE, "n=%lld bytes is not a multiple of 16", (long long)n);
    } else if (kind == IC_CALIB_GATHER) {
        if (!src || !idx) return fail(IC_ERR_NULL, "src and idx must not be NULL");
        if (table_rows < 1) return fail(IC_ERR_SHAPE, "table_rows must be positive");
        if (row_bytes != 1152 && row_bytes != 256) return fail(IC_ERR_UNSUPPORTED, "row_bytes=%d (1152 or 256)", row_bytes);
    } else if (kind >= IC_CALIB_LDS_READ16_PADDED) {
        if (n > INT32_MAX) return fail(IC_ERR_SHAPE, "too many rounds");
    } else if (kind >= IC_CALIB_TILE_GATHER) {
        if (!src || !idx) return fail(IC_ERR_NULL, "src and idx must not be NULL");
        if (table_rows < 1) return fail(IC_ERR_SHAPE, "table_rows must be positive");
        if (row_bytes != 1152) return fail(IC_ERR_UNSUPPORTED, "row_bytes=%d (1152)", row_bytes);
        if (n % 64 != 0) return fail(IC_ERR_SHAPE, "n=%lld rows is not a multiple of 64", (long long)n);
    } else if (n > INT32_MAX) {
        return fail(IC_ERR_SHAPE, "too many rounds");
    }
    hipError_t e = ic::launch_calib(kind, src, dst, idx, n, table_rows, row_bytes, wgs, (hipStream_t)stream);
    if (e != hipSuccess) return fail(IC_ERR_HIP, "calibration launch failed: %s", hipGetErrorString(e));
    return IC_OK;
}

void ic_prof_enable(int32_t on)
{
    std::lock_guard<std::mutex> lk(g_prof_mu);
    g_prof_on = on != 0;
}

ic_status ic_prof_collect(void)
{
    std::lock_guard<std::mutex> lk(g_prof_mu);
    ic_status rc = IC_OK;
    for (ProfRec &r : g_prof_recs) {
        float ms = 0.f;
        hipError_t e = hipEventSynchronize(r.e1);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, r.e0, r.e1);
        if (e == hipSuccess) {
            g_prof_n[r.which] += 1;
            g_prof_ms[r.which] += ms;
        } else {
            rc = fail(IC_ERR_HIP, "event timing failed: %s", hipGetErrorString(e));
        }
        (void)hipEventDestroy(r.e0);
        (void)hipEventDestroy(r.e1);
    }
    g_prof_recs.clear();
    return rc;
}

ic_status ic_prof_get(int32_t which, int64_t *launches, double *total_ms)
{
    if (which < 0 || which >= kProfClasses) return fail(IC_ERR_SHAPE, "kernel class %d outside [0,%d)", which, kProfClasses);
    if (!launches || !total_ms) return fail(IC_ERR_NULL, "output pointers must not be NULL");
    std::lock_guard<std::mutex> lk(g_prof_mu);
    *launches = g_prof_n[which];
    *total_ms = g_prof_ms[which];
    return IC_OK;
}

void ic_prof_reset(void)
{
    std::lock_guard<std::mutex> lk(g_prof_mu);
    for (int i = 0; i < kProfClasses; ++i) {
        g_prof_n[i] = 0;
        g_prof_ms[i] = 0;
    }
}

} // extern "C"
