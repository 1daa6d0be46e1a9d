// Shared device/host declarations of the gfx950 IndexCache library (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "indexcache.h"

namespace ic {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;   // one 16-byte chunk
typedef __attribute__((ext_vector_type(4))) int i32x4;

constexpr int kWave = 64;

// ---- kernel argument blocks ---------------------------------------------------------

// Ragged and paged caches (decode with a full KV cache, paper Sec. 4.3 setting): per-sequence
// lengths and a page table from logical to physical pages.  All-zero = the dense layout.
struct PagedView {
    const int32_t *seq_lens;    // [B] visible length of each sequence (nullptr: every sequence has Lk)
    const int32_t *page_table;  // [B, max_pages] physical page of a logical page (nullptr: not paged)
    int32_t page_shift;         // log2(positions per page), pages hold a power of two >= 64 positions
    int32_t max_pages;
};

// physical row of logical position s of sequence b (paged layout only)
__device__ __forceinline__ int64_t paged_row(const PagedView &pv, int b, int s)
{
    const int32_t page = pv.page_table[(int64_t)b * pv.max_pages + (s >> pv.page_shift)];
    return ((int64_t)page << pv.page_shift) + (s & ((1 << pv.page_shift) - 1));
}

// Small read-only operands (head weights, lengths, page-table entries) are read through the constant address space: with a
// uniform address that is a scalar load, which does not enter the vector-memory queue that waits by position count on.
// (An ordinary load inside such a loop would make the compiler wait for "all its loads", i.e. drain the queue.)
template <typename T> __device__ __forceinline__ T load_uniform(const T *p)
{
    return *(const __attribute__((address_space(4))) T *)(uintptr_t)p;
}

// Inclusive prefix sum over the 64 lanes of a wave on the data-parallel-primitive path of the
// vector ALU (no LDS traffic): shifts by 1, 2, 4, 8 lanes inside each row of 16 lanes, then the
// last lane of rows 0 and 2 is added to rows 1 and 3, then lane 31 to rows 2 and 3.  Lanes
// without a source add zero.  Packed fields are summed independently as long as none overflows.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1, 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2, 3
    return x;
}

// Indexer scoring of query rows [i0, i0+Ri) of sequences [b0, b0+Bc) against their keys.
// Scores land in a strip: row (b-b0)*Ri + (i-i0), element s, row stride ld floats.
struct ScoreArgs {
    const void *q;        // [B,Tq,H_I,d_I]
    const void *k;        // [B,Lk,d_I]
    const float *w;       // [B,Tq,H_I]
    const float *q_scale; // fp8 only
    const float *k_scale; // fp8 only
    float *strip;
    int64_t ld;
    int64_t q_pos0;
    int32_t Tq, Lk, H_I;
    int32_t b0, i0, Ri;   // chunk origin and rows per sequence in the strip
    int32_t n_qblocks;    // ceil(Ri / tokens per workgroup)
    int32_t KC;           // keys per workgroup along grid.y (multiple of 64)
    PagedView pv;         // ragged / paged key cache (the Tq query rows are the LAST Tq positions of a sequence)
};

// Per-row top-k over a strip of scores.
struct SelectArgs {
    const float *strip;
    int64_t ld;
    int64_t q_pos0;
    int32_t Tq, Lk, k_sel;
    int32_t b0, i0, Ri;
    int32_t cache_elems;  // row elements the workgroup may cache in LDS (0 = none)
    int32_t *idx;         // [B,Tq,k_sel]
    float *sel;           // [B,Tq,k_sel] or nullptr
    const int32_t *seq_lens;  // ragged: [B] visible lengths (nullptr: q_pos0 rule)
};

// Candidate lists of rows that are selected in parts (workspace).
struct PartArgs {
    uint32_t *heads;      // [rows][head_words]: threshold key, then the lengths of the row's lists
    uint32_t *lists;      // [rows][2][list entries]: keys, positions; the parts' lists in equal shares
    int32_t n_parts, head_words;
    int32_t slots;        // entries of a list
    uint32_t inv_parts;   // 2^32 / n_parts, rounded up (two parts or more)
};

// One launch covers n_layers layers of one shape that read the same index tensor (a Full layer and the Shared layers
// behind it); its queries are numbered layer by layer, layer * B * Tq + b * Tq + t.
constexpr int kMaxBatchLayers = 8;
struct AttnArgs {
    const void *Q;        // [B,Tq,H_q,d_qk] bf16       (of the first layer; all of them: Qs, KVs, Os below)
    const void *KV;       // [B,Lk,row_elems] bf16
    const int32_t *idx;   // [B,Tq,k_sel]
    void *O;              // [B,Tq,H_q,d_v] bf16
    float *lse;           // [B,Tq,H_q] or nullptr (one layer only)
    void *part_o;         // split partials: [n_layers*B*Tq, n_splits, H_q, d_v], each normalised by its own row sum
    float *part_ml;       // [n_layers*B*Tq, n_splits, H_q, 2] fp32 (running max in log2 units, sum)
    int32_t B, Tq, Lk, H_q, v_off, row_elems, k_sel;
    int32_t n_splits, split_len; // key slots per split (multiple of 64)
    float scale_log2e;    // sm_scale * log2(e)
    PagedView pv;         // ragged / paged KV cache (KV is then the page pool [n_pages << page_shift, row_elems])
    // >= 0: idx comes from the causal top-k of this library with query row t at position causal_pos0 + t, so row t
    // holds min(k_sel, causal_pos0 + t + 1) entries followed by -1 only, and the tiles behind them need no work;
    // < 0: nothing is known about idx
    int64_t causal_pos0;
    int32_t n_layers;
    int32_t row_gap;      // rows of Q, idx, O and lse between two sequences' Tq rows (0: one follows the other)
    const void *Qs[kMaxBatchLayers];
    const void *KVs[kMaxBatchLayers];
    void *Os[kMaxBatchLayers];
    int32_t part_wide;    // 1: the partials are fp32, 0: bf16
};

// Which leading rows of every sequence of an index tensor are whole prefixes, row t = 0 .. pos0 + t and then nothing: per
// chunk of kLeadChunk rows the number of such rows before the first other one.
constexpr int kLeadChunk = 16;
struct LeadArgs {
    const int32_t *idx[IC_MAX_OVERLAP_LAYERS];   // tensors [B,Tq,k_sel]
    int32_t *lead;        // [tensors][B][n_chunks]
    int32_t B, Tq, k_sel, pos0;
    int32_t n_rows, n_chunks;                    // rows looked at per sequence and ceil(n_rows / kLeadChunk)
};

// number of leading rows from one sequence's chunk counts, by a whole wave
__device__ __forceinline__ int lead_rows(const int32_t *lead, int n_chunks)
{
    const int lane = threadIdx.x & 63;
    for (int c0 = 0; c0 < n_chunks; c0 += 64) {
        const int v = c0 + lane < n_chunks ? lead[c0 + lane] : 0;
        const unsigned long long m = __ballot(v < kLeadChunk);
        if (m != 0ull) {
            const int first = __builtin_ctzll(m);
            return kLeadChunk * (c0 + first) + __builtin_amdgcn_readlane(v, first);
        }
    }
    return kLeadChunk * n_chunks;
}

// The rows of a launch whose selection is a whole prefix of the cache.
struct DenseArgs {
    int32_t n_queries;    // per sequence, from row 0
    int32_t pos0;         // row t sees the keys 0 .. pos0 + t, all of them below Lk
    const int32_t *lead;  // [layers][B][n_chunks] or nullptr: fewer rows where these counts say so
    int32_t n_chunks;
};

// The rows that are left: of every sequence of each of n_jobs layers (AttnArgs' Qs, KVs, Os; index tensors of their own), from
// the first row that is not a leading one in both of two tensors up to n_rows.  n_jobs * B is at most kRestSeqs.
constexpr int kRestSeqs = 512;
struct RestArgs {
    const int32_t *idx[kMaxBatchLayers];
    const int32_t *lead[kMaxBatchLayers], *lead2[kMaxBatchLayers];   // [B][n_chunks] chunk counts
    int32_t n_jobs, n_chunks, n_rows;
};

// Comparisons of n_rows rows each.  Rows that are leading in both index tensors of a pair are the same in A and B: their
// similarity is read from `self`, which an earlier launch has left (self_out: it writes those of A's leading rows, and no sum).
struct CosineArgs {
    const unsigned short *A[kMaxBatchLayers], *B[kMaxBatchLayers];
    double *acc[kMaxBatchLayers];                // the sum of the similarities is added here
    const int32_t *lead[kMaxBatchLayers], *lead2[kMaxBatchLayers];   // [B][n_chunks] or nullptr: no such rows
    double *self[kMaxBatchLayers];               // [n_rows] or nullptr: worked out again
    float *per_row;                              // [n_rows] or nullptr (one comparison only)
    int64_t n_rows, row_len;
    int32_t n_chunks, Tq, self_out;
};

// Head-aggregated attention probabilities over the selected rows (the indexer's training target).
struct ProbsArgs {
    const void *Q;        // [B,Tq,H_q,d_qk] bf16
    const void *KV;       // [B,Lk,row_elems] bf16; K = the first d_qk features of a row
    const int32_t *idx;   // [B,Tq,k_sel]
    const float *lse;     // [B,Tq,H_q] natural-log sum-exp of each head over the same rows
    float *probs;         // [B,Tq,k_sel] out, slot order, 0 on empty slots
    int32_t B, Tq, Lk, H_q, row_elems, k_sel;
    float scale_log2e;
};

// Distillation losses of one Full layer's indexer against the layers it serves.
struct DistillArgs {
    const float *probs[IC_MAX_DISTILL_TARGETS];   // m+1 targets, each [nq, k_sel]
    int32_t n_targets, k_sel;
    const float *scores;  // [nq, k_sel] indexer logits at the selected positions (-inf on empty slots)
    double *row_multi;    // [nq] per-row Eq. 1 terms
    double *row_avg;      // [nq] per-row Eq. 2 terms
    float *grad;          // [nq, k_sel] or nullptr
};

// Sum over the 16 lanes of a row (lanes with equal lane / 16) on the data-parallel-primitive path:
// shifts by 1, 2, 4, 8 lanes inside the row; lanes without a source add zero.  Lane 15 of the row
// holds the total.
__device__ __forceinline__ float row16_sum(float x)
{
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x111, 0xf, 0xf, false));
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x112, 0xf, 0xf, false));
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x114, 0xf, 0xf, false));
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x118, 0xf, 0xf, false));
    return x;
}

// ---- launchers (defined next to their kernels) ----------------------------------------

hipError_t launch_score(const ScoreArgs &a, int dtype, int d_I, int Bc, hipStream_t st);
hipError_t launch_fill(float *p, int64_t n, float v, hipStream_t st);
hipError_t launch_select(const SelectArgs &a, int n_rows, int max_row_len, hipStream_t st);
bool topk_short(const ScoreArgs &a, int dtype, int d_I, int n_rows, int64_t max_vis);
hipError_t launch_topk_short(const ScoreArgs &a, const SelectArgs &se, int d_I, int Bc, hipStream_t st);
int select_parts(int n_rows, int max_row_len);
bool select_parts_fit(int k, int row_len);
int select_parts_slots(int n_rows, int max_row_len);
int select_parts_cache(int ragged);
int select_cand_rank(int k, int row_len, int many);
int select_cand_runs(int many);
int select_cand_list(int many);
size_t select_parts_bytes(int n_rows, int max_row_len);
hipError_t launch_select_parts(const SelectArgs &a, int n_rows, int max_row_len, void *ws, hipStream_t st);
hipError_t launch_attn(const AttnArgs &a, int d_qk, int d_v, hipStream_t st);
hipError_t launch_attn_dense(const AttnArgs &a, const DenseArgs &da, hipStream_t st);
hipError_t launch_attn_rest(const AttnArgs &a, const RestArgs &ra, hipStream_t st);
hipError_t launch_lead(const LeadArgs &a, int n_tensors, hipStream_t st);
hipError_t launch_attn_merge(const AttnArgs &a, int d_v, hipStream_t st);
size_t overlap_ws_bytes(int n_layers);
size_t overlap_lds_bytes(int n_layers, int Lk);
hipError_t launch_overlap(const int32_t *const *idx_layers, int n_layers, int64_t nq, int k_sel, int Lk, double *overlap,
                          unsigned long long *inter_out, unsigned long long *sizes_out, void *ws, hipStream_t st);
hipError_t launch_cosine(const void *A, const void *B, int64_t n_rows, int64_t row_len, double *mean, float *per_row,
                         double *acc, hipStream_t st);
hipError_t launch_cosines(const CosineArgs &a, int n, hipStream_t st);
hipError_t launch_sim_init(double *S, int n, hipStream_t st);
hipError_t launch_sim_finish(double *S, int n, int64_t n_rows, hipStream_t st);
hipError_t launch_loss_finish(const double *sims, int n, double *loss, hipStream_t st);
hipError_t launch_probs_stream(const ProbsArgs &a, hipStream_t st);
hipError_t launch_attn_probs(const ProbsArgs &a, int d_qk, hipStream_t st);
hipError_t launch_distill(const DistillArgs &a, int64_t nq, double *loss_multi, double *loss_avg, hipStream_t st);
hipError_t launch_calib(int kind, const void *src, void *dst, const int32_t *idx, int64_t n, int64_t table_rows, int row_bytes,
                        int wgs, hipStream_t st);
bool score_shape_supported(int dtype, int H_I, int d_I);
bool attn_shape_supported(int d_qk, int d_v);

} // namespace ic
