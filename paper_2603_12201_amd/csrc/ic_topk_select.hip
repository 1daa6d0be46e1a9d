// Per-query top-k over a strip of indexer scores (T_t = Top-k(I_t), paper Sec. 3 Notation).
//
// One workgroup per query row.  Scores become order-preserving 32-bit keys.  An MSB-first
// radix select finds the exact key of the k-th largest score and how many entries equal to it
// belong to the result; one ordered pass then emits every position whose key is larger, plus
// the first (lowest-position) entries that tie with it, in ascending position order.
//
//   pass 1   12-bit digit (sign, exponent, 3 mantissa bits) over the whole row, fused with the
//            single read of the row from HBM; rows of up to `cache_elems` keys stay in LDS
//   pass 2,3 12 + 8 bits; only entries that match the prefix found so far touch the histogram,
//            so these are read-mostly sweeps over the cached row.  The sweeps stop as soon as the
//            boundary bin holds exactly the entries still needed (with distinct scores: after
//            pass 2), because then every entry with key >= prefix is selected
//   emit     a thread owns 4 consecutive positions in every sweep.  When every entry equal to the
//            k-th key is selected (the usual case: known from the last histogram) "selected" is
//            the single test key >= tau: per-thread counts of two sweeps packed in one word, one
//            wave scan per word on the DPP path, one scan over the (sweep, wave) cells, two
//            barriers in all.  When ties are cut at the boundary: per-sweep scans of packed
//            greater / equal counts.
// That is the form for whatever the others leave over.  Forms by row length: scores and top-k in one launch (few rows of up
// to 1024 keys), the bins form (launches whose rows have up to 32768), the candidate form (32769 to 131072 keys), the candidate form with a row spread
// over several workgroups (few rows of more than 65536 keys), and the radix select, with the keys cached in LDS (up to
// 32768) or re-reading the row on every sweep.
#include "ic_common.hpp"

namespace ic {

namespace {

__device__ __forceinline__ uint32_t score_key(float x)
{
    uint32_t u = __float_as_uint(x);
    u = (u == 0x80000000u) ? 0u : u;                   // -0 and +0 are the same score
    const uint32_t flip = (uint32_t)((int32_t)u >> 31) | 0x80000000u;   // all ones for negatives, else the sign bit
    return u ^ flip;                                   // larger float <=> larger key
}

__device__ __forceinline__ float key_score(uint32_t key)
{
    const uint32_t u = (key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key;
    return __uint_as_float(u);
}

constexpr int kBins1 = 4096;   // histogram bins: digits of 12, 12 and 8 key bits

// Workgroup-wide descending scan over `nbins` counters: finds the digit d with
// count(bins > d) < need <= count(bins >= d) and writes {d, need - count(bins > d), count(bin d)} to bc.
// Every thread owns BPT consecutive bins, highest bins first.
struct BlockSync {
    __device__ __forceinline__ void operator()() const { __syncthreads(); }
};
// A wave that works by itself: LDS serves it in order, so the compiler has to keep that order.
struct WaveSync {
    __device__ __forceinline__ void operator()() const
    {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
};

template <int NT, int BPT, typename Sync = BlockSync>
__device__ __forceinline__ void find_digit(const uint32_t *cnt, uint32_t need, uint32_t *wsum, uint32_t *bc,
                                           int tid, int lane, int wave, Sync sync = Sync())
{
    constexpr int NW = NT / 64;
    const int top = NT * BPT - 1 - BPT * tid;          // highest bin of this thread
    uint32_t c[BPT];
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
        c[j] = cnt[top - j];
        mine += c[j];
    }
    uint32_t incl = wave_incl_scan(mine);
    if (lane == 63) wsum[wave] = incl;
    sync();
    uint32_t before = 0;
#pragma unroll
    for (int wv = 0; wv < NW; ++wv)
        if (wv < wave) before += wsum[wv];
    incl += before;
    const uint32_t excl = incl - mine;
    if (excl < need && need <= incl) {                 // exactly one thread
        uint32_t run = excl;
#pragma unroll
        for (int j = 0; j < BPT; ++j) {
            if (run < need && need <= run + c[j]) {
                bc[0] = (uint32_t)(top - j);
                bc[1] = need - run;
                bc[2] = c[j];
            }
            run += c[j];
        }
    }
    sync();
}

// The radix select of one row (workgroup-wide; smem: kBins1 + 2 NW + 4 + a.cache_elems words).
template <int NT>
__device__ __forceinline__ void select_row_generic(const SelectArgs &a, uint32_t *smem)
{
    constexpr int NW = NT / 64;
    uint32_t *hist1 = smem;                    // [kBins1]
    uint32_t *wsum = hist1 + kBins1;           // [2][NW] (scan partials / emit totals, double buffered)
    uint32_t *bc = wsum + 2 * NW;              // [4] broadcast: digit, remaining need
    uint32_t *cache = bc + 4;                  // [cache_elems] keys of the row

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = blockIdx.x;
    const int b = a.b0 + r / a.Ri;
    const int i = a.i0 + r % a.Ri;
    if (i >= a.Tq) return;
    // ragged cache: the sequence holds Lk_b keys and its Tq query rows are its last Tq positions
    const int Lk_b = a.seq_lens ? max(0, min(a.seq_lens[b], a.Lk)) : a.Lk;
    int64_t nv64 = (a.seq_lens ? (int64_t)Lk_b - a.Tq : a.q_pos0) + (int64_t)i + 1;
    nv64 = nv64 < 0 ? 0 : (nv64 > Lk_b ? Lk_b : nv64);
    const int nv = (int)nv64;
    const float *row = a.strip + (int64_t)r * a.ld;
    int32_t *oidx = a.idx + ((int64_t)b * a.Tq + i) * a.k_sel;
    float *osel = a.sel ? a.sel + ((int64_t)b * a.Tq + i) * a.k_sel : nullptr;

    if (nv <= a.k_sel) {                       // every visible key is selected
        for (int m = tid; m < a.k_sel; m += NT) {
            oidx[m] = m < nv ? m : -1;
            if (osel) osel[m] = m < nv ? row[m] : -INFINITY;
        }
        return;
    }

    const bool cached = nv <= a.cache_elems;   // workgroup-uniform
    // four consecutive keys starting at p (p % 4 == 0); entries at or beyond nv are unspecified
    auto get_key4 = [&](int p) -> u32x4 {
        u32x4 k4 = u32x4{0u, 0u, 0u, 0u};
        if (p < nv) {
            if (cached) {
                k4 = *(const u32x4 *)(cache + p);
            } else {
                const f32x4 v = *(const f32x4 *)(row + p);
#pragma unroll
                for (int e = 0; e < 4; ++e) k4[e] = score_key(v[e]);
            }
        }
        return k4;
    };

    // ---- pass 1: 12-bit digit, fused with the read of the row ----
    for (int e = tid; e < kBins1; e += NT) hist1[e] = 0;
    __syncthreads();
    {
        // 16-byte loads, kLoadBatch of them in flight per thread: the strip lives in HBM and one
        // workgroup per CU has to cover the whole memory latency by itself.  Rows start 256-byte
        // aligned and are padded to a multiple of 64 floats, so the last vector may run past nv
        // (never past the row); those lanes are masked.
        constexpr int kLoadBatch = 4;
        for (int base = 0; base < nv; base += NT * 4 * kLoadBatch) {
            f32x4 v[kLoadBatch];
#pragma unroll
            for (int u = 0; u < kLoadBatch; ++u) {
                const int p = base + (u * NT + tid) * 4;
                v[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (p < nv) v[u] = *(const f32x4 *)(row + p);
            }
#pragma unroll
            for (int u = 0; u < kLoadBatch; ++u) {
                const int p = base + (u * NT + tid) * 4;
                if (p < nv) {
                    u32x4 k4;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        k4[e] = score_key(v[u][e]);
                        if (p + e < nv) atomicAdd(&hist1[k4[e] >> 20], 1u);
                    }
                    if (cached) *(u32x4 *)(cache + p) = k4;   // cache is 16-byte aligned, p % 4 == 0
                }
            }
        }
    }
    __syncthreads();
    find_digit<NT, kBins1 / NT>(hist1, (uint32_t)a.k_sel, wsum, bc, tid, lane, wave);
    uint32_t prefix = bc[0] << 20, prefix_mask = 0xFFF00000u;
    uint32_t need = bc[1];
    // Once the boundary bin holds exactly as many entries as are still needed, all of them are
    // selected and the remaining digits do not matter: "selected" is key >= prefix (rest zero).
    // With distinct scores that happens after the second digit, which saves the third sweep.
    bool all_sel = bc[2] == need;              // workgroup-uniform
    uint32_t total_eq = bc[2];
    __syncthreads();

    // ---- passes 2 and 3: bits [19:8] and [7:0] of the entries that match the prefix so far ----
#pragma unroll 1
    for (int pass = 0; pass < 2 && !all_sel; ++pass) {
        const int shift = pass == 0 ? 8 : 0;
        const uint32_t dmask = pass == 0 ? 4095u : 255u;
        for (int e = tid; e < kBins1; e += NT) hist1[e] = 0;
        __syncthreads();
        for (int p0 = 0; p0 < nv; p0 += 4 * NT) {
            const int p = p0 + 4 * tid;
            const u32x4 k4 = get_key4(p);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (p + e < nv && (k4[e] & prefix_mask) == prefix) atomicAdd(&hist1[(k4[e] >> shift) & dmask], 1u);
        }
        __syncthreads();
        find_digit<NT, kBins1 / NT>(hist1, need, wsum, bc, tid, lane, wave);
        prefix |= bc[0] << shift;
        prefix_mask |= dmask << shift;
        need = bc[1];
        total_eq = bc[2];
        all_sel = total_eq == need;
        __syncthreads();
    }
    // tau: key of the k-th largest score, or (all_sel) a lower bound of it that no unselected entry
    // reaches.  need_eq: how many of the total_eq entries equal to tau are selected.
    const uint32_t tau = prefix;
    const uint32_t need_eq = need;

    // ---- ordered emit, common case: the row is cached, has at most kFastChunks sweeps, and every
    // entry equal to tau is selected (the k-th score is unique, or all of its ties fit).  Then
    // "selected" is the single test key >= tau and the slot of an entry is the number of selected
    // entries ahead of it in (chunk, wave, lane, element) order: one packed wave scan per chunk
    // pair, one scan over the (chunk, wave) cells, two barriers in all. ----
    constexpr int kFastChunks = 8;
    const int nchunks = (nv + 4 * NT - 1) / (4 * NT);
    if (cached && nchunks <= kFastChunks && all_sel) {
        uint32_t *cellsum = hist1;                     // [kFastChunks / 2][NW]  (the histogram is dead: its barrier is behind us)
        uint32_t *cellbase = cellsum + kFastChunks / 2 * NW;   // [kFastChunks * NW]
        uint32_t cw[kFastChunks / 2], inc[kFastChunks / 2];
#pragma unroll
        for (int j = 0; j < kFastChunks / 2; ++j) {
            uint32_t n2[2] = {0u, 0u};
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int p = (2 * j + h) * 4 * NT + 4 * tid;
                if (2 * j + h < nchunks) {             // workgroup-uniform
                    const u32x4 k4 = get_key4(p);
#pragma unroll
                    for (int e = 0; e < 4; ++e) n2[h] += (p + e < nv && k4[e] >= tau) ? 1u : 0u;
                }
            }
            cw[j] = n2[0] | (n2[1] << 16);
            inc[j] = wave_incl_scan(cw[j]);
        }
        if (lane == 63) {
#pragma unroll
            for (int j = 0; j < kFastChunks / 2; ++j) cellsum[j * NW + wave] = inc[j];
        }
        __syncthreads();
        if (wave == 0) {
            // cells in (chunk, wave) order, 64 at a time
            uint32_t carry = 0;
#pragma unroll
            for (int base = 0; base < kFastChunks * NW; base += 64) {
                const int cell = base + lane, c = cell / NW, w = cell % NW;
                const bool real = cell < kFastChunks * NW;
                const uint32_t v = real ? (cellsum[(c >> 1) * NW + w] >> (16 * (c & 1))) & 0xFFFFu : 0u;
                const uint32_t in = wave_incl_scan(v);
                if (real) cellbase[cell] = carry + in - v;
                carry += __shfl(in, 63);
            }
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < kFastChunks; ++c) {
            if (c >= nchunks) continue;                // workgroup-uniform
            const int p = c * 4 * NT + 4 * tid;
            const u32x4 k4 = get_key4(p);
            uint32_t slot = cellbase[c * NW + wave] + (((inc[c >> 1] - cw[c >> 1]) >> (16 * (c & 1))) & 0xFFFFu);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (p + e < nv && k4[e] >= tau) {
                    if (slot < (uint32_t)a.k_sel) {    // always true for a consistent select
                        oidx[slot] = p + e;
                        if (osel) osel[slot] = key_score(k4[e]);
                    }
                    ++slot;
                }
            }
        }
        return;
    }

    // ---- ordered emit, general case: slot = #greater before + min(#equal before, need_eq) ----
    // A thread owns 4 consecutive positions; the counts of greater / equal entries of ONE chunk
    // (at most 4 * NT of each) travel packed in one word (equal << 16 | greater) through a wave scan
    // and a 16-entry scan of the wave totals.  The totals over all previous chunks are kept in two
    // full words: a row longer than 65535 keys may tie with the k-th score in more than 65535 places.
    static_assert(4 * NT < 65536, "per-chunk counts must fit 16 bits");
    uint32_t run_g = 0, run_e = 0;                     // greater / equal entries of all previous chunks
#pragma unroll 1
    for (int c = 0; c < nchunks; ++c) {
        const int p = c * 4 * NT + 4 * tid;
        const u32x4 k4 = get_key4(p);
        uint32_t gm = 0, em = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (p + e < nv) {
                gm |= ((all_sel ? k4[e] >= tau : k4[e] > tau) ? 1u : 0u) << e;
                em |= ((!all_sel && k4[e] == tau) ? 1u : 0u) << e;
            }
        }
        const uint32_t mine = ((uint32_t)__popc(em) << 16) | (uint32_t)__popc(gm);
        uint32_t incl = mine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t up = __shfl_up(incl, off);
            if (lane >= off) incl += up;
        }
        uint32_t *wt = wsum + (c & 1) * NW;
        if (lane == 63) wt[wave] = incl;
        __syncthreads();
        uint32_t ws = lane < NW ? wt[lane] : 0u;       // scan of the wave totals (NW <= 16)
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
            const uint32_t up = __shfl_up(ws, off);
            if (lane >= off) ws += up;
        }
        const uint32_t waves_before = wave == 0 ? 0u : __shfl(ws, wave - 1);
        const uint32_t chunk_total = __shfl(ws, NW - 1);
        const uint32_t before = waves_before + incl - mine;   // inside this chunk: both fields < 65536
        uint32_t g_before = run_g + (before & 0xFFFFu), e_before = run_e + (before >> 16);
        if ((gm | em) != 0u) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool g = (gm >> e) & 1u, q = (em >> e) & 1u;
                if (g || (q && e_before < need_eq)) {
                    const uint32_t slot = g_before + (e_before < need_eq ? e_before : need_eq);
                    if (slot < (uint32_t)a.k_sel) {    // always true for a consistent select
                        oidx[slot] = p + e;
                        if (osel) osel[slot] = key_score(k4[e]);
                    }
                }
                g_before += g ? 1u : 0u;
                e_before += q ? 1u : 0u;
            }
        }
        run_g += chunk_total & 0xFFFFu;
        run_e += chunk_total >> 16;
    }
}

// The arguments that the way to a row's first load needs, requested together: left alone each is loaded where it is first used, a
// chain of memory latencies in front of a launch of 10 to 20 us.
__device__ __forceinline__ void request_args(const SelectArgs &a)
{
    asm volatile("" ::"s"(a.strip), "s"(a.ld), "s"(a.q_pos0), "s"(a.Tq), "s"(a.Lk), "s"(a.k_sel), "s"(a.b0), "s"(a.i0), "s"(a.Ri), "s"(a.idx), "s"(a.seq_lens));
}

template <int NT>
__global__ __launch_bounds__(NT) void select_kernel(SelectArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
    request_args(a);
    select_row_generic<NT>(a, smem);
}

// ---- candidate form (long rows) ------------------------------------------------------------------
// For rows much longer than k almost every key is far below the k-th score, and pushing all of them through
// the digit histograms (LDS atomics into the few dozen bins a row's exponents fall into) is what the generic
// form spends its time on.  Here the row is read ONCE:
//   sample    4096 keys in 256 short stretches spread over the row -> a histogram of 4096 linear bins between
//             the smallest and the largest sampled key -> a threshold T0 that about 2k keys of the row should reach
//   sweep     one pass over the row: the keys >= T0 go to a candidate list in LDS (one atomic per wave and step: a wave
//             scan places the entries), their maximum is tracked
//   select    one histogram over the candidates with 4096 LINEAR bins between T0 and that maximum (candidates
//             spread over all of them), a scan for the bin of the k-th largest, and an exact ranking
//             (key descending, position ascending) of the few members of that bin
//   emit      selected positions set bits in a bitmap of the row; a prefix count over the bitmap words gives
//             every selected candidate its slot, so positions come out ascending with their scores
// Exact for every input: whenever a step cannot proceed (fewer than k candidates, more than the list holds,
// too many ties in the boundary bin) the workgroup falls back to the generic radix select on the same row.
constexpr int kCandCap = 12288;          // candidate list entries (6 k for k = 2048)
constexpr int kCandMinLen = 8192;        // shorter rows of a launch take the generic form at once
constexpr int kCandMaxLen = 131072;      // bitmap capacity
constexpr int kCandSample = 4096;
constexpr int kBoundaryCap = 1024;       // boundary-bin members ranked exactly
// A second instance for launches of more rows than CUs: half the threads and half the LDS, so that two rows are in flight per CU
// (a row's phases are chains of latencies; a second workgroup fills them), and a threshold nearer to the k-th key.  us, one row per CU /
// two: 257 rows of 41700 keys 39 / 25, 700 62 / 49, 2048 rows of up to 40000 keys 159 / 110, 65536 199 / 166, 131072 294 / 254; with
// scores of which half is a component that decays over 64 keys 700 rows of 41700 64 / 46, 2048 of 65536 221 / 157, of 131072 421 / 361
// (one row that leaves the form is a hundred us at the launch's end), over 256 keys 513 / 251.
constexpr int kCandManyCap = 6112;
// Stretches of the sample, 64 bytes each: neighbouring keys score alike, and fewer and longer ones count for less.  Half of the scores'
// variance in a component that decays over 64 (256) keys, 131072 keys, k = 2048: with 32 stretches of 128 keys 8 (16) per cent of the rows
// left too few or too many candidates for a list of 6112, with 256 none of 120; lists of 704 for every wave overflowed in another 20.
constexpr int kCandRuns = 256;
// Rank in the sample of the threshold that k of nv keys should reach.
__host__ __device__ inline uint32_t cand_rank(int k, int nv, bool many)
{
    uint32_t rank = (uint32_t)(((int64_t)kCandSample * 2 * k) / nv) + 32u;
    if (many) {                                // k of nv keys are `mean` of the sample, give or take its root or, of neighbours, more
        const float mean = (float)kCandSample * (float)k / (float)nv;
        rank = (uint32_t)(mean + 4.5f * __builtin_sqrtf(mean)) + 4u;
    }
    return rank > (uint32_t)kCandSample ? (uint32_t)kCandSample : rank;
}
constexpr int cand_lds_words(int nt, int maxlen, int cap) { return kBins1 + 2 * (nt / 64) + 4 + 16 + 2 * cap + maxlen / 32; }

// Largest value over the 64 lanes of a wave, in every lane (no LDS traffic; lanes without a source keep their own).
__device__ __forceinline__ uint32_t wave_max_dpp(uint32_t x)
{
#define IC_DPP_MAX(ctrl, rows) x = max(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, ctrl, rows, 0xf, false))
    IC_DPP_MAX(0x111, 0xf);              // row_shr:1, 2, 4, 8
    IC_DPP_MAX(0x112, 0xf);
    IC_DPP_MAX(0x114, 0xf);
    IC_DPP_MAX(0x118, 0xf);
    IC_DPP_MAX(0x142, 0xa);              // row_bcast:15 into rows 1, 3
    IC_DPP_MAX(0x143, 0xc);              // row_bcast:31 into rows 2, 3
#undef IC_DPP_MAX
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

template <int NT, int MAXLEN, int CAP, bool MANY>
__global__ __launch_bounds__(NT) void select_cand_kernel(SelectArgs a)
{
    static_assert(kCandSample % (4 * NT) == 0 && (MAXLEN / 32) % NT == 0, "whole sample vectors and bitmap words per thread");
    request_args(a);
    constexpr int NW = NT / 64;
    constexpr int SV = kCandSample / (4 * NT); // sample vectors per thread
    constexpr int BW = MAXLEN / 32 / NT;       // bitmap words per thread
    extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
    uint32_t *hist = smem;                     // [kBins1]  (the generic form's layout starts the same way)
    uint32_t *wsum = hist + kBins1;            // [2 NW]
    uint32_t *bc = wsum + 2 * NW;              // [4]
    uint32_t *misc = bc + 4;                   // [16]: 0 candidate count, 1 largest candidate key, 2 boundary-list count
    uint32_t *ckey = misc + 16;                // [CAP]
    uint32_t *cpos = ckey + CAP;               // [CAP]
    uint32_t *bitmap = cpos + CAP;             // [MAXLEN / 32]
    // once the histograms are read: the boundary bin's members (key, position), then the selected entries ahead of each bitmap word
    uint32_t *wpre = hist;
    static_assert(2 * kBoundaryCap <= kBins1 && MAXLEN / 32 <= kBins1, "they share its space");

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = blockIdx.x;
    const int b = a.b0 + r / a.Ri;
    const int i = a.i0 + r % a.Ri;
    if (i >= a.Tq) return;
    const int Lk_b = a.seq_lens ? max(0, min(a.seq_lens[b], a.Lk)) : a.Lk;
    int64_t nv64 = (a.seq_lens ? (int64_t)Lk_b - a.Tq : a.q_pos0) + (int64_t)i + 1;
    nv64 = nv64 < 0 ? 0 : (nv64 > Lk_b ? Lk_b : nv64);
    const int nv = (int)nv64;
    // The candidate form proper; false = this row takes the generic form (one call site below: a fallback reached
    // through several calls is not inlined, and a kernel argument captured by a real function is copied to scratch
    // memory by every thread of every row).
    auto candidate_form = [&]() -> bool {
    if (nv < kCandMinLen || nv < 4 * a.k_sel) return false;    // (short rows of a ragged launch) workgroup-uniform
    const float *row = a.strip + (int64_t)r * a.ld;
    int32_t *oidx = a.idx + ((int64_t)b * a.Tq + i) * a.k_sel;
    float *osel = a.sel ? a.sel + ((int64_t)b * a.Tq + i) * a.k_sel : nullptr;
    const uint32_t k = (uint32_t)a.k_sel;

    // The row arrives in groups of kGroup vectors per thread, two groups in flight: a single workgroup has to
    // cover the whole memory latency by itself.  The sample and the first group are requested before anything else.
    constexpr int kGroup = 4;
    const int nsteps = (nv + 4 * NT - 1) / (4 * NT);
    auto load_group = [&](int c0, f32x4 (&dst)[kGroup]) {
#pragma unroll
        for (int j = 0; j < kGroup; ++j) {
            const int p = ((c0 + j) * NT + tid) * 4;
            dst[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (p < nv) dst[j] = *(const f32x4 *)(row + p);   // may run past nv inside the row's padding; masked below
        }
    };
    f32x4 ga[kGroup], gb[kGroup];
    f32x4 sv[SV];
#pragma unroll
    for (int u = 0; u < SV; ++u) {
        constexpr int kLanes = kCandSample / kCandRuns / 4;    // to a stretch
        static_assert(kCandMinLen / kCandRuns >= 4 * kLanes && (int64_t)kCandRuns * MAXLEN <= INT32_MAX, "p + 3 < nv");
        const int p = ((u * NT + tid) / kLanes * nv / kCandRuns & ~(4 * kLanes - 1)) + tid % kLanes * 4;
        sv[u] = *(const f32x4 *)(row + p);
    }
    load_group(0, ga);

    // ---- sample: a histogram of 4096 linear bins between the smallest and the largest of
    //      them (the scores of a row share a few exponents: bins of a key digit would be hit a hundred times each,
    //      and LDS atomics on one address take turns) ----
    for (int e = tid; e < kBins1; e += NT) hist[e] = 0;
#pragma unroll
    for (int q = 0; q < BW; ++q) bitmap[BW * tid + q] = 0;
    if (tid < 16) misc[tid] = 0;
    uint32_t skey[4 * SV];
    uint32_t kmx = 0u, kmn = 0xFFFFFFFFu;
#pragma unroll
    for (int e = 0; e < 4 * SV; ++e) {
        skey[e] = score_key(sv[e >> 2][e & 3]);
        kmx = max(kmx, skey[e]);
        kmn = min(kmn, skey[e]);
    }
    {
        const uint32_t mx = wave_max_dpp(kmx);
        const uint32_t mn = ~wave_max_dpp(~kmn);
        if (lane == 0) {
            wsum[wave] = mn;
            wsum[NW + wave] = mx;
        }
    }
    __syncthreads();
    const uint32_t smin = ~wave_max_dpp(~(lane < NW ? wsum[lane] : 0xFFFFFFFFu));
    const uint32_t smax = wave_max_dpp(lane < NW ? wsum[NW + lane] : 0u);
    const uint32_t srange = smax - smin;
    const int sbits = srange ? 32 - __clz((int)srange) : 0;
    const int ssh = sbits > 12 ? sbits - 12 : 0;
#pragma unroll
    for (int e = 0; e < 4 * SV; ++e) atomicAdd(&hist[(skey[e] - smin) >> ssh], 1u);
    __syncthreads();
    find_digit<NT, kBins1 / NT>(hist, cand_rank(a.k_sel, nv, MANY), wsum, bc, tid, lane, wave);
    const uint32_t T0 = smin + (bc[0] << ssh); // a bin's lower edge: at least `want` sampled keys reach it
    __syncthreads();

    // ---- sweep: the row once, the positions of the candidates to the list ----
    // The sweep is bound by vector-ALU instructions (sixteen keys per thread and group), so it does the least per
    // key: one float comparison against the threshold (the key order is the float order) into a bit mask; only the
    // set bits are visited afterwards, and only positions are stored -- the few candidates' keys are read back
    // from the row (still in L2) once the sweep is over.
    // (rows of up to 65536 keys: a workgroup's row is still in L2 when its candidates are read back; longer rows of
    // a full grid push one another out, there the keys are stored during the sweep)
    const bool reread = nv <= 65536;           // workgroup-uniform
    {
        const float T0f = key_score(T0);
        auto sweep_group = [&](int c0, const f32x4 (&v)[kGroup]) {
            uint32_t m = 0;
#pragma unroll
            for (int j = 0; j < kGroup; ++j) {
                const int p = ((c0 + j) * NT + tid) * 4;
#pragma unroll
                for (int e = 0; e < 4; ++e) m |= (uint32_t)((int)(p + e < nv) & (int)(v[j][e] >= T0f)) << (4 * j + e);
            }
            const uint32_t n_t = (uint32_t)__popc(m);
            const uint32_t incl = wave_incl_scan(n_t);
            const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            if (total == 0u) return;               // wave-uniform
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&misc[0], total);
            uint32_t off = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + incl - n_t;
            if (reread) {
                while (m) {
                    const int bit = __builtin_ctz(m);
                    m &= m - 1u;
                    if (off < (uint32_t)CAP) cpos[off] = (uint32_t)(((c0 + (bit >> 2)) * NT + tid) * 4 + (bit & 3));
                    ++off;
                }
            } else {
#pragma unroll
                for (int j = 0; j < kGroup; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if ((m >> (4 * j + e)) & 1u) {
                            if (off < (uint32_t)CAP) {
                                cpos[off] = (uint32_t)(((c0 + j) * NT + tid) * 4 + e);
                                ckey[off] = max(score_key(v[j][e]), T0);
                            }
                            ++off;
                        }
            }
        };
#pragma unroll 1
        for (int c0 = 0; c0 < nsteps; c0 += 2 * kGroup) {
            if (c0 + kGroup < nsteps) load_group(c0 + kGroup, gb);
            sweep_group(c0, ga);
            if (c0 + kGroup >= nsteps) break;
            if (c0 + 2 * kGroup < nsteps) load_group(c0 + 2 * kGroup, ga);
            sweep_group(c0 + kGroup, gb);
        }
    }
    __syncthreads();
    const uint32_t n_cand = misc[0];
    if (n_cand < k || n_cand > (uint32_t)CAP) {    // workgroup-uniform
        __syncthreads();
        return false;
    }
    // the candidates' keys and their maximum
    {
        uint32_t tmax = 0;
        for (uint32_t j = tid; j < n_cand; j += NT) {
            uint32_t key;
            if (reread) {
                key = max(score_key(row[cpos[j]]), T0);   // (>= T0 by construction; the bins below rely on it)
                ckey[j] = key;                 // (read again by this thread only)
            } else {
                key = ckey[j];
            }
            tmax = max(tmax, key);
        }
        tmax = wave_max_dpp(tmax);
        if (lane == 0 && tmax != 0u) atomicMax(&misc[1], tmax);
    }

    // ---- one histogram over the candidates: 4096 linear bins over [T0, kmax] ----
    for (int e = tid; e < kBins1; e += NT) hist[e] = 0;
    __syncthreads();
    const uint32_t kmax = misc[1];
    const uint32_t range = kmax - T0;
    const int nbits = range ? 32 - __clz((int)range) : 0;
    const int sh = nbits > 12 ? nbits - 12 : 0;
    for (uint32_t j = tid; j < n_cand; j += NT) atomicAdd(&hist[(ckey[j] - T0) >> sh], 1u);
    __syncthreads();
    find_digit<NT, kBins1 / NT>(hist, k, wsum, bc, tid, lane, wave);
    const uint32_t bstar = bc[0], need = bc[1], n_b = bc[2];
    __syncthreads();
    const bool ranked = need < n_b;            // the boundary bin is cut: rank its members exactly
    if (ranked && n_b > (uint32_t)kBoundaryCap) return false;

    // ---- mark the selected positions ----
    uint32_t *bl_key = wpre, *bl_pos = wpre + kBoundaryCap;
    for (uint32_t j = tid; j < n_cand; j += NT) {
        const uint32_t bin = (ckey[j] - T0) >> sh;
        if (bin > bstar || (bin == bstar && !ranked)) {
            atomicOr(&bitmap[cpos[j] >> 5], 1u << (cpos[j] & 31u));
        } else if (bin == bstar) {
            const uint32_t s = atomicAdd(&misc[2], 1u);
            bl_key[s] = ckey[j];
            bl_pos[s] = cpos[j];
        }
    }
    __syncthreads();
    if (ranked) {
        for (uint32_t m = tid; m < n_b; m += NT) {
            const uint32_t km = bl_key[m], pm = bl_pos[m];
            uint32_t ahead = 0;                // members that beat this one: larger key, or equal key at a lower position
#pragma unroll 4
            for (uint32_t x = 0; x < n_b; ++x) {       // (no branch: positions would be asked for after their keys)
                const uint32_t kx = bl_key[x], px = bl_pos[x];
                ahead += (uint32_t)(kx > km) | ((uint32_t)(kx == km) & (uint32_t)(px < pm));
            }
            if (ahead < need) atomicOr(&bitmap[pm >> 5], 1u << (pm & 31u));
        }
        __syncthreads();
    }

    // ---- slots: selected entries ahead of every bitmap word ----
    {
        uint32_t wcnt[BW], mine = 0;
#pragma unroll
        for (int q = 0; q < BW; ++q) {
            wcnt[q] = (uint32_t)__popc(bitmap[BW * tid + q]);
            mine += wcnt[q];
        }
        const uint32_t incl = wave_incl_scan(mine);
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();                       // also: every read of the boundary list is over, wpre may be overwritten
        uint32_t before = 0;
#pragma unroll
        for (int wv = 0; wv < NW; ++wv)
            if (wv < wave) before += wsum[wv];
        uint32_t run = before + incl - mine;
#pragma unroll
        for (int q = 0; q < BW; ++q) {
            wpre[BW * tid + q] = run;
            run += wcnt[q];
        }
    }
    __syncthreads();
    for (uint32_t j = tid; j < n_cand; j += NT) {
        const uint32_t pos = cpos[j], word = bitmap[pos >> 5], bit = pos & 31u;
        if ((word >> bit) & 1u) {
            const uint32_t slot = wpre[pos >> 5] + (uint32_t)__popc(word & ((1u << bit) - 1u));
            if (slot < k) {                    // always true for a consistent select
                oidx[slot] = (int32_t)pos;
                if (osel) osel[slot] = key_score(ckey[j]);
            }
        }
    }
    return true;
    };
    if (!candidate_form()) {
        SelectArgs ga = a;
        // the candidate arrays' space serves as the row cache (rows that do not fit it are streamed)
        constexpr int kSpace = 16 + 2 * CAP + MAXLEN / 32;
        ga.cache_elems = kSpace >= 32768 ? 32768 : kSpace / 64 * 64;
        select_row_generic<NT>(ga, smem);
    }
}

struct RowView {
    int b, i, nv;
};
__device__ __forceinline__ RowView row_view(const SelectArgs &a, int r)
{
    RowView v;
    v.b = a.b0 + r / a.Ri;
    v.i = a.i0 + r % a.Ri;
    const int Lk_b = a.seq_lens ? max(0, min(a.seq_lens[v.b], a.Lk)) : a.Lk;
    const int64_t nv64 = (a.seq_lens ? (int64_t)Lk_b - a.Tq : a.q_pos0) + (int64_t)v.i + 1;
    v.nv = (int)(nv64 < 0 ? 0 : (nv64 > Lk_b ? Lk_b : nv64));
    return v;
}

// ---- bins form -----------------------------------------------------------------------------------------------------
// The whole row sits in registers (4 NV scores a thread), and one histogram of NB bins, LINEAR between the row's smallest
// and largest score, finds the bin of the k-th largest: the scores of a row are spread over all of them, while bins of a
// key's leading bits (the radix form's) are hit by a few exponents, a hundred times each, and LDS atomics on one address
// take turns.  The few members of that bin are ranked exactly, which gives the k-th score and the position up to which
// entries equal to it belong to the result.  Where the bin has more members than kRankCap (an outlier stretches the range,
// ties), or a score is no finite number, keys take the scores' place, in bins linear between the smallest and the largest
// one that is left, until that bin is small enough, or all of it is equal and the position is counted.  The selected
// positions leave through a bitmap of the row, in whole lines.
// What bounds it: with few rows a chain of nine barriers, with many their LDS atomics, one per key (before, rows of up to 8192
// keys took the radix form, longer ones the candidate form; us, one row in parentheses the number of them): 10007 keys (1) 13.2
// -> 7.8, 30011 (24) 17.0 -> 14.9, 64 of 1 to 512 (512) 8.7 -> 5.6, 2048 of 1 to 4096 (4096) 27 -> 20, of 6145 to 8192 (2048)
// 44 -> 25, of 12289 to 16384 (4096) 137 -> 67, of 30721 to 32768 (2048) 93 -> 71.  With 64 keys a thread it is no faster
// than the candidate form (64 K keys, 32 rows: 20.6 and 19.4).
constexpr int kBinsLen = 32768;
constexpr int kRankCap = 64;             // (each is compared with all others: 150 ties of 2400 keys cost more than the rest of the row)

template <int NT, int NV, int NB>
struct BinsLds {
    static constexpr int NW = NT / 64;
    static constexpr int kWords = NT * NV / 8; // bitmap
    static constexpr int kList = kRankCap * 2 > IC_MAX_K ? kRankCap * 2 : IC_MAX_K;
    static_assert(NB % NT == 0, "whole bins per thread");
    // the histogram and a place per lane; once it is read the boundary bin's members (keys, positions), then the selected
    // positions, and behind them the bitmap
    uint32_t smem[NB + 64 > kList + kWords ? NB + 64 : kList + kWords];
    uint32_t wsum[NW], bc[4], red[2 * NW];
    uint32_t misc[5];                          // 0 members listed, 1 k-th key, 2 its position, 3 equal ones behind it, 4 odd scores
};

// every visible key is selected (nv <= k)
template <int NT>
__device__ __forceinline__ void select_all(const float *row, int nv, int k, int32_t *oidx, float *osel, int tid)
{
    if (k % 4 == 0 && (uintptr_t)oidx % 16 == 0) {
        for (int s = 4 * tid; s < k; s += 4 * NT)
            *(i32x4 *)(oidx + s) = i32x4{s < nv ? s : -1, s + 1 < nv ? s + 1 : -1, s + 2 < nv ? s + 2 : -1, s + 3 < nv ? s + 3 : -1};
    } else {
        for (int s = tid; s < k; s += NT) oidx[s] = s < nv ? s : -1;
    }
    if (osel)
        for (int s = tid; s < k; s += NT) osel[s] = s < nv ? row[s] : -INFINITY;
}

// One row of nv > k scores (16-byte aligned, readable up to the next multiple of four) by NT threads that sync() brings together.
template <int NT, int NV, int NB, typename Sync>
__device__ __forceinline__ void bins_select(const float *row, int nv, int k, int32_t *oidx, float *osel, BinsLds<NT, NV, NB> &lds, int tid, Sync sync)
{
    constexpr int NW = NT / 64, kList = BinsLds<NT, NV, NB>::kList;
    uint32_t *const smem = lds.smem, *const wsum = lds.wsum, *const bc = lds.bc, *const red = lds.red, *const misc = lds.misc;
    uint32_t *hist = smem, *member = smem, *member_at = smem + kRankCap, *out = smem, *bitmap = smem + kList;
    const int nsteps = (nv + 4 * NT - 1) / (4 * NT);
    u32x4 v[NV];                               // scores, later maybe keys
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int p = (j * NT + tid) * 4;
        if (p < nv) v[j] = *(const u32x4 *)(row + p);          // may run past nv inside the row's padding
    }
    const float f0 = row[0];
    const int lane = tid & 63, wave = tid >> 6;
    for (int e = tid; e < NB; e += NT) hist[e] = 0;
    if (tid < 5) misc[tid] = 0;
    sync();
    // Slots behind the row hold its first score, so that the sweeps below need no test; what they add is taken off the
    // counts again, and their bits off the bitmap.
    const uint32_t pad = (uint32_t)(nsteps * 4 * NT - nv);
    // (opaque values: the compiler would keep the steps' conditions, positions and bins from one sweep to the next)
    auto again = [](int n) { asm volatile("" : "+s"(n)); return n; };
    auto each = [&](auto f) __attribute__((always_inline)) {
        const int steps = again(nsteps);
        int at = 4 * tid;
        asm volatile("" : "+v"(at));
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (j < steps) {                   // workgroup-uniform
#pragma unroll
                for (int e = 0; e < 4; ++e) f(v[j][e], at + j * NT * 4 + e);
            }
    };
    uint32_t lo, hi;
    auto bounds = [&](uint32_t mx, uint32_t mn) {              // of the threads' largest and smallest keys
        mx = wave_max_dpp(mx);
        mn = wave_max_dpp(~mn);
        if constexpr (NW > 1) {
            if (lane == 0) {
                red[wave] = mx;
                red[NW + wave] = mn;
            }
            sync();
            mx = wave_max_dpp(red[lane % NW]);
            mn = wave_max_dpp(red[NW + lane % NW]);
        }
        hi = mx;
        lo = ~mn;
    };
    bool odd;                                  // a score is infinite or none
    {
        float mx = f0, mn = f0, z = 0.f;
        const int end = again(nv);
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (j < nsteps) {
                const int p = (j * NT + tid) * 4;
                if (p + 3 >= end) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[j][e] = p + e < end ? v[j][e] : __float_as_uint(f0);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = __uint_as_float(v[j][e]);
                    mx = fmaxf(mx, x);
                    mn = fminf(mn, x);
                    z = __builtin_fmaf(x, 0.f, z);
                }
            }
        if (__ballot(!(z == 0.f)) != 0ull && lane == 0) misc[4] = 1u;
        bounds(score_key(mx), score_key(mn));
        if constexpr (NW == 1) sync();
        odd = misc[4] != 0u;
    }
    auto mark = [&](auto pred) __attribute__((always_inline)) {    // bit p of the bitmap: pred(key, p); eight lanes make a word
        const int steps = again(nsteps);
        int at = 4 * tid;
        asm volatile("" : "+v"(at));
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (j < steps) {
                uint32_t m = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) m |= (pred(v[j][e], (uint32_t)(at + j * NT * 4 + e)) ? 1u : 0u) << e;
                m <<= 4 * (lane & 7);
                m |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xf, 0xf, true);    // the neighbour in a pair,
                m |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xf, 0xf, true);    // the other pair of four,
                m |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x141, 0xf, 0xf, true);   // the other four of eight lanes
                if ((lane & 7) == 0) bitmap[(at >> 5) + j * (NT / 8)] = m;
            }
    };
    // this thread's 4 NV bits of it, from position at0, and the number of set ones in front of them
    constexpr int MW = NV >= 8 ? NV / 8 : 1;
    const int at0 = tid * 4 * NV;
    auto mine = [&](uint32_t (&m)[MW]) __attribute__((always_inline)) -> uint32_t {
        uint32_t n = 0;
#pragma unroll
        for (int q = 0; q < MW; ++q) {
            const int left = nv - (at0 + 32 * q);
            m[q] = 0;
            if (left > 0) {
                m[q] = bitmap[(at0 >> 5) + q];
                if constexpr (NV < 8) m[q] = (m[q] >> (at0 & 31)) & ((1u << (4 * NV)) - 1);
                if (left < 32) m[q] &= (1u << left) - 1;
            }
            n += (uint32_t)__popc(m[q]);
        }
        uint32_t before = wave_incl_scan(n);
        if (lane == 63) wsum[wave] = before;
        sync();
        before -= n;
#pragma unroll
        for (int wv = 0; wv < NW - 1; ++wv)
            if (wv < wave) before += wsum[wv];
        return before;
    };
    uint32_t need = (uint32_t)k;
    // the members of the boundary bin, listed, ranked (keys descending, positions ascending): the last one wanted
    auto rank = [&](uint32_t n_b) __attribute__((always_inline)) {
        sync();
        for (uint32_t m = tid; m < n_b; m += NT) {
            const uint32_t xm = member[m], pm = member_at[m];
            uint32_t ahead = 0, behind = 0;    // members that beat this one: larger, or equal at a lower position
#pragma unroll 4
            for (uint32_t o = 0; o < n_b; ++o) {
                const uint32_t xo = member[o], po = member_at[o];
                ahead += (uint32_t)(xo > xm) | ((uint32_t)(xo == xm) & (uint32_t)(po < pm));
                behind += (uint32_t)(xo == xm) & (uint32_t)(po > pm);
            }
            if (ahead + 1 == need) {
                misc[1] = xm;
                misc[2] = pm;
                misc[3] = behind;
            }
        }
        sync();
    };
    auto list = [&](uint32_t key, int p) {
        const uint32_t m = atomicAdd(&misc[0], 1u);
        member[m] = key;
        member_at[m] = (uint32_t)p;
    };
    auto clear = [&]() {
        for (int e = tid; e < NB; e += NT) hist[e] = 0;
    };
    // bins of scores
    const float first = key_score(lo), scale = (NB - 0.5f) / (key_score(hi) - first);
    bool scores = false;                       // they decide
    if (!odd && scale > 0.f && scale < 3e38f) {                // (one value only, or a range beyond floats: no bins)
        // (monotone, NB - 1 at most)
        auto bin = [](float x, float from, float by) { return (uint32_t)((x - from) * by); };
        // A ReLU's zeros, or all of a row but its largest scores, would take turns in the lowest bin.  A wave that finds an eighth of its
        // first scores there gives them a place per lane behind the bins, and that bin is what the others leave (one head of 30000 keys,
        // half of them zero: 32.5 us counted, 21.7 so; 2048 rows of 32768 388 / 310).  Asked for every key, that took other rows 0.1 to 1.5
        // us.  A single wave's rows are too short for it to matter.
        constexpr bool all = NW == 1;
        if (tid == 0) {
            if (all || bin(f0, first, scale)) atomicSub(&hist[bin(f0, first, scale)], pad);
            if (!all) atomicAdd(&hist[0], (uint32_t)nv);       // (for the scan, which ends here at the latest)
        }
        if (all || __builtin_expect(__popcll(__ballot(bin(__uint_as_float(v[0][0]), first, scale) == 0u)) < 8, 1))
            each([&](uint32_t x, int) { atomicAdd(&hist[bin(__uint_as_float(x), first, scale)], 1u); });
        else
            each([&](uint32_t x, int) {
                const uint32_t at = bin(__uint_as_float(x), first, scale);
                atomicAdd(&hist[at ? at : NB + lane], 1u);
            });
        sync();
        find_digit<NT, NB / NT>(hist, need, wsum, bc, tid, lane, wave, sync);
        const uint32_t b = bc[0], n_b = all || b ? bc[2] : (uint32_t)(nv - k) + bc[1];
        need = bc[1];
        float from = first;                    // (opaque: bins are worked out again)
        asm volatile("" : "+v"(from));
        if (n_b <= (uint32_t)kRankCap) {
            const int len = again(nv);
            each([&](uint32_t x, int p) {
                if (bin(__uint_as_float(x), from, scale) == b && p < len) list(score_key(__uint_as_float(x)), p);
            });
            rank(n_b);
            scores = true;
        } else {
            uint32_t mx = 0u, mn = 0xFFFFFFFFu;                // (a thread without members has neither)
            each([&](uint32_t x, int) {
                if (bin(__uint_as_float(x), from, scale) == b) {
                    mx = max(mx, score_key(__uint_as_float(x)));
                    mn = min(mn, score_key(__uint_as_float(x)));
                }
            });
            sync();                   // (everybody has read hist, bc and red)
            clear();
            bounds(mx, mn);
        }
    } else if (odd) {                          // (the bounds so far know no NaN)
        uint32_t mx = 0u, mn = 0xFFFFFFFFu;
        each([&](uint32_t x, int) {
            mx = max(mx, score_key(__uint_as_float(x)));
            mn = min(mn, score_key(__uint_as_float(x)));
        });
        sync();
        bounds(mx, mn);
    }
    uint32_t tau, ptau;
    bool cut;                                  // entries equal to tau behind ptau are left out
    if (!scores) {
        // bins of keys
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[j][e] = score_key(__uint_as_float(v[j][e]));
        const uint32_t x0 = score_key(f0);
        while (lo != hi) {
#pragma unroll
            for (int j = 0; j < NV; ++j) asm volatile("" : "+v"(v[j]));   // (nothing is worked out ahead of the loop and kept)
            const int bits = 32 - __clz((int)(hi - lo));
            constexpr int kBits = 31 - __builtin_clz(NB);
            const int sh = bits > kBits ? bits - kBits : 0;
            const uint32_t span = hi - lo;
            if constexpr (NW == 1) sync();
            if (tid == 0 && x0 - lo <= span) atomicSub(&hist[(x0 - lo) >> sh], pad);
            each([&](uint32_t x, int) { if (x - lo <= span) atomicAdd(&hist[(x - lo) >> sh], 1u); });
            sync();
            find_digit<NT, NB / NT>(hist, need, wsum, bc, tid, lane, wave, sync);
            const uint32_t n_b = bc[2];
            need = bc[1];
            // the bin's keys (`from` opaque: differences are worked out again)
            uint32_t from = lo + (bc[0] << sh);
            const uint32_t last = min((1u << sh) - 1u, hi - from);
            asm volatile("" : "+v"(from));
            if (n_b <= (uint32_t)kRankCap) {
                const int len = again(nv);
                each([&](uint32_t x, int p) { if (x - from <= last && p < len) list(x, p); });
                rank(n_b);
                break;
            }
            uint32_t mx = 0u, mn = 0xFFFFFFFFu;
            each([&](uint32_t x, int) {
                if (x - from <= last) {
                    mx = max(mx, x);
                    mn = min(mn, x);
                }
            });
            sync();
            clear();
            bounds(mx, mn);
        }
    }
    if (!scores && lo == hi) {                 // all members are equal: count up to the last one wanted
        sync();
        tau = lo;
        cut = true;
        mark([&](uint32_t x, uint32_t) { return x == tau; });
        sync();
        uint32_t m[MW];
        uint32_t before = mine(m);
#pragma unroll
        for (int q = 0; q < MW; ++q) {
            const uint32_t n = (uint32_t)__popc(m[q]);
            if (before < need && need <= before + n) {
                for (uint32_t d = need - before; d > 1; --d) m[q] &= m[q] - 1;
                misc[2] = (uint32_t)(at0 + 32 * q + __builtin_ctz(m[q]));
            }
            before += n;
        }
        sync();
    } else {
        tau = misc[1];
        cut = misc[3] != 0u;
    }
    ptau = misc[2];
    if (scores) {
        const float t = key_score(tau);
        if (!cut)
            mark([&](uint32_t x, uint32_t) { return __uint_as_float(x) >= t; });
        else
            mark([&](uint32_t x, uint32_t p) { return __uint_as_float(x) > t || (__uint_as_float(x) == t && p <= ptau); });
    } else if (!cut)
        mark([&](uint32_t x, uint32_t) { return x >= tau; });
    else
        mark([&](uint32_t x, uint32_t p) { return x > tau || (x == tau && p <= ptau); });
    sync();
    {
        uint32_t m[MW];
        uint32_t slot = mine(m);
#pragma unroll
        for (int q = 0; q < MW; ++q)
            while (m[q]) {
                if (slot < (uint32_t)k) out[slot] = (uint32_t)(at0 + 32 * q + __builtin_ctz(m[q]));   // (always, for a consistent select)
                m[q] &= m[q] - 1;
                ++slot;
            }
    }
    sync();
    for (int s = tid; s < k; s += NT) {
        oidx[s] = (int32_t)out[s];
        if (osel) osel[s] = key_score(score_key(row[out[s]]));   // (-0 as +0)
    }
}

template <int NT, int NV, int NB, int WPE>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE))) void select_bins_kernel(SelectArgs a)
{
    __shared__ __attribute__((aligned(16))) BinsLds<NT, NV, NB> lds;
    const int tid = threadIdx.x;
    request_args(a);
    const int r = blockIdx.x;
    const RowView rw = row_view(a, r);
    if (rw.i >= a.Tq) return;
    const float *row = a.strip + (int64_t)r * a.ld;
    int32_t *oidx = a.idx + ((int64_t)rw.b * a.Tq + rw.i) * a.k_sel;
    float *osel = a.sel ? a.sel + ((int64_t)rw.b * a.Tq + rw.i) * a.k_sel : nullptr;
    if (rw.nv <= a.k_sel)
        select_all<NT>(row, rw.nv, a.k_sel, oidx, osel, tid);
    else
        bins_select<NT, NV, NB>(row, rw.nv, a.k_sel, oidx, osel, lds, tid, BlockSync());
}

// ---- scores and top-k together (short rows) ----------------------------------------------------------------------
// Rows that see at most kShortLen keys, of up to 32 bf16 heads: a workgroup scores two tokens of a sequence against all of their
// keys, its waves taking every fourth subtile of 32 keys straight from memory (they are in L2), into LDS, and then a wave
// selects a row by itself, in the bins form.  The scores are those of score_kernel, operation for operation.
// What bounds it: one launch and its latencies; 512 rows of up to 512 keys (4 heads of 64) took two launches of 6.6 and 5.6 us.
constexpr int kShortLen = 1024;
constexpr int kShortNB = 512;            // bins
constexpr int kShortRows = 2;            // of a workgroup (4: 512 rows of up to 512 keys 10.0 us, 9.8 with 2)

template <int DI>
__global__ __launch_bounds__(256, 1) void topk_short_kernel(ScoreArgs a, SelectArgs se)
{
    constexpr int KS = DI / 16, NV = kShortLen / 256, TT = kShortRows;
    static_assert(TT <= 4, "a wave per row");
    __shared__ __attribute__((aligned(16))) float score[TT][kShortLen];
    __shared__ __attribute__((aligned(16))) BinsLds<64, NV, kShortNB> lds[TT];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, half = lane >> 5;
    asm volatile("" ::"s"(a.q), "s"(a.k), "s"(a.w), "s"(a.q_pos0), "s"(a.Tq), "s"(a.Lk), "s"(a.H_I), "s"(a.i0), "s"(a.Ri), "s"(a.b0), "s"(se.k_sel), "s"(se.idx), "s"(se.sel));   // (together: see request_args)
    const int b = a.b0 + (int)blockIdx.y, t0 = a.i0 + TT * (int)blockIdx.x, t_end = min(a.i0 + a.Ri, a.Tq);
    auto visible = [&](int t) -> int {
        const int64_t n = a.q_pos0 + t + 1;
        return (int)(n < 0 ? 0 : (n > a.Lk ? a.Lk : n));
    };
    const int most = visible(min(t0 + TT, t_end) - 1);
    // (rows that select all they see need no scores)
    if (most > se.k_sel || se.sel) {
        bf16x8 qa[TT][KS];
        float wr[TT][16];
#pragma unroll
        for (int j = 0; j < TT; ++j) {
            const int64_t trow = (int64_t)b * a.Tq + min(t0 + j, t_end - 1);
            const bool hv = r32 < a.H_I;
            const unsigned short *src = (const unsigned short *)a.q + (trow * a.H_I + (hv ? r32 : 0)) * DI + 8 * half;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                u32x4 x = *(const u32x4 *)(src + 16 * ks);
                if (!hv) x = u32x4{0u, 0u, 0u, 0u};
                qa[j][ks] = __builtin_bit_cast(bf16x8, x);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int h = 8 * (i / 4) + 4 * half + (i % 4);
                const float w = a.w[trow * a.H_I + min(h, a.H_I - 1)];
                wr[j][i] = h < a.H_I ? w : 0.f;
            }
        }
        const unsigned short *kp = (const unsigned short *)a.k + (int64_t)b * a.Lk * DI + 8 * half;
        auto load = [&](int s0, bf16x8 (&kb)[KS]) {
            const unsigned short *src = kp + (int64_t)min(s0 + r32, a.Lk - 1) * DI;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) kb[ks] = *(const bf16x8 *)(src + 16 * ks);
        };
        bf16x8 kb[2][KS];
        load(32 * wave, kb[0]);
#pragma unroll 1
        for (int s0 = 32 * wave; s0 < most; s0 += 256) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {      // two subtiles a turn, each requested one ahead
                const int s = s0 + 128 * u;
                if (s >= most) break;
                load(min(s + 128, a.Lk - 1), kb[u ^ 1]);
#pragma unroll
                for (int j = 0; j < TT; ++j) {
                    f32x16 acc;
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qa[j][ks], kb[u][ks], acc, 0, 0, 0);
                    float x = 0.f;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int bits = __float_as_int(acc[i]);
                        x = fmaf(__int_as_float(bits > 0 ? bits : 0), wr[j][i], x);
                    }
                    const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
                    const float v = __uint_as_float(both[0]) + __uint_as_float(both[1]);
                    if (half == 0) score[j][s + r32] = v;
                }
            }
        }
    }
    __syncthreads();
    const int t = t0 + wave;
    if (wave >= TT || t >= t_end) return;
    const int nv = visible(t);
    int32_t *oidx = se.idx + ((int64_t)b * a.Tq + t) * se.k_sel;
    float *osel = se.sel ? se.sel + ((int64_t)b * a.Tq + t) * se.k_sel : nullptr;
    if (nv <= se.k_sel)
        select_all<64>(score[wave], nv, se.k_sel, oidx, osel, lane);
    else
        bins_select<64, NV, kShortNB>(score[wave], nv, se.k_sel, oidx, osel, lds[wave], lane, WaveSync());
}

// ---- parts form (few long rows) ---------------------------------------------------------------------------------
// A long row of a decode step has one workgroup in the forms above, and that one CU is what bounds it (a 200 000-key row,
// past the candidate form's bitmap, was streamed four times by it: 150 us).  Here a row is cut into parts with a
// workgroup each, and a second launch finishes it:
//   select_part_kernel    every part takes the candidate form's sample of the whole row (the same 4096 keys, so the same
//                         threshold T0), then sweeps its own keys and leaves its candidates in a list of its own in the
//                         workspace.  A part has every n-th block of 32 keys, so that the lists of a row whose best keys lie
//                         together are as long as those of any other
//   select_finish_kernel  one workgroup per row takes all lists into registers (16 slots a thread, requested before their
//                         lengths are known), finds the k-th largest candidate with one histogram and an exact ranking of
//                         its bin, and emits through a bitmap of the row in LDS
// A row that the candidates cannot decide (fewer than k of them, a list that overflowed, too many ties in the boundary
// bin) and a row too short for the sample take the generic radix select in the second launch.
// What bounds it: two launches, each a chain of memory latencies and barriers.  One row of 200 000 keys: 6.1 + 12.3 us with
// lists per wave that the second launch collected in LDS, 5.6 + 9.3 with this (of the second: lists 1.8, histogram and its scan
// 2.1, marking 1.9, ranking 0.5, bitmap scan 1.1, entries 1.1); with 512 threads of 32 slots 12.4, two waves per SIMD do not
// cover their LDS latencies.
constexpr int kPartThreads = 1024;
constexpr int kPartWaves = kPartThreads / 64;
constexpr int kPartMax = 64;             // parts of a row
constexpr int kPartBlock = 32;           // keys of a row that stay together: a line
// Where the form is the better one (scores and select of a call, 2 heads of 64, k = 2048; us, parts / the forms above): one row of 40 000
// keys 20.0 / 21.3, 66 000 20.7 / 27.0, 100 000 21.3 / 30.9, 131 072 22.9 / 36.6; 32 rows of 66 000 34.7 / 38.4, of 131 072 44.8 / 55.3;
// 64 rows 48.2 / 50.3 and 64.1 / 71.8, 96 rows 55.9 / 56.1 and 77 / 81, 128 rows 64.3 / 63.2 and 96 / 97, 200 rows 85 / 80 and 134 / 127.
// Past the candidate form's bitmap one row of 200 000 keys 24.9 / 148, 64 rows of 140 000 70 / 167, 200 rows 142 / 240, 500 rows 316 / 644.
constexpr int kPartFrom = 65536;         // rows have more keys than this ...
constexpr int kPartRows = 64;            // ... and are at most this many: more of them fill the chip by themselves,
constexpr int kPartRowsLong = 512;       // which holds for longer where the alternative streams the row four times
constexpr int kFinishThreads = 1024;
constexpr int kFinishSlots = 16384;      // list entries of a row, its parts' lists in equal shares of them
constexpr int kFinishCap = 12288;        // candidates of a row that are likely to find room in them: the lists' lengths and the threshold scatter
constexpr int kFinishWindow = 1 << 20;   // keys that the bitmap covers at a time

// per row: T0, then the lists' lengths
constexpr int kPartHead = 1 + kPartMax;
// Entries of a part's list, in lines of 32.  (Shares of a power of two, one wave's vector of them or more, left 7 rows, of 36 parts, room
// for 9216 entries: every second row of 500 000 keys overflowed them and took the radix select behind both launches.)
constexpr int kListLine = 32;
inline int part_slots(int n_parts) { return kFinishSlots / kListLine / n_parts * kListLine; }

// rows the sample can speak for
__device__ __forceinline__ bool part_row(const SelectArgs &a, int nv) { return nv >= kCandMinLen && nv >= 4 * a.k_sel; }

__global__ __launch_bounds__(kPartThreads) void select_part_kernel(SelectArgs a, PartArgs pa)
{
    constexpr int NT = kPartThreads, NW = kPartWaves;
    request_args(a);
    __shared__ __attribute__((aligned(16))) uint32_t hist[kBins1];
    __shared__ uint32_t wsum[2 * NW], bc[4], red[2 * NW], n_list;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int part = blockIdx.x, r = blockIdx.y;
    const RowView rv = row_view(a, r);
    if (rv.i >= a.Tq || !part_row(a, rv.nv)) return;
    const int nv = rv.nv;
    const float *row = a.strip + (int64_t)r * a.ld;
    // eight lanes to a block; blocks part, part + n_parts, ...
    constexpr int kGroup = 4;
    f32x4 ga[kGroup];
    auto place = [&](int i0, int j) { return ((i0 + (j * NW + wave) * 8 + (lane >> 3)) * pa.n_parts + part) * kPartBlock + 4 * (lane & 7); };
    auto load_group = [&](int i0) {
#pragma unroll
        for (int j = 0; j < kGroup; ++j) {
            const int p = place(i0, j);
            ga[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (p < nv) ga[j] = *(const f32x4 *)(row + p);     // may run past nv inside the row's padding; masked below
        }
    };
    const int blk = tid >> 5;                                  // 32 blocks of 128 keys spread over the row
    const f32x4 sv = *(const f32x4 *)(row + (int)(((int64_t)blk * nv / 32) & ~(int64_t)3) + (tid & 31) * 4);
    load_group(0);
    static_assert(kCandSample == 4 * NT, "one sample vector per thread");
    for (int e = tid; e < kBins1; e += NT) hist[e] = 0;
    if (tid == 0) n_list = 0;
    uint32_t skey[4], kmx = 0u, kmn = 0xFFFFFFFFu;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        skey[e] = score_key(sv[e]);
        kmx = max(kmx, skey[e]);
        kmn = min(kmn, skey[e]);
    }
    kmx = wave_max_dpp(kmx);
    kmn = wave_max_dpp(~kmn);
    if (lane == 0) {
        red[wave] = kmn;
        red[NW + wave] = kmx;
    }
    __syncthreads();
    const uint32_t smin = ~wave_max_dpp(red[lane % NW]);
    const uint32_t smax = wave_max_dpp(red[NW + lane % NW]);
    const uint32_t srange = smax - smin;
    const int sbits = srange ? 32 - __clz((int)srange) : 0;
    const int ssh = sbits > 12 ? sbits - 12 : 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) atomicAdd(&hist[(skey[e] - smin) >> ssh], 1u);
    __syncthreads();
    find_digit<NT, kBins1 / NT>(hist, cand_rank(a.k_sel, nv, false), wsum, bc, tid, lane, wave);
    const uint32_t T0 = smin + (bc[0] << ssh);
    const float T0f = key_score(T0);

    const uint32_t slots = (uint32_t)pa.slots;
    uint32_t *keys = pa.lists + (size_t)r * 2 * kFinishSlots + part * slots, *pos = keys + kFinishSlots;
    const int n_blk = ((nv + kPartBlock - 1) / kPartBlock - part + pa.n_parts - 1) / pa.n_parts;     // of this part
    for (int i0 = 0; i0 < n_blk; i0 += NW * 8 * kGroup) {      // workgroup-uniform
        if (i0) load_group(i0);
        uint32_t m = 0;
#pragma unroll
        for (int j = 0; j < kGroup; ++j) {
            const int p = place(i0, j);
#pragma unroll
            for (int e = 0; e < 4; ++e) m |= (uint32_t)((int)(p + e < nv) & (int)(ga[j][e] >= T0f)) << (4 * j + e);
        }
        const uint32_t n_t = (uint32_t)__popc(m), incl = wave_incl_scan(n_t);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        if (total == 0u) continue;                             // wave-uniform
        uint32_t first = 0;
        if (lane == 0) first = atomicAdd(&n_list, total);
        uint32_t off = (uint32_t)__builtin_amdgcn_readfirstlane((int)first) + incl - n_t;
#pragma unroll
        for (int j = 0; j < kGroup; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((m >> (4 * j + e)) & 1u) {
                    if (off < slots) {
                        keys[off] = max(score_key(ga[j][e]), T0);
                        pos[off] = (uint32_t)(place(i0, j) + e);
                    }
                    ++off;
                }
    }
    __syncthreads();
    uint32_t *head = pa.heads + (size_t)r * pa.head_words;
    if (tid == 0) head[1 + part] = n_list;
    if (part == 0 && tid == 0) head[0] = T0;
}

constexpr int finish_bitmap_words(int row_len) { return ((row_len < kFinishWindow ? row_len : kFinishWindow) + 127) / 128 * 4; }

__global__ __launch_bounds__(kFinishThreads) void select_finish_kernel(SelectArgs a, PartArgs pa)
{
    constexpr int NT = kFinishThreads, NW = NT / 64, NV = kFinishSlots / NT / 4;
    extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
    uint32_t *hist = smem;                     // [kBins1]  (the generic form's layout starts the same way)
    uint32_t *wsum = hist + kBins1;            // [2 NW]
    uint32_t *bc = wsum + 2 * NW;              // [4]
    __shared__ uint32_t misc[2], red[NW];      // misc: 0 members listed
    uint32_t *bl_key = bc + 4, *bl_pos = bl_key + kBoundaryCap;    // the boundary bin's members
    uint32_t *bitmap = bl_pos + kBoundaryCap;  // [finish_bitmap_words] of the row
    uint16_t *ahead_of = (uint16_t *)hist;     // [kFinishWindow / 128] selected entries ahead of every four words (the histogram is read by then)
    static_assert(kFinishWindow / 128 <= 2 * kBins1 && (kBins1 + 2 * NW + 4) % 4 == 0, "they share its space");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = blockIdx.x;
    request_args(a);
    const RowView rv = row_view(a, r);
    if (rv.i >= a.Tq) return;
    auto finish = [&]() -> bool {              // false: the generic form takes the row (one call site, see the candidate form)
        if (!part_row(a, rv.nv)) return false;
        const uint32_t *head = pa.heads + (size_t)r * pa.head_words;
        const uint32_t *keys = pa.lists + (size_t)r * 2 * kFinishSlots;
        const float *row = a.strip + (int64_t)r * a.ld;
        // A vector's entry: all lists' first lines, then their second ones: empty slots lie together, and waves of them have nothing to
        // do (list behind list 0.8 us longer for 48 lists of 117 entries).
        auto list_of = [&](int j, int &first) {
            const int line = (j * NT + tid) / (kListLine / 4);
            const int of_list = pa.n_parts == 1 ? line : (int)__umulhi((unsigned)line, pa.inv_parts);
            first = of_list * kListLine + 4 * (tid % (kListLine / 4));
            return line - of_list * pa.n_parts;
        };
        u32x4 v[NV], at[NV];
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            int first;
            const int list = list_of(j, first);
            v[j] = u32x4{0u, 0u, 0u, 0u};
            if (first < pa.slots) v[j] = *(const u32x4 *)(keys + list * pa.slots + first);
        }
        const uint32_t T0 = head[0];
        const uint32_t n_lane = lane < pa.n_parts ? head[1 + lane] : 0u;
        const uint32_t n_cand = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(n_lane), 63), k = (uint32_t)a.k_sel;
        if (n_cand < k || __ballot(n_lane > (uint32_t)pa.slots) != 0ull) return false;   // workgroup-uniform
        // slots behind a list's end: key 0, below every candidate (T0 is above the smallest sampled key or a bin's edge)
        uint32_t mx = 0;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            int first;
            const int list = list_of(j, first);
            const int left = first < pa.slots ? (int)__shfl(n_lane, list) - first : 0;
            at[j] = u32x4{0u, 0u, 0u, 0u};
            if (left > 0) at[j] = *(const u32x4 *)(keys + kFinishSlots + list * pa.slots + first);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[j][e] = e < left ? v[j][e] : 0u;
                mx = max(mx, v[j][e]);
            }
        }
        for (int e = tid; e < kBins1; e += NT) hist[e] = 0;
        const int words = finish_bitmap_words(rv.nv);
        for (int e = 4 * tid; e < words; e += 4 * NT) *(u32x4 *)(bitmap + e) = u32x4{0u, 0u, 0u, 0u};
        if (tid == 0) misc[0] = 0;
        mx = wave_max_dpp(mx);
        if (lane == 0) red[wave] = mx;
        __syncthreads();
        const uint32_t range = wave_max_dpp(red[lane % NW]) - T0;
        const int nbits = range ? 32 - __clz((int)range) : 0;
        const int sh = nbits > 12 ? nbits - 12 : 0;
        auto each = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                asm volatile("" : "+v"(v[j]));                 // (bins and tests are not kept from one sweep to the next)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (v[j][e] != 0u) f(v[j][e], at[j][e]);
            }
        };
        each([&](uint32_t x, uint32_t) { atomicAdd(&hist[(x - T0) >> sh], 1u); });
        __syncthreads();
        find_digit<NT, kBins1 / NT>(hist, k, wsum, bc, tid, lane, wave);
        const uint32_t bstar = bc[0], need = bc[1], n_b = bc[2];
        const bool ranked = need < n_b;        // the boundary bin is cut: rank its members exactly
        if (ranked && n_b > (uint32_t)kBoundaryCap) {
            __syncthreads();
            return false;
        }
        // Selected entries of a window set their bits (the first window's, of all rows but the longest: together with the listing)
        auto in_window = [&](uint32_t p, uint32_t w0) { return p - w0 < (uint32_t)kFinishWindow; };
        auto set = [&](uint32_t p, uint32_t w0) { atomicOr(&bitmap[(p - w0) >> 5], 1u << (p & 31u)); };
        const uint32_t least = bstar + (ranked ? 1u : 0u);     // bins from here on are selected whole
        each([&](uint32_t x, uint32_t p) {
            const uint32_t bin = (x - T0) >> sh;
            if (bin >= least) {
                if (in_window(p, 0u)) set(p, 0u);
            } else if (bin == bstar) {
                const uint32_t m = atomicAdd(&misc[0], 1u);
                bl_key[m] = x;
                bl_pos[m] = p;
            }
        });
        __syncthreads();
        bool in = false;                       // this thread's member
        if (ranked) {
            static_assert(kBoundaryCap <= NT, "a member per thread");
            if ((uint32_t)tid < n_b) {
                const uint32_t km = bl_key[tid], pm = bl_pos[tid];
                uint32_t ahead = 0;            // members that beat this one: larger key, or equal key at a lower position
#pragma unroll 4
                for (uint32_t x = 0; x < n_b; ++x) {   // (no branch: positions asked for after their keys took a row with 667 ties from 52 to 98 us)
                    const uint32_t kx = bl_key[x], px = bl_pos[x];
                    ahead += (uint32_t)(kx > km) | ((uint32_t)(kx == km) & (uint32_t)(px < pm));
                }
                in = ahead < need;
                if (in && in_window(pm, 0u)) set(pm, 0u);
            }
            __syncthreads();
        }
        int32_t *oidx = a.idx + ((int64_t)rv.b * a.Tq + rv.i) * a.k_sel;
        float *osel = a.sel ? a.sel + ((int64_t)rv.b * a.Tq + rv.i) * a.k_sel : nullptr;
        uint32_t taken = 0;                    // entries of the windows before
        for (uint32_t w0 = 0; w0 < (uint32_t)rv.nv; w0 += kFinishWindow) {
            if (w0) {
                __syncthreads();
                for (int e = 4 * tid; e < words; e += 4 * NT) *(u32x4 *)(bitmap + e) = u32x4{0u, 0u, 0u, 0u};
                __syncthreads();
                each([&](uint32_t x, uint32_t p) {
                    if ((x - T0) >> sh >= least && in_window(p, w0)) set(p, w0);
                });
                if (in && in_window(bl_pos[tid], w0)) set(bl_pos[tid], w0);
                __syncthreads();
            }
            // a thread's words follow each other
            const int groups = words / 4, mine = (groups + NT - 1) / NT, g0 = min(tid * mine, groups), g1 = min(g0 + mine, groups);
            uint32_t n = 0;
            for (int q = g0; q < g1; ++q) {
                const u32x4 w = *(const u32x4 *)(bitmap + 4 * q);
                n += (uint32_t)(__popc(w[0]) + __popc(w[1]) + __popc(w[2]) + __popc(w[3]));
            }
            uint32_t before = wave_incl_scan(n);
            if (lane == 63) wsum[wave] = before;
            __syncthreads();
            before += taken - n;
#pragma unroll
            for (int wv = 0; wv < NW; ++wv) {
                if (wv < wave) before += wsum[wv];
                taken += wsum[wv];
            }
            for (int q = g0; q < g1; ++q) {
                const u32x4 w = *(const u32x4 *)(bitmap + 4 * q);
                ahead_of[q] = (uint16_t)before;    // (k_sel is at most 2048)
                before += (uint32_t)(__popc(w[0]) + __popc(w[1]) + __popc(w[2]) + __popc(w[3]));
            }
            __syncthreads();
            for (int q = tid; q < groups; q += NT) {           // (neighbouring groups in neighbouring threads: entries that lie together)
                const u32x4 w = *(const u32x4 *)(bitmap + 4 * q);
                uint32_t slot = ahead_of[q];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    uint64_t m = w[2 * u] | (uint64_t)w[2 * u + 1] << 32;
                    while (m) {
                        const uint32_t p = w0 + 128 * (uint32_t)q + 64 * u + (uint32_t)__builtin_ctzll(m);
                        m &= m - 1;
                        if (slot < k) {        // always true for a consistent select
                            oidx[slot] = (int32_t)p;
                            if (osel) osel[slot] = key_score(score_key(row[p]));   // (-0 as +0)
                        }
                        ++slot;
                    }
                }
            }
        }
        return true;
    };
    if (!finish()) {
        __syncthreads();
        select_row_generic<NT>(a, smem);
    }
}
constexpr size_t finish_lds_bytes(int row_len) { return (size_t)(kBins1 + 2 * (kFinishThreads / 64) + 4 + 2 * kBoundaryCap + finish_bitmap_words(row_len)) * 4; }
static_assert(finish_lds_bytes(kFinishWindow) <= 159 * 1024, "fits the LDS, static arrays beside it");

size_t select_lds_bytes(int cache_elems)
{
    return (size_t)(kBins1 + 2 * 16 + 4 + cache_elems) * sizeof(uint32_t);
}

} // namespace

// A row of this length leaves about 2 k + 1 / 128 of its keys as candidates (the rank that select_part_kernel takes from the
// sample).  Where the lists (some kFinishSlots together at any number of parts) are unlikely to hold that many, the row would go to the radix select behind two launches for
// nothing (k = 2048: from 1.05 M keys; 1.1 M keys 775 us without, 780 with them).  The sample scatters by some 14 %: a row
// shortly below the line may still get there, and gains tenfold where it does not (1 M keys 652 / 45 us).
bool select_parts_fit(int k, int row_len) { return (int64_t)2 * k + row_len / 128 <= kFinishCap; }

// Parts of a row when n_rows rows of up to max_row_len keys are selected together: enough for one workgroup per CU,
// of at least 4096 keys (a vector a thread); 0 = the row-per-workgroup forms take the rows.
int select_parts(int n_rows, int max_row_len)
{
    if (n_rows < 1 || max_row_len <= kPartFrom || n_rows > (max_row_len > kCandMaxLen ? kPartRowsLong : kPartRows)) return 0;
    int p = 256 / n_rows;
    const int most = max_row_len / (256 * kPartWaves);
    p = p > most ? most : p;
    return p < 1 ? 1 : (p > kPartMax ? kPartMax : p);
}

// Keys of a row that the radix select keeps in the second launch's LDS, of which a workgroup has its CU's anyway: for sequences that are too
// short for the sample beside long ones (streamed, 31 of 8191 keys beside one of 100 000 took the two launches 22.1 us, cached 20.0).
int select_parts_cache(int ragged) { return ragged ? 24576 : 0; }

// Room in the list of each of them.
int select_parts_slots(int n_rows, int max_row_len)
{
    const int p = select_parts(n_rows, max_row_len);
    return p == 0 ? 0 : part_slots(p);
}

// The candidate forms' sample (rank of the threshold in it, stretches) and the entries of their list, for launches of few or of many rows.
int select_cand_rank(int k, int row_len, int many) { return (int)cand_rank(k, row_len, many != 0); }
int select_cand_runs(int many) { return kCandRuns; }
int select_cand_list(int many) { return many ? kCandManyCap : kCandCap; }

size_t select_parts_bytes(int n_rows, int max_row_len)
{
    return select_parts(n_rows, max_row_len) == 0 ? 0 : (size_t)n_rows * (((kPartHead + 63) / 64 * 64) + 2 * kFinishSlots) * 4;
}

hipError_t launch_select_parts(const SelectArgs &a_in, int n_rows, int max_row_len, void *ws, hipStream_t st)
{
    SelectArgs a = a_in;
    a.cache_elems = select_parts_cache(a.seq_lens != nullptr);
    PartArgs pa;
    pa.n_parts = select_parts(n_rows, max_row_len);
    pa.slots = part_slots(pa.n_parts);
    pa.inv_parts = (uint32_t)((((uint64_t)1 << 32) + pa.n_parts - 1) / pa.n_parts);
    pa.head_words = (kPartHead + 63) / 64 * 64;
    pa.heads = (uint32_t *)ws;
    pa.lists = pa.heads + (size_t)n_rows * pa.head_words;
    const size_t lds = std::max(finish_lds_bytes(max_row_len), select_lds_bytes(a.cache_elems));
    static hipError_t attr = hipFuncSetAttribute((const void *)select_finish_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)finish_lds_bytes(kFinishWindow));
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(select_part_kernel, dim3((unsigned)pa.n_parts, (unsigned)n_rows), dim3(kPartThreads), 0, st, a, pa);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(select_finish_kernel, dim3((unsigned)n_rows), dim3(kFinishThreads), lds, st, a, pa);
    return hipGetLastError();
}

namespace {
template <int NT, int NV, int NB, int WPE>
hipError_t launch_bins(const SelectArgs &a, int n_rows, int max_row_len, hipStream_t st)
{
    if (max_row_len > NT * NV * 4) return hipErrorInvalidValue;
    hipLaunchKernelGGL((select_bins_kernel<NT, NV, NB, WPE>), dim3((unsigned)n_rows), dim3(NT), 0, st, a);
    return hipGetLastError();
}
} // namespace

hipError_t launch_select(const SelectArgs &a_in, int n_rows, int max_row_len, hipStream_t st)
{
    if (n_rows <= 0) return hipSuccess;
    SelectArgs a = a_in;
    a.cache_elems = 0;
    // The bins form, in the smallest workgroup that holds the row: its barriers and its start cost less, and more rows are
    // in flight per CU.  Rows of 16384 keys take 512 threads where there are few of them (1 row of 10007 keys: 7.8 us,
    // 10.5 with 256; 4096 rows of 14336 on average 73 and 67).
    if (max_row_len <= 1024) return launch_bins<128, 2, 512, 8>(a, n_rows, max_row_len, st);
    if (max_row_len <= 2048) return launch_bins<128, 4, 512, 8>(a, n_rows, max_row_len, st);
    if (max_row_len <= 4096) return launch_bins<256, 4, 1024, 8>(a, n_rows, max_row_len, st);
    if (max_row_len <= 8192) return launch_bins<256, 8, 1024, 7>(a, n_rows, max_row_len, st);
    if (max_row_len <= 16384 && n_rows > 512) return launch_bins<256, 16, 2048, 4>(a, n_rows, max_row_len, st);
    if (max_row_len <= 16384) return launch_bins<512, 8, 2048, 6>(a, n_rows, max_row_len, st);
    if (max_row_len <= kBinsLen) return launch_bins<512, 16, 4096, 4>(a, n_rows, max_row_len, st);
    static_assert(4 * IC_MAX_K <= kBinsLen, "a row of the candidate form is four times as long as its selection");
    if (max_row_len <= kCandMaxLen) {
        // one read of the row, a sampled threshold and a candidate list (falls back row by row)
        constexpr int lds = cand_lds_words(1024, kCandMaxLen, kCandCap) * (int)sizeof(uint32_t);
        constexpr int lds_many = cand_lds_words(512, kCandMaxLen, kCandManyCap) * (int)sizeof(uint32_t);
        static_assert(2 * lds_many <= 160 * 1024, "two workgroups per CU");
        static hipError_t attr = hipFuncSetAttribute((const void *)select_cand_kernel<1024, kCandMaxLen, kCandCap, false>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        static hipError_t attr_many = hipFuncSetAttribute((const void *)select_cand_kernel<512, kCandMaxLen, kCandManyCap, true>,
                                                          hipFuncAttributeMaxDynamicSharedMemorySize, lds_many);
        if (attr != hipSuccess) return attr;
        if (attr_many != hipSuccess) return attr_many;
        if (n_rows > 256)
            hipLaunchKernelGGL((select_cand_kernel<512, kCandMaxLen, kCandManyCap, true>), dim3((unsigned)n_rows), dim3(512), lds_many, st, a);
        else
            hipLaunchKernelGGL((select_cand_kernel<1024, kCandMaxLen, kCandCap, false>), dim3((unsigned)n_rows), dim3(1024), lds, st, a);
        return hipGetLastError();
    }
    // longer rows, too many for the parts form, are streamed on every sweep
    hipLaunchKernelGGL((select_kernel<1024>), dim3((unsigned)n_rows), dim3(1024), select_lds_bytes(0), st, a);
    return hipGetLastError();
}

// Rows that topk_short_kernel takes: few enough that the launch it saves counts for more than what score_kernel gains by sharing
// its keys among more rows.  us, two launches / one (the caller's own 9.7 us bound the shorter ones): 4 heads of 64, 512 rows of
// up to 512 keys 12.5 / 9.8, 3 x 512 15.2 / 12.5, 1000 of 1000 14.0 / 12.7, 2 x 1000 18.5 / 19.4; 32 heads of 128, 512 rows of 512
// 13.1 / 11.1, 64 of 900 12.3 / 15.2.  With few rows two launches take 8 to 8.5 us at any of these lengths (up to four rows a
// sequence: the streaming forms of the scores, which spread the keys over the chip) or 10 (more), while here a workgroup goes
// through a row's keys one subtile after another.  One row, 4 heads of 64: 512 keys 7.6 / 7.4, 768 8.2 / 8.7, 1024 7.9 / 9.9; 32 heads:
// 256 7.4 / 7.1, 512 7.5 / 8.1, 1024 8.1 / 10.5; 4 heads of 128: 256 8.1 / 7.6, 320 8.0 / 8.4; 32 heads: 128 8.4 / 8.3, 256 8.2 / 8.7,
// 512 8.2 / 10.7; 64 rows of 512 keys, 32 heads 8.2 / 8.8.  Past 128 keys for each CU the streaming forms take a second round: 64 rows, 4
// heads of 64: 640 9.6 / 8.9, 768 9.6 / 9.2, 1024 9.4 / 10.4, 96 even.  16 rows of one sequence, 32 heads of 64: 768 10.3 / 9.7, 1024 10.2 / 10.9.
bool topk_short(const ScoreArgs &a, int dtype, int d_I, int n_rows, int64_t max_vis)
{
    if (dtype != IC_BF16 || a.H_I > 32 || a.pv.seq_lens || a.pv.page_table) return false;
    if (d_I != 64 && d_I != 128) return false;
    int64_t most = d_I == 64 ? kShortLen : kShortLen / 2;
    if (n_rows < 96 && a.Ri <= 4 && n_rows * max_vis <= 256 * 128) most = a.H_I > 8 ? most / 4 : most / 2;
    else if (n_rows < 96 && d_I == 64) most = most * 3 / 4;
    return max_vis <= most && n_rows * max_vis <= (d_I == 64 ? 1 << 20 : 1 << 18);
}

hipError_t launch_topk_short(const ScoreArgs &a, const SelectArgs &se, int d_I, int Bc, hipStream_t st)
{
    const dim3 grid((unsigned)((a.Ri + kShortRows - 1) / kShortRows), (unsigned)Bc);
    if (d_I == 64)
        hipLaunchKernelGGL(topk_short_kernel<64>, grid, dim3(256), 0, st, a, se);
    else
        hipLaunchKernelGGL(topk_short_kernel<128>, grid, dim3(256), 0, st, a, se);
    return hipGetLastError();
}

} // namespace ic
