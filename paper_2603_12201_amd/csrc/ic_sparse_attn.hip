// Sparse MQA core attention over the selected KV rows (paper Sec. 2.1: the main attention is
// computed only over the top-k subset; MLA form, one shared KV row per position).
//
// MLA rows whose values are their first features (576 / 512) take one of three forms further down: the stream form, one
// workgroup per CU that walks a chain of queries; the row-slab form, one (query, split) per workgroup where there are fewer
// queries than CUs (decode) and one query where their selections are short; the dense form where a row selects all it sees.  Every other supported layout takes the
// small-tile form described here.
//
// Small-tile form: one workgroup (4 waves) per query token and key-slot split; two workgroups
// fit a CU (75 KB of LDS, <= 256 VGPRs each) so that one computes while the other waits for its
// gather.  Tiles of 32 selected rows are gathered with 16-byte coalesced loads (each row is
// contiguous) into a double-buffered LDS tile, row-major.  A wave owns 16 of the 32 heads and half
// of the value columns, and runs its own online softmax over every row of the tile:
//   S^T = K Q^T   v_mfma_f32_16x16x32_bf16, A = tile rows (16-byte LDS reads), B = Q (registers)
//   P   = exp2(S^T * scale*log2e - m)   in the result layout: a lane owns one head, 8 keys
//   O  += P V     same MFMA; P is already an A operand (its contraction slots are whatever keys
//                 the lane holds), and V comes out of the SAME row-major tile through the LDS
//                 transpose read ds_read_b64_tr_b16, which hands a lane one value column of four
//                 consecutive tile rows.  No transposed copy of V is ever made.
// The two waves of a head group compute the same S^T (cheap next to the gather) and therefore
// the same softmax statistics, so no exchange between waves is ever needed.
//
// Splits (both forms): a split stores its own normalised output in bf16 together with its
// reference maximum and row sum; attn_merge_kernel weighs the splits by their share of the total
// row sum.
#include "ic_common.hpp"
#include <algorithm>
#include <cstring>
#include <type_traits>

namespace ic {

namespace {

constexpr int kTile = 32;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// layer of query gq of a launch (several layers share one where they have a few thousand queries together: 32 bits do; the
// division in 64 bits costs every workgroup about 1 us before its first load)
__device__ __forceinline__ int layer_of(const AttnArgs &a, int64_t gq)
{
    return a.n_layers == 1 ? 0 : (int)((unsigned)gq / (unsigned)(a.B * a.Tq));
}

// Tile staging.  A thread owns tile row tid / 8 and the 16-byte chunks (tid % 8) + 8 r of that
// row: eight neighbouring lanes read one full 128-byte line, and no index needs a division.
template <int ROW_F, int LPT, bool PG>
__device__ __forceinline__ void attn_gload(u32x4 (&pre)[LPT], const unsigned short *kv_seq, const int32_t *ti,
                                           int row_elems, int tid, const PagedView &pv, int b)
{
    constexpr int CPR = ROW_F / 8;
    const int row = tid >> 3, c0 = tid & 7;
    const int32_t v = ti[row];                             // empty slots read row 0 (never a page-table entry)
    const int64_t prow = v < 0 ? 0 : (PG && pv.page_table ? paged_row(pv, b, v) : (int64_t)v);
    const unsigned short *src = kv_seq + prow * row_elems + c0 * 8;
#pragma unroll
    for (int r = 0; r < LPT; ++r)
        if (c0 + 8 * r < CPR) pre[r] = *(const u32x4 *)(src + 64 * r);
}

template <int ROW_F, int LPT, int ROWB>
__device__ __forceinline__ void attn_lstore(const u32x4 (&pre)[LPT], unsigned char *tile, int tid)
{
    constexpr int CPR = ROW_F / 8;
    const int row = tid >> 3, c0 = tid & 7;
    unsigned char *dst = tile + row * ROWB + c0 * 16;
#pragma unroll
    for (int r = 0; r < LPT; ++r)
        if (c0 + 8 * r < CPR) *(u32x4 *)(dst + 128 * r) = pre[r];
}

// PG: the KV cache may be ragged and / or paged (a.pv); false compiles the dense layout only.
template <int D_QK, int D_V, int ROW_F, bool PG>
__global__ __launch_bounds__(256, 2) void attn_kernel(AttnArgs a)
{
    constexpr int ROWB = ROW_F * 2 + 16;                  // LDS row stride in bytes
    constexpr int CPR = ROW_F / 8;                        // 16-byte chunks staged per row
    constexpr int LPT = (CPR + 7) / 8;                    // chunk loads per thread per tile (one row per 8 lanes)
    static_assert(kTile * 8 == 256, "256 threads cover the tile rows, 8 lanes per row");
    constexpr int KSTEPS = D_QK / 32;
    constexpr int DVW = D_V / 2;                          // value columns per wave
    constexpr int NB = DVW / 16;
    constexpr int TILEB = kTile * ROWB;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char *tile0 = smem;                          // [2][kTile][ROWB]
    int32_t *tidx = (int32_t *)(smem + 2 * TILEB);        // [3][kTile] validated row ids of a tile

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, g = lane >> 4;
    const int mh = wave & 1, vh = wave >> 1;
    asm volatile("" ::"s"(a.n_layers), "s"(a.B), "s"(a.Tq), "s"(a.Lk), "s"(a.H_q), "s"(a.row_elems), "s"(a.k_sel), "s"(a.split_len), "s"(a.idx));   // (together: see attn_slab_kernel)
    const int64_t gq = blockIdx.x;                        // query of the launch: flattened (layer, b, t)
    const int layer = layer_of(a, gq);
    const int64_t qrow = gq - (int64_t)layer * a.B * a.Tq;
    const int b = (int)((unsigned)qrow / (unsigned)a.Tq);
    const int sp = blockIdx.y;
    const int slot0 = sp * a.split_len;
    const int slot1 = min(slot0 + a.split_len, a.k_sel);
    const int ntiles = (slot1 - slot0 + kTile - 1) / kTile;

    const int32_t *idx_row = a.idx + qrow * a.k_sel;
    const unsigned short *kv_seq = (const unsigned short *)a.KVs[layer] + (PG && a.pv.page_table ? 0 : (int64_t)b * a.Lk * a.row_elems);
    const int Lk_b = PG && a.pv.seq_lens ? min(a.pv.seq_lens[b], a.Lk) : a.Lk;     // ragged cache: rows of this sequence

    auto fetch_idx = [&](int it) -> int32_t {             // threads 0..31: validated row id of a slot
        const int slot = slot0 + it * kTile + tid;
        int32_t v = -1;
        if (it < ntiles && slot < slot1) v = idx_row[slot];
        return (v >= 0 && v < Lk_b) ? v : -1;
    };

    // ---- Q as the B operand of S^T = K Q^T: lane (head l16, k-group g) ----
    const int head = 16 * mh + l16;
    const bool head_ok = head < a.H_q;
    const bool wave_ok = 16 * mh < a.H_q;                 // wave-uniform: any valid head at all
    bf16x8 qreg[KSTEPS];
    {
        const unsigned short *qp = (const unsigned short *)a.Qs[layer] + (qrow * a.H_q + (head_ok ? head : 0)) * D_QK + 8 * g;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            u32x4 raw = u32x4{0u, 0u, 0u, 0u};
            if (head_ok) raw = *(const u32x4 *)(qp + 32 * ks);
            qreg[ks] = __builtin_bit_cast(bf16x8, raw);
        }
    }

    // ---- prologue ----
    if (tid < kTile) {
        tidx[0 * kTile + tid] = fetch_idx(0);
        tidx[1 * kTile + tid] = fetch_idx(1);
    }
    __syncthreads();
    u32x4 pre[LPT];
    if (ntiles > 0) {
        attn_gload<ROW_F, LPT, PG>(pre, kv_seq, tidx, a.row_elems, tid, a.pv, b);
        attn_lstore<ROW_F, LPT, ROWB>(pre, tile0, tid);
    }
    __syncthreads();

    f32x4 oacc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) oacc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY;                              // running max (log2 units) of head l16
    float l_run = 0.f;                                    // this lane's share of the running sum

#pragma unroll 1
    for (int it = 0; it < ntiles; ++it) {
        const int buf = it & 1;
        int32_t nxt_idx = -1;
        if (tid < kTile) nxt_idx = fetch_idx(it + 2);
        if (it + 1 < ntiles) attn_gload<ROW_F, LPT, PG>(pre, kv_seq, tidx + ((it + 1) % 3) * kTile, a.row_elems, tid, a.pv, b);

        if (wave_ok) {
            const unsigned char *tb = tile0 + buf * TILEB;
            // S^T for the tile's 32 rows (two 16-row blocks) x this wave's 16 heads
            f32x4 sacc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) {
#pragma unroll
                for (int blk = 0; blk < 2; ++blk) {
                    const bf16x8 ka = *(const bf16x8 *)(tb + (16 * blk + l16) * ROWB + (32 * ks + 8 * g) * 2);
                    sacc[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qreg[ks], sacc[blk], 0, 0, 0);
                }
            }
            // validity of the lane's 8 key slots: rows 16blk + 4g + i
            const int32_t *ti = tidx + (it % 3) * kTile;
            float z[8];
            bool ok[8];
            float mx = -INFINITY;
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                const i32x4 rv = *(const i32x4 *)(ti + 16 * blk + 4 * g);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    ok[4 * blk + i] = rv[i] >= 0;
                    z[4 * blk + i] = sacc[blk][i] * a.scale_log2e;
                    if (ok[4 * blk + i]) mx = fmaxf(mx, z[4 * blk + i]);
                }
            }
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m_run, mx);
            const float alpha = (m_new == -INFINITY) ? 1.f : fast_exp2(m_run - m_new);
            float psum = 0.f;
            float pv[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                pv[j] = ok[j] ? fast_exp2(z[j] - m_new) : 0.f;
                psum += pv[j];
            }
            l_run = l_run * alpha + psum;
            m_run = m_new;
            // rescale O only when some head's max moved (wave-uniform test)
            if (__ballot(alpha != 1.f) != 0ull) {
                float ar[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) ar[i] = __shfl(alpha, 4 * g + i);   // alpha of head row 4g+i
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) oacc[nb][i] *= ar[i];
            }
            bf16x8 pa;
#pragma unroll
            for (int j = 0; j < 8; ++j) pa[j] = (__bf16)pv[j];
            // O += P V : V columns of 4 consecutive tile rows through the LDS transpose read
            const unsigned char *vb0 = tb + (4 * g + (l16 >> 2)) * ROWB + (a.v_off + DVW * vh + 4 * (l16 & 3)) * 2;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4 *)(vb0 + nb * 32));
                const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4 *)(vb0 + 16 * ROWB + nb * 32));
                typedef __attribute__((ext_vector_type(8))) short s16x8;
                const s16x8 vv = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                oacc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa, __builtin_bit_cast(bf16x8, vv), oacc[nb], 0, 0, 0);
            }
        }

        if (it + 1 < ntiles) attn_lstore<ROW_F, LPT, ROWB>(pre, tile0 + (buf ^ 1) * TILEB, tid);
        if (tid < kTile) tidx[((it + 2) % 3) * kTile + tid] = nxt_idx;
        __syncthreads();
    }
    if (!wave_ok) return;

    // ---- epilogue: this wave's heads x its value columns ----
    float l_tot = l_run + __shfl_xor(l_run, 16);
    l_tot += __shfl_xor(l_tot, 32);                       // every lane: full sum of head l16
    const bool split = a.n_splits > 1;
    if (vh == 0 && g == 0 && head_ok) {
        if (split) {
            float *ml = a.part_ml + ((gq * a.n_splits + sp) * a.H_q + head) * 2;
            ml[0] = m_run;
            ml[1] = l_tot;
        } else if (a.lse) {
            a.lse[qrow * a.H_q + head] =
                (l_tot > 0.f) ? (m_run + __builtin_log2f(l_tot)) * 0.6931471805599453f : -INFINITY;
        }
    }
    // a split stores its own normalised output; the merge weighs the splits by their share of the total row sum
    auto put = [&](auto *o) __attribute__((always_inline)) {
        typedef std::remove_pointer_t<decltype(o)> T;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int hr = 4 * g + i;                     // O row of this lane
            const int hq = 16 * mh + hr;
            const float l = __shfl(l_tot, hr);            // the sum lives in the lanes with l16 == hr
            if (hq >= a.H_q) continue;
            const float inv = (l > 0.f) ? 1.f / l : 0.f;
            T *po = o + hq * D_V + DVW * vh;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) po[16 * nb + l16] = (T)(oacc[nb][i] * inv);
        }
    };
    const int64_t part = (gq * a.n_splits + sp) * a.H_q * D_V;
    if (!split)
        put((__bf16 *)a.Os[layer] + qrow * a.H_q * D_V);
    else if (a.part_wide)
        put((float *)a.part_o + part);
    else
        put((__bf16 *)a.part_o + part);
}

// ---- row-slab form (576/512 MLA rows) --------------------------------------------------
// One workgroup (4 waves, one per SIMD, the whole register file) per CU; tiles of 64 selected
// rows, two tiles resident in LDS.  Wave w owns rows 16w..16w+15 of a tile in the producer role
// and value columns 32w + 128nb + (0..31) in the consumer role:
//   gather    eight lanes fetch one 128-byte line of a row (the access shape the vector memory
//             path serves fastest), 18 loads per lane and tile, refilled in place one tile ahead
//   stage     the wave stores its own 16 rows to the LDS tile (after the barrier of the previous
//             tile, so nobody still reads that buffer) and reads them back in the A-operand
//             layout of v_mfma_f32_16x16x32_bf16: every key byte is written and read once
//   produce   S^T = K Q^T for 16 rows x 32 heads (Q stays in registers), p = 2^(z - m_w) against
//             a lazily updated reference maximum, P and m_w to LDS
//   one barrier per tile
//   consume   M = max over the four m_w; probabilities of wave j are rescaled by 2^(m_j - M) when
//             some m_j differs; O += P V on v_mfma_f32_32x32x16_bf16, whose four contraction
//             steps are exactly the four waves' row groups; V comes out of the same row-major
//             tile through the LDS transpose read, once per element.
// Row sums stay with the producers in their own reference and are combined once at the end.
// The consumer role lags the producer role by one tile (a step = produce tile it, consume tile
// it-1), so the previous tile's operand reads run under the softmax arithmetic and the staging
// stores under the PV MFMAs.
constexpr int kSlabTile = 64;
constexpr float kLazyLog2 = 8.f;

// Tile rows in LDS are padded by 32 bytes (row stride 1184 for rows of 1152) and not swizzled.  Measured on this part
// with every wave of a CU reading: the 16-byte A-operand read of 16 rows (lane = row, same piece in every lane) takes
// 2.3 ticks per instruction with rows 1152 + an odd multiple of 32 bytes apart, as a contiguous read does, and 3.8
// with rows 1152 apart under either of two XOR swizzles; an 8-byte transpose read serves 32 lanes per pass out of 64
// banks of 4 bytes, i.e. 64 contiguous bytes of four rows, and rows 2 x 1184 apart start 64 bytes apart modulo 256:
// conflict-free when the four rows of a pass are two apart (even rows, then odd rows).
constexpr int kSlabPad = 32;

// Reductions over the four 16-lane groups of a wave with the row-swap instructions (plain VALU
// latency, no trip through the LDS crossbar).  permlane16_swap(x, x) yields {[r0,r0,r2,r2],
// [r1,r1,r3,r3]} and permlane32_swap(y, y) yields {[lo,lo],[hi,hi]} in units of 16-lane rows.
__device__ __forceinline__ float xmax16_32(float x)
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

__device__ __forceinline__ float xsum16_32(float x)
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Validity of the 16 rows of a wave from the two ballots over the gather lanes (lane 8r' + piece
// holds row r' of the first / second eight rows): bit r of the result is row r.
__device__ __forceinline__ unsigned rows_mask(unsigned long long ba, unsigned long long bb)
{
    // byte r of a ballot is 0x00 or 0xFF; keep bit 0 of each byte and gather the eight bits in the
    // top byte of a product whose partial sums never collide
    const unsigned long long ones = 0x0101010101010101ull, pack = 0x0102040810204080ull;
    const unsigned lo = (unsigned)(((ba & ones) * pack) >> 56);
    const unsigned hi = (unsigned)(((bb & ones) * pack) >> 56);
    return lo | (hi << 8);
}

// blockIdx.x: query of the launch, flattened (layer, b, t).  SPLIT: blockIdx.y selects a.split_len of its key slots and the result
// is a partial for the merge kernel; otherwise all of them, and O and lse.
template <int D_QK, int D_V, bool PG, bool SPLIT>   // value columns = the first D_V features of a row; PG as above
__global__ __launch_bounds__(256, 1) void attn_slab_kernel(AttnArgs a)
{
    constexpr int KS = D_QK / 32;                         // contraction steps of S^T = 16-byte chunks per gather lane
    constexpr int ROWB = D_QK * 2 + kSlabPad;             // LDS row stride
    static_assert((D_QK * 2) % 128 == 0 && D_V % 128 == 0 && KS % 2 == 0, "row = whole 128-byte windows");
    constexpr int TBUFB = kSlabTile * ROWB;
    constexpr int PSTR = kSlabTile * 2 + 16;              // bytes per head row of the P tile
    constexpr int PBUFB = 32 * PSTR;
    constexpr int NBW = D_V / 4 / 32;                     // 32-column blocks per wave
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char *tbuf = smem;                           // [2][64][ROWB]
    unsigned char *pbuf = smem + 2 * TBUFB;               // [2][32][PSTR]
    float *lbuf = (float *)(pbuf + 2 * PBUFB);            // [4][32] final row sums
    float *abuf = lbuf + 4 * 32;                          // [4][32] per-wave rescale factors

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, g = lane >> 4;
    const int l32 = lane & 31, hh = lane >> 5;
    const int gr = lane >> 3, gp = lane & 7;              // gather role: row (and row + 8), 16-byte piece
    // the arguments that the way to the first gather needs, requested together: left alone, each is loaded where it is first
    // used, a chain of five memory latencies
    // (24 queries in 8 splits: 23.8 us, 23.2 with this)
    asm volatile("" ::"s"(a.n_layers), "s"(a.B), "s"(a.Tq), "s"(a.Lk), "s"(a.H_q), "s"(a.row_elems), "s"(a.k_sel), "s"(a.split_len), "s"(a.row_gap), "s"(a.idx));
    const int sp = (int)blockIdx.y;
    const int slot0 = sp * a.split_len;
    const int slot1 = min(slot0 + a.split_len, a.k_sel);
    const int ntiles = (slot1 - slot0 + kSlabTile - 1) / kSlabTile;
    const int64_t gq = blockIdx.x;
    const int layer = layer_of(a, gq);
    int64_t qrow = gq - (int64_t)layer * a.B * a.Tq;
    const int b = (int)((unsigned)qrow / (unsigned)a.Tq);
    qrow += (int64_t)b * a.row_gap;
    const void *const q_l = a.Qs[layer], *const kv_l = a.KVs[layer];
    asm volatile("" ::"s"(q_l), "s"(kv_l));
    void *const o_l = SPLIT ? nullptr : a.Os[layer];
    const int32_t *idx_row = a.idx + qrow * a.k_sel;
    const unsigned short *kv = (const unsigned short *)kv_l + (PG && a.pv.page_table ? 0 : (int64_t)b * a.Lk * a.row_elems);
    const int len = PG && a.pv.seq_lens ? min(a.pv.seq_lens[b], a.Lk) : a.Lk;   // ragged cache: rows of this sequence

    // Loads inside the tile loop are unconditional (clamped addresses, result discarded when out
    // of range): the wait counters are positional, and a load that may or may not have been
    // issued would force every later wait down to "everything has landed".
    struct Ids { int32_t lo, hi; };                       // validated ids of tile rows 16w+gr and 16w+gr+8
    auto fetch_ids = [&](int it) -> Ids {
        const int s_lo = slot0 + it * kSlabTile + 16 * wave + gr, s_hi = s_lo + 8;
        const int32_t v_lo = idx_row[min(s_lo, a.k_sel - 1)], v_hi = idx_row[min(s_hi, a.k_sel - 1)];
        Ids r;
        // no short-circuit: one basic block, so the loaded ids are not waited for before their use
        r.lo = ((int)(s_lo < slot1) & (int)(v_lo >= 0) & (int)(v_lo < len)) ? v_lo : -1;
        r.hi = ((int)(s_hi < slot1) & (int)(v_hi >= 0) & (int)(v_hi < len)) ? v_hi : -1;
        return r;
    };
    auto row_ptr = [&](int32_t v) {
        // empty slots read row 0 of the cache (never a page-table entry: the sequence may own no page)
        const int64_t prow = v < 0 ? 0 : (PG && a.pv.page_table ? paged_row(a.pv, b, v) : (int64_t)v);
        return kv + prow * a.row_elems + 8 * gp;
    };
    auto ids_mask = [&](const Ids &d) { return rows_mask(__ballot(d.lo >= 0), __ballot(d.hi >= 0)); };

    // Q as the B operand: lane (head 16 hb + l16, features 8 g..) for both head blocks.  All of its
    // loads are issued before anything waits for one of them, and the ids and rows of the first
    // tile are requested in their shadow.
    u32x4 qraw[2][KS];
    auto load_q = [&]() {
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
            const int head = 16 * hb + l16;
            const bool ok = head < a.H_q;
            const unsigned short *qp = (const unsigned short *)q_l + (qrow * a.H_q + (ok ? head : 0)) * D_QK + 8 * g;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                qraw[hb][ks] = u32x4{0u, 0u, 0u, 0u};
                if (ok) qraw[hb][ks] = *(const u32x4 *)(qp + 32 * ks);
            }
        }
    };
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    f32x16 oacc[NBW];
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[nb][i] = 0.f;
    float m_all[2] = {-INFINITY, -INFINITY};              // common reference of all waves, heads 16hb+l16
    float m_ref[2] = {-INFINITY, -INFINITY};              // this wave's current reference
    float m_c = -INFINITY;                                // common reference, head l32
    float l_own[2] = {0.f, 0.f};                          // this lane's share of the wave's row sums (ref m_ref)

    // LDS addresses of the lane in its three roles (byte offsets inside one tile buffer)
    const int st_off = (16 * wave + gr) * ROWB + (gp << 4);                           // + 8 rows for odd chunks
    const int ka_row = (16 * wave + l16) * ROWB;
    const int ka_e = ka_row + (g << 4);                                               // even contraction steps
    const int ka_o = ka_row + ((4 + g) << 4);                                         // odd ones
    // transpose reads: the four rows of a read are two apart; within a group of eight rows the first read takes the
    // even rows (contraction positions 0-3), the second the odd ones (positions 4-7), and P is written in that order
    const int tr_row = 8 * hh + 2 * (l16 >> 2);
    const int tr_slot = 4 * (wave & 1) + 2 * (g & 1) + ((l16 & 3) >> 1);
    const int tr0 = tr_row * ROWB + 128 * (wave >> 1) + (tr_slot << 4) + 8 * (l16 & 1);
    const int tr1 = tr0 + ROWB;

    // The gather registers are refilled chunk by chunk: as soon as chunk ks of tile t+1 has been
    // stored to LDS, the same registers receive chunk ks of tile t+2.
    u32x4 cur[KS];
    auto gload = [&](const Ids &d) {
        const unsigned short *pl = row_ptr(d.lo), *ph = row_ptr(d.hi);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) cur[ks] = *(const u32x4 *)(((ks & 1) ? ph : pl) + 64 * (ks >> 1));
    };
    unsigned vm_cur, vm_n1;
    Ids ids_n2;
    bf16x8 qreg[2][KS];
    // pin Q to the accumulation half of the register file (MFMA reads B operands from there
    // directly): the vector half is needed for the gather and the LDS operands
    auto pin_q = [&]() {
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                u32x4 raw = qraw[hb][ks];
                asm volatile("" : "+a"(raw));
                qreg[hb][ks] = __builtin_bit_cast(bf16x8, raw);
            }
    };
    {
        const Ids d0 = fetch_ids(0), d1 = fetch_ids(1);
        ids_n2 = fetch_ids(2);
        __builtin_amdgcn_sched_barrier(0);
        // One wave loads Q (each load touches 16 rows of it, so four waves loading the same 36 KB keep the CU's one address
        // unit busy for 2.8 us) and hands it over; its loads go out behind the id fetches, so that the ids, and with them the
        // first gather, do not wait for Q
        if (wave_u == 0) load_q();
        gload(d0);
        __builtin_amdgcn_sched_barrier(0);
        {   // Q from wave 0 to the others through the second tile buffer (unused until step 0 stages tile 1)
            unsigned char *mine = tbuf + TBUFB + lane * 16;
            if (wave_u == 0) {
#pragma unroll
                for (int hb = 0; hb < 2; ++hb)
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) *(u32x4 *)(mine + (hb * KS + ks) * 1024) = qraw[hb][ks];
            }
            __syncthreads();
            if (wave_u != 0) {
#pragma unroll
                for (int hb = 0; hb < 2; ++hb)
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) qraw[hb][ks] = *(const u32x4 *)(mine + (hb * KS + ks) * 1024);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        pin_q();
        vm_cur = ids_mask(d0);
        vm_n1 = ids_mask(d1);
        const unsigned short *pl = row_ptr(d1.lo), *ph = row_ptr(d1.hi);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            *(u32x4 *)(tbuf + st_off + (ks & 1) * 8 * ROWB + 128 * (ks >> 1)) = cur[ks];
            cur[ks] = *(const u32x4 *)(((ks & 1) ? ph : pl) + 64 * (ks >> 1));
        }
    }

    // One step = the producer role for tile `it` and the consumer role for tile it-1 (have_prev).
    // stage_next: tile it+1 exists (store it);  load_next2: tile it+2 exists (refill the gather
    // registers).  The LDS pipeline is the busiest unit of this kernel (it spends about as long on
    // a 4-byte access as on a 16-byte one), so everything that crosses it is packed into wide
    // instructions and spread over the step: A-operand reads under the S^T MFMAs, the previous
    // tile's P/V operand reads under the softmax arithmetic, the staging stores under the PV MFMAs.
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    auto step = [&](int it, auto have_prev, auto have_cur, auto stage_next, auto load_next2) {
        constexpr bool kPrev = decltype(have_prev)::value, kCur = decltype(have_cur)::value;
        constexpr bool kStage = decltype(stage_next)::value, kLoad = decltype(load_next2)::value;
        const int buf = it & 1;
        Ids ids_n3 = ids_n2;
        if constexpr (kCur) ids_n3 = fetch_ids(it + 3);
        const unsigned char *tb = tbuf + buf * TBUFB;                 // tile it
        const unsigned char *tp = tbuf + (buf ^ 1) * TBUFB;           // tile it-1
        unsigned char *pb = pbuf + buf * PBUFB;                       // P of tile it
        const unsigned char *pp = pbuf + (buf ^ 1) * PBUFB;           // P of tile it-1

        // reference maxima of tile it-1 first: the softmax of tile it builds on them
        f32x4 mjc = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        if constexpr (kPrev) mjc = *(const f32x4 *)(pp + l32 * PSTR + kSlabTile * 2);

        // consumer operands of tile it-1: probabilities of head l32 and every value operand.  The first of these
        // reads go out under the last S^T MFMAs (kConsPer per contraction step from step kConsFrom on: measured, 3
        // from step 10 on is 2.6 % faster than all of them behind the MFMAs and 2 % faster than all of them under
        // the MFMAs), the rest stream in while the softmax below keeps the vector ALU busy.
        bf16x8 pa[4];
        s16x4 vq[4][NBW][2];
        constexpr int NCR = 4 + 8 * NBW;                  // consumer reads of a step
        constexpr int kConsFrom = KS > 10 ? 10 : KS, kConsPer = 3;
        static_assert((KS - kConsFrom) * kConsPer <= NCR, "no more early reads than there are reads");
        auto cons_read = [&](int n) __attribute__((always_inline)) {
            if constexpr (kPrev) {
                if (n < 4) {
                    pa[n] = *(const bf16x8 *)(pp + l32 * PSTR + (16 * n + 8 * hh) * 2);
                } else if (n < NCR) {
                    const int m = n - 4, j = m / (2 * NBW), nb = (m >> 1) % NBW;
                    vq[j][nb][m & 1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (lds_s16x4 *)(tp + ((m & 1) ? tr1 : tr0) + 16 * j * ROWB + 256 * nb));
                }
            }
        };

        // S^T for the wave's 16 rows x 32 heads: two accumulation chains per head block
        f32x4 s4[2][2];
        if constexpr (kCur) {
#pragma unroll
            for (int hb = 0; hb < 2; ++hb)
#pragma unroll
                for (int par = 0; par < 2; ++par) s4[hb][par] = f32x4{0.f, 0.f, 0.f, 0.f};
            constexpr int KRING = 4;                      // A-operand reads in flight ahead of the MFMAs
            bf16x8 ka[KRING];
            auto ka_read = [&](int ks) { return *(const bf16x8 *)(tb + ((ks & 1) ? ka_o : ka_e) + 128 * (ks >> 1)); };
#pragma unroll
            for (int r = 0; r < KRING; ++r) ka[r] = ka_read(r);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                s4[0][ks & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[ks % KRING], qreg[0][ks], s4[0][ks & 1], 0, 0, 0);
                s4[1][ks & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[ks % KRING], qreg[1][ks], s4[1][ks & 1], 0, 0, 0);
                if (ks + KRING < KS) ka[ks % KRING] = ka_read(ks + KRING);
                if (ks >= kConsFrom) {
#pragma unroll
                    for (int n = (ks - kConsFrom) * kConsPer; n < (ks - kConsFrom + 1) * kConsPer; ++n) cons_read(n);
                }
            }
        }
        {
            constexpr int n0 = kCur ? (KS - kConsFrom) * kConsPer : 0;
#pragma unroll
            for (int n = n0; n < NCR; ++n) cons_read(n);
        }

        float alpha = 1.f, fj[4] = {1.f, 1.f, 1.f, 1.f};
        bool any_f = false;
        if constexpr (kPrev) {
            // new common reference of head l32 (= 16 (g&1) + l16); the producer role needs it for
            // heads l16 and 16 + l16, one of which lives in the neighbouring 16-lane group
            const float m_new_c = fmaxf(fmaxf(mjc[0], mjc[1]), fmaxf(mjc[2], mjc[3]));
            const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(m_new_c), __float_as_uint(m_new_c), false, false);
            m_all[0] = __uint_as_float(sw[0]);            // groups [0,0,2,2]: head l16
            m_all[1] = __uint_as_float(sw[1]);            // groups [1,1,3,3]: head 16 + l16
            alpha = (m_new_c == -INFINITY) ? 1.f : fast_exp2(m_c - m_new_c);
            m_c = m_new_c;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                fj[j] = (m_new_c == -INFINITY) ? 1.f : fast_exp2(mjc[j] - m_new_c);
                any_f |= (fj[j] != 1.f);
            }
        }
        __builtin_amdgcn_sched_barrier(0);

        // producer role: rows 4 g + i of the wave.  A head row of the P tile is 128 bytes of
        // probabilities followed by the four waves' reference maxima in its 16 bytes of padding.
        if constexpr (kCur) {
#pragma unroll
            for (int hb = 0; hb < 2; ++hb) {
                float z[4];
                float mx = -INFINITY;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool ok = (vm_cur >> (4 * g + i)) & 1u;
                    z[i] = ok ? (s4[hb][0][i] + s4[hb][1][i]) * a.scale_log2e : -INFINITY;
                    mx = fmaxf(mx, z[i]);
                }
                mx = xmax16_32(mx);
                // lazy reference: keep the common reference until this tile exceeds it by more than
                // 2^kLazyLog2 (probabilities up to that factor are harmless in bf16/fp32), so that
                // the rescaling paths below run only on real jumps of the maximum
                const float m_new = (mx > m_all[hb] + kLazyLog2) ? mx : m_all[hb];   // m_all >= m_ref always
                const float resc = (m_new == -INFINITY) ? 1.f : fast_exp2(m_ref[hb] - m_new);
                float psum = 0.f;
                short pk[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float p = (z[i] == -INFINITY) ? 0.f : fast_exp2(z[i] - m_new);
                    psum += p;
                    pk[i] = __builtin_bit_cast(short, (__bf16)p);
                }
                l_own[hb] = l_own[hb] * resc + psum;
                m_ref[hb] = m_new;
                unsigned char *prow = pb + (16 * hb + l16) * PSTR;
                // row e of a group of eight sits at contraction position e / 2 + 4 (e % 2) (see the transpose reads):
                // the lane's rows 4 (g & 1) + {0, 2} are neighbours there, and so are its rows 4 (g & 1) + {1, 3}
                typedef __attribute__((ext_vector_type(2))) short s16x2;
                unsigned char *pg = prow + (16 * wave + 8 * (g >> 1) + 2 * (g & 1)) * 2;
                *(s16x2 *)pg = s16x2{pk[0], pk[2]};
                *(s16x2 *)(pg + 8) = s16x2{pk[1], pk[3]};
                if (g == 0) *(float *)(prow + kSlabTile * 2 + 4 * wave) = m_new;
            }
        }
        // P of tile it is written; every wave has all its reads of tile it-1 back
        __syncthreads();

        if constexpr (kPrev) {
            if (__ballot(alpha != 1.f) != 0ull) {
                // the rescale factors of the 16 heads a lane accumulates, through a per-wave LDS row
                float *ab = abuf + wave * 32;
                if (hh == 0) ab[l32] = alpha;
                f32x4 ar[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) ar[q] = *(const f32x4 *)(ab + 8 * q + 4 * hh);
                // The accumulators live in accumulation registers; move each value out and back
                // right here (opaque to the compiler), otherwise it copies all 64 of them to vector
                // registers ahead of the branch in every tile.  The MFMAs that wrote them retired
                // a tile ago and the next MFMA that reads them is far behind the trailing no-ops.
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        float t;
                        asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(t) : "a"(oacc[nb][i]));
                        t *= ar[i >> 2][i & 3];
                        asm volatile("v_accvgpr_write_b32 %0, %1" : "=a"(oacc[nb][i]) : "v"(t));
                    }
                asm volatile("s_nop 7\n\ts_nop 7");
            }
            if (__ballot(any_f) != 0ull) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int e = 0; e < 8; ++e) pa[j][e] = (__bf16)((float)pa[j][e] * fj[j]);
            }
        }
        const unsigned vm_n2 = ids_mask(ids_n2);

        // O += P V for tile it-1, with the staging of tile it+1 (nobody reads that buffer any more)
        // and the gather of tile it+2 issued in the shadow of the MFMAs
        unsigned char *tn = tbuf + (buf ^ 1) * TBUFB + st_off;
        const unsigned short *pl = row_ptr(ids_n2.lo), *ph = row_ptr(ids_n2.hi);
        auto stage = [&](int ks) {
            if constexpr (kStage) {
                if (ks < KS) {
                    *(u32x4 *)(tn + (ks & 1) * 8 * ROWB + 128 * (ks >> 1)) = cur[ks];
                    if constexpr (kLoad) cur[ks] = *(const u32x4 *)(((ks & 1) ? ph : pl) + 64 * (ks >> 1));
                }
            }
        };
        if constexpr (kPrev) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb) {
                    const s16x4 v0 = vq[j][nb][0], v1 = vq[j][nb][1];
                    const s16x8 vv = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                    oacc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa[j], __builtin_bit_cast(bf16x8, vv), oacc[nb], 0, 0, 0);
                    stage(4 * j + nb);
                }
#pragma unroll
            for (int ks = 4 * NBW; ks < KS; ++ks) stage(ks);
            if constexpr (kStage) {
                // keep the order: one MFMA, then one LDS store and (when there is one) one gather load
#pragma unroll
                for (int k = 0; k < 4 * NBW; ++k) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                    if constexpr (kLoad) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                }
            }
        } else {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) stage(ks);
        }
        if constexpr (kCur) {                             // the drain step leaves the stream where it is
            vm_cur = vm_n1;
            vm_n1 = vm_n2;
            ids_n2 = ids_n3;
        }
    };

    // ---- epilogue of a query: combine the producers' row sums, normalise, store ----
    auto finish = [&]() {
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
            const float l = xsum16_32(l_own[hb]);
            // bring the wave's sum to the common reference before publishing it
            const float f = (m_all[hb] == -INFINITY) ? 0.f : fast_exp2(m_ref[hb] - m_all[hb]);
            if (g == 0) lbuf[wave * 32 + 16 * hb + l16] = l * f;
        }
        __syncthreads();
        const float l_head = lbuf[l32] + lbuf[32 + l32] + lbuf[64 + l32] + lbuf[96 + l32];   // head l32
        const float m_head = m_c;
        {
            if constexpr (SPLIT) {
                // partial of this split: its reference maximum and row sum (the output below is
                // normalised by that sum; the merge weighs the splits by their share of the total)
                if (wave == 0 && hh == 0 && l32 < a.H_q) {
                    float *ml = a.part_ml + ((gq * a.n_splits + sp) * a.H_q + l32) * 2;
                    ml[0] = m_head;
                    ml[1] = l_head;
                }
            } else {
                if (wave == 0 && hh == 0 && l32 < a.H_q && a.lse)
                    a.lse[qrow * a.H_q + l32] = l_head > 0.f ? (float)(((double)m_head + (double)__builtin_log2f(l_head)) * 0.6931471805599453) : -INFINITY;
            }
            // accumulator element i belongs to head 8 (i / 4) + 4 hh + i % 4: the sums of the lane's
            // 16 heads come straight from the four waves' partials (independent 16-byte reads; a
            // lane-to-lane shuffle per head would be sixteen dependent trips through the crossbar)
            f32x4 inv4[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x4 l4 = *(const f32x4 *)(lbuf + 8 * q + 4 * hh);
#pragma unroll
                for (int w = 1; w < 4; ++w) l4 += *(const f32x4 *)(lbuf + 32 * w + 8 * q + 4 * hh);
#pragma unroll
                for (int r = 0; r < 4; ++r) inv4[q][r] = (l4[r] > 0.f) ? __builtin_amdgcn_rcpf(l4[r]) : 0.f;
            }
            const bool all_heads = a.H_q >= 32;               // workgroup-uniform
            // the lane's offset into O is recomputed from the thread id here: kept live across the
            // tile loop it is spilled, and its reload waits behind every gather in flight
            int tx = tid;
            asm volatile("" : "+v"(tx));
            const int o_lane = 32 * (tx >> 6) + (tx & 31), o_hh = (tx >> 5) & 1;
            auto put = [&](auto *o_row) __attribute__((always_inline)) {
                typedef std::remove_pointer_t<decltype(o_row)> E;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int hq = 8 * (i >> 2) + 4 * o_hh + (i & 3); // O row (head) of accumulator element i
                    const float inv = inv4[i >> 2][i & 3];
                    if (all_heads || hq < a.H_q) {
#pragma unroll
                        for (int nb = 0; nb < NBW; ++nb) o_row[hq * D_V + 128 * nb] = (E)(oacc[nb][i] * inv);
                    }
                }
            };
            const int64_t part = (gq * a.n_splits + sp) * a.H_q * D_V + o_lane;
            if constexpr (!SPLIT)
                put((__bf16 *)o_l + qrow * a.H_q * D_V + o_lane);
            else if (a.part_wide)
                put((float *)a.part_o + part);
            else
                put((__bf16 *)a.part_o + part);
        }
    };

    constexpr std::true_type T{};
    constexpr std::false_type F{};
    // Step 0 has no previous tile, step ntiles has no current one.  (In this order of cases nothing is spilled; with the short ones
    // first twelve values were, and scratch costs a launch 1.1 us.)
    if (ntiles >= 3) {
        step(0, F, T, T, T);
        int it = 1;
#pragma unroll 1
        for (; it + 2 < ntiles; ++it) step(it, T, T, T, T);
        step(it, T, T, T, F);
        ++it;
        step(it, T, T, F, F);
    } else if (ntiles == 2) {
        step(0, F, T, T, F);
        step(1, T, T, F, F);
    } else {
        step(0, F, T, F, F);
    }
    step(ntiles, T, F, F, F);
    finish();
}

// ---- dense form (rows whose selection is a whole prefix of the cache) ---------------------------------------------
// The first rows of a sequence see no more keys than k: their selection is positions 0 .. n-1, so neighbouring queries
// read the same KV rows and there is nothing to gather.  Here 64 rows of the flattened (query, head) space (two queries of
// 32 heads) share every KV tile: twice the matrix work per byte that crosses LDS, which is what the row-slab form is
// bound by.  One workgroup per CU, tiles of 32 keys in a ring of four LDS buffers, one barrier per tile, eight waves in two
// roles (one of each per SIMD, and about as many matrix clocks for either: 576 and 512 per tile):
//   scores   waves 0-3, (rh, kh) = 32 rows x 16 keys of tile t: the tile as A operand of v_mfma_f32_16x16x32_bf16, every
//            read of it used for two row blocks, Q in registers; softmax against a reference per row that moves only when
//            a score exceeds it by 2^kLazyLog2; P to LDS.  The operand ring runs on into the next tile
//   output   waves 4-7, value columns 128 w .. 128 w + 127 of all 64 rows, of tile t - 2, transposed (O^T += V^T P^T on
//            v_mfma_f32_32x32x16_bf16, V through the transpose read): a lane then owns one row of O, so that factors and
//            row sums are a lane's own and four neighbouring columns leave together.  Its operands are in registers when
//            the step begins; as they are used, those of tile t - 1 take their place, tile t + 2 goes to LDS and tile t + 3
//            is requested
// What counts is the traffic through LDS and what waits for it.  With every wave taking both phases, a wave can hold Q of 16
// rows only, the score operand was 147 KB of 290 KB per tile and a tile took 2700-2900 clocks however the phases were
// arranged (two barriers per 64 keys, one per 32, the two waves of a SIMD in opposite order).  Here it is 74 KB of 200 KB:
// 2400 clocks, 1800 with the operands read a step ahead.  1088 of them are matrix clocks; staging the tiles costs about 300
// (it may not move to the scores waves: 1900).  One layer of 32 heads, 2048 rows of a prefix: 180 us before, 145 now.
// LDS layout as in the row-slab form (rows 1184 bytes apart, transpose reads over rows two apart); the A operand presents
// the tile rows in the order dense_row(), so that the four scores of a lane are neighbours in P.
// A workgroup walks a chain of blocks as one stream of tiles, the next block's Q and first keys behind the last one's, and the outputs
// leave under the next block's first steps: with a workgroup per block, its start (Q, first tile, two steps until the first
// product) and end were about 6 us of the 12 to 25 that a block takes.  Four layers of 3 x 1021 rows 578 -> 511 us.  Where a workgroup
// has one block the chain's start is what counts: its Q and first keys are requested together and it has no step 0 (64 rows, one launch
// 11.1 -> 10.4 us; with a workgroup per block and no chain 9.5).
// Registers.  The two roles need 249 of the 256 that a wave may have: Q of 32 rows takes 144 in the scores waves, the output
// accumulators 128 in the others.  The compiler places all of it: state that it is not told of (registers named in asm
// statements) is only safe as long as it happens to put no value of its own there.

// f(integral_constant 0 .. N-1), in order
template <int N, typename F> __device__ __forceinline__ void unroll(F f)
{
    if constexpr (N > 0) {
        unroll<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

constexpr int kDenseRows = 64;               // (query, head) rows per workgroup
constexpr int kDenseTile = 32;               // keys per tile
constexpr int kDenseRing = 4;
constexpr int kDenseChain = 64;              // blocks of a workgroup, at most (their list is in LDS)

struct DenseShape {
    int n_blk, n_wgs, n_round;               // blocks of a sequence, workgroups, whole rounds of them
    unsigned inv_b, inv_h;                   // 2^32 / B and / H_q, rounded up (inv_b 0: divide)
    int n_whole;                             // several layers: rounds that a layer fills, 2^32 / n_layers, rounded up
    unsigned inv_layers;
};

// tile row (within 16) behind result row r of S^T
__device__ __forceinline__ int dense_row(int r) { return 8 * (r >> 3) + 2 * (r & 3) + ((r >> 2) & 1); }

// MULTI: the rows of a.n_layers layers (with their layer a variable, one layer of 3 x 1021 rows took 1 us of 123 longer).
template <bool PG, bool MULTI>
__device__ __forceinline__ void dense_rows(const AttnArgs &a, const DenseArgs &da, const DenseShape &ds)
{
    constexpr int D_QK = 576, D_V = 512;
    constexpr int KS = D_QK / 32;                         // contraction steps
    constexpr int ROWB = D_QK * 2 + kSlabPad, TBUFB = kDenseTile * ROWB;
    constexpr int PSTR = kDenseTile * 2 + 16, PBUFB = kDenseRows * PSTR;
    constexpr int OSTR = 256 + 16;                        // a wave's 128 columns of an output row
    constexpr int RING = 9;                              // A-operand reads in flight
    static_assert(kDenseRows == 2 * kDenseTile && 32 * OSTR <= 8 * ROWB, "Q takes two tiles' places, half of a wave's outputs its eight rows of one");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char *tbuf = smem;                           // [kDenseRing][32][ROWB]
    unsigned char *pbuf = smem + kDenseRing * TBUFB;      // [2][64 rows][PSTR]
    float *mref = (float *)(pbuf + 2 * PBUFB);            // [64] common references
    float *mnew = mref + kDenseRows;                      // [2][64] per key half: reference of the latest tile, then row sums
    float *fac = mnew + 2 * kDenseRows;                   // [3][64] factors of a moved reference: O, P of either key half
    int *moved = (int *)(fac + 3 * kDenseRows);           // [2] by step; [2] by block: a key some row does not see has no finite score
    int *list = moved + 4;                                // [kDenseChain] queries of the block's sequence, 0: no such block

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, l32 = lane & 31, hh = lane >> 5, g = lane >> 4;
    const int gr = lane >> 3, gp = lane & 7;
    const int w = wave & 3;
    // (requested together, and divided by reciprocals: a division is a tenth of a us, and there are ten in front of the first load)
    asm volatile("" ::"s"(a.Q), "s"(a.KV), "s"(a.B), "s"(a.Tq), "s"(a.Lk), "s"(a.H_q), "s"(a.row_elems), "s"(a.n_layers), "s"(da.n_queries), "s"(da.pos0), "s"(da.lead), "s"(ds.n_blk), "s"(ds.n_wgs), "s"(ds.inv_b), "s"(ds.inv_h));
    auto div_b = [&](int x) -> int { return a.B == 1 ? x : ds.inv_b ? (int)__umulhi((unsigned)x, ds.inv_b) : x / a.B; };
    auto div_h = [&](int x) -> int { return a.H_q == 1 ? x : (int)__umulhi((unsigned)x, ds.inv_h); };
    // blocks of the workgroup, all sequences' blocks of a layer ranked by length: there and back over the workgroups, which evens them
    // out.  Several layers take turns (a layer's blocks share its keys): two rounds each, there and back, as long as they fill them, then
    // one round each, then rank by rank.  Layer behind layer, the long blocks of one fell where the other's short ones should.  us, a
    // launch each / layer behind layer / this: 3 layers of 1021 rows 144 / 158 / 132, 4 of 1000 196 / 207 / 169, of 1024 200 / 183 / 173.
    const int n_blk = ds.n_blk, n_all = n_blk * (MULTI ? a.B * a.n_layers : a.B), n_wgs = ds.n_wgs;
    auto place = [&](int n) -> int { return n & 1 ? n_wgs - 1 - (int)blockIdx.x : (int)blockIdx.x; };      // in round n
    int whole = ds.n_whole, n_layers = a.n_layers;
    unsigned inv_layers = ds.inv_layers;
    if (MULTI) asm volatile("" : "+s"(whole), "+s"(n_layers), "+s"(inv_layers));      // (kept: loaded again for every block they cost a us each)
    auto rank_of = [&](int n, int &layer) -> int {        // rank within the layer of block n of the list
        layer = 0;
        if (!MULTI) return n * n_wgs + place(n);
        const int paired = (whole & ~1) * n_layers, all = whole * n_layers;
        if (n < all && n >= paired) {
            layer = n - paired;
            return (whole - 1) * n_wgs + place(n);
        }
        const bool pair = n < paired;
        const int x = pair ? n >> 1 : (n - all) * n_wgs + place(n), by = (int)__umulhi((unsigned)x, inv_layers);
        layer = x - by * n_layers;
        return pair ? (2 * by + (n & 1)) * n_wgs + place(n) : whole * n_wgs + by;
    };
    int n_list = ds.n_round;
    n_list += n_list * n_wgs + place(n_list) < n_all;
    if (tid < kDenseRows) mref[tid] = mnew[tid] = mnew[kDenseRows + tid] = -INFINITY;
    if (tid < 4) moved[tid] = 0;
    if (da.lead) {
        for (int n = wave; n < n_list; n += 8) {
            int layer;
            const int r = rank_of(n, layer), r_b = div_b(r), b = r - r_b * a.B, R0 = (n_blk - 1 - r_b) * kDenseRows;
            const int nq = __builtin_amdgcn_readfirstlane(min(da.n_queries, lead_rows(da.lead + ((int64_t)layer * a.B + b) * da.n_chunks, da.n_chunks)));
            if (lane == 0) list[n] = R0 < nq * a.H_q ? nq : 0;
        }
        __syncthreads();
    }
    struct Block { int n, odd, layer, b, R0, n_queries, n_rows, nt, t_edge; };  // n = n_list: none
    auto open = [&](int n, int odd) {                     // block n of the list, or the first one behind it that exists
        Block k;
        k.odd = odd;                                      // (odd and even ones alternate)
        int nq = da.n_queries;
        if (da.lead)
            while (n < n_list && (nq = __builtin_amdgcn_readfirstlane(list[n])) == 0) ++n;
        const int r = rank_of(min(n, n_list - 1), k.layer), r_b = div_b(r);
        k.n = n;
        k.b = r - r_b * a.B;
        k.R0 = (n_blk - 1 - r_b) * kDenseRows;
        k.n_queries = nq;
        k.n_rows = nq * a.H_q;                            // flattened rows of a sequence
        k.nt = (da.pos0 + div_h(max(min(k.R0 + kDenseRows, k.n_rows) - 1, 0))) / kDenseTile + 1;
        k.t_edge = (da.pos0 + div_h(k.R0) + 1) / kDenseTile;             // first tile with keys that some row does not see
        return k;
    };
    const Block first = open(0, 0);
    if (first.n == n_list) return;

    // The blocks are one stream of tiles: the two of Q (its rows in the shape of keys), then the block's nt of keys, then the
    // next block's.  Step i: tile i is scored (Q: read), the operands of tile i - 1 and the product of tile i - 2 are taken, tile
    // i + 2 goes to LDS and tile i + 3 into registers.  Barriers: one before step 1 (Q and the first keys are there: there is no step 0)
    // and one at the end of every step, one more within step i + 1 if a reference moved in tile i.
    if (wave < 4) {
        const int rh = w & 1, kh = w >> 1;
        bf16x8 qv[KS][2];
        __syncthreads();
        int lim[2], lim0;                                 // last key the lane's rows see, the smallest of the wave
        const int ka_off = (16 * kh + dense_row(l16)) * ROWB + 16 * g;
        const int pw_off = (32 * rh + l16) * PSTR + 32 * kh + 8 * g;
        float m_c[2] = {-INFINITY, -INFINITY}, l_own[2] = {0.f, 0.f}, psum[2] = {0.f, 0.f};
        bf16x8 ka[RING];
        f32x4 s4[2], odd[2];                              // two accumulation chains, as in the row form: half of the roundings in one
        auto scores = [&](int t) __attribute__((always_inline)) {
            const unsigned char *tb = tbuf + (t & (kDenseRing - 1)) * TBUFB + ka_off;
            const unsigned char *tb1 = tbuf + ((t + 1) & (kDenseRing - 1)) * TBUFB + ka_off;
            unroll<KS>([&](auto ks_c) __attribute__((always_inline)) {
                constexpr int ks = decltype(ks_c)::value;
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    f32x4 &c = ks % 2 ? odd[r] : s4[r];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[ks % RING], qv[ks][r], ks < 2 ? f32x4{0.f, 0.f, 0.f, 0.f} : c, 0, 0, 0);
                }
                ka[ks % RING] = ks + RING < KS ? *(const bf16x8 *)(tb + 64 * (ks + RING)) : *(const bf16x8 *)(tb1 + 64 * (ks + RING - KS));
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        auto softmax = [&](int i, int t, int parity) __attribute__((always_inline)) { // tile t of an even or odd block, step i
            // lane: row l16 of either block, keys dense_row(4 g + i)
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) s4[r][i] += odd[r][i];
            const int key0 = kDenseTile * t + 16 * kh;
            if (key0 + 15 > lim0) {
                const int k0 = key0 + 8 * (g >> 1) + (g & 1);
                float z = 0.f;                            // NaN if any of the scores is not finite
#pragma unroll
                for (int i = 0; i < 4; ++i) z = __builtin_fmaf(s4[1][i], 0.f, __builtin_fmaf(s4[0][i], 0.f, z));
                if (__ballot(z != 0.f) != 0ull) moved[2 + parity] = 1;
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int i = 0; i < 4; ++i) s4[r][i] = k0 + 2 * i <= lim[r] ? s4[r][i] : -INFINITY;
            }
            float m_use[2], mx[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                m_use[r] = m_c[r];
                mx[r] = fmaxf(fmaxf(s4[r][0], s4[r][1]), fmaxf(s4[r][2], s4[r][3])) * a.scale_log2e;
            }
            if (__ballot(mx[0] > m_c[0] + kLazyLog2 || mx[1] > m_c[1] + kLazyLog2) != 0ull) {
                // rare: some row's first keys, or a score far above all before it
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    mx[r] = xmax16_32(mx[r]);
                    m_use[r] = mx[r] > m_c[r] + kLazyLog2 ? mx[r] : m_c[r];
                    if (g == 0) mnew[kDenseRows * kh + 32 * rh + 16 * r + l16] = m_use[r];
                }
                moved[i & 1] = 1;
            }
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const float m_safe = m_use[r] == -INFINITY ? 0.f : m_use[r];   // (no key so far: every p is 2^-inf = 0)
                s16x4 pk;
                float p[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    p[i] = fast_exp2(__builtin_fmaf(s4[r][i], a.scale_log2e, -m_safe));
                    pk[i] = __builtin_bit_cast(short, (__bf16)p[i]);
                }
                *(s16x4 *)(pbuf + (i & 1) * PBUFB + pw_off + 16 * r * PSTR) = pk;
                psum[r] = (p[0] + p[1]) + (p[2] + p[3]);
            }
        };
        // a reference moved in the tile of the step before (flag: uniform over the workgroup); its row sums
        auto settle = [&](int i, int flag) __attribute__((always_inline)) {
            if (__builtin_amdgcn_readfirstlane(flag)) {
                if (tid < kDenseRows) {
                    const float m0 = mnew[tid], m1 = mnew[kDenseRows + tid], m = fmaxf(m0, m1), old = mref[tid];
                    fac[tid] = m == -INFINITY ? 1.f : fast_exp2(old - m);
                    fac[kDenseRows + tid] = m == -INFINITY ? 1.f : fast_exp2(m0 - m);
                    fac[2 * kDenseRows + tid] = m == -INFINITY ? 1.f : fast_exp2(m1 - m);
                    mref[tid] = mnew[tid] = mnew[kDenseRows + tid] = m;
                }
                __syncthreads();                          // (everybody has read the flag)
                if (tid == 0) moved[(i - 1) & 1] = 0;     // next raised behind the barrier that ends this step
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int row = 32 * rh + 16 * r + l16;
                    l_own[r] *= fac[row];
                    psum[r] *= fac[kDenseRows * (1 + kh) + row];
                    m_c[r] = mref[row];
                }
            }
#pragma unroll
            for (int r = 0; r < 2; ++r) l_own[r] += psum[r];
        };
        int i = 0;
        Block k = first;
#pragma unroll 1
        for (;;) {
            // Q's steps.  Of the block before: what its last tile moved, then its sums and references for the output waves, where
            // the factors are otherwise
            if (i > 0) settle(i, moved[(i - 1) & 1]);
            if (k.n < n_list) {                           // (at the start both of its tiles are there)
                const unsigned char *qr = tbuf + ((i + rh) & (kDenseRing - 1)) * TBUFB + l16 * ROWB + 16 * g;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int r = 0; r < 2; ++r) qv[ks][r] = *(const bf16x8 *)(qr + 16 * r * ROWB + 64 * ks);
            }
            if (i > 0) __syncthreads();
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int row = 32 * rh + 16 * r + l16;
                const float l = xsum16_32(l_own[r]);
                if (g == 0) {
                    fac[kDenseRows * kh + row] = l;
                    fac[2 * kDenseRows + row] = m_c[r];   // (either half writes the same)
                }
                l_own[r] = psum[r] = 0.f;
                m_c[r] = -INFINITY;
                lim[r] = da.pos0 + div_h(max(min(k.R0 + row, k.n_rows - 1), 0));
            }
            lim0 = __builtin_amdgcn_readfirstlane(lim[0]);
            if (tid < kDenseRows) mref[tid] = mnew[tid] = mnew[kDenseRows + tid] = -INFINITY;
            if (tid == 0) moved[2 + k.odd] = 0;       // (that of the block before the last one)
            __syncthreads();
            if (k.n == n_list) return;
            i += 2;
#pragma unroll
            for (int r = 0; r < RING; ++r) ka[r] = *(const bf16x8 *)(tbuf + (i & (kDenseRing - 1)) * TBUFB + ka_off + 64 * r);
            scores(i);
            softmax(i, 0, k.odd);
            __syncthreads();
            ++i;
#pragma unroll 1
            for (int t = 1; t < k.nt; ++t, ++i) {
                const int flag = moved[(i - 1) & 1];
                __builtin_amdgcn_sched_barrier(0);
                scores(i);
                settle(i, flag);
                softmax(i, t, k.odd);
                __syncthreads();
            }
            k = open(k.n + 1, k.odd ^ 1);
        }
    } else {
        // A tile is fetched eight lanes to a 128-byte line: rows 8 w + gr, nine lines.
        u32x4 cur[9];
        // the next tile to request: tile aj of block an, Q is 0 and 1; its rows' first addresses and their last rows
        int an, aj, ant, aq_last, ak_last, ab = 0;
        const unsigned short *aq, *ak;
        auto aim = [&](const Block &x) __attribute__((always_inline)) {
            an = x.n;
            aj = 0;
            ant = x.nt;
            aq = (const unsigned short *)(MULTI ? a.Qs[x.layer] : a.Q) + ((int64_t)x.b * a.Tq * a.H_q + x.R0) * D_QK;
            aq_last = x.n_rows - 1 - x.R0;
            ak = (const unsigned short *)(MULTI ? a.KVs[x.layer] : a.KV) + (PG && a.pv.page_table ? 0 : (int64_t)x.b * a.Lk * a.row_elems);
            ak_last = da.pos0 + x.n_queries - 1;
            if constexpr (PG) ab = x.b;
        };
        aim(first);
        auto tile_src = [&]() -> const unsigned short * { // (past the last block: one row of its Q, for nobody)
            const unsigned short *p;
            if (ant == INT32_MAX) {
                p = aq;
            } else if (aj < 2) {
                p = aq + min(32 * aj + 8 * w + gr, aq_last) * D_QK;
            } else {
                const int s0 = (aj - 2) * kDenseTile;                      // (a tile never straddles a page)
                const int64_t row = PG && a.pv.page_table ? paged_row(a.pv, ab, s0) : (int64_t)s0;
                p = ak + (row + min(8 * w + gr, ak_last - s0)) * a.row_elems;
            }
            if (__builtin_expect(++aj - 2 == ant, 0)) {
                const Block nx = open(an + 1, 0);
                if (nx.n < n_list)
                    aim(nx);
                else
                    ant = INT32_MAX;                      // (never to come round)
            }
            return p + 8 * gp;
        };
        auto load = [&]() __attribute__((always_inline)) {
            const unsigned short *p = tile_src();
#pragma unroll
            for (int c = 0; c < 9; ++c) cur[c] = *(const u32x4 *)(p + 64 * c);
        };
        const int st_off = (8 * w + gr) * ROWB + 16 * gp;
        auto store = [&](int t, int c0, int n) __attribute__((always_inline)) {
            unsigned char *d = tbuf + (t & (kDenseRing - 1)) * TBUFB + st_off;
            for (int c = c0; c < c0 + n; ++c) *(u32x4 *)(d + 128 * c) = cur[c];
        };
        {
            u32x4 q0[2][9];                               // Q and the first keys, requested together
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                load();
#pragma unroll
                for (int c = 0; c < 9; ++c) q0[t][c] = cur[c];
            }
            load();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int c = 0; c < 9; ++c) *(u32x4 *)(tbuf + t * TBUFB + st_off + 128 * c) = q0[t][c];
            store(2, 0, 9);
            load();
        }
        f32x16 o_acc[2][4];                               // [rows 32 r ..][columns 32 nb ..]
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int e = 0; e < 16; ++e) o_acc[r][nb][e] = 0.f;
        typedef __attribute__((ext_vector_type(8))) short s16x8;
        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
        const int tr_off = (8 * hh + 2 * (l16 >> 2)) * ROWB + 256 * w + 32 * (g & 1) + 8 * (l16 & 3);
        const int pr_off = l32 * PSTR + 16 * hh;
        // Tiles from this one on hold keys that some row of the workgroup does not see.  Such a row's p is 0 there, but 0 times
        // an infinity or NaN in a later position (an unused one, another token's) would reach its output.  A key with one has
        // no finite score, which the scores waves look for in these tiles; from there on V enters the product with infinities
        // and NaN as 0.  (Done to every such tile without the look, four layers of 3 x 1021 rows took 600 us instead of
        // 575.)  A row that does see such a key is all NaN from its p if the score is +inf or NaN; if it is -inf, p is 0 and
        // only the columns in which the key is not finite are NaN (0 times infinity): they are set when the rows leave.
        bf16x8 pa[2][2];
        s16x4 vq[2][4][2];
        auto finite_v = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int e = 0; e < 4; ++e) vq[s][nb][u][e] = (vq[s][nb][u][e] & 0x7f80) == 0x7f80 ? (short)0 : vq[s][nb][u][e];
        };
        auto read_v = [&](int t, int s, int nb) __attribute__((always_inline)) {
            const unsigned char *tb = tbuf + (t & (kDenseRing - 1)) * TBUFB + tr_off + 16 * s * ROWB + 64 * nb;
#pragma unroll
            for (int u = 0; u < 2; ++u) vq[s][nb][u] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(tb + u * ROWB));
        };
        auto read_p = [&](int t, int s) __attribute__((always_inline)) {
            const unsigned char *pb = pbuf + (t & 1) * PBUFB + pr_off;
#pragma unroll
            for (int r = 0; r < 2; ++r) pa[s][r] = *(const bf16x8 *)(pb + 32 * r * PSTR + 32 * s);
        };
        // Step i: output product of tile i - 2 (kMma) in two steps of 16 keys, from operands read a step ago; those of tile i - 1
        // (kRead: tile t of block k) take their registers, tile i + 2 goes to LDS and tile i + 3 into its registers
        int i = 1;
        Block k = first;
        auto step = [&](int t, auto mma_c, auto read_c) __attribute__((always_inline)) {
            constexpr bool kMma = decltype(mma_c)::value, kRead = decltype(read_c)::value;
            const int flag = kRead ? moved[(i - 1) & 1] : 0;
            const unsigned short *src = tile_src();
            __builtin_amdgcn_sched_barrier(0);
            unroll<8>([&](auto u_c) __attribute__((always_inline)) {
                constexpr int u = decltype(u_c)::value, s = u >> 2, nb = u & 3;
                if constexpr (kMma) {
                    const s16x8 v = {vq[s][nb][0][0], vq[s][nb][0][1], vq[s][nb][0][2], vq[s][nb][0][3], vq[s][nb][1][0], vq[s][nb][1][1], vq[s][nb][1][2], vq[s][nb][1][3]};
#pragma unroll
                    for (int r = 0; r < 2; ++r)
                        o_acc[r][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, v), pa[s][r], o_acc[r][nb], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (kRead) {
                    read_v(i - 1, s, nb);
                    if constexpr (nb == 3) read_p(i - 1, s);
                }
#pragma unroll
                for (int c = u; c < (u == 7 ? 9 : u + 1); ++c) {
                    store(i + 2, c, 1);
                    cur[c] = *(const u32x4 *)(src + 64 * c);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            if (kRead && t >= k.t_edge && __builtin_amdgcn_readfirstlane(moved[2 + k.odd])) finite_v();
            if (kRead && __builtin_amdgcn_readfirstlane(flag)) {       // see above
                __syncthreads();
                if constexpr (kMma) {
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const float f = fac[32 * r + l32];
#pragma unroll
                        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                            for (int e = 0; e < 16; ++e) o_acc[r][nb][e] *= f;
                    }
                }
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const float f = fac[kDenseRows * (1 + s) + 32 * r + l32];
#pragma unroll
                        for (int e = 0; e < 8; ++e) pa[s][r][e] = (__bf16)((float)pa[s][r][e] * f);
                    }
            }
            ++i;
        };
        // Outputs of block k, in halves of 32 rows, through the rows of the ring that this wave fills in this step (nobody else
        // touches them now): a store covers whole lines.  (O is 16-byte aligned: dense_output())
        auto finish = [&]() __attribute__((always_inline)) {
            int ln = lane;                                // (kept from before the loop, what follows from it would be spilled)
            asm volatile("" : "+v"(ln));
            const int c32 = ln & 31, half = ln >> 5;
            unsigned char *ob = tbuf + ((i + 2) & (kDenseRing - 1)) * TBUFB + 8 * w * ROWB;
            const int64_t row0 = (int64_t)k.b * a.Tq * a.H_q + k.R0;
            __bf16 *const o_l = (__bf16 *)(MULTI ? a.Os[k.layer] : a.O);
            const bool odd_keys = __builtin_amdgcn_readfirstlane(moved[2 + k.odd]);    // (rare: see finite_v above)
            unroll<2>([&](auto r_c) __attribute__((always_inline)) {
                constexpr int r = decltype(r_c)::value;
                const float l = fac[32 * r + c32] + fac[kDenseRows + 32 * r + c32];
                const float inv = l > 0.f ? __builtin_amdgcn_rcpf(l) : 0.f;
                // (in 64 bits: the reference of 32 keys leaves a larger logarithm, and so a coarser sum, than that of the row form's 64)
                if (a.lse && w == 0 && half == 0 && k.R0 + 32 * r + c32 < k.n_rows)
                    a.lse[row0 + 32 * r + c32] =
                        l > 0.f ? (float)(((double)fac[2 * kDenseRows + 32 * r + c32] + (double)__builtin_log2f(l)) * 0.6931471805599453) : -INFINITY;
                unroll<16>([&](auto q_c) __attribute__((always_inline)) {
                    constexpr int nb = decltype(q_c)::value >> 2, qd = decltype(q_c)::value & 3;
                    s16x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = __builtin_bit_cast(short, (__bf16)(o_acc[r][nb][4 * qd + e] * inv));
                    *(s16x4 *)(ob + c32 * OSTR + 2 * (32 * nb + 8 * qd + 4 * half)) = o;
                });
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int row = 4 * j + (ln >> 4), R = k.R0 + 32 * r + row;
                    u32x4 o = *(const u32x4 *)(ob + row * OSTR + 16 * (ln & 15));
                    if (odd_keys && R < k.n_rows) {
                        const unsigned short *v0 = (const unsigned short *)(MULTI ? a.KVs[k.layer] : a.KV) + 128 * w + 8 * (ln & 15);
                        for (int key = k.t_edge * kDenseTile; key <= da.pos0 + R / a.H_q; ++key) {
                            const int64_t at = PG && a.pv.page_table ? paged_row(a.pv, k.b, key) : (int64_t)k.b * a.Lk + key;
                            const u32x4 v = *(const u32x4 *)(v0 + at * a.row_elems);
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                if ((v[e] & 0x7f80u) == 0x7f80u) o[e] |= 0x7fc0u;
                                if ((v[e] & 0x7f800000u) == 0x7f800000u) o[e] |= 0x7fc00000u;
                            }
                        }
                    }
                    if (R < k.n_rows) *(u32x4 *)(o_l + (row0 + 32 * r + row) * D_V + 128 * w + 8 * (ln & 15)) = o;
                }
            });
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                    for (int e = 0; e < 16; ++e) o_acc[r][nb][e] = 0.f;
        };
        constexpr std::true_type T{};
        constexpr std::false_type F{};
        __syncthreads();
        step(0, F, F);
        __syncthreads();
        step(0, F, F);
        __syncthreads();
#pragma unroll 1
        for (;;) {
            // tile i - 2 is the second one of Q
            step(0, F, T);
            __syncthreads();
#pragma unroll 1
            for (int t = 1; t < k.nt; ++t) {
                step(t, T, T);
                __syncthreads();
            }
            step(0, T, F);
            __syncthreads();
            const Block nx = open(k.n + 1, k.odd ^ 1);    // tile i - 2 is its first one of Q
            finish();
            if (nx.n == n_list) return;
            k = nx;
            step(0, F, F);
            __syncthreads();
        }
    }
}

template <bool PG>
__global__ __launch_bounds__(512, 2) void attn_dense_kernel(AttnArgs a, DenseArgs da, DenseShape ds)
{
    dense_rows<PG, false>(a, da, ds);
}

template <bool PG>
__global__ __launch_bounds__(512, 2) void attn_layers_dense_kernel(AttnArgs a, DenseArgs da, DenseShape ds)
{
    dense_rows<PG, true>(a, da, ds);
}

// ---- stream form (unsplit rows of 576/512 features) ----------------------------------------------------------------
// One workgroup of eight waves per CU walks queries q0, q0 + gridDim.x, ... as one stream of granules of 32 rows: the 32 heads of
// a query's Q, then its selected rows, then the next query's Q.  A granule is gathered eight lanes to a 128-byte line and passes through
// a ring of four LDS buffers; one barrier per granule ("period").  Two roles, one wave of each per SIMD:
//   scores   waves 0-3 in two pairs, which take alternate granules and have two periods for one.  A wave holds all of Q (144
//            registers, read from Q's granule) and scores 16 rows of it for 32 heads: every score operand crosses LDS once.
//            Softmax against a reference that moves only when a score exceeds it by 2^kLazyLog2; P and the reference to LDS
//   output   waves 4-7, value columns 128 w .. 128 w + 127, O^T += V^T P^T: a lane owns a head, so that references, factors
//            and row sums are a lane's own.  They also bring the granules: two in registers, in flight for two periods, the
//            ids six periods ahead
// In period p granule p + 1 goes to LDS, p and p - 1 are scored, V and P of p - 2 go to registers and the product of p - 3 is
// taken from registers: whatever a wave waits for was requested a period ago, and Q of the next query, its first rows and the
// outputs of the last one take their places in the stream.
// What bounds it.  A wave per SIMD and role issues an instruction every 4 to 5 clocks at best, and what a unit has not taken
// blocks the ones behind it: with every phase in each of four waves (the row-slab form) 32 rows took 1950 clocks, and only the gather, the
// LDS traffic or the MFMAs of a phase were busy at a time.  Here the output waves alone take 1000 clocks, the scores waves alone 1000, both
// 1240, of which the matrix cores are busy 540, and the clock is 1.8 to 1.9 GHz; with rows from beyond L2 (131072 of them, 7.1 TB/s
// across its boundary) 1430 clocks.  2048 queries x 2048 of 32768 rows, 32 heads: 450 us in chains of the row-slab form, 355 here.  Ids requested two periods ahead, addresses worked out at the
// start of a period, outputs stored straight from the accumulators: 20 % slower together.  Three granules in flight need more
// registers than there are and gain nothing where two are enough; with 131072 rows (HBM) both forms take the gather's time.
constexpr int kGranule = 32;                 // selected rows that reach LDS together
constexpr int kStreamRing = 4;               // of them resident
constexpr int kStreamDepth = 2;              // of them in registers on their way there
constexpr int kProbsQueries = 1024;          // PROBS: queries of a workgroup, at most
constexpr int kStreamIds = 4;                // periods between the request of a granule's ids and that of its rows

// PG: the KV cache may be ragged and / or paged.
// MULTI: a.n_layers layers in one launch, or the last rows of several sequences (a.row_gap): a query's place in the tensors
// is then not its number.
// REST: the rows of all sequences of one or more layers (RestArgs) behind those that the dense form has taken.  How many that
// are is device data, so the workgroups, as many as for all rows, find out first and share what is left (one round trip to
// memory, about 1 us).
// PROBS: the scores waves write each row's probability, summed over the heads, with the log-sum-exps that an attention launch
// has left (a.lse) instead of P, to a.O as fp32 [B,Tq,k_sel]; the output waves only bring the granules.  A workgroup per query
// whose four waves gathered and scored 16 rows each on their own loaded Q four times over (36 KB in pieces of 64 bytes) and took 442 us
// for 4096 causal rows, 350 here; 4096 x 2048 of 32768 rows 893 and 589, one query 51 and 32.
template <bool PG, bool MULTI, bool REST, bool PROBS>
__global__ __launch_bounds__(512, 2) void attn_stream_kernel(AttnArgs a, RestArgs ra)
{
    constexpr int D_QK = 576, D_V = 512;
    constexpr int KS = D_QK / 32, KS1 = 12;               // contraction steps; those of a granule's first period (8 .. 14: within 2 %)
    constexpr int ROWB = D_QK * 2 + kSlabPad, GB = kGranule * ROWB;
    constexpr int PSTR = kGranule * 2 + 16, PB = 32 * PSTR;
    constexpr int RING = 6;                               // A-operand reads in flight
    constexpr int D = kStreamDepth, DI = kStreamIds;      // (a set of registers is that of the granule's number modulo D, DI)
    static_assert(DI % D == 0, "the loop is unrolled by DI");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char *tbuf = smem;                           // [kStreamRing][32][ROWB]
    unsigned char *pbuf = smem + kStreamRing * GB;        // [2][32 heads][PSTR]
    float *lsum = (float *)(pbuf + 2 * PB);               // [2 by query][32 heads][4 waves] row sums
    float *lref = lsum + 2 * 32 * 4;                      // [2][32][4] and the references they have
    float *mbuf = lref + 2 * 32 * 4;                      // [2 by granule][32 heads][2 key halves] references of P
    unsigned char *filled = (unsigned char *)(mbuf + 2 * 32 * 2);            // [kStreamRing][32 rows][8] 1: the slot holds an entry

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, l32 = lane & 31, hh = lane >> 5, g = lane >> 4;
    const int w = wave & 3;
    // queries of the workgroup: q0, q0 + gridDim.x, ...
    const unsigned nq_layer = (unsigned)(a.B * a.Tq);
    unsigned nq = MULTI ? nq_layer * a.n_layers : nq_layer;
    // REST: numbers of the sequences' first queries, [n_jobs * B] and their total
    unsigned *const start = (unsigned *)(filled + kStreamRing * kGranule * 8);
    const int n_seq = REST ? ra.n_jobs * a.B : 0;
    if (REST && n_seq == 1) {                             // (every wave for itself)
        nq = (unsigned)max(0, ra.n_rows - __builtin_amdgcn_readfirstlane(min(lead_rows(ra.lead[0], ra.n_chunks), lead_rows(ra.lead2[0], ra.n_chunks))));
    } else if constexpr (REST) {
        // lanes to a sequence: 64 for up to 8 of them, down to 8
        const int bits = n_seq <= 8 ? 6 : (n_seq <= 16 ? 5 : (n_seq <= 32 ? 4 : 3)), per = 1 << bits;
        for (int s = tid >> bits; s < n_seq; s += 512 >> bits) {
            const int job = s / a.B;
            const int64_t o = (int64_t)(s - job * a.B) * ra.n_chunks;
            int t0 = kLeadChunk * ra.n_chunks;            // the first row that is not a leading one
#pragma unroll 4
            for (int c = tid & (per - 1); c < ra.n_chunks; c += per) {
                const int n = min(ra.lead[job][o + c], ra.lead2[job][o + c]);
                t0 = n < kLeadChunk ? min(t0, kLeadChunk * c + n) : t0;
            }
            for (int x = per >> 1; x; x >>= 1) t0 = min(t0, __shfl_xor(t0, x));
            if ((tid & (per - 1)) == 0) start[s] = (unsigned)(ra.n_rows - min(t0, ra.n_rows));
        }
        __syncthreads();
        unsigned carry = 0;
        if (wave == 0) {
            for (int s0 = 0; s0 < n_seq; s0 += 64) {
                const unsigned n = s0 + lane < n_seq ? start[s0 + lane] : 0u, incl = wave_incl_scan(n);
                if (s0 + lane < n_seq) start[s0 + lane] = carry + incl - n;
                carry += (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
            }
            if (lane == 0) start[n_seq] = carry;
        }
        __syncthreads();
        nq = __builtin_amdgcn_readfirstlane(start[n_seq]);
    }
    unsigned q0 = blockIdx.x;
    if ((gridDim.x & 7u) == 0) q0 = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    // (PROBS: every other round the other way round: causal rows hold more and more entries, 8 % more in the last workgroup's of a round)
    auto query = [&](int n) -> unsigned { return (unsigned)n * gridDim.x + (PROBS && (n & 1) ? gridDim.x - 1 - q0 : q0); };
    const int n_mine = (int)(nq / gridDim.x) + (query((int)(nq / gridDim.x)) < nq);
    if (n_mine == 0) return;
    int *const counts = (int *)pbuf;                      // PROBS: [n_mine] granules of the queries
    auto granules = [&](int i) -> int {                   // of the workgroup's query i, at least one
        if constexpr (PROBS) return __builtin_amdgcn_readfirstlane(counts[i]);
        int n = a.k_sel;
        if (a.causal_pos0 >= 0) {
            const unsigned gq = query(i);
            const int64_t held = a.causal_pos0 + (MULTI ? gq % nq_layer : gq) % (unsigned)a.Tq + 1;
            if (held < n) n = (int)held;
        }
        return max(1, (n + kGranule - 1) / kGranule);
    };
    if constexpr (PROBS) {
        // Granules behind the last selected row hold nothing: their zeros are written here (512 entries at a time in flight)
        for (int i = wave; i < n_mine; i += 8) {
            const int32_t *idx_row = a.idx + (int64_t)query(i) * a.k_sel;
            float *out = (float *)a.O + (int64_t)query(i) * a.k_sel;
            int n = 1;
            for (int s0 = 0; s0 < a.k_sel; s0 += 64 * 8) {
                int32_t v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = idx_row[min(s0 + 64 * u + lane, a.k_sel - 1)];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const unsigned long long some = __ballot(v[u] >= 0 && s0 + 64 * u + lane < a.k_sel);
                    if (some != 0ull) n = (s0 + 64 * u) / kGranule + (some >> kGranule ? 2 : 1);
                }
            }
            if (lane == 0) counts[i] = n;
            for (int k = kGranule * n + lane; k < a.k_sel; k += 64) out[k] = 0.f;
        }
        __syncthreads();
    }

    if (wave < 4) {
        const int pair = w >> 1, kh = w & 1;
        bf16x8 qv[KS][2];
        auto load_q = [&](int at) __attribute__((always_inline)) {
            const unsigned char *qr = tbuf + (at & (kStreamRing - 1)) * GB + l16 * ROWB + 16 * g;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int r = 0; r < 2; ++r) qv[ks][r] = *(const bf16x8 *)(qr + 16 * r * ROWB + 64 * ks);
        };
        const int ka_off = (16 * kh + (PROBS ? l16 : dense_row(l16))) * ROWB + 16 * g;
        const int pw_off = l16 * PSTR + 32 * kh + 8 * g;
        float m_c[2] = {-INFINITY, -INFINITY}, l_own[2] = {0.f, 0.f};
        auto publish = [&](int n) __attribute__((always_inline)) {       // row sums of query n, and a new start
            float *ls = lsum + (n & 1) * 128 + w, *lr = lref + (n & 1) * 128 + w;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const float l = xsum16_32(l_own[r]);
                if (g == 0) {
                    ls[4 * (16 * r + l16)] = l;
                    lr[4 * (16 * r + l16)] = m_c[r];
                }
                m_c[r] = -INFINITY;
                l_own[r] = 0.f;
            }
        };
        const float inv_h = 1.f / (float)a.H_q;
        bf16x8 ka[RING];
        f32x4 s4[2], odd[2];                              // two accumulation chains: half of the roundings in one
        auto steps = [&](const unsigned char *tb, auto k0_c, auto k1_c) __attribute__((always_inline)) {
            constexpr int k0 = decltype(k0_c)::value, k1 = decltype(k1_c)::value;
            unroll<k1 - k0>([&](auto i_c) __attribute__((always_inline)) {
                constexpr int ks = k0 + decltype(i_c)::value;
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    f32x4 &c = ks % 2 ? odd[r] : s4[r];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[ks % RING], qv[ks][r], ks < 2 ? f32x4{0.f, 0.f, 0.f, 0.f} : c, 0, 0, 0);
                }
                if constexpr (ks + RING < KS) ka[ks % RING] = *(const bf16x8 *)(tb + 64 * (ks + RING));
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        constexpr std::integral_constant<int, 0> c0{};
        constexpr std::integral_constant<int, KS1> c1{};
        constexpr std::integral_constant<int, KS> c2{};

        __syncthreads();                                  // period -1
        if (pair) __syncthreads();                        // period 0
        int at_q = 0;                                     // the query's Q in the stream, its granules behind it
        // PROBS: log-sum-exps of heads l16 and 16 + l16 (a head that is not there counts nothing), the next query's on their way
        float lse2[2] = {INFINITY, INFINITY};
        auto load_lse = [&](int n, float (&l)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 2; ++r)
                l[r] = 16 * r + l16 < a.H_q ? a.lse[(int64_t)query(n) * a.H_q + 16 * r + l16] * 1.4426950408889634f : INFINITY;
        };
        float lse_n[2];
        if constexpr (PROBS) load_lse(0, lse_n);
#pragma unroll 1
        for (int n = 0; n < n_mine; ++n) {
            const int last = at_q + granules(n);
            const bool own = ((at_q ^ pair) & 1) == 0;    // Q takes the place of a granule of this pair
            if constexpr (PROBS) {
                lse2[0] = lse_n[0];
                lse2[1] = lse_n[1];
                if (n + 1 < n_mine) load_lse(n + 1, lse_n);
            } else {
                if (n > 0) publish(n - 1);
            }
            load_q(at_q);
            if (own) {
                __syncthreads();
                __syncthreads();
            }
#pragma unroll 1
            for (int at = at_q + (own ? 2 : 1); at <= last; at += 2) {
                const unsigned char *tb = tbuf + (at & (kStreamRing - 1)) * GB + ka_off;
#pragma unroll
                for (int r = 0; r < RING; ++r) ka[r] = *(const bf16x8 *)(tb + 64 * r);
                __builtin_amdgcn_sched_barrier(0);
                steps(tb, c0, c1);
                __syncthreads();
                typedef __attribute__((ext_vector_type(2))) float f32x2;
                const int vm = *(const int *)(filled + (at & (kStreamRing - 1)) * 256 + (16 * kh + l16) * 8);
                f32x2 mk[2];
#pragma unroll
                for (int r = 0; r < 2 && !PROBS; ++r) mk[r] = *(const f32x2 *)(mbuf + ((at - 1) & 1) * 64 + 2 * (16 * r + l16));
                __builtin_amdgcn_sched_barrier(0);
                steps(tb, c1, c2);
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int i = 0; i < 4; ++i) s4[r][i] += odd[r][i];
                const unsigned rows = (unsigned)__ballot(vm != 0) & 0xFFFFu;
                if constexpr (PROBS) {
                    // lane: rows 4 g + i of the half, heads l16 and 16 + l16
                    float p[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float sum = 0.f;
#pragma unroll
                        for (int r = 0; r < 2; ++r) {
                            const float e = fast_exp2(__builtin_fmaf(s4[r][i], a.scale_log2e, -lse2[r]));
                            sum += (rows >> (4 * g + i) & 1u) && 16 * r + l16 < a.H_q ? e : 0.f;
                        }
                        p[i] = row16_sum(sum);            // lane 15 of the 16: the sum over the heads
                    }
                    if (l16 == 15) {
                        const int k = kGranule * (at - at_q - 1) + 16 * kh + 4 * g;
                        float *out = (float *)a.O + (int64_t)query(n) * a.k_sel + k;
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (k + i < a.k_sel) out[i] = p[i] * inv_h;
                    }
                    __syncthreads();
                    continue;
                }
                if (rows != 0xFFFFu) {
                    const unsigned mine = rows >> (8 * (g >> 1) + (g & 1));    // the lane's keys are two apart
#pragma unroll
                    for (int r = 0; r < 2; ++r)
#pragma unroll
                        for (int i = 0; i < 4; ++i) s4[r][i] = (mine >> 2 * i) & 1u ? s4[r][i] : -INFINITY;
                }
                float m_use[2], mx[2];
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    m_use[r] = at - 1 > at_q ? fmaxf(m_c[r], fmaxf(mk[r][0], mk[r][1])) : m_c[r];
                    mx[r] = fmaxf(fmaxf(s4[r][0], s4[r][1]), fmaxf(s4[r][2], s4[r][3])) * a.scale_log2e;
                }
                // A pair's first granule takes any larger score for its reference, so that the common one is the largest of 64 rows, as
                // in the row-slab form: a row's largest p is then 1 and not rounded the more often.  (Peaked rows of 100 entries: relative
                // distance from 64 bits 0.00188 with the largest of 32, 0.00181 with this.  It moves the accumulators once more per query: four layers of
                // 440 causal rows 63.6 -> 65.7 us, rows of 2048 entries within the runs.)
                const float lazy = m_c[0] == -INFINITY ? 0.f : kLazyLog2;
                if (__ballot(mx[0] > m_use[0] + lazy || mx[1] > m_use[1] + lazy) != 0ull) {
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        mx[r] = xmax16_32(mx[r]);
                        m_use[r] = mx[r] > m_use[r] + lazy ? mx[r] : m_use[r];
                    }
                }
                if (__ballot(m_use[0] != m_c[0] || m_use[1] != m_c[1]) != 0ull) {
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        l_own[r] *= m_use[r] == m_c[r] ? 1.f : fast_exp2(m_c[r] - m_use[r]);
                        m_c[r] = m_use[r];
                    }
                }
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const float m_safe = m_c[r] == -INFINITY ? 0.f : m_c[r];   // (no key so far: every p is 2^-inf = 0)
                    s16x4 pk;
                    float p[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        p[i] = fast_exp2(__builtin_fmaf(s4[r][i], a.scale_log2e, -m_safe));
                        pk[i] = __builtin_bit_cast(short, (__bf16)p[i]);
                    }
                    *(s16x4 *)(pbuf + (at & 1) * PB + pw_off + 16 * r * PSTR) = pk;
                    if (g == 0) mbuf[(at & 1) * 64 + 2 * (16 * r + l16) + kh] = m_c[r];
                    l_own[r] += (p[0] + p[1]) + (p[2] + p[3]);
                }
                __syncthreads();
            }
            at_q = last + 1;
        }
        if constexpr (!PROBS) publish(n_mine - 1);
        // as many barriers as the output waves have: those of the periods -1 .. at_q + 3, in whole rounds of DI
        const int done = at_q + (((at_q ^ pair) & 1) == 0 ? 1 : 2);
        for (int i = done; i < (at_q + 4 + DI) / DI * DI; ++i) __syncthreads();
        return;
    }

    // ---- output waves ----
    const int gr = lane >> 3, gp = lane & 7;              // gather role: row 8 w + gr, 16-byte piece
    const int my_row = 8 * w + gr;
    struct Place { int n, ng; bool is_q; const int32_t *idx; const unsigned short *kv, *q, *src; int len, b; } pl;
    auto tensor_row = [&](unsigned gq, int &layer, int &b) __attribute__((always_inline)) -> int64_t {
        if constexpr (REST) {
            if (n_seq == 1) {                             // (a look at LDS per query: 333 us for 2048 rows, 327 without)
                layer = b = 0;
                return ra.n_rows - (int)(nq - gq);
            }
            int s = -1;                                   // the last sequence that starts at gq or before it
            for (int s0 = 0; s0 < n_seq; s0 += 64) {
                const int n = __popcll(__ballot(s0 + lane < n_seq && start[min(s0 + lane, n_seq)] <= gq));
                s += n;
                if (n < 64) break;
            }
            layer = s / a.B;
            b = s - layer * a.B;
            return (int64_t)b * a.Tq + ra.n_rows - (int)(__builtin_amdgcn_readfirstlane(start[s + 1]) - gq);
        }
        layer = MULTI ? layer_of(a, gq) : 0;
        const unsigned qq = MULTI ? gq - layer * nq_layer : gq;
        b = (int)(qq / (unsigned)a.Tq);
        return MULTI ? (int64_t)qq + (int64_t)b * a.row_gap : (int64_t)qq;
    };
    auto open = [&](int i) __attribute__((always_inline)) {
        const unsigned gq = query(i);
        int layer;
        const int64_t row = tensor_row(gq, layer, pl.b);
        const void *idx_l = a.idx, *q_l = a.Q, *kv_l = a.KV;
        if (MULTI || (REST && n_seq > 1)) {
            if (REST) asm volatile("");                   // (a branch: the loads' latency is not for one sequence)
            if (REST) idx_l = ra.idx[layer];
            q_l = a.Qs[layer];
            kv_l = a.KVs[layer];
        }
        pl.idx = (const int32_t *)idx_l + row * a.k_sel;
        pl.q = (const unsigned short *)q_l + row * a.H_q * D_QK;
        pl.kv = (const unsigned short *)kv_l + (PG && a.pv.page_table ? 0 : (int64_t)pl.b * a.Lk * a.row_elems);
        pl.len = PG && a.pv.seq_lens ? max(0, min(load_uniform(a.pv.seq_lens + pl.b), a.Lk)) : a.Lk;     // (ids are compared unsigned)
        pl.ng = granules(i);
    };
    pl.n = 0;
    open(0);
    pl.is_q = true;
    pl.src = pl.q;
    // per register set: ids of a granule and what they belong to
    int32_t ids[DI];
    const unsigned short *base[DI];
    int n_slots[DI], len[DI], seq[DI];                    // n_slots < 0: the rows are Q
    int64_t prow[DI];
    int ok_pg[DI];
    const unsigned short *base_pg[DI];
    int n_slots_pg[DI];
    int vm[D];
    u32x4 cur[D][9];
    // the place: granules of the query behind this one, the slots left, the byte of the index row that the lane's slot starts at
    int left = 0, n_run = -1;
    unsigned slot_b = 4 * my_row;
    const unsigned last_b = 4 * (a.k_sel - 1);
    auto request = [&](auto s_c) __attribute__((always_inline)) {
        constexpr int s = decltype(s_c)::value;
        ids[s] = *(const int32_t *)((const char *)pl.idx + min(slot_b, last_b));
        base[s] = pl.src;
        n_slots[s] = n_run;
        len[s] = pl.len;
        seq[s] = pl.b;
    };
    auto advance = [&]() __attribute__((always_inline)) {
        n_run -= kGranule;
        slot_b += 4 * kGranule;
        if (__builtin_expect(--left < 0, 0)) {
            slot_b = 4 * my_row;
            if (pl.is_q && pl.n < n_mine) {               // behind Q: the query's granules
                pl.is_q = false;
                pl.src = pl.kv;
                left = pl.ng - 1;
                n_run = a.k_sel;
            } else {                                      // the next query's Q; at the end of the stream the last one's, for nobody
                if (pl.n < n_mine) ++pl.n;
                if (pl.n < n_mine) open(pl.n);
                pl.is_q = true;
                pl.src = pl.q;
                left = 0;
                n_run = -1;
            }
        }
    };
    auto take = [&](auto s_c) __attribute__((always_inline)) {
        request(s_c);
        advance();
    };
    const int q_row = min(my_row, a.H_q - 1);
    // the ids of a set -> what gather() needs (paged: a table entry per row, requested here)
    auto place = [&](auto s_c) __attribute__((always_inline)) {
        constexpr int s = decltype(s_c)::value;
        if constexpr (PG) {
            const int32_t v = ids[s];
            const bool ok = (int)(my_row < n_slots[s]) & (int)((unsigned)v < (unsigned)len[s]);
            // empty slots read row 0 of the cache (never a page-table entry: the sequence may own no page)
            int64_t row = ok ? v : 0;
            if (a.pv.page_table && ok) row = paged_row(a.pv, seq[s], v);
            prow[s] = row;
            ok_pg[s] = ok;
            base_pg[s] = base[s];
            n_slots_pg[s] = n_slots[s];
        }
    };
    auto gather_src = [&](auto s_c) __attribute__((always_inline)) -> uint64_t {
        constexpr int s = decltype(s_c)::value;
        const bool isq = (PG ? n_slots_pg[s] : n_slots[s]) < 0;
        const int stride = isq ? D_QK : a.row_elems;
        if constexpr (PG) {
            vm[s % D] = ok_pg[s];
            return (uint64_t)base_pg[s] + ((isq ? (int64_t)q_row : prow[s]) * stride + 8 * gp) * 2;
        } else {
            const int32_t v = ids[s];
            const bool ok = (int)(my_row < n_slots[s]) & (int)((unsigned)v < (unsigned)a.Lk);
            vm[s % D] = ok;
            const int row = isq ? q_row : (ok ? v : 0);
            return (uint64_t)base[s] + ((uint64_t)(unsigned)row * (unsigned)(2 * stride) + 16 * gp);
        }
    };
    auto load = [&](auto s_c, uint64_t from, int c0, int n) __attribute__((always_inline)) {
        constexpr int s = decltype(s_c)::value;
#pragma unroll
        for (int c = c0; c < c0 + n; ++c) cur[s][c] = *(const __attribute__((address_space(1))) u32x4 *)(from + 128 * c);
    };
    // Granules 0 .. D - 1 on their way, the source of granule D, the ids behind; requested in the order that the periods
    // below have, so that waits by position find the same queue behind the first period as behind any other.
    uint64_t src, first[D];
    unroll<DI>([&](auto s_c) __attribute__((always_inline)) { take(s_c); });
    if constexpr (PG) unroll<DI>([&](auto s_c) __attribute__((always_inline)) {
        place(s_c);
        take(s_c);
    });
    unroll<D>([&](auto s_c) __attribute__((always_inline)) {
        constexpr int s = decltype(s_c)::value;
        __builtin_amdgcn_sched_barrier(0);
        first[s] = gather_src(s_c);
        place(s_c);
        load(s_c, first[s], 0, 5);
        __builtin_amdgcn_sched_barrier(0);
        take(s_c);
        __builtin_amdgcn_sched_barrier(0);
        load(s_c, first[s], 5, 4);
        __builtin_amdgcn_sched_barrier(0);
    });
    src = gather_src(std::integral_constant<int, D % DI>{});
    place(std::integral_constant<int, D % DI>{});
    take(std::integral_constant<int, D % DI>{});

    f32x16 o_acc[4];                                      // O^T: columns 32 nb .., the lane's row is head l32
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int e = 0; e < 16; ++e) o_acc[nb][e] = 0.f;
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const int st_off = my_row * ROWB + 16 * gp;
    const int tr_off = (8 * hh + 2 * (l16 >> 2)) * ROWB + 256 * w + 32 * (g & 1) + 8 * (l16 & 3);
    const int pr_off = l32 * PSTR + 16 * hh;
    bf16x8 pa[2];
    s16x4 vq[2][4][2];
    float m_c = -INFINITY;                                // reference of the accumulators
    int m = 0, to_q = 4;                                  // Q seen by the product so far, periods until the next one

    // Outputs of a query, through the rows of the ring that this wave is about to fill (nobody else touches them in this
    // period): lanes of a store then cover whole lines.  Straight from the accumulators (8 bytes of 32 rows in each of 16
    // stores) a query's outputs kept the four waves for 5000 clocks.
    auto finish = [&](int slot) __attribute__((always_inline)) {
        int ln = lane;                                    // (kept from before the loop, what follows from it would be spilled)
        asm volatile("" : "+v"(ln));
        const int row_l = ln & 31, half = ln >> 5;
        const f32x4 ls = *(const f32x4 *)(lsum + ((m - 1) & 1) * 128 + 4 * row_l), lr = *(const f32x4 *)(lref + ((m - 1) & 1) * 128 + 4 * row_l);
        float l = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) l += lr[i] == -INFINITY ? 0.f : ls[i] * fast_exp2(lr[i] - m_c);
        const float inv = l > 0.f ? __builtin_amdgcn_rcpf(l) : 0.f;
        int layer, b;
        const unsigned gq = query(m - 1);
        const int64_t row = tensor_row(gq, layer, b);
        if (w == 0 && half == 0 && row_l < a.H_q && a.lse) {
            // (in 64 bits: the reference of 16 keys leaves a larger logarithm, and so a coarser sum, than that of more)
            a.lse[row * a.H_q + row_l] = l > 0.f ? (float)(((double)m_c + (double)__builtin_log2f(l)) * 0.6931471805599453) : -INFINITY;
        }
        constexpr int OSTR = 256 + 16;
        static_assert(32 * OSTR <= 8 * ROWB, "32 heads of 256 bytes");
        unsigned char *ob = tbuf + slot * GB + 8 * w * ROWB;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                s16x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = __builtin_bit_cast(short, (__bf16)(o_acc[nb][4 * qd + e] * inv));
                *(s16x4 *)(ob + row_l * OSTR + (32 * nb + 8 * qd + 4 * half) * 2) = v;
            }
        void *o_l = a.O;
        if (MULTI || (REST && n_seq > 1)) {
            if (REST) asm volatile("");
            o_l = a.Os[layer];
        }
        unsigned short *const o = (unsigned short *)o_l + row * a.H_q * D_V + 128 * w;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int head = 4 * k + (ln >> 4);
            const u32x4 v = *(const u32x4 *)(ob + head * OSTR + 16 * (ln & 15));
            unsigned short *d = o + head * D_V + 8 * (ln & 15);
            if (head < a.H_q) {
                if ((uintptr_t)o % 16 == 0) {
                    *(u32x4 *)d = v;
                } else {                                  // (any address of a bf16 will do)
#pragma unroll
                    for (int e = 0; e < 8; ++e) d[e] = (unsigned short)(v[e / 2] >> 16 * (e & 1));
                }
            }
        }
    };

    // Period p: output product of granule p - 3 from operands read a period ago; those of granule p - 2 take their
    // registers, granule p + 1 goes to LDS and granule p + 1 + D into its registers.  Where granule p - 3 is Q, the outputs of
    // the query before it leave first and the product, of nothing, is dropped.  The source of the next period's gather is
    // worked out here, between the MFMAs.  A wave issues an instruction every 4 to 5 clocks at best and this one has the most
    // of them: unrolled over the ring's buffers, so that their addresses are constants.
    static_assert(DI == kStreamRing, "a period's buffers are known where it is unrolled");
    auto pin = [](auto &x) __attribute__((always_inline)) { asm volatile("" : "+v"(x)); };   // worked out here, not where it is used
    int st[2] = {st_off, st_off + 2 * GB}, vb[2] = {tr_off, tr_off + 2 * GB};     // (offsets have 16 bits)
    pin(st[1]);
    pin(vb[1]);
    auto period = [&](auto s_c) __attribute__((always_inline)) {
        constexpr int g1 = decltype(s_c)::value;          // granule p + 1 modulo DI
        constexpr int s = g1 % D, s_next = (s + 1) % D, g2 = (g1 + 1) % DI;      // g2: granule p - 2
        constexpr std::integral_constant<int, (g1 + 1 + D) % DI> s1{};
        if (__builtin_expect(to_q == 0, 0)) {
            if (!PROBS && m > 0) finish(g1);
        }
        f32x2 mj;
        uint64_t src1 = 0;
        bool moved = false;
        unroll<8>([&](auto i_c) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value, h = i >> 2, nb = i & 3;
            if constexpr (!PROBS) {
                const s16x8 v = {vq[h][nb][0][0], vq[h][nb][0][1], vq[h][nb][0][2], vq[h][nb][0][3], vq[h][nb][1][0], vq[h][nb][1][1], vq[h][nb][1][2], vq[h][nb][1][3]};
                o_acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, v), pa[h], o_acc[nb], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    vq[h][nb][u] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(tbuf + vb[g2 / 2] + (g2 % 2) * GB + 16 * h * ROWB + 64 * nb + u * ROWB));
                if constexpr (nb == 3) pa[h] = *(const bf16x8 *)(pbuf + pr_off + (g2 % 2) * PB + 32 * h);
                if constexpr (i == 0) mj = *(const f32x2 *)(mbuf + (g2 % 2) * 64 + 2 * l32);
            }
#pragma unroll
            for (int c = i; c < (i == 7 ? 9 : i + 1); ++c) *(u32x4 *)(tbuf + st[g1 / 2] + (g1 % 2) * GB + 128 * c) = cur[s][c];
            __builtin_amdgcn_sched_barrier(0);            // (loads ahead of the stores would need registers of their own)
            load(std::integral_constant<int, s>{}, src, i, i == 7 ? 2 : 1);
            if constexpr (i == 3) {
                filled[g2 * 256 + w * 64 + lane] = (unsigned char)vm[s_next];      // granule p + 2
                src1 = gather_src(s1);
                pin(src1);
                pin(vm[s_next]);
                place(s1);
            }
            if constexpr (i == 4) request(s1);
            if constexpr (i == 5) advance();
            if constexpr (i == 6 && !PROBS) moved = __ballot(mj[0] != m_c || mj[1] != m_c) != 0ull;
            __builtin_amdgcn_sched_barrier(0);
        });
        if (PROBS && to_q == 0) {
            to_q = m < n_mine ? granules(m) + 1 : INT32_MAX;
            ++m;
        }
        if (!PROBS && __builtin_expect(moved | (to_q <= 1), 0)) {
            if (to_q != 1) {                              // (granule p - 2 is Q: it has no P)
                // another query, or P of granule p - 2 has another reference than the accumulators
                const bool is_q = to_q == 0;
                const float old = is_q ? -INFINITY : m_c;
                m_c = fmaxf(old, fmaxf(mj[0], mj[1]));
                const float f = old == m_c ? 1.f : fast_exp2(old - m_c);
#pragma unroll
                for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                    for (int e = 0; e < 16; ++e) o_acc[nb][e] = is_q ? 0.f : o_acc[nb][e] * f;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float fp = mj[h] == m_c ? 1.f : fast_exp2(mj[h] - m_c);
#pragma unroll
                    for (int e = 0; e < 8; ++e) pa[h][e] = (__bf16)((float)pa[h][e] * fp);
                }
                if (is_q) {
                    to_q = m < n_mine ? granules(m) + 1 : INT32_MAX;
                    ++m;
                }
            }
        }
        --to_q;
        src = src1;
        __syncthreads();
    };
#pragma unroll 1
    do {
        unroll<DI>([&](auto s_c) __attribute__((always_inline)) { period(s_c); });
    } while (m <= n_mine);
}

// Combine the per-split partials of one (query, head): O = sum_s w_s O_s / sum_s w_s with O_s the split's own
// normalised output and w_s = l_s 2^(m_s-m) its share of the row sum.
// D_V / 8 lanes (16 bytes each) per split, SLOTS splits side by side, and each slot requests all of its splits (8 per batch)
// together with their (maximum, sum) pairs: the launch waits for memory once.  What bounds it is that latency and the launch
// itself; with one thread per four columns walking the splits one batch after the other, a single decode token's 32 splits
// took 14.2 us per layer, now 5.  Up to eight splits are one batch of one slot: then a wave has a (query, head) of 512
// columns to itself, nothing passes through LDS, and no lane is left without a split (with four slots, two splits of 128
// queries x 32 heads kept half of the lanes idle in 4096 workgroups: launch and merge took 45.6 us, 38.6 before that form).
template <int D_V, int SLOTS, bool WIDE>                // WIDE: fp32 partials
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a)
{
    constexpr int LPS = D_V / 8, kBatch = 8;
    constexpr int GROUP = LPS * SLOTS, HEADS = 256 / GROUP;  // threads of a head, heads of a workgroup
    static_assert(SLOTS == 1 || 2 * GROUP >= D_V, "two columns per thread at the end");
    asm volatile("" ::"s"(a.n_layers), "s"(a.B), "s"(a.Tq), "s"(a.H_q), "s"(a.n_splits), "s"(a.row_gap), "s"(a.part_o), "s"(a.part_ml), "s"(a.lse));   // (together: see attn_slab_kernel)
    const int64_t gq = blockIdx.x;
    const int layer = layer_of(a, gq);
    int64_t qrow = gq - (int64_t)layer * a.B * a.Tq;
    if (a.row_gap) qrow += (int64_t)((unsigned)qrow / (unsigned)a.Tq) * a.row_gap;
    const int grp = threadIdx.x / GROUP, tid = threadIdx.x % GROUP;
    const int head = blockIdx.y * HEADS + grp;
    const bool live = head < a.H_q;
    const int h = live ? head : 0;
    constexpr int N16 = WIDE ? 2 : 1, CPL = 8 / N16;       // 16-byte loads of a split per thread, columns in each
    const int slot = tid / LPS, v = (tid % LPS) * CPL;     // columns v + c D_V / N16 + 0 .. CPL - 1: a load of a wave is one stretch
    const float *ml = a.part_ml + ((gq * a.n_splits) * a.H_q + h) * 2;
    const int64_t ml_stride = (int64_t)a.H_q * 2;
    const unsigned char *po = (const unsigned char *)a.part_o + (((gq * a.n_splits) * a.H_q + h) * D_V + v) * (2 * N16);
    const int64_t po_stride = (int64_t)a.H_q * D_V * (2 * N16);
    float m = -INFINITY, l = 0.f, o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = 0.f;
    for (int s0 = slot; s0 < a.n_splits; s0 += SLOTS * kBatch) {
        u32x4 x[kBatch][N16];
        float ms[kBatch], ls[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int s = s0 + SLOTS * j;
#pragma unroll
            for (int c = 0; c < N16; ++c) x[j][c] = u32x4{0u, 0u, 0u, 0u};
            ms[j] = -INFINITY;
            ls[j] = 0.f;
            if (s < a.n_splits) {
#pragma unroll
                for (int c = 0; c < N16; ++c) x[j][c] = *(const u32x4 *)(po + s * po_stride + c * (D_V / N16 * 4));
                ms[j] = ml[s * ml_stride];
                ls[j] = ml[s * ml_stride + 1];
            }
        }
        float mb = m;
#pragma unroll
        for (int j = 0; j < kBatch; ++j) mb = fmaxf(mb, ms[j]);
        const float keep = (m == -INFINITY) ? 0.f : fast_exp2(m - mb);
        m = mb;
        l *= keep;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] *= keep;
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const float sc = (ms[j] == -INFINITY) ? 0.f : ls[j] * fast_exp2(ms[j] - m);   // the split's share of the row sum
            l += sc;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (WIDE) {
                    o[e] += __uint_as_float(x[j][0][e]) * sc;
                    o[4 + e] += __uint_as_float(x[j][1][e]) * sc;
                } else {
                    o[2 * e] += __uint_as_float(x[j][0][e] << 16) * sc;        // bf16 -> fp32 is a shift
                    o[2 * e + 1] += __uint_as_float(x[j][0][e] & 0xFFFF0000u) * sc;
                }
            }
        }
    }
    __bf16 *const out = (__bf16 *)a.Os[layer] + (qrow * a.H_q + h) * D_V;
    if constexpr (SLOTS == 1) {
        if (!live) return;
        const float inv = (l > 0.f) ? 1.f / l : 0.f;
        typedef __attribute__((ext_vector_type(CPL))) __bf16 bf16xc;
#pragma unroll
        for (int c = 0; c < N16; ++c) {
            bf16xc r;
#pragma unroll
            for (int e = 0; e < CPL; ++e) r[e] = (__bf16)(o[CPL * c + e] * inv);
            __bf16 *p = out + v + c * (D_V / N16);
            if ((uintptr_t)a.Os[layer] % 16 == 0) {           // (any other address of a bf16 will do as well)
                *(bf16xc *)p = r;
            } else {
#pragma unroll
                for (int e = 0; e < CPL; ++e) p[e] = r[e];
            }
        }
    } else {
        __shared__ __attribute__((aligned(16))) float o_sh[HEADS][SLOTS][D_V];
        __shared__ float m_sh[HEADS][SLOTS], l_sh[HEADS][SLOTS];
        *(f32x4 *)&o_sh[grp][slot][v] = f32x4{o[0], o[1], o[2], o[3]};
        *(f32x4 *)&o_sh[grp][slot][WIDE ? v + D_V / 2 : v + 4] = f32x4{o[4], o[5], o[6], o[7]};
        if (v == 0) {
            m_sh[grp][slot] = m;
            l_sh[grp][slot] = l;
        }
        __syncthreads();
        // the slots together: two neighbouring columns per thread
        const int c = tid * 2;
        if (!live || c >= D_V) return;
        float mt = -INFINITY, lt = 0.f, t0 = 0.f, t1 = 0.f;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) mt = fmaxf(mt, m_sh[grp][s]);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const float sc = (m_sh[grp][s] == -INFINITY) ? 0.f : fast_exp2(m_sh[grp][s] - mt);
            lt += l_sh[grp][s] * sc;
            t0 += o_sh[grp][s][c] * sc;
            t1 += o_sh[grp][s][c + 1] * sc;
        }
        const float inv = (lt > 0.f) ? 1.f / lt : 0.f;
        out[c] = (__bf16)(t0 * inv);
        out[c + 1] = (__bf16)(t1 * inv);
        m = mt;
        l = lt;
    }
    if (tid == 0 && a.lse) a.lse[qrow * a.H_q + h] = (l > 0.f) ? (m + __builtin_log2f(l)) * 0.6931471805599453f : -INFINITY;
}

template <int D_V, int SLOTS, bool WIDE>
hipError_t launch_merge_t(const AttnArgs &a, hipStream_t st)
{
    const unsigned nq = (unsigned)((int64_t)a.n_layers * a.B * a.Tq), H = (unsigned)a.H_q;
    if (D_V == 512 && a.n_splits <= 8)
        hipLaunchKernelGGL((attn_merge_kernel<512, 1, WIDE>), dim3(nq, (H + 3) / 4), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((attn_merge_kernel<D_V, SLOTS, WIDE>), dim3(nq, H), dim3(256), 0, st, a);
    return hipGetLastError();
}

template <int D_QK, int D_V, int ROW_F>
hipError_t launch_t(const AttnArgs &a, hipStream_t st)
{
    constexpr int ROWB = ROW_F * 2 + 16;
    const size_t lds = (size_t)2 * kTile * ROWB + 3 * kTile * sizeof(int32_t);
    static hipError_t attr = hipFuncSetAttribute((const void *)attn_kernel<D_QK, D_V, ROW_F, false>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    static hipError_t attr_pg = hipFuncSetAttribute((const void *)attn_kernel<D_QK, D_V, ROW_F, true>,
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (attr != hipSuccess) return attr;
    if (attr_pg != hipSuccess) return attr_pg;
    dim3 grid((unsigned)((int64_t)a.n_layers * a.B * a.Tq), (unsigned)a.n_splits);
    if (a.pv.seq_lens || a.pv.page_table)
        hipLaunchKernelGGL((attn_kernel<D_QK, D_V, ROW_F, true>), grid, dim3(256), lds, st, a);
    else
        hipLaunchKernelGGL((attn_kernel<D_QK, D_V, ROW_F, false>), grid, dim3(256), lds, st, a);
    return hipGetLastError();
}

template <bool PG, bool SPLIT>
hipError_t launch_slab(const AttnArgs &a, hipStream_t st)
{
    constexpr int lds = 2 * kSlabTile * (576 * 2 + kSlabPad) + 2 * 32 * (kSlabTile * 2 + 16) + (4 * 32 + 4 * 32) * (int)sizeof(float);
    static hipError_t attr = hipFuncSetAttribute((const void *)attn_slab_kernel<576, 512, PG, SPLIT>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    const dim3 grid((unsigned)((int64_t)a.n_layers * a.B * a.Tq), (unsigned)a.n_splits);
    hipLaunchKernelGGL((attn_slab_kernel<576, 512, PG, SPLIT>), grid, dim3(256), lds, st, a);
    return hipGetLastError();
}

int cu_count()
{
    static int n_cu = 0;
    if (n_cu == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess) n_cu = v;
    }
    return n_cu;
}

constexpr int kStreamLds = kStreamRing * kGranule * (576 * 2 + kSlabPad) + 2 * 32 * (kGranule * 2 + 16) + (4 * 32 * 4 + 2 * 32 * 2) * 4 + kStreamRing * kGranule * 8;

template <bool PG, bool MULTI, bool REST = false, bool PROBS = false>
hipError_t launch_stream(const AttnArgs &a, hipStream_t st, const RestArgs &ra = RestArgs{})
{
    constexpr int lds = kStreamLds + (REST ? (kRestSeqs + 1) * 4 : 0);
    static hipError_t attr = hipFuncSetAttribute((const void *)attn_stream_kernel<PG, MULTI, REST, PROBS>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    int64_t wgs = (int64_t)a.n_layers * a.B * a.Tq;
    const int n_cu = cu_count();                          // one workgroup per CU walks a chain of queries
    if (n_cu <= 0) return hipErrorInvalidDevice;
    if (REST) wgs = (int64_t)ra.n_jobs * a.B * ra.n_rows;
    if (wgs > n_cu) wgs = n_cu;
    // (the counts of a workgroup's queries have to fit where P and the references are otherwise)
    if (PROBS) wgs = std::max(wgs, ((int64_t)a.B * a.Tq + kProbsQueries - 1) / kProbsQueries);
    hipLaunchKernelGGL((attn_stream_kernel<PG, MULTI, REST, PROBS>), dim3((unsigned)wgs), dim3(512), lds, st, a, ra);
    return hipGetLastError();
}

hipError_t launch_mla(const AttnArgs &a, hipStream_t st)
{
    const bool pg = a.pv.seq_lens || a.pv.page_table;
    if (a.n_splits > 1) return pg ? launch_slab<true, true>(a, st) : launch_slab<false, true>(a, st);
    const int n_cu = cu_count();                          // one workgroup per CU, in the stream form a chain of queries
    if (n_cu <= 0) return hipErrorInvalidDevice;
    // Queries that are all resident, of a few tiles: the stream's start (its granules are gathered two behind one another, their
    // ids and table entries before that) is most of the launch.  Stream / row-slab, 160 queries of 512 rows: k = 32 11.0 / 9.2 us,
    // 128 11.9 / 11.3, 160 11.9 / 14.0; paged 13.1 / 10.1, 15.0 / 12.6, 15.3 / 16.7, and 8 queries, k = 192, 14.3 / 12.5.
    const int64_t nq = (int64_t)a.n_layers * a.B * a.Tq, tiles = a.split_len / kSlabTile;
    if (nq <= n_cu && (tiles <= 2 || (pg && tiles == 3 && 4 * nq <= n_cu)))
        return pg ? launch_slab<true, false>(a, st) : launch_slab<false, false>(a, st);
    if (a.n_layers > 1 || a.row_gap) return pg ? launch_stream<true, true>(a, st) : launch_stream<false, true>(a, st);
    return pg ? launch_stream<true, false>(a, st) : launch_stream<false, false>(a, st);
}

// Counts of LeadArgs: a workgroup per chunk, a wave per row, whose entries are all requested before the first is looked at
// (2048 rows of 2048 entries are 16 MB: 5 us; four rows per wave, a kilobyte at a time, were one latency after the other
// and took 23).
__global__ __launch_bounds__(64 * kLeadChunk) void lead_kernel(LeadArgs a)
{
    constexpr int U = 8;
    __shared__ int bad[kLeadChunk];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = blockIdx.x * kLeadChunk + wave, b = blockIdx.y;
    const int held = a.pos0 + row + 1;
    const bool vec = (a.k_sel & 3) == 0 && (uintptr_t)a.idx[blockIdx.z] % 16 == 0;
    bool ok = row < a.n_rows;
    if (ok) {
        const int32_t *p = a.idx[blockIdx.z] + ((int64_t)b * a.Tq + row) * a.k_sel;
        if (vec) {
            for (int s0 = 0; s0 < a.k_sel; s0 += 256 * U) {
                i32x4 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = *(const i32x4 *)(p + min(s0 + 256 * u + 4 * lane, a.k_sel - 4));
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int s = min(s0 + 256 * u + 4 * lane, a.k_sel - 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) ok &= s + e < held ? v[u][e] == s + e : v[u][e] < 0;
                }
            }
        } else {
            for (int s0 = 0; s0 < a.k_sel; s0 += 64 * U) {
                int32_t v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = p[min(s0 + 64 * u + lane, a.k_sel - 1)];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int s = min(s0 + 64 * u + lane, a.k_sel - 1);
                    ok &= s < held ? v[u] == s : v[u] < 0;
                }
            }
        }
    }
    const bool prefix = __ballot(!ok) == 0ull;
    if (lane == 0) bad[wave] = prefix ? kLeadChunk : wave;
    __syncthreads();
    if (threadIdx.x == 0) {
        int first = kLeadChunk;
#pragma unroll
        for (int w = 0; w < kLeadChunk; ++w) first = min(first, bad[w]);
        a.lead[((int64_t)blockIdx.z * a.B + b) * a.n_chunks + blockIdx.x] = first;
    }
}

} // namespace

hipError_t launch_lead(const LeadArgs &a, int n_tensors, hipStream_t st)
{
    hipLaunchKernelGGL(lead_kernel, dim3((unsigned)a.n_chunks, (unsigned)a.B, (unsigned)n_tensors), dim3(64 * kLeadChunk), 0, st, a);
    return hipGetLastError();
}

// Head-aggregated probabilities of 576-feature rows: the stream form without its output product.
hipError_t launch_probs_stream(const ProbsArgs &p, hipStream_t st)
{
    AttnArgs a;
    memset(&a, 0, sizeof a);
    a.Q = p.Q;
    a.KV = p.KV;
    a.idx = p.idx;
    a.lse = const_cast<float *>(p.lse);
    a.O = p.probs;
    a.B = p.B;
    a.Tq = p.Tq;
    a.Lk = p.Lk;
    a.H_q = p.H_q;
    a.row_elems = p.row_elems;
    a.k_sel = p.k_sel;
    a.n_layers = 1;
    a.scale_log2e = p.scale_log2e;
    a.causal_pos0 = -1;
    return launch_stream<false, false, false, true>(a, st);
}

// The rows that RestArgs leaves, unsplit.
hipError_t launch_attn_rest(const AttnArgs &a, const RestArgs &ra, hipStream_t st)
{
    return launch_stream<false, false, true>(a, st, ra);
}

// Rows 0 .. n_queries - 1 of every sequence of a.n_layers layers, row t seeing exactly the keys 0 .. pos0 + t (576 / 512 rows, values
// in front).
hipError_t launch_attn_dense(const AttnArgs &a, const DenseArgs &da, hipStream_t st)
{
    if (da.n_queries <= 0) return hipSuccess;
    constexpr int lds = kDenseRing * kDenseTile * (576 * 2 + kSlabPad) + 2 * kDenseRows * (kDenseTile * 2 + 16) + (6 * kDenseRows + 4 + kDenseChain) * 4;
    typedef void (*Kernel)(AttnArgs, DenseArgs, DenseShape);
    static const Kernel kernels[2][2] = {{attn_dense_kernel<false>, attn_dense_kernel<true>}, {attn_layers_dense_kernel<false>, attn_layers_dense_kernel<true>}};
    static hipError_t attr = [] {
        hipError_t e = hipSuccess;
        for (int i = 0; i < 4 && e == hipSuccess; ++i)
            e = hipFuncSetAttribute((const void *)kernels[i / 2][i % 2], hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        return e;
    }();
    if (attr != hipSuccess) return attr;
    const int64_t blocks = ((int64_t)da.n_queries * a.H_q + kDenseRows - 1) / kDenseRows * a.B * a.n_layers;
    const int n_cu = cu_count();
    if (n_cu <= 0) return hipErrorInvalidDevice;
    const dim3 grid((unsigned)std::max(std::min<int64_t>(blocks, n_cu), (blocks + kDenseChain - 1) / kDenseChain));
    // x * ceil(2^32 / d) >> 32 is x / d as long as x * (d - 1) < 2^32; a sequence has at most IC_MAX_K * IC_MAX_HEADS_Q rows
    auto up = [](int64_t d) { return d > 1 ? (unsigned)((((uint64_t)1 << 32) + d - 1) / d) : 0u; };
    DenseShape ds;
    ds.n_blk = (int)(blocks / a.B / a.n_layers);
    ds.n_wgs = (int)grid.x;
    ds.n_round = (int)(blocks / grid.x);
    ds.inv_b = blocks / a.n_layers * (a.B - 1) < (int64_t)1 << 32 ? up(a.B) : 0u;
    ds.n_whole = (int)(blocks / a.n_layers / grid.x);
    ds.inv_layers = up(a.n_layers);          // (of numbers below grid.x * n_layers)
    ds.inv_h = up(a.H_q);
    hipLaunchKernelGGL(kernels[a.n_layers > 1][a.pv.page_table != nullptr], grid, dim3(512), lds, st, a, da, ds);
    return hipGetLastError();
}

bool attn_shape_supported(int d_qk, int d_v)
{
    return (d_qk == 576 && d_v == 512) || (d_qk == 64 && d_v == 64);
}

hipError_t launch_attn(const AttnArgs &a, int d_qk, int d_v, hipStream_t st)
{
    if ((int64_t)a.B * a.Tq <= 0) return hipSuccess;
    if (d_qk == 576 && d_v == 512) {
        // the stream form, or the row-slab form per split of a query's selection when there are too few queries to fill the
        // chip (decode); rows with the values elsewhere than in their first features take the small-tile form
        if (a.v_off == 0) return launch_mla(a, st);
        return launch_t<576, 512, 576>(a, st);
    }
    if (d_qk == 64 && d_v == 64) return launch_t<64, 64, 128>(a, st);
    return hipErrorInvalidValue;
}

hipError_t launch_attn_merge(const AttnArgs &a, int d_v, hipStream_t st)
{
    if ((int64_t)a.B * a.Tq <= 0) return hipSuccess;
    if (d_v == 512) return a.part_wide ? launch_merge_t<512, 4, true>(a, st) : launch_merge_t<512, 4, false>(a, st);
    if (d_v == 64) return a.part_wide ? launch_merge_t<64, 32, true>(a, st) : launch_merge_t<64, 32, false>(a, st);
    return hipErrorInvalidValue;
}

} // namespace ic
