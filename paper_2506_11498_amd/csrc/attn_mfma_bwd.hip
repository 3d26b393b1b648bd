// LRSA attention backward on bf16 MFMA (gfx950), head_dim 128 or 64.  Gradients of sum(O * dO) with
// the mask constant:  A = exp(scale Q K^T + M - lse), dV = A^T dO, dA = dO V^T,
// D = rowsum(dO * O), dS = A * (dA - D), dQ = scale dS K, dK = scale dS^T Q.
//
// Deterministic, no atomics.  Three launches on one stream:
//   k_bwd_dq          query-outer: a workgroup owns eight (or four) pieces of 32 query rows of one KV group and walks their
//                     key stream exactly like the forward (gather list, then the local window), recomputing A;
//                     it also leaves D[b,hq,t] = dO[t] . O[t] and lse in the units of the logits (mfma_tiles.h) in the workspace
//   k_bwd_dkv         key-outer, two kinds of workgroups in one launch.  GATHER: 256 (four waves: 128) consecutive entries of one
//                     KV head's gather list (sink ++ survivors) x one slice of query chunks -> fp32 partial
//                     dK, dV rows in the workspace.  WINDOW: as many consecutive positions x the queries that see
//                     them through the local window (own chunk causally, the next local_prev chunks in full);
//                     positions outside the gather list are written as final dK, dV, listed ones as one more
//                     fp32 partial.
//   k_bwd_dkv_reduce  listed positions: window partial + the slices, in a fixed order -> dK, dV
// In the key-outer kernel a lane owns one key column of S = Q K^T: K fragments stay in registers for the
// whole walk, the workgroup's V rows in LDS; Q and dO rows stream through LDS 64 (four waves: 32) rows at a time and are read
// both row-wise (for S and dA) and transposed (for dV^T += dO^T A and dK^T += Q^T dS).
#include "mfma_tiles.h"

namespace lrsa {

constexpr int DQ_BN = 64;
constexpr int DQ_PF = 4;                 // LDS operands of the query-outer kernel are read this many MFMAs ahead
// The key-outer kernel, with W = 8 or 4 waves per workgroup (two workgroups of four fit a CU), 32 keys each
constexpr int KV_NB = 1;                                   // 32-key blocks per wave (2 needs one wave per SIMD: measured slower)
template <int W> constexpr int KV_BK = 32 * KV_NB * W;     // keys per workgroup
constexpr int KV_BQ = 32;                                  // query rows per MFMA sub-step
template <int W> constexpr int KV_SUB = W == 8 ? 2 : 1;    // sub-steps per pipeline step (one LDS stage, one barrier)
template <int W> constexpr int KV_ROWS = KV_BQ * KV_SUB<W>;   // query rows per step
constexpr int KV_LD = 64;                                  // floats of lse (and of -D) that a wave copies per step
constexpr int KV_MAX_SLICES = 16;

// ------------------------------------------------------------------------------------ host-side plan
struct BwdPlan {
    int sink_tiles_k, tpc_k;    // dK/dV window mode: key tiles of KV_BK positions in the sink / per chunk
    int kc_lo, ktiles;          // first key chunk and number of key tiles of the window part
    int fq0, fq1;               // query chunks whose rows take part (all of them unless a row window is set)
    int waves, bk;              // of a workgroup of the dK/dV kernel, its keys
    int gl_total, gtiles;       // gather list length per KV head as the last query chunk sees it, its tiles
    int qch, nsl;               // query chunks per slice, slices per gather tile (KV_MAX_SLICES, before they are halved where that fills the chip)
    int hsl, wsl;               // parts that the group's heads are split into: GATHER slices, WINDOW tiles
    int wlo, whi;               // positions [wlo, whi) of the WINDOW tiles
    int gather_wgs, window_wgs; // workgroups of the two parts of the dK/dV launch (multiples of 8)
    int window_first;           // the WINDOW part comes first (its workgroups are the longer ones)
    size_t off_lse2, off_part, off_wpart, off_compact, off_dkc, bytes;   // workspace: D, lse in the logits' units, the fp32 partials of
                                                              // the two parts, condensed K/V, condensed dK/dV (fp32)
};

// first query chunk that sees entry j0 of the gather list
__host__ __device__ __forceinline__ int first_chunk_seeing(const Dims& D, int j0) {
    return j0 < D.S ? 0 : (j0 - D.S) / D.K + D.lp + 1;
}

// (head, query) rows that a CU's workgroup walks per us, as measured
static double rows_per_us(const Dims& D) { return D.d == 64 ? 24.0 : 16.0; }

// Parts that the heads of a group are split into, for launches in which a workgroup is long beside what every CU has to do:
// half of the longest workgroup is idle time at the end of the launch, and every part writes fp32 partials that the
// reduction reads again.  The number of parts with the smallest sum of the two, if it saves a fifth.  `rows`: (head, query)
// rows of a workgroup with one part, `bytes`: partials of one part, `bytes_one`: partials where there is only one part; the us
// that it expects to save are added to `saved`.
// Rates: 16 (head_dim 64: 24) rows per us and CU, as measured; 1 TB/s for partials, fitted with workgroups of eight waves that stored 32
// bytes of a row at a time, as the figures below.  Now that partials leave in whole lines and most such launches have four waves the line
// is on the careful side: backward with 2 TB/s over that with 1, head_dim 128 0.78 to 1.08 of the time (50 training shapes, 14 faster and 6 slower
// by more than 1.5 percent, 0.978 on average), head_dim 64 0.82 to 1.09 (20, 0.962), filling steps 0.84 to 1.02 (12, 0.962); with 4.4 TB/s
// 0.983, 0.955 and 0.965, up to 1.15; with 0.5 TB/s 1.02, 1.05 and 1.09.
// The filling steps live from it: their windows of a few chunks leave about as many workgroups as CUs, of which the WINDOW
// ones (whole chunks, all heads) were twice as long as the others and came last.  32K tokens, 12 heads on 2, lag 1024, four
// chunks per step: dK/dV launches of 7.0 ms in all, the whole training step 12.1 -> 9.5 ms; 11.5K tokens, 8 on 2, lag 479:
// 1.94 -> 1.16 ms.  Training steps of 2.6K tokens in one call 206 -> 155 us (with the finer slices
// of make_plan); long sequences keep one part.  With partials at 4.4 TB/s and a tenth instead of a fifth it split too often:
// 3.5K tokens, 16 heads on 4, 4 requests 505 -> 535 us.
static int head_parts(const Dims& D, double rows, double bytes, double bytes_one, double* saved) {
    const double rate = rows_per_us(D);
    int best = 1;
    const double t_one = 0.5 * rows / rate + bytes_one / 1.0e6;
    double t_best = t_one;
    for (int k = 2; k <= D.G; ++k) {
        const double t = 0.5 * rows * ((D.G + k - 1) / k) / D.G / rate + k * bytes / 1.0e6;
        if (t < 0.8 * t_best) { best = k; t_best = t; }
    }
    *saved += t_one - t_best;
    return best;
}

static int64_t gather_workgroups(const Dims& D, const BwdPlan& P) { return (int64_t(D.B) * D.Hkv * P.nsl * P.hsl + 7) / 8 * 8 * P.gtiles; }
static int64_t window_workgroups(const Dims& D, const BwdPlan& P) { return (int64_t(D.B) * D.Hkv * P.ktiles * P.wsl + 7) / 8 * 8; }

// (head, query) rows that all workgroups of `bk` keys walk
static double kv_rows(const Dims& D, int bk) {
    const int gl = D.fq1 > 0 ? gather_count(D, D.fq1 - 1) : 0, kc_lo = D.fq0 - D.lp > 0 ? D.fq0 - D.lp : 0;
    double chunks = 0.0;   // query chunks that see a list tile, over all tiles
    int64_t j0 = 0;
    for (; j0 < gl && j0 < D.S; j0 += bk) chunks += D.fq1 - D.fq0;   // tiles that begin with a sink token
    // first_chunk_seeing of the others, without a division per tile
    int64_t qf = D.lp + 1 + (j0 - D.S) / D.K, rem = (j0 - D.S) % D.K;
    for (; j0 < gl && qf < D.fq1; j0 += bk) {
        chunks += double(D.fq1 - (qf > D.fq0 ? qf : D.fq0));
        qf += bk / D.K;
        rem += bk % D.K;
        if (rem >= D.K) { rem -= D.K; ++qf; }
    }
    const int64_t ktiles = int64_t(D.fq1 - kc_lo) * ((D.L + bk - 1) / bk) + (D.row_begin == 0 ? (D.S + bk - 1) / bk : 0);
    return double(D.B) * D.Hkv * D.L * D.G * (chunks + 0.75 * (D.lp + 1) * ktiles);
}

// split: with parts of the heads and the finest slices, where their rules ask for them; both take more workspace; slices_of: the waves
// whose slices the plan has, 8 or 4; all_rows: kv_rows of such workgroups where that is known
static BwdPlan plan_of(const Dims& D, bool split, int waves, int slices_of, double all_rows = -1.0) {
    BwdPlan P;
    P.waves = waves;
    P.bk = 32 * P.waves;
    const int step = slices_of == 8 ? KV_ROWS<8> : KV_ROWS<4>;
    const int sink_rows = D.S < D.n ? D.S : D.n;
    P.fq0 = D.fq0;
    P.fq1 = D.fq1;
    const int nqf = D.fq1 - D.fq0;                 // query chunks in the window
    P.sink_tiles_k = D.row_begin == 0 ? (sink_rows + P.bk - 1) / P.bk : 0;   // sink keys see only sink queries here
    P.tpc_k = (D.L + P.bk - 1) / P.bk;
    P.kc_lo = D.fq0 - D.lp > 0 ? D.fq0 - D.lp : 0;  // the local window reaches lp chunks back
    P.ktiles = P.sink_tiles_k + (D.fq1 - P.kc_lo) * P.tpc_k;
    P.gl_total = D.fq1 > 0 ? gather_count(D, D.fq1 - 1) : 0;
    P.gtiles = (P.gl_total + P.bk - 1) / P.bk;
    const int stiles = (P.gl_total + 32 * slices_of - 1) / (32 * slices_of);
    // aim at ~8192 query rows (x G heads) per workgroup, but never more than KV_MAX_SLICES slices.  head_dim 64: rows as the steps of
    // KV_ROWS take them, which end with a chunk (512 rows, lag 2, one head: 351 -> 62 us in the backward; all in one slice before)
    const int64_t rows = D.d == 64 ? (int64_t(D.L) + step - 1) / step * step * D.G : int64_t(D.L) * D.G;   // of a chunk
    int64_t qch = (256 * 32) / rows;
    if (qch < 1) qch = 1;
    const int min_qch = (nqf + KV_MAX_SLICES - 1) / KV_MAX_SLICES;
    if (qch < min_qch) qch = min_qch;
    if (qch < 1) qch = 1;
    // small problems: shorter slices (down to ~1024 query rows x G heads) until the gather workgroups -- about
    // half of the (tile, slice) grid sees any query -- fill the chip twice
    while (qch > min_qch && qch > 1 && (qch / 2) * rows >= 1024 &&
           int64_t(D.B) * D.Hkv * stiles * ((nqf + qch - 1) / qch) * slices_of / 16 < 512)
        qch /= 2;
    // fewer than a quarter as many as CUs: down to 256 rows.  With eight waves and partials stored 32 bytes of a row at a time: 2.6K
    // tokens, 4 heads on 2, 2 requests, 24 workgroups, 164 -> 157 us; 2.2K tokens in filling steps, 4 heads on 1, 710 -> 633; from 84
    // workgroups on it cost more than it gave (4K tokens, 8 heads on 8, 2 requests, 128 of them, 271 -> 295 us).  With the present kernels, 70
    // training shapes of grouped heads: without the finer slices 0.90 to 1.51 of the time (1.002 on average at head_dim 128, 1.048 at 64), up to 32
    // workgroups 0.98 to 1.24 (1.001, 1.012), up to 128 0.80 to 1.06 (0.992, 0.997).
    const int64_t coarse = qch;
    while (split && qch > min_qch && qch > 1 && (qch / 2) * rows >= 256 &&
           int64_t(D.B) * D.Hkv * stiles * ((nqf + qch - 1) / qch) * slices_of / 16 < 64)
        qch /= 2;
    P.qch = int(qch);
    P.nsl = nqf > 0 ? (nqf + P.qch - 1) / P.qch : 0;
    P.off_lse2 = align256(size_t(D.B) * D.Hq * D.lse_stride * 4);
    P.off_part = 2 * P.off_lse2;
    P.wlo = P.sink_tiles_k > 0 ? 0 : D.S + P.kc_lo * D.L;
    P.whi = D.row_end;
    P.hsl = P.wsl = 1;
    const int units = D.B * D.Hkv;
    const double w_rows = double(D.lp + 1) * D.L * D.G, g_rows = P.nsl > 0 ? double(P.qch) * D.L * D.G : 0.0;   // of a workgroup
    if (split && D.G > 1) {
        const double per_cu = (all_rows < 0.0 ? kv_rows(D, P.bk) : all_rows) * P.waves / 2048.0;   // per workgroup that runs at once
        const double row = 2.0 * units * D.d * 4;   // bytes of a row of dK and dV partials of all heads
        // a workgroup shorter than a quarter of a CU's work is no tail worth partials
        double saved = 0.0;
        if (per_cu < 4.0 * w_rows) P.wsl = head_parts(D, w_rows, row * (P.whi - P.wlo), 0.0, &saved);
        if (per_cu < 4.0 * g_rows) P.hsl = head_parts(D, g_rows, 0.5 * row * P.nsl * P.gl_total, 0.5 * row * P.nsl * P.gl_total, &saved);
        // In short launches (under 150 us of work for a CU) parts of one kind are worth nothing while the other kind's workgroups
        // are as long, and parts of one kind alone have to save a quarter of a CU's work.  Of 250 training shapes of 2K to 12K
        // tokens 19 were more than 1.2 percent slower split than whole, by up to 14 (24 heads on 8, 2 requests of 2.5K tokens: 228 ->
        // 260 us); with this rule 12, by up to 6.  Gains of up to 9 percent go with them.  In longer launches it would take as much
        // as it gives (8 heads on 2, 37K tokens, lag 1547: training step 3.28 -> 3.50 ms; 4 on 1, 18K tokens: backward 575 -> 524), and where
        // the slices are the finer ones idle CUs take the parts (8 on 2, 2.1K tokens: 82 -> 94 us without).
        const double one = w_rows > g_rows ? w_rows : g_rows, wp = w_rows * ((D.G + P.wsl - 1) / P.wsl) / D.G,
                     gp = g_rows * ((D.G + P.hsl - 1) / P.hsl) / D.G, work = per_cu / rows_per_us(D);
        if (qch == coarse && work < 150.0 && ((wp > gp ? wp : gp) > 0.95 * one || ((P.wsl == 1 || P.hsl == 1) && saved < 0.25 * work))) P.wsl = P.hsl = 1;
    }
    P.window_first = w_rows * ((D.G + P.wsl - 1) / P.wsl) > g_rows * ((D.G + P.hsl - 1) / P.hsl);
    P.gather_wgs = int(gather_workgroups(D, P));
    P.window_wgs = int(window_workgroups(D, P));
    // slots 0 .. nsl*hsl-1: the GATHER workgroups' slices; the last slot: what the WINDOW workgroups add to listed positions
    const size_t part = size_t(2) * (P.nsl * P.hsl + 1) * D.B * D.Hkv * P.gl_total * D.d * 4;
    P.off_wpart = P.off_part + align256(part);
    P.off_compact = P.off_wpart + (P.wsl > 1 ? align256(size_t(2) * P.wsl * units * (P.whi - P.wlo) * D.d * 4) : 0);
    P.off_dkc = P.off_compact + compact_kv_bytes(D);
    P.bytes = P.off_dkc + (D.compact ? 2 * align256(size_t(D.B) * D.Hkv * P.gl_total * 128 * 4) : 0);
    return P;
}

// Waves per workgroup of the dK/dV kernel.  Two workgroups of four (128 keys each) fit a CU, but read every query row twice, and 32 rows
// per step instead of 64 leave half the time for a step's copies: 1 to 8 percent slower in long launches (backward of 32K tokens, 16
// heads on 8: 5.30 and 5.71 ms; 32 on 8: 8.99 and 9.45).  In short ones their finer grain and the second workgroup's work beside the first
// one's beginning and end count for more: 2 requests of 4K tokens, 8 heads on 8: 186 -> 161 us; 2 requests of 2.5K tokens, 16 on 4: 189 -> 134;
// 4 requests of 4K tokens, 32 on 8: 1016 -> 885.  Short: less than 600 us of work for a CU, and no workgroup that is long beside that (which
// would share its CU: 8.1K tokens, 16 on 4, lag 727, 364 us in a workgroup, 291 for a CU: 520 -> 565 us) unless it is short in itself.  Of 80
// random shapes on this side of the line the backward takes 0.93 of the time (geometric mean), two 1.08.  head_dim 64: always (0.73 to 1.05 of the time with eight over 46 shapes of 1K to 8K tokens, 0.91 on average).
static BwdPlan make_plan(const Dims& D, bool split, bool slices_of_8 = false) {
    int waves = 4;
    if (D.d != 64) {
        const double rate = rows_per_us(D), rows = kv_rows(D, 256), work = rows / 256.0 / rate;   // us for a CU
        if (work >= 600.0) {
            waves = 8;
        } else {
            const BwdPlan P = plan_of(D, true, 8, 8, rows);
            const double w = double(D.lp + 1) * D.L * ((D.G + P.wsl - 1) / P.wsl), g = P.nsl > 0 ? double(P.qch) * D.L * ((D.G + P.hsl - 1) / P.hsl) : 0.0;
            const double longest = (w > g ? w : g) / rate;
            waves = longest <= 0.8 * work || longest <= 100.0 ? 4 : 8;
            if (waves == 8 && split) return P;
        }
    }
    return plan_of(D, split, waves, slices_of_8 ? 8 : waves);
}

// What a plan needs does not grow steadily from one filling step to the next: a split step may need more than a later, longer
// one that is not split (up to three times, in every sixth of 2400 shapes).  A call whose workspace holds the plan without splits, as
// one that was sized for the last step does, takes that plan.  With four waves the slices may come out finer than with eight (five
// of 1500 shapes, up to 1.9 times the partials): a workspace that holds the slices of eight, without parts, is enough as well.
static BwdPlan plan_for(const Dims& D, size_t ws_bytes) {
    const BwdPlan P = make_plan(D, true);
    if (P.bytes <= ws_bytes) return P;
    const BwdPlan whole = make_plan(D, false);
    return whole.bytes <= ws_bytes ? whole : make_plan(D, false, true);
}
size_t attn_bwd_mfma_ws_bytes(const Dims& D) { return make_plan(D, true).bytes; }
void attn_bwd_mfma_parts(const Dims& D, int32_t* gather, int32_t* window) {
    const BwdPlan P = make_plan(D, true);
    *gather = P.hsl;
    *window = P.wsl;
}
void attn_bwd_mfma_plan(const Dims& D, size_t ws_bytes, int32_t* dq_waves, int32_t* waves, int32_t* slices, int32_t* gather, int32_t* window) {
    const BwdPlan P = plan_for(D, ws_bytes);
    *dq_waves = qtile_waves(D);
    *waves = P.waves;
    *slices = P.nsl;
    *gather = P.hsl;
    *window = P.wsl;
}
size_t attn_bwd_mfma_ws_min_bytes(const Dims& D) {
    const size_t whole = make_plan(D, false).bytes, split = attn_bwd_mfma_ws_bytes(D), of_8 = make_plan(D, false, true).bytes;
    const size_t least = whole < split ? whole : split;
    return of_8 < least ? of_8 : least;
}

// the grids of the forward, dQ and dK/dV launches (the reduction's threads are fewer than the bytes of its partials)
bool mfma_grids_fit(const Dims& D) {
    // An upper bound on the work-items of each, for nearly all calls: a workgroup's threads are at most 64 per piece of 32 rows x head and 2 per
    // key, and 512 for the remainder of a segment or list; there are at most 2 * KV_MAX_SLICES slices and as many parts as heads.
    const double heads = double(D.B) * D.Hq, gl = D.fq1 > 0 ? gather_count(D, D.fq1 - 1) : 0;
    const double q = heads * (2.0 * D.S + 576.0 + D.fq1 * (2.0 * D.L + 576.0)), g = (heads * 2.0 * KV_MAX_SLICES + 7.0) * (2.0 * gl + 512.0);
    if (q + g + 4096.0 < 2147483648.0) return true;
    const int64_t units = int64_t(D.B) * D.Hkv;
    const BwdPlan P = make_plan(D, true), P8 = plan_of(D, true, 8, 8);   // also where workgroups have four waves: which shapes are served does not change with it
    return grid_fits(units * tiles_per_unit(D, 8), 512) && grid_fits(units * tiles_per_unit(D, 4), 256) &&
           grid_fits(gather_workgroups(D, P8) + window_workgroups(D, P8), 512) &&
           grid_fits(gather_workgroups(D, P) + window_workgroups(D, P), 64 * P.waves);
}

// ------------------------------------------------------------------------------------ dQ
// One 64-key tile for one wave: per 32 keys S^T and dA^T, then dS^T, then dQ^T += K^T dS^T.
// MASK: the tile holds entries some query of the wave does not see (only the last tiles of a walk).
template <int DH, bool MASK>
__device__ __forceinline__ void dq_tile(const unsigned char* sK, const unsigned char* sV, const bf16x8 (&qf)[KK<DH>],
                                        const bf16x8 (&gf)[KK<DH>], const LaneOffs& lo, f32x16 (&dq)[DB<DH>], int j0, int lim,
                                        int wave_lim_max, float c2, float lse2, float Dq, int lane) {
    constexpr bool CLEAN = MASK && DH == 64;   // keys that a query does not see must not reach it, whatever they hold
    const int g = lane >> 5;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        if (!MASK || j0 + kb * 32 <= wave_lim_max) {  // otherwise these 32 keys are masked for the whole wave
            // MFMAs of S^T (K rows), dA^T (V rows), dQ^T (K transposed, rows 0-15 then 16-31); their LDS operands
            // form one stream that is read DQ_PF ahead.  A = exp(scale S - lse) is written beside the dA MFMAs it
            // does not depend on.
            f32x16 s, dp;
#pragma unroll
            for (int i = 0; i < 16; ++i) { s[i] = 0.0f; dp[i] = 0.0f; }
#define LRSA_DQ_OPND(n)                                                                                      \
    ((n) < N1 ? read_rows_o<DH>(sK, lo, kb * 32, (n)) : (n) < N2 ? read_rows_o<DH>(sV, lo, kb * 32, (n) - N1) \
              : read_cols_o<DH>(sK, lo, kb * 32 + ((n) >= N3 ? 16 : 0), ((n) - N2) % DB<DH>))
            constexpr int N1 = KK<DH>, N2 = 2 * KK<DH>, N3 = N2 + DB<DH>, N4 = N3 + DB<DH>;
            bf16x8 a[DQ_PF];
#pragma unroll
            for (int n = 0; n < DQ_PF; ++n) a[n] = LRSA_DQ_OPND(n);
            Weights<TERMS<DH>> dsf0, dsf1;
#pragma unroll
            for (int n = 0; n < N4; ++n) {
                if (CLEAN && n < N1) s = poison_rows(a[n % DQ_PF], s);
                if (CLEAN && n >= N2) a[n % DQ_PF] = finite_operand(a[n % DQ_PF]);
                if (n < N1) s = mfma32(a[n % DQ_PF], qf[n], s);
                else if (n < N2) dp = mfma32(a[n % DQ_PF], gf[n - N1], dp);
                else if (n < N3) dq[n - N2] = mfma32_w(a[n % DQ_PF], dsf0, dq[n - N2]);
                else dq[n - N3] = mfma32_w(a[n % DQ_PF], dsf1, dq[n - N3]);
                if (n + DQ_PF < N4) a[n % DQ_PF] = LRSA_DQ_OPND(n + DQ_PF);
                if (n >= N1 && n < N2) {
                    constexpr int E = 16 / KK<DH>;
#pragma unroll
                    for (int i = E * (n - N1); i < E * (n - N1) + E; ++i) {
                        float pr = weight<DH>(s[i], c2, lse2);
                        if (MASK) {
                            const int j = j0 + kb * 32 + 8 * (i >> 2) + 4 * g + (i & 3);
                            pr = j <= lim ? pr : 0.0f;
                        }
                        s[i] = pr;
                    }
                }
                if (n == N2 - 1) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        s[i] *= dp[i] - Dq;
                        if (CLEAN) s[i] = j0 + kb * 32 + 8 * (i >> 2) + 4 * g + (i & 3) <= lim ? s[i] : 0.0f;
                    }
                    dsf0 = pack_weights<TERMS<DH>>(s, 0);
                    dsf1 = pack_weights<TERMS<DH>>(s, 8);
                }
            }
#undef LRSA_DQ_OPND
        }
    }
}

// A tile all of whose 64 keys every query of the wave sees: both 32-key halves as ONE stream of MFMAs,
//   S0 | dA0 (+ exp of half 0) | S1 (+ dS of half 0) | dA1 (+ exp of half 1) | dQ0 (+ dS of half 1) | dQ1,
// so that every piece of vector work sits beside MFMAs it does not depend on.  LDS operands are read DQ_PF ahead.
template <int DH>
__device__ __forceinline__ void dq_tile_full(const unsigned char* sK, const unsigned char* sV, const bf16x8 (&qf)[KK<DH>],
                                             const bf16x8 (&gf)[KK<DH>], const LaneOffs& lo_in, f32x16 (&dq)[DB<DH>], float c2,
                                             float lse2, float Dq) {
    // the two offset registers are made opaque here so that the XORed per-block offsets are formed next
    // to each read (one vector op) instead of being kept in registers across the whole walk
    LaneOffs lo = lo_in;
    asm volatile("" : "+v"(lo.row), "+v"(lo.col));
    f32x16 s0, dp0, s1, dp1, zero;
#pragma unroll
    for (int i = 0; i < 16; ++i) zero[i] = 0.0f;
    constexpr int K1 = KK<DH>, N4 = 4 * K1, N5 = N4 + 2 * DB<DH>, N6 = N5 + 2 * DB<DH>;   // ends of the S, dA and dQ groups
    constexpr int E = 16 / K1, ED = 16 / (2 * DB<DH>);   // vector elements beside one MFMA of a group
#define LRSA_DQ_OPND(n)                                                                                        \
    ((n) < K1 ? read_rows_o<DH>(sK, lo, 0, (n)) : (n) < 2 * K1 ? read_rows_o<DH>(sV, lo, 0, (n) - K1)           \
     : (n) < 3 * K1 ? read_rows_o<DH>(sK, lo, 32, (n) - 2 * K1) : (n) < N4 ? read_rows_o<DH>(sV, lo, 32, (n) - 3 * K1) \
     : read_cols_o<DH>(sK, lo, ((n) - N4) / DB<DH> * 16, ((n) - N4) % DB<DH>))
    bf16x8 a[DQ_PF];
#pragma unroll
    for (int n = 0; n < DQ_PF; ++n) a[n] = LRSA_DQ_OPND(n);
    Weights<TERMS<DH>> dsf[4];   // dS of keys 0-15, 16-31, 32-47, 48-63
    // six groups of MFMAs (separate loops: each unrolls fully, so every array index is a constant)
#define LRSA_DQ_NEXT(n) if ((n) + DQ_PF < N6) a[(n) % DQ_PF] = LRSA_DQ_OPND((n) + DQ_PF)
#pragma unroll
    for (int k = 0; k < K1; ++k) {
        s0 = mfma32(a[k % DQ_PF], qf[k], k == 0 ? zero : s0);
        LRSA_DQ_NEXT(k);
    }
#pragma unroll
    for (int k = 0; k < K1; ++k) {
        dp0 = mfma32(a[(K1 + k) % DQ_PF], gf[k], k == 0 ? zero : dp0);
        LRSA_DQ_NEXT(K1 + k);
#pragma unroll
        for (int i = E * k; i < E * k + E; ++i) s0[i] = weight<DH>(s0[i], c2, lse2);
    }
#pragma unroll
    for (int k = 0; k < K1; ++k) {
        s1 = mfma32(a[(2 * K1 + k) % DQ_PF], qf[k], k == 0 ? zero : s1);
        LRSA_DQ_NEXT(2 * K1 + k);
#pragma unroll
        for (int i = E * k; i < E * k + E; ++i) s0[i] *= dp0[i] - Dq;
    }
    dsf[0] = pack_weights<TERMS<DH>>(s0, 0);
    dsf[1] = pack_weights<TERMS<DH>>(s0, 8);
#pragma unroll
    for (int k = 0; k < K1; ++k) {
        dp1 = mfma32(a[(3 * K1 + k) % DQ_PF], gf[k], k == 0 ? zero : dp1);
        LRSA_DQ_NEXT(3 * K1 + k);
#pragma unroll
        for (int i = E * k; i < E * k + E; ++i) s1[i] = weight<DH>(s1[i], c2, lse2);
    }
#pragma unroll
    for (int k = 0; k < 2 * DB<DH>; ++k) {
        dq[k % DB<DH>] = mfma32_w(a[(N4 + k) % DQ_PF], dsf[k / DB<DH>], dq[k % DB<DH>]);
        LRSA_DQ_NEXT(N4 + k);
#pragma unroll
        for (int i = ED * k; i < ED * k + ED; ++i) s1[i] *= dp1[i] - Dq;
    }
    dsf[2] = pack_weights<TERMS<DH>>(s1, 0);
    dsf[3] = pack_weights<TERMS<DH>>(s1, 8);
#pragma unroll
    for (int k = 0; k < 2 * DB<DH>; ++k) {
        dq[k % DB<DH>] = mfma32_w(a[(N5 + k) % DQ_PF], dsf[2 + k / DB<DH>], dq[k % DB<DH>]);
        LRSA_DQ_NEXT(N5 + k);
    }
#undef LRSA_DQ_NEXT
#undef LRSA_DQ_OPND
}

// A wave per piece of 32 query rows of one head, eight or four neighbouring pieces per workgroup, as in the forward (mfma_tiles.h, QTileMap).
// The first tile is asked for before the wave's own rows, and its copies take 32-bit offsets from a scalar base (in 64 bits the
// addresses took 15 registers more, and the variant of four waves spilled; whole backward of 32K tokens, 32 heads on 8,
// 9.55 -> 9.40 ms).
// COMPACT: the rows of the gather list come from the condensed cache Kc, Vc (contiguous), no index is read.
template <int DH, int WAVES, bool COMPACT>
__global__ __launch_bounds__(64 * WAVES, 2) void k_bwd_dq(Dims D, const bf16_t* __restrict__ Q,
                                                           const bf16_t* __restrict__ K,
                                                           const bf16_t* __restrict__ V,
                                                           const bf16_t* __restrict__ O,
                                                           const bf16_t* __restrict__ dO,
                                                           const float* __restrict__ lse,
                                                           float* __restrict__ Dsum, float* __restrict__ lse2_out,
                                                           const int32_t* __restrict__ idx,
                                                           const bf16_t* __restrict__ Kc,
                                                           const bf16_t* __restrict__ Vc,
                                                           bf16_t* __restrict__ dQ, QTileMap M) {
    __shared__ __attribute__((aligned(16))) unsigned char sK0[DQ_BN * ROW_BYTES<DH>];
    __shared__ __attribute__((aligned(16))) unsigned char sV0[DQ_BN * ROW_BYTES<DH>];
    __shared__ __attribute__((aligned(16))) unsigned char sK1[DQ_BN * ROW_BYTES<DH>];
    __shared__ __attribute__((aligned(16))) unsigned char sV1[DQ_BN * ROW_BYTES<DH>];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, g = lane >> 5;
    int b, h, tix, qc, seg_end, tw, head, t_last;
    if (!decode_qtile(M, D, blockIdx.x, b, h, tix) || !qtile_rows(M, D, tix, WAVES, wave, qc, seg_end, tw, head, t_last)) return;   // uniform for the workgroup
    if constexpr (DH == 128) asm volatile("" : "+v"(tw));   // else the walk's branches become scalar, and zeros are kept in registers for them
    const int hq = h * D.G + head;
    const int ng = gather_count(D, qc), cs = window_start(D, qc);
    const int m_max = ng + t_last - cs + 1;
    const int ntiles = (m_max + DQ_BN - 1) / DQ_BN;

    const bf16_t* Kh = K + b * D.ks[0] + h * D.ks[1];
    const bf16_t* Vh = V + b * D.ks[0] + h * D.ks[1];
    const int32_t* idx_h = idx + (int64_t(b) * D.Hkv + h) * D.Ns * D.K;

    const int64_t coff = COMPACT ? (int64_t(b) * D.Hkv + h) * (int64_t(D.S) + int64_t(D.K) * D.Ns) * 128 : 0;
    const bf16_t* Kc_h = Kc + coff;
    const bf16_t* Vc_h = Vc + coff;
    constexpr int RPW = DQ_BN / WAVES, COPIES = RPW / COPY_ROWS<DH>;   // of K (and V) per wave and tile
    int pos[COPIES];   // COMPACT: stream entries; else positions (fetched through idx one tile ahead)
    auto fetch_pos = [&](int tile) {
#pragma unroll
        for (int i = 0; i < COPIES; ++i) {
            int j = tile * DQ_BN + async_row<DH>(RPW * wave + COPY_ROWS<DH> * i, lane);
            j = j < m_max ? j : m_max - 1;
            pos[i] = COMPACT ? j : stream_pos(D, idx_h, j, ng, cs);
        }
    };
    const int wv = __builtin_amdgcn_readfirstlane(wave);   // wave-uniform: LDS destinations are scalars
    auto issue = [&](unsigned char* sK, unsigned char* sV) {
#pragma unroll
        for (int i = 0; i < COPIES; ++i) {
            const int r0 = RPW * wv + COPY_ROWS<DH> * i;
            const int ch = async_chunk<DH>(async_row<DH>(r0, lane), lane) * 8;
            if (COMPACT) {
                async_rows<DH>(stream_row(Kc_h, Kh, D.ks[2], pos[i], ng, cs) + ch, sK, r0);
                async_rows<DH>(stream_row(Vc_h, Vh, D.ks[2], pos[i], ng, cs) + ch, sV, r0);
            } else {
                // byte offset inside the head: below 2^31 (a condition of this kernel, checked on the host)
                const unsigned off = (unsigned(pos[i]) * unsigned(D.ks[2]) + unsigned(ch)) * 2u;
                async_copy16_so(Kh, off, lds_addr(sK) + r0 * ROW_BYTES<DH>);
                async_copy16_so(Vh, off, lds_addr(sV) + r0 * ROW_BYTES<DH>);
            }
        }
    };

    // the first tile is on its way while the wave's own rows are read
    fetch_pos(0);
    issue(sK0, sV0);
    if (ntiles > 1) fetch_pos(1);

    const int tq = tw + l32;
    const int tq_ld = tq < seg_end ? tq : seg_end - 1;
    const int64_t qoff = b * D.qs[0] + hq * D.qs[1] + int64_t(tq_ld) * D.qs[2];
    bf16x8 qf[KK<DH>], gf[KK<DH>];
#pragma unroll
    for (int kk = 0; kk < KK<DH>; ++kk) {
        qf[kk] = *reinterpret_cast<const bf16x8*>(Q + qoff + kk * 16 + g * 8);
        gf[kk] = *reinterpret_cast<const bf16x8*>(dO + qoff + kk * 16 + g * 8);
    }
    // D = rowsum(dO * O) of this lane's row and its lse in the logits' units: used here and, through the workspace,
    // by the key-outer kernel that runs after this one (every (head, query) row belongs to exactly one wave)
    const int64_t rowid = (int64_t(b) * D.Hq + hq) * D.lse_stride + tq_ld;
    const float lse2 = lse[rowid] * LOGIT_UNIT<DH>;
    float Dq = 0.0f;
#pragma unroll
    for (int kk = 0; kk < KK<DH>; ++kk) {
        const bf16x8 o8 = *reinterpret_cast<const bf16x8*>(O + qoff + kk * 16 + g * 8);
#pragma unroll
        for (int i = 0; i < 8; ++i) Dq = __builtin_fmaf(float(o8[i]), float(gf[kk][i]), Dq);
    }
    Dq += __shfl_xor(Dq, 32, 64);
    // head_dim 64: a row that holds an infinity or NaN anywhere is marked for the key-outer kernel by an lse of NaN
    bool odd = false;
    if constexpr (DH == 64) {
        float z = (lse2 + Dq) * 0.0f;
#pragma unroll
        for (int kk = 0; kk < KK<DH>; ++kk)
#pragma unroll
            for (int i = 0; i < 8; ++i) z = __builtin_fmaf(float(qf[kk][i]), 0.0f, __builtin_fmaf(float(gf[kk][i]), 0.0f, z));
        z += __shfl_xor(z, 32, 64);
        odd = z != 0.0f;
    }
    if (tq < seg_end && g == 0) { Dsum[rowid] = odd ? 0.0f : -Dq; lse2_out[rowid] = odd ? NAN : lse2; }   // -D: the key-outer kernel starts its dA sums from it
    const int lim = ng + tq - cs;
    const int wave_lim_max = tw < seg_end ? ng + min(tw + 31, seg_end - 1) - cs : -1;   // a wave without a row only copies

    const float c2 = D.scale * LOGIT_UNIT<DH>;
    const LaneOffs lo = make_lane_offs<DH>(lane);
    const int wave_lim_min = wave_lim_max < 0 ? -1 : ng + tw - cs;   // last stream entry the wave's first query sees
#define LRSA_DQ_TILE(sK, sV, j0_)                                                                              \
    {                                                                                                           \
        const int j0 = (j0_);                                                                                   \
        if (j0 + DQ_BN - 1 <= wave_lim_min)                                                                     \
            dq_tile_full<DH>(sK, sV, qf, gf, lo, dq, c2, lse2, Dq);                                                 \
        else if (j0 <= wave_lim_max)                                                                            \
            dq_tile<DH, true>(sK, sV, qf, gf, lo, dq, j0, lim, wave_lim_max, c2, lse2, Dq, lane);                   \
    }
    f32x16 dq[DB<DH>];
#pragma unroll
    for (int db = 0; db < DB<DH>; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dq[db][i] = 0.0f;

    for (int tile = 0; tile < ntiles; tile += 2) {
        wait_vmcnt<0>();
        __syncthreads();
        if (tile + 1 < ntiles) {
            issue(sK1, sV1);
            if (tile + 2 < ntiles) fetch_pos(tile + 2);
        }
        LRSA_DQ_TILE(sK0, sV0, tile * DQ_BN);
        if (tile + 1 >= ntiles) break;
        wait_vmcnt<0>();
        __syncthreads();
        if (tile + 2 < ntiles) {
            issue(sK0, sV0);
            if (tile + 3 < ntiles) fetch_pos(tile + 3);
        }
        LRSA_DQ_TILE(sK1, sV1, (tile + 1) * DQ_BN);
    }

#undef LRSA_DQ_TILE

    if (tq < seg_end) {
        bf16_t* orow = dQ + b * D.qs[0] + hq * D.qs[1] + int64_t(tq) * D.qs[2];
#pragma unroll
        for (int db = 0; db < DB<DH>; ++db)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                f32x4 v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = dq[db][a * 4 + r] * D.scale;
                *reinterpret_cast<bf16x4*>(orow + db * 32 + a * 8 + g * 4) = __builtin_convertvector(v, bf16x4);
            }
    }
}

// ------------------------------------------------------------------------------------ dK, dV
// One sub-step (32 query rows: rows rowbase .. rowbase+31 of the stage tiles) of the key-outer walk for
// one wave.  sLD holds this wave's copy of the stage rows' lse in the logits' units (floats 0 ..) and -D
// (KV_LD floats on; D = rowsum(dO * O), negated by the query-outer kernel that wrote it).  r0 = first row of the sub-step; rows >= tb are padding.
// lim_u: GATHER (steps never straddle a chunk): the largest gather-list entry the step's chunk sees.
// The wave's K fragments are in registers, its V rows in LDS (sVw): K fragments and the accumulators
// fill the register file.
template <int DH, bool GATHER>
__device__ __forceinline__ void dkv_step(const Dims& D, const unsigned char* sQ, const unsigned char* sG,
                                         const float* sLD, const bf16x8 (&kf)[KV_NB][KK<DH>], const unsigned char* sVw,
                                         const LaneOffs& lo_in, f32x16 (&dk)[KV_NB][DB<DH>], f32x16 (&dv)[KV_NB][DB<DH>], int r0,
                                         int tb, const int (&kcmp)[KV_NB], int lim_u, bool need_mask, float c2, int lane,
                                         int rowbase) {
    const int g = lane >> 5;
    // the two offset registers are made opaque here so that the XORed per-block offsets are formed next
    // to each read (one VALU op) instead of being kept in sixteen registers across the whole walk
    // The lane's offsets with the addresses of the three tiles folded in (the tiles start on 256-byte
    // boundaries): one add per tile and sub-step, then one XOR per read.  The registers are made opaque so
    // that the XORed per-block addresses are formed next to each read instead of being kept across the walk.
    unsigned aQr = lo_in.row + lds_addr(sQ) + rowbase * ROW_BYTES<DH>, aQc = lo_in.col + lds_addr(sQ) + rowbase * ROW_BYTES<DH>;
    unsigned aGr = lo_in.row + lds_addr(sG) + rowbase * ROW_BYTES<DH>, aGc = lo_in.col + lds_addr(sG) + rowbase * ROW_BYTES<DH>;
    unsigned aVr = lo_in.row + lds_addr(sVw);
    asm volatile("" : "+v"(aQr), "+v"(aQc), "+v"(aGr), "+v"(aGc), "+v"(aVr));
    // Four MFMA groups: S, dA, dV, dK (DH / 16 MFMAs per 32-key block each).  The vector work between them is
    // written next to MFMAs it does not depend on -- exp(S) beside the dA group, dS beside the dV group --
    // so that one wave keeps both pipes busy.  Operands are read two ahead of the MFMAs that consume them;
    // an operand read from the Q / dO stage serves all key blocks of the wave.
    bf16x8 a[2];
    f32x16 s[KV_NB], dp[KV_NB];
    // dA - D comes out of the MFMAs themselves: the accumulators start from -D of their rows (sLD holds -D)
#pragma unroll
    for (int a4 = 0; a4 < 4; ++a4) {
        const f32x4 d4 = *reinterpret_cast<const f32x4*>(sLD + KV_LD + rowbase + 8 * a4 + 4 * g);
#pragma unroll
        for (int nb = 0; nb < KV_NB; ++nb)
#pragma unroll
            for (int r = 0; r < 4; ++r) dp[nb][a4 * 4 + r] = d4[r];
    }
#pragma unroll
    for (int nb = 0; nb < KV_NB; ++nb)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[nb][i] = 0.0f;
    a[0] = read_rows_a(aQr, 0);
    a[1] = read_rows_a(aQr, 1);
#pragma unroll
    for (int kk = 0; kk < KK<DH>; ++kk) {
#pragma unroll
        for (int nb = 0; nb < KV_NB; ++nb) s[nb] = mfma32(a[kk & 1], kf[nb][kk], s[nb]);
        a[kk & 1] = kk < KK<DH> - 2 ? read_rows_a(aQr, kk + 2) : read_rows_a(aGr, kk - (KK<DH> - 2));
    }
    // mask bounds: row rho = 8*a4 + 4g + r of the step is visible to key block nb iff mlo[nb] <= 8*a4 + r < mhi
    const int mhi = (tb - r0) - 4 * g;
    int mlo[KV_NB];
#pragma unroll
    for (int nb = 0; nb < KV_NB; ++nb)
        mlo[nb] = GATHER ? (kcmp[nb] <= lim_u ? -64 : 64) : (kcmp[nb] == 0x7fffffff ? 64 : kcmp[nb] - r0 - 4 * g);
    // A = exp(scale S - lse), four values per key block and pair of MFMA rounds; sLD holds lse already in
    // the logits' units.  Only steps that touch the diagonal, a partly visible gather prefix, padding rows or
    // padding keys pay for the mask (wave-uniform flag).
    bf16x8 vb[KV_NB][2];
#pragma unroll
    for (int nb = 0; nb < KV_NB; ++nb) vb[nb][0] = read_rows_a(aVr + nb * 32 * ROW_BYTES<DH>, 0);
#pragma unroll
    for (int kk = 0; kk < KK<DH>; ++kk) {
#pragma unroll
        for (int nb = 0; nb < KV_NB; ++nb) {
            if (kk + 1 < KK<DH>) vb[nb][(kk + 1) & 1] = read_rows_a(aVr + nb * 32 * ROW_BYTES<DH>, kk + 1);
            dp[nb] = mfma32(a[kk & 1], vb[nb][kk & 1], dp[nb]);
        }
        // next operands: the rest of the dO rows, then the first transposed dO operands
        if (kk < KK<DH> - 2) a[kk & 1] = read_rows_a(aGr, kk + 2);
        else a[kk & 1] = read_cols_a<DH>(aGc, 0, kk - (KK<DH> - 2));
        if (kk % (KK<DH> / 4) == 0) {
            const int a4 = kk / (KK<DH> / 4);
            const f32x4 l4 = *reinterpret_cast<const f32x4*>(sLD + rowbase + 8 * a4 + 4 * g);
            if (!need_mask) {
#pragma unroll
                for (int nb = 0; nb < KV_NB; ++nb)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        s[nb][a4 * 4 + r] = weight<DH>(s[nb][a4 * 4 + r], c2, l4[r]);
            } else {
#pragma unroll
                for (int nb = 0; nb < KV_NB; ++nb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float pr = weight<DH>(s[nb][a4 * 4 + r], c2, l4[r]);
                        const int c = 8 * a4 + r;
                        s[nb][a4 * 4 + r] = (c >= mlo[nb] && c < mhi) ? pr : 0.0f;
                    }
            }
        }
    }
    constexpr int NB2 = 2 * DB<DH>;   // MFMAs (one per term of the weights) of the dV group and of the dK group
    Weights<TERMS<DH>> pf[KV_NB][2], dsf[KV_NB][2];
#pragma unroll
    for (int nb = 0; nb < KV_NB; ++nb) { pf[nb][0] = pack_weights<TERMS<DH>>(s[nb], 0); pf[nb][1] = pack_weights<TERMS<DH>>(s[nb], 8); }
    // dV^T += dO^T A (rows 0-15 blocks 0..3, rows 16-31 blocks 0..3) with dS = A * (dA - D) beside it (dp holds dA - D),
    // then dK^T += Q^T dS in the same order
#define LRSA_OPND(n) ((n) < NB2 ? read_cols_a<DH>(aGc, (n) / DB<DH> * 16, (n) % DB<DH>) : read_cols_a<DH>(aQc, ((n) - NB2) / DB<DH> * 16, (n) % DB<DH>))
#pragma unroll
    for (int n = 0; n < NB2; ++n) {
#pragma unroll
        for (int nb = 0; nb < KV_NB; ++nb) dv[nb][n % DB<DH>] = mfma32_w(a[n & 1], pf[nb][n / DB<DH>], dv[nb][n % DB<DH>]);
        a[n & 1] = LRSA_OPND(n + 2);
        if (n % (NB2 / 4) == 0) {
            const int a4 = n / (NB2 / 4);
#pragma unroll
            for (int nb = 0; nb < KV_NB; ++nb)
#pragma unroll
                for (int r = 0; r < 4; ++r) dp[nb][a4 * 4 + r] *= s[nb][a4 * 4 + r];
        }
    }
#pragma unroll
    for (int nb = 0; nb < KV_NB; ++nb) { dsf[nb][0] = pack_weights<TERMS<DH>>(dp[nb], 0); dsf[nb][1] = pack_weights<TERMS<DH>>(dp[nb], 8); }
#pragma unroll
    for (int n = NB2; n < 2 * NB2; ++n) {
#pragma unroll
        for (int nb = 0; nb < KV_NB; ++nb) dk[nb][n % DB<DH>] = mfma32_w(a[n & 1], dsf[nb][(n - NB2) / DB<DH>], dk[nb][n % DB<DH>]);
        if (n + 2 < 2 * NB2) a[n & 1] = LRSA_OPND(n + 2);
    }
#undef LRSA_OPND
}

// Query rows that hold infinities or NaN (the query-outer kernel has made their lse NaN) must make NaN of the sums of the keys that
// see them, and leave the others of the step alone, although a sub-step multiplies its masked pairs by zero: the rows become zeros in
// the stage's tiles.  A = exp(S - lse) is NaN where it is seen and 0 where it is masked.  Every wave clears all of them before
// it reads the tiles: its own reads come after its own writes, and all waves write the same.
template <int DH, int W>
__device__ __forceinline__ void clear_odd_rows(unsigned char* sQ, unsigned char* sG, const float* sLD, int lane) {
    static_assert(KV_ROWS<W> <= 64, "a lane looks at a row");
    const float l = sLD[lane];
    unsigned long long rows = __builtin_amdgcn_ballot_w64(l != l && lane < KV_ROWS<W>);
    if (rows == 0) return;
    for (; rows; rows &= rows - 1) {
        const int r = __builtin_ctzll(rows);
        if (lane * 16 < ROW_BYTES<DH>) {
            *reinterpret_cast<uint4*>(sQ + r * ROW_BYTES<DH> + lane * 16) = uint4{0u, 0u, 0u, 0u};
            *reinterpret_cast<uint4*>(sG + r * ROW_BYTES<DH> + lane * 16) = uint4{0u, 0u, 0u, 0u};
        }
    }
    asm volatile("" ::: "memory");   // the tiles are read through integer addresses
}

// Two stages of KV_ROWS rows, one barrier per step; the copies of the next stage run during the sub-steps of the current one.

// LDS of the dK/dV kernel: two stages of (Q rows, dO rows, per-wave lse|D) -- separate arrays so that reads
// of one stage need not wait for the asynchronous fill of the other -- and the workgroup's V rows
struct KvLds {
    unsigned char *sQ0, *sQ1, *sG0, *sG1;
    float *sL0, *sL1;
    unsigned char* sVk;
};
// one set of arrays for both kinds of workgroup (inside the body's template each would get a set of its own)
template <int DH, int W>
__device__ __forceinline__ KvLds kv_lds() {
    __shared__ __attribute__((aligned(256))) unsigned char sQ0[KV_ROWS<W> * ROW_BYTES<DH>], sQ1[KV_ROWS<W> * ROW_BYTES<DH>];
    __shared__ __attribute__((aligned(256))) unsigned char sG0[KV_ROWS<W> * ROW_BYTES<DH>], sG1[KV_ROWS<W> * ROW_BYTES<DH>];
    __shared__ __attribute__((aligned(16))) float sL0[W * 2 * KV_LD], sL1[W * 2 * KV_LD];
    __shared__ __attribute__((aligned(256))) unsigned char sVk[KV_BK<W> * ROW_BYTES<DH>];
    return KvLds{sQ0, sQ1, sG0, sG1, sL0, sL1, sVk};
}

// The 32 rows of DH sums that a wave holds as columns (lane: key lane % 32, channels of half g), in order: half rows of
// COPY_ROWS rows at a time, lane: row r0 + lane / (DH / 8), channels half * DH / 2 + lane % (DH / 8) * 4 .. +3 -> put(r0, half, value).
// stage: 32 * ROW_BYTES bytes of LDS that only this wave uses; 16-byte pieces swizzled so that neither side meets bank conflicts.
template <int DH, typename Put>
__device__ __forceinline__ void rows_through_lds(unsigned char* stage, const f32x16 (&acc)[DB<DH>], float scale, int lane, Put put) {
    constexpr int PIECES = DH / 8;   // of a half row
    const int l32 = lane & 31, g = lane >> 5;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int db = 0; db < DB<DH> / 2; ++db)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                f32x4 v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = acc[half * (DB<DH> / 2) + db][a * 4 + r] * scale;
                *reinterpret_cast<f32x4*>(stage + l32 * ROW_BYTES<DH> + (((db * 8 + a * 2 + g) ^ (l32 & (PIECES - 1))) << 4)) = v;
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // other lanes' writes
#pragma unroll
        for (int r0 = 0; r0 < 32; r0 += COPY_ROWS<DH>) {
            const int row = r0 + lane / PIECES;
            put(r0, half, *reinterpret_cast<const f32x4*>(stage + row * ROW_BYTES<DH> + (((lane & (PIECES - 1)) ^ (row & (PIECES - 1))) << 4)));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read before the second half is written
    }
}

// gather-list entry of a position, if it is a sink token or a survivor that some query of this call sees there; else -1
__device__ __forceinline__ int listed_entry(const Dims& D, const BwdPlan& P, const int32_t* idx_h, int pos) {
    if (P.gtiles == 0) return -1;
    if (pos < D.S) return pos;
    const int c = (pos - D.S) / D.L;
    if (D.S + (c + 1) * D.K > P.gl_total) return -1;   // chunk c is not compressed for any of them
    const int32_t* rowp = idx_h + int64_t(c) * D.K;
    int lo = 0, hi = D.K - 1;
    while (lo <= hi) {
        const int mid = (lo + hi) >> 1, v = rowp[mid];
        if (v == pos) return D.S + c * D.K + mid;
        if (v < pos) lo = mid + 1; else hi = mid - 1;
    }
    return -1;
}

template <int DH, int W, bool GATHER>
__device__ __forceinline__ void dkv_body(const Dims& D, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
                                         const bf16_t* __restrict__ V, const bf16_t* __restrict__ Kc,
                                         const bf16_t* __restrict__ Vc, const bf16_t* __restrict__ dO,
                                         const float* __restrict__ lse, const float* __restrict__ Dsum,
                                         const int32_t* __restrict__ idx, bf16_t* __restrict__ dK,
                                         bf16_t* __restrict__ dV, float* __restrict__ accK, float* __restrict__ accV,
                                         float* __restrict__ part, float* __restrict__ wpart, const BwdPlan& P,
                                         const int block) {
    const KvLds sh = kv_lds<DH, W>();
    unsigned char *const sQ0 = sh.sQ0, *const sQ1 = sh.sQ1, *const sG0 = sh.sG0, *const sG1 = sh.sG1;
    float *const sL0 = sh.sL0, *const sL1 = sh.sL1;
    unsigned char* const sVk = sh.sVk;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: kept in a scalar register
    const int l32 = lane & 31, g = lane >> 5;
    // ---- which keys, which query rows.  The grid is one-dimensional and workgroup i runs on XCD i % 8
    // (each XCD has its own L2).  GATHER: all list tiles of one (batch, KV head, query slice) stream the
    // same Q and dO rows; they get consecutive slots of ONE XCD, so those rows are fetched from memory once
    // per XCD, not once per tile.  WINDOW: tiles in position order, latest first, spread over the XCDs.
    int key0, key_end;   // key ids of this workgroup: positions (WINDOW) or gather-list entries (GATHER)
    int ta, tb;          // query rows [ta, tb) of every head of the group
    int qa = 0;          // GATHER: first query chunk of the slice
    int slot = 0;        // GATHER: slot of the partials; WINDOW: part of the heads
    int h0, h1;          // heads [h0, h1) of the group
    int unit;
    {
        const int xcd = block & 7, seq = block >> 3;
        if (GATHER) {
            const int grp = xcd + 8 * (seq / P.gtiles);
            const int units = D.B * D.Hkv;
            if (grp >= units * P.nsl * P.hsl) return;
            unit = grp % units;
            slot = P.nsl * P.hsl - 1 - grp / units;   // latest slices (most list tiles) first
            key0 = (seq % P.gtiles) * KV_BK<W>;
            h0 = slot % P.hsl * D.G / P.hsl;
            h1 = (slot % P.hsl + 1) * D.G / P.hsl;
        } else {
            const int w = block % (P.ktiles * P.wsl);
            unit = block / (P.ktiles * P.wsl);
            if (unit >= D.B * D.Hkv) return;
            key0 = P.ktiles - 1 - w / P.wsl;          // tile index for now
            slot = w % P.wsl;
            h0 = slot * D.G / P.wsl;
            h1 = (slot + 1) * D.G / P.wsl;
        }
    }
    const int h = unit % D.Hkv, b = unit / D.Hkv;
    const int32_t* idx_h = idx + (int64_t(b) * D.Hkv + h) * D.Ns * D.K;
    if (GATHER) {
        // slice = query chunks [slice*qch, (slice+1)*qch), of which the tile sees those from qf on
        const int slice = slot / P.hsl;
        key_end = P.gl_total;
        const int qf = first_chunk_seeing(D, key0);
        qa = max(P.fq0 + slice * P.qch, qf);
        const int qb = min(P.fq1, P.fq0 + (slice + 1) * P.qch);
        if (qa >= qb) return;
        ta = D.S + qa * D.L;
        const int64_t e = int64_t(D.S) + int64_t(qb) * D.L;
        tb = e < D.n ? int(e) : D.n;
    } else {
        const int tix = key0;
        if (tix < P.sink_tiles_k) {
            key0 = tix * KV_BK<W>;
            key_end = D.S < D.n ? D.S : D.n;
            tb = key_end < D.row_end ? key_end : D.row_end;   // only sink queries see sink keys through the window
        } else {
            const int tt = tix - P.sink_tiles_k;
            const int kc = P.kc_lo + tt / P.tpc_k;
            key0 = D.S + kc * D.L + (tt % P.tpc_k) * KV_BK<W>;
            const int64_t e = int64_t(D.S) + int64_t(kc + 1) * D.L;
            key_end = e < D.n ? int(e) : D.n;
            const int64_t e2 = int64_t(D.S) + (int64_t(kc) + 1 + D.lp) * D.L;
            tb = e2 < D.row_end ? int(e2) : D.row_end;
        }
        if (key0 >= key_end) return;
        ta = key0 > D.row_begin ? key0 : D.row_begin;
        if (ta >= tb) return;
    }
    // Steps of KV_ROWS rows.  WINDOW: consecutive rows of [ta, tb).  GATHER: chunk by chunk (the last step
    // of a chunk may be partial), so that one step never sees two different gather-list prefixes.
    const int spc = (D.L + KV_ROWS<W> - 1) / KV_ROWS<W>;                               // GATHER: steps per chunk
    const int sph = GATHER ? ((tb - ta + D.L - 1) / D.L) * spc : (tb - ta + KV_ROWS<W> - 1) / KV_ROWS<W>;   // steps per head
    const int nsteps = sph * (h1 - h0);
    // first row, row end and chunk-visible limit of a step
    auto step_rows = [&](int sidx, int& r0, int& rend, int& lim_u) {
        const int w = sidx % sph;
        if (GATHER) {
            const int c = qa + w / spc;
            r0 = D.S + c * D.L + (w % spc) * KV_ROWS<W>;
            const int64_t e = int64_t(D.S) + int64_t(c + 1) * D.L;
            rend = e < tb ? int(e) : tb;
            lim_u = gather_count(D, c) - 1;
        } else {
            r0 = ta + w * KV_ROWS<W>;
            rend = tb;
            lim_u = 0;
        }
    };

    // ---- loader: wave w fills rows 8w .. 8w+7 of the Q and dO tiles (two copies of 4 rows each) and
    // its own lse|D block (one copy each).
    auto issue = [&](int step, unsigned char* sQ, unsigned char* sG, float* sL) {
        const int gi = step / sph;
        int r0, rend, lim_unused;
        step_rows(step, r0, rend, lim_unused);
        const int hq = h * D.G + h0 + gi;
        const int64_t base = b * D.qs[0] + hq * D.qs[1];
#pragma unroll
        for (int i = 0; i < KV_ROWS<W> / (COPY_ROWS<DH> * W); ++i) {
            const int rc = (KV_ROWS<W> / W) * wave + COPY_ROWS<DH> * i;
            const int row = async_row<DH>(rc, lane);
            const int t = min(r0 + row, rend - 1);
            const int64_t off = base + int64_t(t) * D.qs[2] + async_chunk<DH>(row, lane) * 8;
            async_rows<DH>(Q + off, sQ, rc);
            async_rows<DH>(dO + off, sG, rc);
        }
        const int64_t rid = (int64_t(b) * D.Hq + hq) * D.lse_stride + min(r0 + lane, rend - 1);
        async_copy4(lse + rid, sL + wave * 2 * KV_LD);
        async_copy4(Dsum + rid, sL + wave * 2 * KV_LD + KV_LD);
    };

    // the first step's rows are on their way while the keys are read (through idx: two trips to memory)
    issue(0, sQ0, sG0, sL0);

    // ---- this lane's key columns (one per 32-key block): K fragments stay in registers, the V rows
    // go to LDS in the swizzled tile layout (row = key within the workgroup)
    const int wave_key0 = key0 + wave * (32 * KV_NB);
    const bool wave_keys_valid = wave_key0 + 32 * KV_NB - 1 < key_end;
    int kcmp[KV_NB];
    bf16x8 kf[KV_NB][KK<DH>];
#pragma unroll
    for (int nb = 0; nb < KV_NB; ++nb) {
        const int kidn = wave_key0 + nb * 32 + l32;
        const bool kvalid = kidn < key_end;
        const int kid_ld = kvalid ? kidn : key_end - 1;
        kcmp[nb] = kvalid ? kidn : 0x7fffffff;
        // the key's K and V rows: by position, or (GATHER with a condensed cache) row kid of the contiguous copy
        const bf16_t *krow, *vrow_src;
        if (GATHER && D.compact) {
            const int64_t coff = ((int64_t(b) * D.Hkv + h) * P.gl_total + kid_ld) * DH;
            krow = Kc + coff;
            vrow_src = Vc + coff;
        } else {
            const int kpos = GATHER ? (kid_ld < D.S ? kid_ld : idx_h[kid_ld - D.S]) : kid_ld;
            const int64_t koff = b * D.ks[0] + h * D.ks[1] + int64_t(kpos) * D.ks[2];
            krow = K + koff;
            vrow_src = V + koff;
        }
#pragma unroll
        for (int kk = 0; kk < KK<DH>; ++kk) kf[nb][kk] = *reinterpret_cast<const bf16x8*>(krow + kk * 16 + g * 8);
        const int vrow = wave * (32 * KV_NB) + nb * 32 + l32;
#pragma unroll
        for (int kk = 0; kk < KK<DH>; ++kk)
            *reinterpret_cast<bf16x8*>(sVk + tile_off<DH>(vrow, kk * 2 + g)) =
                *reinterpret_cast<const bf16x8*>(vrow_src + kk * 16 + g * 8);
    }
    const unsigned char* sVw = sVk + wave * (32 * KV_NB) * ROW_BYTES<DH>;
    const LaneOffs lo = make_lane_offs<DH>(lane);

    const float c2 = D.scale * LOGIT_UNIT<DH>;
    f32x16 dk[KV_NB][DB<DH>], dv[KV_NB][DB<DH>];
#pragma unroll
    for (int nb = 0; nb < KV_NB; ++nb)
#pragma unroll
        for (int db = 0; db < DB<DH>; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) { dk[nb][db][i] = 0.0f; dv[nb][db][i] = 0.0f; }

#define LRSA_KV_STEP(step, sQ, sG, sL, sQn, sGn, sLn)                                                   \
    {                                                                                                    \
        wait_vmcnt<0>();     /* this wave's copies for `step` have landed */                             \
        __syncthreads();     /* ... everybody's have, and everybody is done with the other stage */      \
        if constexpr (DH == 64) clear_odd_rows<DH, W>(sQ, sG, sL + wave * 2 * KV_LD, lane);              \
        if ((step) + 1 < nsteps) issue((step) + 1, sQn, sGn, sLn);                                       \
        int r0s_, rend_, lim_u_;                                                                         \
        step_rows(step, r0s_, rend_, lim_u_);                                                            \
        _Pragma("unroll 1") for (int sub_ = 0; sub_ < KV_SUB<W>; ++sub_) {                                    \
            const int r0_ = r0s_ + sub_ * KV_BQ;                                                         \
            /* nothing to do: padding rows or keys only, rows that see none of the wave's keys.  The flag */ \
            /* is made opaque so that each sub-step body stays a basic block of its own: merged into one */ \
            /* block the bodies get interleaved and the register file overflows.                        */ \
            int run_ = (r0_ < rend_ && wave_key0 < key_end && (GATHER ? lim_u_ : r0_ + KV_BQ - 1) >= wave_key0) ? 1 : 0; \
            run_ = __builtin_amdgcn_readfirstlane(run_); /* wave-uniform by construction */              \
            asm volatile("" : "+s"(run_));                                                               \
            /* every (row, key) pair of the sub-step visible for this wave? */                           \
            const bool full_ = wave_keys_valid && r0_ + KV_BQ <= rend_ &&                                \
                               (GATHER ? lim_u_ >= wave_key0 + 32 * KV_NB - 1 : r0_ >= wave_key0 + 32 * KV_NB - 1); \
            if (run_)                                                                                    \
                dkv_step<DH, GATHER>(D, sQ, sG, sL + wave * 2 * KV_LD, kf, sVw, lo, dk, dv, r0_, rend_, kcmp, lim_u_, \
                                 !full_, c2, lane, sub_ * KV_BQ);                                        \
        }                                                                                                \
    }

    // the K fragments have arrived before the walk: the compiler then places
    // no vector-memory waits of its own in the loop (they would also wait for the copies in flight)
    wait_all_vmem_known();
#pragma unroll
    for (int nb = 0; nb < KV_NB; ++nb)
#pragma unroll
        for (int kk = 0; kk < KK<DH>; ++kk) pin_loaded(kf[nb][kk]);
    for (int step = 0; step < nsteps; step += 2) {
        LRSA_KV_STEP(step, sQ0, sG0, sL0, sQ1, sG1, sL1);
        if (step + 1 >= nsteps) break;
        LRSA_KV_STEP(step + 1, sQ1, sG1, sL1, sQ0, sG0, sL0);
    }
#undef LRSA_KV_STEP

    const size_t part_stride = size_t(D.B) * D.Hkv * P.gl_total * DH;   // floats per slice
    const size_t part_v = size_t(P.nsl * P.hsl + 1) * part_stride;        // dV partials follow the dK partials
    const int rows_here = key_end - wave_key0;                            // of the wave's 32 keys; the rest is padding
    if (rows_here <= 0) return;
    static_assert(KV_NB == 1, "a wave's keys are one block");
    unsigned char* const stage = sVk + wave * 32 * ROW_BYTES<DH>;
    const int srow = lane / (DH / 8), sch = lane % (DH / 8) * 4;          // row within a store, channel within a half row
    if (GATHER || P.wsl > 1) {
        // WINDOW with the heads in parts: [dK, dV][part][batch, KV head][position][DH], all added by the reduction kernel.
        // A lane holds one key's column: stored as it stands, an instruction would touch 32 rows by 32 bytes each.  Through the wave's
        // own V rows in LDS, which nobody reads any more, it stores whole lines of 4 rows (DH = 64: 8): 4 requests of 2.4K tokens, 8 heads
        // on 2, backward 176 -> 165 us, 3.1K tokens, 12 heads on 2, 134 -> 127 us; nothing where partials are few.
        const size_t wrow = size_t(D.B) * D.Hkv * (P.whi - P.wlo) * DH;
        float* pk = GATHER ? part + size_t(slot) * part_stride + ((size_t(b) * D.Hkv + h) * P.gl_total + wave_key0) * DH
                           : wpart + size_t(slot) * wrow + ((size_t(b) * D.Hkv + h) * (P.whi - P.wlo) + (wave_key0 - P.wlo)) * DH;
        float* pv = pk + (GATHER ? part_v : size_t(P.wsl) * wrow);
        auto put = [&](float* z, const f32x16 (&acc)[DB<DH>], float scale) {
            rows_through_lds<DH>(stage, acc, scale, lane, [&](int r0, int half, const f32x4& v) {
                if (r0 + srow < rows_here) *reinterpret_cast<f32x4*>(z + (r0 + srow) * DH + half * (DH / 2) + sch) = v;
            });
        };
        put(pk, dk[0], D.scale);
        put(pv, dv[0], 1.0f);
    } else {
        // listed positions: fp32 into the extra slot, the reduction kernel adds the slices; others: final.  As they stand (through LDS
        // 2 requests of 3.7K tokens, 8 heads on 8: backward 202 -> 206 us).
        const int kid = wave_key0 + l32;
        if (kid >= key_end) return;
        const int j = listed_entry(D, P, idx_h, kid);
        const int64_t koff = b * D.ks[0] + h * D.ks[1] + int64_t(kid) * D.ks[2];
        float* pk = j >= 0 ? part + size_t(P.nsl * P.hsl) * part_stride + ((size_t(b) * D.Hkv + h) * P.gl_total + j) * DH : nullptr;
#pragma unroll
        for (int db = 0; db < DB<DH>; ++db)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                f32x4 x, y;
#pragma unroll
                for (int r = 0; r < 4; ++r) { x[r] = dk[0][db][a * 4 + r] * D.scale; y[r] = dv[0][db][a * 4 + r]; }
                const int dcol = db * 32 + a * 8 + g * 4;
                if (j >= 0) {
                    *reinterpret_cast<f32x4*>(pk + dcol) = x;
                    *reinterpret_cast<f32x4*>(pk + part_v + dcol) = y;
                } else if (D.acc) {
                    // row window: this call's share is added to the caller's fp32 sums (one writer per element)
                    const int64_t aoff = ((int64_t(b) * D.Hkv + h) * D.n + kid) * DH + dcol;
                    *reinterpret_cast<f32x4*>(accK + aoff) += x;
                    *reinterpret_cast<f32x4*>(accV + aoff) += y;
                } else {
                    *reinterpret_cast<bf16x4*>(dK + koff + dcol) = __builtin_convertvector(x, bf16x4);
                    *reinterpret_cast<bf16x4*>(dV + koff + dcol) = __builtin_convertvector(y, bf16x4);
                }
            }
    }
}

// One launch for all of dK/dV, so that the chip has one tail, not two: the part with the longer workgroups first.
template <int DH, int W>
__global__ __launch_bounds__(64 * W, 2) void k_bwd_dkv(Dims D, const bf16_t* __restrict__ Q,
                                                                                const bf16_t* __restrict__ K,
                                                                                const bf16_t* __restrict__ V,
                                                                                const bf16_t* __restrict__ Kc,
                                                                                const bf16_t* __restrict__ Vc,
                                                                                const bf16_t* __restrict__ dO,
                                                                                const float* __restrict__ lse,
                                                                                const float* __restrict__ Dsum,
                                                                                const int32_t* __restrict__ idx,
                                                                                bf16_t* __restrict__ dK,
                                                                                bf16_t* __restrict__ dV,
                                                                                float* __restrict__ accK,
                                                                                float* __restrict__ accV,
                                                                                float* __restrict__ part,
                                                                                float* __restrict__ wpart, BwdPlan P) {
    const int first = P.window_first ? P.window_wgs : P.gather_wgs;
    const bool in_first = int(blockIdx.x) < first;
    const int block = in_first ? blockIdx.x : blockIdx.x - first;
    if (in_first != bool(P.window_first)) dkv_body<DH, W, true>(D, Q, K, V, Kc, Vc, dO, lse, Dsum, idx, dK, dV, accK, accV, part, wpart, P, block);
    else dkv_body<DH, W, false>(D, Q, K, V, Kc, Vc, dO, lse, Dsum, idx, dK, dV, accK, accV, part, wpart, P, block);
}

// dK, dV of the listed positions (sink tokens and survivors): the WINDOW contribution plus the GATHER slices
// that exist for the entry's list tile, added in a fixed order.  DH / 4 threads per entry, 4 channels each.
// With the heads of the WINDOW tiles in parts, entries whose position is in the window are left to a second range of rows,
// the positions [wlo, whi), listed or not.
template <int DH>
__global__ __launch_bounds__(256) void k_bwd_dkv_reduce(Dims D, const int32_t* __restrict__ idx,
                                                        const float* __restrict__ part, const float* __restrict__ wpart,
                                                        bf16_t* __restrict__ dK,
                                                        bf16_t* __restrict__ dV, float* __restrict__ accK,
                                                        float* __restrict__ accV, float* __restrict__ dKc,
                                                        float* __restrict__ dVc, BwdPlan P) {
    int64_t e = int64_t(blockIdx.x) * (1024 / DH) + threadIdx.x / (DH / 4);   // (b, h, entry), then (b, h, position)
    const int64_t total = int64_t(D.B) * D.Hkv * P.gl_total;
    const int wn = P.whi - P.wlo;
    const int dcol = (threadIdx.x & (DH / 4 - 1)) * 4;
    int j, bh, pos;
    f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f}, y = {0.0f, 0.0f, 0.0f, 0.0f};
    if (e < total) {
        j = int(e % P.gl_total);
        bh = int(e / P.gl_total);
        pos = j < D.S ? j : idx[(int64_t(bh) * D.Ns) * D.K + (j - D.S)];
    } else {
        const int64_t w = e - total;
        if (P.wsl == 1 || w >= int64_t(D.B) * D.Hkv * wn) return;
        bh = int(w / wn);
        pos = P.wlo + int(w % wn);
        j = listed_entry(D, P, idx + (int64_t(bh) * D.Ns) * D.K, pos);
        const size_t wrow = size_t(D.B) * D.Hkv * wn * DH;
        const float* p0 = wpart + size_t(w) * DH + dcol;
        for (int sl = 0; sl < P.wsl; ++sl) {
            x += *reinterpret_cast<const f32x4*>(p0 + size_t(sl) * wrow);
            y += *reinterpret_cast<const f32x4*>(p0 + size_t(P.wsl + sl) * wrow);
        }
        e = int64_t(bh) * P.gl_total + j;
    }
    const int b = bh / D.Hkv, h = bh % D.Hkv;
    // the WINDOW workgroups of this call cover the sink (with a row window: only when its rows are in it) and the
    // key chunks from kc_lo on
    const bool entry = int64_t(blockIdx.x) * (1024 / DH) + threadIdx.x / (DH / 4) < total;
    const bool in_window = pos < D.S ? P.sink_tiles_k > 0 : (pos - D.S) / D.L >= P.kc_lo;
    if (entry && in_window && P.wsl > 1) return;
    if (j >= 0) {
        const size_t part_stride = size_t(D.B) * D.Hkv * P.gl_total * DH;
        const int slots = P.nsl * P.hsl;
        const size_t part_v = size_t(slots + 1) * part_stride;
        const float* p0 = part + size_t(e) * DH + dcol;
        if (in_window && P.wsl == 1) {
            x = *reinterpret_cast<const f32x4*>(p0 + size_t(slots) * part_stride);
            y = *reinterpret_cast<const f32x4*>(p0 + size_t(slots) * part_stride + part_v);
        }
        const int qf0 = first_chunk_seeing(D, j / P.bk * P.bk);
        if (qf0 < P.fq1)
            for (int sl = qf0 > P.fq0 ? (qf0 - P.fq0) / P.qch * P.hsl : 0; sl < slots; ++sl) {
                x += *reinterpret_cast<const f32x4*>(p0 + size_t(sl) * part_stride);
                y += *reinterpret_cast<const f32x4*>(p0 + size_t(sl) * part_stride + part_v);
            }
    }
    if (D.acc) {
        const int64_t aoff = ((int64_t(b) * D.Hkv + h) * D.n + pos) * DH + dcol;
        *reinterpret_cast<f32x4*>(accK + aoff) += x;
        *reinterpret_cast<f32x4*>(accV + aoff) += y;
        return;
    }
    if (dKc && j >= 0) {   // condensed cache: the gradient of the condensed rows is a product of its own, scattered afterwards
        *reinterpret_cast<f32x4*>(dKc + e * DH + dcol) = x;
        *reinterpret_cast<f32x4*>(dVc + e * DH + dcol) = y;
        return;
    }
    const int64_t koff = b * D.ks[0] + h * D.ks[1] + int64_t(pos) * D.ks[2];
    *reinterpret_cast<bf16x4*>(dK + koff + dcol) = __builtin_convertvector(x, bf16x4);
    *reinterpret_cast<bf16x4*>(dV + koff + dcol) = __builtin_convertvector(y, bf16x4);
}

// Condensed cache: dKc, dVc [B, Hkv, gl, 128] fp32 -> rows of dK, dV at the positions of the gather list.  Every
// position occurs once in the list, so the scatter has no collisions and needs no addition.
__global__ __launch_bounds__(256) void k_bwd_scatter_dkv(Dims D, const int32_t* __restrict__ idx,
                                                         const float* __restrict__ dKc, const float* __restrict__ dVc,
                                                         bf16_t* __restrict__ dK, bf16_t* __restrict__ dV, int gl) {
    const int64_t e = int64_t(blockIdx.x) * 8 + (threadIdx.x >> 5);   // (b, h, entry)
    if (e >= int64_t(D.B) * D.Hkv * gl) return;
    const int j = int(e % gl), bh = int(e / gl);
    const int b = bh / D.Hkv, h = bh % D.Hkv;
    const int pos = j < D.S ? j : idx[(int64_t(bh) * D.Ns) * D.K + (j - D.S)];
    const int dcol = (threadIdx.x & 31) * 4;
    const int64_t koff = b * D.ks[0] + h * D.ks[1] + int64_t(pos) * D.ks[2];
    *reinterpret_cast<bf16x4*>(dK + koff + dcol) = __builtin_convertvector(*reinterpret_cast<const f32x4*>(dKc + e * 128 + dcol), bf16x4);
    *reinterpret_cast<bf16x4*>(dV + koff + dcol) = __builtin_convertvector(*reinterpret_cast<const f32x4*>(dVc + e * 128 + dcol), bf16x4);
}

// fp32 sums of a sequence of row-window calls -> dK, dV in the tensors' dtype (32 lanes per row)
__global__ __launch_bounds__(256) void k_bwd_acc_finish(Dims D, const float* __restrict__ accK,
                                                        const float* __restrict__ accV, bf16_t* __restrict__ dK,
                                                        bf16_t* __restrict__ dV) {
    const int64_t e = int64_t(blockIdx.x) * 8 + (threadIdx.x >> 5);   // (b, h, position)
    if (e >= int64_t(D.B) * D.Hkv * D.n) return;
    const int pos = int(e % D.n), bh = int(e / D.n);
    const int b = bh / D.Hkv, h = bh % D.Hkv;
    const int dcol = (threadIdx.x & 31) * 4;
    const f32x4 x = *reinterpret_cast<const f32x4*>(accK + e * 128 + dcol);
    const f32x4 y = *reinterpret_cast<const f32x4*>(accV + e * 128 + dcol);
    const int64_t koff = b * D.ks[0] + h * D.ks[1] + int64_t(pos) * D.ks[2];
    *reinterpret_cast<bf16x4*>(dK + koff + dcol) = __builtin_convertvector(x, bf16x4);
    *reinterpret_cast<bf16x4*>(dV + koff + dcol) = __builtin_convertvector(y, bf16x4);
}

hipError_t launch_bwd_acc_finish(const Dims& D, const float* accK, const float* accV, void* dK, void* dV, hipStream_t st) {
    const int64_t rows = int64_t(D.B) * D.Hkv * D.n;
    LRSA_TIMED_LAUNCH("k_bwd_acc_finish", st, k_bwd_acc_finish, dim3((unsigned)((rows + 7) / 8)), dim3(256), 0, st, D, accK,
                      accV, (bf16_t*)dK, (bf16_t*)dV);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------ launcher
hipError_t launch_attn_bwd_mfma(const Dims& D, const void* Q, const void* K, const void* V, const void* O,
                                const void* dO, const float* lse, const int32_t* idx, void* dQ, void* dK,
                                void* dV, float* accK, float* accV, void* ws, size_t ws_bytes, hipStream_t st) {
    const BwdPlan P = plan_for(D, ws_bytes);
    // D and lse in the logits' units hold the rows of the window only; like the caller's tensors they are addressed by
    // absolute row, hence the shifted bases
    float* Dsum = reinterpret_cast<float*>(ws) - D.row_begin;
    float* lse2 = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + P.off_lse2) - D.row_begin;
    float* part = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + P.off_part);
    const bf16_t *q = (const bf16_t*)Q, *k = (const bf16_t*)K, *v = (const bf16_t*)V, *o = (const bf16_t*)O,
                 *g = (const bf16_t*)dO;

    const bool compact = D.compact && P.gl_total > 0;
    const bf16_t *kc = nullptr, *vc = nullptr;
    {
        const int waves = qtile_waves(D);
        const QTileMap M = make_qtile_map(D, waves);
        const int64_t wgs = M.wgs;
        if (compact && wgs > 0) {
            kc = reinterpret_cast<const bf16_t*>(reinterpret_cast<const char*>(ws) + P.off_compact);
            vc = reinterpret_cast<const bf16_t*>(reinterpret_cast<const char*>(ws) + P.off_compact + compact_kv_bytes(D) / 2);
            const hipError_t e = launch_compact_kv(D, K, V, idx, (void*)kc, (void*)vc, st);
            if (e != hipSuccess) return e;
        }
#define LRSA_DQ_LAUNCH(DH_, W_, C_)                                                                              \
    LRSA_TIMED_LAUNCH("k_bwd_dq", st, (k_bwd_dq<DH_, W_, C_>), dim3((unsigned)wgs), dim3(64 * W_), 0, st, D, q, k, v, o, g, lse, \
                      Dsum, lse2, idx, kc, vc, (bf16_t*)dQ, M)
        if (wgs > 0) {
            if (D.d == 64) LRSA_DQ_LAUNCH(64, 4, false);
            else if (compact) LRSA_DQ_LAUNCH(128, 8, true);
            else if (waves == 4) LRSA_DQ_LAUNCH(128, 4, false);
            else LRSA_DQ_LAUNCH(128, 8, false);
        }
#undef LRSA_DQ_LAUNCH
    }
    float* wpart = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + P.off_wpart);
    const int64_t wgs = int64_t(P.gather_wgs) + P.window_wgs;
    if (wgs > 0)
        LRSA_TIMED_LAUNCH("k_bwd_dkv", st, (D.d == 64 ? k_bwd_dkv<64, 4> : P.waves == 4 ? k_bwd_dkv<128, 4> : k_bwd_dkv<128, 8>), dim3((unsigned)wgs), dim3(64 * P.waves), 0, st, D, q, k, v, kc, vc, g,
                          lse2, Dsum, idx, (bf16_t*)dK, (bf16_t*)dV, accK, accV, part, wpart, P);
    const int64_t entries = int64_t(D.B) * D.Hkv * P.gl_total;
    float *dkc = nullptr, *dvc = nullptr;
    if (compact) {
        dkc = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + P.off_dkc);
        dvc = dkc + align256(size_t(entries) * 128 * 4) / 4;
    }
    const int64_t rows = entries + (P.wsl > 1 ? int64_t(D.B) * D.Hkv * (P.whi - P.wlo) : 0);   // of the reduction
    if (rows > 0)
        LRSA_TIMED_LAUNCH("k_bwd_dkv_reduce", st, (D.d == 64 ? k_bwd_dkv_reduce<64> : k_bwd_dkv_reduce<128>),
                          dim3((unsigned)((rows + 1024 / D.d - 1) / (1024 / D.d))), dim3(256), 0, st, D,
                          idx, part, wpart, (bf16_t*)dK, (bf16_t*)dV, accK, accV, dkc, dvc, P);
    if (entries > 0 && compact)
        LRSA_TIMED_LAUNCH("k_bwd_scatter_dkv", st, k_bwd_scatter_dkv, dim3((unsigned)((entries + 7) / 8)), dim3(256), 0, st, D,
                          idx, dkc, dvc, (bf16_t*)dK, (bf16_t*)dV, P.gl_total);
    return hipGetLastError();
}

}  // namespace lrsa
