// LRSA attention forward on bf16 MFMA (gfx950), head_dim 128 or 64: Eq. 2-3 of the paper under the
// chunked mask, flash style (online softmax, only the log-sum-exp is kept for the backward).
//
// A wave owns a piece of 32 consecutive queries of one head; eight (or four) neighbouring pieces of one KV group and segment (the sink, or
// one chunk) make a workgroup (mfma_tiles.h, QTileMap, fwd_waves).  The keys those queries see form one
// stream: the gather list (sink, then the survivors of the compressed chunks) followed by the
// contiguous local window up to the query itself.  Stream entry j is visible to query t iff
// j <= ng + t - cs, so only the last tiles need a mask.  The stream is walked in tiles of 64
// keys; K and V rows of a tile are copied (gathered by position) asynchronously from global
// memory straight into an LDS ring, row-major and swizzled: of four stages, three tiles ahead, where the workgroup has the CU to itself; of
// two stages, one tile ahead, with four waves, where two workgroups share it and cover for each other.
//
// Per tile and wave:  S^T = K Q^T  (keys x queries, so a lane owns one query column and the
// softmax statistics are per lane), P^T = exp2(S^T - m), O^T += V^T P^T with the accumulator
// registers of S^T reused directly as the B operand and V^T read from the row-major tile with
// transposing LDS reads.
//
// head_dim 64: P^T enters as three bf16 terms (mfma_tiles.h, Weights), which is all of an fp32 weight, twice as many MFMAs
// in all; bound by the vector pipe (exponentials and the split).  8192 tokens, 16 query heads on 4 KV heads, lag 256, 64
// kept: 4.7 ms with the plain fp32-arithmetic kernel (a wave per query row) -> 0.14 ms; backward 14.2 ms -> 0.44 ms.  With two
// terms and logits in log2 units 0.125 and 0.40 ms, but 1.6 per mille of the elements of O are then off the correct rounding
// of the exact value, of dV 2.2 (1K to 4K rows, five kinds of values); now 0.22 and 0.41, the plain kernels 0.21 and 0.40.
#include "mfma_tiles.h"

namespace lrsa {

constexpr int FWD_BN = 64;     // keys per tile

// bf16 and a head's K/V rows within 2 GiB of its first row (the copies use 32-bit byte offsets)
bool mfma_supported(const Dims& D) {
    return D.dtype == 1 && int64_t(D.n) * D.ks[2] * 2 < (int64_t(1) << 31);
}
size_t attn_fwd_mfma_ws_bytes(const Dims& D) { return compact_kv_bytes(D); }

// Copies the K and V rows of every gather-list entry into the condensed cache: 16 lanes per row, 16 rows
// per workgroup.
__global__ __launch_bounds__(256) void k_compact_kv(Dims D, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
                                                    const int32_t* __restrict__ idx, bf16_t* __restrict__ Kc,
                                                    bf16_t* __restrict__ Vc, int gl) {
    const int j = blockIdx.x * 16 + (threadIdx.x >> 4), sub = threadIdx.x & 15;
    const int bh = blockIdx.y;
    if (j >= gl) return;
    const int b = bh / D.Hkv, h = bh % D.Hkv;
    const int pos = j < D.S ? j : idx[int64_t(bh) * D.Ns * D.K + (j - D.S)];
    const int64_t src = b * D.ks[0] + h * D.ks[1] + int64_t(pos) * D.ks[2] + sub * 8;
    const int64_t dst = (int64_t(bh) * gl + j) * 128 + sub * 8;
    *reinterpret_cast<uint4*>(Kc + dst) = *reinterpret_cast<const uint4*>(K + src);
    *reinterpret_cast<uint4*>(Vc + dst) = *reinterpret_cast<const uint4*>(V + src);
}

hipError_t launch_compact_kv(const Dims& D, const void* K, const void* V, const int32_t* idx, void* Kc, void* Vc,
                             hipStream_t st) {
    const int gl = gather_list_len(D);
    if (gl == 0) return hipSuccess;
    LRSA_TIMED_LAUNCH("k_compact_kv", st, k_compact_kv, dim3((gl + 15) / 16, D.B * D.Hkv), dim3(256), 0, st, D,
                      (const bf16_t*)K, (const bf16_t*)V, idx, (bf16_t*)Kc, (bf16_t*)Vc, gl);
    return hipGetLastError();
}

// One 64-key tile of the walk for one wave: S^T = K Q^T, masked online softmax, O^T += V^T P^T.
template <int DH>
struct FwdState {
    float m_run, l_run;
    f32x16 o[DB<DH>];
};

// MASK: the tile holds entries some query of the wave does not see (only the last tiles of a walk).
// The running maximum is refreshed lazily: as long as no query's tile maximum exceeds its reference
// by more than 2^8 (e^5), the old reference is kept (probabilities stay below 256, exact enough in fp32 sums
// and bf16 operands) and the accumulators need no rescaling.
template <int DH, bool MASK>
__device__ __forceinline__ void fwd_tile(const unsigned char* sK, const unsigned char* sV, const bf16x8 (&qf)[KK<DH>],
                                         const LaneOffs& lo_in, FwdState<DH>& st, int j0, int lim, int wave_lim_max,
                                         float c2, int lane) {
    const int g = lane >> 5;
    // DH = 64 (128 registers): the offsets are made opaque so that the XORed per-block offsets are formed next to each
    // read instead of being kept across the walk
    LaneOffs lo = lo_in;
    if constexpr (DH == 64) asm volatile("" : "+v"(lo.row), "+v"(lo.col));
    // MASK tiles: do the second 32 keys hold a visible key for some query of the wave?
    const bool two = !MASK || j0 + 32 <= wave_lim_max;
    f32x16 s[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[kb][i] = 0.0f;
    constexpr bool CLEAN = MASK && DH == 64;   // rows that a query does not see must not reach it, whatever they hold
    if constexpr (CLEAN) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int kk = 0; kk < KK<DH>; ++kk) s[kb] = poison_rows(read_rows_o<DH>(sV, lo, 32 * kb, kk), s[kb]);
    }
    // S^T = K Q^T: operands are read a block ahead of the MFMAs that consume them
    {
        bf16x8 a[KK<DH>];
#pragma unroll
        for (int kk = 0; kk < KK<DH>; ++kk) a[kk] = read_rows_o<DH>(sK, lo, 0, kk);
        if (two && DH == 64) {   // one block of operands at a time: 128 registers, and three other waves of the SIMD to wait behind
#pragma unroll
            for (int kk = 0; kk < KK<DH>; ++kk) s[0] = mfma32(a[kk], qf[kk], s[0]);
#pragma unroll
            for (int kk = 0; kk < KK<DH>; ++kk) a[kk] = read_rows_o<DH>(sK, lo, 32, kk);
#pragma unroll
            for (int kk = 0; kk < KK<DH>; ++kk) s[1] = mfma32(a[kk], qf[kk], s[1]);
        } else if (two) {
            bf16x8 a1[KK<DH>];
#pragma unroll
            for (int kk = 0; kk < KK<DH>; ++kk) {
                s[0] = mfma32(a[kk], qf[kk], s[0]);
                a1[kk] = read_rows_o<DH>(sK, lo, 32, kk);
            }
#pragma unroll
            for (int kk = 0; kk < KK<DH>; ++kk) s[1] = mfma32(a1[kk], qf[kk], s[1]);
            // keep the order written above -- 8 operand reads, then one read per MFMA, then 8 MFMAs: left alone,
            // the compiler moves every read down to just before its MFMA to save registers, and the MFMA then
            // waits out the whole LDS latency (0x100: LDS reads, 0x008: MFMAs)
            __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
        } else {
#pragma unroll
            for (int kk = 0; kk < KK<DH>; ++kk) s[0] = mfma32(a[kk], qf[kk], s[0]);
        }
    }
    // first V^T operands are fetched while the softmax runs
    bf16x8 va[DB<DH>], vb[DB<DH>];
#pragma unroll
    for (int db = 0; db < DB<DH>; ++db) va[db] = read_cols_o<DH>(sV, lo, 0, db);
    float mx = -INFINITY;   // raw (unscaled) tile maximum of this lane's query
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (MASK) {
                const int j = j0 + kb * 32 + 8 * (i >> 2) + 4 * g + (i & 3);
                s[kb][i] = j <= lim ? s[kb][i] : -INFINITY;
            }
            mx = fmaxf(mx, s[kb][i]);
        }
    const lanes_u32x2 x = pair32(__float_as_uint(mx));   // not through LDS, whose queue is full of operand reads
    mx = fmaxf(__uint_as_float(x.x), __uint_as_float(x.y)) * c2;
    if (__builtin_amdgcn_ballot_w64(mx > st.m_run + (DH == 64 ? 5.0f : 8.0f)) != 0) {   // wave-uniform; always taken on the first tile
        const float m_new = fmaxf(st.m_run, mx);   // finite: the first tile holds a visible key for every query
        const float corr = exp_units<DH>(st.m_run - m_new);
        st.l_run *= corr;
        st.m_run = m_new;
#pragma unroll
        for (int db = 0; db < DB<DH>; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) st.o[db][i] *= corr;
    }
    float psum = 0.0f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float pv = weight<DH>(s[kb][i], c2, st.m_run);
            s[kb][i] = pv;
            psum += pv;
        }
    st.l_run += psum;
    // O^T += V^T P^T, 16 keys at a time; the operands of the next 16 keys are read during the MFMAs
#define LRSA_PV(kg, cur, nxt)                                                          \
    {                                                                                  \
        const auto pf = pack_weights<TERMS<DH>>(s[(kg) >> 1], 8 * ((kg) & 1));         \
        _Pragma("unroll") for (int db = 0; db < DB<DH>; ++db) {                        \
            st.o[db] = mfma32_w(cur[db], pf, st.o[db]);                                \
            if ((kg) + 1 < 4) nxt[db] = read_cols_o<DH>(sV, lo, ((kg) + 1) * 16, db);  \
        }                                                                              \
    }
    if constexpr (DH == 64) {   // no registers for a second operand block
#pragma unroll
        for (int kg = 0; kg < 4; ++kg)
            if (kg < 2 || two) {
                // a term at a time, what is left of the weights in their own registers
                f32x16& w = s[kg >> 1];
                if constexpr (CLEAN)
#pragma unroll
                    for (int db = 0; db < DB<DH>; ++db) va[db] = finite_operand(va[db]);
#pragma unroll
                for (int t = 0; t < TERMS<DH>; ++t) {
                    const bf16x8 pf = pack8(w, 8 * (kg & 1));
#pragma unroll
                    for (int db = 0; db < DB<DH>; ++db) {
                        st.o[db] = mfma32(va[db], pf, st.o[db]);
                        if (t + 1 == TERMS<DH> && kg + 1 < 4) va[db] = read_cols_o<DH>(sV, lo, (kg + 1) * 16, db);
                    }
                    if (t + 1 < TERMS<DH>)
#pragma unroll
                        for (int j = 0; j < 8; ++j) w[8 * (kg & 1) + j] -= float(pf[j]);
                }
            }
    } else {
        LRSA_PV(0, va, vb);
        LRSA_PV(1, vb, va);
        if (two) {
            LRSA_PV(2, va, vb);
            LRSA_PV(3, vb, va);
        }
    }
#undef LRSA_PV
}

// COMPACT: the rows of the gather list come from the condensed cache Kc, Vc (contiguous), no index is read.
// DH = 64: three waves per SIMD; the 128 registers of a fourth would spill.
template <int DH, int WAVES, bool COMPACT>
__global__ __launch_bounds__(64 * WAVES, DH == 64 ? 3 : 2) void k_fwd_mfma(Dims D, const bf16_t* __restrict__ Q,
                                                              const bf16_t* __restrict__ K,
                                                              const bf16_t* __restrict__ V,
                                                              const int32_t* __restrict__ idx,
                                                              const bf16_t* __restrict__ Kc,
                                                              const bf16_t* __restrict__ Vc,
                                                              bf16_t* __restrict__ O, float* __restrict__ lse,
                                                              QTileMap M) {
    // the stages, each one array holding the K tile then the V tile; separate arrays per stage so that
    // reads of one stage need not wait for the asynchronous fill of another (the compiler tracks only a
    // handful of such arrays, hence K and V share one)
    constexpr int TILE_BYTES = FWD_BN * ROW_BYTES<DH>;
    constexpr int STAGES = WAVES == 8 ? 4 : 2, RPW = FWD_BN / WAVES;   // ring stages; tile rows a wave copies
    __shared__ __attribute__((aligned(16))) unsigned char sT0[2 * TILE_BYTES], sT1[2 * TILE_BYTES];
    __shared__ __attribute__((aligned(16))) unsigned char sT2[STAGES == 4 ? 2 * TILE_BYTES : 16], sT3[STAGES == 4 ? 2 * TILE_BYTES : 16];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, g = lane >> 5;
    int b, h, tix, qc, seg_end, tw, head, t_last;
    if (!decode_qtile(M, D, blockIdx.x, b, h, tix) || !qtile_rows(M, D, tix, WAVES, wave, qc, seg_end, tw, head, t_last)) return;   // uniform for the workgroup
    if constexpr (DH == 128) asm volatile("" : "+v"(tw));   // else the walk's branches become scalar, and zeros are kept in registers for them
    const int hq = h * D.G + head;
    const int ng = gather_count(D, qc), cs = window_start(D, qc);
    const int m_max = ng + t_last - cs + 1;           // stream entries the last row sees
    const int ntiles = (m_max + FWD_BN - 1) / FWD_BN;

    const bf16_t* Kh = K + b * D.ks[0] + h * D.ks[1];
    const bf16_t* Vh = V + b * D.ks[0] + h * D.ks[1];
    const int32_t* idx_h = idx + (int64_t(b) * D.Hkv + h) * D.Ns * D.K;
    const int64_t coff = COMPACT ? (int64_t(b) * D.Hkv + h) * (int64_t(D.S) + int64_t(D.K) * D.Ns) * 128 : 0;
    const bf16_t* Kc_h = Kc + coff;
    const bf16_t* Vc_h = Vc + coff;

    // this lane's query column
    const int tq = tw + l32;
    const int tq_ld = tq < seg_end ? tq : seg_end - 1;
    bf16x8 qf[KK<DH>];
    {
        const bf16_t* qrow = Q + b * D.qs[0] + hq * D.qs[1] + int64_t(tq_ld) * D.qs[2];
#pragma unroll
        for (int kk = 0; kk < KK<DH>; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qrow + kk * 16 + g * 8);
    }
    const int lim = ng + tq - cs;                                     // last stream entry this query sees
    // ... the wave's last valid query sees; a wave without one only copies
    const int wave_lim_max = tw < seg_end ? ng + min(tw + 31, seg_end - 1) - cs : -1;
    const int wave_lim_min = wave_lim_max < 0 ? -1 : ng + tw - cs;   // ... the wave's first query sees

    // loader: wave w fills tile rows RPW * w .. with asynchronous copies of 4 rows each (DH = 64: of 8 rows),
    // K and V alike; rows past the stream end re-read its last key and are masked.  The stream
    // positions a wave needs per tile are wave-uniform addresses, so they are fetched through the scalar
    // cache (one iteration ahead); the only vector memory operations in the loop are the asynchronous
    // copies, always OPS_PER_TILE per wave and tile, which lets s_waitcnt vmcnt(n) address a tile.
    const int32_t* idx_ld = D.Ns > 0 ? idx_h : reinterpret_cast<const int32_t*>(Kh);   // any readable words
    const int idx_last = D.Ns > 0 ? D.Ns * D.K - 1 : 0;
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    auto pos_entry = [&](int tc, int r) {   // clamped index into idx of row r of the wave's 8 tile rows
        const int e = min(tc * FWD_BN + RPW * wv + r, m_max - 1) - D.S;
        return e < 0 ? 0 : (e > idx_last ? idx_last : e);
    };
    struct Pos { Scalar8 e[RPW / 8]; };
    auto fetch_pos = [&](int tile, Pos& raw) {
        if (COMPACT) return;
        const int tc = tile < ntiles ? tile : ntiles - 1;   // past the end: repeat the last tile (never consumed)
#pragma unroll
        for (int i = 0; i < RPW / 8; ++i) {
            Scalar8& w = raw.e[i];
            w.a0 = smem_load(idx_ld, pos_entry(tc, 8 * i + 0)); w.a1 = smem_load(idx_ld, pos_entry(tc, 8 * i + 1));
            w.a2 = smem_load(idx_ld, pos_entry(tc, 8 * i + 2)); w.a3 = smem_load(idx_ld, pos_entry(tc, 8 * i + 3));
            w.a4 = smem_load(idx_ld, pos_entry(tc, 8 * i + 4)); w.a5 = smem_load(idx_ld, pos_entry(tc, 8 * i + 5));
            w.a6 = smem_load(idx_ld, pos_entry(tc, 8 * i + 6)); w.a7 = smem_load(idx_ld, pos_entry(tc, 8 * i + 7));
        }
    };
    auto wait_pos = [&](Pos& raw) {
        if (!COMPACT)
#pragma unroll
            for (int i = 0; i < RPW / 8; ++i) smem_wait(raw.e[i]);
    };
    // laK, laV: LDS byte addresses of the stage's K tile and V tile (compile-time constants at the call sites)
    auto issue = [&](int tile, Pos& raw, unsigned laK, unsigned laV) {
        const int tc = tile < ntiles ? tile : ntiles - 1;
        const int sub = async_row<DH>(0, lane);                         // this lane's row of a copy
        wait_pos(raw);
#pragma unroll
        for (int i = 0; i < RPW / COPY_ROWS<DH>; ++i) {
            const int r0 = RPW * wv + COPY_ROWS<DH> * i;
            int j = tc * FWD_BN + r0 + sub;
            j = j < m_max ? j : m_max - 1;
            const int ch = async_chunk<DH>(r0 + sub, lane) * 8;
            const unsigned row_la = unsigned(r0) * ROW_BYTES<DH>;       // wave-uniform
            if (COMPACT) {
                async_copy16_la(stream_row(Kc_h, Kh, D.ks[2], j, ng, cs) + ch, laK + row_la);
                async_copy16_la(stream_row(Vc_h, Vh, D.ks[2], j, ng, cs) + ch, laV + row_la);
            } else {
                const Scalar8& w = raw.e[i * COPY_ROWS<DH> / 8];
                const int lo4 = pick4(sub & 3, w.a0, w.a1, w.a2, w.a3), hi4 = pick4(sub & 3, w.a4, w.a5, w.a6, w.a7);
                const int sel = DH == 128 ? (i % 2 == 0 ? lo4 : hi4) : (sub < 4 ? lo4 : hi4);
                const int pos = j < ng ? (j < D.S ? j : sel) : cs + (j - ng);
                // byte offset inside the head: below 2^31 (a condition of this kernel, checked on the host)
                const unsigned off = (unsigned(pos) * unsigned(D.ks[2]) + unsigned(ch)) * 2u;
                async_copy16_so(Kh, off, laK + row_la);
                async_copy16_so(Vh, off, laV + row_la);
            }
        }
    };
    constexpr int OPS_PER_TILE = 2 * RPW / COPY_ROWS<DH>;   // asynchronous copies per wave and tile

    const float c2 = D.scale * LOGIT_UNIT<DH>;
    const LaneOffs lo = make_lane_offs<DH>(lane);
    FwdState<DH> st;
    st.m_run = -INFINITY;
    st.l_run = 0.0f;
#pragma unroll
    for (int db = 0; db < DB<DH>; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) st.o[db][i] = 0.0f;

#define LRSA_FWD_TILE(sK, sV, j0_)                                                                   \
    {                                                                                                \
        const int j0 = (j0_);                                                                        \
        if (j0 + FWD_BN - 1 <= wave_lim_min) fwd_tile<DH, false>(sK, sV, qf, lo, st, j0, lim, wave_lim_max, c2, lane); \
        else if (j0 <= wave_lim_max) fwd_tile<DH, true>(sK, sV, qf, lo, st, j0, lim, wave_lim_max, c2, lane);          \
    }

    // A wave's vector memory operations in order:  A(0) A(1) A(2) | iteration t: A(t+3)   (A = the copies
    // of a tile).  At the top of iteration t the operations issued after A(t) are A(t+1) A(t+2).
    Pos pos;   // of the tile that is copied next
    if constexpr (STAGES == 4) {
        const unsigned la0 = lds_addr(sT0), la1 = lds_addr(sT1), la2 = lds_addr(sT2), la3 = lds_addr(sT3);
        Pos pos1, pos2;      // one trip to memory for all three
        fetch_pos(0, pos); fetch_pos(1, pos1); fetch_pos(2, pos2);
        issue(0, pos, la0, la0 + TILE_BYTES);
        issue(1, pos1, la1, la1 + TILE_BYTES);
        issue(2, pos2, la2, la2 + TILE_BYTES);
        fetch_pos(3, pos);
        wait_all_vmem_known();   // the Q fragments (and the first tiles) are here
#define LRSA_FWD_STEP(t_, sT, laN)                                                                   \
    {                                                                                                \
        wait_vmcnt<2 * OPS_PER_TILE>();   /* this wave's copies for tile t_ have landed */            \
        ring_barrier();                   /* everybody's have; everybody is done with tile t_-1 */   \
        issue((t_) + 3, pos, laN, laN + TILE_BYTES); /* tile t_+3 into the stage tile t_-1 used */    \
        fetch_pos((t_) + 4, pos);         /* after the copies: their wait for positions is for ALL scalar loads */ \
        LRSA_FWD_TILE(sT, sT + TILE_BYTES, (t_) * FWD_BN);                                           \
    }
        for (int tile = 0; tile < ntiles; tile += 4) {
            LRSA_FWD_STEP(tile, sT0, la3);
            if (tile + 1 >= ntiles) break;
            LRSA_FWD_STEP(tile + 1, sT1, la0);
            if (tile + 2 >= ntiles) break;
            LRSA_FWD_STEP(tile + 2, sT2, la1);
            if (tile + 3 >= ntiles) break;
            LRSA_FWD_STEP(tile + 3, sT3, la2);
        }
#undef LRSA_FWD_STEP
    } else {
        const unsigned la0 = lds_addr(sT0), la1 = lds_addr(sT1);
        Pos pos0;
        fetch_pos(0, pos0); fetch_pos(1, pos);
        issue(0, pos0, la0, la0 + TILE_BYTES);
        wait_all_vmem_known();
#define LRSA_FWD_STEP2(t_, sT, laN)                                                                   \
    {                                                                                                \
        wait_vmcnt<0>();                                                                              \
        ring_barrier();                                                                              \
        if ((t_) + 1 < ntiles) {                                                                      \
            issue((t_) + 1, pos, laN, laN + TILE_BYTES);                                              \
            fetch_pos((t_) + 2, pos);                                                                 \
        }                                                                                            \
        LRSA_FWD_TILE(sT, sT + TILE_BYTES, (t_) * FWD_BN);                                           \
    }
        for (int tile = 0; tile < ntiles; tile += 2) {
            LRSA_FWD_STEP2(tile, sT0, la1);
            if (tile + 1 >= ntiles) break;
            LRSA_FWD_STEP2(tile + 1, sT1, la0);
        }
#undef LRSA_FWD_STEP2
    }
    wait_pos(pos);     // the last positions, which nobody uses, must not land in registers that the epilogue has taken
    wait_vmcnt<0>();   // copies issued past the end must land before the workgroup's LDS is released
#undef LRSA_FWD_TILE

    const float l_tot = st.l_run + __shfl_xor(st.l_run, 32, 64);
    // row and head once more, from scalars: kept across the walk they would cost vector registers
    int tw_o, head_o;
    qtile_rows(M, D, tix, WAVES, wv, qc, seg_end, tw_o, head_o, t_last);
    const int hq_o = h * D.G + head_o, tq_o = tw_o + l32;
    if (tq_o < seg_end) {
        const float inv = 1.0f / l_tot;
        bf16_t* orow = O + b * D.qs[0] + hq_o * D.qs[1] + int64_t(tq_o) * D.qs[2];
#pragma unroll
        for (int db = 0; db < DB<DH>; ++db)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                f32x4 v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = st.o[db][a * 4 + r] * inv;
                const bf16x4 pk = __builtin_convertvector(v, bf16x4);
                *reinterpret_cast<bf16x4*>(orow + db * 32 + a * 8 + g * 4) = pk;
            }
        // m in natural units: one rounding at the end
        const float lse_t = DH == 64 ? __builtin_fmaf(__builtin_log2f(l_tot), 0.6931471805599453f, st.m_run)
                                     : (st.m_run + __builtin_log2f(l_tot)) * 0.6931471805599453f;
        if (g == 0) lse[(int64_t(b) * D.Hq + hq_o) * D.lse_stride + tq_o] = lse_t;
    }
}

int attn_mfma_fwd_waves(const Dims& D) { return fwd_waves(D); }

hipError_t launch_attn_fwd_mfma(const Dims& D, const void* Q, const void* K, const void* V, const int32_t* idx,
                                void* O, float* lse, void* ws, hipStream_t st) {
    const int waves = fwd_waves(D);
    const QTileMap M = make_qtile_map(D, waves);
    const int64_t wgs = M.wgs;
    if (wgs == 0) return hipSuccess;
    const bf16_t *q = (const bf16_t*)Q, *k = (const bf16_t*)K, *v = (const bf16_t*)V;
    const bool compact = D.compact && gather_list_len(D) > 0;
    const bf16_t *kc = nullptr, *vc = nullptr;
    if (compact) {
        kc = reinterpret_cast<const bf16_t*>(ws);
        vc = reinterpret_cast<const bf16_t*>(reinterpret_cast<const char*>(ws) + compact_kv_bytes(D) / 2);
        const hipError_t e = launch_compact_kv(D, K, V, idx, (void*)kc, (void*)vc, st);
        if (e != hipSuccess) return e;
    }
#define LRSA_FWD_LAUNCH(DH_, W_, C_)                                                                                   \
    LRSA_TIMED_LAUNCH("k_fwd_mfma", st, (k_fwd_mfma<DH_, W_, C_>), dim3((unsigned)wgs), dim3(64 * W_), 0, st, D, q, k, v, \
                      idx, kc, vc, (bf16_t*)O, lse, M)
    if (D.d == 64) { if (waves == 8) LRSA_FWD_LAUNCH(64, 8, false); else LRSA_FWD_LAUNCH(64, 4, false); }
    else if (compact) LRSA_FWD_LAUNCH(128, 8, true);
    else if (waves == 4) LRSA_FWD_LAUNCH(128, 4, false);
    else LRSA_FWD_LAUNCH(128, 8, false);
#undef LRSA_FWD_LAUNCH
    return hipGetLastError();
}

}  // namespace lrsa
