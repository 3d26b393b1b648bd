// LRSA attention on fp32 data, forward and backward (Eq. 2-3 of the paper under the chunked mask), on the fp32 matrix
// instruction v_mfma_f32_16x16x4_f32 (gfx950), head_dim 64 or 128.  Operands, weights and sums are fp32 throughout.
//
// Nothing is staged in LDS: an operand is read from memory (the caches: rows are shared by neighbouring workgroups) in
// the order the instruction wants it.  Lane l, c = l % 16, q4 = l / 16:
//   A operand: row c, k-slot q4     B operand: column c, k-slot q4     C/D: column c, register i -> row 4*q4 + i
// A contraction over head_dim may take the channels in any order, so the lane reads 16 bytes, channels 16j + 4*q4 .. +3 of
// row c, and feeds them to four instructions ("row fragment").  A contraction over 16 keys (queries) takes register i of a
// C-layout block as its B operand, k-slot q4 being key 4*q4 + i; the A operand, the transpose of a row-major tile, is 16
// bytes of row 4*q4 + i, channels 64*grp + 4c .. +3: one channel for each of four output blocks, whose row m is channel
// 64*grp + 4m + block ("column fragment").
//
// Query-outer (forward, dQ): a workgroup owns 16 query rows of one head; its W waves take the 16-key tiles of
// the visible stream (gather list, then the local window) in turn, each with a softmax state of its own, and are merged in
// LDS in a fixed order.  Key-outer (dK, dV): a workgroup owns 16 keys that are seen by about the same rows -- sink tokens,
// survivors of one chunk (all later rows), or the rest of a chunk (up to the end of the local window) -- and its waves take
// the 16-row query tiles of the group's heads in turn.  Deterministic, no atomics; partial sums go through memory only
// where a problem is too small to fill the chip with one workgroup per 16 keys.
//
// Bound by latency for short sequences (few query tiles: the waves of a workgroup split one row's keys for that reason) and
// by the fp32 matrix rate (157 TFLOP/s) beyond.  Against the plain kernels, which give a query row (a key) to a wave: a
// training step of 1024 rows, one head of 64 channels, 118 -> 58 us; 2-norm errors against 64 bits 0.6 to 0.9 of theirs.
#include "common.h"

namespace lrsa {

typedef float fx4 __attribute__((ext_vector_type(4)));

template <int DH> constexpr int F32_WAVES = DH == 64 ? 16 : 8;   // 128 (256) registers per lane

// Keys of the longest walk: the last query chunk, which may be a short one, the chunk before it, or the sink's last row.
static int64_t longest_walk(const Dims& D) {
    int64_t keys = D.S < D.n ? D.S : D.n;
    for (int q = D.nq - 1; q >= 0 && q >= D.nq - 2; --q) {
        const int64_t end = int64_t(D.S) + (int64_t(q) + 1) * D.L, k = gather_count(D, q) + (end < D.n ? end : D.n) - window_start(D, q);
        keys = k > keys ? k : keys;
    }
    return keys;
}

// Waves of a query-outer workgroup: F32_WAVES, so that few query tiles still fill the chip, or half of that, or four, where there are
// more of them: a wave then takes more than the two or three key tiles that it has of 16 waves, and fewer states are merged.  As long as
//  - the chip holds the waves (head_dim 128: twice as many; with only as many 1.2K tokens, 4 heads on 4, take 31 us instead of 23);
//  - a wave has at most 16 key tiles (head_dim 128: 8) of the longest walk.  It adds its tiles one after another, and their rounding
//    grows with their number: 2-norm error of O against 64 bits, over that with all waves, of the last rows of uncompressed sequences,
//    five kinds of values: head_dim 64, four waves 0.93 to 1.01 up to 1024 keys, 1.00 to 1.04 at 2048, 1.02 to 1.08 at 4096, 1.05 to 1.26
//    at 12288; eight waves 0.94 to 1.005 up to 2048, 1.08 at 12288; head_dim 128, four waves 0.96 to 1.005 up to 512, 1.015 at 768,
//    1.07 at 4096, 1.13 at 12288.  Of dQ, whose error jumps more from one set of rows to the next, 0.77 to 1.05 up to these lines, 1.28 beyond;
//  - sixteen waves of walks beyond 512 keys are more than 1.6 times what the chip holds: with 1.0 to 1.6 times as many eight waves are
//    twice as long and leave the second round's gain behind (2.1K tokens, 2 heads on 1, 33 survivors of 65: forward 20.3 us with sixteen, 24.2
//    with eight; 14 shapes between 1.02 and 1.19 in the forward, up to 1.09 in the backward); up to 512 keys 0.82 to 0.95.
// 2 requests of 2.0K tokens, 8 heads of 64 on 2: forward 97 -> 72 us, backward 345 -> 300.
static int f32_query_waves(const Dims& D, int64_t tiles) {
    const int most = D.d == 64 ? F32_WAVES<64> : F32_WAVES<128>, rounds = D.d == 64 ? 1 : 2, wave_keys = D.d == 64 ? 256 : 128;
    const int64_t keys = longest_walk(D);
    int w = most;
    while (w > 4 && tiles * w > rounds * 256 * int64_t(most) * (w == 16 && keys > 512 ? 1.6 : 1.0) && keys <= w / 2 * wave_keys) w /= 2;
    return w;
}

__device__ __forceinline__ fx4 mfma_f32(float a, float b, fx4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <int DH> struct RowFrag { fx4 v[DH / 16]; };
template <int DH>
__device__ __forceinline__ RowFrag<DH> row_frag(const float* row, int q4) {
    RowFrag<DH> f;
#pragma unroll
    for (int j = 0; j < DH / 16; ++j) f.v[j] = *reinterpret_cast<const fx4*>(row + 16 * j + 4 * q4);
    return f;
}
// rows of a x columns of b, over head_dim; in two chains, whose shorter sums round less than the plain kernels' one chain
template <int DH>
__device__ __forceinline__ fx4 dot_tile(const RowFrag<DH>& a, const RowFrag<DH>& b) {
    fx4 s[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
    for (int j = 0; j < DH / 32; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int k = 0; k < 2; ++k) s[k] = mfma_f32(a.v[2 * j + k][e], b.v[2 * j + k][e], s[k]);
    return s[0] + s[1];
}
// [DH channels x 16 columns] sums: block [grp][e], register r <-> channel 64*grp + 16*q4 + 4*r + e
template <int DH> struct Acc { fx4 v[DH / 64][4]; };
template <int DH>
__device__ __forceinline__ void zero(Acc<DH>& a) {
#pragma unroll
    for (int g = 0; g < DH / 64; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) a.v[g][e] = fx4{0.0f, 0.0f, 0.0f, 0.0f};
}
template <int DH> struct ColFrag { fx4 v[DH / 64]; };
template <int DH>
__device__ __forceinline__ ColFrag<DH> col_frag(const float* row, int c) {
    ColFrag<DH> f;
#pragma unroll
    for (int g = 0; g < DH / 64; ++g) f.v[g] = *reinterpret_cast<const fx4*>(row + 64 * g + 4 * c);
    return f;
}
template <int DH>
__device__ __forceinline__ void add_outer(Acc<DH>& a, const ColFrag<DH>& f, float w) {
#pragma unroll
    for (int g = 0; g < DH / 64; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) a.v[g][e] = mfma_f32(f.v[g][e], w, a.v[g][e]);
}
// a = a * f + t.  The sums of a 16-row tile are formed on their own and then added: a long sum takes a rounding of its own
// magnitude per tile, not per instruction (dV of 1500 rows, 2-norm error against 64 bits: 5.4e-7 -> 4.3e-7, the plain
// kernels' 4.3e-7)
template <int DH>
__device__ __forceinline__ void add_acc(Acc<DH>& a, float f, const Acc<DH>& t) {
#pragma unroll
    for (int g = 0; g < DH / 64; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int r = 0; r < 4; ++r) a.v[g][e][r] = __builtin_fmaf(a.v[g][e][r], f, t.v[g][e][r]);
}
// into row c of a [16][DH + 4] LDS tile (the padding spreads the 16 rows over the banks)
template <int DH> constexpr int LROW = DH + 4;
template <int DH>
__device__ __forceinline__ void put_acc(float* tile, const Acc<DH>& a, int c, int q4) {
#pragma unroll
    for (int g = 0; g < DH / 64; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<fx4*>(tile + c * LROW<DH> + 64 * g + 16 * q4 + 4 * r) = fx4{a.v[g][0][r], a.v[g][1][r], a.v[g][2][r], a.v[g][3][r]};
}
// over the four lanes that hold a column
template <class Op>
__device__ __forceinline__ float col_all(float v, Op op) {
    lanes_u32x2 a = pair32(__float_as_uint(v));
    v = op(__uint_as_float(a.x), __uint_as_float(a.y));
    a = pair16(__float_as_uint(v));
    return op(__uint_as_float(a.x), __uint_as_float(a.y));
}

// A tile in which some (query, key) pairs are masked: a weight of zero times an infinity would be NaN in the sums of a query (key)
// that does not see the row.  The operand's non-finite values become zeros there; the return value says whether the row that this
// lane's register i stands for has any, and the weights of the pairs that do see it become NaN.
template <int DH>
__device__ __forceinline__ bool clean_row(ColFrag<DH>& f, int q4) {
    bool bad = false;
#pragma unroll
    for (int g = 0; g < DH / 64; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool x = !__builtin_isfinite(f.v[g][e]);
            f.v[g][e] = x ? 0.0f : f.v[g][e];
            bad |= x;
        }
    return (__builtin_amdgcn_ballot_w64(bad) >> (16 * q4) & 0xffff) != 0;   // over the 16 lanes that hold the row
}

// Query tiles of 16 rows inside the sink and inside every chunk; the latest (most keys) first.
struct QTiles { int sink, tpc, count; };
static QTiles make_qtiles(const Dims& D) {
    QTiles T;
    T.sink = ((D.S < D.n ? D.S : D.n) + 15) / 16;
    T.tpc = (D.L + 15) / 16;
    T.count = T.sink + D.nq * T.tpc;
    return T;
}
struct QRange { int t0, t_last, ng, cs; };   // rows t0 .. t_last; entries of the gather list, start of the window
__device__ __forceinline__ bool query_rows(const Dims& D, const QTiles& T, int tix, QRange& R) {
    int qc = -1, end = D.S < D.n ? D.S : D.n;
    R.t0 = tix * 16;
    if (tix >= T.sink) {
        const int tt = tix - T.sink;
        qc = tt / T.tpc;
        R.t0 = D.S + qc * D.L + tt % T.tpc * 16;
        const int64_t e = int64_t(D.S) + int64_t(qc + 1) * D.L;
        end = e < D.n ? int(e) : D.n;
    }
    if (R.t0 >= end) return false;
    R.t_last = min(R.t0 + 16, end) - 1;
    R.ng = gather_count(D, qc);
    R.cs = window_start(D, qc);
    return true;
}
__device__ __forceinline__ int stream_row(const Dims& D, const int32_t* idx_h, int j, const QRange& R) {
    if (j < R.ng) return j < D.S ? j : idx_h[j - D.S];
    return R.cs + (j - R.ng);
}

// ------------------------------------------------------------------------------------ forward
template <int DH, int W>
__global__ __launch_bounds__(64 * W, DH == 64 ? 4 : 2) void k_fwd_f32(Dims D, const float* __restrict__ Q, const float* __restrict__ K,
                                                                const float* __restrict__ V, const int32_t* __restrict__ idx,
                                                                float* __restrict__ O, float* __restrict__ lse, QTiles T) {
    __shared__ __attribute__((aligned(16))) float sO[W][16 * LROW<DH>];
    __shared__ float sM[W][16], sL[W][16];
    const int heads = D.B * D.Hq;
    const int bh = blockIdx.x % heads, b = bh / D.Hq, hq = bh % D.Hq, h = hq / D.G;
    QRange R;
    if (!query_rows(D, T, T.count - 1 - int(blockIdx.x) / heads, R)) return;   // uniform for the workgroup
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 15, q4 = lane >> 4;
    const int m_max = R.ng + R.t_last - R.cs + 1;
    const float* Kh = K + b * D.ks[0] + h * D.ks[1];
    const float* Vh = V + b * D.ks[0] + h * D.ks[1];
    const int32_t* idx_h = idx + (int64_t(b) * D.Hkv + h) * D.Ns * D.K;
    const int64_t qoff = b * D.qs[0] + hq * D.qs[1];

    const int tr = min(R.t0 + c, R.t_last);
    const RowFrag<DH> q = row_frag<DH>(Q + qoff + int64_t(tr) * D.qs[2], q4);
    const int lim = R.ng + tr - R.cs;                    // last stream entry the lane's query sees
    const int lim_min = R.ng + R.t0 - R.cs;              // ... the first query sees
    float m = -INFINITY, l = 0.0f;
    Acc<DH> o;
    zero(o);
    for (int j0 = wave * 16; j0 < m_max; j0 += 16 * W) {
        const int pos = stream_row(D, idx_h, min(j0 + c, m_max - 1), R);
        const RowFrag<DH> k = row_frag<DH>(Kh + int64_t(pos) * D.ks[2], q4);
        ColFrag<DH> v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = col_frag<DH>(Vh + int64_t(__shfl(pos, 4 * q4 + i, 64)) * D.ks[2], c);
        fx4 s = dot_tile<DH>(k, q);
        if (j0 + 15 > lim_min) {
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = clean_row<DH>(v[i], q4) ? NAN : s[i];
        }
        float mx = m;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s[i] = j0 + 4 * q4 + i <= lim ? D.scale * s[i] : -INFINITY;
            mx = fmaxf(mx, s[i]);
        }
        mx = col_all(mx, [](float x, float y) { return fmaxf(x, y); });
        const float ref = mx == -INFINITY ? 0.0f : mx;   // a query that has seen no key in this wave yet
        const float corr = expf(m - ref);
        m = mx;
        Acc<DH> t;
        zero(t);
        float ps = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float p = expf(s[i] - ref);
            ps += p;
            add_outer<DH>(t, v[i], p);
        }
        l = __builtin_fmaf(l, corr, ps);
        add_acc<DH>(o, corr, t);
    }
    l = col_all(l, [](float x, float y) { return x + y; });
    put_acc<DH>(sO[wave], o, c, q4);
    if (q4 == 0) { sM[wave][c] = m; sL[wave][c] = l; }
    __syncthreads();
    const int waves = min(W, (m_max + 15) / 16);          // waves that saw a key tile
    for (int e = threadIdx.x; e < 16 * (DH / 4); e += 64 * W) {
        const int row = e / (DH / 4), ch = e % (DH / 4) * 4, t = R.t0 + row;
        if (t > R.t_last) continue;
        float M = -INFINITY;
        for (int w = 0; w < waves; ++w) M = fmaxf(M, sM[w][row]);
        float L = 0.0f;
        fx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int w = 0; w < waves; ++w) {
            const float f = expf(sM[w][row] - M);          // 0 for a wave whose tiles the row does not see
            L += f * sL[w][row];
            acc += f * *reinterpret_cast<const fx4*>(&sO[w][row * LROW<DH> + ch]);
        }
        *reinterpret_cast<fx4*>(O + qoff + int64_t(t) * D.qs[2] + ch) = acc / L;
        if (ch == 0) lse[int64_t(bh) * D.n + t] = M + logf(L);
    }
}

// ------------------------------------------------------------------------------------ backward: dQ (and D)
template <int DH, int W>
__global__ __launch_bounds__(64 * W, DH == 64 ? 4 : 2) void k_bwd_dq_f32(Dims D, const float* __restrict__ Q, const float* __restrict__ K,
                                                                   const float* __restrict__ V, const float* __restrict__ O,
                                                                   const float* __restrict__ dO, const float* __restrict__ lse,
                                                                   const int32_t* __restrict__ idx, float* __restrict__ dQ,
                                                                   float* __restrict__ Dsum, QTiles T) {
    __shared__ __attribute__((aligned(16))) float sQ[W][16 * LROW<DH>];
    const int heads = D.B * D.Hq;
    const int bh = blockIdx.x % heads, b = bh / D.Hq, hq = bh % D.Hq, h = hq / D.G;
    QRange R;
    if (!query_rows(D, T, T.count - 1 - int(blockIdx.x) / heads, R)) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 15, q4 = lane >> 4;
    const int m_max = R.ng + R.t_last - R.cs + 1;
    const float* Kh = K + b * D.ks[0] + h * D.ks[1];
    const float* Vh = V + b * D.ks[0] + h * D.ks[1];
    const int32_t* idx_h = idx + (int64_t(b) * D.Hkv + h) * D.Ns * D.K;
    const int64_t qoff = b * D.qs[0] + hq * D.qs[1];

    const int t = R.t0 + c, tr = min(t, R.t_last);
    const int lim = R.ng + tr - R.cs, lim_min = R.ng + R.t0 - R.cs;
    const RowFrag<DH> q = row_frag<DH>(Q + qoff + int64_t(tr) * D.qs[2], q4), g = row_frag<DH>(dO + qoff + int64_t(tr) * D.qs[2], q4);
    const float ls = lse[int64_t(bh) * D.n + tr];
    float Dt = 0.0f;
    {
        const RowFrag<DH> o = row_frag<DH>(O + qoff + int64_t(tr) * D.qs[2], q4);
#pragma unroll
        for (int j = 0; j < DH / 16; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) Dt = __builtin_fmaf(g.v[j][e], o.v[j][e], Dt);
        Dt = col_all(Dt, [](float x, float y) { return x + y; });
    }
    if (wave == 0 && q4 == 0 && t <= R.t_last) Dsum[int64_t(bh) * D.n + t] = Dt;
    Acc<DH> dq;
    zero(dq);
    for (int j0 = wave * 16; j0 < m_max; j0 += 16 * W) {
        const int pos = stream_row(D, idx_h, min(j0 + c, m_max - 1), R);
        const RowFrag<DH> k = row_frag<DH>(Kh + int64_t(pos) * D.ks[2], q4), v = row_frag<DH>(Vh + int64_t(pos) * D.ks[2], q4);
        ColFrag<DH> kc[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) kc[i] = col_frag<DH>(Kh + int64_t(__shfl(pos, 4 * q4 + i, 64)) * D.ks[2], c);
        fx4 s = dot_tile<DH>(k, q);
        const fx4 dp = dot_tile<DH>(v, g);
        if (j0 + 15 > lim_min) {
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = clean_row<DH>(kc[i], q4) ? NAN : s[i];
        }
        Acc<DH> t16;
        zero(t16);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float ds = expf(D.scale * s[i] - ls) * (dp[i] - Dt);
            add_outer<DH>(t16, kc[i], j0 + 4 * q4 + i <= lim ? ds : 0.0f);
        }
        add_acc<DH>(dq, 1.0f, t16);
    }
    put_acc<DH>(sQ[wave], dq, c, q4);
    __syncthreads();
    const int waves = min(W, (m_max + 15) / 16);
    for (int e = threadIdx.x; e < 16 * (DH / 4); e += 64 * W) {
        const int row = e / (DH / 4), ch = e % (DH / 4) * 4;
        if (R.t0 + row > R.t_last) continue;
        fx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int w = 0; w < waves; ++w) acc += *reinterpret_cast<const fx4*>(&sQ[w][row * LROW<DH> + ch]);
        *reinterpret_cast<fx4*>(dQ + qoff + int64_t(R.t0 + row) * D.qs[2] + ch) = acc * D.scale;
    }
}

// ------------------------------------------------------------------------------------ backward: dK, dV
// Key tiles of one (batch, KV head): first the sink and the survivors chunk by chunk (seen by all later rows: the long
// ones), then per chunk the rest (all of it where the chunk is never compressed).
struct KTiles { int sink, surv, rest, longs, count; };   // tiles of the sink, of a chunk's survivors, of a chunk's rest; totals
static KTiles make_ktiles(const Dims& D) {
    KTiles T;
    T.sink = ((D.S < D.n ? D.S : D.n) + 15) / 16;
    T.surv = (D.K + 15) / 16;
    T.rest = (D.L + 15) / 16;                            // a chunk that is never compressed keeps all its rows in one class
    T.longs = T.sink + D.Ns * T.surv;
    T.count = T.longs + D.nq * T.rest;
    return T;
}

constexpr int F32_KV_WAVES = 8;
constexpr int F32_MAX_SLICES = 8;
// Workgroups that share the query rows of a key tile.  One, unless there are fewer key tiles than fill the chip four times:
// a survivor's rows reach to the end of the sequence, so one workgroup per tile leaves most CUs idle behind the longest
// (a training step of 1024 rows of one head: 69 us with one slice, 58 us with eight).
static int f32_slices(const Dims& D) {
    const int64_t tiles = int64_t(make_ktiles(D).count) * D.B * D.Hkv;
    const int64_t s = tiles > 0 ? 1024 / tiles : 1;
    return int(s < 1 ? 1 : s > F32_MAX_SLICES ? F32_MAX_SLICES : s);
}

// part: [slices][dK, dV][batch, KV head][n][DH] when the rows are shared, else null
template <int DH>
__global__ __launch_bounds__(64 * F32_KV_WAVES) void k_bwd_dkv_f32(Dims D, const float* __restrict__ Q, const float* __restrict__ K,
                                                                    const float* __restrict__ V, const float* __restrict__ dO,
                                                                    const float* __restrict__ lse, const float* __restrict__ Dsum,
                                                                    const int32_t* __restrict__ idx, float* __restrict__ dK,
                                                                    float* __restrict__ dV, float* __restrict__ part, int slices, KTiles T) {
    constexpr int W = F32_KV_WAVES;
    __shared__ __attribute__((aligned(16))) float sK[W][16 * LROW<DH>], sV[W][16 * LROW<DH>];
    __shared__ int sPos[16];
    const int units = D.B * D.Hkv;
    const int bh = blockIdx.x % units, b = bh / D.Hkv, h = bh % D.Hkv, slice = int(blockIdx.x) / units % slices, tile = int(blockIdx.x) / units / slices;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 15, q4 = lane >> 4;
    const int32_t* idx_h = idx + (int64_t(b) * D.Hkv + h) * D.Ns * D.K;
    // the lane's key (the last one again past the tile's end) and the row end of the tile
    int count, key, rend = D.n;
    if (tile < T.sink) {
        count = min(16, (D.S < D.n ? D.S : D.n) - tile * 16);
        key = tile * 16 + min(c, count - 1);
    } else if (tile < T.longs) {
        const int ch = (tile - T.sink) / T.surv, first = (tile - T.sink) % T.surv * 16;
        count = min(16, D.K - first);
        key = idx_h[int64_t(ch) * D.K + first + min(c, count - 1)];
    } else {
        const int ch = (tile - T.longs) / T.rest, first = (tile - T.longs) % T.rest * 16, base = D.S + ch * D.L;
        const int64_t e = int64_t(D.S) + (int64_t(ch) + 1 + D.lp) * D.L;
        rend = e < D.n ? int(e) : D.n;
        const int rows = min(D.L, D.n - base);
        count = min(16, (ch < D.Ns ? D.L - D.K : rows) - first);
        if (count <= 0) return;
        key = first + min(c, count - 1);
        if (ch < D.Ns) {
            // the key-th row that did not survive: as many rows further as there are survivors up to it, found on the
            // ascending list (survivor s has idx[s] - base - s rows that did not survive before it)
            const int32_t* rowp = idx_h + int64_t(ch) * D.K;
            int lo = 0, hi = D.K;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (rowp[mid] - base - mid <= key) lo = mid + 1; else hi = mid;
            }
            key += lo;
        }
        key += base;
    }
    const int first_row = __builtin_amdgcn_readfirstlane(key);     // lane 0 holds the tile's lowest position, lane 15 its highest
    const int last_key = __builtin_amdgcn_readlane(key, 15);
    if (threadIdx.x < 16) sPos[threadIdx.x] = key;
    const int64_t koff = b * D.ks[0] + h * D.ks[1];
    const RowFrag<DH> k = row_frag<DH>(K + koff + int64_t(key) * D.ks[2], q4), v = row_frag<DH>(V + koff + int64_t(key) * D.ks[2], q4);
    Acc<DH> dk, dv;
    zero(dk);
    zero(dv);
    const int tph = (rend - first_row + 15) / 16, tiles = tph * D.G;
    const int i_lo = int(int64_t(tiles) * slice / slices), i_hi = int(int64_t(tiles) * (slice + 1) / slices);
    for (int i0 = i_lo + wave; i0 < i_hi; i0 += W) {
        const int hq = h * D.G + i0 / tph, r0 = first_row + i0 % tph * 16;
        const int64_t qoff = b * D.qs[0] + hq * D.qs[1], rid = (int64_t(b) * D.Hq + hq) * D.n;
        const int tr = min(r0 + c, rend - 1);
        const RowFrag<DH> q = row_frag<DH>(Q + qoff + int64_t(tr) * D.qs[2], q4), g = row_frag<DH>(dO + qoff + int64_t(tr) * D.qs[2], q4);
        ColFrag<DH> gc[4], qc[4];
        float ls[4], Dt[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = min(r0 + 4 * q4 + i, rend - 1);
            gc[i] = col_frag<DH>(dO + qoff + int64_t(t) * D.qs[2], c);
            qc[i] = col_frag<DH>(Q + qoff + int64_t(t) * D.qs[2], c);
            ls[i] = lse[rid + t];
            Dt[i] = Dsum[rid + t];
        }
        fx4 s = dot_tile<DH>(q, k), dp = dot_tile<DH>(g, v);
        const bool masked = r0 < last_key || r0 + 16 > rend;
        bool seen[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) seen[i] = r0 + 4 * q4 + i >= key && r0 + 4 * q4 + i < rend;
        if (masked) {
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = clean_row<DH>(gc[i], q4) ? NAN : s[i];
        }
        Acc<DH> t16;
        zero(t16);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s[i] = expf(D.scale * s[i] - ls[i]);
            add_outer<DH>(t16, gc[i], seen[i] ? s[i] : 0.0f);
        }
        add_acc<DH>(dv, 1.0f, t16);
        if (masked) {
#pragma unroll
            for (int i = 0; i < 4; ++i) dp[i] = clean_row<DH>(qc[i], q4) ? NAN : dp[i];
        }
        zero(t16);
#pragma unroll
        for (int i = 0; i < 4; ++i) add_outer<DH>(t16, qc[i], seen[i] ? s[i] * (dp[i] - Dt[i]) : 0.0f);
        add_acc<DH>(dk, 1.0f, t16);
    }
    put_acc<DH>(sK[wave], dk, c, q4);
    put_acc<DH>(sV[wave], dv, c, q4);
    __syncthreads();
    const int waves = min(W, i_hi - i_lo);
    for (int e = threadIdx.x; e < 2 * 16 * (DH / 4); e += 64 * W) {
        const int z = e / (16 * (DH / 4)), row = e / (DH / 4) % 16, ch = e % (DH / 4) * 4;
        if (row >= count) continue;
        fx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int w = 0; w < waves; ++w) acc += *reinterpret_cast<const fx4*>((z ? sV : sK)[w] + row * LROW<DH> + ch);
        if (z == 0) acc *= D.scale;
        float* dst = part ? part + (((int64_t(slice) * 2 + z) * units + bh) * D.n + sPos[row]) * DH
                          : (z ? dV : dK) + koff + int64_t(sPos[row]) * D.ks[2];
        *reinterpret_cast<fx4*>(dst + ch) = acc;
    }
}

// the slices of every row, in order
template <int DH>
__global__ __launch_bounds__(256) void k_bwd_dkv_f32_sum(Dims D, const float* __restrict__ part, int slices, float* __restrict__ dK, float* __restrict__ dV) {
    const int64_t rows = int64_t(D.B) * D.Hkv * D.n;
    const int64_t e = int64_t(blockIdx.x) * (1024 / DH) + threadIdx.x / (DH / 4);
    const int z = blockIdx.y, ch = threadIdx.x % (DH / 4) * 4;
    if (e >= rows) return;
    fx4 x[F32_MAX_SLICES];
#pragma unroll
    for (int s = 0; s < F32_MAX_SLICES; ++s)
        if (s < slices) x[s] = *reinterpret_cast<const fx4*>(part + ((int64_t(s) * 2 + z) * rows + e) * DH + ch);
    fx4 acc = x[0];
#pragma unroll
    for (int s = 1; s < F32_MAX_SLICES; ++s)
        if (s < slices) acc += x[s];
    const int bh = int(e / D.n), b = bh / D.Hkv, h = bh % D.Hkv;
    *reinterpret_cast<fx4*>((z ? dV : dK) + b * D.ks[0] + h * D.ks[1] + e % D.n * D.ks[2] + ch) = acc;
}

// ------------------------------------------------------------------------------------ launchers
// grid of one dimension: query tiles (key tiles) x heads.  A tile holds up to 16 rows and ends with its chunk, so short chunks reach
// the limit first: lag 2, 131072 tokens, 64 query heads of 64 channels are 2^22 workgroups of 1024 threads.
bool f32_tiles_supported(const Dims& D) {
    const int q_threads = 64 * (D.d == 64 ? F32_WAVES<64> : F32_WAVES<128>);
    return D.dtype == 0 && grid_fits(int64_t(make_qtiles(D).count) * D.B * D.Hq, q_threads) &&
           grid_fits(int64_t(make_ktiles(D).count) * D.B * D.Hkv * f32_slices(D), 64 * F32_KV_WAVES);
}

int attn_f32_query_waves(const Dims& D) { return f32_query_waves(D, int64_t(make_qtiles(D).count) * D.B * D.Hq); }
int attn_f32_key_waves() { return F32_KV_WAVES; }
int attn_f32_slices(const Dims& D) { return f32_slices(D); }

template <int DH>
static hipError_t run_fwd(const Dims& D, const float* Q, const float* K, const float* V, const int32_t* idx, float* O, float* lse, hipStream_t st) {
    const QTiles T = make_qtiles(D);
    constexpr int W = F32_WAVES<DH>;
    const int w = f32_query_waves(D, int64_t(T.count) * D.B * D.Hq);
    LRSA_TIMED_LAUNCH("k_fwd_f32", st, (w == W ? k_fwd_f32<DH, W> : w == 8 ? k_fwd_f32<DH, 8> : k_fwd_f32<DH, 4>), dim3(T.count * D.B * D.Hq),
                      dim3(64 * w), 0, st, D, Q, K, V, idx, O, lse, T);
    return hipGetLastError();
}
hipError_t launch_attn_fwd_f32(const Dims& D, const void* Q, const void* K, const void* V, const int32_t* idx, void* O, float* lse, hipStream_t st) {
    const float *q = (const float*)Q, *k = (const float*)K, *v = (const float*)V;
    return D.d == 64 ? run_fwd<64>(D, q, k, v, idx, (float*)O, lse, st) : run_fwd<128>(D, q, k, v, idx, (float*)O, lse, st);
}

// D of every row, then the slices' partial sums
static size_t f32_part_off(const Dims& D) { return align256(size_t(D.B) * D.Hq * D.n * 4); }
size_t attn_bwd_f32_ws_bytes(const Dims& D) {
    const int slices = f32_slices(D);
    return f32_part_off(D) + (slices > 1 ? size_t(slices) * 2 * D.B * D.Hkv * D.n * D.d * 4 : 0);
}

template <int DH>
static hipError_t run_bwd(const Dims& D, const float* Q, const float* K, const float* V, const float* O, const float* dO, const float* lse,
                          const int32_t* idx, float* dQ, float* dK, float* dV, float* ws, hipStream_t st) {
    float* Dsum = ws;
    const int slices = f32_slices(D);
    float* part = slices > 1 ? reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + f32_part_off(D)) : nullptr;
    const QTiles QT = make_qtiles(D);
    const KTiles KT = make_ktiles(D);
    constexpr int W = F32_WAVES<DH>;
    const int w = f32_query_waves(D, int64_t(QT.count) * D.B * D.Hq);
    LRSA_TIMED_LAUNCH("k_bwd_dq_f32", st, (w == W ? k_bwd_dq_f32<DH, W> : w == 8 ? k_bwd_dq_f32<DH, 8> : k_bwd_dq_f32<DH, 4>),
                      dim3(QT.count * D.B * D.Hq), dim3(64 * w), 0, st, D, Q, K, V, O, dO, lse, idx, dQ, Dsum, QT);
    LRSA_TIMED_LAUNCH("k_bwd_dkv_f32", st, k_bwd_dkv_f32<DH>, dim3(KT.count * D.B * D.Hkv * slices), dim3(64 * F32_KV_WAVES), 0, st, D, Q, K, V, dO,
                      lse, Dsum, idx, dK, dV, part, slices, KT);
    if (part)
        LRSA_TIMED_LAUNCH("k_bwd_dkv_f32_sum", st, k_bwd_dkv_f32_sum<DH>, dim3((unsigned)((int64_t(D.B) * D.Hkv * D.n + 1024 / DH - 1) / (1024 / DH)), 2),
                          dim3(256), 0, st, D, part, slices, dK, dV);
    return hipGetLastError();
}
hipError_t launch_attn_bwd_f32(const Dims& D, const void* Q, const void* K, const void* V, const void* O, const void* dO, const float* lse,
                               const int32_t* idx, void* dQ, void* dK, void* dV, void* ws, hipStream_t st) {
    const float *q = (const float*)Q, *k = (const float*)K, *v = (const float*)V, *o = (const float*)O, *g = (const float*)dO;
    return D.d == 64 ? run_bwd<64>(D, q, k, v, o, g, lse, idx, (float*)dQ, (float*)dK, (float*)dV, (float*)ws, st)
                     : run_bwd<128>(D, q, k, v, o, g, lse, idx, (float*)dQ, (float*)dK, (float*)dV, (float*)ws, st);
}

}  // namespace lrsa
