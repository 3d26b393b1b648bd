// Inference-time use of LagKV compression (the setting of the paper's evaluation tables: the KV cache is
// compressed lag window by lag window while tokens are generated).
//
// Cache of one layer: Kc, Vc [B, Hkv, cap, d_h]; rows [0, len) are valid, the same len for every head:
//   sink rows | K rows per compressed chunk, chunk after chunk | uncompressed tail.
// k_cache_compress  one step for every (batch, KV head): the first L rows of the tail are scored against the
//                   next L (Eq. 4-8, the same block routine as the training-time scoring), their top K are
//                   kept in position order (text after Eq. 8) and the rest of the tail moves down by L - K
//                   rows, in place (Section 3.2, Attention Filling 1: the older chunk shrinks to its survivors,
//                   the newer one stays whole).  An optional array of original positions moves alike.
// With a workspace (lrsa_cache_compress_ws) the same is done by many workgroups and all steps of a call at once:
// k_cache_select_move, k_cache_gather and k_cache_place below.
// k_decode_mfma     single-query attention (Eq. 3, nothing masked) of the G query heads of a KV group over a
//                   slice of the cache rows, bf16, on the matrix cores: fp32 online softmax, partial (max, sum,
//                   output) per slice;
// k_decode_attn     the same for fp32 data, in the vector pipe;
// k_decode_combine  merges the slices.
#include "mfma_tiles.h"
#include "score_block.h"
#include "select_block.h"

#include <mutex>

namespace lrsa {

constexpr int DEC_THREADS = 256;
constexpr int DEC_WAVES = DEC_THREADS / 64;
constexpr int DEC_GMAX = 8;            // query heads of a group handled per pass
constexpr int DEC_MAX_SPLITS = 256;
constexpr int DEC_U = 4;               // rows per lane group and step
constexpr int DEC_TILE = 32;           // rows per wave and step of k_decode_mfma

// Slices of a call of lrsa_decode_attn_static at most, by which its scratch limit is stated.
static int decode_static_splits(const Dims& D, int len) {
    const int want = (512 + D.B * D.Hkv - 1) / (D.B * D.Hkv), most = (len + 255) / 256;
    const int s = want < most ? want : most;
    return s < 1 ? 1 : s > DEC_MAX_SPLITS ? DEC_MAX_SPLITS : s;
}
static size_t part_bytes(const Dims& D, int splits) { return size_t(D.B) * D.Hq * splits * (D.d + 2) * 4; }
// Two workgroups share a CU (registers), so 512 run at once: at most that many, so that none runs alone behind them, or many more
// where 512 / units would leave CUs with half the work of others.  At least 128 rows each, a tile per wave of k_decode_mfma
// (12 heads on 2, 2.3K rows: 18 slices instead of 9, with the rest of k_decode_mfma 24.3 -> 11.3 us; fp32 33.9 -> 21.1 us).
// fp32 with three and more heads per group is bound by the vector pipe, which wants waves: beyond some units it keeps the count of
// decode_static_splits (104 units of 4 heads, 4K rows: 95 us, 108 with 512 / units; 88 units of 3 heads, 3.6K rows: 70 us, 67).
// A call that the scratch of lrsa_decode_attn_static held with decode_static_splits still fits: beyond it the slices stay at that
// number, in both calls, so that they give the same bits (more of them are no gain there: bf16, 512 units of 16 heads, 8K rows
// 356 us, 378 with four slices; 2K rows 124 and 114 us).
static int decode_splits(const Dims& D, int len) {
    const int units = D.B * D.Hkv, most = (len + 127) / 128;
    int s = units <= 128 ? 512 / units : 2048 / units;
    s = s < most ? s : most;
    s = s < 1 ? 1 : s > DEC_MAX_SPLITS ? DEC_MAX_SPLITS : s;
    const int base = decode_static_splits(D, len);
    if (D.dtype == 0 && D.G > 2 && units > (D.G == 3 ? 128 : 84)) return base;
    return s > base && part_bytes(D, s) > DECODE_STATIC_SCRATCH_BYTES ? base : s;
}
size_t decode_ws_bytes(const Dims& D) {
    // per (batch, query head, slice): max, sum, d_h output values
    return align256(size_t(D.B) * D.Hq * DEC_MAX_SPLITS * (D.d + 2) * 4);
}
bool cache_compress_supported(const Dims& D) { return D.L <= FUSED_MAX_L && D.lp == 1; }

// ------------------------------------------------------------------------------------ compression step
// Moves rows in place: row dst0 + i <- row src(i), i = 0 .. count-1, where src(i) >= dst0 + i and src is
// increasing.  Passes of FUSED_THREADS / lpr rows, ascending; within a pass every row is read before any is
// written (a pass never writes a row that a LATER pass still has to read: its sources lie above).
template <typename T, typename SrcFn>
__device__ __forceinline__ void move_rows(T* Z, int64_t stride, int d, int dst0, int count, SrcFn src) {
    constexpr int VEC = Elem<T>::VEC;
    const int lpr = d / VEC, rpp = FUSED_THREADS / lpr;
    const int sub = threadIdx.x % lpr, rg = threadIdx.x / lpr;
    for (int i0 = 0; i0 < count; i0 += rpp) {
        const int i = i0 + rg;
        uint4 v = {0u, 0u, 0u, 0u};
        if (i < count) v = *reinterpret_cast<const uint4*>(Z + int64_t(src(i)) * stride + sub * VEC);
        __syncthreads();   // waits for the loads of every thread as well
        if (i < count) *reinterpret_cast<uint4*>(Z + int64_t(dst0 + i) * stride + sub * VEC) = v;
        __syncthreads();
    }
}
template <typename SrcFn>
__device__ __forceinline__ void move_words(int32_t* A, int dst0, int count, SrcFn src) {
    for (int i0 = 0; i0 < count; i0 += FUSED_THREADS) {
        const int i = i0 + threadIdx.x;
        int32_t v = 0;
        if (i < count) v = A[src(i)];
        __syncthreads();
        if (i < count) A[dst0 + i] = v;
        __syncthreads();
    }
}

template <typename T, int DH>
__global__ __launch_bounds__(FUSED_THREADS) void k_cache_compress(Dims D, T* __restrict__ Kc, T* __restrict__ Vc,
                                                                  int32_t* __restrict__ pos, int len, int done) {
    const int bh = blockIdx.x, b = bh / D.Hkv, h = bh % D.Hkv;
    T* Kh = Kc + b * D.ks[0] + h * D.ks[1];
    T* Vh = Vc + b * D.ks[0] + h * D.ks[1];
    const int base = D.S + D.K * done;     // first row of the chunk to compress
    __shared__ ScoreLds sh;
    __shared__ SelectLds sel;
    __shared__ int32_t keep[FUSED_MAX_L];  // the K surviving rows, relative to base, ascending
    score_chunk_block<T, DH>(D.L, D.ddof, Kh + int64_t(base) * D.ks[2], Kh + int64_t(base + D.L) * D.ks[2],
                         Vh + int64_t(base) * D.ks[2], Vh + int64_t(base + D.L) * D.ks[2], D.ks[2], sh, nullptr);
    __syncthreads();
    select_topk_block<FUSED_THREADS>(reinterpret_cast<const uint32_t*>(sh.sig[0]), D.L, D.K, 0, keep, sel);
    __syncthreads();
    const int rest = len - (base + D.L);   // rows after the compressed chunk: they move down by L - K
    auto from_keep = [&](int i) { return base + keep[i]; };
    auto from_tail = [&](int i) { return base + D.L + i; };
    move_rows<T>(Kh, D.ks[2], D.d, base, D.K, from_keep);
    move_rows<T>(Vh, D.ks[2], D.d, base, D.K, from_keep);
    if (D.K < D.L) {
        move_rows<T>(Kh, D.ks[2], D.d, base + D.K, rest, from_tail);
        move_rows<T>(Vh, D.ks[2], D.d, base + D.K, rest, from_tail);
    }
    if (pos) {
        int32_t* ph = pos + int64_t(bh) * D.n;   // [B, Hkv, cap]
        move_words(ph, base, D.K, from_keep);
        if (D.K < D.L) move_words(ph, base + D.K, rest, from_tail);
    }
}

hipError_t launch_cache_compress(const Dims& D, void* Kc, void* Vc, int32_t* pos, int len, int done, int steps,
                                 hipStream_t st) {
    for (int s = 0; s < steps; ++s) {
        if (D.dtype == 1)
            LRSA_TIMED_LAUNCH("k_cache_compress", st, (D.d == 64 ? k_cache_compress<bf16_t, 64> : k_cache_compress<bf16_t, 128>),
                              dim3(D.B * D.Hkv), dim3(FUSED_THREADS), 0, st, D,
                              (bf16_t*)Kc, (bf16_t*)Vc, pos, len, done);
        else
            LRSA_TIMED_LAUNCH("k_cache_compress", st, (D.d == 64 ? k_cache_compress<float, 64> : k_cache_compress<float, 128>),
                              dim3(D.B * D.Hkv), dim3(FUSED_THREADS), 0, st, D,
                              (float*)Kc, (float*)Vc, pos, len, done);
        len -= D.L - D.K;
        done += 1;
    }
    return hipGetLastError();
}

// ---- the same with a workspace -------------------------------------------------------------------------------------
// All steps at once: step j scores chunk j of the tail against chunk j + 1, both still whole, so the steps do not
// depend on each other; only the rows move afterwards, all towards the front.  Launches:
//   k_minmax, k_sigma      standard deviations of every row of the chunks 0 .. steps-1 (score.hip), over all CUs
//   one step               k_cache_select_move: softmax, selection and the move in place
//   several steps          k_softmax_select, then k_cache_gather (rows to the workspace) and k_cache_place (and back)
// k_cache_compress is bound by one CU's loads per head, two in flight per thread, and repeats the move of the whole tail
// for every step.  Measured against it (bf16, d 128): one step at 8 heads, lag 1024: 50 us -> 22 us (4 + 6 + 12); a
// 32K-token prompt of 2 heads, 30 steps: 9600 us -> 43 us (8 + 12 + 7 + 8 + 8).
// The scores are those of k_cache_compress bit for bit, so the same rows survive.
//
// Row dst of the new cache comes from row src(dst) >= dst of the old one.
struct CacheMove {
    int base;       // first row that moves: sink + survivors of the chunks compressed earlier
    int kept;       // survivors: K per step
    int shift;      // rows after the compressed chunks move down by this much: steps * (L - K)
    int count;      // rows of the new cache from base on
    int bounced;    // of these, rows that go through the workspace (k_cache_gather, k_cache_place)
};
static CacheMove make_move(const Dims& D, int len, int done, int steps) {
    CacheMove M;
    M.base = D.S + D.K * done;
    M.kept = D.K * steps;
    M.shift = steps * (D.L - D.K);
    M.count = len - M.base - M.shift;
    // the rest is copied straight to its place when that place does not overlap where it comes from
    M.bounced = M.count - M.kept > M.shift ? M.count : M.kept;
    return M;
}

// One step.  A workgroup owns 64 bytes of every row of one (batch, KV head, K or V): different workgroups touch
// different bytes, so the move in place needs no ordering between them.  Each takes softmax and selection for itself
// (a chain of short block-wide steps: repeating it costs the CUs nothing that anybody else needs).  Rows move in
// ascending batches of MOVE_U per thread, all loads of a batch in flight together; a batch never writes a row that a
// later batch still has to read (src >= dst), so the only barrier is between its loads and its stores.
constexpr int MOVE_U = 8, MOVE_LANES = 4;
template <typename T>
__global__ __launch_bounds__(FUSED_THREADS) void k_cache_select_move(Dims D, T* __restrict__ Kc, T* __restrict__ Vc,
                                                                     int32_t* __restrict__ pos, const float* __restrict__ sigma,
                                                                     CacheMove M) {
    constexpr int VEC = Elem<T>::VEC, RPP = FUSED_THREADS / MOVE_LANES;
    const int slice = blockIdx.x, z = blockIdx.y, bh = blockIdx.z, b = bh / D.Hkv, h = bh % D.Hkv;
    const int tid = threadIdx.x;
    extern __shared__ float dyn[];          // [L] scores, then [K] surviving rows relative to base, ascending
    int32_t* keep = reinterpret_cast<int32_t*>(dyn + D.L);
    __shared__ float sm[2 * FUSED_THREADS / 64];
    __shared__ SelectLds sel;
    softmax_sum_regs<FUSED_THREADS>(sigma + int64_t(bh) * 2 * D.L, sigma + (int64_t(bh) * 2 + 1) * D.L, sm, D.L, nullptr, dyn);
    __syncthreads();
    select_topk_block<FUSED_THREADS>(reinterpret_cast<const uint32_t*>(dyn), D.L, D.K, 0, keep, sel);
    __syncthreads();
    auto src = [&](int i) { return M.base + (i < M.kept ? keep[i] : M.shift + i); };
    T* Z = (z ? Vc : Kc) + b * D.ks[0] + h * D.ks[1] + (slice * MOVE_LANES + tid % MOVE_LANES) * VEC;
    for (int i0 = tid / MOVE_LANES; i0 - tid / MOVE_LANES < M.count; i0 += MOVE_U * RPP) {
        uint4 v[MOVE_U];
#pragma unroll
        for (int u = 0; u < MOVE_U; ++u)
            if (i0 + u * RPP < M.count) v[u] = *reinterpret_cast<const uint4*>(Z + int64_t(src(i0 + u * RPP)) * D.ks[2]);
#pragma unroll
        for (int u = 0; u < MOVE_U; ++u) asm volatile("" : "+v"(v[u].x), "+v"(v[u].y), "+v"(v[u].z), "+v"(v[u].w));   // arrived
        __syncthreads();
#pragma unroll
        for (int u = 0; u < MOVE_U; ++u)
            if (i0 + u * RPP < M.count) *reinterpret_cast<uint4*>(Z + int64_t(M.base + i0 + u * RPP) * D.ks[2]) = v[u];
    }
    if (pos && slice == 0 && z == 0) move_words(pos + int64_t(bh) * D.n, M.base, M.count, src);
}

// Several steps: the rows that go through the workspace, 16 bytes per thread; rows [B * Hkv * 2][bounced][d], words of
// pos [B * Hkv][bounced] after them.  blockIdx.y: K, V, and the positions.
template <typename T>
__global__ __launch_bounds__(256) void k_cache_gather(Dims D, const T* __restrict__ Kc, const T* __restrict__ Vc,
                                                      const int32_t* __restrict__ pos, const int32_t* __restrict__ idx, CacheMove M,
                                                      T* __restrict__ rows, int32_t* __restrict__ words) {
    const int z = blockIdx.y, bh = blockIdx.z, b = bh / D.Hkv, h = bh % D.Hkv;
    const int e = blockIdx.x * 256 + threadIdx.x;
    const int lpr = z < 2 ? D.d / Elem<T>::VEC : 1;
    const int i = e / lpr, c = e % lpr * Elem<T>::VEC;
    if (i >= M.bounced) return;
    const int from = i < M.kept ? idx[int64_t(bh) * M.kept + i] : M.base + M.shift + i;
    if (z < 2) {
        const T* Z = (z ? Vc : Kc) + b * D.ks[0] + h * D.ks[1];
        *reinterpret_cast<uint4*>(rows + ((int64_t(bh) * 2 + z) * M.bounced + i) * D.d + c) =
            *reinterpret_cast<const uint4*>(Z + int64_t(from) * D.ks[2] + c);
    } else {
        words[int64_t(bh) * M.bounced + i] = pos[int64_t(bh) * D.n + from];
    }
}
template <typename T>
__global__ __launch_bounds__(256) void k_cache_place(Dims D, T* __restrict__ Kc, T* __restrict__ Vc, int32_t* __restrict__ pos,
                                                     CacheMove M, const T* __restrict__ rows, const int32_t* __restrict__ words) {
    const int z = blockIdx.y, bh = blockIdx.z, b = bh / D.Hkv, h = bh % D.Hkv;
    const int e = blockIdx.x * 256 + threadIdx.x;
    const int lpr = z < 2 ? D.d / Elem<T>::VEC : 1;
    const int i = e / lpr, c = e % lpr * Elem<T>::VEC;
    if (i >= M.count) return;
    if (z < 2) {
        T* Z = (z ? Vc : Kc) + b * D.ks[0] + h * D.ks[1];
        *reinterpret_cast<uint4*>(Z + int64_t(M.base + i) * D.ks[2] + c) = *reinterpret_cast<const uint4*>(
            i < M.bounced ? rows + ((int64_t(bh) * 2 + z) * M.bounced + i) * D.d + c : Z + int64_t(M.base + M.shift + i) * D.ks[2] + c);
    } else {
        int32_t* ph = pos + int64_t(bh) * D.n;
        ph[M.base + i] = i < M.bounced ? words[int64_t(bh) * M.bounced + i] : ph[M.base + M.shift + i];
    }
}

namespace {
struct CompressWs { size_t sigma, idx, rows, words, bytes; };   // byte offsets; the min / max partials come first
}
// the tail's chunks as the scored chunks of a sequence
static Dims tail_dims(const Dims& D, int done, int steps) {
    Dims T = D;
    T.S = D.S + D.K * done;
    T.Ns = steps;
    return T;
}
static CompressWs compress_ws(const Dims& D, int len, int done, int steps) {
    CompressWs W = {};
    const size_t heads = size_t(D.B) * D.Hkv;
    const bool bounce = steps > 1;
    const size_t bounced = bounce ? size_t(make_move(D, len, done, steps).bounced) : 0;
    W.sigma = align256(cache_sigma_ws_floats(tail_dims(D, done, steps)) * 4);
    W.idx = W.sigma + align256(heads * 2 * steps * D.L * 4);
    W.rows = W.idx + (bounce ? align256(heads * steps * D.K * 4) : 0);
    W.words = W.rows + align256(heads * 2 * bounced * D.d * (D.dtype == 1 ? 2 : 4));
    W.bytes = W.words + align256(heads * bounced * 4);
    return W;
}
// A single step with a workspace gains from the CUs that k_cache_compress leaves idle, and loses three launches against one and a softmax and
// selection in every workgroup of k_cache_select_move: with the bytes of a chunk it gains, with the heads it loses.  Measured
// with the allocation, call by call to its end, k_cache_compress -> three launches, us: bf16, d 128, 32 heads of K: lag 128
// 27.7 -> 29.3, lag 256 (64 KB) 31.7 -> 31.4; 64 heads: lag 512 45 -> 47, lag 1024 (256 KB) 70 -> 63; 128 heads (device
// time) lag 72 17.5 -> 38, lag 2048 146 -> 159.  fp32, d 128, 16 heads: lag 128 27 -> 29, lag 256 (128 KB) 36 -> 33; 32
// heads, of which k_cache_select_move has two workgroups per CU: lag 256 36 -> 37, lag 512 56 -> 49; 64: lag 1024 106 -> 96.
// Several steps always gain: k_cache_compress takes them one after another.
bool cache_step_is_long(const Dims& D) {
    const int64_t heads = int64_t(D.B) * D.Hkv, row = D.d * (D.dtype == 1 ? 2 : 4), chunk = D.L * row;
    if (heads > 64) return false;
    if (D.dtype == 1) return chunk >= (heads <= 32 ? 64 : 256) * 1024;
    return chunk >= 128 * 1024 * ((heads * 2 * row / (16 * MOVE_LANES) + 255) / 256);
}
size_t cache_compress_ws_bytes(const Dims& D, int len, int done, int steps) { return compress_ws(D, len, done, steps).bytes; }

template <typename T>
static hipError_t run_compress_ws(const Dims& D, T* Kc, T* Vc, int32_t* pos, int len, int done, int steps, void* ws, hipStream_t st) {
    const Dims C = tail_dims(D, done, steps);
    const CompressWs W = compress_ws(D, len, done, steps);
    const CacheMove M = make_move(D, len, done, steps);
    char* w = reinterpret_cast<char*>(ws);
    float* sigma = reinterpret_cast<float*>(w + W.sigma);
    hipError_t e = launch_cache_sigma(C, Kc, Vc, reinterpret_cast<float*>(w), sigma, st);
    if (e != hipSuccess) return e;
    if (steps == 1) {
        LRSA_TIMED_LAUNCH("k_cache_select_move", st, k_cache_select_move<T>, dim3(D.d * int(sizeof(T)) / (16 * MOVE_LANES), 2, D.B * D.Hkv),
                          dim3(FUSED_THREADS), size_t(D.L + D.K) * 4, st, D, Kc, Vc, pos, sigma, M);
        return hipGetLastError();
    }
    int32_t* idx = reinterpret_cast<int32_t*>(w + W.idx);
    T* rows = reinterpret_cast<T*>(w + W.rows);
    int32_t* words = reinterpret_cast<int32_t*>(w + W.words);
    if ((e = launch_cache_select(C, sigma, idx, st)) != hipSuccess) return e;
    const int lpr = D.d / Elem<T>::VEC;
    auto grid = [&](int count) { return dim3((unsigned)((int64_t(count) * lpr + 255) / 256), pos ? 3 : 2, D.B * D.Hkv); };
    LRSA_TIMED_LAUNCH("k_cache_gather", st, k_cache_gather<T>, grid(M.bounced), dim3(256), 0, st, D, Kc, Vc, pos, idx, M, rows, words);
    LRSA_TIMED_LAUNCH("k_cache_place", st, k_cache_place<T>, grid(M.count), dim3(256), 0, st, D, Kc, Vc, pos, M, rows, words);
    return hipGetLastError();
}

hipError_t launch_cache_compress_ws(const Dims& D, void* Kc, void* Vc, int32_t* pos, int len, int done, int steps, void* ws,
                                    hipStream_t st) {
    return D.dtype == 1 ? run_compress_ws(D, (bf16_t*)Kc, (bf16_t*)Vc, pos, len, done, steps, ws, st)
                        : run_compress_ws(D, (float*)Kc, (float*)Vc, pos, len, done, steps, ws, st);
}

// ------------------------------------------------------------------------------------ single-query attention
// (m, l, o) of two disjoint key sets -> of their union
__device__ __forceinline__ void merge_state(float& m, float& l, float m2, float l2, float& a, float& b2) {
    const float mn = fmaxf(m, m2);
    a = m == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m - mn);
    b2 = m2 == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m2 - mn);
    l = l * a + l2 * b2;
    m = mn;
}

// bf16.  One workgroup: the heads of one KV group (16 at a time) x rows [split * per, ...) of the cache; its waves take tiles
// of 32 rows in turn.  Nothing is staged in LDS.  Lane l, c = l % 16, q4 = l / 16, v_mfma_f32_16x16x32_bf16:
//   S = K Q^T   row m of block kb is tile row 8*(m/4) + 4*kb + m%4, column c a head: the lane then holds the logits of tile
//               rows 8*q4 .. +7 of head c, which are the k-slots of its B operand in the second product
//   O^T += V^T P^T   the lane reads DH/16 neighbouring channels of tile rows 8*q4 .. +7 and transposes that block in
//               registers (byte permutes): column e of it is its row of the A operand for the channels (DH/16)*m + e
// The weights enter as three bf16 terms, which hold all 24 bits of them; the matrix pipe has time to spare.
// Bound by reading the cache (325 MB, 8 requests of 9.9K rows on 8 KV heads, 4 query heads each: 83 -> 60.5 us with the
// merge, 5.4 TB/s), by latency for a short one (2.3K rows, 2 KV heads: 24.2 -> 10.7 us).  In the vector pipe, one lane's
// dot products and a shuffle through LDS per row and head bounded it.  Errors against 64 bits as before: O differs from
// the rounded exact value in at most 0.2 % of the elements.
template <int DH> struct VPiece { typedef uint4 type; };
template <> struct VPiece<64> { typedef uint2 type; };
template <int DH> struct DecTile {
    bf16x8 k[2][DH / 32];
    typename VPiece<DH>::type v[8];
};
template <int DH>
__device__ __forceinline__ void load_tile(DecTile<DH>& t, const bf16_t* Kl, const bf16_t* Vl, int64_t stride, int kr, int vr, int last) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        const bf16_t* row = Kl + int64_t(min(kr + 4 * kb, last)) * stride;   // rows past the end repeat the last one, weight 0
#pragma unroll
        for (int kk = 0; kk < DH / 32; ++kk) t.k[kb][kk] = *reinterpret_cast<const bf16x8*>(row + kk * 32);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) t.v[j] = *reinterpret_cast<const typename VPiece<DH>::type*>(Vl + int64_t(min(vr + j, last)) * stride);
}
template <int DH> struct DecState {
    float m, l;          // of head c; l over the lane's own rows
    f32x4 o[DH / 16];
};
template <int DH>
__device__ __forceinline__ void use_tile(DecState<DH>& st, const DecTile<DH>& t, const bf16x8 (&qf)[DH / 32], int r, int r1, float c2) {
    f32x4 s[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
    for (int kk = 0; kk < DH / 32; ++kk)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) s[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t.k[kb][kk], qf[kk], s[kb], 0, 0, 0);
    float p[8], mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        p[j] = r + j < r1 ? s[j >> 2][j & 3] * c2 : -INFINITY;
        mx = fmaxf(mx, p[j]);
    }
    lanes_u32x2 x = pair32(__float_as_uint(mx));
    mx = fmaxf(__uint_as_float(x.x), __uint_as_float(x.y));
    x = pair16(__float_as_uint(mx));
    mx = fmaxf(__uint_as_float(x.x), __uint_as_float(x.y));
    if (__builtin_amdgcn_ballot_w64(mx > st.m) != 0) {       // always on the first tile, whose row 0 is there
        const float mn = fmaxf(st.m, mx), a = __builtin_amdgcn_exp2f(st.m - mn);
        st.m = mn;
        st.l *= a;
#pragma unroll
        for (int e = 0; e < DH / 16; ++e) st.o[e] *= a;
    }
    f32x8 w;
    float ps = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        w[j] = __builtin_amdgcn_exp2f(p[j] - st.m);
        ps += w[j];
    }
    st.l += ps;
    bf16x8 term[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        term[i] = __builtin_convertvector(w, bf16x8);
        w -= __builtin_convertvector(term[i], f32x8);
    }
#pragma unroll
    for (int e = 0; e < DH / 16; ++e) {
        uint32_t a[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t lo = reinterpret_cast<const uint32_t*>(&t.v[2 * i])[e >> 1], hi = reinterpret_cast<const uint32_t*>(&t.v[2 * i + 1])[e >> 1];
            a[i] = __builtin_amdgcn_perm(hi, lo, e & 1 ? 0x07060302u : 0x05040100u);
        }
        const bf16x8 av = __builtin_bit_cast(bf16x8, a);
#pragma unroll
        for (int i = 2; i >= 0; --i) st.o[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, term[i], st.o[e], 0, 0, 0);
    }
}

template <int DH>
__global__ __launch_bounds__(DEC_THREADS, 2) void k_decode_mfma(Dims D, const bf16_t* __restrict__ q, const bf16_t* __restrict__ Kc,
                                                                const bf16_t* __restrict__ Vc, int len, int per, int splits,
                                                                float* __restrict__ part) {
    constexpr int CPL = DH / 16, LROW = DH + 4;              // channels per lane; the padding spreads the heads over the banks
    __shared__ __attribute__((aligned(16))) float sO[DEC_WAVES][16][LROW];
    __shared__ float sM[DEC_WAVES][16], sL[DEC_WAVES][16];
    const int split = blockIdx.x, bh = blockIdx.y, b = bh / D.Hkv, h = bh % D.Hkv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 15, q4 = lane >> 4;
    const int r0 = split * per, r1 = min(len, r0 + per);     // r0 >= r1: an empty slice, its records say so
    const bf16_t* Kl = Kc + b * D.ks[0] + h * D.ks[1] + q4 * 8;
    const bf16_t* Vl = Vc + b * D.ks[0] + h * D.ks[1] + c * CPL;
    const int kr = 8 * (c >> 2) + (c & 3), vr = 8 * q4;
    const float c2 = D.scale * 1.4426950408889634f;          // logits in log2 units

    for (int g0 = 0; g0 < D.G; g0 += 16) {
        const int gn = min(16, D.G - g0);
        const bf16_t* qrow = q + (int64_t(b) * D.Hq + h * D.G + g0 + min(c, gn - 1)) * DH + q4 * 8;
        bf16x8 qf[DH / 32];
#pragma unroll
        for (int kk = 0; kk < DH / 32; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qrow + kk * 32);
        DecState<DH> st;
        st.m = -INFINITY;
        st.l = 0.0f;
#pragma unroll
        for (int e = 0; e < CPL; ++e) st.o[e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        // the next tile's loads are in flight while a tile is used
        constexpr int STEP = DEC_WAVES * DEC_TILE;
        int r = r0 + wave * DEC_TILE;
        if (r < r1) {
            DecTile<DH> A, B;
            load_tile<DH>(A, Kl, Vl, D.ks[2], r + kr, r + vr, r1 - 1);
            for (;;) {
                if (r + STEP < r1) load_tile<DH>(B, Kl, Vl, D.ks[2], r + STEP + kr, r + STEP + vr, r1 - 1);
                use_tile<DH>(st, A, qf, r + vr, r1, c2);
                if ((r += STEP) >= r1) break;
                if (r + STEP < r1) load_tile<DH>(A, Kl, Vl, D.ks[2], r + STEP + kr, r + STEP + vr, r1 - 1);
                use_tile<DH>(st, B, qf, r + vr, r1, c2);
                if ((r += STEP) >= r1) break;
            }
        }
        lanes_u32x2 x = pair32(__float_as_uint(st.l));
        st.l = __uint_as_float(x.x) + __uint_as_float(x.y);
        x = pair16(__float_as_uint(st.l));
        st.l = __uint_as_float(x.x) + __uint_as_float(x.y);
        if (c < gn) {
            if (q4 == 0) { sM[wave][c] = st.m; sL[wave][c] = st.l; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < CPL; e += 4)
                    *reinterpret_cast<f32x4*>(&sO[wave][c][(4 * q4 + i) * CPL + e]) = f32x4{st.o[e][i], st.o[e + 1][i], st.o[e + 2][i], st.o[e + 3][i]};
        }
        __syncthreads();
        for (int e = tid; e < gn * DH; e += DEC_THREADS) {
            const int g = e / DH, ch = e % DH;
            float mm = sM[0][g], ll = sL[0][g], oo = sO[0][g][ch];
#pragma unroll
            for (int w = 1; w < DEC_WAVES; ++w) {
                float a, b2;
                merge_state(mm, ll, sM[w][g], sL[w][g], a, b2);
                oo = oo * a + sO[w][g][ch] * b2;
            }
            float* dst = part + ((int64_t(b) * D.Hq + h * D.G + g0 + g) * splits + split) * (DH + 2);
            dst[2 + ch] = oo;
            if (ch == 0) { dst[0] = mm; dst[1] = ll; }
        }
        __syncthreads();
    }
}

// fp32.  One workgroup: the G heads of one KV group (DEC_GMAX at a time) x rows [r0, r1) of the cache.  A row is
// spread over lpr = 16-byte pieces; a wave reads 64 / lpr rows per step; logits are kept in log2 units.
template <typename T>
__global__ __launch_bounds__(DEC_THREADS) void k_decode_attn(Dims D, const T* __restrict__ q, const T* __restrict__ Kc,
                                                             const T* __restrict__ Vc, int len, int splits,
                                                             float* __restrict__ part) {
    constexpr int VEC = Elem<T>::VEC;
    const int lpr = D.d / VEC, rpw = 64 / lpr;
    const int split = blockIdx.x, bh = blockIdx.y, b = bh / D.Hkv, h = bh % D.Hkv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = lane % lpr, slot = lane / lpr;
    const int per = (len + splits - 1) / splits;
    const int r0 = split * per, r1 = min(len, r0 + per);
    const T* Kh = Kc + b * D.ks[0] + h * D.ks[1];
    const T* Vh = Vc + b * D.ks[0] + h * D.ks[1];
    const float c2 = D.scale * 1.4426950408889634f;
    __shared__ float sM[DEC_WAVES][DEC_GMAX], sL[DEC_WAVES][DEC_GMAX], sO[DEC_WAVES][DEC_GMAX][128];

    for (int g0 = 0; g0 < D.G; g0 += DEC_GMAX) {
        const int gn = min(DEC_GMAX, D.G - g0);
        float qv[DEC_GMAX][VEC], o[DEC_GMAX][VEC], m[DEC_GMAX], l[DEC_GMAX];
#pragma unroll
        for (int g = 0; g < DEC_GMAX; ++g) {
            m[g] = -INFINITY; l[g] = 0.0f;
#pragma unroll
            for (int i = 0; i < VEC; ++i) { o[g][i] = 0.0f; qv[g][i] = 0.0f; }
            if (g < gn) Elem<T>::load(q + (int64_t(b) * D.Hq + h * D.G + g0 + g) * D.d + sub * VEC, qv[g]);
        }
        // DEC_U rows per lane group and step: their loads are in flight together, and the running maximum is
        // refreshed (and the sums rescaled) once per step instead of once per row
        const int step = DEC_WAVES * rpw;
        for (int rb = r0 + wave * rpw + slot; rb < r1; rb += DEC_U * step) {
            float kv[DEC_U][VEC], vv[DEC_U][VEC];
#pragma unroll
            for (int u = 0; u < DEC_U; ++u) {
                const int r = min(rb + u * step, r1 - 1);   // rows past the end repeat the last one, weight 0 below
                Elem<T>::load(Kh + int64_t(r) * D.ks[2] + sub * VEC, kv[u]);
                Elem<T>::load(Vh + int64_t(r) * D.ks[2] + sub * VEC, vv[u]);
            }
#pragma unroll
            for (int g = 0; g < DEC_GMAX; ++g) {
                if (g >= gn) continue;
                float sc[DEC_U], mn = m[g];
#pragma unroll
                for (int u = 0; u < DEC_U; ++u) {
                    float t = 0.0f;
#pragma unroll
                    for (int i = 0; i < VEC; ++i) t = __builtin_fmaf(qv[g][i], kv[u][i], t);
                    sc[u] = t;
                }
                for (int off = lpr >> 1; off > 0; off >>= 1)
#pragma unroll
                    for (int u = 0; u < DEC_U; ++u) sc[u] += __shfl_xor(sc[u], off, 64);
#pragma unroll
                for (int u = 0; u < DEC_U; ++u) {
                    sc[u] = rb + u * step < r1 ? sc[u] * c2 : -INFINITY;
                    mn = fmaxf(mn, sc[u]);
                }
                const float a = __builtin_amdgcn_exp2f(m[g] - mn);   // exp2(-inf) = 0 on the first step; row rb is valid
                float ls = 0.0f;
#pragma unroll
                for (int i = 0; i < VEC; ++i) o[g][i] *= a;
#pragma unroll
                for (int u = 0; u < DEC_U; ++u) {
                    const float pr = __builtin_amdgcn_exp2f(sc[u] - mn);
                    ls += pr;
#pragma unroll
                    for (int i = 0; i < VEC; ++i) o[g][i] = __builtin_fmaf(pr, vv[u][i], o[g][i]);
                }
                l[g] = l[g] * a + ls;
                m[g] = mn;
            }
        }
        // merge the row slots of a wave, then the waves
#pragma unroll
        for (int g = 0; g < DEC_GMAX; ++g) {
            if (g >= gn) continue;
            for (int off = lpr; off < 64; off <<= 1) {
                const float m2 = __shfl_xor(m[g], off, 64), l2 = __shfl_xor(l[g], off, 64);
                float a, b2;
                merge_state(m[g], l[g], m2, l2, a, b2);
#pragma unroll
                for (int i = 0; i < VEC; ++i) o[g][i] = o[g][i] * a + __shfl_xor(o[g][i], off, 64) * b2;
            }
            if (slot == 0) {
                if (sub == 0) { sM[wave][g] = m[g]; sL[wave][g] = l[g]; }
#pragma unroll
                for (int i = 0; i < VEC; ++i) sO[wave][g][sub * VEC + i] = o[g][i];
            }
        }
        __syncthreads();
        for (int e = tid; e < gn * D.d; e += DEC_THREADS) {
            const int g = e / D.d, ch = e % D.d;
            float mm = sM[0][g], ll = sL[0][g], oo = sO[0][g][ch];
            for (int w = 1; w < DEC_WAVES; ++w) {
                float a, b2;
                merge_state(mm, ll, sM[w][g], sL[w][g], a, b2);
                oo = oo * a + sO[w][g][ch] * b2;
            }
            float* dst = part + ((int64_t(b) * D.Hq + h * D.G + g0 + g) * splits + split) * (D.d + 2);
            dst[2 + ch] = oo;
            if (ch == 0) { dst[0] = mm; dst[1] = ll; }
        }
        __syncthreads();
    }
}

// One (batch, query head) per workgroup: the weights of all slices first (two loads per lane and 64 slices), then the
// records are summed by all lanes, two channels each, COMB_U loads in flight; fixed order.
constexpr int COMB_U = 4;
template <typename T>
__global__ __launch_bounds__(DEC_THREADS) void k_decode_combine(Dims D, const float* __restrict__ part, int splits,
                                                                T* __restrict__ O, float* __restrict__ lse) {
    __shared__ float sW[DEC_MAX_SPLITS];
    __shared__ float2 sO[DEC_THREADS];
    const int64_t bhq = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, rec = D.d + 2;
    const float* src = part + bhq * splits * rec;
    float m[DEC_MAX_SPLITS / 64], l[DEC_MAX_SPLITS / 64], M = -INFINITY, L = 0.0f;
#pragma unroll
    for (int i = 0; i < DEC_MAX_SPLITS / 64; ++i) {
        const int s = lane + 64 * i;
        m[i] = -INFINITY; l[i] = 0.0f;
        if (s < splits) {
            const float2 ml = *reinterpret_cast<const float2*>(src + int64_t(s) * rec);
            m[i] = ml.x; l[i] = ml.y;
        }
        M = fmaxf(M, m[i]);
    }
    M = wave_max(M);
#pragma unroll
    for (int i = 0; i < DEC_MAX_SPLITS / 64; ++i) {
        const float w = m[i] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m[i] - M);
        L = __builtin_fmaf(l[i], w, L);
        if (tid < 64) sW[lane + 64 * i] = w;
    }
    L = wave_sum(L);
    __syncthreads();
    const int pairs = D.d / 2, ways = DEC_THREADS / pairs, ch = tid % pairs, way = tid / pairs;
    float2 o = {0.0f, 0.0f};
    for (int s0 = way; s0 < splits; s0 += COMB_U * ways) {
        float2 v[COMB_U];
        float w[COMB_U];
#pragma unroll
        for (int u = 0; u < COMB_U; ++u) {
            const int s = s0 + u * ways, sc = min(s, splits - 1);
            w[u] = s < splits ? sW[sc] : 0.0f;
            v[u] = *reinterpret_cast<const float2*>(src + int64_t(sc) * rec + 2 + 2 * ch);
        }
#pragma unroll
        for (int u = 0; u < COMB_U; ++u) {
            o.x = __builtin_fmaf(w[u], v[u].x, o.x);
            o.y = __builtin_fmaf(w[u], v[u].y, o.y);
        }
    }
    sO[tid] = o;
    __syncthreads();
    if (tid < pairs) {
        for (int w = 1; w < ways; ++w) { o.x += sO[w * pairs + tid].x; o.y += sO[w * pairs + tid].y; }
        Elem<T>::put(O + bhq * D.d + 2 * ch, o.x / L);
        Elem<T>::put(O + bhq * D.d + 2 * ch + 1, o.y / L);
        if (lse && tid == 0)   // one rounding at the end: ln 2 as its fp32 value plus the rest
            lse[bhq] = __builtin_fmaf(M, 0.69314718246459961f, __builtin_fmaf(M, -1.9046542e-9f, __builtin_log2f(L) * 0.6931471805599453f));
    }
}

// ------------------------------------------------------------------------------------ no-allocation variant
// Scratch of lrsa_decode_attn_static: the partial (max, sum, output) records of the slices live in this array
// instead of a caller's workspace.  Every GPU holds its own copy at its own address; the array's name is only a
// host-side handle, so the device address is looked up once per device and that pointer is what the kernels get.
static __device__ __align__(256) unsigned char scratch[DECODE_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

static hipError_t scratch_address(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));   // address of the current device's copy
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

size_t decode_static_need(const Dims& D, int len) {
    return part_bytes(D, decode_static_splits(D, len));
}

hipError_t launch_decode_attn(const Dims& D, const void* q, const void* Kc, const void* Vc, int len, void* O,
                              float* lse, void* ws, hipStream_t st);

// Same kernels, same slices, hence the same bits as launch_decode_attn; the caller has checked
// decode_static_need() <= DECODE_STATIC_SCRATCH_BYTES.  Nothing has to start at zero: every record that the
// combine kernel reads is written by the slice kernel of the same call.
hipError_t launch_decode_attn_static(const Dims& D, const void* q, const void* Kc, const void* Vc, int len, void* O,
                                     float* lse, hipStream_t st) {
    void* part = nullptr;
    const hipError_t e = scratch_address(&part);
    if (e != hipSuccess) return e;
    return launch_decode_attn(D, q, Kc, Vc, len, O, lse, part, st);
}

hipError_t launch_decode_attn(const Dims& D, const void* q, const void* Kc, const void* Vc, int len, void* O,
                              float* lse, void* ws, hipStream_t st) {
    const int splits = decode_splits(D, len);
    float* part = reinterpret_cast<float*>(ws);
    if (D.dtype == 1) {
        const int per = ((len + splits - 1) / splits + DEC_TILE - 1) / DEC_TILE * DEC_TILE;
#define LRSA_DECODE_LAUNCH(DH_)                                                                                              \
    LRSA_TIMED_LAUNCH("k_decode_mfma", st, k_decode_mfma<DH_>, dim3(splits, D.B * D.Hkv), dim3(DEC_THREADS), 0, st, D,       \
                      (const bf16_t*)q, (const bf16_t*)Kc, (const bf16_t*)Vc, len, per, splits, part)
        if (D.d == 64) LRSA_DECODE_LAUNCH(64); else LRSA_DECODE_LAUNCH(128);
#undef LRSA_DECODE_LAUNCH
        LRSA_TIMED_LAUNCH("k_decode_combine", st, k_decode_combine<bf16_t>, dim3(D.B * D.Hq), dim3(DEC_THREADS), 0, st, D, part, splits,
                          (bf16_t*)O, lse);
    } else {
        LRSA_TIMED_LAUNCH("k_decode_attn", st, k_decode_attn<float>, dim3(splits, D.B * D.Hkv), dim3(DEC_THREADS), 0, st, D,
                          (const float*)q, (const float*)Kc, (const float*)Vc, len, splits, part);
        LRSA_TIMED_LAUNCH("k_decode_combine", st, k_decode_combine<float>, dim3(D.B * D.Hq), dim3(DEC_THREADS), 0, st, D, part, splits,
                          (float*)O, lse);
    }
    return hipGetLastError();
}

}  // namespace lrsa
