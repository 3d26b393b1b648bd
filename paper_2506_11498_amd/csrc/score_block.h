// Scoring of ONE lag chunk inside one workgroup of 1024 threads (Eq. 4-8 of the paper): per-channel min / max
// over the rows of the reference chunk (Eq. 4-5), the chunk's rows normalised by them (Eq. 6) and their
// standard deviation over the channels, the softmax over the chunk's tokens for K and for V, summed (Eq. 7-8).
// Used by the training-time scoring kernel (chunks of a sequence) and by the cache compression of the
// inference path (the two oldest uncompressed chunks of a cache): the same arithmetic, hence the same scores.
#pragma once
#include "common.h"

namespace lrsa {

constexpr int FUSED_THREADS = 1024;
constexpr int FUSED_MAX_L = 4096;

struct ScoreLds {
    float red[4][FUSED_THREADS / 64][128];   // per-wave partial min_K, max_K, min_V, max_V
    float s_mn[2][128], s_inv[2][128], s_den[2][128];
    float sig[2][FUSED_MAX_L];
    float sm[2 * FUSED_THREADS / 64];
};

// Kcur / Vcur: row 0 of the chunk to score, Kref / Vref: row 0 of the chunk after it; `stride` elements
// between rows; L <= FUSED_MAX_L rows each.  On return sh.sig[0][r] holds the score of row r (also written
// to out[r] when out is not null); all threads have passed a barrier after the last LDS write they depend on
// only for their own r = tid, tid + 1024, ... -- callers that read other rows synchronise first.
// Eq. 7-8 given the standard deviations: max-subtracted softmax of sig0 over the L tokens, the same for sig1,
// their sum written to sig0[r] (and to out[r] when out is not null).  sig0, sig1: LDS, L floats each, complete
// and visible to the NT threads of the block on entry; sm: 2 * NT/64 floats of LDS.  Each thread touches only rows
// r = tid, tid + NT, ...: callers that read other rows afterwards synchronise first.
template <int NT>
__device__ __forceinline__ void softmax_sum_block(float* sig0, const float* sig1, float* sm, int L,
                                                  float* __restrict__ out) {
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the K and the V value reduced over the block together (one pair of barriers for both)
    auto block_red2 = [&](float& a, float& b, bool is_max) {
        a = is_max ? wave_max(a) : wave_sum(a);
        b = is_max ? wave_max(b) : wave_sum(b);
        __syncthreads();
        if (lane == 0) { sm[wave] = a; sm[NW + wave] = b; }
        __syncthreads();
        float ra = sm[0], rb = sm[NW];
        for (int i = 1; i < NW; ++i) {
            ra = is_max ? fmaxf(ra, sm[i]) : ra + sm[i];
            rb = is_max ? fmaxf(rb, sm[NW + i]) : rb + sm[NW + i];
        }
        a = ra;
        b = rb;
    };
    float mk = -INFINITY, mv = -INFINITY;
    for (int r = tid; r < L; r += NT) { mk = fmaxf(mk, sig0[r]); mv = fmaxf(mv, sig1[r]); }
    block_red2(mk, mv, true);
    float zk = 0.0f, zv = 0.0f;
    for (int r = tid; r < L; r += NT) { zk += expf(sig0[r] - mk); zv += expf(sig1[r] - mv); }
    block_red2(zk, zv, false);
    for (int r = tid; r < L; r += NT) {
        const float sc = expf(sig0[r] - mk) / zk + expf(sig1[r] - mv) / zv;
        if (out) out[r] = sc;
        sig0[r] = sc;     // each thread overwrites only what it alone has read
    }
}

// The same from standard deviations in global memory: a thread keeps its rows r = tid, tid + NT, ... in registers from
// the load to the score.  Scores go to out[r] (global) and key[r] (LDS), where these are not null.  The same values in
// the same order as softmax_sum_block<NT>.
template <int NT>
__device__ __forceinline__ void softmax_sum_regs(const float* __restrict__ sk, const float* __restrict__ sv, float* sm,
                                                 int L, float* __restrict__ out, float* key) {
    constexpr int NW = NT / 64, MAXJ = FUSED_MAX_L / NT;   // rows of a thread: at most MAXJ
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // a row past the chunk counts as -inf (its exponential is 0)
    float vk[MAXJ], vv[MAXJ];
#pragma unroll
    for (int j = 0; j < MAXJ; ++j) {
        const int r = tid + j * NT;
        const bool in = j * NT < L && r < L;
        vk[j] = in ? sk[r] : -INFINITY;
        vv[j] = in ? sv[r] : -INFINITY;
    }
    // the K and the V value reduced over the block together (one pair of barriers for both)
    auto block_red2 = [&](float& a, float& b, bool is_max) {
        a = is_max ? wave_max(a) : wave_sum(a);
        b = is_max ? wave_max(b) : wave_sum(b);
        __syncthreads();
        if (lane == 0) { sm[wave] = a; sm[NW + wave] = b; }
        __syncthreads();
        float ra = sm[0], rb = sm[NW];
        for (int i = 1; i < NW; ++i) {
            ra = is_max ? fmaxf(ra, sm[i]) : ra + sm[i];
            rb = is_max ? fmaxf(rb, sm[NW + i]) : rb + sm[NW + i];
        }
        a = ra;
        b = rb;
    };
    float mk = -INFINITY, mv = -INFINITY;
#pragma unroll
    for (int j = 0; j < MAXJ; ++j) { mk = fmaxf(mk, vk[j]); mv = fmaxf(mv, vv[j]); }
    block_red2(mk, mv, true);
    float zk = 0.0f, zv = 0.0f;
#pragma unroll
    for (int j = 0; j < MAXJ; ++j) {
        if (j * NT < L) {
            vk[j] = expf(vk[j] - mk);
            vv[j] = expf(vv[j] - mv);
            zk += vk[j];
            zv += vv[j];
        }
    }
    block_red2(zk, zv, false);
#pragma unroll
    for (int j = 0; j < MAXJ; ++j) {
        const int r = tid + j * NT;
        if (j * NT < L && r < L) {
            const float sc = vk[j] / zk + vv[j] / zv;      // Eq. 7-8
            if (out) out[r] = sc;
            if (key) key[r] = sc;
        }
    }
}

template <typename T, int DH>
__device__ __forceinline__ void score_chunk_block(int L, int ddof, const T* __restrict__ Kcur,
                                                  const T* __restrict__ Kref, const T* __restrict__ Vcur,
                                                  const T* __restrict__ Vref, int64_t stride, ScoreLds& sh,
                                                  float* __restrict__ out) {
    constexpr int VEC = Elem<T>::VEC;
    constexpr int NW = FUSED_THREADS / 64;
    constexpr int d = DH;
    constexpr int lpr = d / VEC;              // lanes per row
    constexpr int rpp = FUSED_THREADS / lpr;  // rows per pass
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = tid % lpr, rg = tid / lpr;
    const float inv_d = 1.0f / float(d);            // exact: head_dim is a power of two
    const float inv_dof = 1.0f / float(d - ddof);
    // ---- phase 1
    {
        float mn[2][VEC], mx[2][VEC];
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int i = 0; i < VEC; ++i) { mn[z][i] = INFINITY; mx[z][i] = -INFINITY; }
        for (int r = rg; r < L; r += 2 * rpp) {
            // two rows of K and of V in flight
            const int r2 = r + rpp < L ? r + rpp : r;
            float k0[VEC], k1[VEC], v0[VEC], v1[VEC];
            Elem<T>::load(Kref + int64_t(r) * stride + sub * VEC, k0);
            Elem<T>::load(Vref + int64_t(r) * stride + sub * VEC, v0);
            Elem<T>::load(Kref + int64_t(r2) * stride + sub * VEC, k1);
            Elem<T>::load(Vref + int64_t(r2) * stride + sub * VEC, v1);
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                mn[0][i] = fminf(mn[0][i], fminf(k0[i], k1[i])); mx[0][i] = fmaxf(mx[0][i], fmaxf(k0[i], k1[i]));
                mn[1][i] = fminf(mn[1][i], fminf(v0[i], v1[i])); mx[1][i] = fmaxf(mx[1][i], fmaxf(v0[i], v1[i]));
            }
        }
        // lanes of one wave that hold the same channels (different rows)
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            across_groups<lpr>(mn[z], [](float x, float y) { return fminf(x, y); });
            across_groups<lpr>(mx[z], [](float x, float y) { return fmaxf(x, y); });
        }
        if (lane < lpr) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                sh.red[0][wave][lane * VEC + i] = mn[0][i]; sh.red[1][wave][lane * VEC + i] = mx[0][i];
                sh.red[2][wave][lane * VEC + i] = mn[1][i]; sh.red[3][wave][lane * VEC + i] = mx[1][i];
            }
        }
        __syncthreads();
        if (tid < 2 * d) {
            const int z = tid / d, c = tid % d;
            float a = INFINITY, m = -INFINITY;
            for (int w = 0; w < NW; ++w) { a = fminf(a, sh.red[2 * z][w][c]); m = fmaxf(m, sh.red[2 * z + 1][w][c]); }
            float den = m - a;
            den = den == 0.0f ? 1.0f : den;
            sh.s_mn[z][c] = a;
            sh.s_den[z][c] = den;
            sh.s_inv[z][c] = 1.0f / den;
        }
        __syncthreads();
    }
    // ---- phase 2: sigma of every row of chunk p; two rows of K and of V in flight per thread
    {
        float mn[2][VEC], den[2][VEC], inv[2][VEC];
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                mn[z][i] = sh.s_mn[z][sub * VEC + i]; den[z][i] = sh.s_den[z][sub * VEC + i]; inv[z][i] = sh.s_inv[z][sub * VEC + i];
            }
        for (int r = rg; r < L; r += 2 * rpp) {
            const bool has2 = r + rpp < L;
            const int r2 = has2 ? r + rpp : r;
            float x[4][VEC];   // K row r, K row r2, V row r, V row r2
            Elem<T>::load(Kcur + int64_t(r) * stride + sub * VEC, x[0]);
            Elem<T>::load(Kcur + int64_t(r2) * stride + sub * VEC, x[1]);
            Elem<T>::load(Vcur + int64_t(r) * stride + sub * VEC, x[2]);
            Elem<T>::load(Vcur + int64_t(r2) * stride + sub * VEC, x[3]);
            float sm4[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int z = j >> 1;
                float acc = 0.0f;
#pragma unroll
                for (int i = 0; i < VEC; ++i) {
                    const float a0 = x[j][i] - mn[z][i];
                    float q0 = a0 * inv[z][i];
                    q0 = __builtin_fmaf(__builtin_fmaf(-den[z][i], q0, a0), inv[z][i], q0);   // correctly rounded a0 / den
                    x[j][i] = q0;
                    acc += q0;
                }
                sm4[j] = acc;
            }
            group_sums<lpr>(sm4);
            float var4[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float m = sm4[j] * inv_d;
                float acc = 0.0f;
#pragma unroll
                for (int i = 0; i < VEC; ++i) { const float dd = x[j][i] - m; acc += dd * dd; }
                var4[j] = acc;
            }
            group_sums<lpr>(var4);
            if (sub == 0) {
                sh.sig[0][r] = sqrtf(var4[0] * inv_dof);
                sh.sig[1][r] = sqrtf(var4[2] * inv_dof);
                if (has2) {
                    sh.sig[0][r2] = sqrtf(var4[1] * inv_dof);
                    sh.sig[1][r2] = sqrtf(var4[3] * inv_dof);
                }
            }
        }
        __syncthreads();
    }
    // ---- phase 3
    softmax_sum_block<FUSED_THREADS>(sh.sig[0], sh.sig[1], sh.sm, L, out);
}

}  // namespace lrsa
