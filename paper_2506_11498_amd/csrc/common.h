// Internal declarations shared by the LRSA kernels and the C-ABI dispatch (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lrsa {

// Problem description after validation: the ABI struct plus the derived partition
// (sink, P full chunks of the lag size, tail R, nq query chunks, Ns scored chunks).
struct Dims {
    int B, Hq, Hkv, G, n, d;
    int S, L, K, ddof, lp;
    int P, R, nq, Ns;
    float scale;
    int dtype;  // 0 fp32, 1 bf16
    int compact;  // MFMA attention kernels read a condensed copy of the gather list's K/V rows
    int64_t qs[3], ks[3];
    // Attention over a window of query rows (one "filling" step of m chunks): rows [row_begin, row_end), which
    // are the query chunks [fq0, fq1) plus the sink rows when row_begin == 0.  The whole sequence by default.
    int row_begin, row_end, fq0, fq1;
    int64_t lse_stride;   // floats between the lse (and D) rows of consecutive (batch, query head) pairs
    int acc;              // backward adds dK, dV into fp32 accumulators instead of writing them
};

// Number of entries of the gather list "sink ++ survivors of chunks 0..c-1" and the first
// position of the contiguous (fully kept) window, for a query in chunk q (q < 0: sink query).
__host__ __device__ inline int gather_count(const Dims& D, int q) {
    if (q < 0) return 0;
    int c = q - D.lp;
    return D.S + D.K * (c > 0 ? c : 0);
}
__host__ __device__ inline int window_start(const Dims& D, int q) {
    if (q < 0) return 0;
    int c = q - D.lp;
    return D.S + D.L * (c > 0 ? c : 0);
}

// ---- launchers (each enqueues on `st` and returns the first HIP error) ----------------------
size_t score_ws_bytes(const Dims&);
int score_route(const Dims&);
hipError_t launch_score(const Dims&, const void* K, const void* V, float* score, void* ws, hipStream_t st);

hipError_t launch_softmax_select(const Dims&, const float* sigma, float* score, int32_t* idx, hipStream_t st);
bool score_resident_applies(const Dims&);
int score_poll_limit(int polls);
hipError_t launch_score_resident(const Dims&, const void* K, const void* V, float* score, int32_t* idx, float* sigma,
                                 hipStream_t st);

size_t select_ws_bytes(const Dims&);
hipError_t launch_select(const Dims&, const float* score, int32_t* idx, void* ws, hipStream_t st);
hipError_t launch_check_idx(const Dims&, const int32_t* idx, int32_t* bad_rows, hipStream_t st);
size_t decode_ws_bytes(const Dims&);
bool cache_compress_supported(const Dims&);
hipError_t launch_cache_compress(const Dims&, void* Kc, void* Vc, int32_t* pos, int len, int done, int steps, hipStream_t st);
// the same with a workspace: all steps at once over many workgroups
size_t cache_compress_ws_bytes(const Dims&, int len, int done, int steps);
bool cache_step_is_long(const Dims&);   // a single step is the faster one with a workspace
hipError_t launch_cache_compress_ws(const Dims&, void* Kc, void* Vc, int32_t* pos, int len, int done, int steps, void* ws,
                                    hipStream_t st);
size_t cache_sigma_ws_floats(const Dims&);
hipError_t launch_cache_sigma(const Dims&, const void* K, const void* V, float* mm, float* sigma, hipStream_t st);
hipError_t launch_cache_select(const Dims&, const float* sigma, int32_t* idx, hipStream_t st);
hipError_t launch_decode_attn(const Dims&, const void* q, const void* Kc, const void* Vc, int len, void* O, float* lse,
                              void* ws, hipStream_t st);
// lrsa_decode_attn_static: bytes of the library-owned scratch array and what a call needs of it
constexpr size_t DECODE_STATIC_SCRATCH_BYTES = size_t(4) << 20;
size_t decode_static_need(const Dims&, int len);
hipError_t launch_decode_attn_static(const Dims&, const void* q, const void* Kc, const void* Vc, int len, void* O,
                                     float* lse, hipStream_t st);
hipError_t launch_score_select(const Dims&, const void* K, const void* V, float* score, int32_t* idx, void* ws, hipStream_t st);

size_t attn_fwd_generic_ws_bytes(const Dims&);
hipError_t launch_attn_fwd_generic(const Dims&, const void* Q, const void* K, const void* V, const int32_t* idx,
                                   void* O, float* lse, void* ws, hipStream_t st);
size_t attn_bwd_generic_ws_bytes(const Dims&);
hipError_t launch_attn_bwd_generic(const Dims&, const void* Q, const void* K, const void* V, const void* O,
                                   const void* dO, const float* lse, const int32_t* idx, void* dQ, void* dK,
                                   void* dV, void* ws, hipStream_t st);

// fp32 data on the fp32 matrix instruction
bool f32_tiles_supported(const Dims&);
size_t attn_bwd_f32_ws_bytes(const Dims&);
int attn_f32_query_waves(const Dims&);
int attn_f32_key_waves();
int attn_f32_slices(const Dims&);
hipError_t launch_attn_fwd_f32(const Dims&, const void* Q, const void* K, const void* V, const int32_t* idx, void* O, float* lse, hipStream_t st);
hipError_t launch_attn_bwd_f32(const Dims&, const void* Q, const void* K, const void* V, const void* O, const void* dO, const float* lse,
                               const int32_t* idx, void* dQ, void* dK, void* dV, void* ws, hipStream_t st);

bool mfma_supported(const Dims&);
bool mfma_grids_fit(const Dims&);
size_t attn_fwd_mfma_ws_bytes(const Dims&);
hipError_t launch_attn_fwd_mfma(const Dims&, const void* Q, const void* K, const void* V, const int32_t* idx,
                                void* O, float* lse, void* ws, hipStream_t st);
size_t attn_bwd_mfma_ws_bytes(const Dims&);       // for the fastest plan
void attn_bwd_mfma_parts(const Dims&, int32_t* gather, int32_t* window);   // of the fastest plan
int attn_mfma_fwd_waves(const Dims&);
void attn_bwd_mfma_plan(const Dims&, size_t ws_bytes, int32_t* dq_waves, int32_t* waves, int32_t* slices, int32_t* gather, int32_t* window);
size_t attn_bwd_mfma_ws_min_bytes(const Dims&);   // for one without splits: what a call must have
hipError_t launch_attn_bwd_mfma(const Dims&, const void* Q, const void* K, const void* V, const void* O,
                                const void* dO, const float* lse, const int32_t* idx, void* dQ, void* dK,
                                void* dV, float* accK, float* accV, void* ws, size_t ws_bytes, hipStream_t st);
hipError_t launch_bwd_acc_finish(const Dims&, const float* accK, const float* accV, void* dK, void* dV, hipStream_t st);

// A launch has fewer than 2^32 work-items per grid dimension (and fewer than 2^31 workgroups).  The runtime does not refuse a larger
// one: the count wraps and most workgroups never run.
inline bool grid_fits(int64_t workgroups, int threads) { return workgroups < (int64_t(1) << 32) / threads && workgroups < (int64_t(1) << 31); }

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Brackets one kernel launch with HIP events on its stream when timing is switched on
// (lrsa_timing_enable); does nothing otherwise.
class ScopedKernelTimer {
  public:
    ScopedKernelTimer(const char* name, hipStream_t st);
    ~ScopedKernelTimer();
  private:
    hipStream_t st_;
    int slot_;
};
#define LRSA_TIMED_LAUNCH(name, st, ...)            \
    do {                                            \
        ::lrsa::ScopedKernelTimer timer_(name, st); \
        hipLaunchKernelGGL(__VA_ARGS__);            \
    } while (0)

// ---- device helpers ---------------------------------------------------------------------------
#if defined(__HIPCC__)
typedef uint16_t bf16_t;  // raw bfloat16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t x) { return __uint_as_float(uint32_t(x) << 16); }
// round to nearest even (inputs are finite)
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return bf16_t(u >> 16);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
    static constexpr int VEC = 4;  // elements per 16-byte load
    __device__ static __forceinline__ void load(const float* p, float (&out)[4]) {
        float4 v = *reinterpret_cast<const float4*>(p);
        out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
    }
    __device__ static __forceinline__ void unpack(const uint4& v, float (&out)[4]) {   // the 16 bytes of a load
        out[0] = __uint_as_float(v.x); out[1] = __uint_as_float(v.y); out[2] = __uint_as_float(v.z); out[3] = __uint_as_float(v.w);
    }
    __device__ static __forceinline__ float get(const float* p) { return *p; }
    __device__ static __forceinline__ void put(float* p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
    static constexpr int VEC = 8;
    __device__ static __forceinline__ void load(const bf16_t* p, float (&out)[8]) {
        unpack(*reinterpret_cast<const uint4*>(p), out);
    }
    __device__ static __forceinline__ void unpack(const uint4& v, float (&out)[8]) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            out[2 * i] = __uint_as_float(w[i] << 16);
            out[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    __device__ static __forceinline__ float get(const bf16_t* p) { return bf16_to_f32(*p); }
    __device__ static __forceinline__ void put(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};

// ---- reductions and scans over the lanes of a wave -----------------------------------------------------------------
// All in the vector pipe: half-wave and row exchanges by permlane swaps, rotations inside a row of 16 lanes by
// data-parallel primitives.  (A shuffle through LDS costs its latency at every one of the six levels: the block-wide
// chains of softmax and selection take 7.4 us at 240 chunks of 1024 rows, 8.6 us with shuffles.)
typedef unsigned int lanes_u32x2 __attribute__((ext_vector_type(2)));
// {own, other} in some order: the values of lane l and of lane l ^ 32 (l ^ 16)
__device__ __forceinline__ lanes_u32x2 pair32(uint32_t v) { return __builtin_amdgcn_permlane32_swap(v, v, false, false); }
__device__ __forceinline__ lanes_u32x2 pair16(uint32_t v) { return __builtin_amdgcn_permlane16_swap(v, v, false, false); }
template <int N>
__device__ __forceinline__ uint32_t row_ror(uint32_t v) {   // rotation by N inside the row of 16
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x120 | N, 0xf, 0xf, false));
}
// op over all 64 lanes, every lane gets the result; the pairs are those of a butterfly 32, 16, 8, 4, 2, 1
template <class Op>
__device__ __forceinline__ float row16_all(float v, Op op) {
    v = op(v, __uint_as_float(row_ror<8>(__float_as_uint(v))));
    v = op(v, __uint_as_float(row_ror<4>(__float_as_uint(v))));
    v = op(v, __uint_as_float(row_ror<2>(__float_as_uint(v))));
    return op(v, __uint_as_float(row_ror<1>(__float_as_uint(v))));
}
template <class Op>
__device__ __forceinline__ float wave_all(float v, Op op) {
    const lanes_u32x2 a = pair32(__float_as_uint(v));
    v = op(__uint_as_float(a.x), __uint_as_float(a.y));
    const lanes_u32x2 c = pair16(__float_as_uint(v));
    v = op(__uint_as_float(c.x), __uint_as_float(c.y));
    return row16_all(v, op);
}
__device__ __forceinline__ float wave_sum(float v) { return wave_all(v, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float wave_max(float v) { return wave_all(v, [](float a, float b) { return fmaxf(a, b); }); }
// sum over the 16 lanes of a row, every lane gets the total
__device__ __forceinline__ float row16_sum(float v) { return row16_all(v, [](float a, float b) { return a + b; }); }
// sums over aligned groups of 8, 16 or 32 lanes of N values together, so that their chains overlap; every lane gets its group's; the pairs
// are those of a butterfly 16, 8, 4, 2, 1
template <int LANES, int N>
__device__ __forceinline__ void group_sums(float (&v)[N]) {
    static_assert(LANES == 8 || LANES == 16 || LANES == 32, "group size");
    if constexpr (LANES == 8) {
        // of the two row shifts by 4 each writes the half of the lanes whose source lies in their own group of 8
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int x = __float_as_int(v[j]);
            const int up = __builtin_amdgcn_update_dpp(0, x, 0x104, 0xf, 0x5, false);            // row_shl:4 into lanes 0-3 and 8-11
            v[j] += __int_as_float(__builtin_amdgcn_update_dpp(up, x, 0x114, 0xf, 0xa, false));  // row_shr:4 into lanes 4-7 and 12-15
            v[j] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[j]), 0x4e, 0xf, 0xf, false));   // quad_perm 2 3 0 1
            v[j] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v[j]), 0xb1, 0xf, 0xf, false));   // quad_perm 1 0 3 2
        }
    } else {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            if constexpr (LANES == 32) {
                const lanes_u32x2 a = pair16(__float_as_uint(v[j]));
                v[j] = __uint_as_float(a.x) + __uint_as_float(a.y);
            }
            v[j] = row16_sum(v[j]);
        }
    }
}
// op (min or max) of N values over the lanes l, l + LANES, l + 2 * LANES ... of a wave
template <int LANES, int N, class Op>
__device__ __forceinline__ void across_groups(float (&v)[N], Op op) {
    static_assert(LANES == 8 || LANES == 16 || LANES == 32, "group size");
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if constexpr (LANES == 8) v[j] = op(v[j], __uint_as_float(row_ror<8>(__float_as_uint(v[j]))));
        if constexpr (LANES <= 16) {
            const lanes_u32x2 c = pair16(__float_as_uint(v[j]));
            v[j] = op(__uint_as_float(c.x), __uint_as_float(c.y));
        }
        const lanes_u32x2 a = pair32(__float_as_uint(v[j]));
        v[j] = op(__uint_as_float(a.x), __uint_as_float(a.y));
    }
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
    lanes_u32x2 a = pair32(v);
    v = a.x < a.y ? a.x : a.y;
    a = pair16(v);
    v = a.x < a.y ? a.x : a.y;
    uint32_t o = row_ror<8>(v); v = o < v ? o : v;
    o = row_ror<4>(v); v = o < v ? o : v;
    o = row_ror<2>(v); v = o < v ? o : v;
    o = row_ror<1>(v); return o < v ? o : v;
}
// inclusive prefix sum over the 64 lanes (lanes before the first contribute zero)
__device__ __forceinline__ int wave_iscan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return v;
}
#endif

}  // namespace lrsa
