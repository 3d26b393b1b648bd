// Building blocks of the bf16 MFMA attention kernels (gfx950): 32x32x16 MFMA wrappers, the
// swizzled row-major LDS tile that every operand is staged in, and its two read patterns.
//
// MFMA v_mfma_f32_32x32x16_bf16, lane l (l32 = l % 32, g = l / 32):
//   A operand: row l32,  k-slots 8g .. 8g+7        B operand: column l32, k-slots 8g .. 8g+7
//   C/D:       column l32, 16 floats i -> row 8*(i/4) + 4g + i%4
//
// A tile is [rows][DH bf16], DH = head_dim = 128 or 64: a row is 256 bytes = 16 chunks of 16 bytes (128 bytes = 8
// chunks); chunk c of row r is stored at chunk c ^ swz(r).  swz is a bijection on 16 consecutive rows (DH = 64: on 8
// pairs of rows, a pair filling 256 bytes), so row-pattern reads of 16 lanes hit 16 different 16-byte units of the
// 256-byte bank line, and it moves rows r, r+1, r+2, r+3 (pairs of rows) to different 64-byte units, so transposed
// reads of 4 rows x 32 bytes spread over the banks.
#pragma once
#include "common.h"

namespace lrsa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

template <int DH> constexpr int ROW_BYTES = 2 * DH;          // a tile row
template <int DH> constexpr int KK = DH / 16;                // MFMA steps of a contraction over head_dim
template <int DH> constexpr int DB = DH / 32;                // blocks of 32 channels
template <int DH> constexpr int COPY_ROWS = 1024 / (2 * DH); // tile rows one asynchronous wave copy fills

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

template <int DH>
__device__ __forceinline__ int swz(int r) {
    if constexpr (DH == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
    return ((r & 2) << 1) | ((r >> 2) & 3);
}

// byte offset of chunk `c` (16 bytes) of row `r`
template <int DH>
__device__ __forceinline__ int tile_off(int r, int c) { return r * ROW_BYTES<DH> + ((c ^ swz<DH>(r)) << 4); }

// Two read patterns:
//  rows  the tile's rows as MFMA rows/columns and head_dim as the contraction: the lane takes row rb + l32, channels
//        16*kk + 8g .. +7 (one 16-byte LDS read).
//  cols  head_dim as MFMA rows and 16 tile rows as the contraction ("transposed" read): the lane takes channel
//        db*32 + l32 and the 8 k-slots of its half g, where slot j is tile row rb16 + 8*(j/4) + 4g + j%4 -- exactly the
//        rows a C-layout accumulator hands over when its registers 8h .. 8h+7 are reused as the other operand.
//        ds_read_b64_tr_b16 works per 16-lane group: lane i receives, as element e, element i%4 of the 8 bytes that
//        lane 4e + i/4 of its group points at.  So source lane lam points at row 4g + lam/4 (+8 for the second read),
//        channels dbase + 4*(lam%4) .. +3.
// Per-lane byte offsets of the two read patterns inside a tile.  Because the swizzle is an XOR on
// chunk bits that the channel-block index also occupies, the offset of channel block kk (or db, and of
// the second transposing read) is the block-0 offset XOR a compile-time constant: two registers per
// lane describe every read, other row blocks (multiples of 16 rows) are immediates on top.
struct LaneOffs {
    int row;   // read_rows: row l32, channel block 0
    int col;   // read_cols: channel block 0, first transposing read
};
template <int DH>
__device__ __forceinline__ LaneOffs make_lane_offs(int lane) {
    LaneOffs o;
    const int l32 = lane & 31, g = lane >> 5, lam = lane & 15, m = (lane >> 4) & 1;
    o.row = tile_off<DH>(l32, g);
    const int ch = 16 * m + 4 * (lam & 3);
    o.col = tile_off<DH>(4 * g + (lam >> 2), ch >> 3) + (ch & 7) * 2;
    return o;
}
// rb is a multiple of 32, rb16 of 16
template <int DH>
__device__ __forceinline__ bf16x8 read_rows_o(const unsigned char* tile, const LaneOffs& o, int rb, int kk) {
    return *reinterpret_cast<const bf16x8*>(tile + (o.row ^ (kk << 5)) + rb * ROW_BYTES<DH>);
}
template <int DH>
__device__ __forceinline__ bf16x8 read_cols_o(const unsigned char* tile, const LaneOffs& o, int rb16, int db) {
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(tile + (o.col ^ (db << 6)) + rb16 * ROW_BYTES<DH>));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_ptr)(tile + (o.col ^ ((db << 6) | 32)) + (rb16 + 8) * ROW_BYTES<DH>));
    union { s16x4 h[2]; bf16x8 v; } u;
    u.h[0] = lo;
    u.h[1] = hi;
    return u.v;
}

// The same two reads with the tile's LDS address already folded into the lane's offset register (one add
// per tile instead of one per read): valid when the tile starts on a 256-byte boundary, because XORing a
// constant below a row's bytes then commutes with adding the base.  rows16 is a compile-time row offset (multiple of 16).
typedef bf16x8 __attribute__((address_space(3))) * lds_bf16x8_ptr;
__device__ __forceinline__ unsigned lds_addr(const void* p) {
    return (unsigned)(size_t)(__attribute__((address_space(3))) void*)p;
}
__device__ __forceinline__ bf16x8 read_rows_a(unsigned arow, int kk) {
    return *(lds_bf16x8_ptr)(size_t)(arow ^ unsigned(kk << 5));
}
template <int DH>
__device__ __forceinline__ bf16x8 read_cols_a(unsigned acol, int rows16, int db) {
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(size_t)((acol ^ unsigned(db << 6)) + rows16 * ROW_BYTES<DH>));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_ptr)(size_t)((acol ^ unsigned((db << 6) | 32)) + (rows16 + 8) * ROW_BYTES<DH>));
    union { s16x4 h[2]; bf16x8 v; } u;
    u.h[0] = lo;
    u.h[1] = hi;
    return u.v;
}

// registers i0 .. i0+7 of a C-layout accumulator as a bf16 operand
__device__ __forceinline__ bf16x8 pack8(const f32x16& v, int i0) {
    f32x8 t;
#pragma unroll
    for (int j = 0; j < 8; ++j) t[j] = v[i0 + j];
    return __builtin_convertvector(t, bf16x8);
}

// A C-layout block of fp32 weights (probabilities, dS) as MFMA operand.  TERMS == 1: rounded to bf16.  TERMS == 3: as
// the sum of three bf16 numbers (the rounded value, its rounded residual and the residual of that), which hold all 24
// bits: head_dim 64, where the weights are fp32 also in the plain kernels.
template <int TERMS> struct Weights {
    bf16x8 t[TERMS];
};
template <int TERMS>
__device__ __forceinline__ Weights<TERMS> pack_weights(const f32x16& v, int i0) {
    Weights<TERMS> w;
    f32x8 r;
#pragma unroll
    for (int j = 0; j < 8; ++j) r[j] = v[i0 + j];
#pragma unroll
    for (int t = 0; t < TERMS; ++t) {
        w.t[t] = __builtin_convertvector(r, bf16x8);
        if (t + 1 < TERMS)
#pragma unroll
            for (int j = 0; j < 8; ++j) r[j] -= float(w.t[t][j]);
    }
    return w;
}
template <int TERMS>
__device__ __forceinline__ f32x16 mfma32_w(bf16x8 a, const Weights<TERMS>& w, f32x16 c) {
#pragma unroll
    for (int t = TERMS - 1; t >= 0; --t) c = mfma32(a, w.t[t], c);   // the small terms first
    return c;
}
template <int DH> constexpr int TERMS = DH == 64 ? 3 : 1;

// Tiles in which some (query, key) pairs are masked, head_dim 64: a weight of zero times an infinity would be NaN in the sums of a
// query (key) that does not see the row.  finite_operand() makes zeros of an operand's non-finite values; poison_rows() turns
// the logits of a tile's rows that have any into NaN (a product with zeros: 0 otherwise), for the pairs that do see them.
__device__ __forceinline__ bf16x8 finite_operand(bf16x8 a) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 w = __builtin_bit_cast(u32x4, a);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t lo = (w[i] & 0x7f80u) == 0x7f80u ? 0xffff0000u : ~0u, hi = (w[i] & 0x7f800000u) == 0x7f800000u ? 0xffffu : ~0u;
        w[i] &= lo & hi;
    }
    return __builtin_bit_cast(bf16x8, w);
}
__device__ __forceinline__ f32x16 poison_rows(bf16x8 rows, f32x16 s) { return mfma32(rows, bf16x8{}, s); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Units of the logits inside the kernels: log2 units, so that a weight is one fma and one exponential; head_dim 64: natural
// units and a multiplication more, because scale * log2(e) and lse * log2(e) are rounded numbers, whose errors grow with the
// logit (scale = 1/8 is exact) and would show beside weights of 24 bits.
constexpr float LOG2E = 1.4426950408889634f;
template <int DH> constexpr float LOGIT_UNIT = DH == 64 ? 1.0f : LOG2E;   // factor of a natural logit
template <int DH>
__device__ __forceinline__ float exp_units(float x) { return fast_exp2(DH == 64 ? x * LOG2E : x); }
// exp(scale * s - ref); c = scale in the kernel's units
template <int DH>
__device__ __forceinline__ float weight(float s, float c, float ref) { return exp_units<DH>(__builtin_fmaf(s, c, -ref)); }

// ---- asynchronous global -> LDS copies (global_load_lds_dwordx4) --------------------------------
// One wave instruction moves 64 x 16 bytes: lane l's 16 bytes land at lds_base + 16*l (checked on the
// hardware), i.e. COPY_ROWS consecutive tile rows starting at row r0.  The swizzle is applied on
// the global side: the lane whose slot is physical chunk pc of row r fetches logical chunk pc ^ swz(r).
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void gbl_void_t;

// tile row and 16-byte logical chunk this lane fetches when its wave fills COPY_ROWS rows from r0 on
template <int DH>
__device__ __forceinline__ int async_row(int r0, int lane) { return r0 + lane / (DH / 8); }
template <int DH>
__device__ __forceinline__ int async_chunk(int row, int lane) { return (lane & (DH / 8 - 1)) ^ swz<DH>(row); }

// The copies are issued through inline assembly, so the compiler does not know that LDS is written
// behind its back: it would otherwise make LDS reads of OTHER ring stages wait for all copies in flight
// (its alias bookkeeping for such copies is limited).  Ordering is the kernels' own business: they wait
// with wait_vmcnt<n>() for the copies of the stage they are about to read and synchronise the workgroup.
// Hidden operations are harmless for the compiler's own vmcnt arithmetic: vector memory loads complete in
// order, so "at most n outstanding" still implies that everything it knows to be older has arrived.
// M0 (the LDS base of the copy) is saved and restored around the instruction.
__device__ __forceinline__ void async_copy16(const void* src, const void* lds_dst) {
    const unsigned la = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lds_void_t*)lds_dst);   // wave-uniform
    unsigned keep;
    asm volatile(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\ts_mov_b32 m0, %0"
        : "=&s"(keep)
        : "v"(src), "s"(la)
        : "memory");
}
__device__ __forceinline__ void async_copy4(const void* src, const void* lds_dst) {
    const unsigned la = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lds_void_t*)lds_dst);
    unsigned keep;
    asm volatile(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %1, off\n\ts_mov_b32 m0, %0"
        : "=&s"(keep)
        : "v"(src), "s"(la)
        : "memory");
}
// The same copy with the global address given as a wave-uniform base (scalar registers) plus this lane's unsigned
// 32-bit byte offset, and the LDS destination as a wave-uniform byte address: no 64-bit vector arithmetic and no
// pointer conversion per copy.  The caller guarantees offsets below 4 GiB.
__device__ __forceinline__ void async_copy16_so(const void* base, unsigned voff, unsigned lds_byte_addr) {
    unsigned keep;
    asm volatile(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b32 m0, %0"
        : "=&s"(keep)
        : "v"(voff), "s"(base), "s"(lds_byte_addr)
        : "memory");
}
// ... and with a per-lane 64-bit global address (rows that come from two different buffers)
__device__ __forceinline__ void async_copy16_la(const void* src, unsigned lds_byte_addr) {
    unsigned keep;
    asm volatile(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\ts_mov_b32 m0, %0"
        : "=&s"(keep)
        : "v"(src), "s"(lds_byte_addr)
        : "memory");
}
// src: this lane's 16 bytes in global memory; tile: LDS tile base; r0: first of the COPY_ROWS rows (wave-uniform)
template <int DH>
__device__ __forceinline__ void async_rows(const void* src, unsigned char* tile, int r0) {
    async_copy16(src, tile + r0 * ROW_BYTES<DH>);
}

// s_waitcnt vmcnt(0) in the form the compiler understands: every vector memory load it has issued so far
// (Q fragments and the like) is complete afterwards, so it will not place waits of its own for them inside
// the ring loop, where they would also drain the asynchronous copies.
__device__ __forceinline__ void wait_all_vmem_known() { __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8)); }

// Pins a loaded register operand at this point of the program: the empty volatile statement "uses and
// redefines" it, so the load that produced it cannot be moved below (volatile statements keep their order,
// and the asynchronous copies are such statements) and later uses carry no pending-load bookkeeping.
template <class T>
__device__ __forceinline__ void pin_loaded(T& v) {
    asm volatile("" : "+v"(v));
}

// s_waitcnt vmcnt(n) alone
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Scalar-cache load of one 32-bit word at a wave-uniform address, issued explicitly (the compiler only
// picks the scalar path for memory it can prove unwritten, which the asynchronous copies defeat).  The
// result may be used only after smem_wait() on the same variables.
__device__ __forceinline__ int smem_load(const int32_t* base, int index) {
    int v;
    const int off = __builtin_amdgcn_readfirstlane(index * 4);
    asm volatile("s_load_dword %0, %1, %2" : "=s"(v) : "s"(base), "s"(off) : "memory");
    return v;
}
// eight scalars (no array: indexing a private array invites the compiler to move it to memory)
struct Scalar8 { int a0, a1, a2, a3, a4, a5, a6, a7; };
// waits for all outstanding scalar loads (and LDS reads); ties the 8 values to the wait (they are scalar
// registers already: the loads' outputs)
__device__ __forceinline__ void smem_wait(Scalar8& v) {
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+s"(v.a0), "+s"(v.a1), "+s"(v.a2), "+s"(v.a3), "+s"(v.a4), "+s"(v.a5), "+s"(v.a6), "+s"(v.a7)
                 :
                 : "memory");
}
// the one of four scalars that belongs to this lane's quarter q4 = lane / 16 (three conditional moves)
__device__ __forceinline__ int pick4(int q4, int x0, int x1, int x2, int x3) {
    int r = x0;
    r = q4 == 1 ? x1 : r;
    r = q4 == 2 ? x2 : r;
    r = q4 == 3 ? x3 : r;
    return r;
}

// Workgroup barrier without the memory fence of __syncthreads(): the fence would make the compiler wait
// for ALL outstanding vector memory operations, i.e. also for the asynchronous copies of later ring
// stages.  The caller has already waited (wait_vmcnt) for exactly the copies that must have landed; LDS
// reads of the stage about to be refilled have been consumed by MFMAs before the wave gets here.  The
// "memory" clobber keeps the compiler from moving LDS accesses across the barrier.
__device__ __forceinline__ void ring_barrier() { asm volatile("s_barrier" ::: "memory"); }

// position of stream entry j: the gather list (sink positions, then the flattened survivor
// lists) followed by the contiguous window that starts at cs
__device__ __forceinline__ int stream_pos(const Dims& D, const int32_t* idx_h, int j, int ng, int cs) {
    if (j < ng) return j < D.S ? j : idx_h[j - D.S];
    return cs + (j - ng);
}

// x / d for x up to the largest one given on the host, by a multiplication (a division is some thirty dependent instructions, and a
// workgroup needs several before it can ask for its first row): m = ceil(2^32 / d) is exact as long as x * d < 2^32; 0: divide.
struct FastDiv {
    unsigned d, m;
};
inline FastDiv make_fast_div(int64_t d, int64_t x_max) {
    const bool exact = d > 1 && x_max < (int64_t(1) << 32) / d;
    return FastDiv{unsigned(d), exact ? unsigned(((int64_t(1) << 32) + d - 1) / d) : 0u};
}
__host__ __device__ __forceinline__ int fast_div(int x, FastDiv f) {
#if defined(__HIP_DEVICE_COMPILE__)
    const unsigned q = __umulhi(unsigned(x), f.m);   // (a shifted product of 64 bits goes to the vector pipe)
#else
    const unsigned q = unsigned(uint64_t(unsigned(x)) * f.m >> 32);
#endif
    return f.m ? int(q) : f.d == 1 ? x : int(unsigned(x) / f.d);
}

// Which (batch, KV head, query tile) a workgroup of a query-outer kernel takes.
//
// A segment (the sink, or one query chunk) is a list of pieces, 32 rows of one query head each: block of heads by block of heads, rows
// in order, the heads of a block side by side.  A block is the group, or four of its heads where that divides it (with all eight of a
// group side by side 4 requests of 3.5K tokens, 16 heads on 2, lag 109, take 118 us instead of 113: no wave ends early).  All pieces
// of a segment walk the same gather list, so a workgroup takes any `waves` neighbours, one per wave, and the last workgroup of a segment is the only one with idle waves.  (Whole heads x a fixed number of rows per workgroup
// wasted up to half of them: 24 heads on 8, 2 requests of 6.2K tokens, lag 258 -- two tiles of 256 rows per chunk, the second
// with 2 -- forward 538 -> 335 us.)
//
// Orders of the tiles, the heaviest (latest) first in each.  With a multiple of eight heads, consecutive workgroup ids -- which the
// hardware deals round-robin to the 8 XCDs -- belong to 8 different KV heads, so that one XCD's L2 keeps serving the K / V rows of the same
// head until it is done.  Otherwise, and where all workgroups are resident at once, so that nothing is dealt later to a CU that is done
// early, all heads side by side; with two workgroups per CU the second 256 come backwards, so that a long one shares its CU with a
// short one.  2 requests of 4K tokens, 8 heads on 8: forward 51.4 us with the first order, 42.2 with the second; one head after
// another instead of side by side: 9.4K tokens, 12 heads on 4, 144 and 117 us; 16K tokens, 24 on 4, 751 and 701.
struct QTileMap {
    int sink_tiles, tpc, tiles;   // query tiles (of `waves` pieces): in the sink, per chunk, in all
    int tix_lo, tix_hi;           // the tiles that are launched (all of them unless a row window is set)
    int per_unit;                 // workgroups per (batch, KV head)
    int wgs;                      // workgroups of the launch
    int side_by_side, backwards;
    int heads;                    // of a block
    FastDiv by_unit, by_units, by_hkv, by_tpc, by_heads;
};
__host__ __device__ __forceinline__ bool decode_qtile(const QTileMap& M, const Dims& D, int i, int& b, int& h, int& tix) {
    int unit, w;
    if (M.side_by_side) {
        int j = i >> 3;
        if (M.backwards && (j >> 5) == 1) j = 95 - j;
        i = j * 8 + (i & 7);
        w = fast_div(i, M.by_units);
        if (w >= M.per_unit) return false;
        unit = i - w * D.B * D.Hkv;
    } else {
        const int j = i >> 3, e = fast_div(j, M.by_unit);
        unit = (i & 7) + 8 * e;
        w = j - e * M.per_unit;
    }
    b = fast_div(unit, M.by_hkv);
    h = unit - b * D.Hkv;
    tix = M.tix_hi - 1 - w;
    return true;
}
// The rows of tile `tix`: query chunk (-1: sink), end of the segment, first row and head (of the group) of this wave's piece, last row
// of the workgroup; false: it has none.  A wave whose first row is not below seg_end has no piece.
__host__ __device__ __forceinline__ bool qtile_rows(const QTileMap& M, const Dims& D, int tix, int waves, int wave, int& qc, int& seg_end, int& tw,
                                           int& head, int& t_last) {
    int ts, u0, rows;
    if (tix < M.sink_tiles) {
        qc = -1; ts = 0; u0 = tix * waves; rows = seg_end = D.S < D.n ? D.S : D.n;
    } else {
        const int tt = tix - M.sink_tiles;
        qc = fast_div(tt, M.by_tpc);
        ts = D.S + qc * D.L;
        u0 = (tt - qc * M.tpc) * waves;
        const int64_t e = int64_t(D.S) + int64_t(qc + 1) * D.L;
        seg_end = e < D.n ? int(e) : D.n;
        rows = D.L;
    }
    const int block = (rows + 31) / 32 * M.heads;   // pieces of a block of heads
    int u1 = u0 + waves - 1, hb = 0;                // hb: first head of the block that piece u0 is in
    while (u0 >= block && hb + M.heads < D.G) { u0 -= block; u1 -= block; hb += M.heads; }
    const bool next = u1 >= block && hb + M.heads < D.G;   // the tile reaches into the next block, whose first rows are there
    int u = u0 + wave;
    while (u >= block && hb + M.heads < D.G) { u -= block; hb += M.heads; }
    const int rb = fast_div(u, M.by_heads);
    tw = ts + rb * 32;                              // past the segment: no piece
    head = hb + u - rb * M.heads;
    t_last = next ? seg_end - 1 : min(ts + (fast_div(u1, M.by_heads) + 1) * 32, seg_end) - 1;
    return next || ts + fast_div(u0, M.by_heads) * 32 < seg_end;
}

// ---- condensed KV cache --------------------------------------------------------------------------
// Kc, Vc [B, Hkv, gl, 128] bf16, contiguous: row j of a head is the K (V) row of entry j of its gather list
// (sink tokens, then the survivors chunk by chunk); gl = S + K * Ns.
inline int gather_list_len(const Dims& D) { return D.nq > 0 ? D.S + D.K * D.Ns : 0; }
inline size_t compact_kv_bytes(const Dims& D) {
    return D.compact ? 2 * align256(size_t(D.B) * D.Hkv * gather_list_len(D) * 128 * sizeof(bf16_t)) : 0;
}
hipError_t launch_compact_kv(const Dims& D, const void* K, const void* V, const int32_t* idx, void* Kc, void* Vc,
                             hipStream_t st);
// address of the row of stream entry j (gather list, then the contiguous window) with a condensed cache
__device__ __forceinline__ const bf16_t* stream_row(const bf16_t* Zc, const bf16_t* Z, int64_t stride, int j, int ng,
                                                    int cs) {
    return j < ng ? Zc + int64_t(j) * 128 : Z + int64_t(cs + (j - ng)) * stride;
}

// all of a launch's workgroups on the chip at once, or nearly: two per CU of four waves, one of eight
inline bool resident_tiles(int64_t wgs, int waves) { return wgs * waves <= 2048 + 512; }

// tiles of `waves` pieces in a segment of `rows` rows, and in all that is launched for a (batch, KV head)
inline int segment_tiles(const Dims& D, int64_t rows, int waves) { return int(((rows + 31) / 32 * D.G + waves - 1) / waves); }
inline int64_t tiles_per_unit(const Dims& D, int waves) {
    return (D.row_begin == 0 ? segment_tiles(D, D.S < D.n ? D.S : D.n, waves) : 0) + int64_t(D.fq1 - (D.row_begin == 0 ? 0 : D.fq0)) * segment_tiles(D, D.L, waves);
}

inline QTileMap make_qtile_map(const Dims& D, int waves) {
    QTileMap M;
    M.heads = D.G % 4 == 0 ? 4 : D.G;
    M.sink_tiles = segment_tiles(D, D.S < D.n ? D.S : D.n, waves);
    M.tpc = segment_tiles(D, D.L, waves);
    M.tiles = M.sink_tiles + D.nq * M.tpc;
    M.tix_lo = D.row_begin == 0 ? 0 : M.sink_tiles + D.fq0 * M.tpc;
    M.tix_hi = M.sink_tiles + D.fq1 * M.tpc;
    M.per_unit = M.tix_hi - M.tix_lo;
    const int64_t units = int64_t(D.B) * D.Hkv, wgs = units * M.per_unit;
    M.side_by_side = units % 8 != 0 || resident_tiles(wgs, waves);
    M.backwards = waves == 4;
    M.wgs = int(M.side_by_side && wgs < 512 ? (wgs + 255) / 256 * 256 : wgs);   // the second 256 are whole
    M.by_unit = make_fast_div(M.per_unit, wgs);
    M.by_units = make_fast_div(units, M.wgs);
    M.by_hkv = make_fast_div(D.Hkv, units);
    M.by_tpc = make_fast_div(M.tpc, M.tiles);
    M.by_heads = make_fast_div(M.heads, int64_t(M.tpc > M.sink_tiles ? M.tpc : M.sink_tiles) * waves + waves);
    return M;
}

// Waves per workgroup of the forward and dQ kernels.  Eight share one staged K / V tile; four, two workgroups of which fit a CU, copy it
// twice and take 2 to 5 percent longer where the chip is full and the walks are long (32K tokens, 32 heads on 8: forward 2718 us with
// eight, 2819 with four).  Four
//  - where the launch is resident at once or nearly: its longest workgroup is what counts, and it is half as long, runs alone on its
//    SIMDs or is paired with a short one (QTileMap).  Forward with eight and with four: 2.4K tokens, 8 heads on 2, lag 96: 27.8 and 22.9 us; 2
//    requests of 4K tokens, 8 heads on 8, lag 256: 47.1 and 42.2; 14.3K tokens, 4 heads on 4, lag 446, 111 kept: 117 and 104;
//  - where eight would leave more than one wave in ten idle at the ends of the chunks: 4 requests of 2.9K tokens, 12 heads on 4,
//    lag 91, 22 kept: 85.9 and 64.8 us;
//  - for walks of up to a thousand keys, whose beginning and end the other workgroup of the CU covers: 2.5K tokens, 64 heads on 8, lag 128:
//    68.2 and 62.4 us, but 4 requests of 3.4K tokens, 8 on 2, lag 117: 53.2 and 55.7 (28 such shapes without gaps: with eight 0.955 to 1.13 of the
//    time, 1.02 on average); from 1.3K keys on eight are faster again (7.4K tokens, 48 heads on 8: 269 and 274 us);
//  - head_dim 64, whose tiles are half as large: three workgroups share a CU, and the backward never gains from eight by more than 3 percent (0.97
//    to 1.24 of the time with four, 92 shapes); the forward in full launches: fwd_waves.
inline int qtile_waves(const Dims& D) {
    if (D.compact) return 8;
    if (D.d == 64) return 4;
    const int64_t units = int64_t(D.B) * D.Hkv, n4 = units * tiles_per_unit(D, 4), n8 = units * tiles_per_unit(D, 8);
    const int keys = gather_count(D, (D.fq0 + D.fq1) / 2) + D.L + D.L / 2;   // of a walk, about
    return resident_tiles(n4, 4) || 20 * n8 > 11 * n4 || keys <= 1000 ? 4 : 8;
}
// The forward at head_dim 64: eight where four would be three rounds of 768 workgroups and more, and eight leave not more than one wave in
// twenty idle.  Of 58 such shapes it takes 0.92 to 1.02 of the time with four, 0.97 on average (32K tokens, 32 heads on 8: 2950 and
// 2846 us; 2 requests of 7.2K tokens, 16 on 4: 293 and 277); with 1300 to 2000 workgroups 0.96 to 1.09, below that up to 1.43.
inline int fwd_waves(const Dims& D) {
    if (D.compact || D.d != 64) return qtile_waves(D);
    const int64_t units = int64_t(D.B) * D.Hkv, n4 = units * tiles_per_unit(D, 4), n8 = units * tiles_per_unit(D, 8);
    return n4 >= 2048 && 40 * n8 <= 21 * n4 ? 8 : 4;
}

}  // namespace lrsa
