// Building blocks of the bf16 MFMA attention kernels (gfx950, head_dim 128).
//
// Matrix-core instruction used throughout: v_mfma_f32_32x32x16_bf16, D(32x32) += A(32x16) B(16x32).
//   A: lane l holds row l%32,    k = 8*(l/32) + [0,8)      (8 bf16, 4 VGPRs)
//   B: lane l holds column l%32, k = 8*(l/32) + [0,8)
//   D: lane l holds column l%32, rows 8*(r/4) + 4*(l/32) + r%4 for r in [0,16)
// Every product here is arranged so that the index kept per lane (a query, or a key) is the D
// column and the contracted index of the NEXT product is the D row; the fp32 tile then turns
// into the next product's 16-bit operand inside the lane, with no LDS round trip.  The D-row
// order is a permutation of the contracted index; the other operand is fetched from LDS in the
// same permuted order (see k_slot_row below), which a sum does not mind.
#pragma once

#include <type_traits>
#include <utility>

#include "cart_common.h"

namespace cart {
namespace mfma {

// compile-time loop: f(std::integral_constant<int, 0>{}), ..., f(std::integral_constant<int, N-1>{})
template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}

// Masking without compares: entry r of a score block (D row 8 (r/4) + r%4 + 4 g, g folded into
// thr by the caller) is hidden when its row exceeds thr (mask_above) or lies below it
// (mask_below).  bound_r = (thr - row + 1/2) * 1e30 is far above every score where the entry is
// visible and far below where it is hidden, so x = min(x, bound_r) does the job in two plain
// vector instructions per entry, with no condition registers between them (the compare / select
// form goes through scalar registers and costs several times more).  A hidden entry ends up at
// -5e29 or below: its exponential is an exact 0.
__device__ __forceinline__ float vmin_raw(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
template <typename V16>
__device__ __forceinline__ void mask_above(V16& x, int thr) {
    const int t = min(max(thr, -64), 64);
    const float tf = fmaf(static_cast<float>(t), 1.0e30f, 0.5e30f);
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = vmin_raw(x[r], tf - static_cast<float>(8 * (r >> 2) + (r & 3)) * 1.0e30f);
}
template <typename V16>
__device__ __forceinline__ void mask_below(V16& x, int thr) {
    const int t = min(max(thr, -64), 64);
    const float tf = fmaf(static_cast<float>(-t), 1.0e30f, 0.5e30f);
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = vmin_raw(x[r], tf + static_cast<float>(8 * (r >> 2) + (r & 3)) * 1.0e30f);
}

// Rows of sequence b, and where the per-row statistics (lse, delta) of its heads live: the value
// of token i of head h is at stat_b + h * stat_h + i.
//   batched layout (cu == nullptr): rows b*S .. b*S+S-1 of [B,S,...]; statistics [B,Hq,S]
//   packed layout: rows cu[b] .. cu[b+1]-1 of [T,...];                statistics [Hq,T]
struct SeqSpan { size_t t0; size_t stat_b; size_t stat_h; int len; };
__device__ __forceinline__ SeqSpan seq_span(const int32_t* cu, int b, int T, int S, int Hq) {
    SeqSpan sp;
    if (cu) {
        const int c0 = cu[b];
        sp.t0 = static_cast<size_t>(c0);
        sp.len = cu[b + 1] - c0;
        sp.stat_b = sp.t0;
        sp.stat_h = static_cast<size_t>(T);
    } else {
        sp.t0 = static_cast<size_t>(b) * S;
        sp.len = S;
        sp.stat_b = static_cast<size_t>(b) * Hq * S;
        sp.stat_h = static_cast<size_t>(S);
    }
    return sp;
}

// Query-stationary workgroups (forward, dQ): 256 query rows = four units of (64 consecutive tokens,
// one query head), one per wavefront.  The units of a (sequence, KV head) are numbered with the
// group's G heads fastest, and a workgroup takes four in a row: with G = 4 its wavefronts hold the
// four heads of the same 64 tokens, so they all end on the same diagonal tile -- one masked tile per
// workgroup instead of the four (and up to three key tiles a wavefront only waited through) of 256
// consecutive tokens of one head -- and a sequence is rounded up to 64 tokens, not to 256.  The
// wavefronts past the last unit load clamped rows and store nothing.  Against 256 consecutive
// tokens of one head (us): Hq 24 / Hkv 8, S 1024, P 2048, B 32: forward 950 -> 918, dQ 1343 -> 1303;
// 32 / 8, S 2048, P 4096, B 16: forward 2180 both, dQ 3165 -> 3090; 64 packed conversations of 64 ..
// 1024 tokens, P 4096 (a block of 64 tokens spans fewer sequences): forward 2352 -> 2234, dQ 3358 -> 3191.
struct QueryBlock {
    int hk, b, h;       // KV head, sequence, the wavefront's query head
    int q0, q_end;      // tokens of the workgroup
    int wrow0;          // first token of the wavefront
    int part, n_parts;  // which part of the block's key tiles, of how many
    int slot;           // where the part's partial result goes (n_parts > 1)
};
__host__ __device__ inline int query_wgs(int S, int G) { return (((S + 63) / 64) * G + 3) / 4; }

// One workgroup fills a CU, so a launch runs in rounds of one block per CU, and what is left over
// after the whole rounds -- everything, for a small problem -- leaves CUs idle for a block's whole
// length.  Those last blocks may be split along their key tiles into parts of about equal length;
// each part leaves a partial result (128 KB) and the finishing kernel of the call combines them.  All blocks of one KV head are numbered b * nW + (nW-1-w) (heaviest first
// within a sequence); the first e_full of them run whole, the parts of the others are listed (a
// search over the blocks in the kernels took longer than the parts' own set-up).
constexpr int MAX_SPLIT = 256;          // parts per KV head, at most one per CU
struct QuerySplit {
    int e_full;                         // blocks per KV head that run whole
    int n_blocks, n_parts;              // split blocks and their parts, per KV head
    uint32_t part[MAX_SPLIT];           // part i: block (from e_full) | part of the block << 8 | parts of the block << 16
    uint32_t first[MAX_SPLIT];          // split block -> its first part
};
// KV head fastest: with 8 of them blockIdx % 8 (the XCD) is the KV head and each XCD's L2 keeps one
// head's prefix; then the blocks of one sequence, heaviest (longest causal part) first, sequence
// after sequence, so that the workgroups running at one time share one or two sequences' K/V in L2.
__device__ __forceinline__ QueryBlock query_block_of(int hk, int e, int wv, int nW, int G) {
    QueryBlock qb;
    const int u0 = 4 * (nW - 1 - e % nW), u = u0 + wv;
    qb.hk = hk;
    qb.b = e / nW;
    qb.h = hk * G + u % G;
    qb.wrow0 = 64 * (u / G);
    qb.q0 = 64 * (u0 / G);
    qb.q_end = 64 * ((u0 + 3) / G) + 64;
    qb.part = 0;
    qb.n_parts = 1;
    qb.slot = 0;
    return qb;
}
__device__ __forceinline__ QueryBlock query_block(int id, int wv, int Smax, int Hq, int Hkv, const QuerySplit& sp) {
    const int G = Hq / Hkv, hk = id % Hkv, x = id / Hkv;
    const uint32_t it = x < sp.e_full ? 0x10000u : sp.part[x - sp.e_full];
    QueryBlock qb = query_block_of(hk, x < sp.e_full ? x : sp.e_full + (it & 255), wv, query_wgs(Smax, G), G);
    qb.part = (it >> 8) & 255;
    qb.n_parts = it >> 16;
    qb.slot = (x - sp.e_full) * Hkv + hk;
    return qb;
}
// Key tiles of a query block, in the order the kernels take them: the tiles every query of the block
// sees entirely (whole prefix tiles, then own tiles tU0 .. tD-1), then the ones that need a mask (the
// ragged last prefix tile, own tiles tA .. that start before the first key of some query, the own
// tiles from tD on the diagonal).  [lo, hi): the tiles of this part.  A part other than the first
// starts at a tile of the first kind, so that every query has a visible key in it.
struct KeyTiles {
    int nPf, rag, tA, tU0, tD, nLow, nMain, nT, lo, hi;
    __device__ __forceinline__ bool pre(int t) const { return t < nPf || (rag && t == nMain); }
    __device__ __forceinline__ int j0(int t) const {
        const int m = t - nMain - rag;      // among the masked own tiles
        return (t < nPf ? t : t < nMain ? tU0 + t - nPf : (rag && t == nMain) ? nPf : m < nLow ? tA + m : tD + m - nLow) * 64;
    }
};
__device__ __forceinline__ KeyTiles key_tiles(const QueryBlock& qb, int S, int P, const int32_t* row_lo) {
    KeyTiles k;
    const int own_end = min(S, qb.q_end);
    k.nPf = P / 64;
    k.rag = (P % 64) ? 1 : 0;
    const int lo_first = row_lo ? row_lo[qb.q0] : 0, lo_last = row_lo ? row_lo[own_end - 1] : 0;
    k.tA = lo_first / 64;
    k.tU0 = (lo_last + 63) / 64;
    k.tD = qb.q0 / 64;
    const int nOf = max(0, k.tD - k.tU0);
    k.nLow = min(k.tU0, k.tD) - k.tA;
    k.nMain = k.nPf + nOf;
    k.nT = k.nMain + k.rag + k.nLow + (own_end + 63) / 64 - k.tD;
    k.lo = 0;
    k.hi = k.nT;
    if (qb.n_parts == 1) return k;
    const int step = (k.nT + qb.n_parts - 1) / qb.n_parts, last = max(k.nMain - 1, 0);
    k.lo = qb.part == 0 ? 0 : min(qb.part * step, last);
    k.hi = qb.part == qb.n_parts - 1 ? k.nT : min((qb.part + 1) * step, last);
    return k;
}
// (host) Playing a launch through: free_at[0, n) is a heap of the times at which n CUs are free; the next
// workgroup, t long, goes to the one that is free first.  Returns when it ends.  (Looking through all
// the CUs for each workgroup made planning the host's largest item: 32 sequences of 516 tokens, 2 KV
// heads, 152 slots: a forward and backward call 1114 us, 295 of them on the GPU.)
inline float run_next(float* free_at, int n, float t) {
    const float end = free_at[0] + t;
    int m = 0;
    for (int c = 1; c < n; c = 2 * m + 1) {
        if (c + 1 < n && free_at[c + 1] < free_at[c]) ++c;
        if (free_at[c] >= end) break;
        free_at[m] = free_at[c];
        m = c;
    }
    free_at[m] = end;
    return end;
}
// (host) the split of a query-stationary launch: B sequences of at most S tokens; packed rows: own_cap, the most
// own-key tiles of a block (bounded by the longest sequence; 0: batched layout), and whether sequences meet inside blocks.
// us: a block's set-up and store, each key tile, and what a split adds: to the call, for each part of a block
// (the sums run over them in turn), for each workgroup.
enum QueryKernel { QUERY_FWD, QUERY_DQ };
struct SplitCost { float block, tile, fix, part, wg; };
constexpr SplitCost SPLIT_COST[2] = {{9.2f, 1.21f, 3.5f, 0.7f, 0.045f}, {11.f, 1.95f, 4.f, 0.f, 0.05f}};
void plan_query_split(QuerySplit& sp, int B, int S, int G, int Hkv, int P, int own_cap, bool meet, const SplitCost& us);
// The cut of the key-stationary launch: token rows per dZ partial, the partials, and into how many parts the
// query heads that read an own key are split
struct KvPlan { int chunk, n_part, head_parts; };
// partial results of one part: 256 rows x 128 fp32, then (forward) 256 fp32 LSEs
constexpr size_t PART_O_BYTES = 256 * 128 * sizeof(float), PART_L_BYTES = 256 * sizeof(float);

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int HD = 128;           // head_dim
constexpr int ROW_B = HD * 2;     // bytes per key/value/query row, in global memory and in LDS
constexpr float NEG_BIG = -1.0e30f;
constexpr float RESCALE_GAP = 8.0f;   // running max is moved only when exceeded by 2^8

__device__ __forceinline__ f32x16 mma(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// The same product with the result in ordinary vector registers (the compiler's own choice for
// the builtin is an accumulation register whenever a kernel uses those at all) and the B operand
// read from an accumulation register.  The compiler does not know these are matrix-core
// instructions: a consumer on the vector ALU must be at least 20 wait states away.
// Where that distance comes from, kernel by kernel (a product occupies the matrix cores for 32
// cycles, so one product issued in between already covers it; every place states its own margin):
//   forward        S(u+1) written in groups 0-15 of an iteration, first read by the vector ALU
//                  in group 0 of the next one: the 16 O products of groups 16-31 lie between.
//   dQ             block 1's S / dP written up to groups 44 / 45, first read in group 0 of the
//                  next iteration: 3 products between (groups 46, 47, 0); block 0's written up to
//                  groups 46 / 47, first read in group 16: 17 products between.  The masked path
//                  reads them at the top of the iteration and waits 24 states first.
//   dK + dV, A     S(u+1) written in groups 0-15, first read in group 0 of the next iteration:
//                  the 16 dV products between.
//   dK + dV, B     dP(u) written in groups 0-15, first read in group 4 of the next iteration: the
//                  16 dK products and 4 more between.
//   prologues      every first score product is followed by s_nop 15; s_nop 7 (24 states).
// The GPU tests hold the tripwires: the forward and the backward run twice bit-equal, and the
// matrix-core kernels against the vector kernels and the oracle over a sweep of random shapes.
__device__ __forceinline__ void mma_vd_zero(f32x16& d, bf16x8 a, const u32x4& b) {
    asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "a"(b));
}
// d = a b + init (init in its own registers, left unchanged)
__device__ __forceinline__ void mma_vd_first(f32x16& d, bf16x8 a, const u32x4& b, const f32x16& init) {
    asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(a), "a"(b), "v"(init));
}
__device__ __forceinline__ void mma_vd(f32x16& d, bf16x8 a, const u32x4& b) {
    asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b));
}

// LDS tiles are [rows][128] bf16, 256 bytes per row, unpadded; the 16-byte chunk c of row r is
// stored at chunk position c ^ swz(r).  swz is a bijection of r % 16 (16 consecutive rows read
// at one logical chunk hit 16 distinct positions: row-wise ds_read_b128 is conflict-free) whose
// bits 2..3 are r % 4 (4 consecutive rows x 4 consecutive chunks cover all 16 positions: the
// transposing read is conflict-free too).
__device__ __forceinline__ int swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

// row-wise operand fragment: the 8 bf16 at columns [col, col+8) of one row (col % 8 == 0)
__device__ __forceinline__ bf16x8 lds_frag_n(const char* tile, int row, int col) {
    return *reinterpret_cast<const bf16x8*>(tile + row * ROW_B + (((col >> 3) ^ swz(row)) << 4));
}

// Transposed operand fragment for one 16-deep k-step of a [k][n] row-major tile: the lane that
// owns operand row/column n gets the 8 k-values whose k-slots match the D-row order above:
// slots e = 0..3 -> k = k0 + 4g + e, slots 4..7 -> k = k0 + 8 + 4g + (e-4), g = lane/32.
// ds_read_b64_tr_b16: within each block of 16 lanes, lane i receives, for e = 0..3, element i%4 of
// the 8 bytes addressed by lane 4e + i/4; so lane s of a block addresses row k + s/4, columns
// n0 + 4*(s%4) .. +3, and lane i ends up with column n0 + i of rows k .. k+3.
__device__ __forceinline__ bf16x8 lds_frag_t(const char* tile, int k0, int n0, int lane) {
    const int blk = lane >> 4, s = lane & 15, g = lane >> 5;
    const int row = k0 + 4 * g + (s >> 2);
    const int col = n0 + 16 * (blk & 1) + 4 * (s & 3);
    const int half = ((col >> 2) & 1) * 8;
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_ptr)(tile + row * ROW_B + (((col >> 3) ^ swz(row)) << 4) + half));
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_ptr)(tile + (row + 8) * ROW_B + (((col >> 3) ^ swz(row + 8)) << 4) + half));
    s16x8 r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, r);
}

// The same two fragment kinds from precomputed 32-bit LDS byte addresses (per-lane part computed
// once, compile-time offsets added at the use): frag_n_ofs / frag_t_ofs give the per-lane offset
// of a fragment inside a tile whose first row is a multiple of 16.
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint32_t frag_n_ofs(int lane, int t8) {
    const int lc = lane & 31, lg = lane >> 5;
    return lc * ROW_B + (((2 * t8 + lg) ^ swz(lc)) << 4);
}
__device__ __forceinline__ void frag_t_ofs(int lane, int db, uint32_t& lo, uint32_t& hi) {
    const int s = lane & 15, g = lane >> 5;
    const int row = 4 * g + (s >> 2);
    const int col = 32 * db + 16 * ((lane >> 4) & 1) + 4 * (s & 3);
    const int half = ((col >> 2) & 1) * 8;
    lo = row * ROW_B + (((col >> 3) ^ swz(row)) << 4) + half;
    hi = (row + 8) * ROW_B + (((col >> 3) ^ swz(row + 8)) << 4) + half;
}
__device__ __forceinline__ bf16x8 lds_ld_frag(uint32_t addr) {
    return *(const bf16x8 __attribute__((address_space(3)))*)addr;
}
__device__ __forceinline__ f32x4 lds_ld_f32x4(uint32_t addr) {
    return *(const f32x4 __attribute__((address_space(3)))*)addr;
}
__device__ __forceinline__ bf16x8 lds_ld_frag_t(uint32_t lo, uint32_t hi) {
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)lo);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)hi);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// D row held in register r of lane-group g (the k index the next product contracts over)
__device__ __forceinline__ int d_row(int r, int g) { return 8 * (r >> 2) + 4 * g + (r & 3); }

// value held by the lane 32 away
__device__ __forceinline__ float partner(float x) {
    uint32_t u = __float_as_uint(x);
    auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}
__device__ __forceinline__ float partner_max(float x) {
    uint32_t u = __float_as_uint(x);
    auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// 8 fp32 D registers [r0, r0+8) -> one 16-bit operand fragment (same lane, same column)
__device__ __forceinline__ bf16x8 pack_frag(const f32x16& s, int r0) {
    u32x4 w = {pack_bf16x2(s[r0 + 0], s[r0 + 1]), pack_bf16x2(s[r0 + 2], s[r0 + 3]),
               pack_bf16x2(s[r0 + 4], s[r0 + 5]), pack_bf16x2(s[r0 + 6], s[r0 + 7])};
    return __builtin_bit_cast(bf16x8, w);
}

// ---- storing a wavefront's transposed accumulators ---------------------------------------------
// acc[db][cb] holds, for row 32 cb + lane % 32 of the wavefront's 64, columns 32 db + 8 (r/4) +
// 4 (lane/32) + r%4.  Stored from the registers, an instruction touches 32 rows with 16 or 32 bytes
// each, and the 32 to 64 of them take 4-5 us of a workgroup's life; turned around in LDS (the
// wavefront's own 16 or 32 KB, free once the key or query tiles are done with) every store
// instruction writes whole rows.  The 16-byte chunks are swizzled by row so that neither side has
// bank conflicts: a forward block of 256 rows 4.7 -> 3.4 us from its last product to its end (16 sequences
// of 256 tokens, 32 heads, 1024 slots: 88.8 -> 85.7 us a forward call).  Eight reads are requested before
// their stores: with each store's row predicate around its own read the reads went one round trip after the other
// (the same call 82.3 -> 81.5 us, backward 268 -> 267; 256 sequences of 64 tokens, 16 / 16 heads 154 -> 148).
// Rows from n_rows on are not stored; consecutive rows are `pitch` elements apart.
// Returns, per block of 32 rows, the sum of the lane's scaled values (not finite when one is not).
struct RowSums { float s[2]; };
__device__ __forceinline__ RowSums store_rows64(char* lds, const f32x16 (&acc)[4][2], float mul0, float mul1,
                                                   bf16_t* __restrict__ out, size_t pitch, int n_rows, int lane) {
    const int lg = lane >> 5, lc = lane & 31;
    RowSums rs = {};
    if (n_rows <= 0) return rs;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
        const float mul = cb ? mul1 : mul0;
        float sum = 0.f;
        char* row = lds + (32 * cb + lc) * ROW_B + ((lg ^ (lc >> 4)) << 3);
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const float v0 = acc[db][cb][4 * r4] * mul, v1 = acc[db][cb][4 * r4 + 1] * mul,
                            v2 = acc[db][cb][4 * r4 + 2] * mul, v3 = acc[db][cb][4 * r4 + 3] * mul;
                sum += (v0 + v1) + (v2 + v3);
                const u32x2 w = {pack_bf16x2(v0, v1), pack_bf16x2(v2, v3)};
                *reinterpret_cast<u32x2*>(row + (((4 * db + r4) ^ (lc & 15)) << 4)) = w;
            }
        rs.s[cb] = sum;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const int rl = lane >> 4, ch = lane & 15;
#pragma unroll
    for (int i0 = 0; i0 < 16; i0 += 8) {
        u32x4 w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = 4 * (i0 + i) + rl;
            w[i] = *reinterpret_cast<const u32x4*>(lds + r * ROW_B + ((ch ^ (r & 15)) << 4));
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(w[i]));
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = 4 * (i0 + i) + rl;
            if (i & 4) w[i] = u32x4{w[i].z, w[i].w, w[i].x, w[i].y};       // (rows 16-31 of a block: halves stored the other way round)
            if (r < n_rows) *reinterpret_cast<u32x4*>(out + r * pitch + 8 * ch) = w[i];
        }
    }
    return rs;
}
__device__ __forceinline__ RowSums store_rows64(char* lds, const f32x16 (&acc)[4][2], float mul0, float mul1,
                                                float* __restrict__ out, size_t pitch, int n_rows, int lane) {
    const int lg = lane >> 5, lc = lane & 31;
    RowSums rs = {};
    if (n_rows <= 0) return rs;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
        const float mul = cb ? mul1 : mul0;
        float sum = 0.f;
        char* row = lds + (32 * cb + lc) * 2 * ROW_B;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const f32x4 w = {acc[db][cb][4 * r4] * mul, acc[db][cb][4 * r4 + 1] * mul, acc[db][cb][4 * r4 + 2] * mul,
                                 acc[db][cb][4 * r4 + 3] * mul};
                sum += (w[0] + w[1]) + (w[2] + w[3]);
                *reinterpret_cast<f32x4*>(row + (((8 * db + 2 * r4 + lg) ^ lc) << 4)) = w;
            }
        rs.s[cb] = sum;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const int rl = lane >> 5, ch = lane & 31;
#pragma unroll
    for (int i0 = 0; i0 < 32; i0 += 8) {
        f32x4 w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = 2 * (i0 + i) + rl;
            w[i] = *reinterpret_cast<const f32x4*>(lds + r * 2 * ROW_B + ((ch ^ (r & 31)) << 4));
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(w[i]));
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = 2 * (i0 + i) + rl;
            if (r < n_rows) *reinterpret_cast<f32x4*>(out + r * pitch + 4 * ch) = w[i];
        }
    }
    return rs;
}

// The same rows straight from the registers (bf16), for a workgroup with few of them
__device__ __forceinline__ RowSums store_rows64_direct(const f32x16 (&acc)[4][2], float mul0, float mul1, bf16_t* __restrict__ out,
                                                       size_t pitch, int n_rows, int lane) {
    const int lg = lane >> 5, lc = lane & 31;
    RowSums rs = {};
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
        if (32 * cb + lc >= n_rows) continue;
        const float mul = cb ? mul1 : mul0;
        bf16_t* const row = out + (32 * cb + lc) * pitch + 4 * lg;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const float v0 = acc[db][cb][4 * r4] * mul, v1 = acc[db][cb][4 * r4 + 1] * mul,
                            v2 = acc[db][cb][4 * r4 + 2] * mul, v3 = acc[db][cb][4 * r4 + 3] * mul;
                rs.s[cb] += (v0 + v1) + (v2 + v3);
                *reinterpret_cast<u32x2*>(row + 32 * db + 8 * r4) = u32x2{pack_bf16x2(v0, v1), pack_bf16x2(v2, v3)};
            }
    }
    return rs;
}

// ---- direct-to-LDS loads --------------------------------------------------------------------
// The loads are written as inline assembly so that the wait for them sits where the pipeline
// wants it (one s_waitcnt vmcnt(0) in front of the barrier that publishes the tile, a whole
// iteration after the loads went out) and not in front of the next LDS read of any address.
// M0 carries the wave-uniform LDS byte address; lane i's 16 (4) bytes land at M0 + 16 i (4 i).
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)p));
}
// base: wave-uniform global address; voff: per-lane unsigned byte offset from it
__device__ __forceinline__ void dma16(const char* base, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(base), "s"(lds) : "memory", "m0");
}
// (of rows that are read once: not kept in the caches)
__device__ __forceinline__ void dma16_nt(const char* base, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                 :: "v"(voff), "s"(base), "s"(lds) : "memory", "m0");
}
__device__ __forceinline__ void dma4(const char* base, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
                 :: "v"(voff), "s"(base), "s"(lds) : "memory", "m0");
}
// every direct-to-LDS load of this wavefront has landed
__device__ __forceinline__ void dma_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// all but the wavefront's N most recent direct-to-LDS loads have landed
template <int N>
__device__ __forceinline__ void dma_wait_but() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

// Tile of ROWS rows x 256 bytes -> LDS (row r at 256 r, 16-byte chunks swizzled), cooperatively
// by the 4 wavefronts of a 256-thread workgroup.  One load instruction moves 64 chunks = 4 tile
// rows; lane i's chunk lands at (wave-uniform base) + 16 i, so the lane fetches the logical
// chunk that belongs at that position under the swizzle.  Tile row r comes from tensor row
// min(j0 + r, last) of a slice that starts at `base` with `pitch` bytes between rows (base, j0,
// last, pitch wave-uniform; j0 <= last; rows past `last` repeat it and are masked by the
// caller, so their contents never reach a result; 64 * pitch < 2^32).
template <int ROWS>
__device__ __forceinline__ void tile_load_async(char* tile, const char* base, int j0, int last, uint32_t pitch) {
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int PER_WAVE = ROWS / 16;      // instructions per wavefront
    const char* tb = base + static_cast<size_t>(j0) * pitch;
    const int lim = last - j0;
    const uint32_t lds0 = lds_addr(tile);
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
        const int r0 = (PER_WAVE * wv + i) * 4;
        const int r = r0 + (lane >> 4);
        const uint32_t voff = static_cast<uint32_t>(min(r, lim)) * pitch + (((lane & 15) ^ swz(r)) << 4);
        dma16(tb, voff, lds0 + r0 * ROW_B);
    }
}

}  // namespace mfma

// ---- what the two backward files and the forward's planner share (host) ----
// the split of the query blocks, the most parts it can take (attn_mfma_fwd.hip)
void attn_query_split(mfma::QuerySplit& sp, const cart_attn_desc& d, int T, mfma::QueryKernel kind);
size_t attn_query_parts(const cart_attn_desc& d, int T);
// every block in `parts` parts (1: whole); false: more than `most` of them
bool attn_query_split_all(mfma::QuerySplit& sp, const cart_attn_desc& d, int T, int parts, int most);
// key tiles of each workgroup of a KV head in the split launch's order; how many, -1: more than `most`
int attn_query_tiles(const cart_attn_desc& d, int T, const mfma::QuerySplit& sp, int* tiles, int most);
// the fused dK + dV kernel, its cut, the most bytes its partials can take; dQ beside it in one launch (attn_mfma_bwd_kv.hip)
struct KvArgs {
    const bf16_t *q, *k, *v, *zk, *zv, *d_o;
    const float *nlse2, *ndelta;
    bf16_t *dk_own, *dv_own;
    float *part_k, *part_v;             // dZ partials, one per chunk of token rows; or dZ itself (one chunk)
    float *own_k, *own_v;               // partials of own keys, one per part of the heads (head_parts > 1)
    const int32_t* cu;
    int n_tok, chunk, head_parts, Smax, Hq, Hkv, P;
    int own_cols;                       // own-key blocks: 0: a (sequence, part of the heads)'s one after the other; else the first of all own_cols of these, then the second ..
    float c, scale;
    int n_frozen;                       // prefix rows stored as zeros (only where dZ itself is stored)
};
struct DqArgs;
// one_launch: dQ beside dK and dV, behind the first kv_front blocks of the key side (per KV head)
struct BwdPlan { mfma::KvPlan kv; mfma::QuerySplit split; bool one_launch; int kv_front; };
const BwdPlan& plan_bwd(const cart_attn_desc& d, int T);
size_t bwd_kv_most(const cart_attn_desc& d, long tokens);
unsigned bwd_kv_grid(const cart_attn_desc& d, const mfma::KvPlan& plan);
void launch_attn_bwd_kv(const KvArgs& a, unsigned grid, hipStream_t st);
void launch_attn_bwd_stats(const bf16_t* o, const bf16_t* d_o, const float* lse, float* nlse2, float* ndelta, int n_tok, int S, int Hq,
                           hipStream_t st);
void launch_attn_bwd_both(const KvArgs& ka, const DqArgs& qa, const mfma::QuerySplit& sp, unsigned kv_grid, int kv_front, hipStream_t st);
}  // namespace cart
