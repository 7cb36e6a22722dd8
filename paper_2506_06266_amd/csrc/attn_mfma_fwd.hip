// Cartridge attention forward on the matrix cores (bf16 in, fp32 accumulate, head_dim 128):
// Eq. 1 over the cache of Sec. 3.2, [prefix Z (all visible) ; own keys (causal)].
//
// One 256-thread workgroup = 256 query rows of one (sequence, KV head): each of its four wavefronts
// owns 64 consecutive tokens of one query head (see QueryBlock), kept in registers as MFMA operand
// fragments.  Keys/values
// stream through LDS in tiles of 64 (prefix tiles first, then own tiles up to the diagonal),
// four buffers, one barrier per tile, consumed as sub-tiles of 32 keys.  Per sub-tile a
// wavefront computes S^T = K Q^T (keys on the D rows, its queries on the D columns), turns it
// into P = 2^(c S - m) per lane (a lane owns one query) and accumulates O^T += V^T P^T with V
// read through the transposing LDS load.
//
// The softmax reference m of a query is fixed once, from its first sub-tile of keys; there is no
// running max and the O accumulators are never rescaled.  exp2 and the fp32 accumulators cover
// 2^+-126 around that reference, so this is exact unless a later score exceeds the first
// sub-tile's maximum by more than ~80 in natural-log units; then the row sum overflows to
// inf/NaN, and those 64 rows are computed again with a plain running-max loop, by the wavefront itself
// or, in a split block, by attn_fwd_finish_kernel.  The hot loop is one straight-line block per sub-tile with two
// independent instruction streams: the matrix cores work on S(u+1) and on O += V P(u-1) while the
// vector ALU turns S(u) into P(u).
#include <type_traits>

#include "attn_mfma.h"

namespace cart {
using namespace mfma;

constexpr int FWD_BN = 64;    // keys per LDS tile, consumed as two sub-tiles of 32
constexpr int FWD_NBUF = 4;     // tile t in buffer t % 4; loads run two tiles ahead of the barrier that publishes them
constexpr int FWD_TILE_B = FWD_BN * ROW_B;

struct FwdSmem {
    char k[FWD_NBUF][FWD_TILE_B];
    char v[FWD_NBUF][FWD_TILE_B];
};

// 1: fold the softmax scale into Q (one extra bf16 rounding of Q) and the softmax reference into
// the score product's init value, so that an exponent costs no arithmetic of its own.  0: scores
// are scaled in fp32, exponent = fma(score, c, -m): exact, one more vector-ALU instruction per
// element.
#ifndef CART_PRESCALE
#define CART_PRESCALE 0
#endif

// Rows i0 .. i1-1 (tokens of the sequence at t0) of query head h again, with a running-max loop on the
// vector ALU: what a block does whose fixed softmax reference overflowed.  Lane l owns head elements
// 2l, 2l+1, eight keys at a time (a CU holds one of the blocks that come here, with nothing else to hide a
// round trip per key); lse_h: the sequence's LSE values of head h.
__device__ __forceinline__ void recompute_rows(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
    const bf16_t* __restrict__ zk, const bf16_t* __restrict__ zv, bf16_t* __restrict__ o, float* __restrict__ lse_h,
    const int32_t* __restrict__ row_lo, size_t t0, int i0, int i1, int h, int hk, int Hq, int Hkv, int P, float c, int lane) {
    constexpr int U = 8;
    for (int i = i0; i < i1; ++i) {
        const size_t row = (t0 + i) * Hq + h;
        const uint32_t qw = *reinterpret_cast<const uint32_t*>(q + row * HD + 2 * lane);
        const float q0 = __uint_as_float(qw << 16), q1 = __uint_as_float(qw & 0xffff0000u);
        float m = -3.0e38f, l = 0.f, a0 = 0.f, a1 = 0.f;
        const int own0 = row_lo ? row_lo[i] : 0;      // first own key of the row
        const int n = P + (i - own0) + 1;
        for (int j0 = 0; j0 < n; j0 += U) {
            float sc[U], nm = m;
            uint32_t vw[U];
#pragma unroll
            for (int x = 0; x < U; ++x) {
                const int j = min(j0 + x, n - 1);
                const size_t kr = j < P ? static_cast<size_t>(hk) * P + j : (t0 + own0 + (j - P)) * Hkv + hk;
                const uint32_t kw = *reinterpret_cast<const uint32_t*>((j < P ? zk : k) + kr * HD + 2 * lane);
                vw[x] = *reinterpret_cast<const uint32_t*>((j < P ? zv : v) + kr * HD + 2 * lane);
                sc[x] = q0 * __uint_as_float(kw << 16) + q1 * __uint_as_float(kw & 0xffff0000u);
            }
#pragma unroll
            for (int x = 0; x < U; ++x) {
                sc[x] = wave_sum(sc[x]) * c;
                nm = fmaxf(nm, sc[x]);
            }
            const float corr = fast_exp2(m - nm);
            l *= corr;
            a0 *= corr;
            a1 *= corr;
            m = nm;
#pragma unroll
            for (int x = 0; x < U; ++x) {
                const float pj = j0 + x < n ? fast_exp2(sc[x] - m) : 0.f;
                l += pj;
                if (j0 + x < n) {
                    a0 += pj * __uint_as_float(vw[x] << 16);
                    a1 += pj * __uint_as_float(vw[x] & 0xffff0000u);
                }
            }
        }
        const float inv = 1.f / l;
        *reinterpret_cast<uint32_t*>(o + row * HD + 2 * lane) = pack_bf16x2(a0 * inv, a1 * inv);
        if (lane == 0) lse_h[i] = (m + fast_log2(l)) * CART_LN2;
    }
}

// FEW: launches whose blocks have rows for two wavefronts at most and run whole (see launch_attn_fwd_mfma).
// Two wavefronts' stores straight from the registers end sooner than their way through LDS.
template <bool FEW>
__global__ __launch_bounds__(256, 1) void attn_fwd_mfma_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
    const bf16_t* __restrict__ zk, const bf16_t* __restrict__ zv, bf16_t* __restrict__ o,
    float* __restrict__ lse, int* __restrict__ flags, const int32_t* __restrict__ cu,
    const int32_t* __restrict__ row_lo, int n_tok, int Smax, int Hq, int Hkv, int P,
    float c /* scale*log2(e) */, QuerySplit split, float* __restrict__ part_o, float* __restrict__ part_l) {
    __shared__ FwdSmem sm;
    const int lane = threadIdx.x & 63, lg = lane >> 5, lc = lane & 31;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform, in a scalar register
    const QueryBlock qb = FEW ? query_block_of(blockIdx.x % Hkv, blockIdx.x / Hkv, wv, 1, Hq / Hkv)
                              : query_block(blockIdx.x, wv, Smax, Hq, Hkv, split);
    const int hk = qb.hk, b = qb.b, h = qb.h, q0 = qb.q0, wrow0 = qb.wrow0;
    // Rows of sequence b: [t0, t0 + S).  Batched layout: S rows each; packed layout (cu given):
    // rows cu[b] .. cu[b+1]-1 of T, the grid is sized for the longest sequence and a workgroup
    // whose tokens lie past the end of its sequence has nothing to do.
    // Packed layout with a prefix (row_lo given, B = 1, S = all packed rows): query tiles are cut
    // from the packed rows regardless of sequence boundaries -- no sequence ends in a partly
    // filled tile -- and row i sees the own keys row_lo[i] .. i (row_lo = first row of its sequence).
    const SeqSpan sp = seq_span(cu, b, n_tok, Smax, Hq);
    const int S = sp.len;
    const size_t t0 = sp.t0;
    // (a part's overflow flag per wavefront; blocks that run whole have none)
    int* const my_flag = flags + 4 * qb.slot + wv;
    if (q0 >= S) {
        if (lane == 0 && qb.n_parts > 1) *my_flag = 0;
        return;
    }
    const KeyTiles kt = key_tiles(qb, S, P, row_lo);
    float* const my_l = part_l + static_cast<size_t>(qb.slot) * 256 + 64 * wv;
    if (kt.lo >= kt.hi) {      // (fewer tiles than the launch assumed: this part is empty)
        if (lane == 0) *my_flag = 0;
        my_l[lane] = __uint_as_float(0xff800000u);
        return;
    }
    // this wavefront's 64 queries as B-operand fragments: column = query, k = head element
    // They are pinned to accumulation registers (the matrix cores read B operands from there
    // directly), which leaves the ordinary vector registers to the softmax arithmetic.
    u32x4 qraw[2][8];
    int lo_q[2] = {0, 0};     // first own key the lane's queries see
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
        int qi = wrow0 + 32 * cb + lc;
        qi = qi < S ? qi : S - 1;
        if (row_lo) lo_q[cb] = row_lo[qi];
        const bf16_t* qp = q + ((t0 + qi) * Hq + h) * HD + 8 * lg;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const u32x4 w = *reinterpret_cast<const u32x4*>(qp + 16 * t);
#if CART_PRESCALE
            // Q enters every product scaled by c = softmax_scale * log2(e), rounded to bf16 once
            // here: the scores then come out of the matrix cores in log2 units
#pragma unroll
            for (int i = 0; i < 4; ++i)
                qraw[cb][t][i] = pack_bf16x2(__uint_as_float(w[i] << 16) * c, __uint_as_float(w[i] & 0xffff0000u) * c);
#else
            qraw[cb][t] = w;
#endif
        }
    }
    f32x16 acc[4][2];   // O^T: [head-element block][query block]
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][cb][r] = 0.f;
    // keeps Q and the O accumulators in accumulation registers across the loops' control flow
    auto pin = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int t = 0; t < 8; ++t) asm volatile("" : "+a"(qraw[cb][t]));
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) asm volatile("" : "+a"(acc[db][cb]));
    };
    pin();

    // The softmax reference is fixed, so key tiles may come in any order: the unmasked ones (see
    // KeyTiles) run through a loop without masking code, the others through a copy that masks.
    const int nMain = kt.nMain, nT = kt.hi;
    const char* zk_b = reinterpret_cast<const char*>(zk) + static_cast<size_t>(hk) * P * ROW_B;
    const char* zv_b = reinterpret_cast<const char*>(zv) + static_cast<size_t>(hk) * P * ROW_B;
    const uint32_t own_pitch = static_cast<uint32_t>(Hkv) * ROW_B;
    const char* k_b = reinterpret_cast<const char*>(k) + (t0 * Hkv + hk) * ROW_B;
    const char* v_b = reinterpret_cast<const char*>(v) + (t0 * Hkv + hk) * ROW_B;
    auto tile_pre = [&](int t) __attribute__((always_inline)) { return kt.pre(t); };
    auto tile_j0 = [&](int t) __attribute__((always_inline)) { return kt.j0(t); };

    // Direct-to-LDS load of one tile, eight instructions per wavefront (K rows, then V rows),
    // handed out one per matrix-core instruction by the stage below.
    const uint32_t dma_c0 = (lane & 15) ^ (((lane >> 4) & 3) << 2);   // chunk under the swizzle, before ^ i
    struct TileSrc { const char* kb; const char* vb; int lim; uint32_t pitch; uint32_t lds_k, lds_v; };
    auto tile_src = [&](int t, int buf) __attribute__((always_inline)) {
        const bool pre = tile_pre(t);
        const int j0 = tile_j0(t);
        TileSrc ts;
        ts.pitch = pre ? static_cast<uint32_t>(ROW_B) : own_pitch;
        ts.kb = (pre ? zk_b : k_b) + static_cast<size_t>(j0) * ts.pitch;
        ts.vb = (pre ? zv_b : v_b) + static_cast<size_t>(j0) * ts.pitch;
        ts.lim = (pre ? P : S) - 1 - j0;    // rows past the end repeat the last valid row
        ts.lds_k = lds_addr(sm.k[buf]);
        ts.lds_v = lds_addr(sm.v[buf]);
        return ts;
    };
    auto dma_piece = [&](const TileSrc& ts, int n) __attribute__((always_inline)) {
        const int i = n & 3;
        const int r0 = (4 * wv + i) * 4;
        const uint32_t voff = __umul24(min(r0 + (lane >> 4), ts.lim), ts.pitch) + ((dma_c0 ^ i) << 4);
        if (n < 4) dma16(ts.kb, voff, ts.lds_k + r0 * ROW_B);
        else       dma16(ts.vb, voff, ts.lds_v + r0 * ROW_B);
    };
    // hidden entries of the scores of the sub-tile whose first key is j0 (prefix or own) -> very negative
    auto mask = [&](f32x16 (&x)[2], bool pre, int j0) __attribute__((always_inline)) {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            // key j0 + d_row(r, lg) is hidden when it exceeds the lane's last visible key
            mask_above(x[cb], (pre ? P - 1 : wrow0 + 32 * cb + lc) - j0 - 4 * lg);
            // ... or precedes the first key of the query's sequence
            if (row_lo && !pre) mask_below(x[cb], lo_q[cb] - j0 - 4 * lg);
        }
    };

    // Per-lane LDS addresses of the operand fragments, complete except for compile-time offsets;
    // they move from buffer to buffer once per tile (K fragments are fetched one tile ahead of V).
    uint32_t kofs[8], vofs[4][2];
    {
        const uint32_t lk = lds_addr(sm.k[1]), lv = lds_addr(sm.v[0]);
#pragma unroll
        for (int t8 = 0; t8 < 8; ++t8) kofs[t8] = lk + lc * ROW_B + (((2 * t8 + lg) ^ swz(lc)) << 4);
        const int s16 = lane & 15;
        const int row = 4 * lg + (s16 >> 2);
        const int col0 = 16 * ((lane >> 4) & 1) + 4 * (s16 & 3);
        const int half = ((col0 >> 2) & 1) * 8;
#pragma unroll
        for (int db = 0; db < 4; ++db) {
            const int ch = (32 * db + col0) >> 3;
            vofs[db][0] = lv + row * ROW_B + ((ch ^ swz(row)) << 4) + half;
            vofs[db][1] = lv + (row + 8) * ROW_B + ((ch ^ swz(row + 8)) << 4) + half;
        }
    }
    typedef const bf16x8 __attribute__((address_space(3))) * lds_b128;
    typedef s16x4 __attribute__((address_space(3))) * lds_b64;
    // row-wise K fragment t8 of the 32-row half hb of the buffer kofs points at
    auto ld_k = [&](int t8, int hb) __attribute__((always_inline)) {
        return *(lds_b128)(kofs[t8] + hb * 32 * ROW_B);
    };
    // transposed V fragment (k-step ks, head-element block db) of half hb of the buffer at vofs
    auto ld_v = [&](int ks, int db, int hb) __attribute__((always_inline)) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_b64)(vofs[db][0] + (32 * hb + 16 * ks) * ROW_B));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_b64)(vofs[db][1] + (32 * hb + 16 * ks) * ROW_B));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    // -m (the softmax reference of the lane's query) in all 16 registers of a set: the first
    // product of every score chain starts from it, so S arrives as the exponent c s - m
#if CART_PRESCALE
    f32x16 ninit[2];
#else
    float negm[2];
#endif
    float l_run[2] = {0.f, 0.f};
    // Scores live in ordinary vector registers, in two sets used alternately: while the vector
    // ALU reads S(u) from one set the matrix cores write S(u+1) into the other, so no copy sits
    // between the matrix cores' results and the softmax arithmetic.
    f32x16 sa[2], sb[2];
    u32x4 pf[2][2];           // P^T(u-1) as B-operand fragments [query block][k-step]
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) pf[cb][ks] = u32x4{0u, 0u, 0u, 0u};
    bf16x8 ka[8], va[2][4];   // K fragments of sub-tile u+1, V fragments of sub-tile u-1
    // The last two V fragments have a spare register set each (indexed by the parity of the
    // iteration that USES them): the next iteration's copies are requested before this
    // iteration's last use, so no LDS read is issued in the last groups and the wait in front of
    // the tile barrier finds nothing outstanding.
    bf16x8 vb6[2], vb7[2];

    // Iteration u (sub-tile hb of a tile; MASKED: it may hold hidden keys).  On entry: x = S(u),
    // ka = K fragments of sub-tile u+1, va = V fragments of sub-tile u-1, pf = P(u-1); on exit
    // y = S(u+1).  The work is laid out as 32 groups of one matrix-core instruction plus one
    // softmax element and the odd jobs that go with it, fenced so that the scheduler keeps the
    // spread: the matrix cores run S^T(u+1) = K Q^T (groups 0-15) and O^T += V^T P^T(u-1)
    // (groups 16-31) while the vector ALU turns S(u) into P(u); each fragment register is
    // refilled from LDS for the next iteration right after its last use, and the eight
    // direct-to-LDS loads of tile t+2 (DMA, first sub-tile only) ride along in groups 0-7.
    auto stage = [&](auto hb_tag, auto masked_tag, bool pre, int j0, f32x16 (&x)[2], f32x16 (&y)[2],
                     const TileSrc& ts) __attribute__((always_inline)) {
        constexpr int hb = decltype(hb_tag)::value;
        constexpr bool MASKED = decltype(masked_tag)::value;
        if (MASKED) mask(x, pre, j0 + 32 * hb);
        pin();
        float pe[32];
        u32x4 pn[2][2];
#pragma unroll
        for (int g = 0; g < 32; ++g) {
            if (g < 16) {
                const int t8 = g >> 1, cb = g & 1;
#if CART_PRESCALE
                if (t8 == 0) mma_vd_first(y[cb], ka[0], qraw[cb][0], ninit[cb]);
#else
                if (t8 == 0) mma_vd_zero(y[cb], ka[0], qraw[cb][0]);
#endif
                else         mma_vd(y[cb], ka[t8], qraw[cb][t8]);
            } else {
                const int i = g - 16, ks = i >> 3, db = (i >> 1) & 3, cb = i & 1, p = 4 * ks + db;
                const bf16x8 vf_ = p == 6 ? vb6[hb] : p == 7 ? vb7[hb] : va[ks][db];
                acc[db][cb] = mma(vf_, __builtin_bit_cast(bf16x8, pf[cb][ks]), acc[db][cb]);
            }
            __builtin_amdgcn_sched_barrier(0);   // the matrix-core instruction leads its group
            if (hb == 0 && g < 8) dma_piece(ts, g);
            // refill the fragment register the previous two groups used last
            if (g >= 2 && g <= 16 && !(g & 1)) ka[(g - 2) >> 1] = ld_k((g - 2) >> 1, hb);
            if (g >= 18 && g <= 28 && !(g & 1)) {
                const int i = g - 18;
                va[i >> 3][(i >> 1) & 3] = ld_v(i >> 3, (i >> 1) & 3, hb);
            }
            if (g == 25) vb6[1 - hb] = ld_v(1, 2, hb);
            if (g == 27) vb7[1 - hb] = ld_v(1, 3, hb);
            // the LDS reads go out right behind the matrix-core instruction, ahead of the vector ALU work
            __builtin_amdgcn_sched_barrier(0);
            {   // softmax element g; the pair before it is rounded, packed and summed
                const int cb = g >> 4, r = g & 15;
#if CART_PRESCALE
                pe[g] = fast_exp2(x[cb][r]);
#else
                pe[g] = fast_exp2(fmaf(x[cb][r], c, negm[cb]));
#endif
                if (g >= 2 && !(g & 1)) {
                    const int e = g - 2, cbe = e >> 4, re = e & 15;
                    pn[cbe][re >> 3][(re & 7) >> 1] = pack_bf16x2(pe[e], pe[e + 1]);
                    l_run[cbe] += pe[e] + pe[e + 1];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        pn[1][1][3] = pack_bf16x2(pe[30], pe[31]);
        l_run[1] += pe[30] + pe[31];
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) pf[cb][ks] = pn[cb][ks];
        __builtin_amdgcn_sched_barrier(0);
    };
    // the matrix-core results of the inline-assembly products are not tracked by the compiler's
    // hazard logic: before the vector ALU touches them, let the last one retire
    auto settle = [&]() __attribute__((always_inline)) { asm volatile("s_nop 15\n\ts_nop 7" ::: "memory"); };

    {   // tiles 0 and 1 on their way; scores of sub-tile 0 and the softmax reference of every
        // query: its maximum over that sub-tile (which holds a visible key for every query)
        const TileSrc t0 = tile_src(kt.lo, 0);
#pragma unroll
        for (int n = 0; n < 8; ++n) dma_piece(t0, n);
        const TileSrc t1 = tile_src(min(kt.lo + 1, nT - 1), 1);
#pragma unroll
        for (int n = 0; n < 8; ++n) dma_piece(t1, n);
        const TileSrc t2 = tile_src(min(kt.lo + 2, nT - 1), 2);
#pragma unroll
        for (int n = 0; n < 8; ++n) dma_piece(t2, n);
        dma_wait_but<16>();
        __syncthreads();
#pragma unroll
        for (int t8 = 0; t8 < 8; ++t8) ka[t8] = lds_frag_n(sm.k[0], lc, 16 * t8 + 8 * lg);
#pragma unroll
        for (int t8 = 0; t8 < 8; ++t8) {
            if (t8 == 0) { mma_vd_zero(sa[0], ka[0], qraw[0][0]); mma_vd_zero(sa[1], ka[0], qraw[1][0]); }
            else         { mma_vd(sa[0], ka[t8], qraw[0][t8]);    mma_vd(sa[1], ka[t8], qraw[1][t8]); }
        }
        settle();
        mask(sa, tile_pre(kt.lo), tile_j0(kt.lo));
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            float tm = sa[cb][0];
#pragma unroll
            for (int r = 1; r < 16; ++r) tm = fmaxf(tm, sa[cb][r]);
#if CART_PRESCALE
            const float nm = -partner_max(tm);
#pragma unroll
            for (int r = 0; r < 16; ++r) { ninit[cb][r] = nm; sa[cb][r] += nm; }
#else
            negm[cb] = -partner_max(tm) * c;
#endif
        }
#pragma unroll
        for (int t8 = 0; t8 < 8; ++t8) ka[t8] = lds_frag_n(sm.k[0], 32 + lc, 16 * t8 + 8 * lg);   // sub-tile 1
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)     // placeholder for "V of sub-tile -1": multiplied by P = 0
#pragma unroll
            for (int db = 0; db < 4; ++db) va[ks][db] = lds_frag_t(sm.v[0], 16 * ks, 32 * db, lane);
        vb6[0] = va[1][2];
        vb7[0] = va[1][3];
    }
    // Four LDS buffers, tile t in buffer t % 4.  The one barrier per tile opens the iteration of
    // the tile's first sub-tile: it publishes tile t+1 (read from this iteration on; its loads
    // went out two iterations ago, so their memory latency is covered twice over) and retires
    // tile t-1's buffer (its last fragments were fetched in the previous iteration), which then
    // receives tile t+3.
    int buf = 0;
    auto tile_iter = [&](int t, auto masked_tag) __attribute__((always_inline)) {
        const int nbuf = buf + 1 == FWD_NBUF ? 0 : buf + 1;
        const int nnbuf = nbuf + 1 == FWD_NBUF ? 0 : nbuf + 1;
        const int n3buf = nnbuf + 1 == FWD_NBUF ? 0 : nnbuf + 1;
        const TileSrc ts = tile_src(min(t + 3, nT - 1), n3buf);
        const bool pre = tile_pre(t);
        const int j0 = tile_j0(t);
        dma_wait_but<8>();      // tile t+1 has landed (t+2 may still be in flight)
        __syncthreads();
        if (decltype(masked_tag)::value && !pre && j0 > wrow0 + 63) {
            // A diagonal tile that lies entirely behind this wavefront's 64 queries (so do all
            // that follow): nothing to compute -- its share of the loads still goes out, and the
            // state of the pipeline (P and the V fragments of the last visible sub-tile) waits
            // for the drain.  The products skipped are a few per cent of the kernel's, and under
            // these kernels the chip's clock follows the energy spent.
#pragma unroll
            for (int n = 0; n < 8; ++n) dma_piece(ts, n);
        } else {
            stage(std::integral_constant<int, 0>{}, masked_tag, pre, j0, sa, sb, ts);
            stage(std::integral_constant<int, 1>{}, masked_tag, pre, j0, sb, sa, ts);
        }
        // fragment addresses follow the buffers: K to tile t+2's, V to tile t+1's
        const uint32_t dk = nnbuf == 0 ? static_cast<uint32_t>(-(FWD_NBUF - 1) * FWD_TILE_B) : static_cast<uint32_t>(FWD_TILE_B);
        const uint32_t dv = nbuf == 0 ? static_cast<uint32_t>(-(FWD_NBUF - 1) * FWD_TILE_B) : static_cast<uint32_t>(FWD_TILE_B);
#pragma unroll
        for (int t8 = 0; t8 < 8; ++t8) kofs[t8] += dk;
#pragma unroll
        for (int db = 0; db < 4; ++db) { vofs[db][0] += dv; vofs[db][1] += dv; }
        buf = nbuf;
    };
    for (int t = kt.lo; t < min(nMain, nT); ++t) tile_iter(t, std::false_type{});
    for (int t = max(kt.lo, nMain); t < nT; ++t) tile_iter(t, std::true_type{});
    {   // drain: O^T += V^T P^T of the last sub-tile (its V fragments are already in registers)
        pin();
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int db = 0; db < 4; ++db) {
                const int p = 4 * ks + db;
                const bf16x8 vf_ = p == 6 ? vb6[0] : p == 7 ? vb7[0] : va[ks][db];
                acc[db][0] = mma(vf_, __builtin_bit_cast(bf16x8, pf[0][ks]), acc[db][0]);
                acc[db][1] = mma(vf_, __builtin_bit_cast(bf16x8, pf[1][ks]), acc[db][1]);
            }
    }
#if CART_PRESCALE
    float m_ref[2] = {-ninit[0][0], -ninit[1][0]};
#else
    float m_ref[2] = {-negm[0], -negm[1]};
#endif

    // normalise and store, turned around in LDS once nobody reads a tile or has a load in flight
    dma_wait();
    if (!FEW) __syncthreads();
    float l_tot[2], inv[2];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
        const int qi = wrow0 + 32 * cb + lc;
        l_tot[cb] = l_run[cb] + partner(l_run[cb]);
        inv[cb] = 1.f / l_tot[cb];
        const float row_lse = (m_ref[cb] + fast_log2(l_tot[cb])) * CART_LN2;
        if (qi < S && lg == 0) {
            if (qb.n_parts == 1) lse[sp.stat_b + h * sp.stat_h + qi] = row_lse;
            else                 my_l[32 * cb + lc] = row_lse;
        }
    }
    char* const turn = reinterpret_cast<char*>(&sm) + wv * (2 * FWD_TILE_B);
    RowSums rs;
    if (FEW)
        rs = store_rows64_direct(acc, inv[0], inv[1], o + ((t0 + wrow0) * Hq + h) * HD, static_cast<size_t>(Hq) * HD, S - wrow0, lane);
    else if (qb.n_parts == 1)
        rs = store_rows64(turn, acc, inv[0], inv[1], o + ((t0 + wrow0) * Hq + h) * HD, static_cast<size_t>(Hq) * HD, S - wrow0, lane);
    else
        rs = store_rows64(turn, acc, inv[0], inv[1], part_o + (static_cast<size_t>(qb.slot) * 256 + 64 * wv) * HD, HD, S - wrow0, lane);
    // overflow of the fixed-reference softmax shows as a non-finite row sum or output
    bool bad = false;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
        bad |= wrow0 + 32 * cb + lc < S && (!(l_tot[cb] < 3.0e38f) || !(fabsf(rs.s[cb]) < 3.0e38f));
    bad = __any(bad);
    if (qb.n_parts > 1) {      // (a flag per wavefront: a barrier here would wait for the stores, 4-5 us of a block)
        if (lane == 0) *my_flag = bad ? 1 : 0;
    } else if (bad) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // (other lanes stored these rows)
        recompute_rows(q, k, v, zk, zv, o, lse + sp.stat_b + h * sp.stat_h, row_lo, t0, wrow0, min(S, wrow0 + 64), h, hk, Hq, Hkv,
                       P, c, lane);
    }
}

// Finishes the split blocks of a forward call (eight workgroups each, 32 rows apiece): combines the
// parts by their log-sum-exps, or recomputes the rows of a wavefront that raised its overflow flag.  (Blocks
// that run whole recompute their own; left to this kernel, every
// call paid its launch: one sequence of 64 tokens, 128 slots 15.2 -> 12.9 us, 16 x 256, 1024 slots 83.2 -> 81.0.)
__global__ __launch_bounds__(256) void attn_fwd_finish_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
    const bf16_t* __restrict__ zk, const bf16_t* __restrict__ zv, bf16_t* __restrict__ o,
    float* __restrict__ lse, const int* __restrict__ flags, const int32_t* __restrict__ cu,
    const int32_t* __restrict__ row_lo, int n_tok, int Smax, int Hq, int Hkv, int P, float c, QuerySplit split,
    const float* __restrict__ part_o, const float* __restrict__ part_l) {
    const int G = Hq / Hkv, nW = query_wgs(Smax, G);
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r0 = 8 * (blockIdx.x & 7), hk = (blockIdx.x >> 3) % Hkv, blk = (blockIdx.x >> 3) / Hkv, e = split.e_full + blk;
    const int x = split.first[blk], n_parts = split.part[x] >> 16;      // the block's first part, its parts
    if (n_parts == 1) return;               // (a short block among the split ones ran whole)
    const QueryBlock qb = query_block_of(hk, e, wv, nW, G);
    const SeqSpan sp = seq_span(cu, qb.b, n_tok, Smax, Hq);
    const int S = sp.len, h = qb.h, i0 = qb.wrow0 + r0, i1 = min(S, i0 + 8);
    const size_t t0 = sp.t0;
    // Half a wavefront per row, four head elements per lane: two rows per load, eight rows in flight, four parts at a time
    // (past the last one: the last, not used).  The first four leave ahead of the flags, none waits for its LSE (an empty
    // part's are not used): one round trip to memory where there were three (a forward call from a graph, us: 1 x 700
    // tokens, 32 / 8 heads, 1000 slots, in three parts 37.5 -> 36.0; 5 x 333, 8 / 2, 2500 38.3 -> 37.5; 1 x 64, 8 / 8, 8000 34.0 -> 33.6).
    constexpr int R = 4, U = 4;
    const int half = lane >> 5, d4 = 4 * (lane & 31);
    const size_t row0 = (static_cast<size_t>(x) * Hkv + hk) * 256 + 64 * wv + r0 + half;
    float pl[U][R];
    f32x4 po[U][R];
    auto load = [&](int p0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t row = row0 + static_cast<size_t>(min(p0 + u, n_parts - 1)) * Hkv * 256;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                pl[u][r] = part_l[row + 2 * r];
                po[u][r] = *reinterpret_cast<const f32x4*>(part_o + (row + 2 * r) * HD + d4);
            }
        }
    };
    load(0);
    int bad = 0;         // of this wavefront's rows
    for (int p = 0; p < n_parts; ++p) bad |= flags[4 * ((x + p) * Hkv + hk) + wv];
    if (!bad) {
        const float ninf = __uint_as_float(0xff800000u);
        float m[R], l[R];
        f32x4 a[R];
#pragma unroll
        for (int r = 0; r < R; ++r) { m[r] = -3.0e38f; l[r] = 0.f; a[r] = f32x4{0.f, 0.f, 0.f, 0.f}; }
        for (int p0 = 0; p0 < n_parts; p0 += U) {
            if (p0 > 0) load(p0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (p0 + u >= n_parts) break;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float nm = fmaxf(m[r], pl[u][r]), corr = __expf(m[r] - nm), w = __expf(pl[u][r] - nm);
                    l[r] = l[r] * corr + w;
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[r][e] = a[r][e] * corr + (pl[u][r] > ninf ? w * po[u][r][e] : 0.f);
                    m[r] = nm;
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = i0 + 2 * r + half;
            if (i >= i1) continue;
            const float inv = 1.f / l[r];
            u32x2 w = {pack_bf16x2(a[r][0] * inv, a[r][1] * inv), pack_bf16x2(a[r][2] * inv, a[r][3] * inv)};
            *reinterpret_cast<u32x2*>(o + ((t0 + i) * Hq + h) * HD + d4) = w;
            if ((lane & 31) == 0) lse[sp.stat_b + h * sp.stat_h + i] = m[r] + __logf(l[r]);
        }
        return;
    }
    recompute_rows(q, k, v, zk, zv, o, lse + sp.stat_b + h * sp.stat_h, row_lo, t0, i0, i1, h, hk, Hq, Hkv, P, c, lane);
}

// row_lo[i] = first packed row of the sequence that row i belongs to (cu: B+1 offsets, cu[B] = T)
__global__ __launch_bounds__(256) void attn_row_lo_kernel(const int32_t* __restrict__ cu, int B, int T,
                                                          int32_t* __restrict__ row_lo) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= T) return;
    int lo = 0, hi = B;                 // largest b with cu[b] <= i
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cu[mid] <= i) lo = mid; else hi = mid;
    }
    row_lo[i] = cu[lo];
}
int launch_row_lo(const int32_t* cu, int B, int T, int32_t* row_lo, hipStream_t st) {
    hipLaunchKernelGGL(attn_row_lo_kernel, dim3((T + 255) / 256), dim3(256), 0, st, cu, B, T, row_lo);
    return static_cast<int>(hipGetLastError());
}

// Whether and how far to split is decided by playing the launch through: blocks go to the CU that is
// free first, in order.  With many rounds there is little to gain, and blocks of very different lengths (long
// sequences, short prefix) even each other out: not split.
// The forward's times, from calls with every number of parts (us; tiles of the longest block, blocks -> whole;
// 2, 3, 4, 6 parts; * taken):
//   1 x   64 tokens, 32 / 8 heads, 2000 slots  33,  8 -> 48.6; 35.3 30.6 27.8 26.5*     1 x 256, 32 / 8,  512  12, 32 -> 23.6*; 25.8 25.6 27.6 29.4
//   1 x  128,        32 / 8,       1024        18, 16 -> 30.6; 27.5 25.4* 24.6 26.2     1 x  32,  8 / 8,  300   6,  8 -> 15.6*; 17.6 18.4 18.4 20.5
//   1 x  700,        32 / 8,       1000        27, 88 -> 41.9; 40.0 38.0* -             6 x  90, 16 / 4,  700  13, 48 -> 24.2*; 26.7 26.7 29.4 30.2
//   1 x 1024,         8 / 2,          0        16, 32 -> 28.4; 25.6 24.5 24.0* 25.6     2 x  64,  8 / 2,  600  11,  4 -> 22.8; 21.8 20.2 20.7* 22.2
//   1 x 2048,         8 / 2,        256        36, 64 -> 51.8; 39.8 34.4 32.4 31.4      2 x 333,  3 / 3,   31   7, 12 -> 18.1*; 23.7 24.3 25.0 24.9
// Only unmasked tiles are divided (see key_tiles): a part that ends in ten masked ones is no shorter for it (three packed
// sequences of 700, 1 and 90 tokens, 32 / 8 heads, 300 slots: whole 40.6, 2 parts 49.7).
constexpr int SPLIT_MIN_TILES = 4;      // (dQ: 1.95 (n - 1) > 4 + 2 x 0.05; the forward: 6)

// blocks per KV head the chip runs at one time
static int query_slots(int Hkv) {
    const int n = device_cus() / Hkv;
    return n < 1 ? 1 : (n > MAX_SPLIT ? MAX_SPLIT : n);
}

// key tiles of block e of a KV head, the masked ones among them
struct Tiles { int all, masked; };
static Tiles block_tiles(int e, int S, int G, int P, int own_cap, bool meet) {
    const int nW = query_wgs(S, G), w = nW - 1 - e % nW, q_end = 64 * ((4 * w + 3) / G) + 64, tD = 4 * w / G;
    const int upto = ((q_end < S ? q_end : S) + 63) / 64, own = own_cap > 0 && own_cap < upto ? own_cap : upto;
    // (a block in which sequences meet: none of its own tiles is seen whole by all of its rows)
    return Tiles{(P + 63) / 64 + own, (P % 64 ? 1 : 0) + (meet ? own : upto - tD < own ? upto - tD : own)};
}
// the longest of np parts
static int longest(const Tiles& t, int np) {
    const int step = (t.all + np - 1) / np, last = t.all - t.masked - 1, from = (np - 1) * step < last ? (np - 1) * step : last;
    return np == 1 ? t.all : t.all - (from > 0 ? from : 0) > step ? t.all - (from > 0 ? from : 0) : step;
}

void mfma::plan_query_split(QuerySplit& sp, int B, int S, int G, int Hkv, int P, int own_cap, bool meet, const SplitCost& us) {
    const int nW = query_wgs(S, G);
    const long n_all = static_cast<long>(B) * nW;
    const int slots = query_slots(Hkv);
    sp.e_full = static_cast<int>(n_all);
    sp.n_blocks = sp.n_parts = 0;
    if (n_all > 4L * slots || n_all > 2 * MAX_SPLIT || (P + 63) / 64 + (S + 63) / 64 < SPLIT_MIN_TILES) return;
    const int n = static_cast<int>(n_all), left = n % slots;       // the blocks left over after whole rounds
    if (left == 0) return;
    auto tiles = [&](int e) { return block_tiles(e, S, G, P, own_cap, meet); };
    float cu[MAX_SPLIT];                                    // when each CU is free
    for (int i = 0; i < slots; ++i) cu[i] = 0.f;
    float done = 0.f;                                       // when the whole rounds are done
    for (int e = 0; e < n - left; ++e) {
        const float t = run_next(cu, slots, us.block + us.tile * tiles(e).all);
        done = t > done ? t : done;
    }
    Tiles tl[MAX_SPLIT];
    int most = 0;
    for (int i = 0; i < left; ++i) {
        tl[i] = tiles(n - left + i);
        most = tl[i].all > most ? tl[i].all : most;
    }
    int best = 0;                                           // tiles per part, 0: whole
    float best_t = 0.f;
    for (int parts = 1; parts <= 32 && parts <= most; ++parts) {
        const int tps = (most + parts - 1) / parts;
        int items = 0;
        for (int i = 0; i < left; ++i) items += (tl[i].all + tps - 1) / tps;
        if (items > slots) break;
        float c[MAX_SPLIT], end = done;
        for (int i = 0; i < slots; ++i) c[i] = cu[i];
        for (int i = 0; i < left; ++i) {
            const int np = (tl[i].all + tps - 1) / tps;
            for (int p = 0; p < np; ++p) {
                const float len = us.block + us.tile * (p == np - 1 ? longest(tl[i], np) : (tl[i].all + np - 1) / np);
                const float t = n == left ? len : run_next(c, slots, len);
                end = t > end ? t : end;
            }
        }
        if (parts > 1) end += us.fix + us.part * ((most + tps - 1) / tps) + us.wg * items * Hkv;
        if (parts == 1 || end < best_t) {
            best_t = end;
            best = parts == 1 ? 0 : tps;
        }
    }
    if (best == 0) return;
    sp.e_full = n - left;
    sp.n_blocks = left;
    for (int i = 0; i < left; ++i) {
        const uint32_t np = static_cast<uint32_t>((tl[i].all + best - 1) / best);
        sp.first[i] = static_cast<uint32_t>(sp.n_parts);
        for (uint32_t p = 0; p < np; ++p) sp.part[sp.n_parts++] = static_cast<uint32_t>(i) | p << 8 | np << 16;
    }
}
static size_t r256(size_t n) { return (n + 255) & ~static_cast<size_t>(255); }

bool attn_mfma_supported(const cart_attn_desc& d) {
    return d.dtype == CART_BF16 && d.D == 128;
}
// What a split depends on: blocks per sequence, or over the packed rows (a packed batch with a prefix; T > 0)
struct SplitKey { int B, S, G, Hkv, P, own_cap, meet, cus; };
static SplitKey split_key(const cart_attn_desc& d, int T) {
    const int G = d.Hq / d.Hkv;
    const bool rows = T > 0 && d.P > 0;
    // (packed: a block's rows and those of the first one's sequence before it, and the tiles they begin and end inside)
    const int block_rows = 4 % G == 0 ? 256 / G : G % 4 == 0 ? 64 : 128;
    return {rows ? 1 : d.B, rows ? T : d.S, G, d.Hkv, d.P, rows ? (d.S + block_rows + 126) / 64 : 0, rows && d.B > 1, device_cus()};
}
bool attn_query_split_all(mfma::QuerySplit& sp, const cart_attn_desc& d, int T, int parts, int most) {
    const SplitKey k = split_key(d, T);
    const long n = static_cast<long>(k.B) * query_wgs(k.S, k.G);
    sp.n_blocks = sp.n_parts = 0;
    sp.e_full = static_cast<int>(n);
    if (parts == 1) return true;
    most = most < MAX_SPLIT ? most : MAX_SPLIT;
    if (n > most) return false;
    int all = 0;
    for (int e = 0; e < n; ++e) {
        const int t = block_tiles(e, k.S, k.G, k.P, k.own_cap, k.meet != 0).all;
        all = t > all ? t : all;
    }
    const int step = (all + parts - 1) / parts;             // tiles per part, the same for every block
    sp.e_full = 0;
    sp.n_blocks = static_cast<int>(n);
    for (int e = 0; e < n; ++e) {
        const int np = (block_tiles(e, k.S, k.G, k.P, k.own_cap, k.meet != 0).all + step - 1) / step;
        if (sp.n_parts + np > most) return false;
        sp.first[e] = static_cast<uint32_t>(sp.n_parts);
        for (int p = 0; p < np; ++p) sp.part[sp.n_parts++] = static_cast<uint32_t>(e | p << 8 | np << 16);
    }
    return true;
}
int attn_query_tiles(const cart_attn_desc& d, int T, const mfma::QuerySplit& sp, int* tiles, int most) {
    const SplitKey k = split_key(d, T);
    const int n = sp.e_full + sp.n_parts;
    if (n > most) return -1;
    for (int i = 0; i < n; ++i) {
        const uint32_t it = i < sp.e_full ? 0x10000u : sp.part[i - sp.e_full];
        const Tiles t = block_tiles(i < sp.e_full ? i : sp.e_full + static_cast<int>(it & 255), k.S, k.G, k.P, k.own_cap, k.meet != 0);
        const int np = static_cast<int>(it >> 16);
        tiles[i] = static_cast<int>((it >> 8) & 255) == np - 1 ? longest(t, np) : (t.all + np - 1) / np;
    }
    return n;
}
// The layers of a step ask for the same two splits in turn, forward's and dQ's: the thread's last one of either kind is kept with
// all that it depends on (planned again at each call, 32 sequences of 516 tokens, 8 / 2 heads: 18 us a layer).
void attn_query_split(mfma::QuerySplit& sp, const cart_attn_desc& d, int T, mfma::QueryKernel kind) {
    static thread_local SplitKey last[2];
    static thread_local QuerySplit kept[2];
    const int G = d.Hq / d.Hkv;
    const SplitKey k = split_key(d, T);
    SplitKey& l = last[kind];
    if (l.cus != k.cus || l.B != k.B || l.S != k.S || l.G != k.G || l.Hkv != k.Hkv || l.P != k.P || l.own_cap != k.own_cap ||
        l.meet != k.meet) {
        plan_query_split(kept[kind], k.B, k.S, G, d.Hkv, d.P, k.own_cap, k.meet != 0, SPLIT_COST[kind]);
        l = k;
    }
    sp = kept[kind];
}
// The most parts per KV head that this problem or any smaller one is split into: the workspace holds that
// many, so that one kept for a program's largest batch serves its smaller ones (which are split further).
size_t attn_query_parts(const cart_attn_desc& d, int T) {
    const int G = d.Hq / d.Hkv;
    const long by_seq = static_cast<long>(d.B) * query_wgs(d.S, G), by_row = T > 0 ? query_wgs(T, G) : 0;
    const long tiles = (static_cast<long>(d.P) + 63) / 64 + (d.S + 63) / 64 + 6;        // (own_cap at most 6 more than S's)
    const long all = (by_seq > by_row ? by_seq : by_row) * tiles, slots = query_slots(d.Hkv);
    // (No workspace at all for the smallest calls, whose time is the host's: allocating one that is never used took 1.1 us
    // of 10.0.  Parts of one tile each cost more than the tiles saved up to SPLIT_MIN_TILES - 1 of them.)
    if (T == 0 && tiles - 6 < SPLIT_MIN_TILES) return 0;
    return static_cast<size_t>(all < slots ? all : slots);
}
// packed batches: the first row of every row's sequence; split blocks: an overflow flag per wavefront and the
// partial results
size_t attn_mfma_fwd_workspace(const cart_attn_desc& d, int T) {
    const size_t slots = attn_query_parts(d, T) * d.Hkv;
    return r256(slots * 4 * sizeof(int)) + (T > 0 ? r256(static_cast<size_t>(T) * sizeof(int32_t)) : 0) +
           slots * (PART_O_BYTES + PART_L_BYTES);
}

// cu == nullptr: batched layout [B,S,...].  Otherwise the packed layout: d.S is the longest
// sequence, T the number of packed rows, cu (device) the B+1 row offsets.
int launch_attn_fwd_mfma(const cart_attn_desc& d, float scale, const void* q, const void* k,
                         const void* v, const void* zk, const void* zv, void* o, float* lse,
                         void* ws, hipStream_t st, const int32_t* cu, int T) {
    if (!cu) T = 0;
    QuerySplit sp;
    attn_query_split(sp, d, T, QUERY_FWD);
    const size_t slots = static_cast<size_t>(sp.n_parts) * d.Hkv;
    const unsigned n_items = static_cast<unsigned>(sp.e_full + sp.n_parts) * d.Hkv;
    char* w = static_cast<char*>(ws);
    int* flags = reinterpret_cast<int*>(w);
    w += r256(slots * 4 * sizeof(int));
    int32_t* row_lo = nullptr;
    if (T > 0) {
        if (d.P > 0) row_lo = reinterpret_cast<int32_t*>(w);
        w += r256(static_cast<size_t>(T) * sizeof(int32_t));
    }
    float* part_l = reinterpret_cast<float*>(w);
    float* part_o = reinterpret_cast<float*>(w + slots * PART_L_BYTES);
    int S = d.S;
    const bf16_t *Q = static_cast<const bf16_t*>(q), *K = static_cast<const bf16_t*>(k),
                 *V = static_cast<const bf16_t*>(v), *ZK = static_cast<const bf16_t*>(zk),
                 *ZV = static_cast<const bf16_t*>(zv);
    if (row_lo) {          // blocks over the packed rows: the kernels see one sequence of T rows
        launch_row_lo(cu, d.B, T, row_lo, st);
        cu = nullptr;
        S = T;
    }
    trace_begin(st);   // kernel order: forward, finish (nothing between its events when no block is split)
    // Sequences of at most two units (64 tokens of one query head of the KV group), one block each.  With the stores
    // through LDS (us a forward call): 256 sequences of 64 tokens, 16 / 16 heads, 64 slots 148.0, now 130.8; 128 of 128,
    // 32 / 32 heads 198.5, now 178.7.  With four wavefronts' rows LDS is the faster way (see store_rows64).
    const bool few = !row_lo && sp.n_parts == 0 && (S + 63) / 64 * (d.Hq / d.Hkv) <= 2;
    auto forward = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(n_items), dim3(256), 0, st, Q, K, V, ZK, ZV, static_cast<bf16_t*>(o), lse, flags, cu, row_lo, T,
                           S, d.Hq, d.Hkv, d.P, scale * CART_LOG2E, sp, part_o, part_l);
    };
    if (few) forward(attn_fwd_mfma_kernel<true>);
    else     forward(attn_fwd_mfma_kernel<false>);
    trace_mark(st);
    if (sp.n_blocks > 0)
        hipLaunchKernelGGL(attn_fwd_finish_kernel, dim3(static_cast<unsigned>(8 * sp.n_blocks) * d.Hkv), dim3(256), 0, st, Q, K, V, ZK, ZV,
                           static_cast<bf16_t*>(o), lse, flags, cu, row_lo, T, S, d.Hq, d.Hkv, d.P, scale * CART_LOG2E, sp, part_o,
                           part_l);
    trace_mark(st);
    return static_cast<int>(hipGetLastError());
}

}  // namespace cart
