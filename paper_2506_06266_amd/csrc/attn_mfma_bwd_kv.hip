// Key and value gradients of cartridge attention in ONE pass over the queries (bf16, head_dim
// 128): dK, dV of the own tokens and the per-chunk partials of dZ_k, dZ_v (Sec. 3.2: the loss is
// back-propagated into the key and value vectors of Z with the model frozen).
//
// Keys stationary, as in the split dK / dV kernels this replaces, but the scores S and the
// probabilities P are formed once and serve both gradients: 4 contractions per visible (query,
// key) pair (S, dP, dV, dK) instead of 5 (S twice).  One wavefront cannot hold the accumulators of
// both gradients for 64 keys next to the stationary K and V fragments (that is 384 of its 512
// registers before any working set), so the work of a block of 64 keys is split over a PAIR of
// wavefronts on two SIMDs that stream the same Q / dO tiles from LDS:
//   wavefront A ("P"):   S = Q K^T,  P = 2^(c S - lse2),            dV^T += dO^T P
//   wavefront B ("dS"):  dP = dO V^T - delta,  dS = P (dP - delta),  dK^T += Q^T dS
// A hands P over as the bf16 operand fragments it feeds to its own dV product, through a
// double-buffered 4 KB LDS slot; B runs one sub-tile (32 query rows) behind A, so a slot is
// written in one iteration and read in the next, with the workgroup's barrier between them.  A
// workgroup is two such pairs = 128 keys of one (sequence | chunk of token rows, KV head).
//
// Everything else follows the other backward kernels: Q / dO tiles of 64 rows go straight to LDS
// (direct loads, four buffers), each iteration is 32 fenced groups of one matrix-core instruction
// plus its share of LDS reads and vector-ALU work, tiles that need no mask run through a loop
// without masking code, and prefix-slot gradients leave as fp32 partials per chunk of token rows.
#include "attn_bwd_dq.h"

namespace cart {
using namespace mfma;

constexpr int KV_TILE = 64;                       // token rows per LDS tile (two sub-tiles of 32)
constexpr int KV_TILE_B = KV_TILE * ROW_B;
constexpr int KV_NBUF = 4;
constexpr int KV_BUF_B = 2 * KV_TILE_B;           // one buffer: Q tile, dO tile
constexpr int KV_G_OFF = KV_TILE_B;               // dO tile inside a buffer
constexpr int KV_WG_KEYS = 128;                   // keys per workgroup: two pairs of wavefronts x 64
constexpr int KV_SLOT_B = 4096;                   // P of one sub-tile for 64 keys: 4 fragments x 64 lanes x 16 B
constexpr int KV_MIN_CHUNK = 128;                 // fewest token rows per dZ partial

struct KvSmem {
    struct { char q[KV_TILE_B]; char g[KV_TILE_B]; } t[KV_NBUF];
    float nl2[KV_NBUF][KV_TILE];
    float ndl[KV_NBUF][KV_TILE];
    char slot[2][2][KV_SLOT_B];                   // [pair][sub-tile parity]
};

// One LDS block for the workgroup, at file scope: the two roles are separate (not inlined)
// functions, each with a register allocation of its own, that address the same memory.
__shared__ union BwdSmem {
    KvSmem kv;
    DqSmem dq;
} bwd_sm;

// The workgroup barrier without the wait for every outstanding LDS and memory operation that
// __syncthreads() puts in front of it: in the hot loop a wavefront only has to have finished what
// the OTHER wavefronts are about to depend on (A: its direct-to-LDS loads and its P-slot writes;
// B: nothing), and fragment loads for later iterations stay in flight across the barrier.
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }
__device__ __forceinline__ void lds_wait0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// The kernels' arguments (KvArgs and what the one-launch form adds).  The role functions are real calls, and a call passes
// its arguments in vector registers; they get one pointer -- the kernel-argument segment, taken in the kernel itself
// (the builtin that returns it is only meaningful there: inside a called function it yields a null
// pointer) -- make it wave-uniform again and read this block through the scalar cache, so that
// every pointer and size stays in scalar registers.
struct BwdArgs {
    KvArgs kv;
    DqArgs dq;
    unsigned n_front, n_dq;             // workgroups: key-side ones ahead of dQ's, dQ's
    QuerySplit split;
};
#if defined(__HIP_DEVICE_COMPILE__)
#define CART_KERNARG(T) const __attribute__((address_space(4))) T
#else
#define CART_KERNARG(T) const T         // (host pass: never runs)
#endif
template <typename T>
__device__ __forceinline__ CART_KERNARG(T)* kernarg(const T* generic) {
    const uint64_t u = reinterpret_cast<uint64_t>(generic);
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u >> 32)));
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u)));
    return (CART_KERNARG(T)*)((static_cast<uint64_t>(hi) << 32) | static_cast<uint64_t>(lo));
}

// A called function saves the callee-saved half of its registers on entry and reads it back on return:
// 240 of them a wavefront, 240 KB a workgroup out and in again through scratch memory.  The compiler
// drops that for a function of internal linkage whose calls are not marked as tail calls (it then knows
// that the kernel holds nothing across the call), hence `static` and the attribute.
// One sequence of 700 tokens, 32 / 8 heads, 1000 slots: 135 -> 127 us for forward and backward; 64 packed
// conversations of up to 1024: 10.17 -> 10.00 ms; 16 x 2048 over 4096 slots: 9.81 -> 9.71.
template <bool roleB>
[[clang::not_tail_called]] static __device__ __attribute__((noinline)) void kv_role(const KvArgs* args, int block) {
    const KvArgs a = *kernarg(args);
    const bf16_t* __restrict__ q = a.q; const bf16_t* __restrict__ k = a.k; const bf16_t* __restrict__ v = a.v;
    const bf16_t* __restrict__ zk = a.zk; const bf16_t* __restrict__ zv = a.zv; const bf16_t* __restrict__ d_o = a.d_o;
    const float* __restrict__ nlse2 = a.nlse2; const float* __restrict__ ndelta = a.ndelta;
    bf16_t* __restrict__ dk_own = a.dk_own; bf16_t* __restrict__ dv_own = a.dv_own;
    float* __restrict__ part_k = a.part_k; float* __restrict__ part_v = a.part_v;
    const int32_t* __restrict__ cu = a.cu;
    const int n_tok = a.n_tok, chunk = a.chunk, Smax = a.Smax, Hq = a.Hq, Hkv = a.Hkv, P = a.P;
    const float c = a.c, scale = a.scale;
    KvSmem& sm = bwd_sm.kv;
    const int G = Hq / Hkv;
    const int nPb = (P + KV_WG_KEYS - 1) / KV_WG_KEYS, nOb = (Smax + KV_WG_KEYS - 1) / KV_WG_KEYS;
    // workgroup -> (KV head, key block, chunk of token rows | sequence and part of the heads): KV head
    // fastest; the prefix blocks (long streams: every token row of a chunk, all G heads) first
    int id = __builtin_amdgcn_readfirstlane(block);
    const int hk = id % Hkv; id /= Hkv;
    int kb_, b_, g0 = 0, g1 = G;
    SeqSpan sp;
    const int nChunk = (n_tok + chunk - 1) / chunk;
    if (id < nPb * nChunk) {
        kb_ = id % nPb;
        b_ = id / nPb;
        sp.t0 = static_cast<size_t>(b_) * chunk;
        sp.len = min(chunk, n_tok - b_ * chunk);
        sp.stat_b = sp.stat_h = 0;
    } else {
        id -= nPb * nChunk;
        kb_ = nPb + (a.own_cols ? id / a.own_cols : id % nOb);
        id = a.own_cols ? id % a.own_cols : id / nOb;
        b_ = id / a.head_parts;
        g0 = (id % a.head_parts) * (G / a.head_parts);
        g1 = g0 + G / a.head_parts;
        sp = seq_span(cu, b_, n_tok, Smax, Hq);
    }
    const int kb = kb_, b = b_;      // for a prefix block b is the chunk
    const bool pre = kb < nPb;
    const int key0 = (pre ? kb : kb - nPb) * KV_WG_KEYS;
    const int S = sp.len;
    const size_t t0 = sp.t0;
    const int nkeys = pre ? P : S;
    const int lane = threadIdx.x & 63, lg = lane >> 5, lc = lane & 31;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pair = wv >> 1;
    const int wkey0 = key0 + 64 * pair;
    if (!pre && key0 >= S) return;

    // this wavefront's 64 keys as B operands (column = key, k = head element): K for A, V for B
    u32x4 sf[2][8];
    auto load_keys = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int kc = 0; kc < 2; ++kc) {
            const int key = min(wkey0 + 32 * kc + lc, nkeys - 1);
            const size_t row = pre ? static_cast<size_t>(hk) * P + key : (t0 + key) * Hkv + hk;
            const bf16_t* sp_ = (roleB ? (pre ? zv : v) : (pre ? zk : k)) + row * HD + 8 * lg;
#pragma unroll
            for (int t = 0; t < 8; ++t) sf[kc][t] = *reinterpret_cast<const u32x4*>(sp_ + 16 * t);
        }
    };
    f32x16 acc[4][2];   // dV^T (A) or dK^T (B): [head-element block][key block]
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int kc = 0; kc < 2; ++kc)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][kc][r] = 0.f;
    auto pin = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int kc = 0; kc < 2; ++kc)
#pragma unroll
            for (int t = 0; t < 8; ++t) asm volatile("" : "+a"(sf[kc][t]));
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int kc = 0; kc < 2; ++kc) asm volatile("" : "+a"(acc[db][kc]));
    };

    // The stream of query tiles (64 token rows of one head): per head the whole tiles entirely
    // after the block's last key need no mask, the tiles on the diagonal and the ragged last tile
    // do.  Order: the unmasked tiles of every head, then the masked tiles of every head.
    const int nQtAll = (S + KV_TILE - 1) / KV_TILE, nFullEnd = S / KV_TILE;
    const int qt0 = pre ? 0 : key0 / KV_TILE;
    const int qtF0 = pre ? 0 : qt0 + KV_WG_KEYS / KV_TILE;
    const int nFull = max(0, nFullEnd - qtF0);
    const int nM1 = min(qtF0, nQtAll) - qt0;
    const int nM = nM1 + ((nFullEnd < nQtAll && nFullEnd >= qtF0) ? 1 : 0);
    const int nG = g1 - g0, nMain = nG * nFull, nT = nG * (nFull + nM);
    const char* q_c = reinterpret_cast<const char*>(q);
    const char* g_c = reinterpret_cast<const char*>(d_o);
    const uint32_t q_pitch = static_cast<uint32_t>(Hq) * ROW_B;
    int it_ph = nFull > 0 ? 0 : 1, it_g = 0, it_n = 0, it_cnt = 0;
    struct TileSrc { const char* qb; const char* gb; const char* rb; int lim; int i0; uint32_t lds_q, lds_g, lds_r; };
    const uint32_t dma_c0 = (lane & 15) ^ (((lane >> 4) & 3) << 2);
    auto next_tile = [&](int buf) __attribute__((always_inline)) {
        const int qt = it_ph == 0 ? qtF0 + it_n : (it_n < nM1 ? qt0 + it_n : nFullEnd);
        const int h = hk * G + g0 + it_g;
        TileSrc ts;
        ts.i0 = qt * KV_TILE;
        const size_t base = (t0 * Hq + h) * ROW_B + static_cast<size_t>(ts.i0) * q_pitch;
        ts.qb = q_c + base;
        ts.gb = g_c + base;
        ts.lim = S - 1 - ts.i0;
        ts.rb = reinterpret_cast<const char*>((pair ? ndelta : nlse2) + static_cast<size_t>(h) * n_tok + t0 + ts.i0);
        ts.lds_q = lds_addr(sm.t[buf].q);
        ts.lds_g = lds_addr(sm.t[buf].g);
        ts.lds_r = lds_addr(pair ? sm.ndl[buf] : sm.nl2[buf]);
        if (it_cnt < nT - 1) {     // past the end the last tile is fetched again, into a retired buffer
            ++it_cnt;
            ++it_n;
            if (it_n == (it_ph == 0 ? nFull : nM)) {
                it_n = 0;
                if (++it_g == nG) { it_g = 0; ++it_ph; }
            }
        }
        return ts;
    };
    // Direct-to-LDS loads of a tile, all issued by the two A wavefronts (B is the busier role):
    // seventeen each -- 8 x 4 Q rows, 8 x 4 dO rows of the wavefront's half of the tile, and one
    // of the two row-value arrays (pair 0: -lse2, pair 1: -delta).
    auto dma_piece = [&](const TileSrc& ts, int n) __attribute__((always_inline)) {
        if (n == 16) {
            dma4(ts.rb, static_cast<uint32_t>(min(lane, ts.lim)) * 4u, ts.lds_r);
            return;
        }
        const int i = n & 7;
        const int r0 = (8 * pair + i) * 4;
        const uint32_t voff = __umul24(min(r0 + (lane >> 4), ts.lim), q_pitch) + ((dma_c0 ^ (i & 3)) << 4);
        if (n < 8) dma16(ts.qb, voff, ts.lds_q + r0 * ROW_B);
        else       dma16(ts.gb, voff, ts.lds_g + r0 * ROW_B);
    };
    constexpr int KV_DMA = 17, KV_DMA0 = 9;      // pieces per tile; how many of them ride in the first half

    const uint32_t fwd = static_cast<uint32_t>(KV_BUF_B), back = static_cast<uint32_t>(-(KV_NBUF - 1) * KV_BUF_B);
    const uint32_t rfwd = static_cast<uint32_t>(KV_TILE * 4), rback = static_cast<uint32_t>(-(KV_NBUF - 1) * KV_TILE * 4);
    const uint32_t slot0 = lds_addr(sm.slot[pair][0]) + lane * 16;     // fragment f of parity s: + s * SLOT_B + f * 1024

    // The wavefront's 64 rows of dV (A) or dK (B), turned around in LDS (32 KB each, the tile buffers)
    // once every wavefront is done with them; A waits for its direct-to-LDS loads first.
    auto kv_store = [&]() __attribute__((always_inline)) {
        __syncthreads();
        char* const turn = reinterpret_cast<char*>(&sm.t[wv]);
        const float mul = roleB ? scale : 1.f;
        float* const part = roleB ? part_k : part_v;
        float* const own_part = roleB ? a.own_k : a.own_v;
        bf16_t* const own = roleB ? dk_own : dv_own;
        if (pre && wkey0 < a.n_frozen) {        // (zeros, whatever the gradient is)
#pragma unroll
            for (int kc = 0; kc < 2; ++kc)
                if (wkey0 + 32 * kc + lc < a.n_frozen) {
#pragma unroll
                    for (int db = 0; db < 4; ++db)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[db][kc][r] = 0.f;
                }
        }
        if (pre)
            store_rows64(turn, acc, mul, mul, part + ((static_cast<size_t>(b) * Hkv + hk) * P + wkey0) * HD, HD, P - wkey0, lane);
        else if (a.head_parts > 1)
            store_rows64(turn, acc, mul, mul, own_part + ((static_cast<size_t>(g0 / nG) * n_tok + t0 + wkey0) * Hkv + hk) * HD,
                         static_cast<size_t>(Hkv) * HD, S - wkey0, lane);
        else
            store_rows64(turn, acc, mul, mul, own + ((t0 + wkey0) * Hkv + hk) * HD, static_cast<size_t>(Hkv) * HD, S - wkey0, lane);
    };

    if constexpr (!roleB) {
        // =========================================================================================
        // A: S, P, dV.  Iteration u (half hb of tile T): on entry xin = S(u), qa = row-wise Q
        // fragments of sub-tile u+1, nl = -lse2 of sub-tile u, ta = transposed dO fragments of
        // sub-tile u-1, xf = P(u-1).  Matrix cores: S(u+1) (groups 0-15), dV^T += dO^T P(u-1)
        // (groups 16-31); vector ALU: P(u), which goes to the pair's slot at the end.
        // =========================================================================================
        uint32_t qofs[8], tofs[4][2], rofs, rofs_c;
        {
            const uint32_t t1 = lds_addr(sm.t[1].q), tg0 = lds_addr(sm.t[0].g);
#pragma unroll
            for (int t8 = 0; t8 < 8; ++t8) qofs[t8] = t1 + frag_n_ofs(lane, t8);
#pragma unroll
            for (int db = 0; db < 4; ++db) {
                frag_t_ofs(lane, db, tofs[db][0], tofs[db][1]);
                tofs[db][0] += tg0;
                tofs[db][1] += tg0;
            }
            rofs = lds_addr(&sm.nl2[1][4 * lg]);
            rofs_c = lds_addr(&sm.nl2[0][4 * lg]);
        }
        auto ld_q = [&](int t8, int hb) __attribute__((always_inline)) { return lds_ld_frag(qofs[t8] + hb * 32 * ROW_B); };
        auto ld_t = [&](int p, int hb) __attribute__((always_inline)) {
            const int ks = p >> 2, db = p & 3;
            return lds_ld_frag_t(tofs[db][0] + (32 * hb + 16 * ks) * ROW_B, tofs[db][1] + (32 * hb + 16 * ks) * ROW_B);
        };
        auto ld_rows_at = [&](f32x16& d, uint32_t base, int hb) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4 w = lds_ld_f32x4(base + (32 * hb + 8 * j) * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) d[4 * j + e] = w[e];
            }
        };
        // a query row of the sub-tile starting at token i0 is hidden from a key when it precedes
        // it (own keys) or lies past the end of the sequence (clamped tile rows)
        auto mask1 = [&](f32x16& x, int kc, int i0) __attribute__((always_inline)) {
            mask_below(x, (pre ? 0 : wkey0 + 32 * kc + lc) - i0 - 4 * lg);
            mask_above(x, S - 1 - i0 - 4 * lg);
        };
        u32x4 xf[2][2];
#pragma unroll
        for (int kc = 0; kc < 2; ++kc)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) xf[kc][ks] = u32x4{0u, 0u, 0u, 0u};
        bf16x8 qa[8], ta[6];
        f32x16 nl, nl_n;
        f32x16 xa[2], xb[2];

        // The last two transposed fragments have a spare register set each (tb6 / tb7, indexed by
        // the parity of the iteration that USES them), so that the next iteration's copies can be
        // requested before this iteration's last use: nothing is issued to LDS in the last
        // groups, and the wait in front of the barrier finds (almost) nothing outstanding.
        bf16x8 tb6[2], tb7[2];
        auto stage = [&](auto hb_tag, auto masked_tag, int i0, f32x16 (&xin)[2], f32x16 (&xout)[2], const TileSrc& ts,
                         uint32_t wslot) __attribute__((always_inline)) {
            constexpr int hb = decltype(hb_tag)::value;
            constexpr bool MASKED = decltype(masked_tag)::value;
            if (MASKED) { mask1(xin[0], 0, i0 + 32 * hb); mask1(xin[1], 1, i0 + 32 * hb); }
            pin();
            float pe[32];
            u32x4 xn[2][2];
            auto elem = [&](int e) __attribute__((always_inline)) {
                pe[e] = fast_exp2(fmaf(xin[e >> 4][e & 15], c, nl[e & 15]));
            };
            auto pack2 = [&](int e) __attribute__((always_inline)) {     // elements e, e+1 -> their word of P(u)
                xn[e >> 4][(e & 15) >> 3][(e & 7) >> 1] = pack_bf16x2(pe[e], pe[e + 1]);
            };
            auto put = [&](int f) __attribute__((always_inline)) {       // fragment f of P(u) -> the pair's slot
                *(u32x4 __attribute__((address_space(3)))*)(wslot + f * 1024) = xn[f >> 1][f & 1];
            };
            static_for<32>([&](auto gc) __attribute__((always_inline)) {
                constexpr int g = decltype(gc)::value;
                if (g < 16) {
                    const int t8 = g >> 1, kc = g & 1;
                    if (t8 == 0) mma_vd_zero(xout[kc], qa[0], sf[kc][0]);
                    else         mma_vd(xout[kc], qa[t8], sf[kc][t8]);
                } else {
                    const int i = g - 16, ks = i >> 3, db = (i >> 1) & 3, kc = i & 1, pf = 4 * ks + db;
                    const bf16x8 tf = pf == 6 ? tb6[hb] : pf == 7 ? tb7[hb] : ta[pf];
                    acc[db][kc] = mma(tf, __builtin_bit_cast(bf16x8, xf[kc][ks]), acc[db][kc]);
                }
                __builtin_amdgcn_sched_barrier(0);   // the matrix-core instruction leads its group
                if (hb == 0 && g < KV_DMA0) dma_piece(ts, g);
                if (hb == 1 && g < KV_DMA - KV_DMA0) dma_piece(ts, KV_DMA0 + g);
                if (g == 20) ld_rows_at(nl_n, hb ? rofs : rofs_c, 1 - hb);                 // -lse2 of sub-tile u+1
                if (g >= 2 && g <= 16 && !(g & 1)) qa[(g - 2) >> 1] = ld_q((g - 2) >> 1, hb);   // of sub-tile u+2
                if (g >= 18 && g <= 28 && !(g & 1)) ta[(g - 18) >> 1] = ld_t((g - 18) >> 1, hb);   // of sub-tile u
                if (g == 25) tb6[1 - hb] = ld_t(6, hb);
                if (g == 27) tb7[1 - hb] = ld_t(7, hb);
                // P(u) leaves for the pair's slot fragment by fragment, as soon as each is complete
                if (g == 9) put(0);
                if (g == 17) put(1);
                if (g == 21) put(2);
                if (g == 29) put(3);
                __builtin_amdgcn_sched_barrier(0);   // LDS traffic first, then the vector ALU work
                // P(u): one element per group, two in groups 16-19, so that the last fragment is
                // complete four groups before the iteration ends
                if (g < 16) elem(g);
                else if (g < 20) { elem(2 * g - 16); elem(2 * g - 15); }
                else if (g < 28) elem(g + 4);
                if (g >= 2 && g <= 16 && !(g & 1)) pack2(g - 2);
                if (g >= 17 && g <= 20) pack2(2 * g - 18);
                if (g >= 22 && g <= 28 && !(g & 1)) pack2(g + 2);
                __builtin_amdgcn_sched_barrier(0);
            });
            nl = nl_n;
#pragma unroll
            for (int kc = 0; kc < 2; ++kc)
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) xf[kc][ks] = xn[kc][ks];
            __builtin_amdgcn_sched_barrier(0);
        };
        auto settle = [&]() __attribute__((always_inline)) { asm volatile("s_nop 15\n\ts_nop 7" ::: "memory"); };

        int i0_cur, i0_nx;
        {   // prologue: tiles 0 and 1 on their way, scores of sub-tile 0, fragments of sub-tile 1
            const TileSrc t0s = next_tile(0);
            i0_cur = t0s.i0;
#pragma unroll
            for (int n = 0; n < KV_DMA; ++n) dma_piece(t0s, n);
            const TileSrc t1s = next_tile(1);
            i0_nx = t1s.i0;
#pragma unroll
            for (int n = 0; n < KV_DMA; ++n) dma_piece(t1s, n);
            load_keys();      // (behind the tiles: one round trip to memory, not three)
            pin();
            dma_wait();
            __syncthreads();
#pragma unroll
            for (int t8 = 0; t8 < 8; ++t8) qa[t8] = lds_ld_frag(qofs[t8] - KV_BUF_B);        // sub-tile 0
            ld_rows_at(nl, rofs_c, 0);
#pragma unroll
            for (int t8 = 0; t8 < 8; ++t8) {
                if (t8 == 0) { mma_vd_zero(xa[0], qa[0], sf[0][0]); mma_vd_zero(xa[1], qa[0], sf[1][0]); }
                else         { mma_vd(xa[0], qa[t8], sf[0][t8]);    mma_vd(xa[1], qa[t8], sf[1][t8]); }
            }
            settle();
#pragma unroll
            for (int t8 = 0; t8 < 8; ++t8) qa[t8] = lds_ld_frag(qofs[t8] - KV_BUF_B + 32 * ROW_B);   // sub-tile 1
#pragma unroll
            for (int p = 0; p < 6; ++p) ta[p] = ld_t(p, 0);     // placeholder: multiplied by P = 0
            tb6[0] = ld_t(6, 0);
            tb7[0] = ld_t(7, 0);
        }
        int buf = 0;
        auto tile_iter = [&](auto masked_tag) __attribute__((always_inline)) {
            const int nbuf = buf + 1 == KV_NBUF ? 0 : buf + 1;
            const int nnbuf = nbuf + 1 == KV_NBUF ? 0 : nbuf + 1;
            const TileSrc ts = next_tile(nnbuf);
            dma_wait();       // tile T+1 has landed,
            lds_wait0();      // the last P went into its slot,
            wg_barrier();     // and everybody knows
            stage(std::integral_constant<int, 0>{}, masked_tag, i0_cur, xa, xb, ts, slot0);
            lds_wait0();
            wg_barrier();
            stage(std::integral_constant<int, 1>{}, masked_tag, i0_cur, xb, xa, ts, slot0 + KV_SLOT_B);
#pragma unroll
            for (int db = 0; db < 4; ++db) {                 // tile T -> T+1
                tofs[db][0] += nbuf == 0 ? back : fwd;
                tofs[db][1] += nbuf == 0 ? back : fwd;
            }
#pragma unroll
            for (int t8 = 0; t8 < 8; ++t8) qofs[t8] += nnbuf == 0 ? back : fwd;   // tile T+1 -> T+2
            rofs += nnbuf == 0 ? rback : rfwd;
            rofs_c += nbuf == 0 ? rback : rfwd;
            buf = nbuf;
            i0_cur = i0_nx;
            i0_nx = ts.i0;
        };
        for (int ti = 0; ti < nMain; ++ti) tile_iter(std::false_type{});
        for (int ti = nMain; ti < nT; ++ti) tile_iter(std::true_type{});
        __syncthreads();      // B's last iteration: publishes the last P
        {   // drain: the last sub-tile's contribution
            pin();
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int db = 0; db < 4; ++db) {
                    const int pf = 4 * ks + db;
                    const bf16x8 tf = pf == 6 ? tb6[0] : pf == 7 ? tb7[0] : ta[pf];
                    acc[db][0] = mma(tf, __builtin_bit_cast(bf16x8, xf[0][ks]), acc[db][0]);
                    acc[db][1] = mma(tf, __builtin_bit_cast(bf16x8, xf[1][ks]), acc[db][1]);
                }
        }
        dma_wait();
        kv_store();
    } else {
        // =========================================================================================
        // B: dP, dS, dK, one sub-tile behind A.  Iteration u: on entry yin = dP(u-1) - delta,
        // ga = row-wise dO fragments of sub-tile u, nd = -delta of sub-tile u, ta = transposed Q
        // fragments of sub-tile u-2, xf = dS(u-2); the slot of parity (u-1) holds P(u-1).
        // Matrix cores: dP(u) (groups 0-15), dK^T += Q^T dS(u-2) (groups 16-31); vector ALU:
        // dS(u-1) = P(u-1) (dP(u-1) - delta).
        // =========================================================================================
        uint32_t gofs[8], tofs[4][2], rofs;
        {
            const uint32_t tq0 = lds_addr(sm.t[0].q), tg0 = lds_addr(sm.t[0].g);
#pragma unroll
            for (int t8 = 0; t8 < 8; ++t8) gofs[t8] = tg0 + frag_n_ofs(lane, t8);
#pragma unroll
            for (int db = 0; db < 4; ++db) {
                frag_t_ofs(lane, db, tofs[db][0], tofs[db][1]);
                tofs[db][0] += tq0;
                tofs[db][1] += tq0;
            }
            rofs = lds_addr(&sm.ndl[0][4 * lg]);
        }
        auto ld_g = [&](int t8, int half) __attribute__((always_inline)) { return lds_ld_frag(gofs[t8] + half * 32 * ROW_B); };
        auto ld_t = [&](int p, int half) __attribute__((always_inline)) {
            const int ks = p >> 2, db = p & 3;
            return lds_ld_frag_t(tofs[db][0] + (32 * half + 16 * ks) * ROW_B, tofs[db][1] + (32 * half + 16 * ks) * ROW_B);
        };
        auto ld_rows = [&](f32x16& d, int half) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4 w = lds_ld_f32x4(rofs + (32 * half + 8 * j) * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) d[4 * j + e] = w[e];
            }
        };
        u32x4 xf[2][2];
#pragma unroll
        for (int kc = 0; kc < 2; ++kc)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) xf[kc][ks] = u32x4{0u, 0u, 0u, 0u};
        bf16x8 ga[8], ta[8];
        f32x16 nd;
        f32x16 ya[2], yb[2];
#pragma unroll
        for (int kc = 0; kc < 2; ++kc)
#pragma unroll
            for (int r = 0; r < 16; ++r) ya[kc][r] = 0.f;      // "dP(-1)": multiplied by P(-1) = 0
        // P(-1) = 0 in the slot the first iteration reads (parity 1)
#pragma unroll
        for (int f = 0; f < 4; ++f)
            *(u32x4 __attribute__((address_space(3)))*)(slot0 + KV_SLOT_B + f * 1024) = u32x4{0u, 0u, 0u, 0u};

        // vector ALU part: dS(u-1) from the P fragments pw and yin; element e of 32
        auto ds_elem = [&](const u32x4 (&pw)[4], const f32x16 (&yin)[2], float (&w)[32], int e) __attribute__((always_inline)) {
            const int kc = e >> 4, r = e & 15;
            const uint32_t word = pw[2 * kc + (r >> 3)][(r & 7) >> 1];
            const float p = (r & 1) ? __uint_as_float(word & 0xffff0000u) : __uint_as_float(word << 16);
            w[e] = p * yin[kc][r];
        };
        // stage: `half` of the row-wise / row-value reads (sub-tile u+1) and `thalf` of the
        // transposed reads (sub-tile u-1) are fixed per call site
        auto stage = [&](auto hb_tag, f32x16 (&yin)[2], f32x16 (&yout)[2], uint32_t rslot) __attribute__((always_inline)) {
            constexpr int hb = decltype(hb_tag)::value;
            constexpr int half = 1 - hb;        // sub-tile u+1 is half 1 of tile T (hb 0) or half 0 of tile T+1 (hb 1)
            constexpr int thalf = 1 - hb;       // sub-tile u-1 is half 1 of tile T-1 (hb 0) or half 0 of tile T (hb 1)
            pin();
            u32x4 pw[4];
#pragma unroll
            for (int f = 0; f < 4; ++f) pw[f] = *(const u32x4 __attribute__((address_space(3)))*)(rslot + f * 1024);
            float w[32];
            u32x4 xn[2][2];
            static_for<32>([&](auto gc) __attribute__((always_inline)) {
                constexpr int g = decltype(gc)::value;
                if (g < 16) {
                    const int t8 = g >> 1, kc = g & 1;
                    if (t8 == 0) mma_vd_first(yout[kc], ga[0], sf[kc][0], nd);
                    else         mma_vd(yout[kc], ga[t8], sf[kc][t8]);
                } else {
                    const int i = g - 16, ks = i >> 3, db = (i >> 1) & 3, kc = i & 1;
                    acc[db][kc] = mma(ta[4 * ks + db], __builtin_bit_cast(bf16x8, xf[kc][ks]), acc[db][kc]);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (g == 20) ld_rows(nd, half);                                                   // -delta of sub-tile u+1
                if (g >= 2 && g <= 16 && !(g & 1)) ga[(g - 2) >> 1] = ld_g((g - 2) >> 1, half);   // of sub-tile u+1
                if (g >= 18 && !(g & 1)) ta[(g - 18) >> 1] = ld_t((g - 18) >> 1, thalf);          // of sub-tile u-1
                __builtin_amdgcn_sched_barrier(0);
                // dS(u-1): element g-4 from group 4 on (the P fragments were requested at the
                // top), the last four elements double up in the last four groups
                if (g >= 4) ds_elem(pw, yin, w, g - 4);
                if (g >= 28) ds_elem(pw, yin, w, g);
                if (g >= 6 && !(g & 1)) {
                    const int e = g - 6;
                    xn[e >> 4][(e & 15) >> 3][(e & 7) >> 1] = pack_bf16x2(w[e], w[e + 1]);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            ta[7] = ld_t(7, thalf);
            xn[1][1][1] = pack_bf16x2(w[26], w[27]);
            xn[1][1][2] = pack_bf16x2(w[28], w[29]);
            xn[1][1][3] = pack_bf16x2(w[30], w[31]);
#pragma unroll
            for (int kc = 0; kc < 2; ++kc)
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) xf[kc][ks] = xn[kc][ks];
            __builtin_amdgcn_sched_barrier(0);
        };

        load_keys();
        pin();
        {   // prologue: A's barrier publishes tile 0; fragments and row values of sub-tile 0
            __syncthreads();
#pragma unroll
            for (int t8 = 0; t8 < 8; ++t8) ga[t8] = ld_g(t8, 0);
            ld_rows(nd, 0);
#pragma unroll
            for (int p = 0; p < 8; ++p) ta[p] = ld_t(p, 0);     // placeholder: multiplied by dS = 0
        }
        int buf = 0;
        bool first = true;
        auto tile_iter = [&]() __attribute__((always_inline)) {
            const int nbuf = buf + 1 == KV_NBUF ? 0 : buf + 1;
            const int nnbuf = nbuf + 1 == KV_NBUF ? 0 : nbuf + 1;
            wg_barrier();
            // first half: reads P of the previous tile's second sub-tile (parity 1)
            stage(std::integral_constant<int, 0>{}, ya, yb, slot0 + KV_SLOT_B);
            // between the halves the row-wise reads move on to tile T+1 and the transposed reads
            // to tile T (the first tile has no predecessor: they already sit on tile 0)
#pragma unroll
            for (int t8 = 0; t8 < 8; ++t8) gofs[t8] += nbuf == 0 ? back : fwd;
            rofs += nbuf == 0 ? rback : rfwd;
            if (!first) {
#pragma unroll
                for (int db = 0; db < 4; ++db) {
                    tofs[db][0] += buf == 0 ? back : fwd;
                    tofs[db][1] += buf == 0 ? back : fwd;
                }
            }
            wg_barrier();
            stage(std::integral_constant<int, 1>{}, yb, ya, slot0);
            first = false;
            buf = nbuf;
        };
        for (int ti = 0; ti < nT; ++ti) tile_iter();
        __syncthreads();
        {   // tail: dS of the last sub-tile, then the two outstanding dK products
            pin();
            u32x4 pw[4];
#pragma unroll
            for (int f = 0; f < 4; ++f) pw[f] = *(const u32x4 __attribute__((address_space(3)))*)(slot0 + KV_SLOT_B + f * 1024);
            // dK^T += Q^T dS(u-2): fragments of that sub-tile are in registers
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int db = 0; db < 4; ++db) {
                    acc[db][0] = mma(ta[4 * ks + db], __builtin_bit_cast(bf16x8, xf[0][ks]), acc[db][0]);
                    acc[db][1] = mma(ta[4 * ks + db], __builtin_bit_cast(bf16x8, xf[1][ks]), acc[db][1]);
                }
            float w[32];
#pragma unroll
            for (int e = 0; e < 32; ++e) ds_elem(pw, ya, w, e);
#pragma unroll
            for (int e = 0; e < 32; e += 2) xf[e >> 4][(e & 15) >> 3][(e & 7) >> 1] = pack_bf16x2(w[e], w[e + 1]);
            // the last sub-tile is the second half of the last tile, where the transposed reads sit
#pragma unroll
            for (int p = 0; p < 8; ++p) ta[p] = ld_t(p, 1);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int db = 0; db < 4; ++db) {
                    acc[db][0] = mma(ta[4 * ks + db], __builtin_bit_cast(bf16x8, xf[0][ks]), acc[db][0]);
                    acc[db][1] = mma(ta[4 * ks + db], __builtin_bit_cast(bf16x8, xf[1][ks]), acc[db][1]);
                }
        }
        kv_store();
    }
}

// odd wavefronts take role B, even ones role A (wave-uniform: a scalar branch)
__device__ __forceinline__ void kv_block(const KvArgs* args, int block) {
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) & 1) kv_role<true>(args, block);
    else                                                      kv_role<false>(args, block);
}
#if defined(__HIP_DEVICE_COMPILE__)
#define CART_ARGS_PTR(T, args) (const T*)__builtin_amdgcn_kernarg_segment_ptr()       // = &args, the first argument
#else
#define CART_ARGS_PTR(T, args) &args
#endif
__global__ __launch_bounds__(256, 1) void attn_bwd_kv_kernel(KvArgs args) { kv_block(CART_ARGS_PTR(KvArgs, args), blockIdx.x); }

// dQ beside dK and dV: a workgroup of either fills a CU, and apart each launch leaves CUs idle in its last round -- or, of
// a problem with fewer blocks than CUs, for its whole length.  The longest blocks first: prefix blocks, own-key blocks with
// more rows behind them than a dQ block has keys, dQ's, the other own-key blocks.
[[clang::not_tail_called]] static __device__ __attribute__((noinline)) void dq_role(const BwdArgs* args, int block) {
    CART_KERNARG(BwdArgs)* const ap = kernarg(args);
    const DqArgs a = ap->dq;
    const int id = __builtin_amdgcn_readfirstlane(block), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int G = a.Hq / a.Hkv, hk = id % a.Hkv, x = id / a.Hkv, e_full = ap->split.e_full;
    const uint32_t it = x < e_full ? 0x10000u : ap->split.part[x - e_full];
    QueryBlock qb = query_block_of(hk, x < e_full ? x : e_full + (it & 255), wv, query_wgs(a.Smax, G), G);
    qb.part = (it >> 8) & 255;
    qb.n_parts = it >> 16;
    qb.slot = (x - e_full) * a.Hkv + hk;
    dq_block<false>(a, qb, reinterpret_cast<char*>(&bwd_sm), lds_addr(&bwd_sm));
}
__global__ __launch_bounds__(256, 1) void attn_bwd_both_kernel(BwdArgs args) {
    const BwdArgs* const ap = CART_ARGS_PTR(BwdArgs, args);
    const unsigned id = blockIdx.x, n_front = args.n_front, n_dq = args.n_dq;
    if (id < n_front || id >= n_front + n_dq) kv_block(&ap->kv, id < n_front ? id : id - n_dq);
    else                                      dq_role(ap, id - n_front);
}

// -lse log2(e) and -delta = -dO . O of every (token, head), [Hq][all token rows]: 16 lanes a row, 64 tokens of one head a
// workgroup, heads fastest (they are next to each other in memory).  S: tokens per lse row
__global__ __launch_bounds__(256) void attn_bwd_stats_kernel(const bf16_t* __restrict__ o, const bf16_t* __restrict__ d_o,
                                                             const float* __restrict__ lse, float* __restrict__ nlse2,
                                                             float* __restrict__ ndelta, int n_tok, int S, int Hq) {
    const int id = workgroup_id(), h = id % Hq, i0 = id / Hq * 64 + (threadIdx.x >> 6) * 16 + ((threadIdx.x & 63) >> 4);
    const int c = threadIdx.x & 15;
    u32x4 ow[4], gw[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const size_t row = (static_cast<size_t>(min(i0 + 4 * r, n_tok - 1)) * Hq + h) * HD + 8 * c;
        ow[r] = *reinterpret_cast<const u32x4*>(o + row);
        gw[r] = *reinterpret_cast<const u32x4*>(d_o + row);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float x = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x = fmaf(__uint_as_float(ow[r][e] << 16), __uint_as_float(gw[r][e] << 16), x);
            x = fmaf(__uint_as_float(ow[r][e] & 0xffff0000u), __uint_as_float(gw[r][e] & 0xffff0000u), x);
        }
#pragma unroll
        for (int m = 8; m > 0; m >>= 1) x += __shfl_xor(x, m, 16);
        const int i = i0 + 4 * r;
        if (c == 0 && i < n_tok) {
            const size_t st = static_cast<size_t>(h) * n_tok + i;
            ndelta[st] = -x;
            nlse2[st] = -lse[(static_cast<size_t>(i / S) * Hq + h) * S + i % S] * CART_LOG2E;
        }
    }
}

// How the key-stationary launch is cut: token rows per dZ partial (prefix blocks stream chunks of the
// token rows, every head of the group), parts of the heads for own-key blocks (they stream the rows from
// their first key on).  The cheapest by playing each cut through, one KV head's workgroups on its
// share of the CUs, in launch order: a workgroup costs KV_BLOCK_US and, per 64 query rows, 1.4 us
// while most of the chip idles and 1.8 us when it is full (the clock follows the load); partials cost
// their way through memory.  Measured, a whole backward call (us), chunks n / parts of the heads h:
//   B 1  S 700  32 / 8 heads P 1000   n1/h1 117  n2/h1 122  n2/h2  96  n3/h2 113
//   B 4  S 200   8 / 2 heads P 300    n1/h1 107  n4/h1  65  n8/h2  55  n12/h4 53
//   B 16 S 256  32 / 8 heads P 1024   n1/h1 465  n2/h1 308  n3/h1 281  n4/h1 296
//   B 2  S 1024 32 / 8 heads P 2048   n1/h1 308  n2/h1 342  n3/h1 327  n1/h2 314
//   B 1  S 2048 32 / 8 heads P 8192   n1/h1 992  n1/h2 925  n2/h1 1043
//   B 3  S 1659 32 / 8 heads P 723    n1/h1 616  n2/h1 459  n3/h1 512  n6/h1 473
constexpr float KV_BLOCK_US = 10.f, KV_LIGHT_US = 1.4f, KV_FULL_US = 1.8f, KV_US_PER_MB = 0.6f;
constexpr int KV_MAX_CUS = 256;
constexpr int KV_MAX_CHUNKS = 32;
// Partials beyond the first chunk's: 192 MB at most (the cheapest cuts of 6000 problems of up to 8192 slots had
// 178 at most, 99.8 % of them 128)
constexpr size_t KV_MOST_EXTRA = static_cast<size_t>(192) << 20;
static size_t kv_chunk_bytes(const cart_attn_desc& d) { return 2 * static_cast<size_t>(d.Hkv) * d.P * HD * sizeof(float); }
static size_t kv_own_bytes(const cart_attn_desc& d, long tokens, int head_parts) {
    return head_parts > 1 ? 2 * static_cast<size_t>(head_parts) * tokens * d.Hkv * HD * sizeof(float) : 0;
}
// bytes of the partials at their most, for this problem or any smaller one
size_t bwd_kv_most(const cart_attn_desc& d, long tokens) {
    const long chunks = (tokens + KV_MIN_CHUNK - 1) / KV_MIN_CHUNK;
    const size_t extra = static_cast<size_t>((chunks < KV_MAX_CHUNKS ? chunks : KV_MAX_CHUNKS) - 1) * kv_chunk_bytes(d) +
                         kv_own_bytes(d, tokens, d.Hq / d.Hkv);
    return kv_chunk_bytes(d) + (extra < KV_MOST_EXTRA ? extra : KV_MOST_EXTRA);
}

// the partials' way through memory
static float kv_parts_us(const cart_attn_desc& d, long tokens, const KvPlan& p) {
    return KV_US_PER_MB * 1e-6f * 2.f * HD * 4.f * static_cast<float>(d.Hkv) *
           (static_cast<float>(p.n_part) * d.P + (p.head_parts > 1 ? static_cast<float>(p.head_parts) * tokens : 0.f));
}
// The cuts that are considered: f(plan, own-key workgroups per KV head, microseconds of the partials' way)
template <typename F>
static void each_cut(const cart_attn_desc& d, long tokens, int M, F&& f) {
    const int G = d.Hq / d.Hkv, nOb = (d.S + KV_WG_KEYS - 1) / KV_WG_KEYS;
    for (int hp = 1; hp <= G; ++hp) {
        if (G % hp) continue;
        const long n_own = static_cast<long>(nOb) * d.B * hp;
        if (hp > 1 && n_own > 4L * M) break;            // (plenty of own-key workgroups as it is)
        int last = 0;
        for (int n = 1; n <= (d.P > 0 ? KV_MAX_CHUNKS : 1); n += 1 + n / 8) {
            KvPlan p;
            p.chunk = static_cast<int>((((tokens + n - 1) / n) + KV_TILE - 1) / KV_TILE * KV_TILE);
            p.n_part = static_cast<int>((tokens + p.chunk - 1) / p.chunk);
            p.head_parts = hp;
            if (p.n_part == last || (n > 1 && p.chunk < KV_MIN_CHUNK)) break;
            last = p.n_part;
            if (static_cast<size_t>(p.n_part - 1) * kv_chunk_bytes(d) + kv_own_bytes(d, tokens, hp) > KV_MOST_EXTRA) break;
            f(p, n_own, kv_parts_us(d, tokens, p));
        }
    }
}

// The times (us) of the workgroups of one KV head of a cut
struct KvTimes {
    long n_pre, n_own;
    float pre, own_tile;                // a prefix block; 64 query rows of an own-key block
    int nT, nOb, heads;
    float own(int i) const { return KV_BLOCK_US + own_tile * static_cast<float>((nT - 2 * (i % nOb)) * heads); }
    float sum(int B_hp) const {
        float t = pre * static_cast<float>(n_pre);
        for (int kb = 0; kb < nOb; ++kb) t += own(kb) * static_cast<float>(B_hp);
        return t;
    }
};
static KvTimes kv_times(const cart_attn_desc& d, const KvPlan& p) {
    KvTimes t;
    t.nT = (d.S + KV_TILE - 1) / KV_TILE;
    t.nOb = (d.S + KV_WG_KEYS - 1) / KV_WG_KEYS;
    t.heads = d.Hq / d.Hkv / p.head_parts;
    t.n_pre = static_cast<long>((d.P + KV_WG_KEYS - 1) / KV_WG_KEYS) * p.n_part;
    t.n_own = static_cast<long>(t.nOb) * d.B * p.head_parts;
    return t;
}
static void set_tiles(KvTimes& t, const cart_attn_desc& d, const KvPlan& p, float pre_tile, float own_tile) {
    t.own_tile = own_tile;
    t.pre = KV_BLOCK_US + pre_tile * static_cast<float>(p.chunk / KV_TILE * (d.Hq / d.Hkv));
}

// the cut of a launch of its own
static KvPlan search_plan(const cart_attn_desc& d, long tokens, int M) {
    KvPlan best = {};
    float best_t = 0.f;
    each_cut(d, tokens, M, [&](const KvPlan& p, long n_own, float parts_us) {
        KvTimes t = kv_times(d, p);
        const bool full_pre = 4 * t.n_pre >= 3L * M, full_own = 4 * t.n_own >= 3L * M;
        const float half = 0.5f * (KV_FULL_US + KV_LIGHT_US);
        set_tiles(t, d, p, full_pre ? KV_FULL_US : 4 * (t.n_pre + t.n_own) >= 3L * M ? half : KV_LIGHT_US,
                  full_own ? KV_FULL_US : t.n_pre % M ? half : KV_LIGHT_US);
        const long q = t.n_pre / M, r = t.n_pre % M;
        float end = t.pre * static_cast<float>(q + (r ? 1 : 0));
        const float even = t.sum(d.B * p.head_parts) / static_cast<float>(M);
        // (no cut ends before its longest prefix CU or an even spread of all its work: not played through
        // when that is no better already)
        if (best.chunk != 0 && fmaxf(end, even) + parts_us >= best_t) return;
        if (n_own > 512) {
            end = fmaxf(end, even + 0.5f * t.own(0));
        } else {
            float cu[KV_MAX_CUS];                   // a heap of the times at which the CUs are free
            for (int m = 0; m < M; ++m) cu[m] = t.pre * static_cast<float>(q + (m >= M - static_cast<int>(r) ? 1 : 0));
            for (long j = 0; j < n_own; ++j) {
                const float e = run_next(cu, M, t.own(static_cast<int>(j)));
                end = e > end ? e : end;
            }
        }
        end += parts_us;
        if (best.chunk == 0 || end < best_t) {
            best_t = end;
            best = p;
        }
    });
    return best;
}

// One KV head's workgroups played through in launch order, each on the CU that is free first
struct Played {
    float cu[KV_MAX_CUS];
    int n;
    float end;
    explicit Played(int M) : n(M), end(0.f) {
        for (int i = 0; i < n; ++i) cu[i] = 0.f;
    }
    void run(float t) {
        t = run_next(cu, n, t);
        end = t > end ? t : end;
    }
};

// dQ, dK and dV in one launch, or dQ and then dK and dV: by playing both through, the one launch for the two cuts of each
// split of dQ that look best by their work spread evenly.  Its estimate is 4 % further above the measured times than the two
// launches' (8 % either way for one problem), so as good as equal is ahead.  Not where its long blocks are somewhat more than
// one round, prefix blocks many of them: a block's time varies by 8 %, the few of the second round start when the last of the
// first ones end, and little is left to even that out; there it has to be ahead by ONE_LATE.  1400 random batched and packed
// problems of 20 to 1500 us: slower than in two launches by more than 1.5 % 5 (two estimates compared as they come: 10; without
// ONE_LATE: 8 of the first 700), all of them 1.180 times as fast in the geometric mean (1.173; of
// the first 700 1.174, the faster form of each 1.179).  (The one launch played on 15/16 of its CUs and asked to be ahead by 5 % where prefix blocks
// are half of the work: 1 slower of 700, but 54 that are faster in one launch by more than 3 % stayed in two.)
// Launches of many rounds are not looked at: their ends leave less idle than the statistics' own launch costs (32 x 1024
// tokens, 24 / 8 heads, 2048 slots: 2943 us in two, 2970 in one).  Measured, a backward call (us, two launches -> one):
//   1 x 128, 32 / 8 heads, 1024 slots  53 -> 38     2 x 333, 32 / 8, 4096  204 -> 184     1 x 2048, 8 / 2, 256   91 -> 68
//   1 x 700, 32 / 8, 1000              92 -> 86     3 x 1659, 32 / 8, 723  463 -> 429     1 x 567, 32 / 8, 5785  235 -> 211
//   packed: 4 of up to 272, 8 / 2, 1000  60 -> 41;  8 of up to 638, 32 / 8, 1501  343 -> 312
// (own-key blocks as the two launches number them, a sequence's one after the other and all behind dQ's: 1 x 700 92, 3 x 1659 451)
constexpr int BOTH_ITEMS = 1024;        // most workgroups of a KV head that are played through
constexpr float ONE_SHORT = 0.4f;       // of the longest block: a block that long or shorter starts where it finds room
constexpr float ONE_EVEN = 1.015f;      // how far behind two launches the one may look ..
constexpr float ONE_LATE = 1.06f, ONE_LATE_ROUNDS = 1.45f, ONE_LATE_SHARE = 0.43f;      // .. or has to be ahead of them, see above
static bool plan_one_launch(const cart_attn_desc& d, int T, long tokens, int M, BwdPlan& best) {
    constexpr SplitCost us = SPLIT_COST[QUERY_DQ];
    const int most_parts = static_cast<int>(attn_query_parts(d, T));
    int tiles[BOTH_ITEMS];
    auto dq_items = [&](const QuerySplit& sp) { return attn_query_tiles(d, T, sp, tiles, BOTH_ITEMS); };
    auto dq_extra = [&](const QuerySplit& sp) { return sp.n_blocks > 0 ? us.fix + us.wg * static_cast<float>(sp.n_parts * d.Hkv) : 0.f; };
    auto dq_us = [&](int i) { return us.block + us.tile * static_cast<float>(tiles[i]); };
    int n_dq = dq_items(best.split);
    if (n_dq < 0 || best.split.e_full > 4 * M) return false;
    const long key_blocks = (d.P + KV_WG_KEYS - 1) / KV_WG_KEYS + static_cast<long>((d.S + KV_WG_KEYS - 1) / KV_WG_KEYS) * d.B;
    if (key_blocks > BOTH_ITEMS) return false;
    float two_t;                        // when the two launches end
    {
        // (a tile's time, of its time when the chip is full)
        auto light = [&](long blocks) {
            return KV_LIGHT_US / KV_FULL_US + (1.f - KV_LIGHT_US / KV_FULL_US) * fminf(static_cast<float>(blocks) / static_cast<float>(M), 1.f);
        };
        Played dq(M), kv(M);
        const float dq_tile = us.tile * light(n_dq);
        for (int i = 0; i < n_dq; ++i) dq.run(us.block + dq_tile * static_cast<float>(tiles[i]));
        KvTimes t = kv_times(d, best.kv);
        const float kv_tile = KV_FULL_US * light(t.n_pre + t.n_own);
        set_tiles(t, d, best.kv, kv_tile, kv_tile);
        for (long j = 0; j < t.n_pre; ++j) kv.run(t.pre);
        for (long j = 0; j < t.n_own; ++j) kv.run(t.own(static_cast<int>(j % t.nOb)));
        two_t = dq.end + dq_extra(best.split) + kv.end + kv_parts_us(d, tokens, best.kv);
    }
    float one_t = two_t * ONE_EVEN;     // when the cheapest one launch so far ends
    bool one = false, late = false;
    KvPlan one_kv = {};
    QuerySplit one_split;
    int one_front = 0;
    const float stats_us = 4.f + static_cast<float>(tokens) * d.Hq * (2 * ROW_B) / 4.0e6f;
    for (int parts = 1; parts <= 6; ++parts) {
        QuerySplit sp;
        if (!attn_query_split_all(sp, d, T, parts, most_parts)) break;
        n_dq = dq_items(sp);
        if (n_dq < 0) break;
        float dq_sum = 0.f, dq_most = 0.f;
        for (int i = 0; i < n_dq; ++i) {
            dq_sum += dq_us(i);
            dq_most = fmaxf(dq_most, dq_us(i));
        }
        auto longest = [&](const KvTimes& t) { return fmaxf(dq_most, fmaxf(t.n_pre > 0 ? t.pre : 0.f, t.own(0))); };
        // of this split, the two cuts with the least bound
        struct { KvPlan p; float bound, extra; } c[2] = {};
        int n = 0;
        each_cut(d, tokens, M, [&](const KvPlan& p, long n_own, float parts_us) {
            KvTimes t = kv_times(d, p);
            set_tiles(t, d, p, KV_FULL_US, KV_FULL_US);
            if (t.n_pre + n_own > BOTH_ITEMS) return;
            const float extra = parts_us + dq_extra(sp) + stats_us;
            const float sum = dq_sum + t.sum(d.B * p.head_parts);
            const float bound = fmaxf(longest(t), sum / static_cast<float>(M)) + extra;
            if (bound >= one_t) return;
            const int at = n == 0 || bound < c[0].bound ? 0 : n == 1 || bound < c[1].bound ? 1 : 2;
            if (at == 0) c[1] = c[0];
            if (at < 2) { c[at].p = p; c[at].bound = bound; c[at].extra = extra; }
            if (n < 2) ++n;
        });
        for (int i = 0; i < n; ++i) {
            if (c[i].bound >= one_t) continue;
            KvTimes t = kv_times(d, c[i].p);
            set_tiles(t, d, c[i].p, KV_FULL_US, KV_FULL_US);
            const long cols = static_cast<long>(d.B) * c[i].p.head_parts;
            int kb1 = 0;                                // own-key blocks 0 .. kb1 - 1 of each column go ahead of dQ
            while (kb1 < t.nOb && t.own(kb1) > dq_most) ++kb1;
            const float short_us = ONE_SHORT * longest(t);
            long n_long = t.pre > short_us ? t.n_pre : 0;
            for (int j = 0; j < n_dq; ++j) n_long += dq_us(j) > short_us;
            for (int kb = 0; kb < t.nOb; ++kb) n_long += t.own(kb) > short_us ? cols : 0;
            Played w(M);
            for (long j = 0; j < t.n_pre; ++j) w.run(t.pre);
            for (int kb = 0; kb <= t.nOb; ++kb) {
                if (kb == kb1)
                    for (int j = 0; j < n_dq; ++j) w.run(dq_us(j));
                if (kb < t.nOb)
                    for (long j = 0; j < cols; ++j) w.run(t.own(kb));
            }
            if (w.end + c[i].extra < one_t) {
                one_t = w.end + c[i].extra;
                one_kv = c[i].p;
                one_split = sp;
                one_front = static_cast<int>(t.n_pre + kb1 * cols);
                one = true;
                late = n_long > M && static_cast<float>(n_long) <= ONE_LATE_ROUNDS * static_cast<float>(M) &&
                       t.pre * static_cast<float>(t.n_pre) > ONE_LATE_SHARE * (dq_sum + t.sum(d.B * c[i].p.head_parts));
            }
        }
    }
    if (!one || (late && one_t * ONE_LATE > two_t)) return false;
    best.kv = one_kv;
    best.split = one_split;
    best.kv_front = one_front;
    return true;
}

// (the thread's last plan is kept with all that it depends on: the layers of a step ask for the same one in turn)
const BwdPlan& plan_bwd(const cart_attn_desc& d, int T) {
    struct Key { int T, B, S, Hq, Hkv, P, cus; };
    static thread_local Key key;
    static thread_local BwdPlan plan;
    const Key k = {T, d.B, d.S, d.Hq, d.Hkv, d.P, device_cus()};
    if (key.cus != k.cus || key.T != k.T || key.B != k.B || key.S != k.S || key.Hq != k.Hq || key.Hkv != k.Hkv || key.P != k.P) {
        const long tokens = T > 0 ? T : static_cast<long>(d.B) * d.S;
        int M = k.cus / d.Hkv;
        M = M < 1 ? 1 : (M > KV_MAX_CUS ? KV_MAX_CUS : M);
        attn_query_split(plan.split, d, T, QUERY_DQ);
        plan.kv = search_plan(d, tokens, M);
        plan.one_launch = plan_one_launch(d, T, tokens, M, plan);
        key = k;
    }
    return plan;
}

unsigned bwd_kv_grid(const cart_attn_desc& d, const KvPlan& plan) {
    const long nPb = (d.P + KV_WG_KEYS - 1) / KV_WG_KEYS, nOb = (d.S + KV_WG_KEYS - 1) / KV_WG_KEYS;
    return static_cast<unsigned>((nPb * plan.n_part + nOb * d.B * plan.head_parts) * d.Hkv);
}

void launch_attn_bwd_kv(const KvArgs& a, unsigned grid, hipStream_t st) {
    hipLaunchKernelGGL(attn_bwd_kv_kernel, dim3(grid), dim3(256), 0, st, a);
}
void launch_attn_bwd_stats(const bf16_t* o, const bf16_t* d_o, const float* lse, float* nlse2, float* ndelta, int n_tok, int S, int Hq,
                           hipStream_t st) {
    hipLaunchKernelGGL(attn_bwd_stats_kernel, grid_of(static_cast<long>((n_tok + 63) / 64) * Hq), dim3(256), 0, st, o, d_o, lse, nlse2,
                       ndelta, n_tok, S, Hq);
}
void launch_attn_bwd_both(const KvArgs& ka, const DqArgs& qa, const QuerySplit& sp, unsigned kv_grid, int kv_front, hipStream_t st) {
    BwdArgs a;
    a.kv = ka;
    a.dq = qa;
    a.n_front = static_cast<unsigned>(kv_front) * ka.Hkv;
    a.n_dq = static_cast<unsigned>(sp.e_full + sp.n_parts) * ka.Hkv;
    a.split = sp;
    hipLaunchKernelGGL(attn_bwd_both_kernel, dim3(kv_grid + a.n_dq), dim3(256), 0, st, a);
}

}  // namespace cart
