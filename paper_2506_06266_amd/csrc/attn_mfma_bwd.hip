// Cartridge attention backward on the matrix cores (bf16 in, fp32 accumulate, head_dim 128):
// the gradient of Eq. 1 over the cache of Sec. 3.2 with respect to Q, the own K/V and the
// trainable prefix Z (Sec. 3.2 trains Z by back-propagation with the model frozen).
//
// This file: the dQ kernel of the two-launch form (its body in attn_bwd_dq.h; queries stationary: S^T = K Q^T,
// dP^T = V dO^T, dQ^T += K^T dS^T, with P = exp(scale S - lse), dS = P (dP - delta), delta_i = dO_i . O_i formed
// in its prologue and written out for the key-side kernel), the fixed-order reduction of the prefix-gradient partials,
// and the launcher of the whole backward call.  dK, dV and the partials of dZ come from the
// key-stationary kernel of attn_mfma_bwd_kv.hip, which also holds the one-launch form.  The probabilities are recomputed from the saved
// log-sum-exp, so there is no running max and no rescale; nothing uses atomics, so results are
// bit-reproducible.
#include "attn_bwd_dq.h"

namespace cart {
using namespace mfma;

// The row statistics on the way: the two-launch form, whose dK / dV launch comes behind
__global__ __launch_bounds__(256, 1) void attn_bwd_dq_kernel(DqArgs a, QuerySplit split) {
    __shared__ DqSmem sm;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    dq_block<true>(a, query_block(blockIdx.x, wv, a.Smax, a.Hq, a.Hkv, split), reinterpret_cast<char*>(&sm), lds_addr(&sm));
}

// Everything the backward pass leaves as fp32 partials, summed in a fixed order, in one launch (two
// launches for dZ_k and dZ_v alone cost 2 x 5 us and a gap); one 16-byte vector per thread.  Workgroups [0, dz_wgs): dZ_k, dZ_v (one partial per chunk of token rows; rows below
// n_frozen are 0 / left alone; added to the previous value when accumulating); then the split query
// blocks of dQ, 32 workgroups each; then dK, dV of the own tokens when their heads were split.
struct BwdReduce {
    const float *dz_part[2], *dq_part, *own_part[2];
    float* dz[2];
    bf16_t *dq, *own[2];
    long dz_n4, own_n4;                 // vectors per partial
    int dz_parts, own_parts, dz_wgs, dq_wgs, wgs;
    int P, n_frozen, accumulate;
    const int32_t* cu;
    int n_tok, Smax, Hq, Hkv;
};
__device__ __forceinline__ f32x4 sum_parts(const f32x4* __restrict__ src, long i, long stride, int n) {
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int p = 0; p < n; ++p) a += src[p * stride + i];
    return a;
}
__device__ __forceinline__ u32x2 pack4(const f32x4& a) { return u32x2{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3])}; }

__global__ __launch_bounds__(256) void attn_bwd_reduce_kernel(BwdReduce r, QuerySplit split) {
    int id = workgroup_id();
    if (id >= r.wgs) return;
    if (id < r.dz_wgs) {
        const int which = id >= r.dz_wgs / 2;
        const long i = static_cast<long>(id - which * (r.dz_wgs / 2)) * 256 + threadIdx.x;
        if (i >= r.dz_n4) return;
        f32x4 a = {0.f, 0.f, 0.f, 0.f};
        if ((i / (HD / 4)) % r.P >= r.n_frozen)
            a = sum_parts(reinterpret_cast<const f32x4*>(r.dz_part[which]), i, r.dz_n4, r.dz_parts);
        f32x4* dst = reinterpret_cast<f32x4*>(r.dz[which]);
        if (r.accumulate) a += dst[i];
        dst[i] = a;
        return;
    }
    id -= r.dz_wgs;
    if (id < r.dq_wgs) {
        const int hk = (id >> 5) % r.Hkv, blk = (id >> 5) / r.Hkv, G = r.Hq / r.Hkv;
        const int row = 8 * (id & 31) + (threadIdx.x >> 5), d4 = threadIdx.x & 31;      // row of the block, vector of the row
        const int first = split.first[blk], n_parts = split.part[first] >> 16;
        if (n_parts == 1) return;           // (a short block among the split ones ran whole)
        const QueryBlock qb = query_block_of(hk, split.e_full + blk, row >> 6, query_wgs(r.Smax, G), G);
        const SeqSpan sp = seq_span(r.cu, qb.b, r.n_tok, r.Smax, r.Hq);
        const int i = qb.wrow0 + (row & 63);
        if (i >= sp.len) return;
        const f32x4 a = sum_parts(reinterpret_cast<const f32x4*>(r.dq_part) + (static_cast<size_t>(first) * r.Hkv + hk) * (256 * HD / 4),
                                  row * (HD / 4) + d4, static_cast<long>(r.Hkv) * (256 * HD / 4), n_parts);
        reinterpret_cast<u32x2*>(r.dq + ((sp.t0 + i) * r.Hq + qb.h) * HD)[d4] = pack4(a);
        return;
    }
    id -= r.dq_wgs;
    const int half = static_cast<int>((r.own_n4 + 255) / 256), which = id >= half;
    const long i = static_cast<long>(id - which * half) * 256 + threadIdx.x;
    if (i >= r.own_n4) return;
    reinterpret_cast<u32x2*>(r.own[which])[i] =
        pack4(sum_parts(reinterpret_cast<const f32x4*>(r.own_part[which]), i, r.own_n4, r.own_parts));
}

bool attn_mfma_bwd_supported(const cart_attn_desc& d) { return d.dtype == CART_BF16 && d.D == 128; }

static size_t r256(size_t n) { return (n + 255) & ~static_cast<size_t>(255); }

// The workspace of a backward call: -delta and -lse2 (one value per token and head), the dZ partials
// [n_part,Hkv,P,128] for keys and values, the partials of split query blocks and of own keys with
// split heads; packed layout: + the row_lo array.
struct BwdLayout {
    KvPlan kv;
    QuerySplit split;
    bool one_launch;
    int kv_front;
    size_t rows, part, dq, own;
};
static size_t bwd_rows_bytes(const cart_attn_desc& d, long tokens) { return r256(static_cast<size_t>(tokens) * d.Hq * sizeof(float)); }
static void bwd_layout(BwdLayout& w, const cart_attn_desc& d, int T) {
    const long tokens = T > 0 ? T : static_cast<long>(d.B) * d.S;
    const BwdPlan& plan = plan_bwd(d, T);
    w.kv = plan.kv;
    w.split = plan.split;
    w.one_launch = plan.one_launch;
    w.kv_front = plan.kv_front;
    w.rows = bwd_rows_bytes(d, tokens);
    w.part = r256(static_cast<size_t>(w.kv.n_part) * d.Hkv * d.P * HD * sizeof(float));
    w.dq = static_cast<size_t>(w.split.n_parts) * d.Hkv * PART_O_BYTES;
    w.own = w.kv.head_parts > 1 ? r256(static_cast<size_t>(w.kv.head_parts) * tokens * d.Hkv * HD * sizeof(float)) : 0;
}
// (beyond the delta array; the partials at their most for this problem or any smaller one)
size_t attn_mfma_bwd_workspace(const cart_attn_desc& d, int T) {
    const long tokens = T > 0 ? T : static_cast<long>(d.B) * d.S;
    return bwd_rows_bytes(d, tokens) + bwd_kv_most(d, tokens) + attn_query_parts(d, T) * d.Hkv * PART_O_BYTES +
           (T > 0 ? r256(static_cast<size_t>(T) * sizeof(int32_t)) : 0);
}

int launch_attn_bwd_mfma(const cart_attn_desc& d, float scale, const void* q, const void* k,
                         const void* v, const void* zk, const void* zv, const void* o,
                         const float* lse, const void* d_o, void* dq, void* dk, void* dv,
                         float* dzk, float* dzv, void* ws, hipStream_t st, const int32_t* cu, int T) {
    if (!cu) T = 0;
    BwdLayout L;
    bwd_layout(L, d, T);
    const int n_tok = T > 0 ? T : d.B * d.S;
    char* w = static_cast<char*>(ws);
    auto take = [&](size_t bytes) { char* p = w; w += bytes; return p; };
    float* delta = reinterpret_cast<float*>(take(L.rows));
    float* lse2 = reinterpret_cast<float*>(take(L.rows));
    float* part_k = reinterpret_cast<float*>(take(L.part));
    float* part_v = reinterpret_cast<float*>(take(L.part));
    float* part_q = reinterpret_cast<float*>(take(L.dq));
    float* own_k = reinterpret_cast<float*>(take(L.own));
    float* own_v = reinterpret_cast<float*>(take(L.own));
    // packed batch with a prefix: the dQ kernel cuts its query blocks from the packed rows (it sees
    // one sequence of T rows and the first row of every row's sequence)
    int32_t* row_lo = nullptr;
    if (cu && d.P > 0) {
        row_lo = reinterpret_cast<int32_t*>(w);
        launch_row_lo(cu, d.B, T, row_lo, st);
    }
    const int32_t* q_cu = row_lo ? nullptr : cu;
    const int q_S = row_lo ? n_tok : d.S;
    const bf16_t *Q = static_cast<const bf16_t*>(q), *K = static_cast<const bf16_t*>(k),
                 *V = static_cast<const bf16_t*>(v), *ZK = static_cast<const bf16_t*>(zk),
                 *ZV = static_cast<const bf16_t*>(zv), *DO = static_cast<const bf16_t*>(d_o);
    const bf16_t* O = static_cast<const bf16_t*>(o);
    const DqArgs qa = {Q, K, V, ZK, ZV, O, DO, lse, lse2, delta, static_cast<bf16_t*>(dq), q_cu, row_lo, part_q,
                       n_tok, q_S, d.Hq, d.Hkv, d.P, scale * CART_LOG2E, scale};
    // One chunk of token rows that is not added to what dZ holds has nothing to be summed with: its partial is dZ.  Without split heads
    // and query blocks that is the call's last launch saved (us, forward and backward: 3 x 259 tokens, 24 / 8 heads, 4087 slots 224 -> 215; 1 x
    // 796, 5016 258 -> 247; 12 x 75, 32 / 8, 2600 240 -> 232; 32 x 1024, 24 / 8, 2048 3842 -> 3830).
    const bool dz_whole = L.kv.n_part == 1 && !d.dz_accumulate;
    const KvArgs ka = {Q, K, V, ZK, ZV, DO, lse2, delta, static_cast<bf16_t*>(dk), static_cast<bf16_t*>(dv), dz_whole ? dzk : part_k,
                       dz_whole ? dzv : part_v, own_k, own_v, cu, n_tok, L.kv.chunk, L.kv.head_parts, d.S, d.Hq, d.Hkv, d.P,
                       L.one_launch ? d.B * L.kv.head_parts : 0, scale * CART_LOG2E, scale, dz_whole ? d.n_frozen : 0};
    trace_begin(st);   // kernel order: dq (+ row statistics), dk + dv; or the statistics, all three gradients; then the partials' sums
    if (L.one_launch) {
        launch_attn_bwd_stats(O, DO, lse, lse2, delta, n_tok, T > 0 ? T : d.S, d.Hq, st);
        trace_mark(st);
        launch_attn_bwd_both(ka, qa, L.split, bwd_kv_grid(d, L.kv), L.kv_front, st);
    } else {
        hipLaunchKernelGGL(attn_bwd_dq_kernel, dim3(static_cast<unsigned>(L.split.e_full + L.split.n_parts) * d.Hkv), dim3(256), 0, st, qa,
                           L.split);
        trace_mark(st);
        launch_attn_bwd_kv(ka, bwd_kv_grid(d, L.kv), st);
    }
    trace_mark(st);
    BwdReduce r;
    r.dz_part[0] = part_k; r.dz_part[1] = part_v; r.dq_part = part_q; r.own_part[0] = own_k; r.own_part[1] = own_v;
    r.dz[0] = dzk; r.dz[1] = dzv; r.dq = static_cast<bf16_t*>(dq);
    r.own[0] = static_cast<bf16_t*>(dk); r.own[1] = static_cast<bf16_t*>(dv);
    r.dz_n4 = static_cast<long>(d.Hkv) * d.P * HD / 4;
    r.own_n4 = static_cast<long>(n_tok) * d.Hkv * HD / 4;
    r.dz_parts = L.kv.n_part; r.own_parts = L.kv.head_parts;
    r.dz_wgs = dz_whole ? 0 : static_cast<int>((r.dz_n4 + 255) / 256) * 2;
    r.dq_wgs = L.split.n_blocks * d.Hkv * 32;
    r.P = d.P; r.n_frozen = d.n_frozen; r.accumulate = d.dz_accumulate;
    r.cu = q_cu; r.n_tok = n_tok; r.Smax = q_S; r.Hq = d.Hq; r.Hkv = d.Hkv;
    const long own_wgs = L.kv.head_parts > 1 ? (r.own_n4 + 255) / 256 * 2 : 0;
    const long wgs = r.dz_wgs + r.dq_wgs + own_wgs;
    r.wgs = static_cast<int>(wgs);
    if (wgs > 0) hipLaunchKernelGGL(attn_bwd_reduce_kernel, grid_of(wgs), dim3(256), 0, st, r, L.split);
    trace_mark(st);
    return static_cast<int>(hipGetLastError());
}

}  // namespace cart
