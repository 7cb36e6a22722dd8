// Cartridge attention (Eq. 1 over the cache of Sec. 3.2), its gradient, and decode (Sec. 3.3) in fp32
// arithmetic, for fp32 problems and any head_dim <= 256 (bf16 inputs are widened); no atomics, fixed
// summation order.  In-library baseline the bf16 matrix-core kernels are compared with.
//
// The attention kernels run on the fp32 matrix-core instruction v_mfma_f32_16x16x4_f32,
// D(16x16) += A(16x4) B(4x16), all operands and sums fp32:
//   A: lane l holds row l%16, k = l/16;  B: lane l holds column l%16, k = l/16;
//   D: lane l holds column l%16, rows 4 (l/16) + r for r in [0,4).
// Every product keeps the stationary index (a query, or a key) on the D column.  The index the next
// product contracts over is then on the D rows: with its k-step r taken as rows {4g + r}, register r
// of the result is that product's B operand in the same lane, and nothing passes through LDS.
// Operands come straight from memory (16 rows x 64 bytes, or 4 rows x 64 bytes, per load).
//
// One workgroup owns 16 queries of one head (forward, dQ) or 16 keys of one KV head (dK, dV); its
// wavefronts split what is contracted over in blocks of 16 and add up through LDS at the end.  A
// small problem is bound by latency -- its launches, one round trip for the operands, one for the
// sums -- and a large one by the matrix cores.  Against one wavefront per row or key, a serial chain of
// shuffles and exponentials per key, us for forward and backward: 2 sequences of 64 tokens, 2 / 1
// heads of 64, 32 slots: 175 -> 20 (launches); 4 of 256, 8 / 2 heads, 256 slots: head_dim 64 2268 -> 93,
// head_dim 128 2855 -> 175.
#include "cart_common.h"

namespace cart {

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr float VEC_HIDDEN = -3.0e38f;

__device__ __forceinline__ f32x4 mma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
// sum / maximum over the four lanes that hold the same column
__device__ __forceinline__ float col_sum(float v) { v += __shfl_xor(v, 16, CART_WAVE); return v + __shfl_xor(v, 32, CART_WAVE); }
__device__ __forceinline__ float col_max(float v) {
    v = fmaxf(v, __shfl_xor(v, 16, CART_WAVE));
    return fmaxf(v, __shfl_xor(v, 32, CART_WAVE));
}

// Row operand of a contraction over the head elements: k-step (s, e) is element 16 s + 4 (lane/16) + e
template <int NB> struct RowFrag { f32x4 v[NB]; };
__device__ __forceinline__ f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 load4(const bf16_t* p) {
    const u32x2 w = *reinterpret_cast<const u32x2*>(p);
    return f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                 __uint_as_float(w.y & 0xffff0000u)};
}
template <typename T, int NB>
__device__ __forceinline__ RowFrag<NB> row_frag(const T* p, int D, int g) {
    RowFrag<NB> f;
    if (D == 16 * NB) {
#pragma unroll
        for (int s = 0; s < NB; ++s) f.v[s] = load4(p + 16 * s + 4 * g);
    } else if ((D & 3) == 0) {
#pragma unroll
        for (int s = 0; s < NB; ++s) {
            const int d = 16 * s + 4 * g;
            f.v[s] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (d < D) f.v[s] = load4(p + d);
        }
    } else {
#pragma unroll
        for (int s = 0; s < NB; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int d = 16 * s + 4 * g + e;
                f.v[s][e] = d < D ? elem<T>::load(p + d) : 0.f;
            }
    }
    return f;
}
template <int NB>
__device__ __forceinline__ f32x4 contract(const RowFrag<NB>& a, const RowFrag<NB>& b) {
    f32x4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;      // two chains: a product's result is not the next one's input
#pragma unroll
    for (int s = 0; s < NB; ++s)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
            c0 = mma4(a.v[s][e], b.v[s][e], c0);
            c1 = mma4(a.v[s][e + 1], b.v[s][e + 1], c1);
        }
    return c0 + c1;
}
// Column operand of a contraction over a block's rows: element 16 db + lane%16 of rows 4 (lane/16) + r
template <int NB> struct ColFrag { f32x4 v[NB]; };
template <typename T, int NB>
__device__ __forceinline__ ColFrag<NB> col_frag(const T* const (&p)[4], int D, int c) {
    ColFrag<NB> f;
    if (D == 16 * NB) {         // (unguarded: all loads of the block in flight at one time)
#pragma unroll
        for (int db = 0; db < NB; ++db)
#pragma unroll
            for (int r = 0; r < 4; ++r) f.v[db][r] = elem<T>::load(p[r] + 16 * db + c);
    } else {
#pragma unroll
        for (int db = 0; db < NB; ++db)
#pragma unroll
            for (int r = 0; r < 4; ++r) f.v[db][r] = 16 * db + c < D ? elem<T>::load(p[r] + 16 * db + c) : 0.f;
    }
    return f;
}
// acc[db] += X^T w, w the B operand that register r of a result is
template <int NB>
__device__ __forceinline__ void accumulate(f32x4 (&acc)[NB], const ColFrag<NB>& x, const f32x4& w) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int db = 0; db < NB; ++db) acc[db] = mma4(x.v[db][r], w[r], acc[db]);
}
// A hidden pair's weight is 0, and 0 times a NaN or an infinity of the hidden row (padding behind a
// sequence's last token, say) is not.  So a block with hidden pairs and such a row adds its rows one at a
// time, each to the columns that see it.  (A second pass over all blocks by a wavefront whose sums are
// not finite, instead of this check, measured the same on the smallest problem: 31.2 us against 30.2.)  vis: which of the lane's four rows its column sees.
template <int NB> __device__ __forceinline__ bool any_nonfinite(const ColFrag<NB>& x) {
    f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int db = 0; db < NB; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) t[r] = fmaf(x.v[db][r], 0.f, t[r]);
    return __any(t[0] + t[1] + t[2] + t[3] != 0.f);
}
template <int NB>
__device__ __forceinline__ void accumulate_visible(f32x4 (&acc)[NB], const ColFrag<NB>& x, const f32x4& w, uint32_t vis, bool hidden,
                                                   int c, int g) {
    if (__builtin_expect(!hidden || !any_nonfinite(x), 1)) {
        accumulate(acc, x, w);
        return;
    }
#pragma unroll 1
    for (int u = 0; u < 4; ++u) {
        const uint32_t sees = __shfl(vis, 16 * u + c, CART_WAVE);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float wr = __shfl(w[r], 16 * u + c, CART_WAVE);
#pragma unroll
            for (int db = 0; db < NB; ++db)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float xe = __shfl(x.v[db][r], 16 * u + 4 * g + e, CART_WAVE);
                    acc[db][e] = (sees >> r) & 1 ? fmaf(wr, xe, acc[db][e]) : acc[db][e];
                }
        }
    }
}
template <int NB> __device__ __forceinline__ void clear(f32x4 (&acc)[NB]) {
#pragma unroll
    for (int db = 0; db < NB; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
}
// a wavefront's 16 columns x head elements into LDS, [column][element]
template <int NB> __device__ __forceinline__ void to_lds(float* dst, const f32x4 (&acc)[NB], int c, int g) {
#pragma unroll
    for (int db = 0; db < NB; ++db) *reinterpret_cast<f32x4*>(dst + c * (16 * NB + 4) + 16 * db + 4 * g) = acc[db];
}

// Head_dim 128: one wavefront per SIMD, which requests each operand's next block as soon as its products are out (AHEAD; us, 4 x 256
// tokens, 8 / 2 heads, 256 slots: forward 37.6 -> 34.6, backward 319 -> 290).  Two wavefronts on a SIMD cover each
// other (head_dim up to 64: backward 22.7 -> 25.3 at 2 x 64 tokens, 64 slots); below 128 the loads are under conditions and each
// request is waited for at its end (forward, head_dim 96: 7 x 36 tokens, 32 / 8 heads 11.0 -> 12.1, 120 problems of 256 blocks or more
// 1.5 % slower on average); above 128 there are no registers for it (forward 14.0 -> 14.6, 2 x 64 tokens, 4 / 2 heads of 200).
template <int NB> constexpr bool VEC_AHEAD = NB == 8;       // .. in which register layout

// key / value row j of the concatenated cache [prefix ; own] for (sequence b, KV head hk)
template <typename T>
__device__ __forceinline__ const T* cache_row(const T* z, const T* own, int j, int P, int S,
                                              int Hkv, int D, int b, int hk) {
    return j < P ? z + (static_cast<size_t>(hk) * P + j) * D
                 : own + ((static_cast<size_t>(b) * S + (j - P)) * Hkv + hk) * D;
}

template <typename T, int NB, int NW, bool AHEAD>
__global__ __launch_bounds__(64 * NW) void attn_fwd_vector(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, const T* __restrict__ zk,
    const T* __restrict__ zv, T* __restrict__ o, float* __restrict__ lse, int B, int S, int Hq, int Hkv, int D, int P, float scale) {
    constexpr int PITCH = 16 * NB + 4;
    __shared__ float sm_o[NW][16 * PITCH], sm_m[NW][16], sm_l[NW][16];
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nQt = (S + 15) / 16;
    int id = workgroup_id();
    const int i0 = 16 * (id % nQt); id /= nQt;
    const int h = id % Hq, b = id / Hq, hk = h / (Hq / Hkv);
    if (b >= B) return;
    const int i = min(i0 + c, S - 1);
    const RowFrag<NB> qf = row_frag<T, NB>(q + ((static_cast<size_t>(b) * S + i) * Hq + h) * D, D, g);
    const float c2 = scale * CART_LOG2E;
    const int nk = P + min(i0 + 16, S), last = P + i;      // keys of the block; last key the lane's query sees
    f32x4 acc[NB];
    clear(acc);
    float m = VEC_HIDDEN, l = 0.f;
    auto load_k = [&](int j0) __attribute__((always_inline)) {
        return row_frag<T, NB>(cache_row(zk, k, min(j0 + c, nk - 1), P, S, Hkv, D, b, hk), D, g);
    };
    auto load_v = [&](int j0) __attribute__((always_inline)) {
        const T* vr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) vr[r] = cache_row(zv, v, min(j0 + 4 * g + r, nk - 1), P, S, Hkv, D, b, hk);
        return col_frag<T, NB>(vr, D, c);
    };
    RowFrag<NB> kf;
    ColFrag<NB> vc;
    if (AHEAD) { kf = load_k(16 * wv); vc = load_v(16 * wv); }
    for (int j0 = 16 * wv; j0 < nk; j0 += 16 * NW) {
        const bool more = AHEAD && j0 + 16 * NW < nk;
        if (!AHEAD) { kf = load_k(j0); vc = load_v(j0); }
        f32x4 s = contract(kf, qf);
        if (more) kf = load_k(j0 + 16 * NW);
        float tm = VEC_HIDDEN;
        uint32_t vis = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool sees = j0 + 4 * g + r <= last;
            vis |= sees ? 1u << r : 0u;
            s[r] = sees ? s[r] * c2 : VEC_HIDDEN;
            tm = fmaxf(tm, s[r]);
        }
        const float nm = fmaxf(m, col_max(tm)), alpha = fast_exp2(m - nm);
        f32x4 p;
        l *= alpha;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p[r] = (vis >> r) & 1 ? fast_exp2(s[r] - nm) : 0.f;      // (a NaN score reaches the row)
            l += p[r];
        }
        m = nm;
#pragma unroll
        for (int db = 0; db < NB; ++db) acc[db] *= alpha;
        accumulate_visible(acc, vc, p, vis, j0 + 15 > P + i0, c, g);
        if (more) vc = load_v(j0 + 16 * NW);
    }
    l = col_sum(l);
    to_lds(sm_o[wv], acc, c, g);
    if (g == 0) { sm_m[wv][c] = m; sm_l[wv][c] = l; }
    __syncthreads();
    // 16 threads per query, each every 16th head element
    for (int t = threadIdx.x; t < 256; t += 64 * NW) {
        const int qc = t >> 4;
        if (i0 + qc >= S) continue;
        float M = sm_m[0][qc], L = 0.f, w[NW];
#pragma unroll
        for (int u = 1; u < NW; ++u) M = fmaxf(M, sm_m[u][qc]);
#pragma unroll
        for (int u = 0; u < NW; ++u) {
            w[u] = fast_exp2(sm_m[u][qc] - M);
            L += w[u] * sm_l[u][qc];
        }
        const float inv = 1.f / L;
        T* op = o + ((static_cast<size_t>(b) * S + i0 + qc) * Hq + h) * D;
        for (int d = t & 15; d < D; d += 16) {
            float a = 0.f;
#pragma unroll
            for (int u = 0; u < NW; ++u) a = fmaf(w[u], sm_o[u][qc * PITCH + d], a);
            elem<T>::store(op + d, a * inv);
        }
        if ((t & 15) == 0) lse[(static_cast<size_t>(b) * Hq + h) * S + i0 + qc] = (M + fast_log2(L)) * CART_LN2;
    }
}

// ---- backward: dQ blocks and dK / dV blocks -----------------------------------------------------
template <typename T>
struct VecBwd {
    const T *q, *k, *v, *zk, *zv, *o, *d_o;
    const float* lse;
    float* delta;                       // [B,Hq,S], written by the dQ blocks of the two-launch form
    T *dq, *dk, *dv;
    float *dzk, *dzv;
    int B, S, Hq, Hkv, D, P;
    float scale;
    int n_frozen, accumulate;
    int splits;                         // of a prefix block's token rows; more than one: sums into part [splits][2][Hkv,P,D]
    float* part;
};
template <int NB> constexpr int VEC_TURN = 16 * (16 * NB + 4);      // floats of one wavefront's sums in LDS

// delta = dO . O of the lane's row, from its quarter of the head elements
template <int NB>
__device__ __forceinline__ float row_delta(const RowFrag<NB>& of, const RowFrag<NB>& gf) {
    float dl = 0.f;
#pragma unroll
    for (int s = 0; s < NB; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) dl = fmaf(of.v[s][e], gf.v[s][e], dl);
    return col_sum(dl);
}

// dQ of 16 queries of one head.  ONE: in one launch with dK and dV; else also delta[b,h,i], for the dK / dV launch that follows.
template <typename T, int NB, int NW, bool ONE, bool AHEAD>
__device__ __forceinline__ void dq_block(const VecBwd<T>& a, int id, float (*sm_o)[VEC_TURN<NB>]) {
    constexpr int PITCH = 16 * NB + 4;
    const int B = a.B, S = a.S, Hq = a.Hq, Hkv = a.Hkv, D = a.D, P = a.P;
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nQt = (S + 15) / 16;
    const int i0 = 16 * (id % nQt); id /= nQt;
    const int h = id % Hq, b = id / Hq, hk = h / (Hq / Hkv);
    if (b >= B) return;
    const int i = min(i0 + c, S - 1);
    const size_t row = ((static_cast<size_t>(b) * S + i) * Hq + h) * D;
    const size_t st = (static_cast<size_t>(b) * Hq + h) * S + i;
    const int nk = P + min(i0 + 16, S), last = P + i;
    RowFrag<NB> kf, vf;
    ColFrag<NB> kc;
    auto load_rows = [&](int j0) __attribute__((always_inline)) {
        const int jc = min(j0 + c, nk - 1);
        kf = row_frag<T, NB>(cache_row(a.zk, a.k, jc, P, S, Hkv, D, b, hk), D, g);
        vf = row_frag<T, NB>(cache_row(a.zv, a.v, jc, P, S, Hkv, D, b, hk), D, g);
    };
    auto load_cols = [&](int j0) __attribute__((always_inline)) {
        const T* kr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) kr[r] = cache_row(a.zk, a.k, min(j0 + 4 * g + r, nk - 1), P, S, Hkv, D, b, hk);
        kc = col_frag<T, NB>(kr, D, c);
    };
    const RowFrag<NB> qf = row_frag<T, NB>(a.q + row, D, g), gf = row_frag<T, NB>(a.d_o + row, D, g);
    const float c2 = a.scale * CART_LOG2E, l2 = a.lse[st] * CART_LOG2E;
    // (the one launch's first keys are requested ahead of delta's wait for O and dO)
    float dl;
    {
        const RowFrag<NB> of = row_frag<T, NB>(a.o + row, D, g);
        if constexpr (ONE) {
            load_rows(16 * wv);
            load_cols(16 * wv);
            __builtin_amdgcn_sched_barrier(0);
        }
        dl = row_delta(of, gf);
    }
    if (!ONE && wv == 0 && g == 0 && i0 + c < S) a.delta[st] = dl;
    f32x4 acc[NB];
    clear(acc);
    for (int j0 = 16 * wv; j0 < nk; j0 += 16 * NW) {
        const bool more = AHEAD && j0 + 16 * NW < nk;
        if (!ONE || (!AHEAD && j0 != 16 * wv)) { load_rows(j0); load_cols(j0); }
        const f32x4 s = contract(kf, qf), dp = contract(vf, gf);
        if (more) load_rows(j0 + 16 * NW);
        f32x4 ds;
        uint32_t vis = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool sees = j0 + 4 * g + r <= last;
            vis |= sees ? 1u << r : 0u;
            ds[r] = sees ? fast_exp2(fmaf(s[r], c2, -l2)) * (dp[r] - dl) : 0.f;
        }
        accumulate_visible(acc, kc, ds, vis, j0 + 15 > P + i0, c, g);
        if (more) load_cols(j0 + 16 * NW);
    }
    to_lds(sm_o[wv], acc, c, g);
    __syncthreads();
    for (int t16 = threadIdx.x; t16 < 256; t16 += 64 * NW) {
        const int qc = t16 >> 4;
        if (i0 + qc >= S) continue;
        T* op = a.dq + ((static_cast<size_t>(b) * S + i0 + qc) * Hq + h) * D;
        for (int d = t16 & 15; d < D; d += 16) {
            float x = 0.f;
#pragma unroll
            for (int u = 0; u < NW; ++u) x += sm_o[u][qc * PITCH + d];
            elem<T>::store(op + d, x * a.scale);
        }
    }
}

// dK, dV of 16 keys: prefix slots (summed over every sequence, every query head of the group, every
// token) or own keys of one sequence (the group's heads, tokens from the block's first key on).
// ONE: in one launch with dQ, the rows' delta is formed here from O and dO (the same sum in the same order), not read.
template <typename T, int NB, int NW, bool ONE, bool AHEAD>
__device__ __forceinline__ void dkv_block(const VecBwd<T>& a, int id, float (*sm_k)[VEC_TURN<NB>], float (*sm_v)[VEC_TURN<NB>]) {
    constexpr int PITCH = 16 * NB + 4;
    const int B = a.B, S = a.S, Hq = a.Hq, Hkv = a.Hkv, D = a.D, P = a.P;
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nPt = (P + 15) / 16, nSt = (S + 15) / 16, G = Hq / Hkv;
    const bool prefix = id < nPt * Hkv * a.splits;
    if (!prefix) id -= nPt * Hkv * a.splits;
    const int hk = id % Hkv; id /= Hkv;
    const int key0 = 16 * (id % (prefix ? nPt : nSt)), split = prefix ? id / nPt : 0, b_own = prefix ? 0 : id / nSt;
    if (b_own >= B) return;
    const int nkeys = prefix ? P : S;
    auto key_row = [&](int j) { return prefix ? (static_cast<size_t>(hk) * P + j) * D
                                              : ((static_cast<size_t>(b_own) * S + j) * Hkv + hk) * D; };
    const size_t kr = key_row(min(key0 + c, nkeys - 1));
    const RowFrag<NB> kf = row_frag<T, NB>((prefix ? a.zk : a.k) + kr, D, g), vf = row_frag<T, NB>((prefix ? a.zv : a.v) + kr, D, g);
    const float c2 = a.scale * CART_LOG2E;
    f32x4 ak[NB], av[NB];
    clear(ak);
    clear(av);
    // blocks of 16 token rows: (sequence, head of the group, block), from the block's own diagonal on
    const int it0 = prefix ? 0 : key0 / 16, nIt = nSt - it0, all = (prefix ? B : 1) * G * nIt;
    const int first = prefix ? static_cast<int>(static_cast<long>(all) * split / a.splits) : 0;
    const int n = prefix ? static_cast<int>(static_cast<long>(all) * (split + 1) / a.splits) : all;      // blocks [first, n)
    // Of a block: its rows for the scores, lse, delta; then the same rows as columns for the sums
    struct Block { int i0, h, b; };
    auto block = [&](int t) __attribute__((always_inline)) {
        const int u = t / nIt;
        return Block{16 * (it0 + t - u * nIt), hk * G + u % G, prefix ? u / G : b_own};
    };
    auto tok = [&](const Block& x, int i) __attribute__((always_inline)) {
        return ((static_cast<size_t>(x.b) * S + min(i, S - 1)) * Hq + x.h) * D;
    };
    RowFrag<NB> qf, gf, of;
    ColFrag<NB> gc, qc;
    f32x4 l2, dl;
    auto load_rows = [&](const Block& x) __attribute__((always_inline)) {
        const size_t rc = tok(x, x.i0 + c);
        qf = row_frag<T, NB>(a.q + rc, D, g);
        gf = row_frag<T, NB>(a.d_o + rc, D, g);
        if constexpr (ONE) of = row_frag<T, NB>(a.o + rc, D, g);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const size_t st = (static_cast<size_t>(x.b) * Hq + x.h) * S + min(x.i0 + 4 * g + r, S - 1);
            l2[r] = a.lse[st] * CART_LOG2E;
            if (!ONE) dl[r] = a.delta[st];
        }
    };
    auto load_cols = [&](const Block& x, ColFrag<NB>& f, const T* src) __attribute__((always_inline)) {
        const T* pr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) pr[r] = src + tok(x, x.i0 + 4 * g + r);
        f = col_frag<T, NB>(pr, D, c);
    };
    constexpr bool COLS_FIRST = !ONE && NB <= 8;
    Block cur = block(min(first + wv, n - 1));
    if constexpr (AHEAD) {
        load_rows(cur);
        load_cols(cur, gc, a.d_o);
        load_cols(cur, qc, a.q);
    }
    for (int t = first + wv; t < n; t += NW) {
        // (The block after the last is the last again: loads under a condition are all waited for at its end.  The columns
        // not requested ahead come behind the scores: head_dim above 128 has no registers for all four operands of a block --
        // 52 registers of fp32 problems, 128 of bf16 ones, spill as it is -- and two wavefronts on a SIMD are faster so:
        // backward 148 -> 135 us at 4 x 256 tokens, 8 / 2 heads of 64, 256 slots)
        const Block nx = block(AHEAD ? min(t + NW, n - 1) : t);
        if constexpr (!AHEAD) { cur = nx; load_rows(cur); }
        if constexpr (COLS_FIRST) { load_cols(cur, gc, a.d_o); load_cols(cur, qc, a.q); }
        if constexpr (ONE) {
            const float rd = row_delta(of, gf);      // of row i0 + c
#pragma unroll
            for (int r = 0; r < 4; ++r) dl[r] = __shfl(rd, 4 * g + r, CART_WAVE);
        }
        const f32x4 s = contract(qf, kf), dp = contract(gf, vf);
        f32x4 p, ds;
        uint32_t vis = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = cur.i0 + 4 * g + r;
            const bool seen = i < S && (prefix || i >= key0 + c);
            vis |= seen ? 1u << r : 0u;
            p[r] = seen ? fast_exp2(fmaf(s[r], c2, -l2[r])) : 0.f;
            ds[r] = seen ? p[r] * (dp[r] - dl[r]) : 0.f;
        }
        if constexpr (AHEAD) load_rows(nx);
        const bool hidden = cur.i0 + 16 > S || (!prefix && cur.i0 == key0);
        if constexpr (!AHEAD && !COLS_FIRST) {
            asm volatile("" ::: "memory");
            load_cols(cur, gc, a.d_o);
        }
        accumulate_visible(av, gc, p, vis, hidden, c, g);
        if constexpr (AHEAD) load_cols(nx, gc, a.d_o);
        if constexpr (!AHEAD && !COLS_FIRST) {
            asm volatile("" ::: "memory");
            load_cols(cur, qc, a.q);
        }
        accumulate_visible(ak, qc, ds, vis, hidden, c, g);
        if constexpr (AHEAD) load_cols(nx, qc, a.q);
        cur = nx;
    }
    to_lds(sm_k[wv], ak, c, g);
    to_lds(sm_v[wv], av, c, g);
    __syncthreads();
    for (int t = threadIdx.x; t < 256; t += 64 * NW) {
        const int j = key0 + (t >> 4);
        if (j >= nkeys) continue;
        const size_t r = key_row(j);
        for (int d = t & 15; d < D; d += 16) {
            float gk = 0.f, gv = 0.f;
#pragma unroll
            for (int u = 0; u < NW; ++u) {
                gk += sm_k[u][(t >> 4) * PITCH + d];
                gv += sm_v[u][(t >> 4) * PITCH + d];
            }
            if (prefix && a.splits > 1) {
                const size_t all_z = static_cast<size_t>(Hkv) * P * D;
                a.part[2 * split * all_z + r + d] = gk;
                a.part[(2 * split + 1) * all_z + r + d] = gv;
            } else if (prefix) {
                gk = j < a.n_frozen ? 0.f : gk * a.scale;
                gv = j < a.n_frozen ? 0.f : gv;
                if (a.accumulate) { gk += a.dzk[r + d]; gv += a.dzv[r + d]; }
                a.dzk[r + d] = gk;
                a.dzv[r + d] = gv;
            } else {
                elem<T>::store(a.dk + r + d, gk * a.scale);
                elem<T>::store(a.dv + r + d, gv);
            }
        }
    }
}

template <typename T, int NB, int NW>
__global__ __launch_bounds__(64 * NW) void attn_bwd_dq_vector(VecBwd<T> a) {
    __shared__ float sm[NW][VEC_TURN<NB>];
    dq_block<T, NB, NW, false, false>(a, workgroup_id(), sm);
}
template <typename T, int NB, int NW>
__global__ __launch_bounds__(64 * NW) void attn_bwd_dkv_vector(VecBwd<T> a) {
    __shared__ float sm[2][NW][VEC_TURN<NB>];
    dkv_block<T, NB, NW, false, false>(a, workgroup_id(), sm[0], sm[1]);
}
// dZ from the sums of split prefix blocks, in the splits' order
__global__ __launch_bounds__(256) void attn_bwd_dz_vector(const float* __restrict__ part, float* __restrict__ dzk, float* __restrict__ dzv,
                                                          int n, int P, int D, int splits, float scale, int n_frozen, int accumulate) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float gk = 0.f, gv = 0.f;
#pragma unroll 4
    for (int s = 0; s < splits; ++s) {
        gk += part[static_cast<size_t>(2 * s) * n + i];
        gv += part[static_cast<size_t>(2 * s + 1) * n + i];
    }
    const bool frozen = i / D % P < n_frozen;
    gk = frozen ? 0.f : gk * scale;
    gv = frozen ? 0.f : gv;
    if (accumulate) { gk += dzk[i]; gv += dzv[i]; }
    dzk[i] = gk;
    dzv[i] = gv;
}
// Both in one launch, the dK / dV blocks (the longer ones) first
template <typename T, int NB, int NW, bool AHEAD>
__global__ __launch_bounds__(64 * NW) void attn_bwd_vector(VecBwd<T> a, int n_kv) {
    __shared__ float sm[2][NW][VEC_TURN<NB>];
    const int id = workgroup_id();
    if (id < n_kv) dkv_block<T, NB, NW, true, AHEAD>(a, id, sm[0], sm[1]);
    else           dq_block<T, NB, NW, true, AHEAD>(a, id - n_kv, sm[0]);
}

// ---- decode: one wavefront per output row; lane l owns head elements l, l+64, ... ---------------
constexpr int VEC_WAVES = 4;         // wavefronts per workgroup
template <typename T, int E>
__device__ __forceinline__ void load_row(const T* p, int D, int lane, float (&r)[E]) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
        int d = lane + 64 * e;
        r[e] = d < D ? elem<T>::load(p + d) : 0.f;
    }
}
template <int E>
__device__ __forceinline__ float dot_rows(const float (&a)[E], const float (&b)[E]) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) s = fmaf(a[e], b[e], s);
    return wave_sum(s);
}

template <typename T, int E>
__global__ __launch_bounds__(64 * VEC_WAVES) void decode_vector(
    const T* q, const T* zk, const T* zv, const T* k, const T* v, const int32_t* cu, T* o,
    float* lse, int B, int Hq, int Hkv, int D, int P, float scale) {
    const int lane = threadIdx.x & 63;
    const long row = static_cast<long>(blockIdx.x) * VEC_WAVES + (threadIdx.x >> 6);
    if (row >= static_cast<long>(B) * Hq) return;
    const int h = row % Hq, b = row / Hq;
    const int hk = h / (Hq / Hkv);
    const int t0 = cu[b], len = cu[b + 1] - t0;
    float qr[E], acc[E];
    load_row<T, E>(q + row * D, D, lane, qr);
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.f;
    const float c = scale * CART_LOG2E;
    float m = -3.0e38f, l = 0.f;
    for (int j = 0; j < P + len; ++j) {
        const size_t off = j < P ? (static_cast<size_t>(hk) * P + j) * D
                                 : (static_cast<size_t>(t0 + j - P) * Hkv + hk) * D;
        float kr[E], vr[E];
        load_row<T, E>((j < P ? zk : k) + off, D, lane, kr);
        load_row<T, E>((j < P ? zv : v) + off, D, lane, vr);
        float s = dot_rows<E>(qr, kr) * c;
        float nm = fmaxf(m, s);
        float corr = fast_exp2(m - nm), pj = fast_exp2(s - nm);
        l = l * corr + pj;
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = acc[e] * corr + pj * vr[e];
        m = nm;
    }
    const float inv = 1.f / l;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        int d = lane + 64 * e;
        if (d < D) elem<T>::store(o + row * D + d, acc[e] * inv);
    }
    if (lane == 0 && lse) lse[row] = (m + fast_log2(l)) * CART_LN2;
}

static inline unsigned blocks_for(long rows) { return static_cast<unsigned>((rows + VEC_WAVES - 1) / VEC_WAVES); }

// Head elements in blocks of 16, wavefronts per workgroup: as many as their registers allow
#define CART_DISPATCH_NB(D, BODY)                                                  \
    do {                                                                           \
        if ((D) <= 64) { constexpr int NB = 4, NW = 8; BODY; }                     \
        else if ((D) <= 128) { constexpr int NB = 8, NW = 4; BODY; }               \
        else { constexpr int NB = 16, NW = 4; BODY; }                              \
    } while (0)
#define CART_DISPATCH_E(D, BODY)                      \
    do {                                              \
        if ((D) <= 64) { constexpr int E = 1; BODY; } \
        else if ((D) <= 128) { constexpr int E = 2; BODY; } \
        else { constexpr int E = 4; BODY; }           \
    } while (0)

template <typename T>
static void fwd_t(const cart_attn_desc& d, float scale, const void* q, const void* k, const void* v,
                  const void* zk, const void* zv, void* o, float* lse, hipStream_t st) {
    const long wgs = static_cast<long>((d.S + 15) / 16) * d.Hq * d.B;
    const bool ahead = d.D == 128;
    CART_DISPATCH_NB(d.D, hipLaunchKernelGGL((ahead ? attn_fwd_vector<T, NB, NW, VEC_AHEAD<NB>> : attn_fwd_vector<T, NB, NW, false>), grid_of(wgs), dim3(64 * NW), 0, st, (const T*)q,
        (const T*)k, (const T*)v, (const T*)zk, (const T*)zv, (T*)o, lse, d.B, d.S, d.Hq, d.Hkv, d.D, d.P, scale));
}

int launch_attn_fwd_vector(const cart_attn_desc& d, float scale, const void* q, const void* k,
                           const void* v, const void* zk, const void* zv, void* o, float* lse,
                           hipStream_t st) {
    trace_begin(st);
    if (d.dtype == CART_F32) fwd_t<float>(d, scale, q, k, v, zk, zv, o, lse, st);
    else fwd_t<bf16_t>(d, scale, q, k, v, zk, zv, o, lse, st);
    trace_mark(st);
    return static_cast<int>(hipGetLastError());
}

// Into how many parts the token rows of a prefix block are split: it streams those of every sequence, an own-key block one
// sequence's, and a problem of this path's size leaves most CUs idle meanwhile.  Blocks of 16 rows one after the other
// cost a wavefront about VEC_TURN_US each, the sums their launch; no more prefix blocks than CUs.  us a backward call, whole ->
// split: 4 x 128 tokens, 8 / 2 heads of 128, 128 slots 148 -> 47; 4 x 256, 256 slots 291 -> 138, of 64 134 -> 72; 2 x 64, 4 / 2
// heads of 200, 64 slots 71 -> 53; 2 x 64, 8 / 2 heads of 64, 64 slots 22.7 -> 17.5.
constexpr int VEC_MAX_SPLITS = 8;
constexpr float VEC_TURN_US = 3.5f, VEC_SUM_US = 5.f;
static int dz_splits(const cart_attn_desc& d, int NW) {
    const long nSt = (d.S + 15) / 16, nPt = (d.P + 15) / 16, G = d.Hq / d.Hkv;
    if (d.P == 0) return 1;
    // (nor where the blocks keep the CUs busy for as long as a whole prefix block takes: 7 x 208 tokens, 16 / 16 heads of 96, 37
    // slots in five parts 221, whole 211)
    const long all = d.B * G * nSt, even = d.Hkv * (nPt * all + d.B * nSt * G * (nSt + 1) / 2) / (NW * device_cus());
    const long longest_own = (G * nSt + NW - 1) / NW, own = longest_own > even ? longest_own : even;
    int best = 1;
    float best_us = 0.f;
    for (int s = 1; s <= VEC_MAX_SPLITS && s <= all; ++s) {
        if (s > 1 && nPt * d.Hkv * s > device_cus()) break;
        const long turns = ((all + s - 1) / s + NW - 1) / NW;
        const float us = VEC_TURN_US * static_cast<float>(turns > own ? turns : own) + (s > 1 ? VEC_SUM_US : 0.f);
        if (s == 1 || us < best_us) {
            best_us = us;
            best = s;
        }
    }
    return best;
}
// what the sums of split prefix blocks take at most, for this problem or any smaller one
size_t attn_vector_bwd_workspace(const cart_attn_desc& d) {
    if (d.P == 0) return 0;
    const size_t one = 2 * static_cast<size_t>(d.Hkv) * d.P * d.D * sizeof(float), most = 2 * static_cast<size_t>(device_cus()) * 16 * d.D * sizeof(float);
    return VEC_MAX_SPLITS * one < most ? VEC_MAX_SPLITS * one : most;
}

// One launch, each dK / dV block forming the delta of its rows itself: it does not wait for the dQ blocks, and a launch fewer
// (us, fp32, two launches -> one: 2 x 64 tokens, 2 / 1 heads of 64, 32 slots 21.0 -> 17.0; 4 x 256, 8 / 2, 256 slots 162 -> 134; of
// 128 375 -> 339).  The blocks read O's rows besides, and at head_dim up to 64 the dQ blocks share the kernel's 150 registers,
// a workgroup a CU where 125 allow two: with many blocks two launches are ahead.  500 random problems, blocks of dQ + 4 x of
// dK / dV per CU, two launches' time over one's: up to 4 1.47, 4 - 8 1.23, 8 - 12 1.11, 12 - 16 0.99, beyond 0.92 (3 x 560,
// 16 / 16 heads of 32: two 142, one 173); head_dim up to 128, blocks per CU: up to 16 1.18 with several query
// heads a KV head, beyond 0.95 (6 x 434, 24 / 8 of 96: two 637, one 668).  One query head a KV head, whose dK / dV blocks are as many as dQ's: a
// workgroup fills a CU in either form, so the one launch has to save a round (3 x 119, 16 / 16 of 96, 384 blocks of each kind: one
// 43.7, two 49.7; 5 x 94, 480: 52.1, 49.8); to 1.5 blocks per CU the launch and the wait saved outweigh that (1 x 164 28.9, 36.2),
// beyond 4 O's rows any round (7 x 208 two 211, one 242).  At 128 the one launch alone requests ahead: 1.1 with several heads a KV
// head, and with one (6 x 389, 8 / 8, 380 slots: two 472, one 430; 2 x 304, 16 / 16, 67: 134, 128; 6 x 349, 31: 204, 194).
// (Head_dim above 128: no registers for O's rows.)
static bool vec_one_launch(const cart_attn_desc& d, long n_q, long n_kv) {
    const long cus = device_cus();
    if (d.D <= 64) return n_q + 4 * n_kv <= 12 * cus;
    if (d.D >= 128) return d.D == 128;
    const long n = n_q + n_kv;
    auto rounds = [&](long blocks) { return (blocks + cus - 1) / cus; };
    if (d.Hq > d.Hkv) return n <= 16 * cus;
    return 2 * n <= 3 * cus || (n <= 4 * cus && rounds(n) < rounds(n_q) + rounds(n_kv));
}

template <typename T>
static void bwd_t(const cart_attn_desc& d, float scale, const void* q, const void* k, const void* v,
                  const void* zk, const void* zv, const void* o, const float* lse, const void* d_o,
                  void* dq, void* dk, void* dv, float* dzk, float* dzv, void* ws, hipStream_t st) {
    const long nSt = (d.S + 15) / 16, nPt = (d.P + 15) / 16;
    const int splits = dz_splits(d, d.D <= 64 ? 8 : 4);
    const long n_q = nSt * d.Hq * d.B, n_kv = (nPt * splits + nSt * d.B) * d.Hkv;
    const bool one = vec_one_launch(d, n_q, n_kv), ahead = d.D == 128;
    float* const part = reinterpret_cast<float*>(static_cast<char*>(ws) + ((static_cast<size_t>(d.B) * d.Hq * d.S * sizeof(float) + 255) & ~static_cast<size_t>(255)));
    const VecBwd<T> a = {(const T*)q, (const T*)k, (const T*)v, (const T*)zk, (const T*)zv, (const T*)o, (const T*)d_o, lse,
                         static_cast<float*>(ws), (T*)dq, (T*)dk, (T*)dv, dzk, dzv, d.B, d.S, d.Hq, d.Hkv, d.D, d.P, scale,
                         d.n_frozen, d.dz_accumulate, splits, part};
    trace_begin(st);   // kernel order: dq (+ delta), dk/dv/dz; or both in one (nothing between the second's events)
    CART_DISPATCH_NB(d.D, {
        if constexpr (NB <= 8) {
            if (one) {
                hipLaunchKernelGGL((ahead ? attn_bwd_vector<T, NB, NW, VEC_AHEAD<NB>> : attn_bwd_vector<T, NB, NW, false>), grid_of(n_q + n_kv), dim3(64 * NW), 0, st, a, static_cast<int>(n_kv));
                trace_mark(st);
            }
        }
        if (!one) {
            hipLaunchKernelGGL((attn_bwd_dq_vector<T, NB, NW>), grid_of(n_q), dim3(64 * NW), 0, st, a);
            trace_mark(st);
            hipLaunchKernelGGL((attn_bwd_dkv_vector<T, NB, NW>), grid_of(n_kv), dim3(64 * NW), 0, st, a);
        }
        trace_mark(st);
    });
    if (splits > 1) {
        const int n = d.Hkv * d.P * d.D;
        hipLaunchKernelGGL(attn_bwd_dz_vector, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st, part, dzk, dzv, n, d.P, d.D, splits,
                           scale, d.n_frozen, d.dz_accumulate);
        trace_mark(st);
    }
}

int launch_attn_bwd_vector(const cart_attn_desc& d, float scale, const void* q, const void* k,
                           const void* v, const void* zk, const void* zv, const void* o,
                           const float* lse, const void* d_o, void* dq, void* dk, void* dv,
                           float* dzk, float* dzv, void* ws, hipStream_t st) {
    if (d.dtype == CART_F32) bwd_t<float>(d, scale, q, k, v, zk, zv, o, lse, d_o, dq, dk, dv, dzk, dzv, ws, st);
    else bwd_t<bf16_t>(d, scale, q, k, v, zk, zv, o, lse, d_o, dq, dk, dv, dzk, dzv, ws, st);
    return static_cast<int>(hipGetLastError());
}

template <typename T>
static void dec_t(const cart_decode_desc& d, float scale, const void* q, const void* zk,
                  const void* zv, const void* k, const void* v, const int32_t* cu, void* o,
                  float* lse, hipStream_t st) {
    const long rows = static_cast<long>(d.B) * d.Hq;
    CART_DISPATCH_E(d.D, hipLaunchKernelGGL((decode_vector<T, E>), dim3(blocks_for(rows)),
        dim3(64 * VEC_WAVES), 0, st, (const T*)q, (const T*)zk, (const T*)zv, (const T*)k,
        (const T*)v, cu, (T*)o, lse, d.B, d.Hq, d.Hkv, d.D, d.P, scale));
}

int launch_decode_vector(const cart_decode_desc& d, float scale, const void* q, const void* zk,
                         const void* zv, const void* k, const void* v, const int32_t* cu,
                         void* o, float* lse, hipStream_t st) {
    trace_begin(st);
    if (d.dtype == CART_F32) dec_t<float>(d, scale, q, zk, zv, k, v, cu, o, lse, st);
    else dec_t<bf16_t>(d, scale, q, zk, zv, k, v, cu, o, lse, st);
    trace_mark(st);
    return static_cast<int>(hipGetLastError());
}

}  // namespace cart
