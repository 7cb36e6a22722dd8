// Context-distillation loss (Eq. 3, Sec. 4.2, over the teacher's recorded top entries of
// App. A.2) fused with its gradient.  Two readings of the truncated teacher (recorded terms only /
// plus a rest bucket) share the kernels: they differ in one per-row coefficient and in the k
// fix-ups; next-token cross-entropy is the case of one recorded token of probability 1.
//
// A row is cut into an aligned body of 16-byte vectors and up to 2 x (vector - 1) single elements
// around it (rows of a vocabulary that is not a multiple of the vector start anywhere); body and
// singles take the same arithmetic, so every vocabulary size and both data types run the same code.
//
// kl_row_resident: one workgroup per row, the row held in registers (fp32 rows of more than 65536
// logits: also in LDS), so HBM sees each logit read once and each gradient written once; what
// exceeds both is read twice.
#include "attn_mfma.h"
#include "logit_rows.h"

namespace cart {

// A row's K teacher records staged in LDS (four arrays of K words and one of halves, dynamic: at K = 20 they must not
// limit how many workgroups share a CU)
struct KlTeacher {
    uint16_t* own;      // the thread that stores the token's element (kl_owner), 0xffff for ignored entries; up to a multiple of 8
    int* idx;           // token, -1 for ignored entries
    float* t;           // exp(logp), 0 for ignored entries
    float* lp;
    float* x;           // student logit at idx (read before anything is overwritten)
};
extern __shared__ __attribute__((aligned(16))) int kl_records[];
__host__ __device__ inline int kl_up8(int K) { return (K + 7) & ~7; }
inline unsigned kl_record_bytes(int K) { return static_cast<unsigned>(kl_up8(K)) * 2u + static_cast<unsigned>(K) * 16u; }
__device__ __forceinline__ KlTeacher kl_teacher(int K) {
    int* idx = kl_records + kl_up8(K) / 2;
    float* f = reinterpret_cast<float*>(idx);
    return KlTeacher{reinterpret_cast<uint16_t*>(kl_records), idx, f + K, f + 2 * K, f + 3 * K};
}

// KL_n = sum_j t_j (logp_j - x_j + lse) (+ extra, the rest-bucket term), by the first wavefront
__device__ __forceinline__ void kl_row_value(int tid, const KlTeacher& tc, int K, float lse, float extra, float* out) {
    if (tid < CART_WAVE) {
        float a = 0.f;
        for (int j = tid; j < K; j += CART_WAVE) a += tc.t[j] * (tc.lp[j] - tc.x[j] + lse);
        a = wave_sum(a);
        if (tid == 0) *out = a + extra;
    }
}

// Rest-bucket mode, once the row's log2-sum-exp is known.  The first wavefront sums the student's
// mass on the recorded tokens, S = sum_j 2^(x_j log2e - lse2), and leaves in LDS the coefficient
// of the off-support gradient, (M - S) / (1 - S), and the row's extra term
// (1 - M)(log(1 - M) - log(1 - S)); the caller synchronises before reading them.  1 - M is
// floored at 0 and 1 - S at 2^-24, below which fp32 cannot resolve them.
__device__ __forceinline__ void kl_rest_terms(int tid, const KlTeacher& tc, int K, float lse2, float M, float* out2) {
    if (tid < CART_WAVE) {
        float a = 0.f;
        for (int j = tid; j < K; j += CART_WAVE)
            if (tc.idx[j] >= 0) a += fast_exp2(fmaf(tc.x[j], CART_LOG2E, -lse2));
        a = wave_sum(a);
        if (tid == 0) {
            const float rs = fmaxf(1.f - a, 5.9604645e-8f), rt = fmaxf(1.f - M, 0.f);
            out2[0] = (M - a) / rs;
            out2[1] = rt > 0.f ? rt * (__logf(rt) - __logf(rs)) : 0.f;
        }
    }
}

template <typename T> __device__ __forceinline__ u32x4 kl_fill() {
    constexpr uint32_t f = LogitVec<T>::FILL;
    return u32x4{f, f, f, f};
}
template <typename T> __device__ __forceinline__ float kl_vec_max(float mx, const u32x4& w) {
#pragma unroll
    for (int e = 0; e < LogitVec<T>::N; e += 2) mx = max3_raw(mx, LogitVec<T>::bits(w, e), LogitVec<T>::bits(w, e + 1));
    return mx;
}
// The largest of a thread's logits.  bf16: two at a time by their bits, which order as 16-bit integers do while one of them is
// positive (or a zero); where none is, the smallest as unsigned integers is the largest.  A third of the instructions of widening each.
template <typename T, int NV> __device__ __forceinline__ float kl_max(float mx, const u32x4 (&x)[NV]) {
    if constexpr (sizeof(T) == 2) {
        typedef short s16x2 __attribute__((ext_vector_type(2)));
        typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
        s16x2 m[4];                          // (a dependent packed instruction waits a slot)
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t w = x[i][e];
                m[e] = i == 0 ? __builtin_bit_cast(s16x2, w) : __builtin_elementwise_max(m[e], __builtin_bit_cast(s16x2, w));
            }
        m[0] = __builtin_elementwise_max(__builtin_elementwise_max(m[0], m[1]), __builtin_elementwise_max(m[2], m[3]));
        int top = max(static_cast<int>(m[0][0]), static_cast<int>(m[0][1]));
        if (__any(top < 0)) {
            u16x2 l[4];
#pragma unroll
            for (int i = 0; i < NV; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t w = x[i][e];
                    l[e] = i == 0 ? __builtin_bit_cast(u16x2, w) : __builtin_elementwise_min(l[e], __builtin_bit_cast(u16x2, w));
                }
            l[0] = __builtin_elementwise_min(__builtin_elementwise_min(l[0], l[1]), __builtin_elementwise_min(l[2], l[3]));
            if (top < 0) top = min(static_cast<int>(l[0][0]), static_cast<int>(l[0][1]));
        }
        const uint32_t b = static_cast<uint32_t>(top) << 16;
        return max3_raw(mx, b, b);
    } else {
#pragma unroll
        for (int i = 0; i < NV; ++i) mx = kl_vec_max<T>(mx, x[i]);
        return mx;
    }
}
// s0 + s1 += sum of 2^(x log2e + c0)
template <typename T> __device__ __forceinline__ void kl_vec_sum(float& s0, float& s1, const u32x4& w, float c0) {
#pragma unroll
    for (int e = 0; e < LogitVec<T>::N; e += 2) {
        s0 += fast_exp2(fmaf(__uint_as_float(LogitVec<T>::bits(w, e)), CART_LOG2E, c0));
        s1 += fast_exp2(fmaf(__uint_as_float(LogitVec<T>::bits(w, e + 1)), CART_LOG2E, c0));
    }
}
// Gradient off the recorded tokens: g = c 2^(x log2e - lse2), c = scale * M (rest-bucket mode: scale *
// (M - S) / (1 - S)).  bf16: |c| rides in the exponent (c == 0 gives 2^-inf = 0).
struct KlGrad {
    float c, off;
    uint32_t sgn;
};
template <typename T> __device__ __forceinline__ KlGrad kl_grad_coef(float c, float lse2) {
    if (sizeof(T) == 2) return KlGrad{c, -(lse2 - fast_log2(fabsf(c))), static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(c < 0.f ? 0x80008000u : 0u))};
    return KlGrad{c, -lse2, 0u};
}
template <typename T> __device__ __forceinline__ u32x4 kl_vec_grad(const u32x4& w, const KlGrad& g) {
    u32x4 r;
    if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float lo = fast_exp2(fmaf(__uint_as_float(w[e] << 16), CART_LOG2E, g.off));
            const float hi = fast_exp2(fmaf(__uint_as_float(w[e] & 0xffff0000u), CART_LOG2E, g.off));
            r[e] = pack_bf16x2(lo, hi);
        }
        if (g.sgn) {
            asm volatile("");            // (a branch, seldom taken)
            r ^= g.sgn;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            r[e] = __float_as_uint(g.c * fast_exp2(fmaf(__uint_as_float(w[e]), CART_LOG2E, g.off)));
    }
    return r;
}

// A row's vectors in slots that start at a 128-byte line of the tensor: the first `lead` slots of a row
// that starts inside a line belong to the row before it (they are loaded, never used nor stored), and a
// wavefront's store covers whole lines.  With the row's first vector in slot 0 every wavefront wrote two
// parts of lines (4096 rows, us a call: 50257 bf16 181 -> 170, fp32 354 -> 322; 80001 bf16 327 -> 309, fp32
// 551 -> 493).  Rows that nearly fill the registers start at a half or a quarter of a line instead: a wider workgroup, or
// reading the last slots twice, costs more (4096 x 4099 bf16 22.5 us; at twice the width 31.6).
struct KlRow : LogitRow {
    int lead, nslot;    // nslot = lead + nvec
};
template <typename T> __device__ __forceinline__ KlRow kl_row(int n, int V, int lead_mask) {
    KlRow r;
    static_cast<LogitRow&>(r) = logit_row<T>(n, V);
    r.lead = r.nvec > 0 ? static_cast<int>((r.row + r.head) / LogitVec<T>::N) & (lead_mask & 7) : 0;
    r.nslot = r.lead + r.nvec;
    return r;
}
// the thread (of THREADS) that stores element id
template <typename T, int THREADS> __device__ __forceinline__ int kl_owner(const KlRow& r, int id) {
    const int e = id - r.head, v = e / LogitVec<T>::N;
    return e < 0 ? id : v < r.nvec ? (v + r.lead) & (THREADS - 1) : id - r.nvec * LogitVec<T>::N;
}

// The slots of a row as a buffer resource: a load past its end returns 0 and a store past it is
// dropped, and an access takes one 32-bit offset instead of a 64-bit address and a predicate.  Rows of more
// than 1 GB (LONG) reach only their first vectors so: a resource ends below KL_DROP and its offsets below 4 GB.
struct KlBuf {
    __amdgpu_buffer_rsrc_t r;
};
constexpr int KL_DROP = 0x7ffffff0;  // an offset past every resource
template <typename T> __device__ __forceinline__ const T* kl_slots(const T* base, const KlRow& r) {
    return base + (r.row + r.head - static_cast<size_t>(r.lead) * LogitVec<T>::N);
}
template <bool LONG, typename T> __device__ __forceinline__ KlBuf kl_buf(const T* base, const KlRow& r) {
    return KlBuf{__builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(kl_slots(base, r)), 0,
                                                   (LONG ? KL_DROP / 16 : r.nslot) * 16, 0x00027000)};
}
constexpr int KL_NT = 2;             // cache policy: non-temporal
constexpr int KL_AHEAD = 4;          // turns ahead of its use that a vector which is not resident is requested
// what of a row is not resident: nothing; read a turn at a time; KL_AHEAD turns ahead (see launch_rows)
enum KlRemainder { KL_NONE, KL_BY_TURN, KL_TURNS_AHEAD };
template <int AUX> __device__ __forceinline__ u32x4 kl_ld(const KlBuf& b, int off) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(b.r, off, 0, AUX));
}
__device__ __forceinline__ void kl_st(const KlBuf& b, u32x4 w, int off) {
    __builtin_amdgcn_raw_buffer_store_b128(w, b.r, off, 0, KL_NT);
}

// Makes the register-resident row opaque to the optimiser between sweeps; otherwise the
// unpacked fp32 copies of one sweep are kept alive for the next one and spill.
#define KL_FORGET(x)                                                                      \
    _Pragma("unroll") for (int i_ = 0; i_ < NV; ++i_)                                   \
        asm volatile("" : "+v"(x[i_]))

// One row per workgroup at a time: THREADS x (NV vectors in registers + NL in LDS) are resident, the
// rest of a longer row is read twice.  The launcher takes the smallest of 128 x 4 and 256 x 4 (2048 such threads a CU, 64
// registers each), 256 x 16 (four workgroups per CU cover each other's loads and reductions), 512 x 16 and
// 1024 x 16 (1024 a CU, 128 registers each) whose registers hold the row.  At 1024 nothing else runs on the CU:
// the workgroup walks rows n, n + gridDim.x, ... and fetches the next row's vectors and teacher
// records into the registers (LDS slots) of the current row as its last sweep releases them.
// Bound by HBM, one read and one write of the tensor.  Kernel time in us against one-workgroup-per-
// row kernels that took whole-vector bf16 rows at 1024 threads whatever their length and read every
// other row twice, element by element (rows x vocabulary):
//   16384 x 128256 bf16  1649 -> 1593 (5.28 TB/s)     4096 x 32000 bf16  153 -> 100
//    1024 x  50257 bf16   146 ->   47                16384 x  1000 fp32   54 ->  47
//    2048 x 128256 fp32   785 ->  397 (10 more without the LDS part)
// Rows of whole vectors leave the arithmetic little to hide behind, so it is kept short: the maxima two at a time, what is past the
// row's end and a negative coefficient behind branches.  And nothing lives in scratch (but three registers of bf16 rows past 1 GB): the thread's number is opaque each row, or what
// follows from it (LDS and record addresses) is kept across the sweeps at the price of up to 26 registers' reloads, each of which waits
// for every store and load ahead of it.  Both, and the groups of the last sweep (us a call): 16384 x 128256 bf16 1557 -> 1530, 4000 402 ->
// 391, 200 26.0 -> 22.2; 1024 x 50257 bf16 44.4 -> 41.5; 16000 x 32000 bf16 387 -> 384; 2048 x 128256 fp32 400 -> 386 (8192 x 32000 371 -> 374,
// 25001 296 -> 291).
// PF: at 1024 threads the CU has nothing to send for while its one workgroup forms maxima and sums.  The first PF vectors of the next row
// are requested into LDS ahead of them, the others by the last sweep as ever (us a call, bf16: 16384 x 128256 1529 -> 1502, 600 71.0 ->
// 67.7, 4000 x 100000 318 -> 301, x 66000 232 -> 229; four of the sixteen 1581; requested as early as the last sweep 1544.  fp32 rows,
// whose sums are half as long, 380 -> 385; workgroups of 512, two a CU, 277 -> 282).
template <typename T, int THREADS, int NV, int NL, KlRemainder REM, bool LONG = false, int PF = 0>
__global__ __launch_bounds__(THREADS, NV > 4 ? 4 : 8) void kl_row_resident(const T* logits, const int32_t* idx,
                                                              const float* logp, T* dlogits, float* row_kl,
                                                              int N, int V, int K, float scale, int mode /* rest bucket | lead mask << 1 */) {
    constexpr int GRP = PF > 0 ? PF : NV < 8 ? NV : THREADS == 1024 || (THREADS == 512 && sizeof(T) == 2) ? 16 : 8;
    constexpr int NW = THREADS / CART_WAVE, VE = LogitVec<T>::N;
    const KlTeacher tc = kl_teacher(K);
    __shared__ float red_c[NW], red_m[NW], red_sum[NW], rest_terms[2];
    __shared__ __attribute__((aligned(16))) u32x4 lds_x[NL + PF > 0 ? (NL + PF) * THREADS : 1];
    int tid = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    int n = blockIdx.x;
    if (n >= N) return;
    KlRow R = kl_row<T>(n, V, mode >> 1);

    // vector i of the next row's LDS part, straight into the thread's own slot (clamped to the row)
    auto lds_fetch = [&](const T* base, const KlRow& r, int i) __attribute__((always_inline)) {
        const int v = min((NV + i) * THREADS + tid, max(r.nslot - 1, 0));
        mfma::dma16(reinterpret_cast<const char*>(kl_slots(base, r)), static_cast<uint32_t>(v) * 16u,
                    mfma::lds_addr(lds_x + i * THREADS + wv * CART_WAVE));
    };
    // the first PF vectors of a row to come, likewise
    auto fetch_ahead = [&](int m) __attribute__((always_inline)) {
        const KlRow r = kl_row<T>(m, V, mode >> 1);
        const char* const base = reinterpret_cast<const char*>(kl_slots(logits, r));
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the slots have been read
#pragma unroll
        for (int i = 0; i < PF; ++i)
            mfma::dma16_nt(base, static_cast<uint32_t>(min(i * THREADS + tid, max(r.nslot - 1, 0))) * 16u,
                           mfma::lds_addr(lds_x + i * THREADS + wv * CART_WAVE));
    };
    u32x4 x[NV];
    constexpr int STEP = THREADS * 16;
    float xs = -3.0e38f;          // the thread's single element
    int my_id = -1;               // the thread's teacher record (record tid; more of them by a loop)
    float my_lp = 0.f, my_x = 0.f;
    // The records of row m are two dependent round trips: tokens and log-probabilities first ...
    auto fetch_record = [&](int m) __attribute__((always_inline)) {
        if (tid < K) {
            my_id = idx[static_cast<size_t>(m) * K + tid];
            if (logp) my_lp = logp[static_cast<size_t>(m) * K + tid];
        }
    };
    // ... then the logits of the tokens
    auto fetch_logit = [&](const LogitRow& r) __attribute__((always_inline)) {
        if (my_id >= V) my_id = -1;
        if (my_id >= 0) my_x = elem<T>::load(logits + r.row + my_id);
    };
    {
        const KlBuf src = kl_buf<LONG>(logits, R);
        fetch_record(n);          // (ahead of the row: what depends on it need not wait for the row)
#pragma unroll
        for (int i = 0; i < NV; ++i) x[i] = kl_ld<KL_NT>(src, tid * 16 + i * STEP);
        if constexpr (NL > 0) {
#pragma unroll
            for (int i = 0; i < NL; ++i) lds_fetch(logits, R, i);
        }
        if (tid < R.head + R.tail) xs = elem<T>::load(logits + R.row + logit_single<T>(R, tid));
        fetch_logit(R);
        if constexpr (PF > 0) {
            if (n + static_cast<int>(gridDim.x) < N) fetch_ahead(n + static_cast<int>(gridDim.x));
        }
    }
    for (;;) {
        asm volatile("" : "+v"(tid));
        // teacher records into LDS
        float m_part = 0.f;
        for (int j = tid; j < K; j += THREADS) {
            int id = my_id;
            float lp = my_lp, xj = my_x;
            if (j >= THREADS) {        // (more records than threads)
                id = idx[static_cast<size_t>(n) * K + j];
                lp = logp ? logp[static_cast<size_t>(n) * K + j] : 0.f;
                if (id < 0 || id >= V) id = -1;
                xj = id >= 0 ? elem<T>::load(logits + R.row + id) : 0.f;
            }
            const float t = id >= 0 ? __expf(lp) : 0.f;
            tc.own[j] = static_cast<uint16_t>(id >= 0 ? kl_owner<T, THREADS>(R, id) : 0xffff);
            tc.idx[j] = id >= 0 ? id : -1;
            tc.t[j] = t;
            tc.lp[j] = id >= 0 ? lp : 0.f;
            tc.x[j] = id >= 0 ? xj : 0.f;
            m_part += t;
        }
        if (tid < kl_up8(K) - K) tc.own[K + tid] = 0xffff;
        const int n_next = n + static_cast<int>(gridDim.x);
        const bool more = n_next < N;
        if (more) fetch_record(n_next);

        // sweep 1, the thread's maximum.  It is the thread's own reference for the exponentials (no
        // barrier between the sweeps); kept above -2e38 so that c0 stays finite.
        float mx = fmaxf(xs, -2.0e38f);
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if ((i + 1) * THREADS > R.nslot) {
                asm volatile("");        // (a branch, seldom taken: selects for every vector else)
                if (i * THREADS + tid >= R.nslot) x[i] = kl_fill<T>();
            }
        if (tid < R.lead) x[0] = kl_fill<T>();
        mx = kl_max<T>(mx, x);
        if constexpr (NL > 0) {
            mfma::dma_wait();            // the LDS part (each thread reads only what its own lane fetched)
#pragma unroll
            for (int i = 0; i < NL; ++i)
                if ((NV + i) * THREADS + tid < R.nslot) mx = kl_vec_max<T>(mx, lds_x[i * THREADS + tid]);
        }
        KL_FORGET(x);
        // sweep 2: sum of 2^((x - reference) log2e)
        float c0 = -mx * CART_LOG2E;
        float s0 = fast_exp2(fmaf(xs, CART_LOG2E, c0)), s1 = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (i * THREADS < R.nslot) kl_vec_sum<T>(s0, s1, x[i], c0);
            asm volatile("" : "+v"(s0), "+v"(s1));   // summed here: the compiler would sink the adds behind all the exponentials
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (NL > 0) {
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                if ((NV + i) * THREADS + tid < R.nslot) kl_vec_sum<T>(s0, s1, lds_x[i * THREADS + tid], c0);
                asm volatile("" : "+v"(s0), "+v"(s1));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        KL_FORGET(x);
        float sum = s0 + s1;
        const KlBuf src = kl_buf<LONG>(logits, R), dst = kl_buf<LONG>(dlogits, R);
        // What is not resident; KL_TURNS_AHEAD: each vector requested KL_AHEAD turns ahead of its use (past the row's end:
        // zeros).  One at a time, every turn is a round trip to memory with nothing else on the CU (us a call when it was chosen, 2048 rows
        // of 128256 fp32 logits 421, 2 / 3 / 4 / 6 / 8 ahead 410 / 408 / 403 / 406 / 408; the two forms now: see kl_ahead).
        constexpr int REST = (NV + NL) * THREADS;
        auto rest = [&](int v) __attribute__((always_inline)) {
            if constexpr (LONG) return reinterpret_cast<const u32x4*>(kl_slots(logits, R))[min(v, max(R.nslot - 1, 0))];
            else return kl_ld<0>(src, v * 16);
        };
        auto rest_sum = [&](const u32x4& w) __attribute__((always_inline)) {
            const float m1 = kl_vec_max<T>(mx, w);
            if (m1 > mx) {
                const float c1 = -m1 * CART_LOG2E;
                sum *= fast_exp2(c1 - c0);
                mx = m1;
                c0 = c1;
            }
            s0 = s1 = 0.f;
            kl_vec_sum<T>(s0, s1, w, c0);
            sum += s0 + s1;
        };
        if constexpr (REM == KL_BY_TURN) {
            for (int v = REST + tid; v < R.nslot; v += THREADS) rest_sum(rest(v));
        } else if constexpr (REM == KL_TURNS_AHEAD) {
            u32x4 w[KL_AHEAD];
#pragma unroll
            for (int i = 0; i < KL_AHEAD; ++i) w[i] = rest(REST + i * THREADS + tid);
            for (int v0 = REST; v0 < R.nslot; v0 += KL_AHEAD * THREADS) {
#pragma unroll
                for (int i = 0; i < KL_AHEAD; ++i) {
                    if (i > 0 && v0 + i * THREADS >= R.nslot) break;
                    const int v = v0 + i * THREADS + tid;
                    u32x4 wi = w[i];
                    w[i] = rest(v + KL_AHEAD * THREADS);
                    if (v >= R.nslot) wi = kl_fill<T>();
                    rest_sum(wi);
                }
            }
        }
        // the row's sum, relative to the largest reference
        const float wc = -wave_max(-c0);
        sum = wave_sum(sum * fast_exp2(wc - c0));
        m_part = wave_sum(m_part);
        if ((tid & 63) == 0) { red_c[wv] = wc; red_sum[wv] = sum; red_m[wv] = m_part; }
        __syncthreads();
        float M = 0.f, gc = red_c[0];
#pragma unroll
        for (int w = 0; w < NW; ++w) { gc = fminf(gc, red_c[w]); M += red_m[w]; }
        sum = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) sum += red_sum[w] * fast_exp2(gc - red_c[w]);
        const float lse2 = fast_log2(sum) - gc;          // log2 of the softmax denominator

        // sweep 3: the gradient, a group of vectors at a time: their stores, then the loads of the same
        // vectors of the next row into their registers.  One store and one load in turn turns the
        // memory bus around too often (16384 rows of 128256 bf16 logits, us: groups of 1 / 2 / 4 / 8 /
        // 16 vectors -> 1674 / 1672 / 1627 / 1605 / 1603; 2048 fp32 rows: 434 / 433 / 426 / 419 / 415).  Where more than one
        // workgroup shares a CU groups of 8 do as well or better, but for bf16 in two of them (8 / 16: 8192 x 50257 bf16 308 / 304;
        // 8192 x 32000 fp32 374 / 379; 16000 x 32000 bf16 384 / 389; 4000 x 100000 bf16, alone on the CU 325 / 315).
        float coef = M, extra = 0.f;
        if (mode & 1) {
            kl_rest_terms(tid, tc, K, lse2, M, rest_terms);
            __syncthreads();
            coef = rest_terms[0];
            extra = rest_terms[1];
        }
        const KlGrad g = kl_grad_coef<T>(scale * coef, lse2);
        const KlRow Rn = kl_row<T>(more ? n_next : n, V, mode >> 1);
        if (more) fetch_logit(Rn);
        if (tid < R.head + R.tail)
            elem<T>::store(dlogits + R.row + logit_single<T>(R, tid), g.c * fast_exp2(fmaf(xs, CART_LOG2E, -lse2)));
        xs = -3.0e38f;
        if (more && tid < Rn.head + Rn.tail) xs = elem<T>::load(logits + Rn.row + logit_single<T>(Rn, tid));
        // (the last read of these vectors, as the stores next to it: 512 rows of 300000 fp32 288 -> 265, 1024 of 200000 347 -> 328)
        auto rest_nt = [&](int v) __attribute__((always_inline)) {
            if constexpr (LONG) return rest(v);
            else return kl_ld<KL_NT>(src, v * 16);
        };
        auto rest_grad = [&](int v, const u32x4& w) __attribute__((always_inline)) {
            if constexpr (LONG) {
                if (v < R.nslot) reinterpret_cast<u32x4*>(const_cast<T*>(kl_slots(dlogits, R)))[v] = kl_vec_grad<T>(w, g);
            } else {
                kl_st(dst, kl_vec_grad<T>(w, g), v * 16);
            }
        };
        if constexpr (REM == KL_BY_TURN) {
            for (int v = REST + tid; v < R.nslot; v += THREADS) rest_grad(v, kl_ld<KL_NT>(src, v * 16));
        } else if constexpr (REM == KL_TURNS_AHEAD) {
            u32x4 w[KL_AHEAD];
#pragma unroll
            for (int i = 0; i < KL_AHEAD; ++i) w[i] = rest_nt(REST + i * THREADS + tid);
            for (int v0 = REST; v0 < R.nslot; v0 += KL_AHEAD * THREADS) {
#pragma unroll
                for (int i = 0; i < KL_AHEAD; ++i) {
                    if (i > 0 && v0 + i * THREADS >= R.nslot) break;
                    const int v = v0 + i * THREADS + tid;
                    const u32x4 wi = w[i];
                    w[i] = rest_nt(v + KL_AHEAD * THREADS);
                    rest_grad(v, wi);
                }
            }
        }
        const KlBuf src_next = kl_buf<LONG>(logits, Rn);
#pragma unroll
        for (int i0 = 0; i0 < NV; i0 += GRP) {
#pragma unroll
            for (int i = i0; i < i0 + GRP; ++i) {
                if (i * THREADS < R.nslot) kl_st(dst, kl_vec_grad<T>(x[i], g), i == 0 && tid < R.lead ? KL_DROP : tid * 16 + i * STEP);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (more && i0 >= PF) {
#pragma unroll
                for (int i = i0; i < i0 + GRP; ++i) x[i] = kl_ld<KL_NT>(src_next, tid * 16 + i * STEP);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (NL > 0) {
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                kl_st(dst, kl_vec_grad<T>(lds_x[i * THREADS + tid], g), tid * 16 + (NV + i) * STEP);
                __builtin_amdgcn_sched_barrier(0);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the slots have been read
            if (more) {
#pragma unroll
                for (int i = 0; i < NL; ++i) lds_fetch(logits, Rn, i);
            }
        }
        // recorded tokens: the thread that stored the element's vector rewrites that element, so
        // the two stores to one address are in program order.  Every thread passes every record, eight owners
        // a read, and a wavefront's threads rewrite the first of their own at one time, then the second.  (One
        // record after the other, its owner worked out on the spot: 1000 records, 4096 rows of 32000 fp32 logits 1425 us, now 390; 20
        // records, 1024 x 50257 bf16 47.5, now 42.9.  Reading further ahead or sixteen owners at a time costs spills: 4096 x 4104
        // bf16, 20 records 24.8, sixteen 29.3.)
#pragma unroll 1
        for (int j0 = 0; j0 < K; j0 += 8) {
            const u32x4 o = *reinterpret_cast<const u32x4*>(tc.own + j0);
            uint32_t mine = 0u;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (((o[e >> 1] >> (16 * (e & 1))) & 0xffffu) == static_cast<uint32_t>(tid)) mine |= 1u << e;
            while (mine) {
                const int j = j0 + __builtin_ctz(mine);
                mine &= mine - 1;
                const float s = fast_exp2(fmaf(tc.x[j], CART_LOG2E, -lse2));
                elem<T>::store(dlogits + R.row + tc.idx[j], scale * ((mode & 1 ? 1.f : M) * s - tc.t[j]));
            }
        }
        kl_row_value(tid, tc, K, lse2 * CART_LN2, extra, row_kl + n);
        if (!more) break;
        n = n_next;
        R = Rn;
        __syncthreads();    // the teacher staging area and the reduction arrays are reused
        if constexpr (PF > 0) {
            // The wait is for everything: the first half, requested a row ago, the gradient's stores, and the second half requested
            // behind them, whose maxima are formed next in any case.  The row after it is requested once all that is there.
            mfma::dma_wait();
#pragma unroll
            for (int i = 0; i < PF; ++i) x[i] = lds_x[i * THREADS + tid];
            if (n + static_cast<int>(gridDim.x) < N) fetch_ahead(n + static_cast<int>(gridDim.x));
        }
    }
}

// loss = scale * sum_n row_kl[n]: one workgroup, fixed summation order, fp64 accumulation.  A launch and a few
// round trips: 16384 rows 5.8 -> 4.0 us with two barriers' worth of tree instead of eleven.
__global__ __launch_bounds__(1024) void kl_reduce_rows(const float* row_kl, int N, float scale,
                                                       float* loss) {
    __shared__ double red[1024 / CART_WAVE];
    double a = 0.0;
#pragma unroll 8
    for (int i = threadIdx.x; i < N; i += 1024) a += static_cast<double>(row_kl[i]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, CART_WAVE);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
        a = red[0];
#pragma unroll
        for (int w = 1; w < 1024 / CART_WAVE; ++w) a += red[w];
        *loss = static_cast<float>(static_cast<double>(scale) * a);
    }
}

template <typename T, int THREADS, int NV, int NL, KlRemainder REM = KL_NONE, bool LONG = false, int PF = 0>
static void resident(const cart_kl_desc& d, const void* logits, const int32_t* idx, const float* logp, void* d_logits,
                     float* rows, hipStream_t st) {
    const int slots = device_cus() * ((NV > 4 ? 1024 : 2048) / THREADS);      // workgroups the chip keeps resident
    const int spare = (NV + NL) * THREADS - d.V / LogitVec<T>::N;
    const int lead_mask = spare < 0 || spare >= 7 ? 7 : spare >= 3 ? 3 : spare >= 1 ? 1 : 0;
    hipLaunchKernelGGL((kl_row_resident<T, THREADS, NV, NL, REM, LONG, PF>), dim3(static_cast<unsigned>(d.N < slots ? d.N : slots)),
                       dim3(THREADS), kl_record_bytes(d.K), st, static_cast<const T*>(logits), idx, logp,
                       static_cast<T*>(d_logits), rows, d.N, d.V, d.K, d.scale, (d.mode == CART_KL_REST ? 1 : 0) | lead_mask << 1);
}
// Whether a remainder of `rest` vectors is requested ahead.  Up to two turns there is nothing to request ahead; and with few turns of rows
// on few CUs memory answers a turn sooner than the longer loop's code arrives.
// fp32, us a call one at a time / ahead:  rows        32             65             128            256            1024
//   103122, 2 turns                              17.5 / 18.1    18.7 / 19.3    24.4 / 24.8    39.8 / 40.3    156.0 / 157.7
//   110000, 3                                    18.8 / 19.0    19.8 / 19.9    25.5 / 25.2    42.4 / 42.1    175.1 / 171.7
//   128256, 8                                    21.1 / 21.4    23.1 / 22.5    29.3 / 28.6    48.2 / 47.9    205.6 / 196.7
//   200000, 25                                   33.8 / 31.2    35.5 / 32.4    48.1 / 43.6    80.2 / 76.9    341.1 / 318.7
// (bf16 alike: 145000, 2 turns, 1024 rows 116.8 / 117.7; 160000, 4 turns 128.0 / 127.6, 64 rows 20.9 / 21.2)
static bool kl_ahead(long rest, int rows) {
    const long turns = (rest + 1023) / 1024;
    return turns > 2 && (2L * rows >= device_cus() || turns * rows >= 2L * device_cus() || turns > 12);
}
template <typename T, int NL>
static void launch_rows(const cart_kl_desc& d, const void* logits, const int32_t* idx, const float* logp, void* d_logits,
                        float* rows, hipStream_t st) {
    const long nvec = d.V / LogitVec<T>::N;
    if (nvec <= 128 * 4) resident<T, 128, 4, 0>(d, logits, idx, logp, d_logits, rows, st);
    else if (nvec <= 256 * 4) resident<T, 256, 4, 0>(d, logits, idx, logp, d_logits, rows, st);
    else if (nvec <= 256 * 16) resident<T, 256, 16, 0>(d, logits, idx, logp, d_logits, rows, st);
    else if (nvec <= 512 * 16) resident<T, 512, 16, 0>(d, logits, idx, logp, d_logits, rows, st);
    else if (nvec <= 1024 * 16) resident<T, 1024, 16, 0, KL_NONE, false, sizeof(T) == 2 ? 8 : 0>(d, logits, idx, logp, d_logits, rows, st);
    else if (nvec >= 1L << 26) resident<T, 1024, 16, NL, KL_TURNS_AHEAD, true>(d, logits, idx, logp, d_logits, rows, st);
    else if (kl_ahead(nvec - 1024 * (16 + NL), d.N)) resident<T, 1024, 16, NL, KL_TURNS_AHEAD>(d, logits, idx, logp, d_logits, rows, st);
    else resident<T, 1024, 16, NL, KL_BY_TURN>(d, logits, idx, logp, d_logits, rows, st);
}

int launch_kl(const cart_kl_desc& d, const void* logits, const int32_t* idx, const float* logp,
              float* loss, void* d_logits, float* row_kl, void* ws, hipStream_t st) {
    float* rows = row_kl ? row_kl : static_cast<float*>(ws);
    trace_begin(st);   // kernel order: row kernel, loss reduce
    // (a bf16 row too long for the registers alone is rare: no LDS part for it)
    if (d.logits_dtype == CART_BF16) launch_rows<bf16_t, 0>(d, logits, idx, logp, d_logits, rows, st);
    else launch_rows<float, 8>(d, logits, idx, logp, d_logits, rows, st);
    trace_mark(st);
    hipLaunchKernelGGL(kl_reduce_rows, dim3(1), dim3(1024), 0, st, rows, d.N, d.scale, loss);
    trace_mark(st);
    return static_cast<int>(hipGetLastError());
}

}  // namespace cart
