// Teacher records (App. A.2 "Training Objective": the top output probabilities of the teacher are
// collected while it generates): per position, the K most probable tokens and their
// log-probabilities, by descending probability, the lower token index first among equal logits.
//
// topk_row: one workgroup per position, one pass over its logits.  Every vocabulary size and both
// data types: a row is an aligned body of 16-byte vectors and up to 14 single elements around it.
#include "logit_rows.h"

namespace cart {

// order-preserving 32-bit key of an fp32 (a bf16 widened to fp32): larger key <=> larger value
__device__ __forceinline__ uint32_t f32_key(float x) {
    uint32_t u = __float_as_uint(x);
    if (u == 0x80000000u) u = 0u;        // -0 and +0 are one value (ties go by index)
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float f32_key_value(uint32_t key) {
    return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

// (key, index) -> one 64-bit word whose order is "larger value first, then lower index"
__device__ __forceinline__ uint64_t order_word(uint32_t key, uint32_t idx) {
    return (static_cast<uint64_t>(key) << 32) | (0xffffffffu - idx);
}
__device__ __forceinline__ uint32_t word_index(uint64_t w) { return 0xffffffffu - static_cast<uint32_t>(w); }

// Every listed logit counts the listed ones that precede it: that is its output position (positions from K on are dropped).
template <int THREADS>
__device__ __forceinline__ void write_ranked(const uint64_t* list, int cnt, int K, int32_t* idx_out, float* logp_out, float lse) {
    const ulonglong2* pairs = reinterpret_cast<const ulonglong2*>(list);
    for (int t = threadIdx.x; t < cnt; t += THREADS) {
        const uint64_t me = list[t];
        int rank = 0;
#pragma unroll 4
        for (int j = 0; j < cnt / 2; ++j) {
            const ulonglong2 w = pairs[j];
            rank += (w.x > me) + (w.y > me);
        }
        if (cnt & 1) rank += list[cnt - 1] > me;
        if (rank < K) {
            idx_out[rank] = static_cast<int32_t>(word_index(me));
            logp_out[rank] = f32_key_value(static_cast<uint32_t>(me >> 32)) - lse;
        }
    }
}

// Lists the K best of a row, whatever it holds, and at most a quarter more (or 128); returns how many.  The K-th largest key two
// bits at a time, and where too many logits reach it the index of the last of its equals that belongs, two bits at a
// time too; each step counts the row's logits against three candidates.  The row is read again for every step, from
// cache: 16 steps at most for the key of an fp32 (8 of a bf16), fewer where a candidate leaves few enough.  (K rounds of "the best one below the last winner" instead, us: 4096
// rows of 1024 bf16 logits, K = 1024 15300, now 268; of 4096, K = 600 10780, now 191;
// of 32000, K = 1000 10460, now 3420; 16384 of 256, K = 40 404, now 59.)
template <typename T, int THREADS, int CAP>
__device__ __forceinline__ int list_best(const T* row, const LogitRow& R, int V, int K, int (*count)[4], uint64_t* list, int* list_n) {
    constexpr int VE = LogitVec<T>::N, LOW_BIT = sizeof(T) == 2 ? 16 : 0;      // (the keys of bf16 values differ in their upper halves)
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const u32x4* src = reinterpret_cast<const u32x4*>(row + R.head);
    // f(upper bits of the key, index, whether there is such a logit), whole wavefronts at a time
    auto each = [&](auto f) __attribute__((always_inline)) {
        for (int v0 = wv * CART_WAVE; v0 < R.nvec; v0 += THREADS) {
            const int v = v0 + lane;
            const bool ok = v < R.nvec;
            const u32x4 w = src[ok ? v : 0];
#pragma unroll
            for (int e = 0; e < VE; ++e)
                f(f32_key(__uint_as_float(LogitVec<T>::bits(w, e))) >> LOW_BIT, static_cast<uint32_t>(R.head + VE * v + e), ok);
        }
        if (wv == 0) {
            const bool ok = lane < R.head + R.tail;
            const int i = ok ? logit_single<T>(R, lane) : 0;
            f(f32_key(elem<T>::load(row + i)) >> LOW_BIT, static_cast<uint32_t>(i), ok);
        }
    };
    // The row's logits for which each of three conditions holds.  Counters in rotation: those of the next step
    // are cleared while everyone is past the barrier behind which they were last read.
    int step = 0;
    auto count3 = [&](auto cond, int (&c)[3]) __attribute__((always_inline)) {
        int n[3] = {0, 0, 0};
        each([&](uint32_t key, uint32_t i, bool ok) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 3; ++j) n[j] += __popcll(__ballot(ok && cond(key, i, j)));
        });
        const int next = step == 2 ? 0 : step + 1;
        if (tid < 3) count[next][tid] = 0;
        if (lane < 3) atomicAdd(&count[step][lane], lane == 0 ? n[0] : lane == 1 ? n[1] : n[2]);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 3; ++j) c[j] = count[step][j];
        step = next;
    };
    __syncthreads();                        // (the counters and the list's may still be read)
    if (tid < 3) count[0][tid] = 0;
    if (tid == 0) *list_n = 0;
    __syncthreads();
    // t: the K-th key as far as decided, reached by `ge` logits; `gt` logits lie above all keys that begin like it
    uint32_t t = 0, upto = 0xffffffffu;
    const int most = min(max(K + K / 4, 128), CAP);          // (ranking 128 is cheaper than a step)
    int ge = V, gt = 0;
    for (int bit = 30 - LOW_BIT; bit >= 0 && ge > most; bit -= 2) {
        int c[3];
        count3([&](uint32_t key, uint32_t, int j) __attribute__((always_inline)) { return key >= (t | static_cast<uint32_t>(j + 1) << bit); }, c);
        const int j = (c[0] >= K) + (c[1] >= K) + (c[2] >= K);
        gt = j == 0 ? c[0] : j == 1 ? c[1] : j == 2 ? c[2] : gt;
        ge = j == 0 ? ge : c[j - 1];
        t |= static_cast<uint32_t>(j) << bit;
    }
    if (ge > most) {                        // t is the K-th key itself: of its equals the K - gt with the lowest indices
        uint32_t last = 0;
        for (int bit = (31 - __clz(V)) & ~1; bit >= 0; bit -= 2) {
            int c[3];
            count3([&](uint32_t key, uint32_t i, int j) __attribute__((always_inline)) {
                return key == t && i < (last | static_cast<uint32_t>(j + 1) << bit);
            }, c);
            last |= static_cast<uint32_t>((c[0] < K - gt) + (c[1] < K - gt) + (c[2] < K - gt)) << bit;
        }
        upto = last;
        ge = K;
    }
    each([&](uint32_t key, uint32_t i, bool ok) __attribute__((always_inline)) {
        if (ok && (key > t || (key == t && i <= upto))) {
            const int pos = atomicAdd(list_n, 1);
            list[pos] = order_word(f32_key(elem<T>::load(row + i)), i);
        }
    });
    __syncthreads();
    return ge;
}

// One pass: the log-sum-exp and, per thread, the maxima of its three best vectors and which the
// best two are.  tau = the K-th largest of the threads' maxima: K distinct logits are >= tau, so
// every winner is.  The logits >= tau (K plus a few) are listed: a thread whose best (two) vectors
// reach tau reads those vectors again, one whose third reaches it too reads all of its vectors.
// Each listed logit then counts the listed logits that precede it; that is its output position.
// A row whose list does not fit (thousands of ties at the top, K near the number of threads), or with fewer than K
// threads that hold a logit above -inf, takes list_best's instead.
//   Bound by HBM (one read of the row) with the arithmetic close behind: the exponential of every
// logit, and for the candidates eight plain instructions per VECTOR (three of them v_med3 / v_max
// on the maxima).  Keeping the two best LOGITS of a thread instead took seven per logit in 87 % of
// the vectors: 16384 rows of 128256 bf16 logits 801 -> 693 us (6.07 TB/s).  Rows that are not whole
// vectors and fp32 rows used to take the selection rounds: 1024 x 50257 bf16 1422 -> 26 us, 2048 x
// 128256 fp32 6320 -> 178 us (5.9 TB/s).  The last vectors of a row used to be one round trip
// after the other (with the rule of TOPK_ONCE_BYTES; us): 16384 rows of 128256 bf16 704 -> 665 (6.3 TB/s), 2264 114 -> 97, 3000 of 8000
// 18.7 -> 16.0; fp32 1500 of 128256 138 -> 124, 3000 of 8000 24.9 -> 21.8.
// ONCE: the rows are not kept in the caches (see TOPK_ONCE_BYTES).
template <typename T, int THREADS, int CAP, bool ONCE>
__global__ __launch_bounds__(THREADS, 8) void topk_row(const T* logits, int32_t* idx_out, float* logp_out, int N, int V, int K) {
    constexpr int NW = THREADS / CART_WAVE, VE = LogitVec<T>::N, PER_LANE = THREADS / CART_WAVE;
    constexpr int LOW_BIT = sizeof(T) == 2 ? 16 : 0;      // (the keys of bf16 values differ in their upper halves)
    __shared__ float red_max[NW], red_sum[NW];
    __shared__ int counts[3][4];
    __shared__ uint32_t all_kmax[THREADS];
    __shared__ __attribute__((aligned(16))) uint64_t list[CAP];
    __shared__ int list_n;
    __shared__ uint32_t tau_s;
    const int n = workgroup_id(), tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (n >= N) return;
    const LogitRow R = logit_row<T>(n, V);
    const T* row = logits + R.row;
    const u32x4* src = reinterpret_cast<const u32x4*>(row + R.head);
    idx_out += static_cast<size_t>(n) * K;
    logp_out += static_cast<size_t>(n) * K;
    if (tid == 0) list_n = 0;

    const float ninf = __uint_as_float(0xff800000u);
    float t1 = ninf, t2 = ninf, t3 = ninf;     // the largest vector maxima of the thread, descending
    int p1 = -1, p2 = -1;                      // vectors of t1 and t2; -1: the thread's single element
    float ref = -3.0e38f, sum = 0.f;           // sum of 2^(x log2e - ref); ref moves up to the largest maximum so far
    auto note = [&](float vm, int v) __attribute__((always_inline)) {
        const bool c1 = vm > t1, c2 = vm > t2;
        p2 = c1 ? p1 : (c2 ? v : p2);
        p1 = c1 ? v : p1;
        t3 = __builtin_amdgcn_fmed3f(t3, t2, vm);
        t2 = __builtin_amdgcn_fmed3f(t2, t1, vm);
        t1 = c1 ? vm : t1;
        const float need = fmaxf(vm, -3.0e38f) * CART_LOG2E;
        if (need > ref) {                      // (rare after the first few vectors)
            sum *= fast_exp2(ref - need);
            ref = need;
        }
    };
    auto take = [&](const u32x4& w, int v) __attribute__((always_inline)) {
        float vm = ninf;                       // (a NaN never becomes a maximum)
#pragma unroll
        for (int e = 0; e < VE; e += 2) vm = max3_raw(vm, LogitVec<T>::bits(w, e), LogitVec<T>::bits(w, e + 1));
        note(vm, v);
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int e = 0; e < VE; e += 2) {
            s0 += fast_exp2(fmaf(__uint_as_float(LogitVec<T>::bits(w, e)), CART_LOG2E, -ref));
            s1 += fast_exp2(fmaf(__uint_as_float(LogitVec<T>::bits(w, e + 1)), CART_LOG2E, -ref));
        }
        sum += s0 + s1;
    };
    if (tid < R.head + R.tail) {
        const float x = elem<T>::load(row + logit_single<T>(R, tid));
        note(max3_raw(ninf, __float_as_uint(x), __float_as_uint(x)), -1);
        sum += fast_exp2(fmaf(x, CART_LOG2E, -ref));
    }
    // Four vectors in flight.  A thread's last turn may hold fewer: loaded together all the same (past the row's end its last
    // vector, not taken).  Rows that are not kept take every turn through that form, whose loop is shorter (us, one form for the whole
    // turns / this for all: 4000 rows of 50257 bf16 75.8 / 73.5, 900 of 100001 42.2 / 40.1); others do not gain where a launch is few
    // rounds of rows (300 of 128256 bf16 23.9 / 25.5, 715 of 50257 17.4 / 18.0).
    int v0 = 0;
    if constexpr (!ONCE) {
        for (; v0 + 4 * THREADS <= R.nvec; v0 += 4 * THREADS) {
            u32x4 w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = src[v0 + tid + i * THREADS];
#pragma unroll
            for (int i = 0; i < 4; ++i) take(w[i], v0 + tid + i * THREADS);
        }
    }
    for (int v = v0 + tid; v < R.nvec; v += 4 * THREADS) {
        u32x4 w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32x4* const from = src + min(v + i * THREADS, R.nvec - 1);
            if constexpr (ONCE) w[i] = __builtin_nontemporal_load(from);
            else if (i == 0 || v0 + i * THREADS < R.nvec) w[i] = *from;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (v + i * THREADS < R.nvec) take(w[i], v + i * THREADS);
    }

    all_kmax[tid] = f32_key(t1);
    const float wref = wave_max(ref);
    sum = wave_sum(sum * fast_exp2(ref - wref));
    if (lane == 0) { red_max[wv] = wref; red_sum[wv] = sum; }
    __syncthreads();
    // tau, bit by bit from the top, by the first wavefront.  Of the 32 bits of an fp32 key the lower ones only tell a few candidates more or
    // less apart: any bound that K maxima reach will do.  With K up to a quarter of the threads so will one that somewhat more reach; with
    // more records every further maximum brings further logits of its thread, and the list, ranked at the square of its length, outgrows
    // what the bits cost (us, all bits / a bound that up to K + K/4 + 8 reach / this: 42 rows of 50257, K = 20 14.3 / 10.8 / 10.8, 500 31.8 / 32.0 / 30.0,
    // 800 75 / 127 / 73; 4096 of 8000, K = 128 44.6 / 51.5 / 41.5, 850 745 / 3877 / 725, its list past CAP; 500 of 32000, K = 256 31.6 / 39.7 / 30.8).
    // The 16 bits of a bf16 cost less than a longer list: 524 of 32000, K = 5 11.6, 14.1 so.
    // (rows of up to 128 logits and fewer vectors than records are listed whole: us, 16884 rows of 3 fp32, K = 1 34, now 19.6;
    // 20000 of 120, K = 100 66, now 48)
    const bool whole = V <= 128 && K > V / VE;
    if (wv == 0 && !whole) {
        uint32_t mine[PER_LANE];
#pragma unroll
        for (int j = 0; j < PER_LANE; ++j) mine[j] = all_kmax[64 * j + lane];
        uint32_t t = 0;
        const int enough = K + (K <= THREADS / 4 ? min(K / 4 + 8, 32) : 0);
        for (int bit = 31; bit >= LOW_BIT; --bit) {
            const uint32_t cand = t | (1u << bit);
            int c = 0;
#pragma unroll
            for (int j = 0; j < PER_LANE; ++j) c += __popcll(__ballot(mine[j] >= cand));
            if (c >= K) {
                t = cand;
                if (LOW_BIT == 0 && c <= enough) break;
            }
        }
        if (lane == 0) tau_s = t;
    }
    float gref = red_max[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) gref = fmaxf(gref, red_max[w]);
    sum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) sum += red_sum[w] * fast_exp2(red_max[w] - gref);
    const float lse = (gref + fast_log2(sum)) * CART_LN2;
    __syncthreads();
    const float tau = whole ? ninf : f32_key_value(tau_s);
    const bool listed = tau > ninf;
    if (listed && t1 >= tau) {
        auto put = [&](float x, uint32_t i) __attribute__((always_inline)) {
            if (x >= tau) {
                const int pos = atomicAdd(&list_n, 1);
                if (pos < CAP) list[pos] = order_word(f32_key(x), i);
            }
        };
        auto put_vec = [&](int pv) __attribute__((always_inline)) {
            const u32x4 w = src[pv];
#pragma unroll
            for (int e = 0; e < VE; ++e) put(__uint_as_float(LogitVec<T>::bits(w, e)), static_cast<uint32_t>(R.head + VE * pv + e));
        };
        if (t3 >= tau) {
            for (int u = tid; u < R.nvec; u += THREADS) put_vec(u);
            p1 = p2 = tid < R.head + R.tail ? -1 : -2;
        }
        if (p1 >= 0) put_vec(p1);
        if (t2 >= tau && p2 >= 0) put_vec(p2);
        if (p1 == -1 || (t2 >= tau && p2 == -1)) {
            const int i = logit_single<T>(R, tid);
            put(elem<T>::load(row + i), static_cast<uint32_t>(i));
        }
    }
    __syncthreads();
    int cnt = list_n;
    if (!listed || cnt < K || cnt > CAP) cnt = list_best<T, THREADS, CAP>(row, R, V, K, counts, list, &list_n);
    write_ranked<THREADS>(list, cnt, K, idx_out, logp_out, lse);
}

// Past a size the logits drive each other out of the memory-side cache on their way through, and what a later call or kernel
// could still find there: not kept then.  us a call, kept / not (two tensors in turn; behind 512 MB of other traffic), bf16
// 128256 a row: 98 MB 26.4 / 26.1, 29.8 / 29.9; 130 MB 35.4 / 35.4, 39.7 / 38.9; 200 MB 52.3 / 44.9, 54.4 / 48.8; 1 GB 184 / 174, 186 / 171.
// (Two calls' logits fit in the 256 MB that the memory side caches up to about the line.)  The price: what the candidates' threads read again
// comes from memory too.  With records for more than an eighth of the threads that takes the gain back or up to 10 % more, but not at every size (us, kept /
// not: 4096 x 20000 bf16, K = 20 37.1 / 34.7, 48 41.8 / 42.7, 64 45.6 / 47.3; 2048 x 20000 fp32, K = 20 36.6 / 32.0, 64 40.1 / 41.0, 128 51.0 / 54.3; 16384 x 32000
// bf16, K = 20 190 / 177, 64 214 / 212, 128 276 / 303; 2000 x 50257, K = 20 44.6 / 38.3, 64 52.2 / 50.9, 192 76.3 / 66.4).
constexpr size_t TOPK_ONCE_BYTES = static_cast<size_t>(144) << 20;

template <typename T>
static void launch_rows(const cart_topk_desc& d, const void* logits, int32_t* idx, float* logp, hipStream_t st) {
    const T* x = static_cast<const T*>(logits);
    // Threads by the length of the row: about 16 vectors per thread balance what a row costs besides
    // its loads (reductions, tau, list) against the workgroups a CU overlaps.  256 / 512 / 1024
    // threads, us for 4096 rows of V bf16 logits: V 128256 207 / 188 / 191 (16384 rows 724 / 703 /
    // 693, 1024 fp32 rows 140 / 107 / 97), 50257 84 / 81 / 106, 16000 35 / 45 / 71, 4096 15 / 24 / 56;
    // 256 rows of 128256: 45 / 25 / 18.  K records take K threads with a vector each, so
    // 512 or 1024 from half of the threads on.  Rows of fewer vectors than records are listed by list_best at any width: narrow
    // where there are rows for the chip, wide where one row's time counts.  256 / 512 / 1024 threads, bf16 rows of 1024 logits:
    // 4096 rows, K = 257 84 / 119 / 247, K = 1000 301 / 320 / 418; 256 rows, K = 600 46 / 39 / 36, K = 1000 75 / 51 / 45 (before rows
    // of little more than K logits were listed whole).
    const long nvec = d.V / LogitVec<T>::N;
    const int few = d.K > nvec ? (d.K <= 256 ? 256 : d.N <= device_cus() ? 1024 : d.K <= 512 ? 256 : 512) : 0;
    const bool once = static_cast<size_t>(d.N) * d.V * sizeof(T) > TOPK_ONCE_BYTES;
    auto launch = [&](auto kept, auto not_kept, int threads) {
        hipLaunchKernelGGL(once ? not_kept : kept, grid_of(d.N), dim3(threads), 0, st, x, idx, logp, d.N, d.V, d.K);
    };
    if (few == 256 || (few == 0 && nvec <= 4096 && d.K <= 128))       launch(topk_row<T, 256, 1024, false>, topk_row<T, 256, 1024, true>, 256);
    else if (few == 512 || (few == 0 && nvec <= 12288 && d.K <= 256)) launch(topk_row<T, 512, 2048, false>, topk_row<T, 512, 2048, true>, 512);
    else                                                              launch(topk_row<T, 1024, 4096, false>, topk_row<T, 1024, 4096, true>, 1024);
}

int launch_topk(const cart_topk_desc& d, const void* logits, int32_t* idx, float* logp, hipStream_t st) {
    trace_begin(st);   // kernel order: the row kernel
    if (d.logits_dtype == CART_BF16) launch_rows<bf16_t>(d, logits, idx, logp, st);
    else launch_rows<float>(d, logits, idx, logp, st);
    trace_mark(st);
    return static_cast<int>(hipGetLastError());
}

}  // namespace cart
