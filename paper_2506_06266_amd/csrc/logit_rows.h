// Rows of a [N][V] tensor of logits as 16-byte vectors, for the loss and the top-k kernels.
#pragma once

#include "cart_common.h"

namespace cart {

// max of a float and two raw fp32 bit patterns in one instruction, without the NaN-quieting
// moves the compiler would add around fmaxf for values it cannot prove canonical
__device__ __forceinline__ float max3_raw(float a, uint32_t b, uint32_t c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// One 16-byte vector of logits: its elements widened to fp32.
template <typename T> struct LogitVec;
template <> struct LogitVec<bf16_t> {
    static constexpr int N = 8;
    static constexpr uint32_t FILL = 0xff7fff7fu;      // two bf16 of the most negative finite value
    static __device__ __forceinline__ uint32_t bits(const u32x4& w, int e) {
        return (e & 1) ? (w[e >> 1] & 0xffff0000u) : (w[e >> 1] << 16);
    }
};
template <> struct LogitVec<float> {
    static constexpr int N = 4;
    static constexpr uint32_t FILL = 0xff7fffffu;
    static __device__ __forceinline__ uint32_t bits(const u32x4& w, int e) { return w[e]; }
};
// Row n of [N][V]: `head` single elements, nvec whole vectors, `tail` single elements.  The base of
// the tensor is 16-byte aligned.  Single element s (of head + tail <= 14) belongs to thread s of the
// workgroup, vector v to thread v % THREADS.
struct LogitRow {
    size_t row;
    int head, nvec, tail;
};
template <typename T> __device__ __forceinline__ LogitRow logit_row(int n, int V) {
    constexpr int VE = LogitVec<T>::N;
    LogitRow r;
    r.row = static_cast<size_t>(n) * V;
    r.head = min(static_cast<int>((VE - (r.row & (VE - 1))) & (VE - 1)), V);
    r.nvec = (V - r.head) / VE;
    r.tail = V - r.head - r.nvec * VE;
    return r;
}
// element index of single s
template <typename T> __device__ __forceinline__ int logit_single(const LogitRow& r, int s) {
    return s < r.head ? s : s + r.nvec * LogitVec<T>::N;
}
}  // namespace cart
