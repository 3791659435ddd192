// knnf_networks.h -- register networks over unsigned keys, shared by the filter
// kernels (device code only).  The tiles issue one vector instruction after
// another, so the count of instructions is what a network costs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace knnf {
namespace {

__device__ __forceinline__ uint32_t med3u(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ void cx(uint32_t& a, uint32_t& b) {
    const uint32_t lo = min(a, b);
    b = max(a, b);
    a = lo;
}

// Ascending order of four elements.
__device__ __forceinline__ void sort4(uint32_t& a, uint32_t& b, uint32_t& c, uint32_t& d) {
    const uint32_t lo = min(min(a, b), c), md = med3u(a, b, c), hi = max(max(a, b), c);
    a = min(lo, d);
    b = med3u(lo, md, d);
    c = med3u(md, hi, d);
    d = max(hi, d);
}
// Ascending order of two sorted pairs (a, b), (c, d).
__device__ __forceinline__ void merge22(uint32_t& a, uint32_t& b, uint32_t& c, uint32_t& d) {
    const uint32_t lo = min(a, c), t = max(a, c), hi = max(b, d);
    const uint32_t m1 = min(min(t, b), d), m2 = med3u(t, b, d);
    a = lo;
    b = m1;
    c = m2;
    d = hi;
}
// Ascending order of a cyclic bitonic sequence of four.
__device__ __forceinline__ void bitonic4(uint32_t& a, uint32_t& b, uint32_t& c, uint32_t& d) {
    const uint32_t lo = min(b, d), hi = max(b, d);
    const uint32_t y0 = min(min(a, c), lo), y1 = med3u(a, c, lo);
    const uint32_t y2 = med3u(a, c, hi), y3 = max(max(a, c), hi);
    a = y0;
    b = y1;
    c = y2;
    d = y3;
}

// Ascending order of x[0], x[S], x[2 S], ... (N elements, both halves sorted).
template <int N, int S>
__device__ __forceinline__ void merge_halves(uint32_t* x) {
    if constexpr (N == 4) {
        merge22(x[0], x[S], x[2 * S], x[3 * S]);
    } else {
        merge_halves<N / 2, 2 * S>(x);  // Batcher: even and odd elements, then neighbours
        merge_halves<N / 2, 2 * S>(x + S);
#pragma unroll
        for (int i = 1; i + 1 < N; i += 2) cx(x[i * S], x[(i + 1) * S]);
    }
}
// Ascending sort of the lane's E elements.
template <int E>
__device__ __forceinline__ void lane_sort(uint32_t* x) {
    if constexpr (E == 4) {
        sort4(x[0], x[1], x[2], x[3]);
    } else {
        lane_sort<E / 2>(x);
        lane_sort<E / 2>(x + E / 2);
        merge_halves<E, 1>(x);
    }
}
// Ascending order of the lane's bitonic sequence.
template <int E>
__device__ __forceinline__ void lane_merge(uint32_t* x) {
    if constexpr (E == 4) {
        bitonic4(x[0], x[1], x[2], x[3]);
    } else {
#pragma unroll
        for (int r = 0; r < E / 2; ++r) cx(x[r], x[r + E / 2]);
        lane_merge<E / 2>(x);
        lane_merge<E / 2>(x + E / 2);
    }
}
// Keep the smaller (keep = 0) or larger (all ones) of each element and its
// partner in the lane that CTRL selects, the registers mirrored or not.
template <int CTRL, bool MIRROR, int E>
__device__ __forceinline__ void cross(uint32_t (&x)[E], uint32_t keep) {
    uint32_t t[E];
#pragma unroll
    for (int r = 0; r < E; ++r)
        t[r] = (uint32_t)__builtin_amdgcn_mov_dpp((int)x[MIRROR ? E - 1 - r : r], CTRL, 0xF, 0xF, false);
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] = med3u(x[r], t[r], keep);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_XOR3 = 0x1B, DPP_XOR7 = 0x141, DPP_XOR15 = 0x140;
// cross with lane L ^ 4, by way of L ^ 7.
template <int E>
__device__ __forceinline__ void cross_xor4(uint32_t (&x)[E], uint32_t keep) {
    uint32_t t[E];
#pragma unroll
    for (int r = 0; r < E; ++r)
        t[r] = (uint32_t)__builtin_amdgcn_mov_dpp(
            __builtin_amdgcn_mov_dpp((int)x[r], DPP_XOR7, 0xF, 0xF, false), DPP_XOR3, 0xF, 0xF, false);
#pragma unroll
    for (int r = 0; r < E; ++r) x[r] = med3u(x[r], t[r], keep);
}

}  // namespace
}  // namespace knnf
