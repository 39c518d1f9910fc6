// Convolutions of 32-bit words of length 2^13 .. 2^19 on the matrix cores, in three
// launches: N = 256 Q, element t = t1 + Q t2, frequency u = u2 + 256 u1.
//   columns: length-256 transforms over t2 of f and g, times w^(t1 u2), into
//     scratch rows of digits Y[u2 Q + t1];
//   rows: the convolution of each pair of rows (the kernels of wave.hpp for
//     length Q), times w^-(s1 u2), over the row of f;
//   inverse columns: length-256 inverse transforms over u2, canonical store.
// The frequency order stays inside, so nothing is transposed in memory.  Memory moves
// 16, 12 and 8 bytes per element; the columns and the inverse columns are bound by
// that (62 and 24 us per 2^24 elements, 4.3 and 5.6 TB/s), the rows by vector issue (46
// us, 60 above 2^16).  m = 13631489, against the fp64 four-step kernels: one item of 2^16
// 13.2 -> 12.0 us, of 2^19 21.2 -> 15.6; 2^22 elements of 2^16 48 -> 38, of 2^19 61 -> 41; 2^24
// of 2^18 172 -> 138; 2^26 of 2^18 637 -> 540, of 2^19 703 -> 539.  Slower: the phases of
// successive groups side by side in one launch (2^24 elements of 2^16 162 us against 130),
// and workgroups of one die that keep an item's scratch in its L2 and wait for each
// other between the phases (2^26 elements of 2^16 660 against 513).
#pragma once
#include "trans.hpp"

namespace nttmi {

// Items at offs[i], or back to back (offs null); scratch 2N words per item, rows of f
// and then of g.
template <int n, int V>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5 - V, 5 - V))) void k_four_cols(
    const uint32_t* f, const uint32_t* g, const uint64_t* __restrict__ offs, uint32_t* Y, I8Plan p) {
    constexpr uint32_t N = 1u << n, CB = N / 4096 / V;
    __shared__ v4i xch[V][1024];
    const uint32_t id = col_id<V>(), half = id / CB;
    const uint64_t off = offs ? offs[half / 2] : (uint64_t)(half / 2) * N;
    cols_block<n, FORWARD, false, V>((half & 1 ? g : f) + off, Y + (uint64_t)half * N, id % CB, p,
                                     xch);
}
template <int n, bool SMALL, int V>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5 - V, 5 - V))) void k_four_inv(
    const uint32_t* Y, uint32_t* h, const uint64_t* __restrict__ offs, I8Plan p) {
    constexpr uint32_t N = 1u << n, CB = N / 4096 / V;
    __shared__ v4i xch[V][1024];
    const uint32_t id = col_id<V>(), item = id / CB;
    const uint64_t off = offs ? offs[item] : (uint64_t)item * N;
    cols_block<n, INVERSE, SMALL, V>(Y + (uint64_t)item * 2 * N, h + off, id % CB, p, xch);
}
template <int n, int V>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5 - V, 5 - V))) void k_four_crt(const uint32_t* Y,
                                                                                                    Combine crt, I8Plan p) {
    constexpr uint32_t N = 1u << n, CB = N / 4096 / V;
    __shared__ v4i xch[V][1024];
    const uint32_t id = col_id<V>(), item = id / CB;
    crt.h += (uint64_t)item * N;
    cols_block<n, INVERSE, false, V, true>(Y + (uint64_t)item * 2 * N, (uint32_t*)crt.a1 + (uint64_t)item * N, id % CB, p,
                                           xch, crt);
}
template <int n, bool SMALL, class Point>
__device__ __forceinline__ void four_rows(uint32_t* Y, int rounds, const I8Plan& p, const Point& point) {
    constexpr int la = n - 8;
    constexpr uint32_t N = 1u << n, CH = N / 4096;
    if constexpr (la <= 8) {
        const uint32_t per = CH / rounds, item = blockIdx.x / per, bx = blockIdx.x % per;
        uint32_t* y = Y + (uint64_t)item * 2 * N;
        tiny_block<la, SMALL, true>(y, y + N, y, N, rounds, p, bx, (const v4i*)p.tti, point);
    } else {
        __shared__ v4i xch[3][1024];
        const uint32_t item = blockIdx.x / CH, bx = blockIdx.x % CH;
        uint32_t* y = Y + (uint64_t)item * 2 * N;
        mid_block<la, SMALL, true>(y, y + N, y, N, p, bx, (const v4i*)p.tti, xch, point);
    }
}
template <int n, bool SMALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_four_rows(uint32_t* Y, int rounds,
                                                                                             I8Plan p) {
    four_rows<n, SMALL>(Y, rounds, p, PointMul{});
}
template <int n, bool SMALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_four_div(uint32_t* Y, int rounds,
                                                                                            I8Plan p, Quotient q) {
    four_rows<n, SMALL>(Y, rounds, p, PointDiv(q));
}

}  // namespace nttmi
