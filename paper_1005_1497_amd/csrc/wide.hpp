// Convolutions of 32-bit words of length 2^13 and 2^14 on the matrix cores, each
// start to finish in one workgroup: operands are read and results written once,
// and everything in between stays in registers and LDS.
//
// N = 4096 R, element t = t' + 4096 k, frequency u = j + R u'.  Transform j < R of
// 4096 points, of inputs sum_k w_R^(j k) x(t' + 4096 k) twisted by w^(j t'), is that
// of wave.hpp on four waves.  The twist is a product over the digits of t', so the
// tables of transform j take it in (first step: the digit p2, second: p1, twiddles:
// t0), and the sum over k is part of the first step's contraction: its sums run on
// over R matrices and R inputs, which costs matrix instructions but no vector ones
// and no exchange.  The inverse is the mirror image: its last step contracts over
// (j, p0) for each k.
//
// 2^13: four waves and 48 KB of LDS, three workgroups per CU (168 registers); the
// transforms j = 0, 1 one after the other, what the second needs waiting in one LDS
// buffer and 16 registers.  Bound by vector issue, as k_conv_mid (81 vector and 9
// matrix instructions per element, three waves per SIMD).  2^26 elements,
// m = 13631489, against the fp64 kernels with a scratch in memory (36 bytes per
// element): 447 -> 267 us; 2^24: 137 -> 64.
// 2^14: eight waves of 240 registers and all 160 KB of a CU's LDS, two groups of
// waves with two transforms each; the next item's words are loaded during the last
// step.  Bound by its two waves per SIMD going through the matrix-heavy first and
// last steps together.  2^26 elements 463 -> 359 us, 2^24: 152 -> 90.
// A step of its own over k, exchanged through LDS, took 102 vector instructions per
// element and 370 us at 2^13, 385 at 2^14; with 128 registers (16 waves per CU) it
// spilled and took 532 and 641.  2^15 and 2^16 that way: 488 and 990 us, no gain over
// the four-step kernels (453, 513).
#pragma once
#include "wave.hpp"

namespace nttmi {

struct WideTab {   // 16-byte units: shared part, then one part per j
    static constexpr int W = 0, TK = 192, TB = TK + 128, J = TB + 16 * 128;
    // per j: inverse's first and second steps, matrices, twiddles, and for each k the first step and the last
    static constexpr int V1 = 0, U = 192, M = 384, TF = M + 16 * 192, F = TF + 16 * 128;
    __device__ static constexpr int L(int R) { return F + R * 192; }
    __device__ static constexpr int size(int R) { return F + 2 * R * 192; }
};

template <int n>
struct WideG {
    static constexpr int N = 1 << n, R = N / 4096;
    static constexpr int WAVES = 2 * R, GROUPS = R / 2;   // a group of four waves per transform: two rounds
    static constexpr int PW = 16 / WAVES;                 // values of p1 per wave in the first and last steps
};

// Word of an exchange buffer for element (g, i), column c, register p (16-byte
// pieces of a row permuted by two bits of the column, as mid_put has them).
__device__ __forceinline__ int wide_at(int row, int c, int p) { return ((row * 16 + c) * 4 + ((p >> 2) ^ (c >> 2))) * 4 + (p & 3); }
template <int PW>
__device__ __forceinline__ void wide_put(v4i* b, const v4i (&v)[PW], int wave, int gr, int c) {
    if constexpr (PW == 4)
        mid_put(b, v, wave, gr, c);
    else {
        typedef int v2i __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int i = 0; i < 4; ++i) *(v2i*)((int*)b + wide_at(4 * gr + i, c, 2 * wave)) = v2i{v[0][i], v[1][i]};
    }
}
// registers p = PW wave + k, elements (g, i)
template <int PW>
__device__ __forceinline__ void wide_get(const v4i* b, v4i (&v)[PW], int wave, int gr, int c) {
#pragma unroll
    for (int k = 0; k < PW; ++k) v[k] = b[((PW * wave + k) * 16 + c) * 4 + (gr ^ (c >> 2))];
}

// matrices and twiddles of the second step
struct WideM {
    Mat M[4];
    Tw tw[4];
};
__device__ __forceinline__ void ld_m(WideM& m, const v4i* tj, int w4, int lane) {
    using T = WideTab;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        m.M[k] = ld_mat(tj + T::M + (4 * w4 + k) * 192, lane);
        m.tw[k] = ld_tw(tj + T::TF + (4 * w4 + k) * 128, lane);
    }
}
// Transform j between the exchanges: x, y (registers 4 w4 + k: u0) -> x (registers p0).
template <bool SMALL, class Point>
__device__ __forceinline__ void wide_core(v4i (&x)[4], v4i (&y)[4], const WideM& m, const v4i* ts, const v4i* tj, int w4,
                                         int lane, const I8K& C, const Point& point) {
    using T = WideTab;
    const Init ti = init_tight(C);
    const Mat W = ld_mat(ts + T::W, lane), V = ld_mat(tj + T::V1, lane);
    const Tw tk = ld_tw(ts + T::TK, lane);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        x[k] = fold4_tw(digit_sums<TURN>(m.M[k], x[k], ti), m.tw[k], C);
        y[k] = fold4_tw(digit_sums<TURN>(m.M[k], y[k], ti), m.tw[k], C);
    }
    const Mat U = ld_mat(tj + T::U, lane);
    Tw tb[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) tb[k] = ld_tw(ts + T::TB + (4 * w4 + k) * 128, lane);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        x[k] = fold4_tight(digit_sums<KEEP>(W, x[k], ti), C);
        y[k] = fold4_tight(digit_sums<KEEP>(W, y[k], ti), C);
        if constexpr (!Point::DIV) x[k] = mul4_fg<SMALL>(x[k], y[k], C);
    }
    if constexpr (Point::DIV) point(x, y, C);
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = fold4_tw(digit_sums<TURN>(V, x[k], ti), tk, C);
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = fold4_tw(digit_sums<KEEP>(U, x[k], ti), tb[k], C);
}

// MODE 0: no extra reductions, 1: of the results (m < R 2.2e6), 2: also before the products (small moduli)
// CRT: the combining store instead of h's (items back to back).
template <int n, int MODE, class Point, bool CRT = false>
__device__ __forceinline__ void wide_block(const uint32_t* f, const uint32_t* g, uint32_t* h, const uint64_t* offs,
                                           uint32_t count, I8Plan p, const Point& point, const Combine& crt = Combine{}) {
    using G = WideG<n>;
    using T = WideTab;
    constexpr int R = G::R, PW = G::PW;
    constexpr bool SMALL = MODE == 2;
    __shared__ v4i xch[n == 13 ? 3 : 10][1024];
    int lane = threadIdx.x & 63, gr = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), group = wave >> 2, w4 = wave & 3;
    const I8K C(p.C);
    const v4i* ts = (const v4i*)p.tab;
    auto tab = [&](int j) { return ts + T::J + j * T::size(R); };
    const uint32_t lw = (uint32_t)(c + 1024 * gr);
    auto at_word = [&](int q, int k, int i) -> uint32_t { return k * 4096 + i * 256 + (wave * PW + q) * 16; };
    // (past the last item: empty, at an address whose words are there all the same, since
    // the scalar offsets are outside the check)
    auto buf = [&](const uint32_t* a, uint32_t item) {
        const uint64_t off = item >= count ? 0 : offs ? offs[item] : (uint64_t)item * G::N;
        return wave_buf(a + off, item < count ? G::N * 4 : 0);
    };
    auto load = [&](const uint32_t* a, uint32_t item, v4i (&v)[PW][R]) {
        const auto b = buf(a, item);
#pragma unroll
        for (int q = 0; q < PW; ++q)
#pragma unroll
            for (int k = 0; k < R; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    v[q][k][i] = (int)__builtin_amdgcn_raw_buffer_load_b32(b, lw * 4, at_word(q, k, i) * 4, 0);
    };
    auto digits = [&](v4i (&v)[PW][R]) {
#pragma unroll
        for (int q = 0; q < PW; ++q)
#pragma unroll
            for (int k = 0; k < R; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[q][k][i] ^= (int)DIG;
    };
    // sum over k of the matrices' products
    auto sums = [&](const Mat (&A)[R], const v4i (&v)[R], const Init& in) {
        Sums s = digit_sums<KEEP>(A[0], v[0], in);
#pragma unroll
        for (int k = 1; k < R; ++k) s = digit_sums<KEEP>(A[k], v[k], Init{s.s0, s.s1, s.s2});
        return s;
    };
    auto first = [&](int j, const Mat (&A)[R], const v4i (&v)[PW][R], v4i (&out)[PW]) {
        const Init lo = init_loose(C);
        const Init in = j == 0 ? init_raw(lo, C, [&](int i) { return gr == 0 && i == 0; }) : lo;
#pragma unroll
        for (int q = 0; q < PW; ++q) out[q] = fold4_loose(sums(A, v[q], in), C);
    };
    auto mats = [&](Mat (&A)[R], int at, int step) {
#pragma unroll
        for (int k = 0; k < R; ++k) A[k] = ld_mat(ts + T::J + at + k * step, lane);
    };
    // the last step's outputs k, from (j, q)
    auto last = [&](const v4i (&a)[PW][R], uint32_t item, Mat (&A)[R]) {
        const Init ti = init_tight(C);
        const uint64_t at = (uint64_t)item * G::N;
        const auto bh = CRT ? wave_buf(crt.h + at, G::N * 8) : buf(h, item);
        uint32_t a1[CRT ? R : 1][PW][4];
        if constexpr (CRT) {
            const auto ba = wave_buf(crt.a1 + at, G::N * 4);
#pragma unroll
            for (int k = 0; k < R; ++k)
#pragma unroll
                for (int q = 0; q < PW; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        a1[k][q][i] = __builtin_amdgcn_raw_buffer_load_b32(ba, lw * 4, at_word(q, k, i) * 4, 0);
        }
#pragma unroll
        for (int k = 0; k < R; ++k) {
            Mat B[R];
            if (k + 1 < R) {
                B[0] = A[0];   // (j = 0: no factors w_R^(j k))
#pragma unroll
                for (int j = 1; j < R; ++j) B[j] = ld_mat(tab(j) + T::L(R) + (k + 1) * 192, lane);
            }
#pragma unroll
            for (int q = 0; q < PW; ++q) {
                const v4i r = fold4_tight(sums(A, a[q], ti), C);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (CRT)
                        __builtin_amdgcn_raw_buffer_store_b64(combined<MODE != 0>(r[i], a1[k][q][i], crt, C), bh, lw * 8,
                                                              at_word(q, k, i) * 8, 0);
                    else st_out<true>(bh, out_word<MODE != 0>(r[i], C), lw, at_word(q, k, i));
                }
            }
            if (k + 1 < R)
#pragma unroll
                for (int j = 0; j < R; ++j) A[j] = B[j];
        }
    };
    v4i fr[PW][R], gw[PW][R];
    if constexpr (n == 13) {
        const uint32_t item = blockIdx.x;
        load(f, item, fr);
        load(g, item, gw);
        Mat A[2], B[2];
        A[0] = A[1] = ld_mat(tab(0) + T::F, lane);
        mats(B, T::size(R) + T::F, 192);
        v4i x[4], y[4], t[4];
        digits(fr);
        first(0, A, fr, x);
        mid_put(xch[0], x, wave, gr, c);
        first(1, B, fr, x);
        mid_put(xch[1], x, wave, gr, c);
        digits(gw);
        first(0, A, gw, x);
        mid_put(xch[2], x, wave, gr, c);
        first(1, B, gw, t);
        WideM m;
        ld_m(m, tab(0), w4, lane);
        __syncthreads();
        mid_get(xch[0], x, wave, gr, c);
        mid_get(xch[2], y, wave, gr, c);
        wide_core<SMALL>(x, y, m, ts, tab(0), w4, lane, C, point);
        v4i z[4];
        mid_get(xch[1], z, wave, gr, c);
        __syncthreads();
        mid_put(xch[0], t, wave, gr, c);
        mid_put(xch[2], x, wave, gr, c);
        ld_m(m, tab(1), w4, lane);
        __syncthreads();
        mid_get(xch[0], y, wave, gr, c);
        wide_core<SMALL>(z, y, m, ts, tab(1), w4, lane, C, point);
        mid_put(xch[1], z, wave, gr, c);
        __syncthreads();
        mid_get(xch[2], x, wave, gr, c);
        mid_get(xch[1], y, wave, gr, c);
        v4i a[4][2];
#pragma unroll
        for (int q = 0; q < 4; ++q) a[q][0] = x[q], a[q][1] = y[q];
        Mat L[R];
        mats(L, T::L(R), T::size(R));
        last(a, item, L);
    } else {
        uint32_t item = blockIdx.x;
        load(f, item, fr);
        load(g, item, gw);
        for (; item < count; item += gridDim.x) {
            // (or the loop's invariant addresses take the registers)
            asm volatile("" : "+s"(ts));
            asm volatile("" : "+v"(lane));
            gr = lane >> 4, c = lane & 15;
            digits(fr);
            digits(gw);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                // (w_R^(j k) repeats with k: R / gcd(j, R) matrices)
                Mat A[R];
                const int per = j == 0 ? 1 : j == 2 ? 2 : 4;
#pragma unroll
                for (int k = 0; k < R; ++k) A[k] = k < per ? ld_mat(tab(j) + T::F + k * 192, lane) : A[k % per];
                v4i x[PW];
                first(j, A, fr, x);
                wide_put<PW>(xch[j], x, wave, gr, c);
                first(j, A, gw, x);
                wide_put<PW>(xch[4 + j], x, wave, gr, c);
            }
            WideM m;
            ld_m(m, tab(group), w4, lane);
            __syncthreads();
            v4i x[4], y[4];
            wide_get<4>(xch[group], x, w4, gr, c);
            wide_get<4>(xch[4 + group], y, w4, gr, c);
            wide_core<SMALL>(x, y, m, ts, tab(group), w4, lane, C, point);
            wide_put<4>(xch[8 + group], x, w4, gr, c);
            ld_m(m, tab(2 + group), w4, lane);
            wide_get<4>(xch[2 + group], x, w4, gr, c);
            wide_get<4>(xch[6 + group], y, w4, gr, c);
            __syncthreads();   // xch[group] is read
            wide_core<SMALL>(x, y, m, ts, tab(2 + group), w4, lane, C, point);
            wide_put<4>(xch[group], x, w4, gr, c);
            Mat L[R];
            mats(L, T::L(R), T::size(R));
            load(f, item + gridDim.x, fr);
            load(g, item + gridDim.x, gw);
            __syncthreads();
            v4i a[PW][R];
#pragma unroll
            for (int j = 0; j < R; ++j) {
                v4i t[PW];
                wide_get<PW>(xch[j < 2 ? 8 + j : j - 2], t, wave, gr, c);
#pragma unroll
                for (int q = 0; q < PW; ++q) a[q][j] = t[q];
            }
            __syncthreads();   // xch[0], xch[1] are read
            last(a, item, L);
        }
    }
}

template <int n, int MODE>
__global__ __launch_bounds__(64 * WideG<n>::WAVES) __attribute__((amdgpu_waves_per_eu(n == 13 ? 3 : 2, n == 13 ? 3 : 2))) void
k_conv_wide(const uint32_t* f, const uint32_t* g, uint32_t* h, const uint64_t* __restrict__ offs, uint32_t count, I8Plan p) {
    wide_block<n, MODE>(f, g, h, offs, count, p, PointMul{});
}
template <int n, int MODE>
__global__ __launch_bounds__(64 * WideG<n>::WAVES) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_div_wide(
    const uint32_t* f, const uint32_t* g, uint32_t* h, const uint64_t* __restrict__ offs, uint32_t count, I8Plan p,
    Quotient q) {
    wide_block<n, MODE>(f, g, h, offs, count, p, PointDiv(q));
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_crt_wide(
    const uint32_t* f, const uint32_t* g, uint32_t count, I8Plan p, Combine crt) {
    wide_block<13, 0, PointMul, true>(f, g, nullptr, nullptr, count, p, PointMul{}, crt);
}

}  // namespace nttmi
