// Convolutions of 32-bit words of length 2^5 .. 2^12 on the matrix cores.
//
// A sequence is read as digits of its index, and a step contracts one digit
// (i8dft.hpp).  In a wave's registers one digit (4 bits) lies in the lane group
// and register element (g, i), one in the lane's column c, and the others name
// registers and waves.  Sequences shorter than the digits allow fill up with the
// sequence number s: the matrix is then block diagonal.
#pragma once
#include "arith.hpp"
#include "i8dft.hpp"

namespace nttmi {

// A wave's buffer over `bytes` valid bytes: loads beyond read 0 and stores beyond are
// dropped, by a check that covers the lane's offset and the instruction's constant but not
// a scalar offset.  Where a chunk may be a part of one, all of the offset is therefore in
// those two: the accessors below take the lane's word and a constant one (up to 1023 words
// it is in the instruction itself).  WHOLE: everything accessed is in the buffer, and the
// second word may be a scalar (2^24 elements of 2^15, rows in three launches: four
// registers spilled otherwise, 600 integer convolutions 345 -> 353 us).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t wave_buf(const void* p, uint32_t bytes) {
    // (uniform by construction; said so, or the descriptor would be taken lane by lane)
    const uint64_t a = (uint64_t)(uintptr_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)(((uint64_t)hi << 32) | lo), (short)0,
                                             __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
}
template <bool WHOLE = false>
__device__ __forceinline__ uint32_t ld_word(__amdgpu_buffer_rsrc_t b, uint32_t lane_word, uint32_t word) {
    if constexpr (WHOLE) return __builtin_amdgcn_raw_buffer_load_b32(b, lane_word * 4, word * 4, 0);
    else return __builtin_amdgcn_raw_buffer_load_b32(b, (lane_word + word) * 4, 0, 0);
}
template <bool WHOLE = false>
__device__ __forceinline__ int ld_raw(__amdgpu_buffer_rsrc_t b, uint32_t lane_word, uint32_t word) {
    return (int)(ld_word<WHOLE>(b, lane_word, word) ^ DIG);
}
template <bool WHOLE = false>
__device__ __forceinline__ void st_out(__amdgpu_buffer_rsrc_t b, uint32_t x, uint32_t lane_word, uint32_t word) {
    if constexpr (WHOLE) __builtin_amdgcn_raw_buffer_store_b32(x, b, lane_word * 4, word * 4, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(x, b, (lane_word + word) * 4, 0, 0);
}
__device__ __forceinline__ void st_out2(__amdgpu_buffer_rsrc_t b, v2u x, uint32_t lane_word, uint32_t word) {
    __builtin_amdgcn_raw_buffer_store_b64(x, b, (lane_word + word) * 8, 0, 0);
}
// Sixteen bytes at once.  With a scalar register as offset the compiler would leave no
// wait before the next write to the stored registers, and the last lanes of the store
// read what that write put there; all of the offset is in the lanes.
typedef unsigned v4u __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void st_out4(__amdgpu_buffer_rsrc_t b, v4u x, uint32_t word) {
    __builtin_amdgcn_raw_buffer_store_b128(x, b, word * 4, 0, 0);
}

// The pointwise steps over four registers of spectra (tight residues).
// x <- x y, as digits:
struct PointMul {   // (register by register, where the kernels form them)
    static constexpr bool DIV = false;
};
// x <- y / x, as digits: the lane's sixteen divisors are inverted together
// (Montgomery's simultaneous inversion): one Fermat power of their product, then each
// inverse from the prefix products.  A zero divisor sets the flag and enters as 1.
// In fp64: a product modulo m is four instructions there, and leaves no residue too
// large for the next one.  (2^23 elements of 2^13: 92 -> 55 us.)
struct PointDiv {
    static constexpr bool DIV = true;
    ModC M;
    uint32_t* singular;
    __device__ __forceinline__ explicit PointDiv(const Quotient& q) : M(q.M), singular(q.singular) {}
    // valid: the registers (bits) that hold a sequence of the batch
    __device__ __forceinline__ void operator()(v4i (&x)[4], const v4i (&y)[4], const I8K& C, uint32_t valid = 15) const {
        double c[16];
        bool zero = false;
        auto divisor = [&](int i) {
            const double r = reduce((double)x[i >> 2][i & 3], M);
            zero |= r == 0.0 && ((valid >> (i >> 2)) & 1);
            return r == 0.0 ? 1.0 : r;
        };
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const double r = divisor(i);
            c[i] = i == 0 ? r : mulmod_var(c[i - 1], r, M);
        }
        if (zero) atomicOr(singular, 1u);
        const uint32_t e = C.m - 2;
        double inv = pow_mod<W32>(c[15], e, 31 - __builtin_clz(e), M);
#pragma unroll
        for (int i = 15; i >= 0; --i) {
            const double ri = i == 0 ? inv : mulmod_var(inv, c[i - 1], M);
            if (i > 0) inv = mulmod_var(inv, divisor(i), M);   // (formed again rather than kept)
            const double q = mulmod_var(ri, (double)y[i >> 2][i & 3], M);
            x[i >> 2][i & 3] = (int)(((uint32_t)(int32_t)q + DIG) ^ DIG);
        }
    }
};

// The combining store's word for the tight residue r of the launch's modulus.
template <bool SMALL>
__device__ __forceinline__ v2u combined(int r, uint32_t a1, const Combine& crt, const I8K& C) {
    const int b = reduce_i((int)out_word<SMALL>(r, C) - (int)a1, C);   // (both below 2^24)
    const float q = __builtin_fmaf((float)b, crt.cq, MAGIC);
    const uint32_t t = canon_i((int32_t)mad24u(fbits(q), C.m, mad24s(b, crt.c, (uint32_t)C.it)), C);
    const uint64_t h = a1 + (uint64_t)crt.m1 * t;
    return v2u{(uint32_t)h, (uint32_t)(h >> 32)};
}

// ROWS (of tiny_block and mid_block): the row phase of a longer transform
// (four.hpp).  f and g are an item's rows of digits in scratch; the rows'
// convolutions, times the twiddles rtt (four words per lane, in the order of the
// registers), go to h as digits.  CRT: the combining store instead of h's.

// ------------------------------------------------------------------ N <= 2^8
// N = 16 B, B <= 16; a block of 256 consecutive elements (16 / B sequences) is
// four registers of a wave, and a convolution never leaves the registers:
// forward, t = t0 + 16 t', u = U + B u2: over (s, t') [c: t0 -> (s, U)], times
// w^(t0 U), over t0; inverse, position p = p0 + B p', result v0 + 16 v1: over p'
// [c: (s, p0) -> v0], times w^-(p0 v0), over (s, p0) with N^-1.
constexpr int TINY_BLOCKS = 4;   // blocks per wave and pass (1024 elements)
constexpr int TINY_ROUNDS = 4;   // passes per wave, at most
template <int n, bool SMALL, bool ROWS, class Point, bool CRT = false>
__device__ __forceinline__ void tiny_block(const uint32_t* f, const uint32_t* g, uint32_t* h, uint64_t words,
                                           int rounds, const I8Plan& p, uint32_t bx, const v4i* rtt, const Point& point,
                                           const Combine& crt = Combine{}) {
    constexpr int B = (1 << n) / 16;
    const int lane = threadIdx.x & 63, gr = lane >> 4, c = lane & 15;
    const I8K C(p.C);
    const v4i* t = (const v4i*)p.tab;
    const Mat A1 = ld_mat(t, lane), A2 = ld_mat(t + 192, lane), A3 = ld_mat(t + 384, lane), A4 = ld_mat(t + 576, lane);
    const Tw T1 = ld_tw(t + 768, lane), T2 = ld_tw(t + 768 + 128, lane);
    const Init ti = init_tight(C), raw = ROWS ? ti : init_raw(ti, C, [&](int) { return (c & (B - 1)) == 0; });
    const uint32_t lw = (uint32_t)(c + 64 * gr);
    constexpr uint32_t CH = 256 * TINY_BLOCKS;
    int nx[TINY_BLOCKS][4], ny[TINY_BLOCKS][4];   // the next blocks' words, loaded ahead
    auto load = [&](const uint32_t* src, uint64_t at, int (&v)[TINY_BLOCKS][4]) {
        const uint64_t a = at < words ? at : 0;
        const auto bu = wave_buf(src + a, at < words ? (uint32_t)(words - a < CH ? words - a : CH) * 4 : 0u);
        uint32_t ll = lw;
        if constexpr (!ROWS) asm volatile("" : "+v"(ll));   // (as below)
#pragma unroll
        for (int b = 0; b < TINY_BLOCKS; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                v[b][i] = (int)ld_word<ROWS>(bu, ll, 256 * b + 16 * i);
    };
    // a workgroup's passes lie together
    const uint64_t first = (uint64_t)bx * (4 * CH) * rounds +
                           (uint64_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * CH;
    constexpr uint64_t step = 4 * CH;
    load(f, first, nx);
    load(g, first, ny);
    for (int r = 0; r < rounds; ++r) {
        const uint64_t at = first + r * step;
        if (at >= words) break;
        const uint32_t bytes = (uint32_t)(words - at < CH ? words - at : CH) * 4;
        const auto bh = CRT ? wave_buf(crt.h + at, 2 * bytes) : wave_buf(h + at, bytes);
        v4i x[TINY_BLOCKS], y[TINY_BLOCKS];
#pragma unroll
        for (int b = 0; b < TINY_BLOCKS; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[b][i] = nx[b][i] ^ (ROWS ? 0 : (int)DIG);
                y[b][i] = ny[b][i] ^ (ROWS ? 0 : (int)DIG);
            }
        v4i tt[TINY_BLOCKS];
        if constexpr (ROWS) {
#pragma unroll
            for (int b = 0; b < TINY_BLOCKS; ++b) tt[b] = rtt[(at / 256 + b) * 64 + lane];
        }
        __builtin_amdgcn_sched_barrier(0);
        if (r + 1 < rounds) {
            load(f, at + step, nx);
            load(g, at + step, ny);
        }
        __builtin_amdgcn_sched_barrier(0);
        auto forward = [&](int b) {
            x[b] = fold4_tw(digit_sums<TURN>(A1, x[b], raw), T1, C);
            y[b] = fold4_tw(digit_sums<TURN>(A1, y[b], raw), T1, C);
            x[b] = fold4_tight(digit_sums<KEEP>(A2, x[b], ti), C);
            y[b] = fold4_tight(digit_sums<KEEP>(A2, y[b], ti), C);
        };
        if constexpr (Point::DIV) {
#pragma unroll
            for (int b = 0; b < TINY_BLOCKS; ++b) forward(b);
            uint32_t valid = 0;
#pragma unroll
            for (int b = 0; b < TINY_BLOCKS; ++b) valid |= (uint32_t)(at + 256 * b + (c / B) * 16 * B < words) << b;
            point(x, y, C, valid);
        }
        uint32_t ls = lw;
        if constexpr (!ROWS) asm volatile("" : "+v"(ls));   // (or each offset is a sum of its own, formed before the loop and held)
#pragma unroll
        for (int b = 0; b < TINY_BLOCKS; ++b) {
            if constexpr (!Point::DIV) {
                forward(b);
                x[b] = mul4_fg<SMALL>(x[b], y[b], C);
            }
            uint32_t a1[4];   // (here: loaded before the transforms they spilled 11 registers)
            if constexpr (CRT) {
                const auto ba = wave_buf(crt.a1 + at, bytes);
#pragma unroll
                for (int i = 0; i < 4; ++i) a1[i] = ld_word(ba, ls, 256 * b + 16 * i);
            }
            x[b] = fold4_tw(digit_sums<TURN>(A3, x[b], ti), T2, C);
            const Sums s = digit_sums<KEEP>(A4, x[b], ti);
            x[b] = ROWS ? fold4_w(s, tt[b], C) : fold4_tight(s, C);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (CRT) st_out2(bh, combined<SMALL>(x[b][i], a1[i], crt, C), ls, 256 * b + 16 * i);
                else st_out<ROWS>(bh, ROWS ? (uint32_t)x[b][i] : out_word<SMALL>(x[b][i], C), ls, 256 * b + 16 * i);
            }
        }
    }
}

template <int n, bool SMALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_conv_tiny(
    const uint32_t* f, const uint32_t* g, uint32_t* h, uint64_t words, int rounds, I8Plan p) {
    tiny_block<n, SMALL, false>(f, g, h, words, rounds, p, blockIdx.x, nullptr, PointMul{});
}
template <int n, bool SMALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_div_tiny(
    const uint32_t* f, const uint32_t* g, uint32_t* h, uint64_t words, int rounds, I8Plan p, Quotient q) {
    tiny_block<n, SMALL, false>(f, g, h, words, rounds, p, blockIdx.x, nullptr, PointDiv(q));
}
template <int n>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_crt_tiny(
    const uint32_t* f, const uint32_t* g, uint64_t words, int rounds, I8Plan p, Combine crt) {
    tiny_block<n, false, false, PointMul, true>(f, g, nullptr, words, rounds, p, blockIdx.x, nullptr, PointMul{}, crt);
}

// ------------------------------------------------------------------ 2^9 .. 2^12
// N = 256 R1, R1 = 2 .. 16; a chunk of 4096 elements (16 / R1 sequences) in the
// registers of the four waves of a workgroup, four registers each.
// Forward, t = t0 + 16 p1 + 16 R1 p2, u = u0 + 16 u1 + 16 R1 u2:
//   register (s, p1): over p2 (c: t0 stays), exchange (s, p1) against u0,
//   register u0: over (s, p1), with w^(16 p1 u0) in the register's own matrix
//   [c: t0 -> (s, u1)], times w^(t0 (u0 + 16 u1)), over t0 (c stays).
// Inverse, position p0 + 16 p1 + 16 R1 p2, the same registers: register p0: over
// p2 [c: (s, p1) -> v0], times w^-(16 p1 v0), over (s, p1) with N^-1 (c stays),
// times w^-(p0 (v0 + 16 v1)), exchange p0 against (s, v1), register (s, v1):
// over p0.  Loads and stores are rows of 16 consecutive words.
// An exchange goes through LDS rows of 16 words, the words of one row the four
// waves' four registers each: 16-byte accesses on both sides, the four pieces of
// a row permuted by two bits of the column so that 16 rows touch every bank.
// One chunk per workgroup, three workgroups per CU; its loads and those of its
// matrices go out together.  Bound by vector issue (81 vector and 7 matrix
// instructions per element).  2^26 elements, m = 13631489, against the LDS
// kernel's fp64 butterflies: 2^12 341 -> 240 us, 2^9 290 -> 234 us; 2^18
// elements 10.7 -> 6.9 and 9.0 -> 7.0 us.  Slower: one wave per chunk with the
// transposes by lane-group swaps and no barrier (242 us, 73 against 59 us at
// 2^24 elements: 8 waves per CU), persistent workgroups at two per CU (262 us).
struct MidTab {   // 16-byte units, as in the plan's table
    static constexpr int W = 0, V = 192, U = 384, M = 576, TF = M + 16 * 192, TK = TF + 16 * 128, TB = TK + 128;
};
__device__ __forceinline__ void mid_put(v4i* x, const v4i (&v)[4], int wave, int gr, int c) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
        x[((4 * gr + i) * 16 + c) * 4 + (wave ^ (c >> 2))] = v4i{v[0][i], v[1][i], v[2][i], v[3][i]};
}
__device__ __forceinline__ void mid_get(const v4i* x, v4i (&v)[4], int wave, int gr, int c) {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = x[((4 * wave + k) * 16 + c) * 4 + (gr ^ (c >> 2))];
}
// First word of register r's element i in lane 0; a sum, mid_word(4 w + k, i) =
// mid_word(4 w, 0) + mid_word(k, i) for k < 4: the wave's part goes to the lane's offset.
template <int n>
__device__ constexpr uint32_t mid_word(int r, int i) {
    constexpr int R1 = (1 << n) / 256;
    return (uint32_t)((r / R1) * (1 << n) + 16 * (r % R1) + 16 * R1 * i);
}
template <int n, bool SMALL, bool ROWS, class Point, bool CRT = false>
__device__ __forceinline__ void mid_block(const uint32_t* f, const uint32_t* g, uint32_t* h, uint64_t words,
                                          const I8Plan& p, uint32_t bx, const v4i* rtt, v4i (*xch)[1024], const Point& point,
                                          const Combine& crt = Combine{}) {
    constexpr int R1 = (1 << n) / 256, N = 1 << n;
    using T = MidTab;
    // xch: f, g, the inverse: two barriers
    const int lane = threadIdx.x & 63, gr = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t at = (uint64_t)bx * 4096;
    const uint32_t bytes = (uint32_t)(words - at < 4096 ? words - at : 4096) * 4;
    const auto bf = wave_buf(f + at, bytes), bg = wave_buf(g + at, bytes),
               bh = CRT ? wave_buf(crt.h + at, 2 * bytes) : wave_buf(h + at, bytes);
    const uint32_t lw = (uint32_t)(c + 16 * R1 * 4 * gr) + (ROWS ? 0 : mid_word<n>(4 * wave, 0));
    auto at_word = [&](int k, int i) { return mid_word<n>(ROWS ? 4 * wave + k : k, i); };
    v4i x[4], y[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) x[k][i] = ld_raw<ROWS>(bf, lw, at_word(k, i)) ^ (ROWS ? (int)DIG : 0);
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) y[k][i] = ld_raw<ROWS>(bg, lw, at_word(k, i)) ^ (ROWS ? (int)DIG : 0);
    const I8K C(p.C);
    const v4i* t = (const v4i*)p.tab;
    const Mat W = ld_mat(t + T::W, lane);
    Mat M[4];
    Tw tw[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        M[k] = ld_mat(t + T::M + (4 * wave + k) * 192, lane);
        tw[k] = ld_tw(t + T::TF + (4 * wave + k) * 128, lane);
    }
    const Init lo = init_loose(C), ti = init_tight(C);
    const Init raw = ROWS ? lo : init_raw(lo, C, [&](int i) { return gr == 0 && i == 0; });
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = fold4_loose(digit_sums<KEEP>(W, x[k], raw), C);
    mid_put(xch[0], x, wave, gr, c);
#pragma unroll
    for (int k = 0; k < 4; ++k) y[k] = fold4_loose(digit_sums<KEEP>(W, y[k], raw), C);
    mid_put(xch[1], y, wave, gr, c);
    __syncthreads();
    mid_get(xch[0], x, wave, gr, c);
    mid_get(xch[1], y, wave, gr, c);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        x[k] = fold4_tw(digit_sums<TURN>(M[k], x[k], ti), tw[k], C);
        y[k] = fold4_tw(digit_sums<TURN>(M[k], y[k], ti), tw[k], C);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) tw[k] = ld_tw(t + T::TB + (4 * wave + k) * 128, lane);
    const Mat V = ld_mat(t + T::V, lane), U = ld_mat(t + T::U, lane);
    const Tw tk = ld_tw(t + T::TK, lane);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        x[k] = fold4_tight(digit_sums<KEEP>(W, x[k], ti), C);
        y[k] = fold4_tight(digit_sums<KEEP>(W, y[k], ti), C);
        if constexpr (!Point::DIV) x[k] = mul4_fg<SMALL>(x[k], y[k], C);
    }
    if constexpr (Point::DIV) point(x, y, C, at + (c / R1) * N < words ? 15 : 0);
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = fold4_tw(digit_sums<TURN>(V, x[k], ti), tk, C);
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = fold4_tw(digit_sums<KEEP>(U, x[k], ti), tw[k], C);
    mid_put(xch[2], x, wave, gr, c);
    v4i tt[4];
    if constexpr (ROWS) {
#pragma unroll
        for (int k = 0; k < 4; ++k) tt[k] = rtt[((uint64_t)bx * 16 + 4 * wave + k) * 64 + lane];
    }
    uint32_t a1[4][4];
    if constexpr (CRT) {
        const auto ba = wave_buf(crt.a1 + at, bytes);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) a1[k][i] = ld_word(ba, lw, at_word(k, i));
    }
    __syncthreads();
    mid_get(xch[2], x, wave, gr, c);
    const uint32_t ls = ROWS ? lw : keep(lw);   // (or sixteen sums for the stores are formed and held with the loads')
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const Sums s = digit_sums<KEEP>(V, x[k], ti);
        x[k] = ROWS ? fold4_w(s, tt[k], C) : fold4_tight(s, C);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (CRT) st_out2(bh, combined<SMALL>(x[k][i], a1[k][i], crt, C), ls, at_word(k, i));
            else st_out<ROWS>(bh, ROWS ? (uint32_t)x[k][i] : out_word<SMALL>(x[k][i], C), ls, at_word(k, i));
        }
    }
}

template <int n, bool SMALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_conv_mid(
    const uint32_t* f, const uint32_t* g, uint32_t* h, uint64_t words, I8Plan p) {
    __shared__ v4i xch[3][1024];
    mid_block<n, SMALL, false>(f, g, h, words, p, blockIdx.x, nullptr, xch, PointMul{});
}
template <int n, bool SMALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_div_mid(
    const uint32_t* f, const uint32_t* g, uint32_t* h, uint64_t words, I8Plan p, Quotient q) {
    __shared__ v4i xch[3][1024];
    mid_block<n, SMALL, false>(f, g, h, words, p, blockIdx.x, nullptr, xch, PointDiv(q));
}
template <int n>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_crt_mid(
    const uint32_t* f, const uint32_t* g, uint64_t words, I8Plan p, Combine crt) {
    __shared__ v4i xch[3][1024];
    mid_block<n, false, false, PointMul, true>(f, g, nullptr, words, p, blockIdx.x, nullptr, xch, PointMul{}, crt);
}

// ------------------------------------------------------------------ transforms
// The inverse halves of the convolutions above by themselves, natural order on
// both sides, from tables of w for a forward transform and of w^-1 and N^-1 for an
// inverse one: each word is read and written once.  This half rather than the
// forward one, because the short pieces lie on the side of the loads (2^26 elements
// of 2^6: 105 us, the forward half 139; of 2^10: 128 and 188).  Bound by memory from
// 2^24 elements on (2^26, against the LDS kernel's fp64 butterflies: 2^5 241 -> 145 us,
// 2^8 103 -> 100, 2^9 124 -> 119; 2^24 elements of 2^8 25 -> 22, of 2^10 36 -> 27, of 2^12 40 -> 28).
// N <= 2^8: inputs p0 + B p', register element p', column (s, p0).  One pass per wave:
// beyond the memory-side cache several passes with the next one's words loaded ahead
// are slower (2^25.3 elements of 2^8 60 against 64 us).
template <int n, bool SMALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_ntt_tiny(const uint32_t* f,
                                                                                            uint32_t* h, uint64_t words,
                                                                                            I8Plan p) {
    constexpr int B = (1 << n) / 16;
    constexpr uint32_t CH = 256 * TINY_BLOCKS;
    const int lane = threadIdx.x & 63, gr = lane >> 4, c = lane & 15;
    const uint64_t at = ((uint64_t)blockIdx.x * 4 + (uint64_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * CH;
    if (at >= words) return;
    const uint32_t bytes = (uint32_t)(words - at < CH ? words - at : CH) * 4;
    const auto bf = wave_buf(f + at, bytes), bh = wave_buf(h + at, bytes);
    const uint32_t li = (uint32_t)((c / B) * 16 * B + c % B + 4 * B * gr), lo = (uint32_t)(c + 64 * gr);
    v4i x[TINY_BLOCKS];
#pragma unroll
    for (int b = 0; b < TINY_BLOCKS; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) x[b][i] = ld_raw(bf, li, 256 * b + B * i);
    const I8K C(p.C);
    const v4i* t = (const v4i*)p.tab;
    const Mat A1 = ld_mat(t + 384, lane), A2 = ld_mat(t + 576, lane);
    const Tw T1 = ld_tw(t + 768 + 128, lane);
    const Init ti = init_tight(C), raw = init_raw(ti, C, [&](int) { return c == 0; });
#pragma unroll
    for (int b = 0; b < TINY_BLOCKS; ++b) {
        x[b] = fold4_tw(digit_sums<TURN>(A1, x[b], raw), T1, C);
        x[b] = fold4_tight(digit_sums<KEEP>(A2, x[b], ti), C);
#pragma unroll
        for (int i = 0; i < 4; ++i) st_out(bh, out_word<SMALL>(x[b][i], C), lo, 256 * b + 16 * i);
    }
}

// 2^9 .. 2^12: inputs p0 + 16 (p1 + R1 p2) with p0 in the registers: 16 consecutive
// bytes per lane, and a row of 64 in the four waves.  Four waves per SIMD: five are even
// (2^24 elements of 2^9 26.7 against 27.3 us, 2^25.3 77 / 77, 2^26 119 / 121), and spill where
// the two steps share a loop.
template <int n, bool SMALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_ntt_mid(const uint32_t* f,
                                                                                           uint32_t* h, uint64_t words,
                                                                                           I8Plan p) {
    constexpr int R1 = (1 << n) / 256, N = 1 << n;
    using T = MidTab;
    __shared__ v4i xch[1024];
    const int lane = threadIdx.x & 63, gr = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t at = (uint64_t)blockIdx.x * 4096;
    const uint32_t bytes = (uint32_t)(words - at < 4096 ? words - at : 4096) * 4;
    const auto bf = wave_buf(f + at, bytes), bh = wave_buf(h + at, bytes);
    const uint32_t li = (uint32_t)((c / R1) * N + 16 * (c % R1) + 16 * R1 * 4 * gr + 4 * wave),
                   lo = (uint32_t)(c + 16 * R1 * 4 * gr) + mid_word<n>(4 * wave, 0);
    v4i x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(bf, (li + 16 * R1 * i) * 4, 0, 0);
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k][i] = (int)(v[k] ^ DIG);
    }
    const I8K C(p.C);
    const v4i* t = (const v4i*)p.tab;
    const Mat V = ld_mat(t + T::V, lane), U = ld_mat(t + T::U, lane);
    const Tw tk = ld_tw(t + T::TK, lane);
    Tw tw[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) tw[k] = ld_tw(t + T::TB + (4 * wave + k) * 128, lane);
    const Init ti = init_tight(C), raw = init_raw(ti, C, [&](int) { return c == 0; });
    // (two loops: 106 registers, 116 with both steps in one)
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = fold4_tw(digit_sums<TURN>(V, x[k], raw), tk, C);
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = fold4_tw(digit_sums<KEEP>(U, x[k], ti), tw[k], C);
    mid_put(xch, x, wave, gr, c);
    __syncthreads();
    mid_get(xch, x, wave, gr, c);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        x[k] = fold4_tight(digit_sums<KEEP>(V, x[k], ti), C);
#pragma unroll
        for (int i = 0; i < 4; ++i) st_out(bh, out_word<SMALL>(x[k][i], C), lo, mid_word<n>(k, i));
    }
}

}  // namespace nttmi
