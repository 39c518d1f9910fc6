// Transforms of 32-bit words on the matrix cores (gfx950), one wave at a time.
//
// A radix-16 step of Eq. 2 is a product by a 16 x 16 matrix of powers of the
// root.  A residue is held as a 32-bit integer whose four bytes are signed
// digits (x = sum_a d_a 256^a, -128 <= d_a < 128), and a matrix entry enters as
// the three signed digits of each of 256^a w mod m, so that one
// v_mfma_i32_16x16x64_i8 per digit of the entries forms, exactly, the sums
//   s_c = sum_{r, a} d_a(x_r) digit_c(256^a w^(u r) mod m),   c = 0, 1, 2,
// and X(u) = s_0 + 256 s_1 + 65536 s_2 modulo m.  |s_c| <= 64 * 128 * 128 = 2^20.
// The matrix pipe does the contraction; the vector units only fold the three
// sums into one residue: four 32-bit instructions and one XOR that turns it
// into digits again, against about ten 64-bit ones for a radix-16 butterfly
// with its twiddles in fp64 (5.75 instructions per element and pass with the
// matrix instructions counted, 10.5 before).
//
// Twiddles: those between the two steps of a transform of length up to 256 are
// folded into the matrices of the second step (one matrix per u0); a single
// element-wise product per element and transform is left.
//
// Range.  loose: r = X + q m with q the rounded quotient of 65536 s_2 alone,
// |r| <= 256 |s_1| + |s_0| + m < 2^29: an int32, digits of the next step.
// tight: q from 256 (256 s_2 + s_1): |r| <= 0.502 m + 2^20, below 2^23 for
// m <= I8_MAX_M, as the 24-bit products of the element-wise steps need.  The
// quotients come from 32-bit floats and may be off by one; every sum and
// product that enters a result is an integer modulo 2^32 whose true value fits
// 32 bits, so results are exact.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch.hpp"

namespace nttmi {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

constexpr uint32_t DIG = 0x80808080u;   // x + DIG, XOR DIG: the signed digits of x

// 24-bit products as single instructions (the empty asm keeps the compiler from
// regrouping the additions across them).
__device__ __forceinline__ uint32_t keep(uint32_t x) {
    asm("" : "+v"(x));
    return x;
}
__device__ __forceinline__ uint32_t lshl8_add(uint32_t a, uint32_t b) { return keep((a << 8) + b); }
__device__ __forceinline__ uint32_t mad24u(uint32_t a, uint32_t b, uint32_t c) {
    return keep((uint32_t)__umul24(a, b) + c);
}
__device__ __forceinline__ uint32_t mad24s(int32_t a, int32_t b, uint32_t c) {
    return keep((uint32_t)__mul24(a, b) + c);
}
__device__ __forceinline__ float keep(float x) {
    asm("" : "+v"(x));
    return x;
}
// The constants as the kernels hold them: the multipliers of the quotients in
// vector registers, since a float multiply-add with a scalar operand takes
// twice the time of one without (4.2 against 2.7 clocks per wave).
struct I8K : I8C {
    float vk16, vmg2, vk8, vmi;
    __device__ __forceinline__ explicit I8K(const I8C& c) : I8C(c), vk16(keep(c.k16)), vmg2(keep(c.mg2)), vk8(keep(c.k8)), vmi(keep(c.mi)) {}
};
__device__ __forceinline__ uint32_t fbits(float f) { return __builtin_bit_cast(uint32_t, f); }

// One radix-16 step of 16 columns: the three digit sums.  Data: lane l holds
// column l % 16, inputs 4 (l / 16) .. + 3.  Matrix fragment: lane l holds output
// l % 16, inputs 4 (l / 16) .. + 3.  With the matrix as the first operand the
// outputs 4 (l / 16) .. + 3 of column l % 16 come back (the column stays in the
// lane); with the data as the first operand lane l gets output l % 16 of the
// columns 4 (l / 16) .. + 3, which is the data layout of a next step over the
// columns' own index: two steps follow one another with nothing moved.
struct Mat {
    v4i a[3];
};
__device__ __forceinline__ Mat ld_mat(const v4i* t, int lane) {
    Mat A;
#pragma unroll
    for (int c = 0; c < 3; ++c) A.a[c] = t[c * 64 + lane];
    return A;
}
__device__ __forceinline__ v4i splat(uint32_t x) { return v4i{(int)x, (int)x, (int)x, (int)x}; }
// accumulators' initial values
struct Init {
    v4i s0, s1, s2;
};
struct Sums {
    v4i s0, s1, s2;
};
enum { KEEP = 0, TURN = 1 };   // the column stays in the lane; the output goes there
template <int TYPE>
__device__ __forceinline__ Sums digit_sums(const Mat& A, const v4i& x, const Init& in) {
    Sums s;
    if constexpr (TYPE == KEEP) {
        s.s2 = __builtin_amdgcn_mfma_i32_16x16x64_i8(A.a[2], x, in.s2, 0, 0, 0);
        s.s1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(A.a[1], x, in.s1, 0, 0, 0);
        s.s0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(A.a[0], x, in.s0, 0, 0, 0);
    } else {
        s.s2 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x, A.a[2], in.s2, 0, 0, 0);
        s.s1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x, A.a[1], in.s1, 0, 0, 0);
        s.s0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(x, A.a[0], in.s0, 0, 0, 0);
    }
    return s;
}

// The float 1.5 2^23 + q carries the integer q in its low bits: as the 24-bit
// operand of a product it is 0x400000 + q, whose constant part the initial
// values take away (I8C::il, I8C::it).
constexpr float MAGIC = 12582912.0f;

// s2 starts at the bits of MAGIC, so that it reads as the float MAGIC + s_2
// (its low half is zero: s2 << 16 is unchanged).
__device__ __forceinline__ Init init_loose(const I8K& C) {
    return Init{splat((uint32_t)C.il), splat(0), splat(0x4B400000u)};
}
__device__ __forceinline__ Init init_tight(const I8K& C) { return Init{splat((uint32_t)C.it), splat(0), splat(0)}; }

// signed digits of the loose residue
__device__ __forceinline__ uint32_t fold_loose(int s0, int s1, int s2, const I8K& C) {
    const float q = __builtin_fmaf(__builtin_bit_cast(float, s2), C.vk16, C.vmg2);
    const uint32_t t = lshl8_add(lshl8_add((uint32_t)s2, (uint32_t)s1), (uint32_t)s0);
    return mad24u(fbits(q), C.m, t) ^ DIG;
}
// the tight residue itself
__device__ __forceinline__ int32_t fold_tight(int s0, int s1, int s2, const I8K& C) {
    const uint32_t a = lshl8_add((uint32_t)s2, (uint32_t)s1);
    const float q = __builtin_fmaf((float)(int32_t)a, C.vk8, MAGIC);
    return (int32_t)mad24u(fbits(q), C.m, lshl8_add(a, (uint32_t)s0));
}
// |r| <= m/2 + 1 from |r| < 2^24 (moduli so small that the unreduced s_0 counts)
__device__ __forceinline__ int32_t reduce_i(int32_t r, const I8K& C) {
    const float q = __builtin_fmaf((float)r, C.vmi, MAGIC);
    return (int32_t)mad24u(fbits(q), C.m, (uint32_t)r + (uint32_t)C.it);
}
// b w mod m for a tight b, as digits: w a balanced residue, wq = -w / m.
__device__ __forceinline__ uint32_t mul_tw_i(int32_t b, int32_t w, float wq, const I8K& C) {
    const float q = __builtin_fmaf((float)b, wq, MAGIC);
    return mad24u(fbits(q), C.m, mad24s(b, w, (uint32_t)C.il)) ^ DIG;
}
// F G mod m for two tight residues, as digits.  |F G| / m < 2^23 may pass the
// range of MAGIC, so the quotient is taken as the integer 2^23 + q.
__device__ __forceinline__ uint32_t mul_fg_i(int32_t F, int32_t G, const I8K& C) {
    const uint32_t q = (uint32_t)__builtin_fmaf((float)F * C.vmi, (float)G, 8388608.0f);
    return mad24u(q, C.m, mad24s(F, G, (uint32_t)C.ip)) ^ DIG;
}
// canonical residue of a tight one (Appendix A)
__device__ __forceinline__ uint32_t canon_i(int32_t r, const I8K& C) {
    const uint32_t u = (uint32_t)r, v = u + C.m;   // r < 0 is the larger unsigned value
    return u < v ? u : v;
}

// The four residues of one step as digits (loose), as tight residues, and as
// digits times the element-wise twiddles tw = (w0, -w0/m, w1, -w1/m), (w2, ...).
__device__ __forceinline__ v4i fold4_loose(const Sums& s, const I8K& C) {
    v4i r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = (int)fold_loose(s.s0[i], s.s1[i], s.s2[i], C);
    return r;
}
__device__ __forceinline__ v4i fold4_tight(const Sums& s, const I8K& C) {
    v4i r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = fold_tight(s.s0[i], s.s1[i], s.s2[i], C);
    return r;
}
struct Tw {
    v4i p[2];
};
__device__ __forceinline__ Tw ld_tw(const v4i* t, int lane) { return Tw{{t[2 * lane], t[2 * lane + 1]}}; }
__device__ __forceinline__ v4i fold4_tw(const Sums& s, const Tw& tw, const I8K& C) {
    v4i r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int w = tw.p[i >> 1][2 * (i & 1)], wq = tw.p[i >> 1][2 * (i & 1) + 1];
        r[i] = (int)mul_tw_i(fold_tight(s.s0[i], s.s1[i], s.s2[i], C), w, __builtin_bit_cast(float, wq), C);
    }
    return r;
}
__device__ __forceinline__ v4i mul4_tw(const v4i& b, const Tw& tw, const I8K& C) {
    v4i r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int w = tw.p[i >> 1][2 * (i & 1)], wq = tw.p[i >> 1][2 * (i & 1) + 1];
        r[i] = (int)mul_tw_i(b[i], w, __builtin_bit_cast(float, wq), C);
    }
    return r;
}
// the same with the residues w alone (w / m formed here)
__device__ __forceinline__ v4i fold4_w(const Sums& s, const v4i& w, const I8K& C) {
    v4i r;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        r[i] = (int)mul_tw_i(fold_tight(s.s0[i], s.s1[i], s.s2[i], C), w[i], (float)w[i] * C.vmi, C);
    return r;
}
// F G as digits, of four tight residues each
template <bool SMALL>
__device__ __forceinline__ v4i mul4_fg(v4i F, v4i G, const I8K& C) {
    v4i r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int a = F[i], b = G[i];
        if constexpr (SMALL) {
            a = reduce_i(a, C);
            b = reduce_i(b, C);
        }
        r[i] = (int)mul_fg_i(a, b, C);
    }
    return r;
}
template <bool SMALL>
__device__ __forceinline__ uint32_t out_word(int r, const I8K& C) {
    if constexpr (SMALL) r = reduce_i(r, C);
    return canon_i(r, C);
}

// Initial values of a first step over raw words (x XOR DIG holds the digits of
// x - DIG): its outputs of index 0 take the correction R DIG mod m, R the
// step's radix, in digits.  zero(i): whether the lane's result i is one of them.
template <class Z>
__device__ __forceinline__ Init init_raw(const Init& base, const I8K& C, Z zero) {
    Init in = base;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool z = zero(i);
        in.s0[i] += z ? C.c0 : 0;
        in.s1[i] += z ? C.c1 : 0;
        in.s2[i] += z ? C.c2 : 0;
    }
    return in;
}

}  // namespace nttmi
