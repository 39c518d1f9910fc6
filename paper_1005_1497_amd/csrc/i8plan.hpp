// Host side of the matrix-core transforms: constants and tables of one plan.
#pragma once
#include <cstring>
#include <vector>

#include "launch.hpp"
#include "numtheory.hpp"

namespace nttmi {

// The signed digits of a residue: three of the representative that fits them
// (any window of m <= 2^24 consecutive integers from -8421504 on does).
inline void i8_digits(uint64_t x, uint64_t m, int8_t d[3]) {
    int64_t v = (int64_t)(x % m);
    if (v > 8355711) v -= (int64_t)m;
    for (int c = 0; c < 3; ++c) {
        d[c] = (int8_t)(uint8_t)(v & 255);
        v = (v - d[c]) >> 8;
    }
}

// Appends the fragments of a 16 x 16 matrix (row: output, column: input) in the
// lanes' order: plane c, lane l = 16 g + row, bytes 4 i + a the digit c of
// 256^a M[row][4 g + i].
template <class F>
inline void i8_matrix(std::vector<int8_t>& out, uint64_t m, F entry) {
    const size_t at = out.size();
    out.resize(at + 3 * 64 * 16);
    for (int l = 0; l < 64; ++l)
        for (int i = 0; i < 4; ++i) {
            uint64_t x = entry(l & 15, 4 * (l >> 4) + i) % m;
            for (int a = 0; a < 4; ++a) {
                int8_t d[3];
                i8_digits(x, m, d);
                for (int c = 0; c < 3; ++c) out[at + (size_t)(c * 64 + l) * 16 + 4 * i + a] = d[c];
                x = x * 256 % m;
            }
        }
}

inline void i8_pair(std::vector<int8_t>& out, uint64_t w, uint64_t m) {
    int64_t b = (int64_t)(w % m);
    if (2 * b > (int64_t)m) b -= (int64_t)m;
    const int32_t wi = (int32_t)b;
    const float wq = (float)(-(double)b / (double)m);
    const size_t at = out.size();
    out.resize(at + 8);
    std::memcpy(&out[at], &wi, 4);
    std::memcpy(&out[at + 4], &wq, 4);
}

// radix: of the first step (the correction for raw words)
inline I8C make_i8c(uint64_t m, int radix) {
    I8C C{};
    const uint32_t mu = (uint32_t)m, dig = 0x80808080u;
    C.m = mu;
    C.small = m < (1u << 21) ? 1u : 0u;
    C.k16 = (float)(-65536.0 / (double)m);
    C.mg2 = (float)(12582912.0 - 12582912.0 * (double)C.k16);
    C.k8 = (float)(-256.0 / (double)m);
    C.mi = (float)(-1.0 / (double)m);
    C.it = (int32_t)(0u - 0x400000u * mu);
    C.il = (int32_t)(dig - 0x400000u * mu);
    C.ip = (int32_t)(dig - 0x800000u * mu);
    int8_t d[3];
    i8_digits(((uint64_t)dig % m) * (uint64_t)radix, m, d);
    C.c0 = d[0];
    C.c1 = d[1];
    C.c2 = d[2];
    return C;
}

// Appends N residues w(r, l, i) (r < N / 256, lane l, i < 4) as words in (-m/2, m/2].
template <class F>
inline void i8_words(std::vector<int8_t>& out, uint64_t N, uint64_t m, F w) {
    const size_t at = out.size();
    out.resize(at + 4 * N);
    int8_t* p = &out[at];
    for (uint64_t r = 0; r < N / 256; ++r)
        for (uint64_t l = 0; l < 64; ++l)
            for (uint64_t i = 0; i < 4; ++i, p += 4) {
                const uint64_t x = w(r, l, i);
                const int32_t b = (int32_t)(2 * x > m ? (int64_t)x - (int64_t)m : (int64_t)x);
                std::memcpy(p, &b, 4);
            }
}

// Tables of the kernels in wave.hpp; w^e = P(e) for e < N.
template <class PW>
inline std::vector<int8_t> i8_wave_tables(int n, uint64_t m, uint64_t ninv, PW P, I8C* C) {
    const int N = 1 << n;
    std::vector<int8_t> t;
    auto fw = [&](uint64_t e) -> uint64_t { return P(e & (N - 1)); };
    auto bw = [&](uint64_t e) -> uint64_t { return P((0 - e) & (N - 1)); };
    auto w16 = [&](int row, int in) { return fw((uint64_t)(N / 16) * row * in); };
    auto v16 = [&](int row, int in) { return bw((uint64_t)(N / 16) * row * in); };
    if (n <= 8) {
        const int B = N / 16;
        i8_matrix(t, m, [&](int row, int in) -> uint64_t {
            return row / B != in / B ? 0 : fw((uint64_t)16 * (row % B) * (in % B));
        });
        i8_matrix(t, m, w16);
        i8_matrix(t, m, v16);
        i8_matrix(t, m, [&](int row, int in) -> uint64_t {
            return row / B != in / B ? 0 : mulmod64(bw((uint64_t)16 * (row % B) * (in % B)), ninv, m);
        });
        for (int l = 0; l < 64; ++l)
            for (int i = 0; i < 4; ++i) i8_pair(t, fw((uint64_t)(4 * (l >> 4) + i) * ((l & 15) % B)), m);
        for (int l = 0; l < 64; ++l)
            for (int i = 0; i < 4; ++i) i8_pair(t, bw((uint64_t)((4 * (l >> 4) + i) % B) * (l & 15)), m);
        *C = make_i8c(m, B);
        return t;
    }
    const int R1 = N / 256;
    i8_matrix(t, m, w16);
    i8_matrix(t, m, v16);
    i8_matrix(t, m, [&](int row, int in) -> uint64_t {
        return row / R1 != in / R1 ? 0 : mulmod64(bw((uint64_t)256 * (row % R1) * (in % R1)), ninv, m);
    });
    for (int u0 = 0; u0 < 16; ++u0)
        i8_matrix(t, m, [&](int row, int in) -> uint64_t {
            return row / R1 != in / R1 ? 0 : fw((uint64_t)256 * (row % R1) * (in % R1) + (uint64_t)16 * (in % R1) * u0);
        });
    for (int u0 = 0; u0 < 16; ++u0)
        for (int l = 0; l < 64; ++l)
            for (int i = 0; i < 4; ++i)
                i8_pair(t, fw((uint64_t)(4 * (l >> 4) + i) * (u0 + 16 * ((l & 15) % R1))), m);
    for (int l = 0; l < 64; ++l)
        for (int i = 0; i < 4; ++i) i8_pair(t, bw((uint64_t)16 * ((4 * (l >> 4) + i) % R1) * (l & 15)), m);
    for (int p0 = 0; p0 < 16; ++p0)
        for (int l = 0; l < 64; ++l)
            for (int i = 0; i < 4; ++i)
                i8_pair(t, bw((uint64_t)p0 * ((l & 15) + 16 * ((4 * (l >> 4) + i) % R1))), m);
    *C = make_i8c(m, 16);
    return t;
}

// Tables of the kernels in trans.hpp, N = 2^n = 256 Q; w^e = P(e) for e < N, the
// transform's root (its inverse for the inverse), scale = 1 (N^-1).
template <class PW>
inline std::vector<int8_t> i8_trans_tables(int n, uint64_t m, uint64_t scale, PW P, I8C* C) {
    const uint64_t N = 1ull << n, Q = N / 256, R = Q > 256 ? Q / 256 : 1, B = Q / R / 16;
    auto fw = [&](uint64_t e) -> uint64_t { return P(e & (N - 1)); };
    std::vector<int8_t> t;
    // columns: w_256 = w^Q
    i8_matrix(t, m, [&](int row, int in) { return fw(Q * 16 * row * in); });
    for (int u0 = 0; u0 < 16; ++u0)
        i8_matrix(t, m, [&](int row, int in) { return fw(Q * (16 * row * in + in * u0)); });
    // rows, t1 = t0 + 16 p1 + 16 B k, u1 = j + R (U + B u2'): w_Q = w^256
    i8_matrix(t, m, [&](int row, int in) { return mulmod64(fw(N / 16 * row * in), scale, m); });
    for (uint64_t j = 0; j < R; ++j) {
        for (uint64_t k = 0; k < R; ++k)
            i8_matrix(t, m, [&](int row, int in) -> uint64_t {
                const uint64_t p1 = in % B;
                return row / B != in / B ? 0 : fw(256 * 16 * (R * (row % B) * p1 + j * (p1 + B * k)));
            });
        for (int l = 0; l < 64; ++l)
            for (int i = 0; i < 4; ++i) i8_pair(t, fw((uint64_t)256 * (4 * (l >> 4) + i) * (j + R * ((l & 15) % B))), m);
    }
    // blocks of 32 columns; register u0; columns t1 = 2 c, then 2 c + 1; u2 = u0 + 16 (4 g + i):
    // residues in (-m/2, m/2]
    i8_words(t, N, m, [&](uint64_t r, uint64_t l, uint64_t i) {
        return fw((32 * (r / 32) + 2 * (l & 15) + r % 2) * (r / 2 % 16 + 16 * (4 * (l >> 4) + i)));
    });
    *C = make_i8c(m, 16);
    return t;
}

// Tables of the rows of four.hpp, N = 2^n = 256 Q: those of wave.hpp for length Q
// (with the N^-1 of the whole) and, from `tti` on, the twiddles w^-(s1 u2) as residues
// in (-m/2, m/2] in the order of the row kernels' registers.
template <class PW>
inline std::vector<int8_t> i8_four_tables(int n, uint64_t m, uint64_t ninv, PW P, size_t* tti, I8C* C) {
    const int la = n - 8;
    const uint64_t N = 1ull << n, A = 1ull << la;
    std::vector<int8_t> t = i8_wave_tables(la, m, ninv, [&](uint64_t e) { return P(256 * e); }, C);
    *tti = t.size();
    i8_words(t, N, m, [&](uint64_t r, uint64_t l, uint64_t i) {
        const uint64_t k = 4 * (l >> 4) + i, c = l & 15;
        // the element's place in the scratch: blocks of 256 in order, or chunks of
        // 4096 whose registers are (row, v1)
        uint64_t e = 256 * r + 16 * k + c;
        if (la > 8) {
            const uint64_t R1 = A / 256, q = r % 16;
            e = 4096 * (r / 16) + (q / R1) * A + c + 16 * (q % R1) + 16 * R1 * k;
        }
        return P((0 - (e & (A - 1)) * (e >> la)) & (N - 1));
    });
    return t;
}

// Tables of the kernels in wide.hpp, N = 2^n = 4096 R; w^e = P(e) for e < N.
template <class PW>
inline std::vector<int8_t> i8_wide_tables(int n, uint64_t m, uint64_t ninv, PW P, I8C* C) {
    const uint64_t N = 1ull << n;
    const int R = (int)(N / 4096);
    std::vector<int8_t> t;
    auto fw = [&](uint64_t e) -> uint64_t { return P(e & (N - 1)); };
    auto bw = [&](uint64_t e) -> uint64_t { return P((0 - e) & (N - 1)); };
    const uint64_t h16 = N / 16, h256 = (uint64_t)16 * R, h4096 = (uint64_t)R;   // exponents of w_16, w_256, w_4096
    // shared: the plain step, w_256^-(p1 v0), w_4096^-(p0 (v0 + 16 v1))
    i8_matrix(t, m, [&](int row, int in) { return fw(h16 * row * in); });
    for (int l = 0; l < 64; ++l)
        for (int i = 0; i < 4; ++i) i8_pair(t, bw(h256 * (uint64_t)(4 * (l >> 4) + i) * (l & 15)), m);
    for (int p0 = 0; p0 < 16; ++p0)
        for (int l = 0; l < 64; ++l)
            for (int i = 0; i < 4; ++i)
                i8_pair(t, bw(h4096 * (uint64_t)p0 * ((l & 15) + 16 * (4 * (l >> 4) + i))), m);
    // per j, with the twist w^(j t') of the inputs and w^-(j t') of the outputs
    for (uint64_t j = 0; j < (uint64_t)R; ++j) {
        i8_matrix(t, m, [&](int row, int in) { return bw(h16 * row * in + j * row); });
        i8_matrix(t, m, [&](int row, int in) { return mulmod64(bw(h16 * row * in + 16 * j * row), ninv, m); });
        for (int u0 = 0; u0 < 16; ++u0)
            i8_matrix(t, m, [&](int row, int in) { return fw(h16 * row * in + h256 * in * u0 + 16 * j * in); });
        for (int u0 = 0; u0 < 16; ++u0)
            for (int l = 0; l < 64; ++l)
                for (int i = 0; i < 4; ++i) {
                    const uint64_t t0 = 4 * (l >> 4) + i;
                    i8_pair(t, fw(h4096 * t0 * (u0 + 16 * (l & 15)) + j * t0), m);
                }
        for (int k = 0; k < R; ++k)
            i8_matrix(t, m, [&](int row, int in) { return fw(h16 * row * in + 256 * j * in + N / R * j * k); });
        for (int k = 0; k < R; ++k)
            i8_matrix(t, m, [&](int row, int in) { return bw(h16 * row * in + 256 * j * row + N / R * j * k); });
    }
    *C = make_i8c(m, 16 * R);
    return t;
}

}  // namespace nttmi
