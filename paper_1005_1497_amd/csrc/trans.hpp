// Transforms of 32-bit words of length 2^13 .. 2^19 on the matrix cores, natural
// order, in two launches: N = 256 Q, t = t1 + Q t2, u = u2 + 256 u1.
//   columns: length-256 transforms over t2, times w^(t1 u2), into scratch as digits;
//   rows: length-Q transforms over t1, stored transposed.
// Rows longer than 256 split into R = Q / 256 transforms of 256 points (t1 = t' + 256 k,
// u1 = j + R u'), a workgroup each: the sum over k runs on in the first step's matrix
// products, with the twist w_Q^(j t') in its tables, and the R workgroups of a row find
// its words in their die's L2.
// Scratch: row u2 = k + 16 (s + S q), k < 16, S = 256 / Q (Q < 256), is words
// S Q k + Q s + t1 of chunk q of 16 S rows, so that the four registers of a lane in the
// second launch are four neighbouring rows, and its stores rows of 64 bytes.
// Both launches move 8 bytes per element (the scratch in the memory-side cache) and
// are bound by that up to R = 4; at R = 8 by the first step's matrix instructions.
// Forward / inverse, m = 13631489, 2^24 elements, against the fp64 four-step
// kernels: 2^13 74 / 127 -> 47 / 47 us, 2^16 79 / 100 -> 48 / 48, 2^19 107 / 140 -> 77 / 75; 2^26
// of 2^16 304 / 400 -> 209 / 208; one row of 2^16 9.2 / 9.8 -> 6.9 / 6.9.
#pragma once
#include "wave.hpp"

namespace nttmi {

template <int n>
struct TransG {
    static constexpr uint32_t N = 1u << n, Q = N / 256, S = Q < 256 ? 256 / Q : 1, R = Q > 256 ? Q / 256 : 1;
    static constexpr uint32_t B = Q / R / 16;
};
template <int n>
struct TransTab {   // 16-byte units: columns' matrices, rows' (for each j: R first steps, twiddles), w^(t1 u2) as words
    static constexpr uint32_t R = TransG<n>::R;
    static constexpr int W = 0, M = 192, A2 = M + 16 * 192, J = A2 + 192, SIZE = R * 192 + 128, TT = J + R * SIZE;
};

// Workgroups go round the eight dies, each with its own L2; two neighbouring
// blocks of 16 columns share every cache line of 128 bytes, so workgroups whose
// numbers differ by eight take them (the last few of a number that is no multiple
// of 16 keep their order).
__device__ __forceinline__ uint32_t pair_blocks(uint32_t id, uint32_t blocks) {
    const uint32_t r = id & 15;
    return (id | 15) < blocks ? (id & ~15u) + 2 * (r & 7) + (r >> 3) : id;
}

// Columns: 16 V of them in the registers of four waves, V neighbours to a lane.  V = 2
// makes a row's piece a whole cache line and has more loads in flight (2^26 elements,
// forward columns of two operands: 341 -> 250 us, inverse 148 -> 105); V = 1 is for few
// blocks, where a workgroup's own time counts (one item of 2^19 17.4 -> 15.6 us).  t2 = p1 + 16 p2, u2 = u0 + 16 u1: register p1 over
// p2, exchange p1 against u0, register u0 over p1 with w_256^(p1 u0) in its matrix (the
// column stays in the lane).  TRANSFORM: words to digits times w^(t1 u2), the rows as
// above; FORWARD: the rows in their order; INVERSE: digits, the rows in their order, to
// words.
enum { TRANSFORM, FORWARD, INVERSE };
// CRT: INVERSE with the combining store instead (dst: this item's residues of the other
// modulus, read only; crt.h: its results).
template <int n, int KIND, bool SMALL, int V, bool CRT = false>
__device__ __forceinline__ void cols_block(const uint32_t* src, uint32_t* dst, uint32_t bx, const I8Plan& p,
                                           v4i (*xch)[1024], const Combine& crt = Combine{}) {
    using G = TransG<n>;
    using T = TransTab<n>;
    constexpr uint32_t N = G::N, Q = G::Q, S = KIND == TRANSFORM ? G::S : 1;
    const int lane = threadIdx.x & 63, gr = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const auto bs = wave_buf(src, N * 4), bd = wave_buf(dst, N * 4);
    // row 4 wave + k + 16 (4 g + i), columns V c ..
    const uint32_t lw = V * (uint32_t)c + 64 * Q * (uint32_t)gr;
    auto at_word = [&](int k, int i) { return 16 * V * bx + Q * (uint32_t)(4 * wave + k + 16 * i); };
    v4i x[V][4], tt[V][4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (V == 2) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(bs, lw * 4, at_word(k, i) * 4, 0);
                x[0][k][i] = (int)v[0];
                x[1][k][i] = (int)v[1];
            } else
                x[0][k][i] = (int)__builtin_amdgcn_raw_buffer_load_b32(bs, lw * 4, at_word(k, i) * 4, 0);
        }
    uint32_t a1[CRT ? 4 : 1][4][V];
    if constexpr (CRT)
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (V == 2) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b64(bd, lw * 4, at_word(k, i) * 4, 0);
                    a1[k][i][0] = v[0], a1[k][i][1] = v[1];
                } else
                    a1[k][i][0] = __builtin_amdgcn_raw_buffer_load_b32(bd, lw * 4, at_word(k, i) * 4, 0);
            }
    const I8K C(p.C);
    const v4i* t = (const v4i*)p.tab;
    const Mat W = ld_mat(t + T::W, lane);
    Mat M[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) M[k] = ld_mat(t + T::M + (4 * wave + k) * 192, lane);
    if constexpr (KIND != INVERSE)
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int s = 0; s < V; ++s) {   // (in the order of V = 2)
                const uint32_t b = V == 2 ? bx : bx / 2, odd = V == 2 ? s : c & 1,
                               at = V == 2 ? lane : 16 * gr + 8 * (bx & 1) + (c >> 1);
                tt[s][k] = t[T::TT + ((b * 16 + 4 * wave + k) * 2 + odd) * 64 + at];
            }
    const Init lo = init_loose(C), ti = init_tight(C);
    const Init raw = KIND == INVERSE ? lo : init_raw(lo, C, [&](int i) { return gr == 0 && i == 0; });
#pragma unroll
    for (int s = 0; s < V; ++s) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if constexpr (KIND != INVERSE)
#pragma unroll
                for (int i = 0; i < 4; ++i) x[s][k][i] ^= (int)DIG;
            x[s][k] = fold4_loose(digit_sums<KEEP>(W, x[s][k], raw), C);
        }
        mid_put(xch[s], x[s], wave, gr, c);
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < V; ++s) mid_get(xch[s], x[s], wave, gr, c);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int s = 0; s < V; ++s) {
            const Sums sum = digit_sums<KEEP>(M[k], x[s][k], ti);
            x[s][k] = KIND == INVERSE ? fold4_tight(sum, C) : fold4_w(sum, tt[s][k], C);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t o[V];
#pragma unroll
            for (int s = 0; s < V; ++s) o[s] = KIND == INVERSE && !CRT ? out_word<SMALL>(x[s][k][i], C) : (uint32_t)x[s][k][i];
            const uint32_t u1 = (uint32_t)(4 * gr + i);
            const uint32_t lo = KIND == TRANSFORM ? (u1 / S) * (16 * S * Q) + (u1 % S) * Q + V * (uint32_t)c : lw,
                           at = KIND == TRANSFORM ? S * Q * (4 * wave + k) + 16 * V * bx : at_word(k, i);
            if constexpr (CRT) {
                const auto bh = wave_buf(crt.h, N * 8);
                v2u r[V];
#pragma unroll
                for (int s = 0; s < V; ++s) r[s] = combined<SMALL>(x[s][k][i], a1[k][i][s], crt, C);
                if constexpr (V == 2) st_out4(bh, v4u{r[0][0], r[0][1], r[1][0], r[1][1]}, (lo + at) * 2);
                else __builtin_amdgcn_raw_buffer_store_b64(r[0], bh, lo * 8, at * 8, 0);
            } else if constexpr (V == 2)
                __builtin_amdgcn_raw_buffer_store_b64(v2u{o[0], o[1]}, bd, lo * 4, at * 4, 0);
            else st_out<true>(bd, o[0], lo, at);
        }
    }
}

// Block of a column kernel's workgroup: for V = 1 neighbours share every cache line.
template <int V>
__device__ __forceinline__ uint32_t col_id() {
    return V == 2 ? blockIdx.x : pair_blocks(blockIdx.x, gridDim.x);
}

template <int n, int V>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5 - V, 5 - V))) void k_ntt_cols(const uint32_t* f,
                                                                                                    uint32_t* Y, I8Plan p) {
    constexpr uint32_t N = 1u << n, CB = N / 4096 / V;
    __shared__ v4i xch[V][1024];
    const uint32_t id = col_id<V>();
    const uint64_t at = (uint64_t)(id / CB) * N;
    cols_block<n, TRANSFORM, false, V>(f + at, Y + at, id % CB, p, xch);
}

// Rows: 4096 outputs, a chunk's for one j.
template <int n, bool SMALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_ntt_rows(const uint32_t* Y,
                                                                                            uint32_t* h, I8Plan p) {
    using G = TransG<n>;
    using T = TransTab<n>;
    constexpr uint32_t N = G::N, Q = G::Q, S = G::S, R = G::R, CH = N / 4096, B = G::B;
    __shared__ v4i xch[1024];
    const int lane = threadIdx.x & 63, gr = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the R workgroups of a chunk on one die, one after the other, and neighbouring
    // chunks too
    const uint32_t id = blockIdx.x, j = (id / 8) % R, pq = pair_blocks(id / (8 * R) * 8 + id % 8, gridDim.x / R),
                   item = pq / (CH / R), q = pq % (CH / R);
    const auto by = wave_buf(Y + (uint64_t)pq * 4096 * R, 4096 * R * 4), bh = wave_buf(h + (uint64_t)item * N, N * 4);
    const v4i* t = (const v4i*)p.tab;
    const v4i* tj = t + T::J + j * T::SIZE;
    v4i x[4][R];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < (int)R; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                x[k][r][i] = (int)__builtin_amdgcn_raw_buffer_load_b32(
                    by, (uint32_t)(c + 64 * gr) * 4, (S * Q * (4 * wave + k) + 256 * r + 16 * i) * 4, 0);
    const I8K C(p.C);
    const Mat A2 = ld_mat(t + T::A2, lane);
    const Tw T1 = ld_tw(tj + R * 192, lane);
    const Init ti = init_tight(C);
    Sums s[4];
#pragma unroll
    for (int r = 0; r < (int)R; ++r) {
        const Mat A1 = ld_mat(tj + r * 192, lane);
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k] = digit_sums<TURN>(A1, x[k][r], r ? Init{s[k].s0, s[k].s1, s[k].s2} : ti);
    }
    v4i o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if constexpr (R > 1) {   // (s_0 of R sums is too large for the 24-bit products)
            v4i v = fold4_tight(s[k], C);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = reduce_i(v[i], C);
            o[k] = mul4_tw(v, T1, C);
        } else
            o[k] = fold4_tw(s[k], T1, C);
        o[k] = fold4_tight(digit_sums<KEEP>(A2, o[k], ti), C);
#pragma unroll
        for (int i = 0; i < 4; ++i) o[k][i] = (int)out_word<SMALL>(o[k][i], C);
    }
    // element (g, i), column (s, U): row 4 wave + k + 16 s, output u1 = j + R (U + B (4 g + i))
    mid_put(xch, o, wave, gr, c);
    __syncthreads();
    mid_get(xch, o, wave, gr, c);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t u1 = j + R * ((uint32_t)c % B + B * (uint32_t)(4 * wave + k));
        st_out4(bh, __builtin_bit_cast(v4u, o[k]), 4 * (uint32_t)gr + 16 * ((uint32_t)c / B) + 256 * u1 + 16 * S * q);
    }
}

}  // namespace nttmi
