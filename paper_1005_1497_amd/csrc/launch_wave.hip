// Launchers of the matrix-core convolutions and transforms of 32-bit words, lengths 2^5 .. 2^12.
#include <algorithm>

#include "i8plan.hpp"
#include "wave.hpp"

namespace nttmi {

// Passes of a workgroup up to 2^8: one, or up to TINY_ROUNDS where every CU has
// its three workgroups all the same (convolutions, 2^26 elements of 2^8: 172 us
// with 4 passes, against 181 with a fixed share per resident wave; 2^18: 5.6 us
// with one, 13.8 with four).
static int tiny_rounds(uint64_t words, uint32_t cus) {
    const uint64_t fill = 3ull * (cus ? cus : 1) * 4 * 256 * TINY_BLOCKS;
    return (int)std::min<uint64_t>(std::max<uint64_t>(words / fill, 1), TINY_ROUNDS);
}

hipError_t launch_conv_wave(int logn, const void* f, const void* g, void* h, uint32_t count, const I8Plan& p,
                            uint32_t cus, hipStream_t st, const Quotient* div, const Combine* crt) {
    if (count == 0) return hipSuccess;
    const uint64_t words = (uint64_t)count << logn;
    const uint32_t *ff = (const uint32_t*)f, *gg = (const uint32_t*)g;
    uint32_t* hh = (uint32_t*)h;
    const int rounds = tiny_rounds(words, cus);   // above 2^8: a workgroup per chunk
    const uint64_t share = 4ull * rounds * 256 * TINY_BLOCKS;
    const dim3 tiny((uint32_t)((words + share - 1) / share)), mid((uint32_t)((words + 4095) / 4096)), wg(256);
    if (crt) {
        if (p.C.small || div) return hipErrorInvalidValue;
        switch (logn) {
#define TINY(n)                                                                                             \
    case n:                                                                                                 \
        hipLaunchKernelGGL((k_crt_tiny<n>), tiny, wg, 0, st, ff, gg, words, rounds, p, *crt);               \
        break;
#define MID(n)                                                                                              \
    case n:                                                                                                 \
        hipLaunchKernelGGL((k_crt_mid<n>), mid, wg, 0, st, ff, gg, words, p, *crt);                         \
        break;
            TINY(5) TINY(6) TINY(7) TINY(8) MID(9) MID(10) MID(11) MID(12)
#undef TINY
#undef MID
            default:
                return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    switch (logn * 4 + (div ? 2 : 0) + (p.C.small ? 1 : 0)) {
#define TINY(n, s)                                                                                          \
    case n * 4 + s:                                                                                         \
        hipLaunchKernelGGL((k_conv_tiny<n, s>), tiny, wg, 0, st, ff, gg, hh, words, rounds, p);             \
        break;                                                                                              \
    case n * 4 + 2 + s:                                                                                     \
        hipLaunchKernelGGL((k_div_tiny<n, s>), tiny, wg, 0, st, ff, gg, hh, words, rounds, p, *div);        \
        break;
#define MID(n, s)                                                                                           \
    case n * 4 + s:                                                                                         \
        hipLaunchKernelGGL((k_conv_mid<n, s>), mid, wg, 0, st, ff, gg, hh, words, p);                       \
        break;                                                                                              \
    case n * 4 + 2 + s:                                                                                     \
        hipLaunchKernelGGL((k_div_mid<n, s>), mid, wg, 0, st, ff, gg, hh, words, p, *div);                  \
        break;
#define BOTH(K, n) K(n, 0) K(n, 1)
        BOTH(TINY, 5) BOTH(TINY, 6) BOTH(TINY, 7) BOTH(TINY, 8) BOTH(MID, 9) BOTH(MID, 10) BOTH(MID, 11) BOTH(MID, 12)
#undef BOTH
#undef TINY
#undef MID
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_ntt_wave(int logn, bool inv, const void* x, void* X, uint32_t batch, const I8Plan& pl, hipStream_t st) {
    if (batch == 0) return hipSuccess;
    const uint64_t words = (uint64_t)batch << logn;
    const uint32_t* xx = (const uint32_t*)x;
    uint32_t* hh = (uint32_t*)X;
    I8Plan p = pl;
    if (!inv) p.tab = pl.fwd;
    p.C = make_i8c(p.C.m, 16);   // (the correction for raw words: a first step of radix 16)
    const dim3 chunks((uint32_t)((words + 4095) / 4096)), wg(256);   // of 4096 elements
    switch (logn * 2 + (p.C.small ? 1 : 0)) {
#define TINY(n, s)                                                                                             \
    case n * 2 + s:                                                                                            \
        hipLaunchKernelGGL((k_ntt_tiny<n, s>), chunks, wg, 0, st, xx, hh, words, p);                           \
        break;
#define MID(n, s)                                                                                              \
    case n * 2 + s:                                                                                            \
        hipLaunchKernelGGL((k_ntt_mid<n, s>), chunks, wg, 0, st, xx, hh, words, p);                            \
        break;
#define BOTH(K, n) K(n, 0) K(n, 1)
        BOTH(TINY, 5) BOTH(TINY, 6) BOTH(TINY, 7) BOTH(TINY, 8) BOTH(MID, 9) BOTH(MID, 10) BOTH(MID, 11) BOTH(MID, 12)
#undef BOTH
#undef TINY
#undef MID
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace nttmi
