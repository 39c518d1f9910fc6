// Launchers of the matrix-core convolutions of 32-bit words, lengths 2^5 .. 2^12.
#include <algorithm>

#include "wave.hpp"

namespace nttmi {

hipError_t launch_conv_wave(int logn, const void* f, const void* g, void* h, uint32_t count, const I8Plan& p,
                            uint32_t cus, hipStream_t st) {
    if (count == 0) return hipSuccess;
    const uint64_t words = (uint64_t)count << logn;
    const uint32_t *ff = (const uint32_t*)f, *gg = (const uint32_t*)g;
    uint32_t* hh = (uint32_t*)h;
    // up to 2^8: workgroups of 4 waves, each one pass, or up to TINY_ROUNDS where
    // every CU has its three workgroups all the same (2^26 elements of 2^8: 172
    // us with 4 passes, against 181 with a fixed share per resident wave; 2^18:
    // 5.6 us with one, 13.8 with four); above: a workgroup per chunk
    const uint64_t fill = 3ull * (cus ? cus : 1) * 4 * 256 * TINY_BLOCKS;
    const int rounds = (int)std::min<uint64_t>(std::max<uint64_t>(words / fill, 1), TINY_ROUNDS);
    const uint64_t share = 4ull * rounds * 256 * TINY_BLOCKS;
    const dim3 tiny((uint32_t)((words + share - 1) / share)), mid((uint32_t)((words + 4095) / 4096)), wg(256);
    switch (logn) {
#define TINY(n)                                                                                                    \
    case n:                                                                                                        \
        if (p.C.small) hipLaunchKernelGGL((k_conv_tiny<n, true>), tiny, wg, 0, st, ff, gg, hh, words, rounds, p);  \
        else hipLaunchKernelGGL((k_conv_tiny<n, false>), tiny, wg, 0, st, ff, gg, hh, words, rounds, p);           \
        break;
#define MID(n)                                                                                                     \
    case n:                                                                                                        \
        if (p.C.small) hipLaunchKernelGGL((k_conv_mid<n, true>), mid, wg, 0, st, ff, gg, hh, words, p);            \
        else hipLaunchKernelGGL((k_conv_mid<n, false>), mid, wg, 0, st, ff, gg, hh, words, p);                     \
        break;
        TINY(5) TINY(6) TINY(7) TINY(8) MID(9) MID(10) MID(11) MID(12)
#undef TINY
#undef MID
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace nttmi
