// Launcher of the three-launch matrix-core convolutions (32-bit words, 2^13 .. 2^19).
#include <algorithm>

#include "four.hpp"

namespace nttmi {

// (2^13 comes as single convolutions alone, and 2^14 without the combining store by fewer
// items than 32 columns to a workgroup ask for: what these never take is not there.)
template <int n, bool SMALL>
static void four_t(const uint32_t* f, const uint32_t* g, uint32_t* h, const uint64_t* offs, uint32_t count, uint32_t group,
                   uint32_t* Y, uint32_t cus, const I8Plan* trans, const I8Plan& rows, hipStream_t st,
                   const Quotient* div, const Combine* crt) {
    constexpr uint32_t N = 1u << n, CH = N / 4096;
    const dim3 wg(256);
    for (uint32_t i = 0; i < count; i += group) {
        const uint32_t k = std::min(group, count - i);
        const uint64_t at = offs ? 0 : (uint64_t)i * N;
        const uint64_t* o = offs ? offs + i : nullptr;
        const uint32_t blocks = k * CH;
        if (n >= 14 && two_each(2 * blocks, cus)) {
            if constexpr (n >= 14)
                hipLaunchKernelGGL((k_four_cols<n, 2>), dim3(blocks), wg, 0, st, f + at, g + at, o, Y, trans[0]);
        } else
            hipLaunchKernelGGL((k_four_cols<n, 1>), dim3(2 * blocks), wg, 0, st, f + at, g + at, o, Y, trans[0]);
        // two passes per workgroup where every CU has its three all the same
        const int rounds = n <= 16 && two_each(blocks, cus) ? 2 : 1;
        const dim3 grid(blocks / rounds);
        if (n >= 14 && div) {
            if constexpr (n >= 14) hipLaunchKernelGGL((k_four_div<n, SMALL>), grid, wg, 0, st, Y, rounds, rows, *div);
        } else
            hipLaunchKernelGGL((k_four_rows<n, SMALL>), grid, wg, 0, st, Y, rounds, rows);
        if (n >= 14 && crt) {
            if constexpr (n >= 14) {
                Combine c = *crt;
                c.a1 += at;
                c.h += at;
                if (two_each(blocks, cus))
                    hipLaunchKernelGGL((k_four_crt<n, 2>), dim3(blocks / 2), wg, 0, st, Y, c, trans[1]);
                else
                    hipLaunchKernelGGL((k_four_crt<n, 1>), dim3(blocks), wg, 0, st, Y, c, trans[1]);
            }
        } else if (n >= 15 && two_each(blocks, cus)) {
            if constexpr (n >= 15)
                hipLaunchKernelGGL((k_four_inv<n, SMALL, 2>), dim3(blocks / 2), wg, 0, st, Y, h + at, o, trans[1]);
        } else
            hipLaunchKernelGGL((k_four_inv<n, SMALL, 1>), dim3(blocks), wg, 0, st, Y, h + at, o, trans[1]);
    }
}

hipError_t launch_conv_four(int logn, const void* f, const void* g, void* h, const uint64_t* offs, uint32_t count, uint32_t group,
                            void* scratch, uint32_t cus, const I8Plan* trans, const I8Plan& rows, hipStream_t st,
                            const Quotient* div, const Combine* crt) {
    if (count == 0) return hipSuccess;
    if (group == 0 || (crt && (offs || rows.C.small)) || (logn == 13 && (div || crt))) return hipErrorInvalidValue;
    switch (logn) {
#define CASE(n)                                                                                                         \
    case n:                                                                                                             \
        if (rows.C.small)                                                                                               \
            four_t<n, true>((const uint32_t*)f, (const uint32_t*)g, (uint32_t*)h, offs, count, group, (uint32_t*)scratch,\
                            cus, trans, rows, st, div, crt);                                                            \
        else                                                                                                            \
            four_t<n, false>((const uint32_t*)f, (const uint32_t*)g, (uint32_t*)h, offs, count, group, (uint32_t*)scratch,\
                             cus, trans, rows, st, div, crt);                                                           \
        return hipGetLastError();
        CASE(13) CASE(14) CASE(15) CASE(16) CASE(17) CASE(18) CASE(19)
#undef CASE
        default:
            return hipErrorInvalidValue;
    }
}

}  // namespace nttmi
