// Launcher of the three-launch matrix-core convolutions (32-bit words, 2^13 .. 2^19).
#include <algorithm>

#include "four.hpp"

namespace nttmi {

template <int n, bool SMALL>
static void four_t(const uint32_t* f, const uint32_t* g, uint32_t* h, const uint64_t* offs, uint32_t count, uint32_t group,
                   uint32_t* Y, const I8Plan* trans, const I8Plan& rows, hipStream_t st, const Quotient* div,
                   const Combine* crt) {
    constexpr uint32_t N = 1u << n, CH = N / 4096;
    for (uint32_t i = 0; i < count; i += group) {
        const uint32_t k = std::min(group, count - i);
        const uint64_t at = offs ? 0 : (uint64_t)i * N;
        const uint64_t* o = offs ? offs + i : nullptr;
        const uint32_t blocks = k * CH, wg = 256;
        if (wide_cols(2 * blocks)) hipLaunchKernelGGL((k_four_cols<n, 2>), dim3(blocks), dim3(wg), 0, st, f + at, g + at, o, Y, trans[0]);
        else hipLaunchKernelGGL((k_four_cols<n, 1>), dim3(2 * blocks), dim3(wg), 0, st, f + at, g + at, o, Y, trans[0]);
        // two passes per workgroup where every CU has its three all the same
        const int rounds = n <= 16 && k * CH >= 768 * 2 ? 2 : 1;
        const dim3 grid(k * CH / rounds);
        if (div) hipLaunchKernelGGL((k_four_div<n, SMALL>), grid, dim3(256), 0, st, Y, rounds, rows, *div);
        else hipLaunchKernelGGL((k_four_rows<n, SMALL>), grid, dim3(256), 0, st, Y, rounds, rows);
        if (crt) {
            Combine o = *crt;
            o.a1 += at;
            o.h += at;
            if (wide_cols(blocks)) hipLaunchKernelGGL((k_four_crt<n, 2>), dim3(blocks / 2), dim3(wg), 0, st, Y, o, trans[1]);
            else hipLaunchKernelGGL((k_four_crt<n, 1>), dim3(blocks), dim3(wg), 0, st, Y, o, trans[1]);
        } else if (wide_cols(blocks)) hipLaunchKernelGGL((k_four_inv<n, SMALL, 2>), dim3(blocks / 2), dim3(wg), 0, st, Y, h + at, o, trans[1]);
        else hipLaunchKernelGGL((k_four_inv<n, SMALL, 1>), dim3(blocks), dim3(wg), 0, st, Y, h + at, o, trans[1]);
    }
}

hipError_t launch_conv_four(int logn, const void* f, const void* g, void* h, const uint64_t* offs, uint32_t count, uint32_t group,
                            void* scratch, const I8Plan* trans, const I8Plan& rows, hipStream_t st,
                            const Quotient* div, const Combine* crt) {
    if (count == 0) return hipSuccess;
    if (group == 0 || (crt && (offs || rows.C.small))) return hipErrorInvalidValue;
    switch (logn) {
#define CASE(n)                                                                                                     \
    case n:                                                                                                         \
        if (rows.C.small)                                                                                           \
            four_t<n, true>((const uint32_t*)f, (const uint32_t*)g, (uint32_t*)h, offs, count, group,                    \
                            (uint32_t*)scratch, trans, rows, st, div, crt);                                                   \
        else                                                                                                        \
            four_t<n, false>((const uint32_t*)f, (const uint32_t*)g, (uint32_t*)h, offs, count, group,                   \
                             (uint32_t*)scratch, trans, rows, st, div, crt);                                                  \
        return hipGetLastError();
        CASE(13) CASE(14) CASE(15) CASE(16) CASE(17) CASE(18) CASE(19)
#undef CASE
        default:
            return hipErrorInvalidValue;
    }
}

}  // namespace nttmi
