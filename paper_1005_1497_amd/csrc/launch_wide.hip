// Launcher of the one-workgroup matrix-core convolutions (32-bit words, 2^13 and 2^14).
#include "wide.hpp"

namespace nttmi {

hipError_t launch_conv_wide(int logn, const void* f, const void* g, void* h, const uint64_t* offs, uint32_t count,
                            uint32_t cus, const I8Plan& p, hipStream_t st, const Quotient* div,
                            const Combine* crt) {
    if (count == 0) return hipSuccess;
    // 2^14: one workgroup takes a CU (160 KB of LDS) and loads ahead of its next
    // item; 2^13: three share one, and the hardware hands out the next
    const uint32_t grid = logn == 14 && cus && cus < count ? cus : count;
    const uint32_t *ff = (const uint32_t*)f, *gg = (const uint32_t*)g;
    // the last step's sums over R transforms: |r| <= 0.502 m + R 2^20 has to stay below m
    const int mode = p.C.small ? 2 : p.C.m < (2200000u << (logn - 12));
    if (crt) {
        if (offs || logn != 13 || mode) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_crt_wide, dim3(grid), dim3(256), 0, st, ff, gg, count, p, *crt);
        return hipGetLastError();
    }
    switch (logn * 8 + (div ? 4 : 0) + mode) {
#define CASE(n, mode)                                                                                                  \
    case n * 8 + mode:                                                                                                 \
        hipLaunchKernelGGL((k_conv_wide<n, mode>), dim3(grid), dim3(64 * WideG<n>::WAVES), 0, st, ff, gg,              \
                           (uint32_t*)h, offs, count, p);                                                              \
        return hipGetLastError();                                                                                      \
    case n * 8 + 4 + mode:                                                                                             \
        hipLaunchKernelGGL((k_div_wide<n, mode>), dim3(grid), dim3(64 * WideG<n>::WAVES), 0, st, ff, gg,               \
                           (uint32_t*)h, offs, count, p, *div);                                                        \
        return hipGetLastError();
        CASE(13, 0) CASE(13, 1) CASE(13, 2) CASE(14, 0) CASE(14, 1) CASE(14, 2)
#undef CASE
        default:
            return hipErrorInvalidValue;
    }
}

}  // namespace nttmi
