// Launcher of the matrix-core transforms of 32-bit words, lengths 2^13 .. 2^19.
#include "trans.hpp"

namespace nttmi {

hipError_t launch_ntt_trans(int logn, const void* x, void* X, uint32_t rows, void* scratch, uint32_t cus,
                            const I8Plan& p, hipStream_t st) {
    if (rows == 0) return hipSuccess;
    const uint32_t blocks = rows << (logn - 12);   // of 4096 outputs
    switch (logn) {
#define CASE(n)                                                                                                      \
    case n:                                                                                                          \
        if (two_each(blocks, cus))                                                                                   \
            hipLaunchKernelGGL((k_ntt_cols<n, 2>), dim3(blocks / 2), dim3(256), 0, st, (const uint32_t*)x,           \
                               (uint32_t*)scratch, p);                                                               \
        else                                                                                                         \
            hipLaunchKernelGGL((k_ntt_cols<n, 1>), dim3(blocks), dim3(256), 0, st, (const uint32_t*)x,               \
                               (uint32_t*)scratch, p);                                                               \
        if (p.C.small)                                                                                               \
            hipLaunchKernelGGL((k_ntt_rows<n, true>), dim3(blocks), dim3(256), 0, st, (const uint32_t*)scratch,      \
                               (uint32_t*)X, p);                                                                     \
        else                                                                                                         \
            hipLaunchKernelGGL((k_ntt_rows<n, false>), dim3(blocks), dim3(256), 0, st, (const uint32_t*)scratch,     \
                               (uint32_t*)X, p);                                                                     \
        return hipGetLastError();
        CASE(13) CASE(14) CASE(15) CASE(16) CASE(17) CASE(18) CASE(19)
#undef CASE
        default:
            return hipErrorInvalidValue;
    }
}

}  // namespace nttmi
