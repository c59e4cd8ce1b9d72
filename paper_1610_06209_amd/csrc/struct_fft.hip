// Dispatch of the one-kernel G_struct members (struct_fft_kernels.hpp) and their kernels up to n = 2^12.
#include "struct_fft_kernels.hpp"
namespace spinner {
#define CASE(NT) case NT: return log2p > NT ? launch_struct_fft_nt<NT, true>(p, s) : launch_struct_fft_nt<NT, false>(p, s);
hipError_t launch_struct_fft(const float* x, const float* d1, const float* d2, const float2* spec, const float2* tw, float* out,
                             long long batch, int log2n, int log2p, int m, int reverse, float factor, hipStream_t s)
{
    if (batch <= 0) return hipSuccess;
    const StructFftParams p{x, d1, d2, spec, tw, out, batch, m, reverse, factor};
    switch (log2n) {
        CASE(9) CASE(10) CASE(11) CASE(12)
    case 13: return launch_struct_fft_13(log2p > 13, p, s);
    case 14: return launch_struct_fft_14(log2p > 14, p, s);
    default: return hipErrorInvalidValue;
    }
}
#undef CASE
}  // namespace spinner
