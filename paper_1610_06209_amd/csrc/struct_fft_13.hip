// One-kernel G_struct members of n = 2^13 (struct_fft_kernels.hpp).
#include "struct_fft_kernels.hpp"
namespace spinner {
hipError_t launch_struct_fft_13(bool padded, const StructFftParams& p, hipStream_t s)
{
    if (padded && p.batch <= 32) return launch_struct_fft_nt<13, true, true>(p, s);
    return padded ? launch_struct_fft_nt<13, true>(p, s) : launch_struct_fft_nt<13, false>(p, s);
}
}  // namespace spinner
