// One-kernel G_struct members of n = 2^14 (struct_fft_kernels.hpp).
#include "struct_fft_kernels.hpp"
namespace spinner {
hipError_t launch_struct_fft_14(bool padded, const StructFftParams& p, hipStream_t s)
{
    return padded ? launch_struct_fft_nt<14, true>(p, s) : launch_struct_fft_nt<14, false>(p, s);
}
}  // namespace spinner
