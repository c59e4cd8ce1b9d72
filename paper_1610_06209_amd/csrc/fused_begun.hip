// Fused three-round kernels, first-m-rows epilogue, fp32 diagonals, for vectors that arrive with the first diagonal and the first
// transform's low kColumnBits stages behind them (the sketch's transposition does both on the way; sizes: sketch_begun_pays).
#include "launch.hpp"
namespace spinner {
template <int NT, int PRUNE>
static hipError_t launch_begun(const TileParams& p, long long tiles, hipStream_t s)
{
    return launch_tile<float, NT, NT, 3, false, EPI_STORE_NONE, false, PRUNE, true, void, kColumnBits>(p, tiles, s);
}
hipError_t launch_fused_begun(int log2n, int prune, const TileParams& p, long long tiles, hipStream_t s)
{
    if (prune >= kPruneBits) {
        switch (log2n) {
        case 11: return launch_begun<11, kPruneBits>(p, tiles, s);
        case 13: return launch_begun<13, kPruneBits>(p, tiles, s);
        case 14: return launch_begun<14, kPruneBits>(p, tiles, s);
        case 15: return launch_begun<15, kPruneBits>(p, tiles, s);
        case 16: return launch_begun<16, kPruneBits>(p, tiles, s);
        default: return hipErrorInvalidValue;
        }
    }
    switch (log2n) {
    case 11: return launch_begun<11, 0>(p, tiles, s);
    case 15: return launch_begun<15, 0>(p, tiles, s);
    case 16: return launch_begun<16, 0>(p, tiles, s);
    default: return hipErrorInvalidValue;
    }
}
}  // namespace spinner
