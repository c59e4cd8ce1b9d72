// Parameter blocks of the adaptive-layer kernels (see layer_kernels.hpp).
#pragma once

namespace spinner {

// n = 2^15, 2^16: values are brought back by 2^-8, the next whole power at n^-1/2 or below, after a transform
constexpr int wide_shrink_log(int log2n) { return (log2n + 1) / 2; }

struct LayerForwardParams {
    const float* x;
    const float* d[3];
    float* y;
    float* saved1;
    float* saved2;
    long long batch;
    float factor;            // scale * n^{-3/2}; 2^15, 2^16: times 2^(2 wide_shrink_log), what the values were shrunk by
    float norm;              // n^{-1/2}
    float norm2;             // 2^15, 2^16: 2^wide_shrink_log / n; an argument because the compiler joins a constant with the shrinking
                             // of the values and then spills 182 registers (2^16, batch 1024 239 -> 435 us)
};

struct LayerBackwardParams {
    const float* dy;
    const float* x;
    const float* saved1;
    const float* saved2;
    const float* d[3];
    float* dx;
    float* partial;          // sums over the vectors of a slot or of a workgroup (unscaled): floats [slots][3][n] where a tile
                             // spans several waves, else doubles [workgroups][3][n]
    long long batch;
    long long slots;         // number of (workgroup, tile slot) pairs = stride between the vectors of one slot
    float factor;            // scale * n^{-3/2}
};

}  // namespace spinner
