// Adaptive-layer kernels: forward with saved activations, backward, n = 2^4 .. 2^14; n = 2^15 and 2^16 in one kernel forward and with
// the signals in memory backward; batch sums of the backward pass above 2^14.
#include "launch.hpp"
#include "layer_kernels.hpp"
namespace spinner {
// 16 values per thread up to n = 2^12, 32 above: the backward kernel keeps three running sums per
// value in registers beside the signal itself
constexpr int layer_rmax(int nt) { return nt <= 5 ? 2 : (nt <= 9 ? 3 : (nt <= 12 ? 4 : 5)); }
template <int NT>
using LayerGeom = TileGeom<NT, layer_rmax(NT), 4>;

// dd[i] = factor * sum over the rows of partial[row][i], summed in fp64 in a fixed order.  A block owns one 128-byte line of
// columns; its row lanes walk the rows and are then added up through LDS.  Bound by the latency of a row lane's loads one behind
// the other, so a block takes 1024 threads unless there are few rows (whole backward pass with 256 / 1024 threads, in us:
// n = 2048, batch 500 14.9 / 13.3, n = 2^14, 500 91 / 81, 20 17.0 / 17.9).
template <typename T, int THREADS>
__global__ void __launch_bounds__(THREADS) layer_reduce_kernel(const T* __restrict__ partial, long long rows, long long len,
                                                            double factor, float* __restrict__ dd)
{
    constexpr int COLS = 128 / sizeof(T), LANES = THREADS / COLS;
    __shared__ double sh[LANES][COLS + 1];
    const int tx = threadIdx.x % COLS, ty = threadIdx.x / COLS;
    const long long i = (long long)blockIdx.x * COLS + tx;
    double s = 0.0;
    if (i < len) {
        long long k = ty;
        for (; k + 3 * LANES < rows; k += 4 * LANES) {        // four independent loads in flight per thread
            const T a0 = partial[k * len + i], a1 = partial[(k + LANES) * len + i];
            const T a2 = partial[(k + 2 * LANES) * len + i], a3 = partial[(k + 3 * LANES) * len + i];
            s += ((double)a0 + (double)a1) + ((double)a2 + (double)a3);
        }
        for (; k < rows; k += LANES) s += (double)partial[k * len + i];
    }
    sh[ty][tx] = s;
    __syncthreads();
    if (ty < 8) {
#pragma unroll
        for (int r = 8; r < LANES; r += 8) s += sh[ty + r][tx];
        sh[ty][tx] = s;
    }
    __syncthreads();
    if (ty == 0 && i < len) {
#pragma unroll
        for (int r = 1; r < 8; ++r) s += sh[r][tx];
        dd[i] = (float)(factor * s);
    }
}

template <typename T>
static hipError_t launch_reduce(const T* partial, long long rows, long long len, double factor, float* dd, hipStream_t s)
{
    const long long cols = 128 / sizeof(T), blocks = (len + cols - 1) / cols;
    if (rows > 32) hipLaunchKernelGGL((layer_reduce_kernel<T, 1024>), dim3((unsigned)blocks), dim3(1024), 0, s, partial, rows, len, factor, dd);
    else hipLaunchKernelGGL((layer_reduce_kernel<T, 256>), dim3((unsigned)blocks), dim3(256), 0, s, partial, rows, len, factor, dd);
    return hipGetLastError();
}

// Above the fused range the backward pass materialises the signal that arrives at each diagonal; the gradient of
// that diagonal is then a sum over the batch of (signal x activation), per coordinate.  Block (bx, by) owns four
// coordinates per thread and the vectors by, by + S, by + 2S, ... (S = gridDim.y) and writes row `by` of `partial`
// (fp64 sums, rounded once); layer_reduce_kernel adds the S rows in fp64 in a fixed order.  With d1 != null the same
// sweep also writes dx = factor d1 .* g (the last step of the backward pass).
__global__ void __launch_bounds__(256) layer_large_dd_kernel(const float* __restrict__ g, const float* __restrict__ a, long long n,
                                                             long long batch, float* __restrict__ partial,
                                                             const float* __restrict__ d1, float* __restrict__ dx, float factor)
{
    const long long i = ((long long)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= n) return;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    float4 dv = make_float4(0.f, 0.f, 0.f, 0.f);
    if (d1) {
        dv = *reinterpret_cast<const float4*>(d1 + i);
        dv.x *= factor; dv.y *= factor; dv.z *= factor; dv.w *= factor;
    }
    for (long long b = blockIdx.y; b < batch; b += gridDim.y) {
        const float4 gv = *reinterpret_cast<const float4*>(g + b * n + i);
        const float4 av = *reinterpret_cast<const float4*>(a + b * n + i);
        s0 += (double)gv.x * (double)av.x; s1 += (double)gv.y * (double)av.y;
        s2 += (double)gv.z * (double)av.z; s3 += (double)gv.w * (double)av.w;
        if (d1) *reinterpret_cast<float4*>(dx + b * n + i) = make_float4(dv.x * gv.x, dv.y * gv.y, dv.z * gv.z, dv.w * gv.w);
    }
    *reinterpret_cast<float4*>(partial + (long long)blockIdx.y * n + i) = make_float4((float)s0, (float)s1, (float)s2, (float)s3);
}

// rows of `partial` the large-n backward pass uses: enough blocks to fill the chip, never more than the batch
long long layer_large_slabs(int log2n, long long batch)
{
    const long long per_row = ((1LL << log2n) / 4 + 255) / 256;       // blocks along the coordinates
    long long slabs = (2048 + per_row - 1) / per_row;
    if (slabs > batch) slabs = batch;
    if (slabs > 1024) slabs = 1024;
    return slabs < 1 ? 1 : slabs;
}

hipError_t launch_layer_large_dd(const float* g, const float* a, int log2n, long long batch, float* partial, float* dd,
                                 const float* d1, float* dx, hipStream_t s, double factor)
{
    const long long n = 1LL << log2n;
    const long long per_row = (n / 4 + 255) / 256;
    const long long slabs = layer_large_slabs(log2n, batch);
    if (per_row > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(layer_large_dd_kernel, dim3((unsigned)per_row, (unsigned)slabs), dim3(256), 0, s, g, a, n, batch, partial, d1, dx, (float)factor);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_reduce(partial, slabs, n, factor, dd, s);
}

// The backward pass of a large batch bypasses cache retention (non-temporal hint on dy, x, the saved activations and dx);
// what a training step of a smaller one moves (nine tensors of batch * n floats) is partly still in the 256 MB memory-side
// cache when the next call reads it.  Backward pass inside a step without / with the hint, in us: n = 2^12, batch 65536 1064 ->
// 960, 16384 295 -> 250, n = 2^10, batch 65536 308 -> 267; whole step at 2^24 elements 137 -> 117, at 2^23 64 -> 76.  The
// forward pass, which writes three tensors for the one it reads, loses with it (782 -> 852, batch 16384 191 -> 202).
constexpr int kLayerBackwardStreamLog = 24;
static bool layer_streams(int log2n, long long batch) { return (batch << log2n) >= (1LL << kLayerBackwardStreamLog); }

template <int NT>
static hipError_t forward_nt(const LayerForwardParams& p, hipStream_t s)
{
    using G = LayerGeom<NT>;
    const long long blocks = (p.batch + G::TILES_PER_WG - 1) / G::TILES_PER_WG;
    if (blocks <= 0) return hipSuccess;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((layer_forward_kernel<G>), dim3((unsigned)blocks), dim3(G::THREADS), 0, s, p);
    return hipGetLastError();
}

// Rows of 3 n floats that the workspace holds; where a tile spans several waves, also the tiles that the backward kernel runs.
template <int NT>
static long long slots_nt(long long batch)
{
    using G = LayerGeom<NT>;
    // four workgroups for each of the 256 compute units (as many as the kernel's registers let a compute unit hold
    // where it is compiled for a given number of waves per SIMD), fewer when the batch is small
    // (32 values per thread: two waves per SIMD, 512 workgroups are resident)
    long long wgs = (G::R == 16 && G::WB > 0) ? 256 * 4 * kLayerBackwardWaves / G::WAVES : (G::R == 32 ? 512 : 1024);
    const long long need = (batch + G::TILES_PER_WG - 1) / G::TILES_PER_WG;
    if (wgs > need) wgs = need;
    // small vectors put many tiles into one workgroup: keep the number of partial rows bounded
    if (wgs * G::TILES_PER_WG > 8192) wgs = 8192 / G::TILES_PER_WG;
    return wgs * G::TILES_PER_WG;
}

// Workgroups of the backward kernel.  Where a workgroup holds several tiles it adds them up itself and leaves one row of doubles,
// which the workspace (sized for a row of floats per tile and at most 8192 of them) holds for 2048 workgroups and more.  Against
// a row of floats per tile, which let n = 16 have 128 workgroups and n = 256 write 8192 rows, in us: n = 16, batch 20000 50 -> 7,
// 337332 143 -> 27; n = 64, 65536 vectors 66 -> 20; n = 256, 1024 vectors 12.4 -> 7.4, 52357 101 -> 57; n = 512, 8000 45 -> 22; n = 1024,
// 16384 96 -> 74.  768 / 1024 / 1280 / 1536 workgroups: n = 16, batch 10^6 80 / 69 / 65 / 63; n = 64, 500000 112 / 109 / 111 / 133; n = 256,
// 200000 182 / 173 / 174 / 220; n = 1024, 65536 257 / 242 / 298 / 273 (four waves per SIMD are what 126 registers leave there).
template <int NT>
static long long workgroups_nt(long long batch)
{
    using G = LayerGeom<NT>;
    if (G::WB > 0) return slots_nt<NT>(batch);
    const long long need = (batch + G::TILES_PER_WG - 1) / G::TILES_PER_WG, most = NT <= 5 ? 1536 : 1024;
    static_assert(G::WB > 0 || (G::TILES_PER_WG >= 4 && G::TILES_PER_WG <= 64), "a workgroup's doubles fit its tiles' floats");
    return need < most ? need : most;
}

template <int NT>
static hipError_t backward_nt(const LayerBackwardParams& p0, double factor, float* dd, hipStream_t s)
{
    using G = LayerGeom<NT>;
    LayerBackwardParams p = p0;
    const long long blocks = workgroups_nt<NT>(p.batch);
    p.slots = blocks * G::TILES_PER_WG;
    if (blocks <= 0) return hipSuccess;
    if (layer_streams(NT, p.batch)) hipLaunchKernelGGL((layer_backward_kernel<G, true>), dim3((unsigned)blocks), dim3(G::THREADS), 0, s, p);
    else hipLaunchKernelGGL((layer_backward_kernel<G, false>), dim3((unsigned)blocks), dim3(G::THREADS), 0, s, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if constexpr (G::WB > 0) return launch_reduce(p.partial, blocks, 3LL << NT, factor, dd, s);
    else return launch_reduce(reinterpret_cast<const double*>(p.partial), blocks, 3LL << NT, factor, dd, s);
}

#define CASES(F, ...) switch (log2n) { case 4: return F<4>(__VA_ARGS__); case 5: return F<5>(__VA_ARGS__); case 6: return F<6>(__VA_ARGS__); \
    case 7: return F<7>(__VA_ARGS__); case 8: return F<8>(__VA_ARGS__); case 9: return F<9>(__VA_ARGS__); case 10: return F<10>(__VA_ARGS__); \
    case 11: return F<11>(__VA_ARGS__); case 12: return F<12>(__VA_ARGS__); case 13: return F<13>(__VA_ARGS__); case 14: return F<14>(__VA_ARGS__); \
    default: break; }

// n = 2^15, 2^16 on the geometries of the fused plain kernels
template <typename G>
static hipError_t forward_wide(const LayerForwardParams& p, hipStream_t s)
{
    if (p.batch <= 0) return hipSuccess;
    if (p.batch > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((layer_forward_kernel<G, true>), dim3((unsigned)p.batch), dim3(G::THREADS), 0, s, p);
    return hipGetLastError();
}
// first = p0 H (da .* in) (da null: p0 H in), and with db second = p1 H (db .* first)
template <typename G>
static hipError_t signals_wide(const float* in, const float* da, const float* db, float* first, float* second, float p0, float p1, long long batch,
                               hipStream_t s)
{
    if (batch <= 0) return hipSuccess;
    if (batch > 0x7fffffffLL || (da && db)) return hipErrorInvalidConfiguration;
    if (da) hipLaunchKernelGGL((layer_signals_kernel<G, true, false>), dim3((unsigned)batch), dim3(G::THREADS), 0, s, in, da, db, first, second, p0, p1);
    else hipLaunchKernelGGL((layer_signals_kernel<G, false, true>), dim3((unsigned)batch), dim3(G::THREADS), 0, s, in, da, db, first, second, p0, p1);
    return hipGetLastError();
}
hipError_t launch_layer_signals(int log2n, const float* in, const float* da, const float* db, float* first, float* second, float p0, float p1,
                                long long batch, hipStream_t s)
{
    if (log2n == 15) return signals_wide<GeomFor<float, 15>>(in, da, db, first, second, p0, p1, batch, s);
    if (log2n == 16) return signals_wide<GeomFor<float, 16>>(in, da, db, first, second, p0, p1, batch, s);
    return hipErrorInvalidValue;
}

hipError_t launch_layer_forward(int log2n, const LayerForwardParams& p, hipStream_t s)
{
    if (log2n == 15) return forward_wide<GeomFor<float, 15>>(p, s);
    if (log2n == 16) return forward_wide<GeomFor<float, 16>>(p, s);
    CASES(forward_nt, p, s)
    return hipErrorInvalidValue;
}
long long layer_backward_slots(int log2n, long long batch)
{
    CASES(slots_nt, batch)
    return 0;
}
hipError_t launch_layer_backward(int log2n, const LayerBackwardParams& p, double factor, float* dd, hipStream_t s)
{
    CASES(backward_nt, p, factor, dd, s)
    return hipErrorInvalidValue;
}
#undef CASES
}  // namespace spinner
