// Newton-sketch helpers: transposition with optional row weights (the sketch acts on the columns
// of a row-major data matrix) and the Gram matrix B^T B on the fp32 matrix pipe.
#include <mutex>

#include "launch.hpp"
namespace spinner {

// dst[c][r] = src[r][c] * (row_scale ? row_scale[r] : 1), src is [rows][cols] row-major.
// 64 x 64 tiles through LDS (row padded by one word), both sides coalesced.  All sixteen loads of a thread are
// issued before the first is used: rows and columns past the end are clamped to the last one (and not stored), so
// that no load sits under a condition.
// Tiles are numbered along the columns and every XCD takes runs of eight (workgroups go to the eight XCDs in turn): a row
// whose length is no multiple of 32 floats shares a 128-byte line between neighbouring tiles, which one L2 then fetches once.
// Sketch with two transpositions, plain numbering -> runs of eight, in us: n = 2^16, d = 500 119.3 -> 110.7 (d = 512 112.1 ->
// 112.2), 2^15, d = 1000 101.5 -> 95.6, 2^13, d = 1999 67.9 -> 62.3; runs of four and of 32 alike.  Tiles of 128 rows: no gain.
constexpr int kTransposeXcdLog = 3;
template <bool SCALED>
__global__ void __launch_bounds__(256) transpose_scale_kernel(const float* __restrict__ src, long long rows, long long cols,
                                                              unsigned gx, const float* __restrict__ row_scale, float* __restrict__ dst)
{
    __shared__ float tile[64][65];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const unsigned tl = (unsigned)xcd_tile(blockIdx.x, gridDim.x, kTransposeXcdLog);
    const long long r0 = (long long)(tl / gx) * 64, c0 = (long long)(tl % gx) * 64;
    const long long cc = c0 + tx < cols ? c0 + tx : cols - 1;
    float v[16], w[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const long long r = r0 + ty + 4 * k;
        const long long rr = r < rows ? r : rows - 1;
        v[k] = src[rr * cols + cc];
        w[k] = SCALED ? row_scale[rr] : 1.0f;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) tile[ty + 4 * k][tx] = SCALED ? v[k] * w[k] : v[k];
    __syncthreads();
    const long long r = r0 + tx;
    if (r0 + 64 <= rows && c0 + 64 <= cols) {
#pragma unroll
        for (int k = 0; k < 16; ++k) dst[(c0 + ty + 4 * k) * rows + r] = tile[tx][ty + 4 * k];
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const long long c = c0 + ty + 4 * k;
            if (r < rows && c < cols) dst[c * rows + r] = tile[tx][ty + 4 * k];
        }
    }
}

hipError_t launch_transpose_scale(const float* src, long long rows, long long cols, const float* row_scale, float* dst,
                                  hipStream_t s)
{
    if (rows <= 0 || cols <= 0) return hipSuccess;
    const long long gx = (cols + 63) / 64, gy = (rows + 63) / 64;
    if (gx > 0xffffffLL || gy > 0xffffffLL || gx * gy > 0xffffffLL) return hipErrorInvalidConfiguration;      // 2^32 threads per grid
    const dim3 grid((unsigned)(gx * gy));
    if (row_scale) hipLaunchKernelGGL(transpose_scale_kernel<true>, grid, dim3(256), 0, s, src, rows, cols, (unsigned)gx, row_scale, dst);
    else hipLaunchKernelGGL(transpose_scale_kernel<false>, grid, dim3(256), 0, s, src, rows, cols, (unsigned)gx, row_scale, dst);
    return hipGetLastError();
}

// dst[c][r] = src[r][c] * (row_scale ? row_scale[r] : 1) * diag[r], with the transform over the low kColumnBits index bits of r
// done on the way (unnormalised).  rows: a multiple of 2^kColumnBits.
// A tile is 256 rows of 32 columns, 32 KiB of LDS.  On the way in lanes 0 .. 31 are the columns and a thread holds 32 rows: row bits
// 0, 1, 4, 6, 7 are transformed between its registers; the wave is row bits 2, 3 and the upper half of the lanes row bit 5.
// On the way out a lane is four rows, so those three are lane bits 0, 1, 3 and take one DPP instruction each; the factor that
// such stages leave on a lane (-1 to the number of the three that are set) is taken from the rows when they are scaled.
// A column of the tile is 64 pieces of 16 bytes, piece q in place q ^ column: both sides touch 64 different pieces of all banks.
// Bound: memory, as the transposition alone (46 us for 2 x 131 MB at n = 2^16, d = 500, where that takes 44): the arithmetic hides behind it,
// and the projection that follows has eight stages and a diagonal less (68 -> 62 us there).  With tiles of 64 columns, whose 64 KiB leave two
// of them on a compute unit, 51 us; with the non-temporal hint on the loads a line that two tiles share comes twice (131 for 126 us in all).
// Runs of 4 / 8 / 16 / 32 tiles per XCD, d = 500: 127.5 / 127.2 / 125.9 / 125.5 us in all, n = 2^13, d = 333: 27.0 / 27.0 / 26.3 / 26.8.
constexpr int kColumnRows = 1 << kColumnBits, kColumnTile = 32, kColumnXcdLog = 4;
static_assert(kColumnBits == 8, "rows of a tile: five bits in registers, two in the wave, one in the lanes");
template <bool SCALED>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
transpose_transform_kernel(const float* __restrict__ src, long long rows, long long cols, unsigned gx, const float* __restrict__ row_scale,
                           const float* __restrict__ diag, float* __restrict__ dst)
{
    __shared__ float4 tile[kColumnTile * 64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lc = lane & 31, up = lane >> 5;
    const unsigned tl = (unsigned)xcd_tile(blockIdx.x, gridDim.x, kColumnXcdLog);
    const long long r0 = (long long)(tl / gx) * kColumnRows, c0 = (long long)(tl % gx) * kColumnTile;
    const long long cc = c0 + lc < cols ? lc : cols - 1 - c0;      // columns past the last one read it and are not stored
    float v[32];
    // register 4 a + i: row 4 wave + 32 up + i + 16 (a & 1) + 64 (a >> 1)
    {
        const float* in = src + (r0 + 4 * wave) * cols + c0;
        const long long own = 32 * up * cols + cc;
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
            for (int i = 0; i < 4; ++i) v[4 * a + i] = in[(16 * (a & 1) + 64 * (a >> 1) + i) * cols + own];
        const unsigned sign = (unsigned)((__builtin_popcount(wave) + up) & 1) << 31;
        const float *w = row_scale + r0 + 4 * wave + 32 * up, *d = diag + r0 + 4 * wave + 32 * up;
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            const int r = 16 * (a & 1) + 64 * (a >> 1);
            if constexpr (SCALED) {
                const float4 t = *reinterpret_cast<const float4*>(w + r);
                v[4 * a] *= t.x; v[4 * a + 1] *= t.y; v[4 * a + 2] *= t.z; v[4 * a + 3] *= t.w;
            }
            const float4 t = *reinterpret_cast<const float4*>(d + r);
            v[4 * a] *= __uint_as_float(__float_as_uint(t.x) ^ sign); v[4 * a + 1] *= __uint_as_float(__float_as_uint(t.y) ^ sign);
            v[4 * a + 2] *= __uint_as_float(__float_as_uint(t.z) ^ sign); v[4 * a + 3] *= __uint_as_float(__float_as_uint(t.w) ^ sign);
        }
    }
    static_for<0, 5>([&](auto q) { reg_stage<q.value>(v); });
#pragma unroll
    for (int a = 0; a < 8; ++a)
        tile[lc * 64 + ((wave + 8 * up + 4 * (a & 1) + 16 * (a >> 1)) ^ lc)] = make_float4(v[4 * a], v[4 * a + 1], v[4 * a + 2], v[4 * a + 3]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int col = 8 * wave + k;
        const float4 t = tile[col * 64 + (lane ^ col)];
        v[4 * k] = t.x; v[4 * k + 1] = t.y; v[4 * k + 2] = t.z; v[4 * k + 3] = t.w;
    }
    lane_stage_fmac_dpp<0>(v, lane & 1 ? 1.0f : -1.0f);
    lane_stage_fmac_dpp<1>(v, lane & 2 ? 1.0f : -1.0f);
    lane_stage_fmac_dpp<3>(v, lane & 8 ? 1.0f : -1.0f);
    float* out = dst + (c0 + 8 * wave) * rows + r0;
    const int left = (int)(cols - c0 < kColumnTile ? cols - c0 : kColumnTile) - 8 * wave;
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (k < left) *reinterpret_cast<float4*>(out + k * rows + 4 * lane) = make_float4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
}

hipError_t launch_transpose_transform(const float* src, long long rows, long long cols, const float* row_scale, const float* diag,
                                      float* dst, hipStream_t s)
{
    if (rows <= 0 || cols <= 0) return hipSuccess;
    if (rows % kColumnRows) return hipErrorInvalidValue;
    const long long gx = (cols + kColumnTile - 1) / kColumnTile, gy = rows / kColumnRows;
    if (gx > 0xffffffLL || gy > 0xffffffLL || gx * gy > 0xffffffLL) return hipErrorInvalidConfiguration;      // 2^32 threads per grid
    const dim3 grid((unsigned)(gx * gy));
    if (row_scale) hipLaunchKernelGGL(transpose_transform_kernel<true>, grid, dim3(256), 0, s, src, rows, cols, (unsigned)gx, row_scale, diag, dst);
    else hipLaunchKernelGGL(transpose_transform_kernel<false>, grid, dim3(256), 0, s, src, rows, cols, (unsigned)gx, row_scale, diag, dst);
    return hipGetLastError();
}

// G = B^T B for B [m][d] row-major: G[a][b] = sum_k B[k][a] B[k][b], on the fp32 matrix pipe (v_mfma_f32_32x32x2_f32).
// G is symmetric, so only the 64 x 64 tiles on and above the diagonal are computed and each is stored twice.  A
// workgroup owns one tile (of one slab of rows); its four waves take a quarter of the rows each, hold the whole tile
// (2 x 2 MFMA tiles) and are added up through LDS at the end, in a fixed order.  Both operands are rows of B as they
// lie: lane l supplies row k + l / 32 of columns 2 (l % 32) and 2 (l % 32) + 1, one for either MFMA tile (EVEN: one 8-byte
// load, which an even d aligns; else two), so they come straight from memory into registers, a group of UNROLL row
// pairs ahead of the group being multiplied; no barrier stands in the loop.
// What bounds it: the matrix pipe at large d (busy 43 % of the time at d = 4096, the rest waits for loads that miss the
// L2), latency below.  Measured against all 128 x 128 tiles of G staged through LDS, m = 2048, in us: d = 64 13.9 -> 12.3,
// 256 17.4 -> 14.4, 500 26.5 -> 17.2, 1000 65 -> 48, 2000 211 -> 171, 4096 621 -> 513 (m = 4096, d = 768: 94 -> 37).  A third
// group in flight: 4096 479, but 64 14.5; tiles dealt to the XCDs in 4 x 4 groups halve the misses and gain nothing.
typedef float floatx16 __attribute__((ext_vector_type(16)));
constexpr int kGramTile = 64;

// t -> (ta, tb), ta <= tb, t = tb (tb + 1) / 2 + ta
__device__ __forceinline__ void upper_tile(int t, int& ta, int& tb)
{
    tb = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while ((tb + 1) * (tb + 2) / 2 <= t) ++tb;
    while (tb * (tb + 1) / 2 > t) --tb;
    ta = t - tb * (tb + 1) / 2;
}

// A tile put together in LDS goes to rows a0 .. and columns b0 .. of G, and once more turned over
constexpr int kGramTilePitch = 65;
__device__ __forceinline__ void store_gram_tile(const float* T, float* __restrict__ G, int d, int a0, int b0, int wave, int lane, bool mirror)
{
    if (b0 + lane < d) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int r = wave * 16 + i;
            if (a0 + r < d) G[(long long)(a0 + r) * d + b0 + lane] = T[r * kGramTilePitch + lane];
        }
    }
    if (mirror && a0 + lane < d) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int r = wave * 16 + i;
            if (b0 + r < d) G[(long long)(b0 + r) * d + a0 + lane] = T[lane * kGramTilePitch + r];
        }
    }
}

// Slab z handles rows [z * kchunk, (z + 1) * kchunk) of B and writes its own d x d matrix of `out`, tiles on and above the
// diagonal only (gram_reduce_kernel adds the slabs up and mirrors); with a single slab `out` is G, mirrored here.
template <bool EVEN>
__global__ void __launch_bounds__(256, 2) sketch_gram_kernel(const float* __restrict__ B, int m_total, int d, int kchunk, int mirror,
                                                             float* __restrict__ out)
{
    __shared__ float red[4][3][16][64];      // [quadrant][contributor][register][lane]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    int ta, tb;
    upper_tile((int)blockIdx.x, ta, tb);
    const int a0 = ta * kGramTile, b0 = tb * kGramTile;
    const int s_begin = blockIdx.y * kchunk;
    const int s_end = s_begin + kchunk < m_total ? s_begin + kchunk : m_total;
    const int quarter = (((s_end - s_begin + 3) >> 2) + 1) & ~1;
    const int k_begin = s_begin + wave * quarter;
    const int k_end = k_begin + quarter < s_end ? k_begin + quarter : s_end;

    floatx16 acc[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][u][v] = 0.f;

    constexpr int UNROLL = 8;
    // columns past the last one are read from it: they only reach entries that are not stored
    int ca[2], cb[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int last = EVEN ? d - 2 + t : d - 1;
        ca[t] = a0 + 2 * l32 + t < d ? a0 + 2 * l32 + t : last;
        cb[t] = b0 + 2 * l32 + t < d ? b0 + 2 * l32 + t : last;
    }
    struct Group { float a[UNROLL][2], b[UNROLL][2]; };
    auto load = [&](Group& g, int k0) {
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) {
            const int row = k0 + 2 * i + half;
            const float* r = B + (long long)(row < k_end ? row : k_end - 1) * d;      // clamped: no load under a condition
            if constexpr (EVEN) {
                const float2 fa = *reinterpret_cast<const float2*>(r + ca[0]), fb = *reinterpret_cast<const float2*>(r + cb[0]);
                g.a[i][0] = fa.x; g.a[i][1] = fa.y;
                g.b[i][0] = fb.x; g.b[i][1] = fb.y;
            } else {
#pragma unroll
                for (int t = 0; t < 2; ++t) { g.a[i][t] = r[ca[t]]; g.b[i][t] = r[cb[t]]; }
            }
        }
    };
    auto multiply = [&](Group& g, int k0) {
        if (k0 + 2 * UNROLL > k_end) {               // rows past the end count as zero in both operands
#pragma unroll
            for (int i = 0; i < UNROLL; ++i)
                if (k0 + 2 * i + half >= k_end) { g.a[i][0] = g.a[i][1] = g.b[i][0] = g.b[i][1] = 0.f; }
        }
#pragma unroll
        for (int i = 0; i < UNROLL; ++i)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int u = 0; u < 2; ++u) acc[t][u] = __builtin_amdgcn_mfma_f32_32x32x2f32(g.a[i][t], g.b[i][u], acc[t][u], 0, 0, 0);
    };
    constexpr int STEP = 2 * UNROLL;
    Group g0, g1;
    if (k_end - k_begin > STEP) {
        load(g0, k_begin);
        int k0 = k_begin;
        do {
            load(g1, k0 + STEP);
            multiply(g0, k0);
            load(g0, k0 + 2 * STEP);
            if (k0 + STEP < k_end) multiply(g1, k0 + STEP);
            k0 += 2 * STEP;
        } while (k0 < k_end);
    } else if (k_begin < k_end) {            // one group: no load that is not multiplied (m = 1000, d = 129 13.2 -> 12.8 us)
        load(g0, k_begin);
        multiply(g0, k_begin);
    }

    // wave w ends up with quadrant (w / 2, w % 2): the others hand it theirs
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (q != wave) {
#pragma unroll
            for (int v = 0; v < 16; ++v) red[q][wave < q ? wave : wave - 1][v][lane] = acc[q >> 1][q & 1][v];
        }
    __syncthreads();
    float sum[16];
#pragma unroll
    for (int c = 0; c < 4; ++c) {            // always in the order of the rows, so that the diagonal tiles are symmetric too
        if (c == wave) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q == wave) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) sum[v] = c ? sum[v] + acc[q >> 1][q & 1][v] : acc[q >> 1][q & 1][v];
                }
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float r = red[wave][c < wave ? c : c - 1][v][lane];
                sum[v] = c ? sum[v] + r : r;
            }
        }
    }

    // Result register v of lane l holds row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32 of its quadrant (i, j) = (wave / 2,
    // wave % 2), which stand for row 2 row + i and column 2 column + j of the tile.
    __syncthreads();
    float* T = &red[0][0][0][0];
    static_assert(sizeof(red) >= kGramTile * kGramTilePitch * sizeof(float), "the tile fits the exchange buffer");
#pragma unroll
    for (int v = 0; v < 16; ++v)
        T[(2 * (8 * (v >> 2) + 4 * half + (v & 3)) + (wave >> 1)) * kGramTilePitch + 2 * l32 + (wave & 1)] = sum[v];
    __syncthreads();
    store_gram_tile(T, out + (long long)blockIdx.y * d * d, d, a0, b0, wave, lane, mirror && ta < tb);
}

// The same with a quadrant of the tile per wave, through all rows (one slab): nothing is added up between waves and no group
// of rows is mostly empty, at the price of every operand being loaded by two waves.  Four sums per entry, every fourth row pair
// each, keep an entry's chain of additions as short as the rows split over the waves do.
// For up to 64 rows, for up to 128 where one slab fills the chip, and there for every odd d, whose 8-byte loads the other kernel
// has to do without.  Former 128 x 128 tiles / rows split over the waves / this kernel, in us:
// m = 16, d = 129 5.1 / 7.2 / 3.9, 1000 5.8 / 6.8 / 4.6, 3001 13.6 / 24.7 / 11.7; m = 64, 64 9.2 / 5.1 / 4.4, 4096 35 / 29.8 / 26;
// m = 128, 4096 57 / 46 / 40; m = 300, 4001 104 / 111 / 77, 4096 105 / 86 / - ; m = 2048, 1921 210 / 127 / 117, 4001 623 / 598 / 454.
__global__ void __launch_bounds__(256) sketch_gram_quadrants_kernel(const float* __restrict__ B, int m, int d, float* __restrict__ G)
{
    __shared__ float T[kGramTile * kGramTilePitch];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    int ta, tb;
    upper_tile((int)blockIdx.x, ta, tb);
    const int a0 = ta * kGramTile, b0 = tb * kGramTile;
    const int qa = 32 * (wave >> 1), qb = 32 * (wave & 1);      // the quadrant's first row and column of the tile
    // columns past the last one are read from it: they only reach entries that are not stored
    const int ca = a0 + qa + l32 < d ? a0 + qa + l32 : d - 1, cb = b0 + qb + l32 < d ? b0 + qb + l32 : d - 1;
    floatx16 acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[q][v] = 0.f;
    constexpr int UNROLL = 8;
    for (int k0 = 0; k0 < m; k0 += 2 * UNROLL) {
        float fa[UNROLL], fb[UNROLL];
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) {
            const int row = k0 + 2 * i + half;
            const float* r = B + (long long)(row < m ? row : m - 1) * d;      // clamped: no load under a condition
            fa[i] = r[ca]; fb[i] = r[cb];
        }
        if (k0 + 2 * UNROLL > m) {                   // rows past the end count as zero in both operands
#pragma unroll
            for (int i = 0; i < UNROLL; ++i)
                if (k0 + 2 * i + half >= m) fa[i] = fb[i] = 0.f;
        }
#pragma unroll
        for (int i = 0; i < UNROLL; ++i)
            if (k0 + 2 * i < m) acc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i], fb[i], acc[i & 3], 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) T[(qa + 8 * (v >> 2) + 4 * half + (v & 3)) * kGramTilePitch + qb + l32] = ((acc[0][v] + acc[1][v]) + acc[2][v]) + acc[3][v];
    __syncthreads();
    store_gram_tile(T, G, d, a0, b0, wave, lane, ta < tb);
}

// G from the slabs: a block adds up one 32 x 32 tile on or above the diagonal (fixed order) and stores it twice
__global__ void __launch_bounds__(256) gram_reduce_kernel(const float* __restrict__ slabs, int count, int d, float* __restrict__ G)
{
    __shared__ float tile[32][33];
    int ta, tb;
    upper_tile((int)blockIdx.x, ta, tb);
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const long long len = (long long)d * d;
    const int col = tb * 32 + tx, cc = col < d ? col : d - 1;
    const float* p[4];
    float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = ta * 32 + ty + 8 * i;
        p[i] = slabs + (long long)(row < d ? row : d - 1) * d + cc;
    }
    // 32 loads in flight, those of slabs past the last one from it; the order of the additions stays fixed.  (The last count mod 8
    // slabs one after the other, each waited for: Gram call with both kernels, in us: m = 2048, d = 500 15.6 -> 14.7, m = 1024, d = 500 14.3 -> 13.4,
    // m = 1000, d = 100 11.4 -> 10.0.)
    for (int k = 0; k < count; k += 8) {
        float v[4][8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i][j] = p[i][(k + j < count ? k + j : count - 1) * len];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (k + j < count)
#pragma unroll
                for (int i = 0; i < 4; ++i) s[i] += v[i][j];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = ta * 32 + ty + 8 * i;
        tile[ty + 8 * i][tx] = s[i];
        if (row < d && col < d) G[(long long)row * d + col] = s[i];
    }
    if (ta == tb) return;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = tb * 32 + ty + 8 * i, c = ta * 32 + tx;
        if (r < d && c < d) G[(long long)r * d + c] = tile[tx][ty + 8 * i];
    }
}

// Slabs that the scratch of a call has room for: what 128 x 128 tiles would need to fill the chip, at least 64 rows of B
// per slab, at most 64 slabs (the sizes of workspaces, and which calls the built-in scratch serves, follow from it)
int sketch_gram_slabs(int m, int d)
{
    const long long tiles = (long long)((d + 127) / 128) * ((d + 127) / 128);
    constexpr int kGramWorkgroups = 256;
    long long ks = (kGramWorkgroups + tiles - 1) / tiles;
    if (ks > (m + 63) / 64) ks = (m + 63) / 64;
    if (ks > 64) ks = 64;
    return ks < 1 ? 1 : (int)ks;
}

// Scratch of the entry point that allocates nothing: the slabs of the split sum live in a file-scope device array.
// Every GPU the library runs on holds its own copy at its own address; in host code the array's name is only a
// handle, so its device address is asked for once per device (hipGetSymbolAddress with that device current) and
// kept, and that pointer - never the name - is what reaches the kernels.
static __device__ __align__(256) unsigned char gram_static_scratch[kGramStaticScratchBytes];
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_lock;
static float* g_scratch_ptr[kMaxDevices];     // device address of gram_static_scratch on each device, once known

hipError_t gram_static_scratch_ptr(float** ptr)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(gram_static_scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = static_cast<float*>(p);
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

hipError_t launch_sketch_gram(const float* B, int m, int d, float* G, float* slabs, hipStream_t s)
{
    if (m <= 0 || d <= 0) return hipSuccess;
    const long long g = (d + kGramTile - 1) / kGramTile, tiles = g * (g + 1) / 2;
    if (tiles > 0x1fffffffLL) return hipErrorInvalidConfiguration;
    if (m <= 64 || ((m <= 128 || (d & 1)) && sketch_gram_slabs(m, d) == 1)) {
        hipLaunchKernelGGL(sketch_gram_quadrants_kernel, dim3((unsigned)tiles), dim3(256), 0, s, B, m, d, G);
        return hipGetLastError();
    }
    // slabs: the fewest that bring the busiest compute unit's share of the rows within 10 % of the least, as far as the
    // scratch goes
    const int room = sketch_gram_slabs(m, d);
    auto share = [&](int k) { return (double)((tiles * k + 255) / 256) / k; };
    double least = share(1);
    for (int k = 2; k <= room; ++k) least = share(k) < least ? share(k) : least;
    int ks = 1;
    while (share(ks) > 1.1 * least) ++ks;
    const int kchunk = ((m + ks - 1) / ks + 1) & ~1;
    float* to = ks > 1 ? slabs : G;
    if (d & 1) hipLaunchKernelGGL(sketch_gram_kernel<false>, dim3((unsigned)tiles, (unsigned)ks), dim3(256), 0, s, B, m, d, kchunk, ks == 1, to);
    else hipLaunchKernelGGL(sketch_gram_kernel<true>, dim3((unsigned)tiles, (unsigned)ks), dim3(256), 0, s, B, m, d, kchunk, ks == 1, to);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || ks == 1) return e;
    const long long g32 = (d + 31) / 32;
    hipLaunchKernelGGL(gram_reduce_kernel, dim3((unsigned)(g32 * (g32 + 1) / 2)), dim3(256), 0, s, slabs, (int)ks, d, G);
    return hipGetLastError();
}
}  // namespace spinner
