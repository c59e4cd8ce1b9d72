// Fused three-round kernels with the sign-code epilogue (angular-kernel features),
// n = 2^8 .. 2^16, with fp32 diagonals or packed sign words; the last round is pruned
// when m <= n / 16.  Also the code-packing kernel used above the fused range and the
// Hamming-distance Gram kernel.
#include "launch.hpp"
namespace spinner {
// The epilogue needs a whole wave per 256 coordinates (six lane bits per tile), so the
// values per thread are capped at n / 64.
template <typename TU, int NT>
using GeomCodeFrom = TileGeom<NT, clamp_rmax(NT, (TU::rmax < NT - 6 ? TU::rmax : NT - 6)),
                              TU::waves, TU::min_waves, TU::trips>;
// Without pruning, n = 2^12 .. 2^14 take the wide exchanges of the plain kernels, loading in layout 1 so that
// the three rounds end in layout 0, where a wave's lanes hold index bits 2..7 (one code word per register).
template <int NT> struct CodeWide { static constexpr int rmax = NT >= 13 ? 6 : 5, waves = 4, min_waves = NT >= 13 ? 4 : 0, trips = 2, wide = 1, start = 1, chunk = kLaneChunk; };
template <int NT, bool PRUNED>
using GeomCode = std::conditional_t<PRUNED, GeomCodeFrom<PrunedTuning<float, NT>, NT>,
                                    std::conditional_t<has_wide_words(NT), GeomFrom<CodeWide<NT>, NT>, GeomCodeFrom<Tuning<float, NT>, NT>>>;

template <int NT, bool SIGNS, int PRUNE>
static hipError_t launch_code_tile(const TileParams& p, long long tiles, hipStream_t stream)
{
    using G = GeomCode<NT, (PRUNE > 0)>;
    static_assert(G::TILES_PER_WG >= 1 && G::LB == 6, "one tile per wave or several waves per tile");
    const long long blocks = (tiles + G::TILES_PER_WG - 1) / G::TILES_PER_WG;
    if (blocks <= 0) return hipSuccess;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    TileParams q = p;
    q.xcd_group_log = SIGNS ? xcd_group_log_for<G>() : -1;
    hipLaunchKernelGGL((spinner_tile_kernel<float, G, NT, 3, true, EPI_STORE_SIGNBITS, SIGNS, PRUNE>),
                       dim3((unsigned)blocks), dim3(G::THREADS), 0, stream, q);
    return hipGetLastError();
}

#define CASE(NT) case NT: return signs ? launch_code_tile<NT, true, 0>(p, tiles, s) : launch_code_tile<NT, false, 0>(p, tiles, s);
#define PCASE(NT) case NT: return signs ? launch_code_tile<NT, true, kPruneBits>(p, tiles, s) \
                                        : launch_code_tile<NT, false, kPruneBits>(p, tiles, s);
hipError_t launch_fused_signbits(int log2n, bool signs, int prune, const TileParams& p, long long tiles, hipStream_t s)
{
    if (prune >= kPruneBits) {
        switch (log2n) {
            PCASE(12) PCASE(13) PCASE(14)
        default: break;
        }
    }
    switch (log2n) {
        CASE(8) CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14) CASE(15) CASE(16)
    default: return hipErrorInvalidValue;
    }
}
#undef CASE
#undef PCASE

// One wave per code word: lane l looks at coordinate ((w >> 2) << 8) | (l << 2) | (w & 3)
// of its vector and the wave's ballot of "negative" is the word.
__global__ void __launch_bounds__(256) pack_codes_kernel(const float* __restrict__ y, long long y_stride,
                                                         unsigned long long* __restrict__ codes, int words_per_vec,
                                                         long long total_words)
{
    const long long gw = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (gw >= total_words) return;
    const long long vec = gw / words_per_vec;
    const int w = (int)(gw - vec * words_per_vec);
    const long long e = ((long long)(w >> 2) << 8) | (lane << 2) | (w & 3);
    const unsigned long long mk = __ballot(y[vec * y_stride + e] < 0.0f);
    if (lane == 0) codes[gw] = mk;
}

hipError_t launch_pack_codes(const float* y, long long y_stride, unsigned long long* codes, int m, long long batch, hipStream_t s)
{
    const int words = m / 64;
    const long long total = batch * words;
    const long long blocks = (total + 3) / 4;
    if (blocks <= 0) return hipSuccess;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(pack_codes_kernel, dim3((unsigned)blocks), dim3(256), 0, s, y, y_stride, codes, words, total);
    return hipGetLastError();
}

// out[i][j] = 1 - popcount(a_i xor b_j) / m.  With the code bits as numbers +1 (0) and -1 (1),
//     popcount(a xor b) = (m - <a, b>) / 2,
// and the table of inner products <a_i, b_j> is a dense contraction over the m code bits: it runs on the matrix
// pipe in the narrowest format that holds +-1, fp4 (E2M1, 0x2 = 1.0, bit 3 the sign; v_mfma_scale_f32_32x32x64_f8f6f4 with
// unit scales; products and fp32 sums of at most 2^24 ones: exact).  A workgroup of four waves owns 128 x 128 pairs
// (each wave 64 x 64 = 2 x 2 tiles) and walks the code words in chunks of 16 staged in LDS; the next chunk is already in
// registers while one is multiplied.  A row is read from LDS 16 bytes per lane (rows padded to 144 bytes: the sixteen
// lanes of a phase cover all banks once): lane group g = lane / 32 takes the g-th 16 bytes of every 32, that is the operand
// dwords of four instructions.  An instruction's operand is a dword of code bits spread into nibbles: dword q of the fp4
// vector holds bits q, q + 4, .., q + 28, each moved to bit 3 of its nibble by doubling and joined with 1.0 by one
// three-operand logic instruction (shifts and v_and_or issue at half its rate).  Which bit lands in which of the 64
// k-slots does not matter, as long as both operands are spread the same way.
// Bound: per code word a wave has four operands to spread at 19 cycles beside four products at 32 (4.9 PFLOP/s of 10.1 for
// long codes, at the clock the chip holds under them), and the results' way out: rows of `out` that are no multiple of 64
// bytes long take twice the write requests.  Against bits as 0 / 1 with the rows' weights counted on the way, half words read
// from LDS and tiles dealt to the XCDs one by one, in us: 16384 x 16384, m = 256 284 -> 191, m = 4096 656 -> 622, m = 16384
// 1808 -> 1785; 16384 x 10007, m = 256 255 -> 154, m = 4096 479 -> 420; 4096 x 4096, m = 1024 23.3 -> 18.3.  Bands of one or
// eight tile rows: 435, 428 at 16384 x 10007, m = 4096.
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef int intx8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
constexpr int kGramRows = 128, kGramCols = 128, kGramChunk = 16;      // chunk: code words per row
constexpr int kGramPitch = kGramChunk / 2 + 1;                        // LDS row, in 16-byte units
constexpr unsigned kGramBand = 4;                                     // tile rows per band (see the kernel)

// the 32 bits of w as 32 fp4 numbers (+1.0 or -1.0) in four dwords
__device__ __forceinline__ intx8 spread_bits_fp4(unsigned w, unsigned sign, unsigned one)
{
    intx8 f = {0, 0, 0, 0, 0, 0, 0, 0};
    f[3] = (int)__builtin_amdgcn_bitop3_b32(w, sign, one, 0xEA);      // (w & sign) | one
    w += w;
    f[2] = (int)__builtin_amdgcn_bitop3_b32(w, sign, one, 0xEA);
    w += w;
    f[1] = (int)__builtin_amdgcn_bitop3_b32(w, sign, one, 0xEA);
    w += w;
    f[0] = (int)__builtin_amdgcn_bitop3_b32(w, sign, one, 0xEA);
    return f;
}

// Three workgroups per compute unit cost 20 bytes of scratch per thread.
// LINES: rows of `out` are whole 128-byte lines (nb a multiple of 32) and bypass cache retention (4096 x 4096, m = 1024 18.2 ->
// 16.4 us; 16384 x 16384, m = 4096 625 -> 607); the pieces of other rows' lines have to meet in the L2 (16384 x 10007, m = 256:
// 152 us, with the hint 338)
template <bool LINES>
__global__ void __launch_bounds__(256, 3) hamming_gram_kernel(const uintx4* __restrict__ a, long long na, const uintx4* __restrict__ b,
                                                           long long nb, int words, float inv_m, unsigned gx, unsigned gy, float* __restrict__ out)
{
    __shared__ uintx4 sa[kGramRows * kGramPitch];
    __shared__ uintx4 sb[kGramCols * kGramPitch];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wr = wave >> 1, wc = wave & 1, g = lane >> 5, l32 = lane & 31;
    // Tiles in bands of four tile rows, column by column, and an equal run of that order per XCD (workgroups go to the eight
    // XCDs in turn): the tiles in flight on an XCD share their codes in its L2, and the two halves of a 128-byte line of
    // `out` that straddles two tiles (rows of any length are allowed) meet there instead of leaving two L2s in pieces
    const unsigned total = gx * gy, xcd = blockIdx.x & 7, longer = total & 7;      // the first `longer` XCDs take one tile more
    const unsigned tile = xcd * (total >> 3) + (xcd < longer ? xcd : longer) + (blockIdx.x >> 3);
    const unsigned band = tile / (kGramBand * gx), in_band = tile - band * kGramBand * gx;
    const unsigned height = gy - kGramBand * band < kGramBand ? gy - kGramBand * band : kGramBand;
    const unsigned tj = in_band / height, ti = kGramBand * band + in_band - tj * height;
    const long long i0 = (long long)ti * kGramRows, j0 = (long long)tj * kGramCols;
    floatx16 acc[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][u][v] = 0.0f;
    const int scale = 0x7f7f7f7f;                    // scale exponents (E8M0): 2^0
    unsigned sign = 0x88888888u, one = 0x22222222u;
    asm("" : "+v"(sign), "+v"(one));                 // in vector registers: scalar operands halve the issue rate

    // staging: 128 rows of 8 16-byte pieces per operand, four pieces per thread and operand; rows and pieces past the end
    // are read from the last one (they reach no stored result)
    const int srow = threadIdx.x >> 3, scol = threadIdx.x & 7;
    const int pieces = words >> 1;                   // 16-byte pieces per row (words is a multiple of 4)
    const uintx4* ra[4];
    const uintx4* rb[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const long long i = i0 + t * 32 + srow, j = j0 + t * 32 + srow;
        ra[t] = a + (i < na ? i : na - 1) * pieces;
        rb[t] = b + (j < nb ? j : nb - 1) * pieces;
    }
    uintx4 pa[4], pb[4];
    auto load = [&](int piece0) {
        const int c = piece0 + scol < pieces ? piece0 + scol : pieces - 1;
#pragma unroll
        for (int t = 0; t < 4; ++t) { pa[t] = ra[t][c]; pb[t] = rb[t][c]; }
    };
    load(0);
    const uintx4* ha = sa + (wr * 64 + l32) * kGramPitch + g;
    const uintx4* hb = sb + (wc * 64 + l32) * kGramPitch + g;
    for (int p0 = 0; p0 < pieces; p0 += kGramChunk / 2) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            sa[(t * 32 + srow) * kGramPitch + scol] = pa[t];
            sb[(t * 32 + srow) * kGramPitch + scol] = pb[t];
        }
        __syncthreads();
        if (p0 + kGramChunk / 2 < pieces) load(p0 + kGramChunk / 2);
        const int steps = pieces - p0 < kGramChunk / 2 ? pieces - p0 : kGramChunk / 2;
        for (int s = 0; s < steps; s += 2) {
            uintx4 qa[2], qb[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) { qa[t] = ha[t * 32 * kGramPitch + s]; qb[t] = hb[t * 32 * kGramPitch + s]; }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                intx8 fa[2], fb[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    fa[t] = spread_bits_fp4(qa[t][k], sign, one);
                    fb[t] = spread_bits_fp4(qb[t][k], sign, one);
                }
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        acc[t][u] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fa[t], fb[u], acc[t][u], 4, 4, 0, scale, 0, scale);
            }
        }
        __syncthreads();
    }
    // result register v of lane l holds row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32 of its 32 x 32 tile
    const int m = words * 64;
    const long long i = i0 + wr * 64 + 4 * g, j = j0 + wc * 64 + l32;
    float* dst = out + i * nb + j;
    const int rows = na - i < 64 ? (int)(na - i) : 64, cols = nb - j < 64 ? (int)(nb - j) : 64;      // what is left below and right of it
    auto store = [&](auto whole) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = t * 32 + 8 * (v >> 2) + (v & 3);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int dh = (m - (int)acc[t][u][v]) >> 1;
                    const float k = 1.0f - (float)dh * inv_m;
                    if (decltype(whole)::value || (r < rows && u * 32 < cols)) {
                        if constexpr (LINES) __builtin_nontemporal_store(k, dst + r * nb + u * 32);
                        else dst[r * nb + u * 32] = k;
                    }
                }
            }
    };
    if (i0 + kGramRows <= na && j0 + kGramCols <= nb) store(std::true_type{});
    else store(std::false_type{});
}

hipError_t launch_hamming_gram(const unsigned long long* a, long long na, const unsigned long long* b, long long nb, int m,
                               float* out, hipStream_t s)
{
    if (na <= 0 || nb <= 0) return hipSuccess;
    const long long gx = (nb + kGramCols - 1) / kGramCols, gy = (na + kGramRows - 1) / kGramRows;
    // one workgroup of 256 threads per tile, and a grid holds fewer than 2^32 threads; the caller keeps gy below 2^16
    if (gx > 0xffffffLL || gx * gy > 0xffffffLL) return hipErrorInvalidConfiguration;
    const auto kernel = (nb & 31) == 0 ? hamming_gram_kernel<true> : hamming_gram_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(gx * gy)), dim3(256), 0, s, reinterpret_cast<const uintx4*>(a), na,
                       reinterpret_cast<const uintx4*>(b), nb, m / 64, 1.0f / (float)m, (unsigned)gx, (unsigned)gy, out);
    return hipGetLastError();
}
}  // namespace spinner
