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

// out[i][j] = 1 - popcount(a_i xor b_j) / m.  The table of inner products of the code bits is a dense contraction and runs on the
// matrix pipe in the narrowest format, fp4 (E2M1; v_mfma_scale_f32_32x32x64_f8f6f4).  A nibble of code bits is four planes, and a
// plane is an operand as it lies: masked with 0x1, 0x2, 0x4 its numbers are 0 or 0.5, 1, 2 (whose weight the scale exponents of
// the instruction take out: every common bit counts 4), masked with 0x8 and joined with 0x2 they are +1 or -1.  So the four dwords
// that a lane reads at once are the operands of four instructions at one logic instruction a dword.  With the rows' bits in planes
// 0 to 2 counted apart (w),
//     popcount(a xor b) = w(a) + w(b) + m / 8 - S / 2,      S = sum of the four products,
// where all is whole numbers below 2^24 up to m = 2^22 (kGramMixed); longer codes (kGramCounted) take plane 3 as 0 or 2 as well, and then
// popcount = w(a) + w(b) - S / 2 with S four times the common bits: w(a) - S / 2 lies between -w(a) and w(a), so that it and the distance
// are whole numbers up to m, exact in fp32 to m = 2^24 (w(a) + w(b) by itself is not, from 2^23 on).  Codes beyond that (kGramSigned) take
// every bit as +1 or -1: popcount = (m - S) / 2, where S stays small for unrelated codes and a sum of whole 64s for equal and opposite
// ones, so that these remain exact; a dword of bits is then spread over four operand dwords at seven instructions (counted / signed,
// in ms: 1024 x 2048 codes of 2^25 bits 71.2 / 72.1, 5 x 70 of 2^26 111 / 115).
// Which bit lands in which of the 64 k-slots does not matter, as long as both operands are laid out the same way.
// A workgroup of four waves owns 128 x 128 pairs (each wave 64 x 64 = 2 x 2 tiles) and walks the code words in chunks of 8, which
// loads write to LDS directly, one chunk ahead into the other of two buffers: a barrier a chunk.  The 16-byte pieces of a row lie
// exchanged by its number, so that the sixteen lanes of a phase cover all banks once.  Lane group g = lane / 32 takes the pieces
// of parity g.
// Bound: the matrix pipe, which takes 34 to 37 cycles per product (random codes: the longer) with up to four vector instructions
// beside it and 2.6 more for each further one, and the results' way out: rows of `out` that are no multiple of 64 bytes long take
// twice the write requests.  A product takes 49 cycles here for long codes (6.1 PFLOP/s of 10.1).  Against +1 / -1 in all planes
// (shifts and seven instructions an operand dword), staged through registers, in us: 16384 x 10007, m = 4096 333 -> 294, m = 256
// 150 -> 147; 16384 x 16384, m = 16384 1700 -> 1450, m = 4096 505 -> 443, m = 256 190 -> 192; 700 x 11000, m = 4096 28 -> 22;
// 12000 x 300, m = 8192 33 -> 28; 4096 x 4096, m = 1024 16.5 -> 16.3.  Workgroups per compute unit, 16384 x 10007 (m = 256, 4096): two
// 140, 305, three 147, 298, four 158, 294, but 16384 x 16384 three 443, two 466 and 9001 x 4999, m = 768, 33 and 38: three.  Results put
// in order through LDS and stored in whole lines: 148, 329.  Bands of one or eight tile rows cost 2 to 4 %.
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef int intx8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
constexpr int kGramRows = 128, kGramCols = 128, kGramChunk = 8;       // chunk: code words per row
constexpr int kGramPieces = kGramChunk / 2;                           // 16-byte pieces of a row's chunk
constexpr unsigned kGramBand = 4;                                     // tile rows per band (see the kernel)
constexpr unsigned kGramSpareLds = 14 << 10;                          // asked for and not used: three workgroups per compute unit, not four
enum { kGramMixed, kGramCounted, kGramSigned };                       // forms of the operands, see above
constexpr int kGramMixedBits = 1 << 22, kGramCountedBits = 1 << 24;   // longest codes of the first two

// operand P of four from 128 code bits, 32 fp4 numbers: plane P of them, signed codes dword P
template <int P, int FORM>
__device__ __forceinline__ intx8 code_operand(uintx4 w, unsigned sign, unsigned one)
{
    intx8 f = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if constexpr (FORM == kGramSigned) f[k] = (int)__builtin_amdgcn_bitop3_b32(w[P] << (3 - k), sign, one, 0xEA);
        else if constexpr (P < 3) f[k] = (int)(w[k] & (0x11111111u << P));
        else if constexpr (FORM == kGramCounted) f[k] = (int)((w[k] >> 1) & 0x44444444u);
        else f[k] = (int)__builtin_amdgcn_bitop3_b32(w[k], sign, one, 0xEA);      // (w & sign) | one
    }
    return f;
}

// LINES: rows of `out` are whole 128-byte lines (nb a multiple of 32) and bypass cache retention (4096 x 4096, m = 1024 18.2 ->
// 16.4 us; 16384 x 16384, m = 4096 625 -> 607); the pieces of other rows' lines have to meet in the L2 (16384 x 10007, m = 256:
// 152 us, with the hint 338)
// FEW: few tiles of short codes, ragged ones among them, are over soon enough that fetching the instructions counts (those of the stores with
// checks lie behind the rest), and half as many in the chunk gain more than an index known in advance.  Unrolled / not, in us: 300 x 300,
// m = 256 5.06 / 4.74, m = 1024 6.17 / 5.92; 100 x 5000, m = 512 5.84 / 5.50, m = 1024 6.57 / 6.37; 2000 x 2000, m = 256 6.89 / 6.63, m = 1024 8.18 / 8.01;
// 12000 x 300, m = 1024 9.17 / 9.03; but whole tiles, 1024 x 1024, m = 1024, 4.91 / 4.97, 4096 x 2048, m = 512, 7.83 / 8.03, more tiles, 700 x 11000, m = 256, 8.88 /
// 8.98, longer codes, 1000 x 1000, m = 4096, 11.64 / 11.90, 16384 x 10007, m = 4096, 294.8 / 297.5
template <bool LINES, int FORM, bool FEW>
__global__ void __launch_bounds__(256, 3) hamming_gram_kernel(const uintx4* __restrict__ a, long long na, const uintx4* __restrict__ b,
                                                           long long nb, int words, float inv_m, unsigned gx, unsigned gy, float* __restrict__ out)
{
    // rows of a, then of b; two arrays, each read and written in code of its own, so that the compiler sees that what is read is
    // not what the loads in flight write and does not wait for them
    __shared__ uintx4 even[(kGramRows + kGramCols) * kGramPieces], odd[(kGramRows + kGramCols) * kGramPieces];
    __shared__ float weights[kGramRows + kGramCols];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
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
    unsigned sign = 0x88888888u, one = 0x22222222u;
    asm("" : "+v"(sign), "+v"(one));                 // in vector registers: scalar operands halve the issue rate

    // staging: a wave brings 64 rows, 16 of them an instruction, lane l the piece of its row that lands at l mod 4; rows and
    // pieces past the end are read from the last one (they reach no stored result)
    const int pieces = words >> 1;                   // 16-byte pieces per row (words is a multiple of 4)
    const int swap = (l32 >> 2) & 3;                 // piece p of row r lies at p xor (r / 4 mod 4)
    const int spiece = (lane & 3) ^ (lane >> 4);
    const uintx4* rows[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int r = (wave & 1) * 64 + t * 16 + (lane >> 2);
        const long long i = i0 + r, j = j0 + r;
        rows[t] = wave < 2 ? a + (i < na ? i : na - 1) * pieces : b + (j < nb ? j : nb - 1) * pieces;
    }
    auto load = [&](int piece0, uintx4* buffer) {
        const int c = piece0 + spiece < pieces ? piece0 + spiece : pieces - 1;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(rows[t] + c),
                                             (__attribute__((address_space(3))) void*)(buffer + (wave * 64 + t * 16) * kGramPieces), 16, 0, 0);
    };
    int weight = 0;                                   // of the row that this thread counts
    auto chunk = [&](int p0, const uintx4* now, uintx4* next) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wave's rows are in place
        __syncthreads();                                      // everyone's are, and the other buffer has been read
        if (p0 + kGramPieces < pieces) load(p0 + kGramPieces, next);
        const uintx4* ha = now + (wr * 64 + l32) * kGramPieces;
        const uintx4* hb = now + (kGramRows + wc * 64 + l32) * kGramPieces;
        const uintx4* hw = now + threadIdx.x * kGramPieces;
        const int have = pieces - p0 < kGramPieces ? pieces - p0 : kGramPieces;      // 2 or 4
        const auto two_pieces = [&](int s) {
            uintx4 qa[2], qb[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                qa[t] = ha[t * 32 * kGramPieces + ((s + g) ^ swap)];
                qb[t] = hb[t * 32 * kGramPieces + ((s + g) ^ swap)];
            }
            const uintx4 w0 = hw[s ^ swap], w1 = hw[(s + 1) ^ swap];
            static_for<0, 4>([&](auto plane) {
                constexpr int P = plane.value;
                constexpr int scale = (int)(0x01010101u * (FORM != kGramSigned && P < 2 ? 0x7fu + 2 - P : 0x7fu));      // exponents (E8M0)
                intx8 fa[2], fb[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    fa[t] = code_operand<P, FORM>(qa[t], sign, one);
                    fb[t] = code_operand<P, FORM>(qb[t], sign, one);
                }
                constexpr unsigned counted = FORM == kGramMixed ? 0x77777777u : ~0u;
                if constexpr (FORM != kGramSigned) weight += __popc(w0[P] & counted) + __popc(w1[P] & counted);
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        acc[t][u] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fa[t], fb[u], acc[t][u], 4, 4, 0, scale, 0, scale);
            });
        };
        if constexpr (FEW) {
#pragma unroll 1
            for (int s = 0; s < have; s += 2) two_pieces(s);
        } else {
#pragma unroll
            for (int s = 0; s < kGramPieces; s += 2) {
                if (s >= have) break;
                two_pieces(s);
            }
        }
    };
    load(0, even);
    for (int p0 = 0; p0 < pieces; p0 += 2 * kGramPieces) {
        chunk(p0, even, odd);
        if (p0 + kGramPieces < pieces) chunk(p0 + kGramPieces, odd, even);
    }
    weights[threadIdx.x] = (float)(weight + (FORM == kGramMixed && threadIdx.x < kGramRows ? words * 8 : 0));
    __syncthreads();
    // result register v of lane l holds row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32 of its 32 x 32 tile
    const long long i = i0 + wr * 64 + 4 * g, j = j0 + wc * 64 + l32;
    float* dst = out + i * nb + j;
    const int left = na - i < 64 ? (int)(na - i) : 64, cols = nb - j < 64 ? (int)(nb - j) : 64;      // what is left below and right of it
    const float* wa = weights + wr * 64 + 4 * g;
    const float* wb = weights + kGramRows + wc * 64 + l32;
    auto store = [&](auto whole) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = t * 32 + 8 * (v >> 2) + (v & 3);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const float dh = FORM == kGramSigned ? (float)((64u * words - (unsigned)(int)acc[t][u][v]) >> 1)
                                                         : __builtin_fmaf(acc[t][u][v], -0.5f, wa[r]) + wb[u * 32];      // both steps exact, in this order
                    const float k = __builtin_fmaf(-dh, inv_m, 1.0f);
                    if (decltype(whole)::value || (r < left && u * 32 < cols)) {
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
    const bool lines = (nb & 31) == 0;
    const bool ragged = na % kGramRows != 0 || nb % kGramCols != 0;
    const bool few = ragged && m <= 2 * 64 * kGramChunk && gx * gy <= 2 * kComputeUnits;
    const auto kernel = m > kGramCountedBits ? (lines ? hamming_gram_kernel<true, kGramSigned, false> : hamming_gram_kernel<false, kGramSigned, false>)
                        : m > kGramMixedBits ? (lines ? hamming_gram_kernel<true, kGramCounted, false> : hamming_gram_kernel<false, kGramCounted, false>)
                        : few                ? (lines ? hamming_gram_kernel<true, kGramMixed, true> : hamming_gram_kernel<false, kGramMixed, true>)
                                             : (lines ? hamming_gram_kernel<true, kGramMixed, false> : hamming_gram_kernel<false, kGramMixed, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(gx * gy)), dim3(256), kGramSpareLds, s, reinterpret_cast<const uintx4*>(a), na,
                       reinterpret_cast<const uintx4*>(b), nb, m / 64, 1.0f / (float)m, (unsigned)gx, (unsigned)gy, out);
    return hipGetLastError();
}
}  // namespace spinner
