// Fused three-round kernels, cos/sin random-feature epilogue, n = 2^4 .. 2^16.
// Up to 2^14 the butterflies run in fp64: with w = scale * y of magnitude ~10^2 the rounding
// of 3 log2(n) fp32 stages alone would exceed a 1e-5 relative feature error.
#include "launch.hpp"
#include "allreg.hpp"
namespace spinner {

// ------------------------------------------------------------------ feature kernel with every butterfly between registers
// The fp64 feature map is bound by the vector ALU, and a lane butterfly on fp64 values costs two lane moves
// and an addition at half rate.  For the sizes below (n = 2^(2r), one wave per 64 / 2^r vectors, +-1 diagonals
// as lane masks) all 3 * 2r stages are register stages of the two layouts of allreg.hpp; fp64 values cross the
// wave-private exchange buffer in two trips (low words, high words), so the buffer stays 4 bytes per element.
// x arrives through the same buffer after coalesced 16-byte loads; the three exchanges end in layout B, where
// register j of consecutive lanes holds consecutive coordinates: the cos and sin rows are written 4 bytes per
// lane, 64 lanes on 256 consecutive bytes.
template <typename G>
__device__ __forceinline__ void feat_ar_flip(double (&v)[G::R], const unsigned long long* words)
{
    sign_words_t w = (sign_words_t)words;
#pragma unroll
    for (int j = 0; j < G::R; ++j) flip_by_mask(v[j], w[j]);
}

template <typename G>
__device__ __forceinline__ void feat_ar_a_to_b(double (&v)[G::R], float4* pa, float* pb)
{
    int4* ia = reinterpret_cast<int4*>(pa);
    int* ib = reinterpret_cast<int*>(pb);
    int lo[G::R];
#pragma unroll
    for (int k = 0; k < G::R / 4; ++k)
        ia[k] = make_int4(__double2loint(v[4 * k]), __double2loint(v[4 * k + 1]), __double2loint(v[4 * k + 2]), __double2loint(v[4 * k + 3]));
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < G::R; ++j) lo[j] = ib[j * G::STRIDE];
    wave_lds_fence();
#pragma unroll
    for (int k = 0; k < G::R / 4; ++k)
        ia[k] = make_int4(__double2hiint(v[4 * k]), __double2hiint(v[4 * k + 1]), __double2hiint(v[4 * k + 2]), __double2hiint(v[4 * k + 3]));
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < G::R; ++j) v[j] = __hiloint2double(ib[j * G::STRIDE], lo[j]);
    wave_lds_fence();
}

// The same with one word per access, a lane's row 2^r + 1 words from the next, so that both sides touch different banks: low and high words lie in every
// other register, and the 16 bytes of one kind above are put together by four moves, their pairs taken apart by two more (n = 4096: 384 moves per
// vector).  The loads are written as atomic ones, which nothing joins into pairs.
// 16 bytes / one word, in us: n = 4096, sign words, 131072 vectors 1223 / 1200, first 1000, 8000 vectors 65.4 / 62.5; fp32 diagonals, 131072 1388 /
// 1336, L = 4, 32768 1333 / 1323, L = 3, first 2000, 8000 213 / 200; n = 1024, fp32 diagonals 298 / 293, L = 4 264 / 261, but sign words 277.7 / 282.9.
__device__ __forceinline__ int lds_word(const int* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT); }
template <typename G>
__device__ __forceinline__ void feat_ar_a_to_b_words(double (&v)[G::R], float* w, int l)
{
    int* ia = reinterpret_cast<int*>(w) + l * (G::R + 1);
    const int* ib = reinterpret_cast<const int*>(w) + l;
    int lo[G::R];
#pragma unroll
    for (int j = 0; j < G::R; ++j) ia[j] = __double2loint(v[j]);
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < G::R; ++j) lo[j] = lds_word(ib + j * (G::R + 1));
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < G::R; ++j) ia[j] = __double2hiint(v[j]);
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < G::R; ++j) v[j] = __hiloint2double(lds_word(ib + j * (G::R + 1)), lo[j]);
    wave_lds_fence();
}

template <typename G>
__device__ __forceinline__ void feat_ar_b_to_a(double (&v)[G::R], float4* pa, float* pb)
{
    int4* ia = reinterpret_cast<int4*>(pa);
    int* ib = reinterpret_cast<int*>(pb);
    int lo[G::R];
#pragma unroll
    for (int j = 0; j < G::R; ++j) ib[j * G::STRIDE] = __double2loint(v[j]);
    wave_lds_fence();
#pragma unroll
    for (int k = 0; k < G::R / 4; ++k) {
        const int4 t = ia[k];
        lo[4 * k] = t.x; lo[4 * k + 1] = t.y; lo[4 * k + 2] = t.z; lo[4 * k + 3] = t.w;
    }
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < G::R; ++j) ib[j * G::STRIDE] = __double2hiint(v[j]);
    wave_lds_fence();
#pragma unroll
    for (int k = 0; k < G::R / 4; ++k) {
        const int4 t = ia[k];
        v[4 * k] = __hiloint2double(t.x, lo[4 * k]);
        v[4 * k + 1] = __hiloint2double(t.y, lo[4 * k + 1]);
        v[4 * k + 2] = __hiloint2double(t.z, lo[4 * k + 2]);
        v[4 * k + 3] = __hiloint2double(t.w, lo[4 * k + 3]);
    }
    wave_lds_fence();
}

// fp32 diagonals for the same kernel.  In layout A a thread's entries are 2^r consecutive floats: the diagonal goes
// through the exchange buffer like x (coalesced 16-byte loads, 16-byte reads in layout A).  In layout B register j of
// consecutive lanes wants consecutive entries: 4-byte loads, 64 lanes on 256 consecutive bytes (the diagonal is
// cache-resident).
// Both are asked for a phase ahead of the use, D1 with x: two waves per SIMD leave the wait for them exposed otherwise (n = 4096, L = 4,
// batch 32768 1347 -> 1322 us; n = 1024, L = 4, 32768 273 -> 261; n = 1024, one block, 131072 297 -> 292; n = 4096, one block, 131072 1370 and
// 1375).  Lane masks a phase ahead in the same way gained nothing (n = 4096, 131072 1224 and 1221, m = 1000 68 and 72).
template <typename G>
struct ArDiagA {
    v4f t[G::R / 4];
    __device__ __forceinline__ void load(const float* d, unsigned at)      // at: the lane's first entry, 4 l
    {
#pragma unroll
        for (int k = 0; k < G::R / 4; ++k) t[k] = *reinterpret_cast<const v4f*>(d + 4 * k * G::LANES + at);
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void multiply(double (&v)[G::R], float* put, const float4* pa) const      // put: where that entry goes
    {
#pragma unroll
        for (int k = 0; k < G::R / 4; ++k) *reinterpret_cast<v4f*>(put + 4 * k * G::STRIDE) = t[k];
        wave_lds_fence();
#pragma unroll
        for (int k = 0; k < G::R / 4; ++k) {
            const float4 f = pa[k];
            v[4 * k] *= (double)f.x; v[4 * k + 1] *= (double)f.y; v[4 * k + 2] *= (double)f.z; v[4 * k + 3] *= (double)f.w;
        }
        wave_lds_fence();
    }
};
template <typename G>
struct ArDiagB {
    float t[G::R];
    __device__ __forceinline__ void load(const float* d, unsigned ebase)
    {
#pragma unroll
        for (int j = 0; j < G::R; ++j) t[j] = (d + (j << G::r))[ebase];
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void multiply(double (&v)[G::R]) const
    {
#pragma unroll
        for (int j = 0; j < G::R; ++j) v[j] *= (double)t[j];
    }
};

template <bool STREAM>
__device__ __forceinline__ void store1(float* p, float v)
{
    if constexpr (STREAM) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// BLOCKS: L stacked blocks (fp32 triples [L][3][n] from p.d[0] on, block l in columns [l m, (l + 1) m) of the cos and of the
// sin part), one wave per block and vector (or pair of vectors).  This kernel cannot keep x beside its 64 fp64 values per thread, so a
// vector's L workgroups each read it, and they have to do so from one L2: workgroups go to the eight XCDs in turn
// (workgroup b to XCD b mod 8), so the L blocks of a vector are workgroups eight apart.  Against the kernel of blocks.hip,
// which keeps x in registers but needs lane stages on fp64 values: L = 4, 2^27 elements in all, 2^10 336 -> 290 us, 2^12
// 393 -> 337 us; n = 4096, L = 4, batch 32768: 1512 -> 1372 us.  Bound: fp64 vector ALU, then HBM (779 us).
// STREAM: results bypass cache retention.  At n = 2^10 a store of a vector is one 128-byte line when rows and blocks are whole
// lines; the pieces of other rows' lines should meet in the L2.  Sign words, hint -> none, in us: m = 1001, batch 4096 19.1 ->
// 14.7, 16384 76 -> 46; m = 1000, 16384 61 -> 45; m = 640 (whole lines), 52428 86 -> 89.  Short rows lose less by pieces than by
// retention: m = 500 33.6 -> 35.3, m = 333 29.2 -> 35.0 (16384).  At n = 2^12 a store is two lines and the hint stays.
template <typename G, bool SIGNS, bool STREAM, bool BLOCKS = false>
__global__ void __launch_bounds__(G::THREADS) __attribute__((amdgpu_waves_per_eu(G::r >= 6 ? 2 : 4)))
spinner_feature_ar_kernel(TileParams p, int L)
{
    static_assert(!BLOCKS || (!SIGNS && G::WAVES == 1), "stacked blocks: fp32 diagonals, one wave per workgroup");
    static_assert(G::LB == G::r, "no lane bit is shared by the two layouts");
    constexpr int R = G::R, r = G::r, n = 1 << G::NT;
    constexpr bool WORDS = r >= 6 || !SIGNS;        // see feat_ar_a_to_b_words
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int g = lane >> G::LB, l = lane & (G::LANES - 1);
    long long wvec = ((long long)blockIdx.x * G::WAVES + wave) * G::TPW;     // first vector of this wave (wave-uniform)
    if constexpr (BLOCKS) {
        const unsigned q = blockIdx.x >> 3, vgroup = q / (unsigned)L, block = q - vgroup * (unsigned)L;
        wvec = ((long long)vgroup * 8 + (blockIdx.x & 7)) * G::TPW;
#pragma unroll
        for (int k = 0; k < 3; ++k) p.d[k] += (long long)block * 3 * n;
        p.out += (long long)block * p.m;
    }
    // a wave with no vector at all leaves (the exchange buffer is private to the wave: no barrier waits for it)
    if (wvec >= p.batch) return;

    __shared__ float4 lds_store[G::WAVES * G::TPW * G::VEC_WORDS / 4];
    float* w = reinterpret_cast<float*>(lds_store) + (wave * G::TPW + g) * G::VEC_WORDS;
    float4* pa = ar_ptr_a<G>(w, l);
    float* pb = ar_ptr_b<G>(w, l);
    constexpr int W = n / 64 < 4 ? 4 : n / 64;      // sign words per diagonal
    const unsigned long long* hw = p.sw[0] + 3 * W; // lane masks behind the triple's sign words: [3 diagonals][2 layouts][R]
    const int ebase = ar_base_b<G>(l);              // layout B: register j holds coordinate ebase + (j << r)
    const long long so = p.sin_off;

    {
        const long long vec = wvec + g;
        const bool active = vec < p.batch;
        double v[R];
        ArDiagA<G> da;
        ArDiagB<G> db;
        // x: coalesced 16-byte loads, then through the buffer into layout A
        const float* src = p.x + (active ? vec : 0) * p.in_stride;
        const unsigned at = 4 * l;
        float* put = w + ar_word_of<G>(at);             // a lane's pieces lie 4 LANES floats apart, four rows of the buffer
        if constexpr (SIGNS) {          // each piece as it arrives (n = 1024, 30000 vectors 68.7 -> 67.4 us, n = 4096 alike)
            src += at;
#pragma unroll
            for (int k = 0; k < R / 4; ++k) {
                const float4 t = load4<true>(src + 4 * k * G::LANES);      // a vector past the end reads the first one
                *reinterpret_cast<float4*>(w + ar_word_of<G>(4 * (k * G::LANES + l))) = t;
            }
        } else {
            float4 t[R / 4];
#pragma unroll
            for (int k = 0; k < R / 4; ++k) t[k] = load4<!BLOCKS>(src + 4 * k * G::LANES + at);
            da.load(p.d[0], at);
#pragma unroll
            for (int k = 0; k < R / 4; ++k) *reinterpret_cast<float4*>(put + 4 * k * G::STRIDE) = t[k];
        }
        wave_lds_fence();
#pragma unroll
        for (int k = 0; k < R / 4; ++k) {
            const float4 f = pa[k];
            v[4 * k] = (double)f.x; v[4 * k + 1] = (double)f.y; v[4 * k + 2] = (double)f.z; v[4 * k + 3] = (double)f.w;
        }
        wave_lds_fence();

        // D1 in layout A, D2 in layout B, D3 in layout A
        if constexpr (SIGNS) feat_ar_flip<G>(v, hw);
        else da.multiply(v, put, pa);
        ar_stages<G>(v);
        if constexpr (WORDS) feat_ar_a_to_b_words<G>(v, w, l); else feat_ar_a_to_b<G>(v, pa, pb);
        if constexpr (!SIGNS) db.load(p.d[1], ebase);
        ar_stages<G>(v);
        if constexpr (SIGNS) feat_ar_flip<G>(v, hw + 3 * R);
        else db.multiply(v);
        ar_stages<G>(v);
        feat_ar_b_to_a<G>(v, pa, pb);
        if constexpr (!SIGNS) da.load(p.d[2], at);
        ar_stages<G>(v);
        if constexpr (SIGNS) feat_ar_flip<G>(v, hw + 4 * R);
        else da.multiply(v, put, pa);
        ar_stages<G>(v);
        if constexpr (WORDS) feat_ar_a_to_b_words<G>(v, w, l); else feat_ar_a_to_b<G>(v, pa, pb);
        ar_stages<G>(v);

        float* dst = p.out + (active ? vec : 0) * p.out_stride + ebase;
        if (p.m == n) {                         // every coordinate is kept: straight-line stores
#pragma unroll
            for (int j = 0; j < R; ++j) {
                float sn, cs;
                feature_sincos(v[j], p, 0.0f, sn, cs);
                if (G::TPW == 1 || active) {
                    store1<STREAM>(dst + (j << r), cs * p.inv_sqrt_m);
                    store1<STREAM>(dst + so + (j << r), sn * p.inv_sqrt_m);
                }
            }
        } else {
            const int m = active ? p.m : 0;
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if ((j << r) >= p.m) return;      // no lane has another coordinate to keep (n = 4096, batch 4096, m = 512 37.8 -> 35.3 us)
                float sn, cs;
                feature_sincos(v[j], p, 0.0f, sn, cs);
                if (ebase + (j << r) < m) {
                    store1<STREAM>(dst + (j << r), cs * p.inv_sqrt_m);
                    store1<STREAM>(dst + so + (j << r), sn * p.inv_sqrt_m);
                }
            }
        }
    }
}

// one wave per workgroup (each wave owns its vectors and its exchange buffer): measured 3-4 % faster than two
constexpr int kFeatureArWaves = 1;
template <int NT>
static bool feature_ar_streams(int m) { return NT != 10 || (m & 31) == 0 || m < (1 << NT) / 2; }
// n = 2^13, 2^14 without the limit of 128 registers (launch.hpp), for batches of at most one tile per compute unit: nothing is gained from more of
// them there, and lane stages in larger batches wait less often (at 2^14 the limit also spills one or two registers).  With / without the limit, in us:
// 2^14, fp32 diagonals, m = n, batch 64 16.4 / 15.9, 256 20.2 / 19.9, m = 1001, 256 18.3 / 17.1, sign words, m = n, 64 16.3 / 16.0, m = 1001, 256 17.5 / 17.1;
// 2^13, fp32 diagonals, m = n, 64 10.1 / 10.0, 256 11.6 / 11.4, m = 500, 256 9.9 / 9.8, but two and three tiles per compute unit: m = n, 400 15.5 / 15.9, 700
// 20.7 / 21.3, m = 500, 512 14.0 / 14.5, 768 18.2 / 19.1
struct FeatureFewTuning : NotWide { static constexpr int rmax = 5, waves = 4, min_waves = 0, trips = 0; };
template <int NT, bool SIGNS>
static hipError_t launch_cossin(const TileParams& p, long long tiles, hipStream_t s)
{
    if constexpr (feature_ar_log2r(NT) != 0) {
        using GA = HashArGeom<NT, feature_ar_log2r(NT), kFeatureArWaves>;
        const long long blocks = (tiles + GA::VECS_PER_WG - 1) / GA::VECS_PER_WG;
        if (blocks <= 0) return hipSuccess;
        if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
        const auto kernel = feature_ar_streams<NT>(p.m) ? spinner_feature_ar_kernel<GA, SIGNS, true> : spinner_feature_ar_kernel<GA, SIGNS, NT != 10>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(GA::THREADS), 0, s, p, 1);
        return hipGetLastError();
    } else {
        if constexpr (NT == 14 || (NT == 13 && !SIGNS)) {
            if (tiles <= kComputeUnits)
                return launch_tile<double, NT, NT, 3, true, EPI_STORE_COSSIN, SIGNS, 0, true, GeomFrom<FeatureFewTuning, NT>>(p, tiles, s);
        }
        return launch_tile<double, NT, NT, 3, true, EPI_STORE_COSSIN, SIGNS>(p, tiles, s);
    }
}

// p as for one block (out_stride = the whole row, sin_off = L m, inv_sqrt_m = 1 / sqrt(L m))
template <int NT>
static hipError_t launch_feature_blocks_nt(const TileParams& p, const float* diag_sets, int L, hipStream_t s)
{
    using GA = HashArGeom<NT, feature_ar_log2r(NT), kFeatureArWaves>;
    const auto kernel = feature_ar_streams<NT>(p.m) ? spinner_feature_ar_kernel<GA, false, true, true> : spinner_feature_ar_kernel<GA, false, NT != 10, true>;
    // one workgroup per block and group of vectors, in slices of at most 2^24 workgroups (a grid holds 2^32 threads)
    for (int l0 = 0; l0 < L; l0 += 1 << 21) {
        const int nl = L - l0 < (1 << 21) ? L - l0 : 1 << 21;
        const long long slice = (long long)((1 << 21) / nl) * 8 * GA::VECS_PER_WG;
        TileParams q = p;
        for (int k = 0; k < 3; ++k) q.d[k] = diag_sets + ((3LL * l0 + k) << NT);
        for (long long b0 = 0; b0 < p.batch; b0 += slice) {
            q.batch = p.batch - b0 < slice ? p.batch - b0 : slice;
            q.x = p.x + b0 * p.in_stride;
            q.out = p.out + b0 * p.out_stride + (long long)l0 * p.m;
            const long long groups = (q.batch + GA::VECS_PER_WG - 1) / GA::VECS_PER_WG;
            hipLaunchKernelGGL(kernel, dim3((unsigned)(8 * ((groups + 7) / 8) * nl)), dim3(GA::THREADS), 0, s, q, nl);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}
hipError_t launch_feature_blocks_ar(int log2n, const TileParams& p, const float* diag_sets, int L, hipStream_t s)
{
    switch (log2n) {
    case 10: return launch_feature_blocks_nt<10>(p, diag_sets, L, s);
    case 12: return launch_feature_blocks_nt<12>(p, diag_sets, L, s);
    default: return hipErrorInvalidValue;
    }
}

#define CASE(NT) case NT: return signs ? launch_cossin<NT, true>(p, tiles, s) : launch_cossin<NT, false>(p, tiles, s);
// n = 2^15, 2^16: fp64 values do not fit a compute unit; fp32 butterflies on the plain kernels' geometries.  At 2^16 sine and cosine
// beside 64 values in 128 registers spill 27 of them (92 bytes per thread with sign words, 100 with fp32 diagonals); 2^15 none
#define WIDECASE(NT) case NT: return signs ? launch_tile<float, NT, NT, 3, true, EPI_STORE_COSSIN, true>(p, tiles, s) \
                                           : launch_tile<float, NT, NT, 3, true, EPI_STORE_COSSIN, false>(p, tiles, s);
hipError_t launch_fused_cossin(int log2n, bool signs, const TileParams& p, long long tiles, hipStream_t s)
{
    switch (log2n) {
        CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14)
        WIDECASE(15) WIDECASE(16)
    default: return hipErrorInvalidValue;
    }
}
#undef WIDECASE
#undef CASE
}  // namespace spinner
