// G_struct D2 H D1 x for n = 2^9 .. 2^14 in one kernel: Hadamard stages, forward transforms, spectrum product and
// inverse transforms of two vectors (the real and imaginary parts of n complex points) with every stage between
// registers and one trip through LDS per group of index bits.
//
// The 2n-point cyclic convolution of a Toeplitz, Hankel or skew-circulant block splits exactly: the first
// decimation-in-frequency stage of the zero-padded input only copies it (even frequencies: a cyclic transform of n
// points) and multiplies it by exp(-i pi k / n) (odd frequencies: a skew-cyclic transform of n points).  So the block
// is two n-point convolutions whose results are added, and the spectrum as the preparation leaves it (bit-reversed
// order) holds the cyclic one in its first half and the skew one in its second.  Both run in the same n-point buffer,
// one after the other.
//
// The n = 2^LOGN points are three groups of index bits (B0 top, B1, B2 low; at most r = log2 R each).  In the phase of
// a group every thread holds R points that differ in that group's bits (and, if it has fewer than r, in the top bits)
// and runs its stages between registers with constant twiddles; one factor exp(-2 pi i j q / 2^(lo + b)) per point
// (j the point's bits below the group, q its frequency in the group) joins a group to the next.  A phase reads and
// writes the same positions, so an exchange is: write, one barrier, read.  Hadamard phases run middle, low, top and the
// top one goes straight into the transform's top phase; the low phase holds the forward stages, the spectrum product
// and the inverse stages.  Six exchanges for a circulant block, ten for the others (the general kernel in
// structured.hip took ten and sixteen round trips at these sizes, of twice the points for the padded kinds: n = 4096,
// batch 16383, Toeplitz 315 -> 251 us).  n = 2^13 and 2^14 are held to two waves per SIMD and the padded kinds spill 100 and 72
// bytes per thread there (2^10 and 2^11: 16 and 20).
#include "launch.hpp"
#include "allreg.hpp"
namespace spinner {

struct StructFftParams {
    const float* x;        // [batch][n]
    const float* d1;       // [n]
    const float* d2;       // [n]
    const float2* spec;    // [P] spectrum in bit-reversed order, P = n or 2n
    const float2* tw;      // [P/2] exp(-2 pi i k / P)
    float* out;            // [batch][m]
    long long batch;
    int m, reverse;
    float factor;
};

namespace fft {

struct alignas(8) C { float x, y; };
__device__ __forceinline__ C mul(C a, C b) { return {__builtin_fmaf(-a.y, b.y, a.x * b.x), __builtin_fmaf(a.x, b.y, a.y * b.x)}; }
__device__ __forceinline__ C mul_conj(C a, C b) { return {__builtin_fmaf(a.y, b.y, a.x * b.x), __builtin_fmaf(-a.x, b.y, a.y * b.x)}; }

// cos(2 pi K / 32) and sin(2 pi K / 32), K = 0 .. 8
constexpr float kCos32[9] = {1.0f, 0.98078528040323044f, 0.92387953251128676f, 0.83146961230254524f, 0.70710678118654752f,
                             0.55557023301960222f, 0.38268343236508977f, 0.19509032201612827f, 0.0f};
constexpr float cos32(int k) { return k <= 8 ? kCos32[k] : -kCos32[16 - k]; }      // k = 0 .. 16
constexpr float sin32(int k) { return k <= 8 ? kCos32[8 - k] : kCos32[k - 8]; }

// a * exp(-2 pi i K / 32) (CONJ: exp(+2 pi i K / 32)), K = 0 .. 15
template <int K, bool CONJ>
__device__ __forceinline__ C rot32(C a)
{
    constexpr float h = 0.70710678118654752f;
    if constexpr (K == 0) return a;
    else if constexpr (K == 8) { if constexpr (CONJ) return {-a.y, a.x}; else return {a.y, -a.x}; }
    else if constexpr (K == 4) { if constexpr (CONJ) return {(a.x - a.y) * h, (a.x + a.y) * h}; else return {(a.x + a.y) * h, (a.y - a.x) * h}; }
    else if constexpr (K == 12) { if constexpr (CONJ) return {(a.x + a.y) * -h, (a.x - a.y) * h}; else return {(a.y - a.x) * h, (a.x + a.y) * -h}; }
    else {
        constexpr float c = cos32(K), s = sin32(K);
        if constexpr (CONJ) return {__builtin_fmaf(a.y, -s, a.x * c), __builtin_fmaf(a.x, s, a.y * c)};
        else return {__builtin_fmaf(a.y, s, a.x * c), __builtin_fmaf(a.x, -s, a.y * c)};
    }
}

constexpr int bit_reverse(int v, int bits)
{
    int r = 0;
    for (int i = 0; i < bits; ++i) r |= ((v >> i) & 1) << (bits - 1 - i);
    return r;
}

// Index bits of the three groups and the points per thread, by size
template <int LOGN> struct Plan;
template <> struct Plan<9>  { static constexpr int r = 3, b[3] = {3, 3, 3}; };
template <> struct Plan<10> { static constexpr int r = 4, b[3] = {4, 3, 3}; };
template <> struct Plan<11> { static constexpr int r = 4, b[3] = {4, 4, 3}; };
template <> struct Plan<12> { static constexpr int r = 4, b[3] = {4, 4, 4}; };
template <> struct Plan<13> { static constexpr int r = 5, b[3] = {5, 4, 4}; };
template <> struct Plan<14> { static constexpr int r = 5, b[3] = {5, 5, 4}; };

template <int LOGN>
struct Geo {
    static constexpr int r = Plan<LOGN>::r, R = 1 << r, N = 1 << LOGN, T = N >> r;
    static constexpr int bits(int g) { return Plan<LOGN>::b[g]; }
    static constexpr int lo(int g) { return g == 2 ? 0 : (g == 1 ? Plan<LOGN>::b[2] : Plan<LOGN>::b[2] + Plan<LOGN>::b[1]); }
    // the part of a point's index that register k contributes in the phase of group g
    static constexpr int reg_index(int g, int k)
    {
        const int b = bits(g), e = r - b;
        return ((k & ((1 << b) - 1)) << lo(g)) | ((k >> b) << (LOGN - e));
    }
    // the part that the thread contributes
    static constexpr __host__ __device__ __forceinline__ int base_index(int g, int t) { return (t & ((1 << lo(g)) - 1)) | ((t >> lo(g)) << (lo(g) + bits(g))); }
    // one unused 8-byte slot after every 16 points keeps the strided accesses of a phase on different banks; index
    // parts with disjoint bits add up, so a register's part of the address is a constant
    static constexpr __host__ __device__ int pad(int i) { return i + (i >> 4); }
    // the wave id stands for the same index bits in both phases: a wave then reads what it wrote itself
    static constexpr bool within_waves(int from, int to)
    {
        for (int bit = 64; bit < T; bit <<= 1)
            if (base_index(from, bit) != base_index(to, bit)) return false;
        return true;
    }
    static constexpr int LDS_POINTS = N + N / 16;
};

// 2^B points of each of the R >> B sub-transforms a thread holds: natural order in, bit-reversed out
template <int B, int R>
__device__ __forceinline__ void forward_regs(C (&v)[R])
{
    static_for<0, B>([&](auto st) {
        constexpr int s = B - 1 - st.value;                   // register bit of this stage
        static_for<0, R>([&](auto kk) {
            constexpr int k = kk.value;
            if constexpr (!(k & (1 << s))) {
                const C a = v[k], c = v[k | (1 << s)];
                v[k] = {a.x + c.x, a.y + c.y};
                v[k | (1 << s)] = rot32<(k & ((1 << s) - 1)) * (16 >> s), false>(C{a.x - c.x, a.y - c.y});
            }
        });
    });
}
template <int B, int R>
__device__ __forceinline__ void inverse_regs(C (&v)[R])
{
    static_for<0, B>([&](auto st) {
        constexpr int s = st.value;
        static_for<0, R>([&](auto kk) {
            constexpr int k = kk.value;
            if constexpr (!(k & (1 << s))) {
                const C c = rot32<(k & ((1 << s) - 1)) * (16 >> s), true>(v[k | (1 << s)]);
                const C a = v[k];
                v[k] = {a.x + c.x, a.y + c.y};
                v[k | (1 << s)] = {a.x - c.x, a.y - c.y};
            }
        });
    });
}
template <int B, int R>
__device__ __forceinline__ void hadamard_regs(C (&v)[R])
{
#pragma unroll
    for (int s = 0; s < B; ++s)
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (!(k & (1 << s))) {
                const C a = v[k], c = v[k | (1 << s)];
                v[k] = {a.x + c.x, a.y + c.y};
                v[k | (1 << s)] = {a.x - c.x, a.y - c.y};
            }
}

// Multiplies point bit_reverse(q) by the product of the powers p2[i] with bit i of q set (times w), for every q: a walk
// down the bits of q, so that only one factor per bit is held at a time.  UNIT: w is 1.
template <int R, int B, int LEFT, int Q, bool INVERSE, bool UNIT>
__device__ __forceinline__ void join_walk(C (&v)[R], const C (&p2)[B], C w)
{
    if constexpr (LEFT == 0) {
        if constexpr (!UNIT) {
            static_for<0, (R >> B)>([&](auto s) {
                constexpr int k = bit_reverse(Q, B) | (s.value << B);
                v[k] = INVERSE ? mul_conj(v[k], w) : mul(v[k], w);
            });
        }
    } else {
        join_walk<R, B, LEFT - 1, Q, INVERSE, UNIT>(v, p2, w);
        C u = p2[LEFT - 1];
        if constexpr (!UNIT) u = mul(w, u);
        join_walk<R, B, LEFT - 1, Q | (1 << (LEFT - 1)), INVERSE, false>(v, p2, u);
    }
}

// The factors that join group g to the group below: point (q, j) times exp(-2 pi i j q / 2^(lo + b)), q the frequency
// that sits at position bit_reverse(q); SKEW: times exp(-2 pi i j / 2n) as well (see the skew transform below).  The
// powers of two of the base come from the table, the others are products of at most B - 1 of them.  The table is asked
// a phase ahead of the use.
template <typename G, int g, bool SKEW>
struct JoinFactors {
    static constexpr int b = G::bits(g), lo = G::lo(g);
    static_assert(lo > 0, "nothing joins the lowest group");
    C p2[b], base;
    __device__ __forceinline__ void load(const float2* __restrict__ tw, int log2p, int t)
    {
        // an opaque copy per call: kept from one of a kernel's up to four uses of a group to the next (as the compiler
        // would), the factors take the registers of the points
        int j = t & ((1 << lo) - 1);
        asm volatile("" : "+v"(j));
        const int sh = log2p - lo - b;
#pragma unroll
        for (int i = 0; i < b; ++i) {
            const float2 f = tw[(j << i) << sh];
            p2[i] = {f.x, f.y};
        }
        base = {1.0f, 0.0f};
        if constexpr (SKEW) {
            const float2 f = tw[j];                           // table of 2n points: exp(-2 pi i j / 2n)
            base = {f.x, f.y};
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    template <bool INVERSE>
    __device__ __forceinline__ void apply(C (&v)[G::R]) const
    {
        join_walk<G::R, b, b, 0, INVERSE, !SKEW>(v, p2, base);
        __builtin_amdgcn_sched_barrier(0);
    }
};

// Registers of group FROM's phase to those of group TO's.  A thread writes the positions that it read in the exchange before, so
// one barrier is enough, and none where the data stay within the waves.
template <typename G, int FROM, int TO>
__device__ __forceinline__ void exchange(C (&v)[G::R], C* X, int t)
{
    C* a = X + G::pad(G::base_index(FROM, t));
    static_for<0, G::R>([&](auto k) { a[G::pad(G::reg_index(FROM, k.value))] = v[k.value]; });
    if constexpr (G::within_waves(FROM, TO)) wave_lds_fence();
    else __syncthreads();
    const C* c = X + G::pad(G::base_index(TO, t));
    static_for<0, G::R>([&](auto k) { v[k.value] = c[G::pad(G::reg_index(TO, k.value))]; });
    __builtin_amdgcn_sched_barrier(0);
}

// v (natural order, top phase) convolved with the part of the spectrum at `spec`: cyclic, or skew-cyclic with
// exp(-i pi k / n) on point k before and its conjugate after.  k = j + q0 2^lo0, so that factor is a constant power of
// exp(-i pi / 2^B0) per register times exp(-i pi j / n), which the joining factors of the top group take along.
template <typename G, bool SKEW>
__device__ __forceinline__ void convolve(C (&v)[G::R], C* X, const float2* __restrict__ spec, const float2* __restrict__ tw, int log2p, int t)
{
    constexpr int B0 = G::bits(0), B1 = G::bits(1), B2 = G::bits(2);
    if constexpr (SKEW) {
        static_assert(B0 >= 3 && B0 <= 5, "constant factors exp(-i pi k / 2^B0)");
        if constexpr (B0 <= 4) {
            static_for<0, G::R>([&](auto k) { v[k.value] = rot32<k.value * (16 >> B0), false>(v[k.value]); });
        } else {
            // powers of exp(-i pi / 32): an even one is in the table of constants, an odd one times the first
            constexpr float c1 = 0.99518472667219689f, s1 = 0.09801714032956060f;
            static_for<0, G::R>([&](auto k) {
                C u = rot32<k.value / 2, false>(v[k.value]);
                if constexpr (k.value & 1) u = {__builtin_fmaf(u.y, s1, u.x * c1), __builtin_fmaf(u.x, -s1, u.y * c1)};
                v[k.value] = u;
            });
        }
    }
    JoinFactors<G, 0, SKEW> f0;
    JoinFactors<G, 1, false> f1;
    f0.load(tw, log2p, t);
    forward_regs<B0>(v);
    f0.template apply<false>(v);
    f1.load(tw, log2p, t);
    exchange<G, 0, 1>(v, X, t);
    forward_regs<B1>(v);
    f1.template apply<false>(v);
    exchange<G, 1, 2>(v, X, t);
    forward_regs<B2>(v);
    {
        // a thread's points of the low phase are runs of 2^B2 consecutive ones: 16-byte loads of two spectrum points
        const float2* s = spec + G::base_index(2, t);
        static_for<0, G::R / 2>([&](auto k2) {
            const float4 f = *reinterpret_cast<const float4*>(s + G::reg_index(2, 2 * k2.value));
            v[2 * k2.value] = mul(v[2 * k2.value], C{f.x, f.y});
            v[2 * k2.value + 1] = mul(v[2 * k2.value + 1], C{f.z, f.w});
            if constexpr ((k2.value & 3) == 3) __builtin_amdgcn_sched_barrier(0);
        });
    }
    inverse_regs<B2>(v);
    f1.load(tw, log2p, t);
    exchange<G, 2, 1>(v, X, t);
    f1.template apply<true>(v);
    f0.load(tw, log2p, t);
    inverse_regs<B1>(v);
    exchange<G, 1, 0>(v, X, t);
    f0.template apply<true>(v);
    inverse_regs<B0>(v);
    if constexpr (SKEW) {
        if constexpr (B0 <= 4) {
            static_for<0, G::R>([&](auto k) { v[k.value] = rot32<k.value * (16 >> B0), true>(v[k.value]); });
        } else {
            constexpr float c1 = 0.99518472667219689f, s1 = 0.09801714032956060f;
            static_for<0, G::R>([&](auto k) {
                C u = rot32<k.value / 2, true>(v[k.value]);
                if constexpr (k.value & 1) u = {__builtin_fmaf(u.y, -s1, u.x * c1), __builtin_fmaf(u.x, s1, u.y * c1)};
                v[k.value] = u;
            });
        }
    }
}
}  // namespace fft

// HALVES: the padded kinds (P = 2n); else a circulant (P = n)
template <int LOGN, bool HALVES>
__global__ void __launch_bounds__(fft::Geo<LOGN>::T) __attribute__((amdgpu_waves_per_eu(fft::Geo<LOGN>::R == 32 ? 2 : 4)))
struct_fft_kernel(StructFftParams p)
{
    using G = fft::Geo<LOGN>;
    using fft::C;
    constexpr int N = G::N, R = G::R, LOGP = LOGN + (HALVES ? 1 : 0);
    extern __shared__ char lds_bytes[];
    C* X = reinterpret_cast<C*>(lds_bytes);
    const int t = threadIdx.x;
    const long long v0 = 2LL * blockIdx.x, v1 = v0 + 1;
    const bool two = v1 < p.batch;
    C v[R];
    {
        const int e = G::base_index(1, t);
        const float* __restrict__ x0 = p.x + v0 * N + e;
        const float* __restrict__ x1 = p.x + (two ? v1 : v0) * N + e;      // a lone last vector is read twice, its copy dropped
        const float* __restrict__ d1 = p.d1 + e;
        // Hankel: G acts on the reversed vector.  Reversing the 2^LOGN outputs of a Hadamard transform (complementing
        // every index bit) is flipping the inputs of odd parity.
        const unsigned flip = p.reverse ? 0x80000000u : 0u;
        const unsigned par = (__popc(e) & 1) ? flip : 0u;
        static_for<0, R>([&](auto k) {
            constexpr int i = G::reg_index(1, k.value);
            constexpr bool odd = __builtin_parity(i) != 0;
            const float d = __uint_as_float(__float_as_uint(d1[i]) ^ (odd ? par ^ flip : par));
            v[k.value] = {x0[i] * d, x1[i] * d};
        });
    }
    fft::hadamard_regs<G::bits(1)>(v);
    fft::exchange<G, 1, 2>(v, X, t);
    fft::hadamard_regs<G::bits(2)>(v);
    fft::exchange<G, 2, 0>(v, X, t);
    fft::hadamard_regs<G::bits(0)>(v);
    {
        const int e = G::base_index(0, t);
        const float* __restrict__ d2 = p.reverse ? p.d2 + (N - 1 - e) : p.d2 + e;
        float d[R];
        if (p.reverse) static_for<0, R>([&](auto k) { d[k.value] = d2[-G::reg_index(0, k.value)]; });
        else static_for<0, R>([&](auto k) { d[k.value] = d2[G::reg_index(0, k.value)]; });
        static_for<0, R>([&](auto k) { v[k.value].x *= d[k.value]; v[k.value].y *= d[k.value]; });
    }
    if constexpr (HALVES) {
        C u[R];
        static_for<0, R>([&](auto k) { u[k.value] = v[k.value]; });
        fft::convolve<G, false>(u, X, p.spec, p.tw, LOGP, t);
        fft::convolve<G, true>(v, X, p.spec + N, p.tw, LOGP, t);
        static_for<0, R>([&](auto k) { v[k.value].x += u[k.value].x; v[k.value].y += u[k.value].y; });
    } else {
        fft::convolve<G, false>(v, X, p.spec, p.tw, LOGP, t);
    }
    const int e = G::base_index(0, t);
    // The non-temporal hint on the stores, without / with it, Toeplitz, in us: n = 4096, 2^22 elements 20.6 / 18.3, 2^24 61.3 /
    // 59.5, 2^26 280 / 243; rows that are no whole lines, m = 4095 21.0 / 18.6, 64.2 / 64.2, 258 / 231, m = 2561 19.2 / 18.6,
    // 61.4 / 63.5, 246 / 214, n = 2^14, m = 16383 41.9 / 41.3, 89.7 / 94.8, 359 / 344.  With a reader of the result behind it the
    // two differ by less than 5 % either way.
    float* o0 = p.out + v0 * p.m;
    float* o1 = o0 + p.m;
    static_for<0, R>([&](auto k) {
        const int i = e + G::reg_index(0, k.value);
        if (i < p.m) {
            __builtin_nontemporal_store(v[k.value].x * p.factor, o0 + i);
            if (two) __builtin_nontemporal_store(v[k.value].y * p.factor, o1 + i);
        }
    });
}

template <int LOGN, bool HALVES>
static hipError_t launch_struct_fft_nt(const StructFftParams& p, hipStream_t s)
{
    using G = fft::Geo<LOGN>;
    constexpr size_t lds = (size_t)G::LDS_POINTS * sizeof(fft::C);
    const long long blocks = (p.batch + 1) / 2;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    if constexpr (lds > 65536) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(struct_fft_kernel<LOGN, HALVES>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((struct_fft_kernel<LOGN, HALVES>), dim3((unsigned)blocks), dim3(G::T), lds, s, p);
    return hipGetLastError();
}

#define CASE(NT) case NT: return log2p > NT ? launch_struct_fft_nt<NT, true>(p, s) : launch_struct_fft_nt<NT, false>(p, s);
hipError_t launch_struct_fft(const float* x, const float* d1, const float* d2, const float2* spec, const float2* tw, float* out,
                             long long batch, int log2n, int log2p, int m, int reverse, float factor, hipStream_t s)
{
    if (batch <= 0) return hipSuccess;
    const StructFftParams p{x, d1, d2, spec, tw, out, batch, m, reverse, factor};
    switch (log2n) {
        CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14)
    default: return hipErrorInvalidValue;
    }
}
#undef CASE
}  // namespace spinner
