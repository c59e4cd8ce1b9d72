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
// and runs its stages between registers, every butterfly with its twiddle in six fused operations (see "Twiddles").  A phase
// reads and writes the same positions, so an exchange is: write, one barrier, read.  Hadamard phases run middle, low, top and the
// top one goes straight into the transform's top phase; the low phase holds the forward stages, the spectrum product
// and the inverse stages.  Six exchanges for a circulant block, ten for the others.  Bound by vector-ALU issue (3214 instructions per
// thread and pair of vectors at n = 2^12, padded, 0.24 per cycle and SIMD of about 0.4 with 3.7 waves there) and what the exchanges leave
// exposed (LDS pipe 38 % busy, a quarter of the waves' time waiting for anything but issue).
// In us, Toeplitz: the general kernel in structured.hip / twiddles between the groups as factors of every point / this form: n = 4096,
// batch 16383 315 / 244 / 226; n = 2^13, 8192 - / 306 / 250, 1024 - / 43.5 / 35.2; n = 2^14, 4096 - / 351 / 305; n = 2048, 32768 - / 226 / 201.
// n = 2^13 and 2^14 are held to two waves per SIMD.
#pragma once
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

// cos(2 pi K / 64), K = 0 .. 16
constexpr float kCos64[17] = {1.0f, 0.99518472667219689f, 0.98078528040323044f, 0.95694033573220886f, 0.92387953251128676f,
                              0.88192126434835503f, 0.83146961230254524f, 0.77301045336273696f, 0.70710678118654752f,
                              0.63439328416364550f, 0.55557023301960222f, 0.47139673682599764f, 0.38268343236508977f,
                              0.29028467725446236f, 0.19509032201612827f, 0.09801714032956060f, 0.0f};
constexpr float cos64(int k) { return k <= 16 ? kCos64[k] : -kCos64[32 - k]; }      // k = 0 .. 32
constexpr float sin64(int k) { return k <= 16 ? kCos64[16 - k] : kCos64[k - 16]; }

// cos a - 1 and sin a for angles up to pi / 16: what the series leave out is below 1e-13
constexpr double cosm1_near_0(double a) { return -a * a / 2 * (1.0 - a * a / 12 * (1.0 - a * a / 30 * (1.0 - a * a / 56))); }
constexpr double sin_near_0(double a) { return a * (1.0 - a * a / 6 * (1.0 - a * a / 20 * (1.0 - a * a / 42))); }

// a * exp(-2 pi i K / 64) (CONJ: exp(+2 pi i K / 64)), K = 0 .. 31
template <int K, bool CONJ>
__device__ __forceinline__ C rot64(C a)
{
    constexpr float h = 0.70710678118654752f;
    if constexpr (K == 0) return a;
    else if constexpr (K == 16) { if constexpr (CONJ) return {-a.y, a.x}; else return {a.y, -a.x}; }
    else if constexpr (K == 8) { if constexpr (CONJ) return {(a.x - a.y) * h, (a.x + a.y) * h}; else return {(a.x + a.y) * h, (a.y - a.x) * h}; }
    else if constexpr (K == 24) { if constexpr (CONJ) return {(a.x + a.y) * -h, (a.x - a.y) * h}; else return {(a.y - a.x) * h, (a.x + a.y) * -h}; }
    else {
        constexpr float c = cos64(K), s = sin64(K);
        if constexpr (CONJ) return {__builtin_fmaf(a.y, -s, a.x * c), __builtin_fmaf(a.x, s, a.y * c)};
        else return {__builtin_fmaf(a.y, s, a.x * c), __builtin_fmaf(a.x, -s, a.y * c)};
    }
}

// (a, c) -> (a + w c, a - w c) (CONJ: with the conjugate of w) in six fused operations, the difference as 2 a minus the sum, or
// (APART) in eight, without the sum's rounding in it
template <bool CONJ, bool APART = false>
__device__ __forceinline__ void butterfly(C& a, C& c, C w)
{
    const float wy = CONJ ? -w.y : w.y;
    const C u = {__builtin_fmaf(w.x, c.x, __builtin_fmaf(-wy, c.y, a.x)), __builtin_fmaf(w.x, c.y, __builtin_fmaf(wy, c.x, a.y))};
    if constexpr (APART)
        c = {__builtin_fmaf(-w.x, c.x, __builtin_fmaf(wy, c.y, a.x)), __builtin_fmaf(-w.x, c.y, __builtin_fmaf(-wy, c.x, a.y))};
    else
        c = {__builtin_fmaf(2.0f, a.x, -u.x), __builtin_fmaf(2.0f, a.y, -u.y)};
    a = u;
}
// the same with w = exp(-2 pi i K / 64), K = 0 .. 31; four additions where w is 1 or -i
template <int K, bool CONJ>
__device__ __forceinline__ void butterfly_const(C& a, C& c)
{
    if constexpr (K == 0 || K == 16) {
        const C t = rot64<K, CONJ>(c), b = a;
        a = {b.x + t.x, b.y + t.y};
        c = {b.x - t.x, b.y - t.y};
    } else if constexpr (K == 8 || K == 24) {
        constexpr float h = K == 8 ? 0.70710678118654752f : -0.70710678118654752f;
        const C t = (K == 8) != CONJ ? C{c.x + c.y, c.y - c.x} : C{c.x - c.y, c.x + c.y}, b = a;
        a = {__builtin_fmaf(h, t.x, b.x), __builtin_fmaf(h, t.y, b.y)};
        c = {__builtin_fmaf(-h, t.x, b.x), __builtin_fmaf(-h, t.y, b.y)};
    } else {
        butterfly<CONJ>(a, c, C{cos64(K), -sin64(K)});
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
    static constexpr int LOGN_ = LOGN, r = Plan<LOGN>::r, R = 1 << r, N = 1 << LOGN, T = N >> r;
    static constexpr int bits(int g) { return Plan<LOGN>::b[g]; }
    static constexpr int lo(int g) { return g == 2 ? 0 : (g == 1 ? Plan<LOGN>::b[2] : Plan<LOGN>::b[2] + Plan<LOGN>::b[1]); }
    // the part of a point's index that register k contributes in the phase of group g
    static constexpr int reg_index(int g, int k)
    {
        const int b = bits(g), e = r - b;
        return ((k & ((1 << b) - 1)) << lo(g)) | ((k >> b) << (LOGN - e));
    }
    // The part that the thread contributes.  In the two lower phases the wave id stands for bits 4 and up of the thread's
    // number, below the lanes' upper two: a wave then reads its factors of the low phase, which lie in the table in the
    // order of reversed bits, in runs of four.
    static constexpr __host__ __device__ __forceinline__ int placed(int t)
    {
        constexpr int waves = T / 64;
        return waves <= 1 ? t : (t & 15) | (t >> 6) << 4 | ((t >> 4) & 3) * (waves << 4);
    }
    static constexpr __host__ __device__ __forceinline__ int base_index(int g, int t)
    {
        const int p = g ? placed(t) : t;
        return (p & ((1 << lo(g)) - 1)) | ((p >> lo(g)) << (lo(g) + bits(g)));
    }
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

// Where the two results of a butterfly are formed apart (eight fused operations), so that the sum's rounding does not enter the
// difference: as far as it takes for the convolution's error to be no larger than with one factor per point between the phases.
// Error over 2^26 values in units of 1e-7 of the norm, that form / this one / this one without any phase apart but, of a
// circulant, the last (512: the middle too, and a factor by squaring): circulant 2^9 1.735 / 1.728 / 1.789, 2^10 1.945 / 1.935 / 1.983, 2^11 2.129 /
// 2.112 / 2.112, 2^12 2.210 / 2.202 / 2.238, 2^13 2.408 / 2.399 / 2.451, 2^14 2.594 / 2.593 / 2.599; Toeplitz 2^9 1.919 / 1.913 / 1.946, 2^10 2.150 /
// 2.146 / 2.167, 2^11 2.325 / 2.316 / 2.316, 2^12 2.388 / 2.385 / 2.392, 2^13 2.625 / 2.529 / 2.529.
// CLOSE: up to 32 vectors of a padded kind of 2^13, which the general kernel (whose error is smaller there, 2.497 for Toeplitz) served
// before: 2.479 against 2.529 for the form of larger batches, 32 vectors 24.9 against 24.1 us (the general kernel 25.4).
template <typename G, bool PADDED, bool CLOSE>
struct Apart {
    static constexpr int n = G::LOGN_;
    static constexpr bool forward = CLOSE || (!PADDED && (n == 9 || n == 10 || n == 13));                   // forward, middle phase
    static constexpr bool low = PADDED ? n == 9 || n == 12 : n == 12 || n == 14;                            // forward, last stage of all
    static constexpr bool middle = CLOSE || (PADDED ? n <= 10 : n != 11 && n != 14), last = !PADDED;        // backward
};

// The second diagonal asked for two phases ahead of its use, the spectrum in two halves ahead of the low stages and ahead of the first products: where
// the registers of two waves per SIMD have room for it.  As they are needed / ahead, in us: 2^13 Toeplitz, 4096 vectors 120.3 / 112.6, circulant 83.1 /
// 75.8, skew-circulant, 30 vectors 25.0 / 23.0; 2^14 circulant, 2048 vectors 101.9 / 98.3, but Toeplitz 150.3 / 160.4.  Below, with
// four waves per SIMD: 2^12 Toeplitz, 16383 vectors 226.6 / 230.5, 2^11, 16384 86.9 / 103.8, 2^10, 32768 81.0 / 92.3, circulants 155.5 / 156.9, 58.1 / 58.0, 55.1 / 55.5.
template <typename G, bool PADDED>
constexpr bool asks_ahead = G::LOGN_ == 13 || (G::LOGN_ == 14 && !PADDED);

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

// Twiddles.  A transform forward runs from the top index bit down with the twiddle on the second input of a butterfly; stage t
// of all (0 at the top) has W = exp(-2 pi i (rev(beta) + shift) / 2^(t + 1)), beta the t bits above, which are transformed
// already, rev their reversal, shift 0 for the cyclic transform and 1/2 for the skew one, which needs no other factor.  Backward it
// runs from the bottom bit up with the conjugates of exp(-2 pi i j / 2^(s + 1)) on the second input, j the s bits below.  A
// thread's part of either is one factor per stage and group from the table; what its registers add is a constant turn.  The
// factors of a group are asked a phase ahead of the use.
template <typename G, int g, bool SKEW, bool PADDED>
struct ForwardTwiddles {
    static constexpr int b = G::bits(g), lo = G::lo(g), above = G::LOGN_ - lo - b, e = G::r - b;
    static_assert(g > 0 && e <= 1, "constants in the top group; at most one more index bit in the registers");
    // three bits in the low phase, padded kinds: the middle stage's factor is the last one's square, a scattered read less (n = 512,
    // batch 65536, Toeplitz 110 -> 102 us; with four bits and two squares the result's error would grow by 3 to 6 %, a circulant's by 2 %)
    static constexpr bool SQUARE = g == 2 && b == 3 && PADDED;
    C w[b];
    __device__ __forceinline__ void load(const float2* __restrict__ tw, int log2p, int t)
    {
        // an opaque copy per call: kept from one of a kernel's uses of a group to the next (as the compiler would), the
        // factors take the registers of the points
        unsigned beta = (unsigned)G::placed(t) >> lo;
        asm volatile("" : "+v"(beta));
        const unsigned rev = (__brev(beta) >> (32 - (above - e))) << e;
#pragma unroll
        for (int i = 0; i < b; ++i) {
            if (SQUARE && i == 1) continue;
            const float2 f = tw[SKEW ? (2 * rev + 1) << (log2p - above - 2 - i) : rev << (log2p - above - 1 - i)];
            w[i] = {f.x, f.y};
        }
        __builtin_amdgcn_sched_barrier(0);
    }
};
template <typename G, int g, bool SKEW>
struct InverseTwiddles {
    static constexpr int b = G::bits(g), lo = G::lo(g);
    static_assert(lo > 0, "constants in the lowest group");
    C w[b], base;
    __device__ __forceinline__ void load(const float2* __restrict__ tw, int log2p, int t)
    {
        int j = t & ((1 << lo) - 1);
        asm volatile("" : "+v"(j));
#pragma unroll
        for (int s = 0; s < b; ++s) {
            const float2 f = tw[j << (log2p - lo - s - 1)];
            w[s] = {f.x, f.y};
        }
        if constexpr (SKEW) {
            const float2 f = tw[j];                           // table of 2n points: exp(-2 pi i j / 2n)
            base = {f.x, f.y};
        }
        __builtin_amdgcn_sched_barrier(0);
    }
};

// The butterflies of one stage between registers FIRST + k and FIRST + (k | 2^s), k < 2^B, with twiddles w exp(-2 pi i q / 2^(D + 1)),
// q the value of the D bits of k that turn the factor: those above s, reversed (forward, D = B - 1 - s), or those below (backward,
// D = s).  Each turned factor is made once; those of the second half are -i times those of the first.
template <bool INVERSE, bool APART, int s, int B, int FIRST, int R>
__device__ __forceinline__ void turned_stage(C (&v)[R], C w)
{
    constexpr int D = INVERSE ? s : B - 1 - s, HALF = D ? 1 << (D - 1) : 1;
    static_for<0, HALF>([&](auto q) {
        const C u = rot64<(q.value << 5 >> D), false>(w);
        constexpr int first = FIRST + (INVERSE ? q.value : bit_reverse(q.value, D) << (s + 1));
        constexpr int second = FIRST + (INVERSE ? q.value + HALF : bit_reverse(q.value + HALF, D) << (s + 1));
#pragma unroll
        for (int m = 0; m < (1 << (B - 1 - D)); ++m) {
            const int k = m << (INVERSE ? s + 1 : 0);
            butterfly<INVERSE, APART>(v[first + k], v[(first + k) | (1 << s)], u);
            if constexpr (D > 0) butterfly<INVERSE, APART>(v[second + k], v[(second + k) | (1 << s)], C{u.y, -u.x});
        }
    });
}

// group 0 forward: constants alone
template <int B, bool SKEW, int R>
__device__ __forceinline__ void forward_top(C (&v)[R])
{
    static_assert((1 << B) == R, "the top group fills the registers");
    static_for<0, B>([&](auto st) {
        constexpr int s = B - 1 - st.value;
        static_for<0, R>([&](auto k) {
            constexpr int K = (bit_reverse(k.value >> (s + 1), st.value) << 5 >> st.value) + (SKEW ? 16 >> st.value : 0);
            if constexpr (!(k.value & (1 << s))) butterfly_const<K, false>(v[k.value], v[k.value | (1 << s)]);
        });
        if constexpr (R > 16) __builtin_amdgcn_sched_barrier(0);
    });
}
// APART: from this stage of the group on
template <int APART, typename G, int g, bool SKEW, bool PADDED>
__device__ __forceinline__ void forward_group(C (&v)[G::R], ForwardTwiddles<G, g, SKEW, PADDED>& f)
{
    constexpr int B = G::bits(g), above = ForwardTwiddles<G, g, SKEW, PADDED>::above;
    if constexpr (ForwardTwiddles<G, g, SKEW, PADDED>::SQUARE) f.w[1] = mul(f.w[2], f.w[2]);
    static_for<0, B>([&](auto st) {
        constexpr int s = B - 1 - st.value;
        turned_stage<false, (st.value >= APART), s, B, 0>(v, f.w[st.value]);
        // the top index bit, where the registers hold it, turns the factors of its half by 2 pi / 2^(above + st + 1)
        if constexpr (G::R >> B == 2) {
            constexpr double a = 6.283185307179586476925286766559 / (double)(2 << (above + st.value));
            constexpr float less = (float)cosm1_near_0(a), sine = (float)sin_near_0(a);
            const C w = f.w[st.value];      // one rounding: what the turn adds is small
            turned_stage<false, (st.value >= APART), s, B, (1 << B)>(v, C{w.x + __builtin_fmaf(w.x, less, w.y * sine), w.y + __builtin_fmaf(w.y, less, w.x * -sine)});
        }
        if constexpr (G::R > 16) __builtin_amdgcn_sched_barrier(0);
    });
    __builtin_amdgcn_sched_barrier(0);
}
// group 2 backward: constants alone
template <int B, int R>
__device__ __forceinline__ void inverse_bottom(C (&v)[R])
{
    static_for<0, B>([&](auto s) {
        static_for<0, R>([&](auto k) {
            if constexpr (!(k.value & (1 << s.value)))
                butterfly_const<((k.value & ((1 << s.value) - 1)) << 5 >> s.value), true>(v[k.value], v[k.value | (1 << s.value)]);
        });
    });
}
// SKEW (the top group): the result times the conjugate of base as well, which the first stage takes along
template <typename G, int g, bool SKEW, bool APART>
__device__ __forceinline__ void inverse_group(C (&v)[G::R], const InverseTwiddles<G, g, SKEW>& f)
{
    constexpr int B = G::bits(g);
    C w0 = f.w[0];
    if constexpr (SKEW) {
        w0 = mul(w0, f.base);
        static_for<0, G::R>([&](auto k) { if constexpr (!(k.value & 1)) v[k.value] = mul_conj(v[k.value], f.base); });
    }
    static_for<0, B>([&](auto s) {
        static_for<0, (G::R >> B)>([&](auto q) { turned_stage<true, APART, s.value, B, (q.value << B)>(v, s.value ? f.w[s.value] : w0); });
        if constexpr (G::R > 16) __builtin_amdgcn_sched_barrier(0);
    });
    __builtin_amdgcn_sched_barrier(0);
}

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

// v (natural order, top phase) convolved with the part of the spectrum at `spec`: cyclic, or skew-cyclic, whose results take
// exp(+i pi k / n) on point k = j + q0 2^lo0: a constant power of exp(i pi / 2^B0) per register times the conjugate of exp(-i pi j / n).
// PADDED: one of the two halves of a padded kind.
template <typename G, bool SKEW, bool PADDED, bool CLOSE>
__device__ __forceinline__ void convolve(C (&v)[G::R], C* X, const float2* __restrict__ spec, const float2* __restrict__ tw, int log2p, int t)
{
    constexpr int B0 = G::bits(0), B1 = G::bits(1), B2 = G::bits(2);
    using A = Apart<G, PADDED, CLOSE>;
    // a thread's points of the low phase are runs of 2^B2 consecutive ones: 16-byte loads of two spectrum points
    constexpr int HALF = G::R / 4;
    constexpr bool AHEAD = asks_ahead<G, PADDED>;
    float4 first[HALF], second[HALF];
    {
        ForwardTwiddles<G, 1, SKEW, PADDED> f1;
        ForwardTwiddles<G, 2, SKEW, PADDED> f2;
        f1.load(tw, log2p, t);
        forward_top<B0, SKEW>(v);
        exchange<G, 0, 1>(v, X, t);
        f2.load(tw, log2p, t);
        forward_group<(A::forward ? 0 : B1), G, 1, SKEW, PADDED>(v, f1);
        exchange<G, 1, 2>(v, X, t);
        if constexpr (AHEAD) {
            const float2* s = spec + G::base_index(2, t);
            static_for<0, HALF>([&](auto k) { first[k.value] = *reinterpret_cast<const float4*>(s + G::reg_index(2, 2 * k.value)); });
            __builtin_amdgcn_sched_barrier(0);
        }
        forward_group<(A::low ? B2 - 1 : B2), G, 2, SKEW, PADDED>(v, f2);
    }
    {
        const float2* s = spec + G::base_index(2, t);
        if constexpr (AHEAD) {
            static_for<0, HALF>([&](auto k) { second[k.value] = *reinterpret_cast<const float4*>(s + G::reg_index(2, 2 * (HALF + k.value))); });
            __builtin_amdgcn_sched_barrier(0);
        }
        static_for<0, G::R / 2>([&](auto k2) {
            float4 f;
            if constexpr (!AHEAD) f = *reinterpret_cast<const float4*>(s + G::reg_index(2, 2 * k2.value));
            else if constexpr (k2.value < HALF) f = first[k2.value];
            else f = second[k2.value - HALF];
            v[2 * k2.value] = mul(v[2 * k2.value], C{f.x, f.y});
            v[2 * k2.value + 1] = mul(v[2 * k2.value + 1], C{f.z, f.w});
            if constexpr ((k2.value & 3) == 3) __builtin_amdgcn_sched_barrier(0);
        });
    }
    InverseTwiddles<G, 1, false> f1;
    InverseTwiddles<G, 0, SKEW> f0;
    inverse_bottom<B2>(v);
    f1.load(tw, log2p, t);
    exchange<G, 2, 1>(v, X, t);
    f0.load(tw, log2p, t);
    inverse_group<G, 1, false, A::middle>(v, f1);
    exchange<G, 1, 0>(v, X, t);
    inverse_group<G, 0, SKEW, A::last>(v, f0);
    if constexpr (SKEW) static_for<0, G::R>([&](auto k) { v[k.value] = rot64<k.value * (32 >> B0), true>(v[k.value]); });
}
}  // namespace fft

// HALVES: the padded kinds (P = 2n); else a circulant (P = n)
template <int LOGN, bool HALVES, bool CLOSE>
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
    constexpr bool AHEAD = fft::asks_ahead<G, HALVES>;
    if constexpr (!AHEAD) {
        fft::hadamard_regs<G::bits(2)>(v);
        fft::exchange<G, 2, 0>(v, X, t);
        fft::hadamard_regs<G::bits(0)>(v);
    }
    {
        const int e = G::base_index(0, t);
        const float* __restrict__ d2 = p.reverse ? p.d2 + (N - 1 - e) : p.d2 + e;
        float d[R];
        if (p.reverse) static_for<0, R>([&](auto k) { d[k.value] = d2[-G::reg_index(0, k.value)]; });
        else static_for<0, R>([&](auto k) { d[k.value] = d2[G::reg_index(0, k.value)]; });
        if constexpr (AHEAD) {
            __builtin_amdgcn_sched_barrier(0);
            fft::hadamard_regs<G::bits(2)>(v);
            fft::exchange<G, 2, 0>(v, X, t);
            fft::hadamard_regs<G::bits(0)>(v);
        }
        static_for<0, R>([&](auto k) { v[k.value].x *= d[k.value]; v[k.value].y *= d[k.value]; });
    }
    if constexpr (HALVES) {
        C u[R];
        static_for<0, R>([&](auto k) { u[k.value] = v[k.value]; });
        fft::convolve<G, false, true, CLOSE>(u, X, p.spec, p.tw, LOGP, t);
        fft::convolve<G, true, true, CLOSE>(v, X, p.spec + N, p.tw, LOGP, t);
        static_for<0, R>([&](auto k) { v[k.value].x += u[k.value].x; v[k.value].y += u[k.value].y; });
    } else {
        fft::convolve<G, false, false, CLOSE>(v, X, p.spec, p.tw, LOGP, t);
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

template <int LOGN, bool HALVES, bool CLOSE = false>
inline hipError_t launch_struct_fft_nt(const StructFftParams& p, hipStream_t s)
{
    using G = fft::Geo<LOGN>;
    constexpr size_t lds = (size_t)G::LDS_POINTS * sizeof(fft::C);
    const long long blocks = (p.batch + 1) / 2;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    if constexpr (lds > 65536) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(struct_fft_kernel<LOGN, HALVES, CLOSE>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((struct_fft_kernel<LOGN, HALVES, CLOSE>), dim3((unsigned)blocks), dim3(G::T), lds, s, p);
    return hipGetLastError();
}

// sizes whose kernels are compiled by themselves (struct_fft_13.hip, struct_fft_14.hip: a minute each); padded: P = 2n
hipError_t launch_struct_fft_13(bool padded, const StructFftParams& p, hipStream_t s);
hipError_t launch_struct_fft_14(bool padded, const StructFftParams& p, hipStream_t s);
}  // namespace spinner
