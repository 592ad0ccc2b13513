// Line pairs of any length N whose prime factors are small, by a mixed-radix transform.
//
// The pair formulation is that of line_fft.hpp: z = v_a + i v_b, one DFT of length N, and the
// post-twiddle per pair (k, N-k); it holds for odd N too (v[n] = x[2n] for 2n < N, v[N-1-n] =
// x[2n+1]).  The DFT runs as autosorting passes over LDS: with s the product of the radices done
// and u = k + s j (k < s, j < N / (R s)), a pass of radix R reads z[u + (N/R) r], r < R, and writes
//   (DFT_R)_p W_N^{s j p}  to  u + s j (R - 1) + s p.
// Radices 16, 8, 4, 2, 3, 5, 7, 11, 13 are straight-line codes; a larger prime takes sums over its half length.
#pragma once
#include <hip/hip_runtime.h>

#include "line_fft.hpp"

namespace dct {

constexpr int kMixStages = 8; // a length up to 1024 takes at most 6 (729 = 3^6)
constexpr int kMixRadix = 13; // largest prime with a straight-line code

// Pairs and threads per workgroup for a length: as many pairs as 16 values per thread hold, a power of
// two.  256 threads where 8 pairs (16 columns, 64 bytes of a row) fit them, else 512 (4 pairs at n > 512:
// 1000 x 600 3 % slower, 768 x 768 2 % faster; 16 pairs of 257 .. 512 in 512 threads: 384 x 384 round
// trip 246 us against 237).
struct MixShape {
    int slots, threads;
};
constexpr MixShape mix_shape(int n)
{
    return n > 512 ? MixShape{8, 512} : n > 256 ? MixShape{8, 256} : n > 128 ? MixShape{16, 256}
         : n > 32 ? MixShape{32, 256} : n > 16 ? MixShape{128, 256} : MixShape{256, 256};
}

// Larger primes p: tables of the factors cos, sin(2 pi jk / p) in blocks of kPrimeBlock values of k,
// (cos, sin) of block b, j = 1 .. H, k = b kPrimeBlock + i at (b H + j - 1) kPrimeBlock + i (zeros past
// k = H = (p - 1) / 2), for p = kMixRadix + 4 .. kMaxPrime (1004 = 4 * 251), one after another.
constexpr int kPrimeBlock = 8, kMaxPrime = 251;
constexpr bool is_prime(int p)
{
    for (int f = 2; f * f <= p; ++f)
        if (p % f == 0) return false;
    return p > 1;
}
constexpr int prime_table_size(int p) { return (p / 2 + kPrimeBlock) / kPrimeBlock * (p / 2) * kPrimeBlock; }
// Where the table of each prime begins; the last entry is the size of all.
struct PrimeOffsets {
    int at[kMaxPrime + 2] = {};
    constexpr PrimeOffsets()
    {
        for (int q = kMixRadix + 1; q <= kMaxPrime; ++q) at[q + 1] = at[q] + (is_prime(q) ? prime_table_size(q) : 0);
    }
};
inline constexpr PrimeOffsets kPrimeOffsets;
constexpr int prime_table_offset(int p) { return kPrimeOffsets.at[p]; }

struct MixPlan {
    int n = 0, stages = 0;
    int radix[kMixStages] = {};
    int s[kMixStages] = {};         // product of the radices before
    float inv_s[kMixStages] = {};   // 1 / s
};

// The radices of n: odd ones first (their strided writes touch all LDS banks), the largest power of
// two last (its writes are contiguous).  False for lengths left to the dense products: those with a
// prime factor so large that fewer than 32 butterflies (of the workgroup's pairs) share it, where most
// lanes of the prime's pass would idle: p and 2p from p = 131, 3p from p = 89, 252 lengths in all.
inline bool mix_plan(int n, MixPlan& p)
{
    p = MixPlan{};
    p.n = n;
    int q = n, lg = 0, odd[kMixStages], no = 0;
    for (; q % 2 == 0; q /= 2) ++lg;
    for (int f = 3; q > 1; f = f * f > q ? q : f + 2) // what is left once f * f > q is prime
        while (q % f == 0) {
            if (f > kMixRadix && n / f * mix_shape(n).slots < 32) return false;
            odd[no++] = f;
            q /= f;
        }
    for (int i = no - 1; i >= 0; --i) p.radix[p.stages++] = odd[i];
    // 2^lg in the fewest passes of at most 4 bits, the larger ones last
    const int passes = (lg + 3) / 4;
    for (int i = 0; i < passes; ++i) p.radix[p.stages++] = 1 << (lg / passes + (i >= passes - lg % passes ? 1 : 0));
    int s = 1;
    for (int i = 0; i < p.stages; ++i) {
        p.s[i] = s;
        p.inv_s[i] = 1.0f / s;
        s *= p.radix[i];
    }
    return true;
}

// Tables of every length 8 .. 1024, one after another: W_n^e, e < n, then c_k, k <= n / 2.
constexpr int mix_table_size(int n) { return n + n / 2 + 1; }
constexpr int mix_table_offset(int n)
{
    // sum over 8 <= i < n of i + floor(i / 2) + 1
    const int a = (n - 1) * n / 2 - 28, h = (n / 2) * ((n - 1) / 2) - 12;
    return a + h + (n - 8);
}

namespace mix {

// floor(i / d) for i < 2^20, inv = 1 / d: the rounding error of the product, below i / d * 2^-22, stays
// under the 1 / (2 d) that the half adds.
__device__ __forceinline__ int div(int i, float inv) { return (int)(((float)i + 0.5f) * inv); }

template <int R> struct OddRoots;
template <> struct OddRoots<3> {
    static constexpr float c[3] = {1.f, -0.5f, -0.5f};
    static constexpr float s[3] = {0.f, 0.866025404f, -0.866025404f};
};
template <> struct OddRoots<5> {
    static constexpr float c[5] = {1.f, 0.309016994f, -0.809016994f, -0.809016994f, 0.309016994f};
    static constexpr float s[5] = {0.f, 0.951056516f, 0.587785252f, -0.587785252f, -0.951056516f};
};
template <> struct OddRoots<7> {
    static constexpr float c[7] = {1.f, 0.623489802f, -0.222520934f, -0.900968868f, -0.900968868f, -0.222520934f, 0.623489802f};
    static constexpr float s[7] = {0.f, 0.781831482f, 0.974927912f, 0.433883739f, -0.433883739f, -0.974927912f, -0.781831482f};
};
template <> struct OddRoots<11> {
    static constexpr float c[11] = {1.f, 0.841253533f, 0.415415013f, -0.142314838f, -0.654860734f, -0.959492974f, -0.959492974f, -0.654860734f, -0.142314838f, 0.415415013f, 0.841253533f};
    static constexpr float s[11] = {0.f, 0.540640817f, 0.909631995f, 0.989821442f, 0.755749574f, 0.281732557f, -0.281732557f, -0.755749574f, -0.989821442f, -0.909631995f, -0.540640817f};
};
template <> struct OddRoots<13> {
    static constexpr float c[13] = {1.f, 0.885456026f, 0.568064747f, 0.12053668f, -0.354604887f, -0.748510748f, -0.970941817f, -0.970941817f, -0.748510748f, -0.354604887f, 0.12053668f, 0.568064747f, 0.885456026f};
    static constexpr float s[13] = {0.f, 0.464723172f, 0.822983866f, 0.992708874f, 0.935016243f, 0.663122658f, 0.239315664f, -0.239315664f, -0.663122658f, -0.935016243f, -0.992708874f, -0.822983866f, -0.464723172f};
};

// DFT of odd length R (forward): X_k, X_{R-k} = sum_j cos(2 pi jk / R) (x_j + x_{R-j}) -+ i sum_j sin(..) (x_j - x_{R-j}).
template <int R>
__device__ __forceinline__ void dft_odd(cf* v)
{
    constexpr int H = (R - 1) / 2;
    cf t[H], d[H];
#pragma unroll
    for (int j = 0; j < H; ++j) {
        t[j] = cadd(v[1 + j], v[R - 1 - j]);
        d[j] = csub(v[1 + j], v[R - 1 - j]);
    }
    const cf x0 = v[0];
    cf sum = x0;
#pragma unroll
    for (int j = 0; j < H; ++j) sum = cadd(sum, t[j]);
    v[0] = sum;
#pragma unroll
    for (int k = 1; k <= H; ++k) {
        cf a = x0, b = {0.f, 0.f};
#pragma unroll
        for (int j = 1; j <= H; ++j) {
            const float c = OddRoots<R>::c[(j * k) % R], s = OddRoots<R>::s[(j * k) % R];
            a = {a.x + c * t[j - 1].x, a.y + c * t[j - 1].y};
            b = j == 1 ? cf{s * d[0].x, s * d[0].y} : cf{b.x + s * d[j - 1].x, b.y + s * d[j - 1].y};
        }
        v[k] = {a.x + b.y, a.y - b.x};     // a - i b
        v[R - k] = {a.x - b.y, a.y + b.x}; // a + i b
    }
}

template <int R>
__device__ __forceinline__ void dft(cf* v)
{
    if constexpr (R % 2 == 0) line::dft<R, false>(v);
    else dft_odd<R>(v);
}

} // namespace mix
} // namespace dct
