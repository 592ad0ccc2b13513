// Line pairs of any length N whose prime factors are small, by a mixed-radix transform.
//
// The pair formulation is that of line_fft.hpp: z = v_a + i v_b, one DFT of length N, and the
// post-twiddle per pair (k, N-k); it holds for odd N too (v[n] = x[2n] for 2n < N, v[N-1-n] =
// x[2n+1]).  The DFT runs as autosorting passes over LDS: with s the product of the radices done
// and u = k + s j (k < s, j < N / (R s)), a pass of radix R reads z[u + (N/R) r], r < R, and writes
//   (DFT_R)_p W_N^{s j p}  to  u + s j (R - 1) + s p.
// Radices 16, 8, 4, 2, 3, 5, 7, 11, 13 are straight-line codes; a larger prime takes a plain sum.
#pragma once
#include <hip/hip_runtime.h>

#include "line_fft.hpp"

namespace dct {

constexpr int kMixStages = 8; // a length up to 1024 takes at most 6 (729 = 3^6)
// Largest prime factor that takes the mixed-radix path, and the largest with a straight-line code.
// A prime between the two is a plain sum of that many terms per output, worth it on long axes only
// (n >= 8 times the prime: 1020 = 60 * 17 takes 65 us against 346 for the dense product in 1020 x 700
// images, but 29 alone lost to it).
constexpr int kMixPrime = 23, kMixRadix = 13;

struct MixPlan {
    int n = 0, stages = 0;
    int radix[kMixStages] = {};
    int s[kMixStages] = {};         // product of the radices before
    float inv_s[kMixStages] = {};   // 1 / s
};

// The radices of n: odd ones first (their strided writes touch all LDS banks), the largest power of
// two last (its writes are contiguous).  False if n has a prime factor above kMixPrime.
inline bool mix_plan(int n, MixPlan& p)
{
    p = MixPlan{};
    p.n = n;
    int m = n, odd[kMixStages * 2], no = 0;
    for (int f = 3; f <= kMixPrime; f += 2)
        while (m % f == 0) {
            if (f > kMixRadix && n < 8 * f) return false;
            odd[no++] = f;
            m /= f;
        }
    if (m & (m - 1)) return false;
    for (int i = no - 1; i >= 0; --i) p.radix[p.stages++] = odd[i];
    int lg = 0;
    while ((1 << lg) < m) ++lg;
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
