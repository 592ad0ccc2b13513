// One-dimensional orthonormal DCT-II / DCT-III of a PAIR of real lines, shared by N / 32 threads.
//
// Two lines a, b of length N travel as one complex line.  With the even-odd reordering
//   v[n] = x[2n] (n < N/2),  v[N-1-n] = x[2n+1],      z = v_a + i v_b,   Z = DFT_N(z),
// and c_k = (a_k / 2) exp(-i pi k / 2N) (a_k: the scale of eq. 1), every pair (k, N-k) gives four
// coefficients in place:  U = Z_k + conj Z_{N-k},  D = Z_k - conj Z_{N-k},
//   X_a[k] = Re(c U),  X_a[N-k] = -Im(c U),  X_b[k] = Im(c D),  X_b[N-k] = Re(c D).
// The inverse is the transposed graph with the same constants (Section 2.2, Prop. 2).
//
// The table holds c_k / S with a power of two S (line_scale), and the last butterflies of the DFT, in
// either direction, multiply by S.  Forward, U and D then do not leave the range of float32 where Z
// does not (a single value of 3e38 came out as infinities); inverse, the factors that multiply first are
// near 1/2, so that subnormal coefficients keep their bits (256 x 256 inverse of 1e-40: 2.4e-4 without).
//
// The DFT is N = R1 * R2 * 16 (R2 = 1 leaves out the middle stage), n = r1 + T1 m, T1 = N / R1,
// r1 = r2 + 16 m2, k = j3 + T3 q, T3 = N / 16, j3 = p + R1 p2:
//   stage 1  radix R1 over m, times W_N^{r1 p}
//   stage 2  radix R2 over m2, times W_{T1}^{r2 p2}
//   stage 3  radix 16 over r2
// A thread holds 32 complex values.  Its stage-1 butterflies come in pairs (r1, T1-1-r1), which
// together own both members of x[2n], x[2n+1], and its two stage-3 butterflies are (j3, T3-j3),
// which own both members of every pair (k, N-k): so lines enter and leave HBM straight from
// registers, and only the stages in between exchange data through LDS.
#pragma once
#include <hip/hip_runtime.h>

#include "dct1d.hpp"

namespace dct {

// Stages, and the table of a length (complex entries):
//   [0, N)           W_N^{r1 p} at p * T1 + r1           (copied to LDS by each workgroup)
//   [N, N + N / 2)   c_k / S of slot q, thread t, at q * TPL + t (likewise; slots below)
//   MID .. + T1      W_{T1}^{r2 p2} at 16 p2 + r2
struct LinePlan {
    int n, r1, r2;
};
constexpr LinePlan line_plan(int n)
{
    return n == 1024 ? LinePlan{n, 16, 4} : n == 512 ? LinePlan{n, 16, 2} : LinePlan{n, n / 16, 1};
}
constexpr int line_table_size(int n) { return n + n / 2 + n / line_plan(n).r1; }
// S: c_k / S lies between 0.35 and 0.5, so that neither the inverse's first products nor the sum of the
// two that a single coefficient has overflow, and the last layer's roundings stay below c's own.
constexpr float line_scale(int n) { return n <= 64 ? 0.25f : n <= 256 ? 0.125f : 0.0625f; }
// The factor of the unpaired coefficients 0 and N / 2.
inline float line_s0(int n) { return (float)(1.0 / __builtin_sqrt((double)n)) / line_scale(n); }

template <int N>
struct LineCfg {
    static constexpr int R1 = line_plan(N).r1, R2 = line_plan(N).r2, R3 = 16;
    static_assert(R1 * R2 * R3 == N, "N = R1 R2 16");
    static constexpr int T1 = N / R1, T3 = N / 16, TPL = N / 32; // TPL: threads per line pair
    static constexpr int NB = 32 / R1;                           // stage-1 butterflies per thread
    static constexpr int TAB = N + N / 2, MID = TAB;             // entries kept in LDS
    static constexpr int SH = line_scale(N) == 0.25f ? 2 : line_scale(N) == 0.125f ? 3 : 4; // S = 2^-SH
    static_assert(line_scale(N) * (1 << SH) == 1.f, "S is a power of two");
    // normalised transforms (NORM below): halvings at the end of the forward's first stage, 2^-SHN <= 1 / sqrt N
    static constexpr int SHN = SH + 1;
};

namespace line {

__device__ __forceinline__ cf mul_mi(cf a) { return {a.y, -a.x}; }
__device__ __forceinline__ cf mul_pi(cf a) { return {-a.y, a.x}; }
// a times -i (forward) or +i (inverse)
template <bool INV>
__device__ __forceinline__ cf rot(cf a) { return INV ? mul_pi(a) : mul_mi(a); }
// a times exp(-+ i phi) in three multiply-adds, (t, s) = (tan phi / 2, sin phi): three shears.  One
// operation less than the product with (cos phi, sin phi), and the shears' determinant is one whatever
// their factors are rounded to, so that these turns neither shrink nor stretch what passes them: with
// products the 512 x 512 round trip was 2.62e-7 off, with shears 2.21e-7 (forward 1.70e-7, 1.56e-7).
template <bool INV>
__device__ __forceinline__ cf turn(cf a, float t, float s)
{
    if (INV) {
        t = -t;
        s = -s;
    }
    const float x = __builtin_fmaf(t, a.y, a.x), y = __builtin_fmaf(-s, x, a.y);
    return {__builtin_fmaf(t, y, x), y};
}
// The turns by pi / 8 and pi / 4; those by more are quarter turns of these.
constexpr float kTan16 = 0.19891236737965800f, kSin8 = 0.38268343236508977f;  // tan pi / 16, sin pi / 8
constexpr float kTan8 = 0.41421356237309505f, kSin4 = 0.70710678118654752f;   // tan pi / 8, sin pi / 4
template <bool INV>
__device__ __forceinline__ cf turn1(cf a) { return turn<INV>(a, kTan16, kSin8); }
template <bool INV>
__device__ __forceinline__ cf turn2(cf a) { return turn<INV>(a, kTan8, kSin4); }
template <bool INV>
__device__ __forceinline__ cf turn3(cf a) { return turn<INV>(rot<INV>(a), -kTan16, -kSin8); }

// (a + b, a - b) / 2^SH, the halvings folded into the additions
template <int SH>
__device__ __forceinline__ void butterfly(cf& a, cf& b)
{
    if constexpr (SH == 0) {
        const cf t = a;
        a = cadd(t, b);
        b = csub(t, b);
    } else {
        constexpr float S = 1.f / (1 << SH);
        const cf t = {S * a.x, S * a.y};
        a = {__builtin_fmaf(S, b.x, t.x), __builtin_fmaf(S, b.y, t.y)};
        b = {__builtin_fmaf(-S, b.x, t.x), __builtin_fmaf(-S, b.y, t.y)};
    }
}

// The DFTs of R values, times 2^-SH.
template <bool INV, int SH = 0>
__device__ __forceinline__ void dft4(cf& a, cf& b, cf& c, cf& d)
{
    cf t0 = cadd(a, c), t1 = csub(a, c), t2 = cadd(b, d), t3 = rot<INV>(csub(b, d));
    butterfly<SH>(t0, t2);
    butterfly<SH>(t1, t3);
    a = t0;
    b = t1;
    c = t2;
    d = t3;
}

template <bool INV, int SH = 0>
__device__ __forceinline__ void dft8(cf* v)
{
    dft4<INV>(v[0], v[2], v[4], v[6]);
    dft4<INV>(v[1], v[3], v[5], v[7]);
    cf o0 = v[1], o1 = turn2<INV>(v[3]), o2 = rot<INV>(v[5]), o3 = turn2<INV>(rot<INV>(v[7]));
    cf e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
    butterfly<SH>(e0, o0);
    butterfly<SH>(e1, o1);
    butterfly<SH>(e2, o2);
    butterfly<SH>(e3, o3);
    v[0] = e0; v[1] = e1; v[2] = e2; v[3] = e3;
    v[4] = o0; v[5] = o1; v[6] = o2; v[7] = o3;
}

template <bool INV, int SH = 0>
__device__ __forceinline__ void dft16(cf* v)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) dft4<INV>(v[i], v[i + 4], v[i + 8], v[i + 12]);
    // v[i + 4 p] now holds output p of column i; times W_16^{i p}
    v[5] = turn1<INV>(v[5]);
    v[6] = turn2<INV>(v[6]);
    v[7] = turn3<INV>(v[7]);
    v[9] = turn2<INV>(v[9]);
    v[10] = rot<INV>(v[10]);
    v[11] = turn2<INV>(rot<INV>(v[11]));
    v[13] = turn3<INV>(v[13]);
    v[14] = turn2<INV>(rot<INV>(v[14]));
    v[15] = turn1<INV>(cf{-v[15].x, -v[15].y});
#pragma unroll
    for (int p = 0; p < 4; ++p) dft4<INV, SH>(v[4 * p], v[4 * p + 1], v[4 * p + 2], v[4 * p + 3]);
    // output p + 4 q sits at v[4 p + q]: transpose
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = p + 1; q < 4; ++q) {
            const cf t = v[4 * p + q];
            v[4 * p + q] = v[4 * q + p];
            v[4 * q + p] = t;
        }
}

template <int R, bool INV, int SH = 0>
__device__ __forceinline__ void dft(cf* v)
{
    if constexpr (R == 2) butterfly<SH>(v[0], v[1]);
    else if constexpr (R == 4) dft4<INV, SH>(v[0], v[1], v[2], v[3]);
    else if constexpr (R == 8) dft8<INV, SH>(v);
    else if constexpr (R == 16) dft16<INV, SH>(v);
}

// Times a table twiddle (conjugated for the inverse).
template <bool INV>
__device__ __forceinline__ cf tmul(cf a, float2 w) { return INV ? cmulc(a, w) : cmul(a, w); }

// Table entries are read through the global address space (a lane-dependent index).
typedef const DCT_GLOBAL float2* tabptr;

// Where an exchanged value lies in LDS.  Every index is a per-thread base plus a compile-time
// constant (no XOR permutation), so each access is one instruction with an immediate offset and no
// address registers.  The pitches keep both sides of each exchange free of bank conflicts (32 banks):
//   exchange 1, (p, r1) at p * PITCH1 + r1: written and read along r1 (the read side of N = 1024
//     spans two p per 32 lanes, 8 banks apart: two lanes share 8 of the banks)
//   exchange 2, (j3, r2) at 17 j3 + r2: written along r2, read along j3
// Rows: the pair slots one after another, SLOT apart, an odd multiple of TPL modulo 32 (the 32 / TPL
// slots of 32 lanes then cover all banks); columns: the slots fastest.
constexpr int spread(int size, int tpl) { return size % (2 * tpl) == tpl ? size : spread(size + 1, tpl); }
template <int N, bool COLS, int SLOTS>
struct Place {
    using C = LineCfg<N>;
    static constexpr int PITCH1 = !COLS && N == 1024 ? C::T1 + 8 : C::T1;
    static constexpr int EX1 = C::R2 > 1 ? C::R1 * PITCH1 : 0, EX2 = C::T3 * 17;
    static constexpr int SIZE = EX1 > EX2 ? EX1 : EX2;
    static constexpr int SLOT = COLS || C::TPL >= 32 ? SIZE : spread(SIZE, C::TPL);
    static constexpr int FLOATS = C::TPL > 1 ? SLOT * SLOTS : 0; // one thread has the whole pair
    __device__ static int at(int e, int ps) { return COLS ? e * SLOTS + ps : ps * SLOT + e; }
    __device__ static int ex1(int p, int r1, int ps) { return at(p * PITCH1 + r1, ps); }
    __device__ static int ex2(int j3, int r2, int ps) { return at(17 * j3 + r2, ps); }
};

// Index of the thread's butterflies: stage 1 butterfly i (i < NB1; the second half mirrors the
// first), stage 3 butterfly 0 / 1.
template <int N>
__device__ __forceinline__ int r1_of(int t, int i)
{
    using C = LineCfg<N>;
    constexpr int NB = 32 / C::R1;
    return i < NB / 2 ? t + C::TPL * i : C::T1 - 1 - (t + C::TPL * (i - NB / 2));
}
template <int N>
__device__ __forceinline__ int j3_of(int t, int i)
{
    using C = LineCfg<N>;
    return i == 0 ? t : (t == 0 ? C::T3 / 2 : C::T3 - t);
}

// One exchange through LDS, real parts and then imaginary parts through the same floats.
// put(i) / get(i): LDS index of value i on the writing / reading side.  sync(): all threads of the
// lines involved have passed (a wavefront-local exchange needs only the wavefront's own order).
template <class PUT, class GET, class SYNC>
__device__ __forceinline__ void exchange(float* lds, cf (&v)[32], PUT put, GET get, SYNC sync)
{
    float re[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) lds[put(i)] = v[i].x;
    sync();
#pragma unroll
    for (int i = 0; i < 32; ++i) re[i] = lds[get(i)];
    sync();
#pragma unroll
    for (int i = 0; i < 32; ++i) lds[put(i)] = v[i].y;
    sync();
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = {re[i], lds[get(i)]};
    sync();
}

// Middle-stage value i: butterfly i / R2, member i % R2; p of the butterfly.
template <int N>
struct Mid {
    using C = LineCfg<N>;
    __device__ static int r2(int t) { return t & 15; }
    __device__ static int p(int t, int i) { return (t >> 4) + (C::TPL / 16) * (i / C::R2); }
};

// The twiddles: the workgroup's LDS copy of the table and, in registers, the middle stage's factors
// (the same for all of a thread's middle butterflies).  Read from memory between the stages they
// would queue behind the other wavefronts' line traffic and stall the wavefront once per stage;
// formed from a few loaded powers they would cost precision.
template <int N>
struct Twiddles {
    using C = LineCfg<N>;
    const float2* tab; // LDS
    float2 m[C::R2 > 1 ? C::R2 : 2];

    __device__ __forceinline__ void load(tabptr g, int t)
    {
        if constexpr (C::R2 > 1) {
#pragma unroll
            for (int k = 1; k < C::R2; ++k) m[k] = g[C::MID + 16 * k + (t & 15)];
        }
    }
    // v[p] *= W_N^{r1 p} (conjugated for the inverse), p < R1
    template <bool INV>
    __device__ __forceinline__ void stage1(cf* v, int r1) const
    {
#pragma unroll
        for (int p = 1; p < C::R1; ++p) v[p] = tmul<INV>(v[p], tab[p * C::T1 + r1]);
    }
    __device__ __forceinline__ float2 slot(int q, int t) const { return tab[N + q * C::TPL + t]; }
};

// NORM: no intermediate value is much larger than the result can be, at the price of a few bits of
// subnormal arrays.  Forward, the first stage (sums of 16 values) multiplies by 2^-SHN instead of the last
// by S; inverse, the table's factors are reduced to c_k first.  fwd_c, inv_c: what the table's factors and
// the unpaired coefficients' then take.
template <int N, bool NORM>
struct Norm {
    using C = LineCfg<N>;
    static constexpr int FIRST = NORM ? C::SHN : 0, LAST = NORM ? 0 : C::SH, INV_LAST = NORM ? 0 : C::SH;
    static constexpr float fwd_c = NORM ? (float)(1 << (C::SHN - C::SH)) : 1.f;
    static constexpr float inv_c = NORM ? 1.f / (1 << C::SH) : 1.f;
};

// Forward: v[i * R1 + m] = z[r1_of(i) + T1 m]  ->  v[16 i + q] = S Z[j3_of(i) + T3 q].
template <int N, class P, bool NORM = false, class SYNC>
__device__ __forceinline__ void fft_forward(cf (&v)[32], float* lds, int t, int ps, const Twiddles<N>& w, SYNC sync)
{
    using C = LineCfg<N>;
    constexpr int R1 = C::R1, R2 = C::R2;
#pragma unroll
    for (int i = 0; i < C::NB; ++i) {
        dft<R1, false, Norm<N, NORM>::FIRST>(v + i * R1);
        w.template stage1<false>(v + i * R1, r1_of<N>(t, i));
    }
    if constexpr (R2 > 1) {
        exchange(
            lds, v, [&](int i) { return P::ex1(i % R1, r1_of<N>(t, i / R1), ps); },
            [&](int i) { return P::ex1(Mid<N>::p(t, i), Mid<N>::r2(t) + 16 * (i % R2), ps); }, sync);
#pragma unroll
        for (int i = 0; i < 32; i += R2) {
            dft<R2, false>(v + i);
#pragma unroll
            for (int k = 1; k < R2; ++k) v[i + k] = cmul(v[i + k], w.m[k]);
        }
        exchange(
            lds, v, [&](int i) { return P::ex2(Mid<N>::p(t, i) + R1 * (i % R2), Mid<N>::r2(t), ps); },
            [&](int i) { return P::ex2(j3_of<N>(t, i / 16), i % 16, ps); }, sync);
    } else if constexpr (C::TPL == 1) {
        cf u[32]; // one thread has the whole pair: r1 = i, or 15 - (i - 8)
#pragma unroll
        for (int i = 0; i < 32; ++i) u[16 * (i % R1) + (i / R1 < 8 ? i / R1 : 23 - i / R1)] = v[i];
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = u[i];
    } else {
        exchange(
            lds, v, [&](int i) { return P::ex2(i % R1, r1_of<N>(t, i / R1), ps); },
            [&](int i) { return P::ex2(j3_of<N>(t, i / 16), i % 16, ps); }, sync);
    }
    dft16<false, Norm<N, NORM>::LAST>(v);
    dft16<false, Norm<N, NORM>::LAST>(v + 16);
}

// The transposed graph: v[16 i + q] = Z[j3_of(i) + T3 q]  ->  v[i * R1 + m] = S z[r1_of(i) + T1 m].
template <int N, class P, bool NORM = false, class SYNC>
__device__ __forceinline__ void fft_inverse(cf (&v)[32], float* lds, int t, int ps, const Twiddles<N>& w, SYNC sync)
{
    using C = LineCfg<N>;
    constexpr int R1 = C::R1, R2 = C::R2;
    dft16<true>(v);
    dft16<true>(v + 16);
    if constexpr (R2 > 1) {
        exchange(
            lds, v, [&](int i) { return P::ex2(j3_of<N>(t, i / 16), i % 16, ps); },
            [&](int i) { return P::ex2(Mid<N>::p(t, i) + R1 * (i % R2), Mid<N>::r2(t), ps); }, sync);
#pragma unroll
        for (int i = 0; i < 32; i += R2) {
#pragma unroll
            for (int k = 1; k < R2; ++k) v[i + k] = cmulc(v[i + k], w.m[k]);
            dft<R2, true>(v + i);
        }
        exchange(
            lds, v, [&](int i) { return P::ex1(Mid<N>::p(t, i), Mid<N>::r2(t) + 16 * (i % R2), ps); },
            [&](int i) { return P::ex1(i % R1, r1_of<N>(t, i / R1), ps); }, sync);
    } else if constexpr (C::TPL == 1) {
        cf u[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) u[i] = v[16 * (i % R1) + (i / R1 < 8 ? i / R1 : 23 - i / R1)];
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = u[i];
    } else {
        exchange(
            lds, v, [&](int i) { return P::ex2(j3_of<N>(t, i / 16), i % 16, ps); },
            [&](int i) { return P::ex2(i % R1, r1_of<N>(t, i / R1), ps); }, sync);
    }
#pragma unroll
    for (int i = 0; i < C::NB; ++i) {
        w.template stage1<true>(v + i * R1, r1_of<N>(t, i));
        dft<R1, true, Norm<N, NORM>::INV_LAST>(v + i * R1);
    }
}

// Slot q of the thread's 16 coefficient pairs (k_lo, k_hi = N - k_lo): k_lo = t + T3 q, the partner in
// the mirrored butterfly.  Thread 0 holds butterflies 0 and T3/2, each its own mirror: slots 0-7 are
// k_lo = T3 q (slot 0: the two unpaired coefficients 0 and N/2), slots 8-15 k_lo = T3/2 + T3 q.  So
// k_lo < N/2 exactly for q < 8.

// The same indices as a non-negative lane part plus a constant (32-bit unsigned offsets).
// Sample x[2n] (with x[2n+1]) of stage-1 butterfly i, member m < R1 / 2: 2n = n_lane + n_const.
template <int N>
__device__ __forceinline__ int n_lane(int t, int i)
{
    return i < LineCfg<N>::NB / 2 ? 2 * t : 2 * (LineCfg<N>::TPL - 1 - t);
}
template <int N>
__host__ __device__ constexpr int n_const(int i, int m)
{
    using C = LineCfg<N>;
    return 2 * C::TPL * (i < C::NB / 2 ? i : C::NB - 1 - (i - C::NB / 2)) + 2 * C::T1 * m;
}
// The butterfly that owns x[2n+1] (as its member R1 - 1 - m).
template <int N>
__host__ __device__ constexpr int mirror(int i)
{
    return i < LineCfg<N>::NB / 2 ? i + LineCfg<N>::NB / 2 : i - LineCfg<N>::NB / 2;
}
// Coefficients of slot q: k_lo = lo_lane + lo_const, k_hi = hi_lane + hi_const.
template <int N>
__device__ __forceinline__ int lo_lane(int t, int q) { return q < 8 || t != 0 ? t : LineCfg<N>::T3 / 2; }
template <int N>
__host__ __device__ constexpr int lo_const(int q) { return LineCfg<N>::T3 * q; }
template <int N>
__device__ __forceinline__ int hi_lane(int t, int q)
{
    return q == 0 ? (t == 0 ? 0 : N / 2 - t) : LineCfg<N>::TPL - lo_lane<N>(t, q);
}
template <int N>
__host__ __device__ constexpr int hi_const(int q) { return q == 0 ? N / 2 : N - LineCfg<N>::TPL - LineCfg<N>::T3 * q; }

__device__ __forceinline__ cf pick(bool c, cf a, cf b) { return {c ? a.x : b.x, c ? a.y : b.y}; }

// Z pairs <-> slots (lo[q], hi[q]).
__device__ __forceinline__ void to_slots(const cf (&v)[32], bool t0, cf (&lo)[16], cf (&hi)[16])
{
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        lo[q] = v[q];
        hi[q] = pick(t0, q == 0 ? v[8] : v[16 - q], v[31 - q]);
        lo[8 + q] = pick(t0, v[24 + q], v[8 + q]);
        hi[8 + q] = v[23 - q];
    }
}
__device__ __forceinline__ void from_slots(cf (&v)[32], bool t0, const cf (&lo)[16], const cf (&hi)[16])
{
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        v[q] = lo[q];
        v[8 + q] = pick(t0, hi[q == 0 ? 0 : 8 - q], lo[8 + q]);
        v[16 + q] = hi[15 - q];
        v[24 + q] = pick(t0, lo[8 + q], hi[7 - q]);
    }
}

// Coefficients of slot q from its Z pair, and back.  xa, xb: (X[k_lo], X[k_hi]) of lines a and b.
template <int N>
__device__ __forceinline__ void slot_forward(cf lo, cf hi, bool single, float2 c, float s0, cf& xa, cf& xb)
{
    const cf u = {lo.x + hi.x, lo.y - hi.y}, d = {lo.x - hi.x, lo.y + hi.y};
    xa = {c.x * u.x - c.y * u.y, -(c.x * u.y + c.y * u.x)};
    xb = {c.x * d.y + c.y * d.x, c.x * d.x - c.y * d.y};
    if (single) {
        xa = {s0 * lo.x, s0 * hi.x};
        xb = {s0 * lo.y, s0 * hi.y};
    }
}
template <int N>
__device__ __forceinline__ void slot_inverse(cf xa, cf xb, bool single, float2 c, float s0, cf& lo, cf& hi)
{
    const cf s = {xa.x + xb.y, xb.x - xa.y}, d = {xa.x - xb.y, -xa.y - xb.x};
    lo = {c.x * s.x + c.y * s.y, c.x * s.y - c.y * s.x};     // conj(c) s
    hi = {c.x * d.x + c.y * d.y, c.y * d.x - c.x * d.y};     // conj(conj(c) d)
    if (single) {
        lo = {s0 * xa.x, s0 * xb.x};
        hi = {s0 * xa.y, s0 * xb.y};
    }
}

} // namespace line
} // namespace dct
