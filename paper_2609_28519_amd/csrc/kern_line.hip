// Axes of 512 and 1024, and of 256 beside them (power-of-two shapes beyond the fused kernels, Section
// 7.1): a row pass and a column pass over HBM, the second in place on the output.  Each pass reads
// and writes every element once and transforms its lines two at a time as one complex line shared by
// N / 32 threads (line_fft.hpp).  Axes of at most 128 in such a shape take the one-thread-per-line
// kernels.
//
// Bound: HBM.  Two passes move 16 B per element, 350 us per 2^27 elements at the copy rate
// (6.1 TB/s).  What decides the rate below that is how many wavefronts a CU holds and how often
// each of them waits:
//   * 32 complex values per thread: 64 data registers, 12-16 wavefronts per CU.  One thread per line
//     and 256 values per lane (the form that these kernels replaced) ran at one wavefront per SIMD.
//   * a wavefront waits for memory once: the twiddles come from an LDS copy, not from memory between
//     the stages (which cost 60 us per pass of 270).
//   * rows: a wavefront owns its lines, so its exchanges need no barrier; lines enter as 8-byte and
//     leave as 16-byte accesses of consecutive lanes (4-byte stores: 610 us for 8 x 1024 forward, 400
//     us now).
//   * columns: a tile is 16 or 32 neighbouring columns (64 or 128 bytes of each row), and 16
//     neighbouring tiles run on the same XCD, whose L2 then sees whole 128-byte lines (1024 x 1024
//     forward with 16-column tiles: 544 us apart, 432 us together).
// 2^27 floats, out of place, us before -> now (forward / inverse / round trip):
//   1024 x 1024  981 -> 439, 952 -> 431, 1626 -> 473      8 x 1024   815 -> 411, 773 -> 420, 1131 -> 424
//   512 x 512    678 -> 421, 745 -> 424, 809 -> 449       1024 x 8   679 -> 399, 647 -> 395, 894 -> 412
// Whole images run the normalised forms (Norm, line_fft.hpp), at the same speed.
#include <hip/hip_runtime.h>

#include "internal.hpp"
#include "line_fft.hpp"

namespace dct {
namespace {

// A tile is a wavefront's worth of row pairs, or PAIRS neighbouring column pairs.  Rows: every
// wavefront of the workgroup has a tile of its own and they share only the twiddle copy.
constexpr int kRowWaves = 4;
template <int N, bool COLS, int PAIRS>
struct Shape {
    static constexpr int TPL = LineCfg<N>::TPL;
    static constexpr int SLOTS = COLS ? PAIRS : 64 / TPL; // pairs per tile
    static constexpr int TILES = COLS ? 1 : kRowWaves;    // tiles per workgroup
    static constexpr int NT = SLOTS * TPL * TILES;
};

// Barriers that wait for LDS only, not for the loads and stores in flight.
template <bool WAVE>
__device__ __forceinline__ void lds_sync()
{
    // one wavefront's LDS accesses happen in program order
    if (WAVE) asm volatile("" ::: "memory");
    else asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int N, int DIR, bool COLS, int PAIRS, bool NORM>
__global__ void __launch_bounds__((Shape<N, COLS, PAIRS>::NT), COLS && PAIRS == 16 && N >= 512 ? 4 : 3)
k_line(Addr a, uint32_t total, uint32_t tiles, uint32_t pairs, int32_t es, int32_t ls, float s0,
       const float2* __restrict__ tab_in)
{
    using C = LineCfg<N>;
    using S = Shape<N, COLS, PAIRS>;
    using P = line::Place<N, COLS, S::SLOTS>;
    constexpr int R1 = C::R1, NB = C::NB;
    __shared__ __attribute__((aligned(16))) float lds_all[2 * C::TAB + S::TILES * P::FLOATS];
    const int wave = COLS ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int th = COLS ? threadIdx.x : threadIdx.x & 63;
    float* lds = lds_all + 2 * C::TAB + wave * P::FLOATS;
    const int ps = COLS ? th % S::SLOTS : th / C::TPL;
    const int t = COLS ? th / S::SLOTS : th % C::TPL;
    // column tiles: 16 neighbours share an XCD (workgroups go to the 8 XCDs in turn)
    uint32_t blk = blockIdx.x;
    if (COLS && (blk | 127u) < gridDim.x) blk = (blk & ~127u) | ((blk & 7) << 4) | ((blk & 127u) >> 3);
    const uint32_t tile0 = blk * S::TILES + wave;
    const uint32_t tile = tile0 < total ? tile0 : total - 1;
    const uint32_t b = tile / tiles;
    const uint32_t pr0 = (tile % tiles) * S::SLOTS + ps;
    // slots past the last pair (tile) transform a copy of it and store nothing
    const bool ok = tile0 < total && pr0 < pairs;
    const uint32_t line_off = 2 * (pr0 < pairs ? pr0 : pairs - 1) * (uint32_t)ls;
    // wave-uniform array base, 32-bit byte offsets (an array is at most 4 MiB)
    const DCT_GLOBAL char* src = reinterpret_cast<const DCT_GLOBAL char*>(uniform_ptr(a.src(b)));
    DCT_GLOBAL char* dst = reinterpret_cast<DCT_GLOBAL char*>(uniform_ptr(a.dst(b)));
    const line::tabptr tab = (line::tabptr)tab_in;
    auto sync = [] { lds_sync<!COLS>(); };
    const bool t0 = t == 0;
    // the twiddle copy, requested before the lines (threads past its end repeat its last entry)
    constexpr int COPIES = (C::TAB / 2 + S::NT - 1) / S::NT;
    float4 tc[COPIES];
    auto tc_at = [](int i) {
        const int e = threadIdx.x + S::NT * i;
        return S::NT * (i + 1) <= C::TAB / 2 ? e : e < C::TAB / 2 ? e : C::TAB / 2 - 1;
    };
#pragma unroll
    for (int i = 0; i < COPIES; ++i) tc[i] = *(reinterpret_cast<const gfloat4*>(tab) + tc_at(i));
    line::Twiddles<N> tw;
    tw.tab = reinterpret_cast<const float2*>(lds_all);
    tw.load(tab, t);
    cf v[32];
    // element k = t_part + c of the pair's lines: lane offset of t_part, uniform offset of c
    auto lane = [&](int tp) { return (line_off + (uint32_t)(tp * es)) * 4u; };
    auto ld1 = [&](uint32_t o, int c) { return *reinterpret_cast<const gfloat*>(src + (uint32_t)(c * 4) + o); };
    auto ld2 = [&](uint32_t o, int c) { return *reinterpret_cast<const DCT_GLOBAL float2*>(src + (uint32_t)(c * 4) + o); };
    auto load_k = [&](uint32_t o, int c) -> cf { // both lines' element
        if constexpr (COLS) {
            const float2 f = ld2(o, c * es);
            return {f.x, f.y};
        } else {
            return {ld1(o, c), ld1(o + (uint32_t)ls * 4u, c)};
        }
    };
    auto store_k = [&](uint32_t o, int c, float xa, float xb) {
        if (!ok) return;
        if constexpr (COLS) {
            *reinterpret_cast<DCT_GLOBAL float2*>(dst + (uint32_t)(c * es * 4) + o) = make_float2(xa, xb);
        } else {
            *reinterpret_cast<gfloat*>(dst + c * 4 + o) = xa;
            *reinterpret_cast<gfloat*>(dst + c * 4 + (o + (uint32_t)ls * 4u)) = xb;
        }
    };
    using F = line::Norm<N, NORM>;
    auto scaled = [](float2 c, float f) { return f == 1.f ? c : make_float2(c.x * f, c.y * f); };
    auto lo_lane = [&](int q) { return line::lo_lane<N>(t, q); };
    auto hi_lane = [&](int q) { return line::hi_lane<N>(t, q); };
    if constexpr (DIR == DCT2D_INVERSE) {
        cf lo[16], hi[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            lo[q] = load_k(lane(lo_lane(q)), line::lo_const<N>(q));
            hi[q] = load_k(lane(hi_lane(q)), line::hi_const<N>(q));
        }
#pragma unroll
        for (int i = 0; i < COPIES; ++i) *(reinterpret_cast<float4*>(lds_all) + tc_at(i)) = tc[i];
        lds_sync<false>();
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            cf l, h;
            line::slot_inverse<N>({lo[q].x, hi[q].x}, {lo[q].y, hi[q].y}, q == 0 && t0,
                                  scaled(tw.slot(q, t), F::inv_c), s0 * F::inv_c, l, h);
            lo[q] = l;
            hi[q] = h;
        }
        line::from_slots(v, t0, lo, hi);
    } else {
        // x[2n], x[2n+1] for n = r1 + T1 m, m < R1 / 2, r1 over the thread's butterflies
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int mi = line::mirror<N>(i);
            const uint32_t o_in = lane(line::n_lane<N>(t, i));
#pragma unroll
            for (int m = 0; m < R1 / 2; ++m) {
                const int c = line::n_const<N>(i, m);
                cf e, o;
                if constexpr (COLS) {
                    e = load_k(o_in, c);
                    o = load_k(o_in, c + 1);
                } else {
                    const float2 fa = ld2(o_in, c), fb = ld2(o_in + (uint32_t)ls * 4u, c);
                    e = {fa.x, fb.x};
                    o = {fa.y, fb.y};
                }
                v[i * R1 + m] = e;
                v[mi * R1 + R1 - 1 - m] = o;
            }
        }
#pragma unroll
        for (int i = 0; i < COPIES; ++i) *(reinterpret_cast<float4*>(lds_all) + tc_at(i)) = tc[i];
        lds_sync<false>();
        line::fft_forward<N, P, NORM>(v, lds, t, ps, tw, sync);
        cf lo[16], hi[16];
        line::to_slots(v, t0, lo, hi);
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            cf xa, xb;
            const float2 c = tw.slot(q, t);
            line::slot_forward<N>(lo[q], hi[q], q == 0 && t0, scaled(c, F::fwd_c), s0 * F::fwd_c, xa, xb);
            if constexpr (DIR == DCT2D_ROUNDTRIP) {
                line::slot_inverse<N>(xa, xb, q == 0 && t0, scaled(c, F::inv_c), s0 * F::inv_c, lo[q], hi[q]);
            } else if constexpr (COLS) {
                store_k(lane(lo_lane(q)), line::lo_const<N>(q), xa.x, xb.x);
                store_k(lane(hi_lane(q)), line::hi_const<N>(q), xa.y, xb.y);
            } else {
                lo[q] = xa;
                hi[q] = xb;
            }
        }
        if constexpr (DIR == DCT2D_FORWARD && !COLS) {
            // rows: one line at a time through LDS, so that it leaves as whole 16-byte groups
            float* row = lds + ps * P::SLOT;
#pragma unroll
            for (int l = 0; l < 2; ++l) {
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const cf x = l ? hi[q] : lo[q];
                    row[lo_lane(q) + line::lo_const<N>(q)] = x.x;
                    row[hi_lane(q) + line::hi_const<N>(q)] = x.y;
                }
                sync();
                const uint32_t o = lane(4 * t) + (l ? (uint32_t)ls * 4u : 0u);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float4 f = *reinterpret_cast<const float4*>(row + 4 * (t + C::TPL * i));
                    if (ok) *reinterpret_cast<gfloat4*>(dst + 16 * C::TPL * i + o) = f;
                }
                sync();
            }
        }
        if constexpr (DIR == DCT2D_FORWARD) return;
        line::from_slots(v, t0, lo, hi);
    }
    line::fft_inverse<N, P, NORM>(v, lds, t, ps, tw, sync);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int mi = line::mirror<N>(i);
        const uint32_t o_out = lane(line::n_lane<N>(t, i));
#pragma unroll
        for (int m = 0; m < R1 / 2; ++m) {
            const int c = line::n_const<N>(i, m);
            const cf e = v[i * R1 + m], o = v[mi * R1 + R1 - 1 - m];
            if constexpr (COLS) {
                store_k(o_out, c, e.x, e.y);
                store_k(o_out, c + 1, o.x, o.y);
            } else if (ok) {
                *reinterpret_cast<DCT_GLOBAL float2*>(dst + c * 4 + o_out) = make_float2(e.x, o.x);
                *reinterpret_cast<DCT_GLOBAL float2*>(dst + c * 4 + (o_out + (uint32_t)ls * 4u)) = make_float2(e.y, o.y);
            }
        }
    }
}

template <int N, int DIR, bool COLS, int PAIRS, bool NORM>
int run(const DeviceTables* t, const Addr& a, int64_t batch, int lines, int es, int ls, hipStream_t s)
{
    using S = Shape<N, COLS, PAIRS>;
    const int64_t tiles = (lines / 2 + S::SLOTS - 1) / S::SLOTS, total = batch * tiles;
    if (total > 0x7fffffff) return DCT2D_ERR_ARG;
    k_line<N, DIR, COLS, PAIRS, NORM><<<(unsigned)((total + S::TILES - 1) / S::TILES), S::NT, 0, s>>>(
        a, (uint32_t)total, (uint32_t)tiles, (uint32_t)(lines / 2), es, ls, line_s0(N), line_tab_for(t, N));
    return hipGetLastError() == hipSuccess ? DCT2D_OK : DCT2D_ERR_HIP;
}

template <int N, bool COLS, int PAIRS, bool NORM>
int run_dir(const DeviceTables* t, const Addr& a, int64_t batch, int lines, int es, int ls, int dir, hipStream_t s)
{
    switch (dir) {
    case DCT2D_FORWARD: return run<N, DCT2D_FORWARD, COLS, PAIRS, NORM>(t, a, batch, lines, es, ls, s);
    case DCT2D_INVERSE: return run<N, DCT2D_INVERSE, COLS, PAIRS, NORM>(t, a, batch, lines, es, ls, s);
    default: return run<N, DCT2D_ROUNDTRIP, COLS, PAIRS, NORM>(t, a, batch, lines, es, ls, s);
    }
}

// Column tiles.  32 columns (16 pairs) keep 128-byte accesses but take 512 threads at N = 1024, whose
// 128 registers the forward and the round trip overflow; 16 columns run with 168 registers (512 x 512: forward
// 422 / 439, round trip 515 / 480 us for 32 / 16 columns; 1024 x 1024: forward 436 / 435, round trip
// 593 / 524).  An array of 8 columns is one tile.
template <int N, bool NORM>
int run_cols(const DeviceTables* t, const Addr& a, int64_t batch, int cols, int dir, hipStream_t s)
{
    if (cols < 16) return run_dir<N, true, 4, NORM>(t, a, batch, cols, cols, 1, dir, s);
    if (dir == DCT2D_ROUNDTRIP) return run<N, DCT2D_ROUNDTRIP, true, 8, NORM>(t, a, batch, cols, cols, 1, s);
    if constexpr (N <= 512) {
        if (cols >= 32)
            return dir == DCT2D_FORWARD ? run<N, DCT2D_FORWARD, true, 16, NORM>(t, a, batch, cols, cols, 1, s)
                                        : run<N, DCT2D_INVERSE, true, 16, NORM>(t, a, batch, cols, cols, 1, s);
    }
    return dir == DCT2D_FORWARD ? run<N, DCT2D_FORWARD, true, 8, NORM>(t, a, batch, cols, cols, 1, s)
                                : run<N, DCT2D_INVERSE, true, 8, NORM>(t, a, batch, cols, cols, 1, s);
}

template <int N, bool NORM>
int run_axis(const DeviceTables* t, const Addr& a, int64_t batch, int rows, int cols, bool column_pass, int dir, hipStream_t s)
{
    return column_pass ? run_cols<N, NORM>(t, a, batch, cols, dir, s)
                       : run_dir<N, false, 1, NORM>(t, a, batch, rows, 1, cols, dir, s);
}

} // namespace

bool line_axis(int n) { return is_pow2(n) || mix_smooth(n); }

int launch_line_axis(const DeviceTables* t, const Addr& a, int64_t batch, int rows, int cols, bool column_pass,
                     int dir, bool norm, hipStream_t s)
{
    const int len = column_pass ? rows : cols;
    // a pair of rows needs an even number of them; k_mix takes any
    if (!is_pow2(len) || (len >= 256 && !column_pass && (rows & 1)))
        return launch_mix_axis(t, a, batch, rows, cols, column_pass, dir, s);
    switch (len) {
    case 1024:
        return norm ? run_axis<1024, true>(t, a, batch, rows, cols, column_pass, dir, s)
                    : run_axis<1024, false>(t, a, batch, rows, cols, column_pass, dir, s);
    case 512:
        return norm ? run_axis<512, true>(t, a, batch, rows, cols, column_pass, dir, s)
                    : run_axis<512, false>(t, a, batch, rows, cols, column_pass, dir, s);
    case 256:
        return norm ? run_axis<256, true>(t, a, batch, rows, cols, column_pass, dir, s)
                    : run_axis<256, false>(t, a, batch, rows, cols, column_pass, dir, s);
    default: return launch_short_line_pass(t, a, batch, len, column_pass ? cols : rows, column_pass, dir, norm, s);
    }
}

int launch_long(const DeviceTables* t, const Job& j)
{
    if (j.dir != DCT2D_FORWARD && j.dir != DCT2D_INVERSE && j.dir != DCT2D_ROUNDTRIP) return DCT2D_ERR_ARG;
    const Addr first = j.addr();
    const Addr in_place{j.out, j.out, j.out_stride, j.out_stride, j.out_idx, j.out_idx, j.out_slot, j.out_slot};
    // rows first (input -> output), then columns in place on the output
    int rc = launch_line_axis(t, first, j.batch, j.rows, j.cols, false, j.dir, false, j.stream);
    if (rc == DCT2D_OK) rc = launch_line_axis(t, in_place, j.batch, j.rows, j.cols, true, j.dir, false, j.stream);
    return rc;
}

} // namespace dct
