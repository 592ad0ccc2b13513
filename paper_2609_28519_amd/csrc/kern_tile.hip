// Arrays with both axes 32 .. 256 and one of 128 or 256 (128 x 128 aside, which k_split128 runs faster):
// one array per workgroup, held whole in registers, 64 values per thread, read from HBM once and written
// once.  The transforms are those of line pairs (line_fft.hpp): row pairs straight from HBM, the
// coefficients through LDS to the threads of their columns, column pairs, and out (or back through LDS
// for the inverse rows).  Every line pair lies within one wavefront, so its exchange needs no barrier;
// the workgroup meets at the transpositions only.
//
// Bound: HBM where several workgroups share a CU (64 x 256 and below: 5.3 TB/s forward), else the sum of
// the phases.  A 256 x 256 array takes the whole register file of a CU, so loads, arithmetic and stores
// of an array overlap only across its own 16 wavefronts: the round trip issues 140 million wave
// instructions (180 us) and 125 us of LDS beside 177 us of HBM, and takes 391.
//   * 64 values per thread and at most 128 registers: 16 wavefronts per CU, twice those of k_split256
//     and four times those of k_rect256_db.  Nothing may spill for that: at 300 bytes of scratch per
//     thread the 256 x 256 round trip took 700 us, at 84 (the row pass's offsets held across the columns)
//     403, and that of 128 x 256 346 instead of 295.
//   * the LDS tile holds half an array: a transposition is two rounds (transpose below).
// 2^27 floats, out of place, us, the best kernel before -> now (forward / inverse / round trip):
//   256 x 256  300 -> 255, 304 -> 284, 430 -> 391    128 x 256  496 -> 205, 424 -> 206, 535 -> 285
//   256 x 128  487 -> 220, 476 -> 221, 620 -> 324    64 x 256   297 -> 203, 284 -> 205, 474 -> 259
//   256 x 64   281 -> 257, 260 -> 262, 468 -> 334    32 x 256   288 -> 193, 268 -> 195, 476 -> 226
//   256 x 32   291 -> 210, 251 -> 252, 450 -> 303    64 x 128   434 -> 202, 432 -> 199, 501 -> 250
//   128 x 64   433 -> 217, 429 -> 255, 496 -> 316    32 x 128   454 -> 206, 486 -> 199, 579 -> 270
//   128 x 32   482 -> 205, 479 -> 265, 587 -> 307
// (Tall arrays trail wide ones.  Their rows are short: with W = 64 two lanes share a row pair, and a wavefront
// instruction takes 16 bytes of each of 32 pairs; the 256 x 64 forward reads 1.3 to 1.5 times its input and writes
// its output once.)
#include <hip/hip_runtime.h>

#include "internal.hpp"
#include "line_fft.hpp"

namespace dct {
namespace {

__device__ __forceinline__ void wg_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int H, int W>
struct TileCfg {
    static constexpr int NT = H * W / 64; // 64 values per thread
    static constexpr int WAVES = NT / 64;
    static constexpr int RS = 64 / LineCfg<W>::TPL, CS = 64 / LineCfg<H>::TPL; // pairs per wavefront
    using RP = line::Place<W, false, RS>;
    using CP = line::Place<H, true, CS>;
    // transposition by halves: H x W/2 (rows to columns), H/2 x W (back); one wavefront: whole
    static constexpr int HALVES = WAVES > 1 ? 2 : 1;
    static constexpr int PT = W / HALVES + 4, PB = W + 8;
    static constexpr int XW = RP::FLOATS > CP::FLOATS ? RP::FLOATS : CP::FLOATS; // exchange floats per wavefront
    static constexpr int mx(int a, int b) { return a > b ? a : b; }
    static constexpr int LDS = mx(mx(WAVES * XW, H * PT), H / HALVES * PB);
    // wavefronts per SIMD that the registers are held to: a CU takes 1024 threads of the larger
    // shapes (two workgroups, or one), 768 of the smaller
    static constexpr int OCC = NT >= 256 ? 4 : 3;
    static constexpr int TABW = 2 * LineCfg<W>::TAB, TABH = H == W ? 0 : 2 * LineCfg<H>::TAB;
};

// The slots exist here, and instructions do not move across (interleaved over several slots, their
// temporaries spill).
__device__ __forceinline__ void settle(cf (&lo)[16], cf (&hi)[16])
{
#pragma unroll
    for (int q = 0; q < 16; ++q) asm volatile("" : "+v"(lo[q].x), "+v"(lo[q].y), "+v"(hi[q].x), "+v"(hi[q].y));
}
__device__ __forceinline__ void pin(cf& a, cf& b) { asm volatile("" : "+v"(a.x), "+v"(a.y), "+v"(b.x), "+v"(b.y)); }
__device__ __forceinline__ void in_order() { __builtin_amdgcn_sched_barrier(0); }

// A transposition through LDS in halves: every wavefront writes its half-0 values, the first half of
// the wavefronts read theirs, and the same for half 1.  The two kinds of wavefront run codes of their
// own with the same barriers: as conditions inside one code, the values that are read count as live
// from the first to the last of them and spill.
template <int HALVES, class PUT, class GET>
__device__ __forceinline__ void transpose(bool first, PUT put, GET get)
{
    if (HALVES == 1) {
        put(0);
        wg_sync();
        get(0);
        wg_sync();
    } else if (first) {
        put(0);
        wg_sync();
        get(0);
        wg_sync();
        put(1);
        wg_sync();
        wg_sync();
    } else {
        put(0);
        wg_sync();
        wg_sync();
        put(1);
        wg_sync();
        get(1);
        wg_sync();
    }
}

// After a barrier the wavefronts of a SIMD run at different priorities, so that the first ones reach
// their stores (or the next barrier) while the others still compute (256 x 128 round trip 382 -> 364 us).
template <int WAVES>
__device__ __forceinline__ void stagger(int wave)
{
    if constexpr (WAVES >= 8) {
        switch (wave >> 2) {
        case 0: __builtin_amdgcn_s_setprio(0); break;
        case 1: __builtin_amdgcn_s_setprio(1); break;
        case 2: __builtin_amdgcn_s_setprio(2); break;
        default: __builtin_amdgcn_s_setprio(3); break;
        }
    }
}

template <int H, int W, int DIR>
__global__ void __launch_bounds__((TileCfg<H, W>::NT), (TileCfg<H, W>::OCC))
k_tile(Addr a, int64_t batch, float s0w, float s0h, const float2* __restrict__ tabw, const float2* __restrict__ tabh)
{
    using C = TileCfg<H, W>;
    using LW = LineCfg<W>;
    using LH = LineCfg<H>;
    __shared__ __attribute__((aligned(16))) float lds[C::TABW + C::TABH + C::LDS];
    float* const T = lds + C::TABW + C::TABH;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int i = threadIdx.x; i < C::TABW / 4; i += C::NT)
        *reinterpret_cast<float4*>(lds + 4 * i) = *((const gfloat4*)tabw + i);
    if constexpr (H != W)
        for (int i = threadIdx.x; i < C::TABH / 4; i += C::NT)
            *reinterpret_cast<float4*>(lds + C::TABW + 4 * i) = *((const gfloat4*)tabh + i);
    line::Twiddles<W> tw;
    line::Twiddles<H> th;
    tw.tab = reinterpret_cast<const float2*>(lds);
    th.tab = reinterpret_cast<const float2*>(lds + (H == W ? 0 : C::TABW));
    wg_sync();
    auto wave_sync = [] { asm volatile("" ::: "memory"); }; // a wavefront's LDS accesses are in order
    float* const X = T + wave * C::XW;

    for (int64_t blk = blockIdx.x; blk < batch; blk += gridDim.x) {
        const DCT_GLOBAL char* src = reinterpret_cast<const DCT_GLOBAL char*>(uniform_ptr(a.src(blk)));
        DCT_GLOBAL char* dst = reinterpret_cast<DCT_GLOBAL char*>(uniform_ptr(a.dst(blk)));
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane)); // the offsets below are formed per array, not held across the loop
        // row pass: slot-major lanes, row pair wave * RS + rps; column pass: the slots fastest
        const int rps = lane / LW::TPL, rt = lane % LW::TPL, row = 2 * (wave * C::RS + rps);
        const int cps = lane % C::CS, ct = lane / C::CS, col = 2 * (wave * C::CS + cps);
        const bool r0 = rt == 0, c0 = ct == 0;
        cf v[32], lo[16], hi[16];

        if constexpr (DIR != DCT2D_INVERSE) {
            // ---- rows -> coefficients lo[q] = (Xa[k_lo], Xa[k_hi]), hi[q] = those of row b
#pragma unroll
            for (int i = 0; i < LW::NB; ++i) {
                const uint32_t o = 4u * (uint32_t)(row * W + line::n_lane<W>(rt, i));
#pragma unroll
                for (int m = 0; m < LW::R1 / 2; ++m) {
                    const float2 fa = *reinterpret_cast<const DCT_GLOBAL float2*>(src + 4 * line::n_const<W>(i, m) + o);
                    const float2 fb = *reinterpret_cast<const DCT_GLOBAL float2*>(src + 4 * (W + line::n_const<W>(i, m)) + o);
                    v[i * LW::R1 + m] = {fa.x, fb.x};
                    v[line::mirror<W>(i) * LW::R1 + LW::R1 - 1 - m] = {fa.y, fb.y};
                }
            }
            line::fft_forward<W, typename C::RP>(v, X, rt, rps, tw, wave_sync);
            line::to_slots(v, r0, lo, hi);
            settle(lo, hi);
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                cf xa, xb;
                line::slot_forward<W>(lo[q], hi[q], q == 0 && r0, tw.slot(q, rt), s0w, xa, xb);
                lo[q] = xa;
                hi[q] = xb;
                in_order();
            }
            // ---- to columns, by halves of the row
            auto put = [&](int h) {
                float* p = T + row * C::PT;
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    if (C::HALVES == 1) {
                        const int kl = line::lo_lane<W>(rt, q) + line::lo_const<W>(q), kh = line::hi_lane<W>(rt, q) + line::hi_const<W>(q);
                        p[kl] = lo[q].x; p[kl + C::PT] = hi[q].x;
                        p[kh] = lo[q].y; p[kh + C::PT] = hi[q].y;
                    } else {
                        // q < 8: k_lo lies in the first half and k_hi in the second; q >= 8 the reverse
                        const bool use_lo = (q < 8) == (h == 0);
                        const int k = (use_lo ? line::lo_lane<W>(rt, q) + line::lo_const<W>(q)
                                              : line::hi_lane<W>(rt, q) + line::hi_const<W>(q)) - h * (W / 2);
                        p[k] = use_lo ? lo[q].x : lo[q].y;
                        p[k + C::PT] = use_lo ? hi[q].x : hi[q].y;
                    }
                }
            };
            auto get = [&](int h) {
                const float* p = T + col - h * (W / 2);
#pragma unroll
                for (int i = 0; i < LH::NB; ++i) {
                    const int nl = line::n_lane<H>(ct, i);
#pragma unroll
                    for (int m = 0; m < LH::R1 / 2; ++m) {
                        const float2 e = *reinterpret_cast<const float2*>(p + (nl + line::n_const<H>(i, m)) * C::PT);
                        const float2 f = *reinterpret_cast<const float2*>(p + (nl + line::n_const<H>(i, m) + 1) * C::PT);
                        v[i * LH::R1 + m] = {e.x, e.y};
                        v[line::mirror<H>(i) * LH::R1 + LH::R1 - 1 - m] = {f.x, f.y};
                    }
                }
            };
            wg_sync();
            transpose<C::HALVES>(wave < C::WAVES / 2, put, get);
            stagger<C::WAVES>(wave);
            line::fft_forward<H, typename C::CP>(v, X, ct, cps, th, wave_sync);
            line::to_slots(v, c0, lo, hi);
            settle(lo, hi);
        }
        // ---- columns: coefficients out, or back
        const uint32_t co = 4u * (uint32_t)col;
        auto at = [&](int lane_k, int const_k) { return (uint32_t)(lane_k * W * 4) + co + (uint32_t)(const_k * W * 4); };
        if constexpr (DIR == DCT2D_INVERSE) {
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const float2 l = *reinterpret_cast<const DCT_GLOBAL float2*>(src + at(line::lo_lane<H>(ct, q), line::lo_const<H>(q)));
                const float2 h = *reinterpret_cast<const DCT_GLOBAL float2*>(src + at(line::hi_lane<H>(ct, q), line::hi_const<H>(q)));
                lo[q] = {l.x, h.x};
                hi[q] = {l.y, h.y};
            }
        }
        const DCT_GLOBAL char* lam = DIR == DIR_FILTER ? reinterpret_cast<const DCT_GLOBAL char*>(uniform_ptr(a.lam_for(blk))) : nullptr;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            cf xa, xb;
            const float2 c = th.slot(q, ct);
            if constexpr (DIR != DCT2D_INVERSE) line::slot_forward<H>(lo[q], hi[q], q == 0 && c0, c, s0h, xa, xb);
            else { xa = lo[q]; xb = hi[q]; }
            if constexpr (DIR == DCT2D_FORWARD) {
                *reinterpret_cast<DCT_GLOBAL float2*>(dst + at(line::lo_lane<H>(ct, q), line::lo_const<H>(q))) = make_float2(xa.x, xb.x);
                *reinterpret_cast<DCT_GLOBAL float2*>(dst + at(line::hi_lane<H>(ct, q), line::hi_const<H>(q))) = make_float2(xa.y, xb.y);
            } else {
                // opaque before and after the multiply, in the round trip too: no product is contracted into
                // the neighbouring operations, so multipliers of one reproduce the round trip bit for bit
                if constexpr (DIR >= DCT2D_ROUNDTRIP) pin(xa, xb);
                if constexpr (DIR == DIR_FILTER) {
                    // the multipliers are 4-byte aligned
                    const gfloat* l = reinterpret_cast<const gfloat*>(lam + at(line::lo_lane<H>(ct, q), line::lo_const<H>(q)));
                    const gfloat* h = reinterpret_cast<const gfloat*>(lam + at(line::hi_lane<H>(ct, q), line::hi_const<H>(q)));
                    xa = {xa.x * l[0], xa.y * h[0]};
                    xb = {xb.x * l[1], xb.y * h[1]};
                }
                if constexpr (DIR >= DCT2D_ROUNDTRIP) pin(xa, xb);
                line::slot_inverse<H>(xa, xb, q == 0 && c0, c, s0h, lo[q], hi[q]);
            }
            in_order();
        }
        if constexpr (DIR != DCT2D_FORWARD) {
            settle(lo, hi);
            line::from_slots(v, c0, lo, hi);
            line::fft_inverse<H, typename C::CP>(v, X, ct, cps, th, wave_sync);
            // formed anew: the first row pass's offsets are not held across the columns (84 bytes of scratch)
            asm volatile("" : "+v"(lane));
            const int rps = lane / LW::TPL, rt = lane % LW::TPL, row = 2 * (wave * C::RS + rps);
            const bool r0 = rt == 0;
            // ---- back to rows, by halves of the columns
            auto put = [&](int h) {
#pragma unroll
                for (int i = 0; i < LH::NB; ++i) {
                    const int nl = line::n_lane<H>(ct, i);
                    float* p = T + nl * C::PB + col;
#pragma unroll
                    for (int m = 0; m < LH::R1 / 2; ++m) {
                        // the half of rows 2n, 2n + 1, the same in every lane
                        const int in = LH::R1 > 2 ? m / (LH::R1 / 4) : i / (LH::NB / 2);
                        if (C::HALVES == 1 || in == h) {
                            const int r = line::n_const<H>(i, m) - (C::HALVES == 1 ? 0 : h * (H / 2));
                            const cf e = v[i * LH::R1 + m], f = v[line::mirror<H>(i) * LH::R1 + LH::R1 - 1 - m];
                            *reinterpret_cast<float2*>(p + r * C::PB) = make_float2(e.x, e.y);
                            *reinterpret_cast<float2*>(p + (r + 1) * C::PB) = make_float2(f.x, f.y);
                        }
                    }
                }
            };
            auto get = [&](int h) {
                const float* p = T + (row - (C::HALVES == 1 ? 0 : h * (H / 2))) * C::PB;
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int kl = line::lo_lane<W>(rt, q) + line::lo_const<W>(q), kh = line::hi_lane<W>(rt, q) + line::hi_const<W>(q);
                    lo[q] = {p[kl], p[kh]};
                    hi[q] = {p[kl + C::PB], p[kh + C::PB]};
                }
            };
            wg_sync();
            transpose<C::HALVES>(wave < C::WAVES / 2, put, get);
            stagger<C::WAVES>(wave);
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                cf l, h;
                line::slot_inverse<W>(lo[q], hi[q], q == 0 && r0, tw.slot(q, rt), s0w, l, h);
                lo[q] = l;
                hi[q] = h;
                in_order();
            }
            settle(lo, hi);
            line::from_slots(v, r0, lo, hi);
            line::fft_inverse<W, typename C::RP>(v, X, rt, rps, tw, wave_sync);
#pragma unroll
            for (int i = 0; i < LW::NB; ++i) {
                const uint32_t o = 4u * (uint32_t)(row * W + line::n_lane<W>(rt, i));
#pragma unroll
                for (int m = 0; m < LW::R1 / 2; ++m) {
                    const cf e = v[i * LW::R1 + m], f = v[line::mirror<W>(i) * LW::R1 + LW::R1 - 1 - m];
                    *reinterpret_cast<DCT_GLOBAL float2*>(dst + 4 * line::n_const<W>(i, m) + o) = make_float2(e.x, f.x);
                    *reinterpret_cast<DCT_GLOBAL float2*>(dst + 4 * (W + line::n_const<W>(i, m)) + o) = make_float2(e.y, f.y);
                }
            }
        }
    }
}

template <int H, int W, int DIR>
int tile_run(const DeviceTables* t, const Job& j, bool persistent)
{
    using C = TileCfg<H, W>;
    int64_t grid = j.batch;
    if (persistent && grid > (int64_t)t->num_cu * (1024 / C::NT)) grid = (int64_t)t->num_cu * (1024 / C::NT);
    if (grid > 0x7fffffff) grid = 0x7fffffff;
    k_tile<H, W, DIR><<<(unsigned)grid, C::NT, 0, j.stream>>>(j.addr(), j.batch, line_s0(W), line_s0(H),
                                                              line_tab_for(t, W), line_tab_for(t, H));
    return hipGetLastError() == hipSuccess ? DCT2D_OK : DCT2D_ERR_HIP;
}

template <int H, int W>
int tile_dir(const DeviceTables* t, const Job& j, bool persistent)
{
    switch (j.dir) {
    case DCT2D_FORWARD: return tile_run<H, W, DCT2D_FORWARD>(t, j, persistent);
    case DCT2D_INVERSE: return tile_run<H, W, DCT2D_INVERSE>(t, j, persistent);
    case DIR_FILTER: return tile_run<H, W, DIR_FILTER>(t, j, persistent);
    default: return tile_run<H, W, DCT2D_ROUNDTRIP>(t, j, persistent);
    }
}

} // namespace

bool tile_shape(int rows, int cols)
{
    return is_pow2(rows) && is_pow2(cols) && rows >= 32 && cols >= 32 && rows <= 256 && cols <= 256 &&
           (rows >= 128 || cols >= 128) && !(rows == 128 && cols == 128);
}

int launch_tile(const DeviceTables* t, const Job& j, bool persistent)
{
    switch (j.rows * 1024 + j.cols) {
    case 256 * 1024 + 256: return tile_dir<256, 256>(t, j, persistent);
    case 256 * 1024 + 128: return tile_dir<256, 128>(t, j, persistent);
    case 128 * 1024 + 256: return tile_dir<128, 256>(t, j, persistent);
    case 256 * 1024 + 64: return tile_dir<256, 64>(t, j, persistent);
    case 64 * 1024 + 256: return tile_dir<64, 256>(t, j, persistent);
    case 256 * 1024 + 32: return tile_dir<256, 32>(t, j, persistent);
    case 32 * 1024 + 256: return tile_dir<32, 256>(t, j, persistent);
    case 128 * 1024 + 64: return tile_dir<128, 64>(t, j, persistent);
    case 64 * 1024 + 128: return tile_dir<64, 128>(t, j, persistent);
    case 128 * 1024 + 32: return tile_dir<128, 32>(t, j, persistent);
    case 32 * 1024 + 128: return tile_dir<32, 128>(t, j, persistent);
    default: return DCT2D_ERR_SIZE;
    }
}

} // namespace dct
