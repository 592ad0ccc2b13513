// Bands: one axis of 8 or 16, the other of 128 or 256.  A wavefront owns a tile of whole arrays with 4096
// values, 64 per thread; the data crosses HBM once each way and no barrier couples wavefronts (four of
// them share a workgroup for its copy of the twiddles).  The long lines are transformed in pairs
// (line_fft.hpp), the short ones by a thread each (dct1d.hpp), and the tile changes hands through the
// wavefront's part of LDS.
//   wide (rows of 128, 256): row pairs straight from HBM | a lane per column, 2 or 4 columns each, which
//     leave in whole 256-byte runs
//   tall: a lane per row, 4 or 8 rows each, straight from HBM | column pairs
// Bound: HBM; the LDS tile allows two workgroups (8 wavefronts) per CU.
// 2^27 floats, out of place, us, the best other variant -> this one, forward / inverse / round trip (the copy
// ceiling is 176):
//     8 x 128   468 451 698 -> 230 261 247     128 x 8    429 441 636 -> 242 240 321
//    16 x 128   441 450 700 -> 216 222 251    128 x 16    432 435 654 -> 209 258 311
//     8 x 256   284 260 443 -> 223 238 237     256 x 8    315 319 505 -> 229 234 317
//    16 x 256   282 263 456 -> 202 205 239    256 x 16    328 301 511 -> 202 260 304
#include "fp32_common.hpp"
#include "line_fft.hpp"

namespace dct {
namespace {

constexpr int kBandWaves = 4;

__device__ __forceinline__ void wave_sync() { asm volatile("" ::: "memory"); } // a wavefront's LDS accesses are in order

// Long axis N, short axis S.
template <int N, int S, bool WIDE>
struct BandCfg {
    static constexpr int A = 4096 / (N * S), LINES = A * S; // arrays and long lines per tile
    static constexpr int PAIRS = 64 / LineCfg<N>::TPL;
    static_assert(2 * PAIRS == LINES, "a wavefront holds the tile's line pairs");
    using P = line::Place<N, !WIDE, PAIRS>;
    // wide: row r of the tile at r * PT; tall: row r unpadded, its 16-byte groups XOR-permuted by a row
    // key (both a lane per row and the column pairs of one row then touch different banks)
    static constexpr int PT = N + 4;
    static constexpr int TILE = WIDE ? LINES * PT : N * LINES;
    static constexpr int FLOATS = TILE > P::FLOATS ? TILE : P::FLOATS;
    static constexpr int TAB = 2 * LineCfg<N>::TAB;
    __device__ static int key(int r) { return LINES == 16 ? (r >> 1) & 3 : r & 7; }
    __device__ static int at(int r, int c) { return r * LINES + (((c >> 2) ^ key(r)) << 2) + (c & 3); }
};

__device__ __forceinline__ void pin4(cf& a, cf& b)
{
    asm volatile("" : "+v"(a.x), "+v"(a.y), "+v"(b.x), "+v"(b.y));
}

template <int N>
__device__ __forceinline__ void copy_table(float* lds, const float2* tab)
{
    for (int i = threadIdx.x; i < 2 * LineCfg<N>::TAB / 4; i += 64 * kBandWaves)
        *reinterpret_cast<float4*>(lds + 4 * i) = *((const gfloat4*)tab + i);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int H, int W, int DIR>
__global__ void __launch_bounds__(64 * kBandWaves, 2)
k_band_wide(Addr a, int64_t batch, float s0, const float2* __restrict__ tab, const float2* __restrict__ twh_in)
{
    using C = BandCfg<W, H, true>;
    using L = LineCfg<W>;
    __shared__ __attribute__((aligned(16))) float lds[C::TAB + kBandWaves * C::FLOATS];
    copy_table<W>(lds, tab);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t b0 = ((int64_t)blockIdx.x * kBandWaves + wave) * C::A;
    if (b0 >= batch) return;
    float* const T = lds + C::TAB + wave * C::FLOATS;
    line::Twiddles<W> tw;
    tw.tab = reinterpret_cast<const float2*>(lds);
    const int ps = lane / L::TPL, t = lane % L::TPL, row = 2 * ps;
    const bool t0 = t == 0;
    // the row pair's array (a slot past the batch transforms a copy of the last array and stores nothing)
    const int64_t bl = b0 + row / H;
    const bool ok = bl < batch;
    cf v[32], lo[16], hi[16];
    if constexpr (DIR != DCT2D_INVERSE) {
        const gfloat* src = a.src(ok ? bl : batch - 1) + row % H * W;
#pragma unroll
        for (int i = 0; i < L::NB; ++i) {
            const gfloat* p = src + line::n_lane<W>(t, i);
#pragma unroll
            for (int m = 0; m < L::R1 / 2; ++m) {
                const float2 fa = *reinterpret_cast<const DCT_GLOBAL float2*>(p + line::n_const<W>(i, m));
                const float2 fb = *reinterpret_cast<const DCT_GLOBAL float2*>(p + W + line::n_const<W>(i, m));
                v[i * L::R1 + m] = {fa.x, fb.x};
                v[line::mirror<W>(i) * L::R1 + L::R1 - 1 - m] = {fa.y, fb.y};
            }
        }
        line::fft_forward<W, typename C::P>(v, T, t, ps, tw, wave_sync);
        line::to_slots(v, t0, lo, hi);
        float* p = T + row * C::PT;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            cf xa, xb;
            line::slot_forward<W>(lo[q], hi[q], q == 0 && t0, tw.slot(q, t), s0, xa, xb);
            const int kl = line::lo_lane<W>(t, q) + line::lo_const<W>(q), kh = line::hi_lane<W>(t, q) + line::hi_const<W>(q);
            p[kl] = xa.x;
            p[kh] = xa.y;
            p[kl + C::PT] = xb.x;
            p[kh + C::PT] = xb.y;
        }
        wave_sync();
    }
    // ---- columns: lane's column lane + 64 i of every array
#pragma unroll 1
    for (int i = 0; i < W / 64; ++i) {
        const int c = lane + 64 * i;
#pragma unroll 1
        for (int k = 0; k < C::A; ++k) {
            const int64_t b = b0 + k < batch ? b0 + k : batch - 1;
            const twptr twh = per_iteration(twh_in);
            float* p = T + k * H * C::PT + c;
            float x[H];
            if constexpr (DIR == DCT2D_INVERSE) {
                const gfloat* src = a.src(b) + c;
#pragma unroll
                for (int r = 0; r < H; ++r) x[r] = src[r * W];
            } else {
#pragma unroll
                for (int r = 0; r < H; ++r) x[r] = p[r * C::PT];
            }
            if constexpr (DIR == DIR_FILTER) filter1d<H>(x, a.lam_for(b) + c, W, twh);
            else apply1d<H, DIR>(x, twh);
            if constexpr (DIR == DCT2D_FORWARD) {
                gfloat* dst = a.dst(b) + c;
                if (b0 + k < batch)
#pragma unroll
                    for (int r = 0; r < H; ++r) dst[r * W] = x[r];
            } else {
#pragma unroll
                for (int r = 0; r < H; ++r) p[r * C::PT] = x[r];
            }
        }
    }
    if constexpr (DIR == DCT2D_FORWARD) return;
    wave_sync();
    {
        const float* p = T + row * C::PT;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int kl = line::lo_lane<W>(t, q) + line::lo_const<W>(q), kh = line::hi_lane<W>(t, q) + line::hi_const<W>(q);
            const cf xa = {p[kl], p[kh]}, xb = {p[kl + C::PT], p[kh + C::PT]};
            line::slot_inverse<W>(xa, xb, q == 0 && t0, tw.slot(q, t), s0, lo[q], hi[q]);
        }
    }
    line::from_slots(v, t0, lo, hi);
    wave_sync();
    line::fft_inverse<W, typename C::P>(v, T, t, ps, tw, wave_sync);
    if (ok) {
        gfloat* dst = a.dst(bl) + row % H * W;
#pragma unroll
        for (int i = 0; i < L::NB; ++i) {
            gfloat* p = dst + line::n_lane<W>(t, i);
#pragma unroll
            for (int m = 0; m < L::R1 / 2; ++m) {
                const cf e = v[i * L::R1 + m], f = v[line::mirror<W>(i) * L::R1 + L::R1 - 1 - m];
                *reinterpret_cast<DCT_GLOBAL float2*>(p + line::n_const<W>(i, m)) = make_float2(e.x, f.x);
                *reinterpret_cast<DCT_GLOBAL float2*>(p + W + line::n_const<W>(i, m)) = make_float2(e.y, f.y);
            }
        }
    }
}

template <int H, int W, int DIR>
__global__ void __launch_bounds__(64 * kBandWaves, 2)
k_band_tall(Addr a, int64_t batch, float s0, const float2* __restrict__ tab, const float2* __restrict__ tww_in)
{
    using C = BandCfg<H, W, false>;
    using L = LineCfg<H>;
    __shared__ __attribute__((aligned(16))) float lds[C::TAB + kBandWaves * C::FLOATS];
    copy_table<H>(lds, tab);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t b0 = ((int64_t)blockIdx.x * kBandWaves + wave) * C::A;
    if (b0 >= batch) return;
    float* const T = lds + C::TAB + wave * C::FLOATS;
    line::Twiddles<H> tw;
    tw.tab = reinterpret_cast<const float2*>(lds);
    const int ps = lane % C::PAIRS, t = lane / C::PAIRS, col = 2 * ps;
    const bool t0 = t == 0;
    const int64_t bl = b0 + col / W;
    const bool ok = bl < batch;
    cf v[32], lo[16], hi[16];
    // rows: lane's row (64 i + lane) % H of array 64 i / H
    auto rows = [&](auto inv) {
        constexpr bool INV = decltype(inv)::value;
#pragma unroll 1
        for (int i = 0; i < C::A * H / 64; ++i) {
            const int k = 64 * i / H, r = 64 * i % H + lane;
            const int64_t b = b0 + k < batch ? b0 + k : batch - 1;
            const twptr tww = per_iteration(tww_in);
            float x[W];
            if constexpr (!INV) {
                const gfloat* src = a.src(b) + r * W;
#pragma unroll
                for (int j = 0; j < W / 4; ++j) {
                    const float4 f = *reinterpret_cast<const gfloat4*>(src + 4 * j);
                    x[4 * j] = f.x; x[4 * j + 1] = f.y; x[4 * j + 2] = f.z; x[4 * j + 3] = f.w;
                }
                dct2_ortho<W>(x, tww);
#pragma unroll
                for (int j = 0; j < W / 4; ++j)
                    *reinterpret_cast<float4*>(T + C::at(r, k * W + 4 * j)) = make_float4(x[4 * j], x[4 * j + 1], x[4 * j + 2], x[4 * j + 3]);
            } else {
#pragma unroll
                for (int j = 0; j < W / 4; ++j) {
                    const float4 f = *reinterpret_cast<const float4*>(T + C::at(r, k * W + 4 * j));
                    x[4 * j] = f.x; x[4 * j + 1] = f.y; x[4 * j + 2] = f.z; x[4 * j + 3] = f.w;
                }
                dct3_ortho<W>(x, tww);
                gfloat* dst = a.dst(b) + r * W;
                if (b0 + k < batch)
#pragma unroll
                    for (int j = 0; j < W / 4; ++j)
                        *reinterpret_cast<gfloat4*>(dst + 4 * j) = make_float4(x[4 * j], x[4 * j + 1], x[4 * j + 2], x[4 * j + 3]);
            }
        }
    };
    const gfloat* src = a.src(ok ? bl : batch - 1) + col % W;
    if constexpr (DIR != DCT2D_INVERSE) {
        rows(std::false_type{});
        wave_sync();
#pragma unroll
        for (int i = 0; i < L::NB; ++i) {
            const int nl = line::n_lane<H>(t, i);
#pragma unroll
            for (int m = 0; m < L::R1 / 2; ++m) {
                const int r = nl + line::n_const<H>(i, m);
                const float2 e = *reinterpret_cast<const float2*>(T + C::at(r, col)), f = *reinterpret_cast<const float2*>(T + C::at(r + 1, col));
                v[i * L::R1 + m] = {e.x, e.y};
                v[line::mirror<H>(i) * L::R1 + L::R1 - 1 - m] = {f.x, f.y};
            }
        }
        wave_sync();
        line::fft_forward<H, typename C::P>(v, T, t, ps, tw, wave_sync);
        line::to_slots(v, t0, lo, hi);
    } else {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const float2 l = *reinterpret_cast<const DCT_GLOBAL float2*>(src + (line::lo_lane<H>(t, q) + line::lo_const<H>(q)) * W);
            const float2 h = *reinterpret_cast<const DCT_GLOBAL float2*>(src + (line::hi_lane<H>(t, q) + line::hi_const<H>(q)) * W);
            lo[q] = {l.x, h.x};
            hi[q] = {l.y, h.y};
        }
    }
    gfloat* dst = a.dst(ok ? bl : batch - 1) + col % W;
    const gfloat* lam = DIR == DIR_FILTER ? a.lam_for(ok ? bl : batch - 1) + col % W : nullptr;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        cf xa, xb;
        const float2 c = tw.slot(q, t);
        const int kl = (line::lo_lane<H>(t, q) + line::lo_const<H>(q)) * W, kh = (line::hi_lane<H>(t, q) + line::hi_const<H>(q)) * W;
        if constexpr (DIR != DCT2D_INVERSE) line::slot_forward<H>(lo[q], hi[q], q == 0 && t0, c, s0, xa, xb);
        else { xa = lo[q]; xb = hi[q]; }
        if constexpr (DIR == DCT2D_FORWARD) {
            if (ok) {
                *reinterpret_cast<DCT_GLOBAL float2*>(dst + kl) = make_float2(xa.x, xb.x);
                *reinterpret_cast<DCT_GLOBAL float2*>(dst + kh) = make_float2(xa.y, xb.y);
            }
        } else {
            // opaque around the multiply, so that multipliers of one reproduce the round trip bit for bit
            if constexpr (DIR >= DCT2D_ROUNDTRIP) pin4(xa, xb);
            if constexpr (DIR == DIR_FILTER) {
                xa = {xa.x * lam[kl], xa.y * lam[kh]};
                xb = {xb.x * lam[kl + 1], xb.y * lam[kh + 1]};
            }
            if constexpr (DIR >= DCT2D_ROUNDTRIP) pin4(xa, xb);
            line::slot_inverse<H>(xa, xb, q == 0 && t0, c, s0, lo[q], hi[q]);
        }
    }
    if constexpr (DIR == DCT2D_FORWARD) return;
    line::from_slots(v, t0, lo, hi);
    line::fft_inverse<H, typename C::P>(v, T, t, ps, tw, wave_sync);
#pragma unroll
    for (int i = 0; i < L::NB; ++i) {
        const int nl = line::n_lane<H>(t, i);
#pragma unroll
        for (int m = 0; m < L::R1 / 2; ++m) {
            const int r = nl + line::n_const<H>(i, m);
            const cf e = v[i * L::R1 + m], f = v[line::mirror<H>(i) * L::R1 + L::R1 - 1 - m];
            *reinterpret_cast<float2*>(T + C::at(r, col)) = make_float2(e.x, e.y);
            *reinterpret_cast<float2*>(T + C::at(r + 1, col)) = make_float2(f.x, f.y);
        }
    }
    wave_sync();
    rows(std::true_type{});
}

template <int H, int W, int DIR>
int band_run(const DeviceTables* t, const Job& j)
{
    constexpr int N = H > W ? H : W, PER = 4096 / (H * W) * kBandWaves;
    const int64_t grid = (j.batch + PER - 1) / PER;
    if (grid > 0x7fffffff) return DCT2D_ERR_ARG;
    const float s0 = line_s0(N);
    if constexpr (W > H)
        k_band_wide<H, W, DIR><<<(unsigned)grid, 64 * kBandWaves, 0, j.stream>>>(j.addr(), j.batch, s0, line_tab_for(t, N), tw_for(t, H));
    else
        k_band_tall<H, W, DIR><<<(unsigned)grid, 64 * kBandWaves, 0, j.stream>>>(j.addr(), j.batch, s0, line_tab_for(t, N), tw_for(t, W));
    return hipGetLastError() == hipSuccess ? DCT2D_OK : DCT2D_ERR_HIP;
}

template <int H, int W>
int band_dir(const DeviceTables* t, const Job& j)
{
    switch (j.dir) {
    case DCT2D_FORWARD: return band_run<H, W, DCT2D_FORWARD>(t, j);
    case DCT2D_INVERSE: return band_run<H, W, DCT2D_INVERSE>(t, j);
    case DIR_FILTER: return band_run<H, W, DIR_FILTER>(t, j);
    default: return band_run<H, W, DCT2D_ROUNDTRIP>(t, j);
    }
}

} // namespace

bool band_shape(int rows, int cols)
{
    const int s = rows < cols ? rows : cols, l = rows < cols ? cols : rows;
    return (s == 8 || s == 16) && (l == 128 || l == 256);
}

int launch_band(const DeviceTables* t, const Job& j)
{
    switch (j.rows * 1024 + j.cols) {
    case 8 * 1024 + 128: return band_dir<8, 128>(t, j);
    case 16 * 1024 + 128: return band_dir<16, 128>(t, j);
    case 8 * 1024 + 256: return band_dir<8, 256>(t, j);
    case 16 * 1024 + 256: return band_dir<16, 256>(t, j);
    case 128 * 1024 + 8: return band_dir<128, 8>(t, j);
    case 128 * 1024 + 16: return band_dir<128, 16>(t, j);
    case 256 * 1024 + 8: return band_dir<256, 8>(t, j);
    case 256 * 1024 + 16: return band_dir<256, 16>(t, j);
    default: return DCT2D_ERR_SIZE;
    }
}

} // namespace dct
