// Axes whose length is not a power of two, 8 .. 1024 (image axes such as 384, 600, 720, 1000; also
// 256 .. 1024 in images with an odd number of rows), all but p, 2p and 3p with a large prime p (mix_plan):
// one pass over HBM per axis, in place or not, each line pair transformed by a mixed-radix DFT in LDS
// (mix_fft.hpp).  No workspace and no dense table.
//
// A workgroup holds 8 or more pairs (16 values per thread), the pairs fastest in LDS, so that every
// pass reads and writes it without bank conflicts whatever the radices; twiddles come from an LDS copy
// of the length's table.  Rows are transposed on the way in and out, 128 contiguous bytes of 8 rows
// per wavefront instruction.
//
// Bound: the passes take 270 - 330 us per 2^27 elements against 178 at the copy rate.  80 to 110
// million wave instructions on the vector ALU (about 100 us) and 10 to 14 million on LDS (60 to 110 us)
// do not fully overlap with HBM at the 16 wavefronts per CU that the registers allow.
// 2^25 floats, out of place, us, the dense products before -> now (forward / round trip):
//   512 x 384  340 -> 123, 645 -> 146     600 x 1000  616 -> 153, 1193 -> 239
//   768 x 768  532 -> 132, 1018 -> 196    720 x 480   480 -> 142, 923 -> 217
// With a large prime factor the prime's pass is bound by the vector ALU, about R multiply-adds per
// complex value; 10^7 floats, forward: 822 x 712 (137, 89) 583 -> 168 us, 1004 x 1004 (251) 807 -> 349,
// 961 x 1020 (31, 17) 821 -> 87.
#include <hip/hip_runtime.h>

#include "internal.hpp"
#include "mix_fft.hpp"

namespace dct {
namespace {


__device__ __forceinline__ void mix_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

struct MixArgs {
    Addr a;
    MixPlan plan;
    uint32_t total;     // pairs of the whole batch
    uint32_t per_array; // pairs per array
    int lines;          // lines per array
    int es, ls;         // element and line stride
    const float2* tab;
    const float2* prime;       // factors of the large prime radices
    int prime_at[kMixStages];  // where those of each stage's begin
    float down, up;            // 2^-e, 2^e (see k_mix)
};

// LDS: the table (W, then c) from byte 0, then value e of slot l at (e * SLOTS + l).
extern __shared__ __attribute__((aligned(16))) char mix_lds[];

__device__ __forceinline__ float2& lds2(uint32_t byte) { return *reinterpret_cast<float2*>(mix_lds + byte); }

template <int R, int SLOTS, int NT>
__device__ __forceinline__ void mix_pass(uint32_t zb, const MixArgs& g, int stage, int tid)
{
    constexpr int IT = (16 + R - 1) / R;
    const int n = g.plan.n, m = n / R, s = g.plan.s[stage], total = SLOTS * m;
    const bool last = s * R == n;
    const uint32_t in_step = (uint32_t)(m * SLOTS * 8), out_step = (uint32_t)(s * SLOTS * 8);
    cf v[IT][R];
    uint32_t at[IT], sj8[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const int idx = tid + NT * i;
        if (idx < total) {
            const int u = idx / SLOTS;
            uint32_t o = zb + (uint32_t)idx * 8u;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float2 f = lds2(o);
                v[i][r] = {f.x, f.y};
                o += in_step;
            }
            const uint32_t sj = __umul24(s, mix::div(u, g.plan.inv_s[stage]));
            at[i] = zb + (uint32_t)idx * 8u + __umul24(sj, (R - 1) * SLOTS * 8);
            sj8[i] = sj * 8u;
        }
    }
    mix_sync();
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const int idx = tid + NT * i;
        if (idx < total) {
            mix::dft<R>(v[i]);
            uint32_t o = at[i], e = sj8[i];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                cf f = v[i][r];
                if (r > 0) {
                    if (!last) f = cmul(f, lds2(e));
                    e += sj8[i];
                }
                lds2(o) = make_float2(f.x, f.y);
                o += out_step;
            }
        }
    }
    mix_sync();
}

// A prime radix without a code of its own, R = 2 H + 1: with t_j = x_j + x_{R-j}, d_j = x_j - x_{R-j},
//   X_k, X_{R-k} = (x_0 + sum_j cos(2 pi jk / R) t_j) -+ i sum_j sin(2 pi jk / R) d_j,   k <= H.
// A lane has one butterfly, a wavefront kPrimeBlock values of k for 64 butterflies: the factors are
// the same in every lane (scalar loads from the prime's table), and one pair of LDS reads serves 4
// kPrimeBlock multiply-adds.  Outputs wait in registers until every wavefront has read its inputs;
// mix_plan admits lengths whose wavefronts then have at most two such tasks each.
template <int SLOTS, int NT>
__device__ __forceinline__ void mix_pass_prime(uint32_t zb, const MixArgs& g, int stage, int tid)
{
    constexpr int KB = kPrimeBlock, NW = NT / 64;
    const int n = g.plan.n, R = g.plan.radix[stage], H = R / 2, m = n / R, s = g.plan.s[stage], total = SLOTS * m;
    const uint32_t step = (uint32_t)(m * SLOTS * 8);
    const int groups = (total + 63) / 64, tasks = groups * ((H + KB) / KB);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    cf lo[2][KB], hi[2][KB];
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const int task = wave + NW * w;
        if (task < tasks) {
            const int blk = task / groups, b0 = (task - blk * groups) * 64 + lane, b = b0 < total ? b0 : total - 1;
            uint32_t o1 = zb + (uint32_t)b * 8u, o2 = o1 + (uint32_t)R * step;
            twptr f = (twptr)g.prime + g.prime_at[stage] + blk * H * KB;
            const float2 x0 = lds2(o1);
            cf ca[KB], sb[KB];
#pragma unroll
            for (int k = 0; k < KB; ++k) {
                ca[k] = {x0.x, x0.y};
                sb[k] = {0.f, 0.f};
            }
            // sums of 16 terms, then the sum of those: half the rounding error of one long sum at R = 251
            for (int j0 = 0; j0 < H; j0 += 16) {
                cf pc[KB], ps[KB];
#pragma unroll
                for (int k = 0; k < KB; ++k) pc[k] = ps[k] = {0.f, 0.f};
                const int end = H - j0 < 16 ? H - j0 : 16;
#pragma unroll 2
                for (int j = 0; j < end; ++j) {
                    o1 += step;
                    o2 -= step;
                    const float2 x1 = lds2(o1), x2 = lds2(o2);
                    const cf t = {x1.x + x2.x, x1.y + x2.y}, d = {x1.x - x2.x, x1.y - x2.y};
#pragma unroll
                    for (int k = 0; k < KB; ++k) {
                        const float2 c = f[k];
                        pc[k] = {pc[k].x + c.x * t.x, pc[k].y + c.x * t.y};
                        ps[k] = {ps[k].x + c.y * d.x, ps[k].y + c.y * d.y};
                    }
                    f += KB;
                }
#pragma unroll
                for (int k = 0; k < KB; ++k) {
                    ca[k] = cadd(ca[k], pc[k]);
                    sb[k] = cadd(sb[k], ps[k]);
                }
            }
#pragma unroll
            for (int k = 0; k < KB; ++k) {
                lo[w][k] = {ca[k].x + sb[k].y, ca[k].y - sb[k].x};
                hi[w][k] = {ca[k].x - sb[k].y, ca[k].y + sb[k].x};
            }
        }
    }
    mix_sync();
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const int task = wave + NW * w;
        if (task < tasks) {
            const int blk = task / groups, b = (task - blk * groups) * 64 + lane;
            if (b < total) {
                const int u = b / SLOTS, sj = s * mix::div(u, g.plan.inv_s[stage]);
                auto put = [&](cf x, int k) {
                    const cf y = cmul(x, lds2(8u * (uint32_t)(sj * k)));
                    lds2(zb + 8u * (uint32_t)((u + sj * (R - 1) + s * k) * SLOTS + b % SLOTS)) = make_float2(y.x, y.y);
                };
#pragma unroll
                for (int i = 0; i < KB; ++i) {
                    const int k = blk * KB + i;
                    if (k <= H) put(lo[w][i], k);
                    if (k > 0 && k <= H) put(hi[w][i], R - k);
                }
            }
        }
    }
    mix_sync();
}

template <int SLOTS, int NT>
__device__ __forceinline__ void mix_dft(uint32_t zb, const MixArgs& g)
{
    for (int st = 0; st < g.plan.stages; ++st) {
        // opaque, so that the addresses of every radix are formed here and not ahead of the loop, where
        // they would fill the registers
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        switch (g.plan.radix[st]) {
        case 2: mix_pass<2, SLOTS, NT>(zb, g, st, tid); break;
        case 3: mix_pass<3, SLOTS, NT>(zb, g, st, tid); break;
        case 4: mix_pass<4, SLOTS, NT>(zb, g, st, tid); break;
        case 5: mix_pass<5, SLOTS, NT>(zb, g, st, tid); break;
        case 7: mix_pass<7, SLOTS, NT>(zb, g, st, tid); break;
        case 8: mix_pass<8, SLOTS, NT>(zb, g, st, tid); break;
        case 11: mix_pass<11, SLOTS, NT>(zb, g, st, tid); break;
        case 13: mix_pass<13, SLOTS, NT>(zb, g, st, tid); break;
        case 16: mix_pass<16, SLOTS, NT>(zb, g, st, tid); break;
        default: mix_pass_prime<SLOTS, NT>(zb, g, st, tid); break;
        }
    }
}

// v index of sample j of a line
__device__ __forceinline__ int v_of(int j, int n) { return j & 1 ? n - 1 - (j >> 1) : j >> 1; }

// The inverse transform is the forward DFT with real and imaginary parts exchanged at both ends.
//
// Range: no intermediate value is much larger than the result can be, as in a product with Q_n.  Forward, the
// lines enter times 2^-e, 1 / sqrt n to 2 / sqrt n, which the factors c_k undo (unscaled, a constant image of 5e35 in
// 512 x 384, whose largest coefficient is 2.2e38, came out as infinities).  Inverse, c_k, about 0.7 / sqrt n,
// comes first and does this by itself.
template <int DIR, bool COLS, int SLOTS, int NT>
__global__ void __launch_bounds__(NT, 4) k_mix(MixArgs g)
{
    const int n = g.plan.n, half = n / 2 + 1;
    const uint32_t cb = 8u * (uint32_t)n, zb = (cb + 8u * (uint32_t)half + 15u) & ~15u;
    const DCT_GLOBAL float2* tab = (const DCT_GLOBAL float2*)g.tab;
    for (int i = threadIdx.x; i < n + half; i += NT) {
        float2 f = tab[i];
        if (DIR == DCT2D_FORWARD && i >= n) f = make_float2(f.x * g.up, f.y * g.up);
        lds2(8u * (uint32_t)i) = f;
    }

    // column tiles: 16 neighbours share an XCD
    uint32_t blk = blockIdx.x;
    if (COLS && (blk | 127u) < gridDim.x) blk = (blk & ~127u) | ((blk & 7) << 4) | ((blk & 127u) >> 3);
    const int slot = COLS ? threadIdx.x % SLOTS : 0;
    const gfloat* src = nullptr; // columns: the thread's column pair
    gfloat* dst = nullptr;
    bool col_ok = false;
    if constexpr (COLS) {
        const uint32_t q0 = blk * (uint32_t)SLOTS + slot;
        col_ok = q0 < g.total;
        const uint32_t q = col_ok ? q0 : g.total - 1, b = q / g.per_array;
        src = g.a.src(b) + 2 * (q - b * g.per_array);
        dst = g.a.dst(b) + 2 * (q - b * g.per_array);
    }
    auto val = [&](int e, int l) -> float2& { return lds2(zb + 8u * (uint32_t)(e * SLOTS + l)); };
    // rows: item i of the thread is four samples 4 q4 .. 4 q4 + 3 of the pair in slot l; the lanes of a
    // wavefront cover 8 slots x 8 groups, 128 contiguous bytes of each row (4 x 16 where there are 4)
    constexpr int SL = SLOTS < 8 ? SLOTS : 8, QL = 64 / SL, SG = SLOTS / SL, QI = SLOTS >= NT ? 8 : 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto item = [&](int i, int& l, int& q4) {
        const int tile = wave + NT / 64 * i;
        l = tile % SG * SL + lane % SL;
        q4 = tile / SG * QL + lane / SL;
        return 4 * q4 < n;
    };
    // pair of slot l: offset of its rows from the array's start, second: the distance of its second row
    auto row_of = [&](int l, uint32_t& b, int64_t& off, int& second) {
        const uint32_t q0 = blk * (uint32_t)SLOTS + l, q = q0 < g.total ? q0 : g.total - 1;
        b = q / g.per_array;
        const int r = 2 * (int)(q - b * g.per_array);
        off = (int64_t)r * g.ls;
        second = r + 1 < g.lines ? g.ls : 0;
        return q0 < g.total;
    };

    // ---- in ------------------------------------------------------------------------------
    if constexpr (COLS) {
        float2 f[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int j = threadIdx.x / SLOTS + NT / SLOTS * i;
            if (j < n) f[i] = *reinterpret_cast<const DCT_GLOBAL float2*>(src + (int64_t)j * g.es);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int j = threadIdx.x / SLOTS + NT / SLOTS * i;
            if (j < n) {
                if constexpr (DIR == DCT2D_INVERSE) val(j, slot) = f[i];
                else val(v_of(j, n), slot) = make_float2(f[i].x * g.down, f[i].y * g.down);
            }
        }
    } else {
        float4 fa[QI], fb[QI];
#pragma unroll
        for (int i = 0; i < QI; ++i) {
            int l, q4;
            if (item(i, l, q4)) {
                uint32_t b;
                int64_t off;
                int second;
                row_of(l, b, off, second);
                const gfloat* p = g.a.src(b) + off + 4 * q4;
                fa[i] = *reinterpret_cast<const gfloat4*>(p);
                fb[i] = *reinterpret_cast<const gfloat4*>(p + second);
            }
        }
#pragma unroll
        for (int i = 0; i < QI; ++i) {
            int l, q4;
            if (item(i, l, q4)) {
                float4 a = fa[i], b = fb[i];
                if constexpr (DIR != DCT2D_INVERSE) {
                    a = make_float4(a.x * g.down, a.y * g.down, a.z * g.down, a.w * g.down);
                    b = make_float4(b.x * g.down, b.y * g.down, b.z * g.down, b.w * g.down);
                }
                const int e0 = DIR == DCT2D_INVERSE ? 4 * q4 : 2 * q4, e1 = DIR == DCT2D_INVERSE ? e0 + 1 : n - 1 - 2 * q4;
                const int e2 = DIR == DCT2D_INVERSE ? e0 + 2 : e0 + 1, e3 = DIR == DCT2D_INVERSE ? e0 + 3 : e1 - 1;
                val(e0, l) = make_float2(a.x, b.x);
                val(e1, l) = make_float2(a.y, b.y);
                val(e2, l) = make_float2(a.z, b.z);
                val(e3, l) = make_float2(a.w, b.w);
            }
        }
    }
    mix_sync();
    if constexpr (DIR != DCT2D_INVERSE) mix_dft<SLOTS, NT>(zb, g);

    // ---- coefficient pairs (k, n - k) -------------------------------------------------------
    for (int idx = threadIdx.x; idx < SLOTS * half; idx += NT) {
        const int l = COLS ? slot : idx % SLOTS, k = idx / SLOTS, kh = k == 0 ? 0 : n - k;
        float2 &plo = val(k, l), &phi = val(kh, l);
        const float2 zl = plo, zh = phi, ck = lds2(cb + 8u * (uint32_t)k);
        cf xa, xb, lo, hi;
        if constexpr (DIR != DCT2D_INVERSE) {
            const float2 cu = DIR == DCT2D_FORWARD ? ck : make_float2(ck.x * g.up, ck.y * g.up);
            line::slot_forward<0>({zl.x, zl.y}, {zh.x, zh.y}, false, cu, 0.f, xa, xb);
        } else {
            xa = {zl.x, zh.x};
            xb = {zl.y, zh.y};
        }
        if constexpr (DIR == DCT2D_FORWARD) {
            if constexpr (COLS) {
                if (col_ok) {
                    *reinterpret_cast<DCT_GLOBAL float2*>(dst + (int64_t)k * g.es) = make_float2(xa.x, xb.x);
                    if (kh != k) *reinterpret_cast<DCT_GLOBAL float2*>(dst + (int64_t)kh * g.es) = make_float2(xa.y, xb.y);
                }
            } else {
                plo = make_float2(xa.x, xb.x);
                if (kh != k) phi = make_float2(xa.y, xb.y);
            }
        } else {
            if (k == 0) xa.y = xb.y = 0.f; // coefficient 0 has no partner
            line::slot_inverse<0>(xa, xb, false, ck, 0.f, lo, hi);
            if (k == 0) lo = cadd(lo, hi);
            plo = make_float2(lo.y, lo.x);
            if (kh != k) phi = make_float2(hi.y, hi.x);
        }
    }
    if constexpr (DIR == DCT2D_FORWARD && COLS) return;
    mix_sync();
    if constexpr (DIR != DCT2D_FORWARD) mix_dft<SLOTS, NT>(zb, g);

    // ---- out -----------------------------------------------------------------------------
    if constexpr (COLS) {
        for (int j = threadIdx.x / SLOTS; j < n; j += NT / SLOTS) {
            const float2 f = val(v_of(j, n), slot);
            if (col_ok) *reinterpret_cast<DCT_GLOBAL float2*>(dst + (int64_t)j * g.es) = make_float2(f.y, f.x);
        }
    } else {
#pragma unroll
        for (int i = 0; i < QI; ++i) {
            int l, q4;
            if (item(i, l, q4)) {
                uint32_t b;
                int64_t off;
                int second;
                const bool ok = row_of(l, b, off, second);
                const int e0 = DIR == DCT2D_FORWARD ? 4 * q4 : 2 * q4, e1 = DIR == DCT2D_FORWARD ? e0 + 1 : n - 1 - 2 * q4;
                const int e2 = DIR == DCT2D_FORWARD ? e0 + 2 : e0 + 1, e3 = DIR == DCT2D_FORWARD ? e0 + 3 : e1 - 1;
                const float2 f0 = val(e0, l), f1 = val(e1, l), f2 = val(e2, l), f3 = val(e3, l);
                const float4 x = make_float4(f0.x, f1.x, f2.x, f3.x), y = make_float4(f0.y, f1.y, f2.y, f3.y);
                if (ok) {
                    gfloat* o = g.a.dst(b) + off + 4 * q4;
                    *reinterpret_cast<gfloat4*>(o) = DIR == DCT2D_FORWARD ? x : y;
                    if (second) *reinterpret_cast<gfloat4*>(o + second) = DIR == DCT2D_FORWARD ? y : x;
                }
            }
        }
    }
}

template <bool COLS, int SLOTS, int NT>
int mix_run(const MixArgs& g, int dir, hipStream_t s)
{
    const unsigned grid = (unsigned)(((int64_t)g.total + SLOTS - 1) / SLOTS);
    const size_t lds = sizeof(float2) * ((size_t)SLOTS * g.plan.n + mix_table_size(g.plan.n) + 1);
    switch (dir) {
    case DCT2D_FORWARD: k_mix<DCT2D_FORWARD, COLS, SLOTS, NT><<<grid, NT, lds, s>>>(g); break;
    case DCT2D_INVERSE: k_mix<DCT2D_INVERSE, COLS, SLOTS, NT><<<grid, NT, lds, s>>>(g); break;
    default: k_mix<DCT2D_ROUNDTRIP, COLS, SLOTS, NT><<<grid, NT, lds, s>>>(g); break;
    }
    return hipGetLastError() == hipSuccess ? DCT2D_OK : DCT2D_ERR_HIP;
}

template <bool COLS>
int mix_slots(const MixArgs& g, int dir, hipStream_t s)
{
    const MixShape shape = mix_shape(g.plan.n);
    switch (shape.slots) {
    case 8: return shape.threads == 512 ? mix_run<COLS, 8, 512>(g, dir, s) : mix_run<COLS, 8, 256>(g, dir, s);
    case 16: return mix_run<COLS, 16, 256>(g, dir, s);
    case 32: return mix_run<COLS, 32, 256>(g, dir, s);
    case 128: return mix_run<COLS, 128, 256>(g, dir, s);
    default: return mix_run<COLS, 256, 256>(g, dir, s);
    }
}

} // namespace

bool mix_smooth(int n)
{
    MixPlan p;
    return mix_plan(n, p);
}

int launch_mix_axis(const DeviceTables* t, const Addr& a, int64_t batch, int rows, int cols, bool column_pass, int dir,
                    hipStream_t s)
{
    const int n = column_pass ? rows : cols;
    MixArgs g{};
    if (!mix_plan(n, g.plan)) return DCT2D_ERR_SIZE;
    g.a = a;
    g.lines = column_pass ? cols : rows;
    g.es = column_pass ? cols : 1;
    g.ls = column_pass ? 1 : cols;
    g.tab = t->mix_tab + mix_table_offset(n);
    g.prime = t->prime_tab;
    for (int i = 0; i < g.plan.stages; ++i)
        if (g.plan.radix[i] > 16) g.prime_at[i] = prime_table_offset(g.plan.radix[i]);
    g.up = 1.f;
    while (4.f * g.up * g.up <= n) g.up *= 2.f; // the largest power of two up to sqrt n
    g.down = 1.f / g.up;
    g.per_array = (uint32_t)((g.lines + 1) / 2);
    const int64_t total = batch * g.per_array;
    if (total > 0x7fffffff) return DCT2D_ERR_ARG;
    g.total = (uint32_t)total;
    return column_pass ? mix_slots<true>(g, dir, s) : mix_slots<false>(g, dir, s);
}

} // namespace dct
