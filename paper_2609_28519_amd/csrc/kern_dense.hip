// Dense column pass for whole images: the transform of length L = rows along the columns of a batch
// of h x w images, by a float32 matrix product with the dense Q_L of eq. 1 (Section 2.1; arbitrary
// axes, Section 7.1).  Used for the image heights that the line transforms leave out, p and 2p with a
// prime p of 131 or more and 3p with one of 89 or more (252 of the lengths 8 .. 1024); zero-padding would
// change the transform.  (Widths are multiples of 4 and never among them.)
//
// Q_L's even rows are symmetric and its odd rows antisymmetric about the middle, so with
// E = ceil(L / 2)
//   forward  Y[2k]   = sum_{n < E} Q_L[2k][n]   (x[n] + x[L-1-n])
//            Y[2k+1] = sum_{n < E} Q_L[2k+1][n] (x[n] - x[L-1-n])
//   inverse  a[n] = sum_k Q_L[2k][n] Y[2k],  b[n] = sum_k Q_L[2k+1][n] Y[2k+1],  n < E,
//            x[n] = a[n] + b[n],  x[L-1-n] = a[n] - b[n]
// (odd L: the middle sample n = E - 1 enters once, and b[E-1] = 0): two products of half the depth,
// with the butterflies fused into the operand loads (forward) or the stores (inverse).
//
// A 256-thread workgroup computes the 64 x 64 tiles of both products for the same positions on the
// matrix cores in float32 (v_mfma_f32_32x32x2f32, each wavefront a 32 x 32 sub-tile of each), over the
// depth in chunks of 16 staged in LDS, the next chunk fetched into registers meanwhile.  The 16
// products of a chunk are summed in a fresh accumulator that is then added to the running sum
// (blocked summation), which keeps the float32 accumulation error near 4 unit roundoffs at L = 1024 instead of growing like
// sqrt(L/6).
// Bound: the matrix cores, 157 TFLOP/s of float32.  The plain product on the vector ALU that these
// lengths took before did twice the operations (10^7 floats in images of 997 x 600, both passes: 509 -> 212 us forward).
#include <hip/hip_runtime.h>

#include "internal.hpp"

namespace dct {
namespace {

constexpr int BM = 64, BN = 64, BK = 16;
typedef float f32x16 __attribute__((ext_vector_type(16)));

// One chunk's operands as loaded from HBM, before the butterflies: u, v from the image (four
// neighbouring columns), b1, b2 from Q_L's even and odd rows; zeros outside the matrices.
struct Chunk {
    float4 u, v;
    float b1[4], b2[4];
};

template <bool INV>
__device__ __forceinline__ Chunk fetch(const gfloat* x, const gfloat* q, int L, int cols, int i0, int j0, int k0, int t)
{
    const int E = (L + 1) / 2;
    Chunk r{};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // forward: output pair h = i0 + t / 4, depth n; inverse: output sample n, depth pair k
        const int h = INV ? k0 + t / 16 : i0 + t / 4, n = INV ? i0 + 4 * (t % 16) + i : k0 + 4 * (t % 4) + i;
        if (h < E && n < E) {
            r.b1[i] = q[(int64_t)(2 * h) * L + n];
            if (2 * h + 1 < L) r.b2[i] = q[(int64_t)(2 * h + 1) * L + n];
        }
    }
    const int k = k0 + t / 16, j = j0 + 4 * (t % 16);
    if (k < E && j < cols) {
        const int hi = INV ? 2 * k + 1 : L - 1 - k;
        r.u = *reinterpret_cast<const gfloat4*>(x + (int64_t)(INV ? 2 * k : k) * cols + j);
        if (INV ? hi < L : hi > k) r.v = *reinterpret_cast<const gfloat4*>(x + (int64_t)hi * cols + j);
    }
    return r;
}

// The chunk into the LDS operand tiles: A (BM x BK, k-major), B (BK x BN), 1 of the even and 2 of the
// odd product.
template <bool INV>
__device__ __forceinline__ void stage(const Chunk& r, bool middle, float (*A1)[BM + 4], float (*A2)[BM + 4],
                                      float (*B1)[BN + 4], float (*B2)[BN + 4], int t)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = INV ? t / 16 : 4 * (t % 4) + i, m = INV ? 4 * (t % 16) + i : t / 4;
        A1[k][m] = r.b1[i];
        A2[k][m] = r.b2[i];
    }
    float4 p = r.u, m = r.v;
    if (!INV) {
        p = make_float4(r.u.x + r.v.x, r.u.y + r.v.y, r.u.z + r.v.z, r.u.w + r.v.w);
        m = make_float4(r.u.x - r.v.x, r.u.y - r.v.y, r.u.z - r.v.z, r.u.w - r.v.w);
        if (middle) m = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    *reinterpret_cast<float4*>(&B1[t / 16][4 * (t % 16)]) = p;
    *reinterpret_cast<float4*>(&B2[t / 16][4 * (t % 16)]) = m;
}

template <bool INV>
__global__ void __launch_bounds__(256) k_dense_cols(Addr a, const float* __restrict__ q_in, int L, int cols)
{
    __shared__ __attribute__((aligned(16))) float A1[BK][BM + 4];
    __shared__ __attribute__((aligned(16))) float A2[BK][BM + 4];
    __shared__ __attribute__((aligned(16))) float B1[BK][BN + 4];
    __shared__ __attribute__((aligned(16))) float B2[BK][BN + 4];
    const int t = threadIdx.x, E = (L + 1) / 2;
    const gfloat* x = a.src(blockIdx.z);
    gfloat* dst = a.dst(blockIdx.z);
    const gfloat* q = (const gfloat*)q_in;
    const int i0 = blockIdx.y * BM, j0 = blockIdx.x * BN;
    const int lane = t & 63, wi = (t >> 6) >> 1, wj = (t >> 6) & 1;
    f32x16 acc1, acc2;
#pragma unroll
    for (int r = 0; r < 16; ++r) { acc1[r] = 0.f; acc2[r] = 0.f; }
    Chunk nx = fetch<INV>(x, q, L, cols, i0, j0, 0, t);
    for (int k0 = 0; k0 < E; k0 += BK) {
        // a depth row past the matrix is all zeros; the middle sample of an odd L has no partner
        stage<INV>(nx, k0 + t / 16 == L - 1 - (k0 + t / 16), A1, A2, B1, B2, t);
        if (k0 + BK < E) nx = fetch<INV>(x, q, L, cols, i0, j0, k0 + BK, t);
        __syncthreads();
        // v_mfma_f32_32x32x2f32 takes A[i][k] from lane i + 32 k and B[k][j] from lane j + 32 k
        f32x16 p1, p2;
#pragma unroll
        for (int r = 0; r < 16; ++r) { p1[r] = 0.f; p2[r] = 0.f; }
#pragma unroll
        for (int kk = 0; kk < BK / 2; ++kk) {
            const int k = 2 * kk + (lane >> 5);
            p1 = __builtin_amdgcn_mfma_f32_32x32x2f32(A1[k][32 * wi + (lane & 31)], B1[k][32 * wj + (lane & 31)], p1, 0, 0, 0);
            p2 = __builtin_amdgcn_mfma_f32_32x32x2f32(A2[k][32 * wi + (lane & 31)], B2[k][32 * wj + (lane & 31)], p2, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) { acc1[r] += p1[r]; acc2[r] += p2[r]; }
        __syncthreads();
    }
    // register r of the lane holds sub-tile row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32
    const int j = j0 + 32 * wj + (lane & 31);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = i0 + 32 * wi + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (i >= E || j >= cols) continue;
        if (INV) {
            dst[(int64_t)i * cols + j] = acc1[r] + acc2[r];
            if (L - 1 - i != i) dst[(int64_t)(L - 1 - i) * cols + j] = acc1[r] - acc2[r];
        } else {
            dst[(int64_t)(2 * i) * cols + j] = acc1[r];
            if (2 * i + 1 < L) dst[(int64_t)(2 * i + 1) * cols + j] = acc2[r];
        }
    }
}

} // namespace

// The column pass of `count` images of rows x cols (cols a multiple of 4), read through a.src and
// written through a.dst, which must not overlap.  q: dense Q_rows, row-major, float32.
int launch_dense_columns(const Addr& a, int64_t count, int rows, int cols, bool inverse, const float* q, hipStream_t s)
{
    if (count <= 0) return DCT2D_OK;
    if (count > 65535) return DCT2D_ERR_ARG;
    const dim3 grid((cols + BN - 1) / BN, ((rows + 1) / 2 + BM - 1) / BM, (unsigned)count);
    if (inverse) k_dense_cols<true><<<grid, 256, 0, s>>>(a, q, rows, cols);
    else k_dense_cols<false><<<grid, 256, 0, s>>>(a, q, rows, cols);
    return hipGetLastError() == hipSuccess ? DCT2D_OK : DCT2D_ERR_HIP;
}

} // namespace dct
