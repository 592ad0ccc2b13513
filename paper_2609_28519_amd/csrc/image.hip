// Batched transforms of whole images of any shape with both axes in [8, 1024] (columns a
// multiple of 4): the strided-batch counterpart of the ragged planner's image classes.
//
// Shapes whose axes are both powers of two go to the kernels of the basic calls: up to 256
// the frozen float32-accurate path, with an axis of 512 or 1024 the two-pass line kernels
// (kern_line.hip).  Every other shape is computed exactly, without zero-padding, axis by axis
// (launch_image): a power-of-two axis by the line kernels, other lengths (384, 600, 1000) by the
// mixed-radix kernels (kern_mix.hip), each in place on the output; heights
// p, 2p and 3p with a large prime p (mix_plan) from the dense Q_n of eq. 1 (FP64-generated, rounded to float32,
// kern_dense.hip).  The dense pass writes its output tile from whole input columns, so it goes
// through a workspace of one float32 image per image of the batch.
//
// dct2d_image_transform takes its workspace from the stream-ordered allocator
// (hipMallocAsync / hipFreeAsync on the caller's stream, so concurrent calls on different
// streams never share it) and keeps one dense Q_n per device and length, built on first
// use.  dct2d_image_transform_noalloc is the same computation for callers that cannot
// allocate: its Q tables and workspace live in `scratch`, a fixed device array of this
// file, and the batch is processed in chunks that fit.
#include <hip/hip_runtime.h>

#include <map>
#include <mutex>
#include <utility>

#include "internal.hpp"

using namespace dct;

namespace {

// ---- the no-allocation scratch ---------------------------------------------------------
// 64 MiB per device, held from the library's load until the process ends.  Layout per
// call of a height that takes the dense product: Q_rows, then the workspace, 256-byte
// aligned.  The largest (1021 x 1024) needs 4 MiB of table and 4 MiB per image of
// workspace, so every accepted shape fits at least one image per chunk (other shapes do not
// use the scratch).
constexpr size_t kScratchBytes = size_t(64) << 20;
__device__ __align__(256) float scratch[kScratchBytes / sizeof(float)];

constexpr int kMaxDevices = 64;
std::mutex g_mu;
// device address of `scratch` per device (the host-side name is only a stand-in)
float* g_scratch[kMaxDevices] = {};
// dense Q_n cache of the allocating entry point: (device, n) -> device table
std::map<std::pair<int, int>, float*> g_q;

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

// Images per launch of the passes without a workspace.  A launch holds fewer than 2^32 threads and the line
// kernels count their tiles in 31 bits; a pass has at most a thread per 7 values (33 x 33: 32 pairs to
// 256 threads) and a pair to at least 14, so 2^34 values at a time stay inside both.
int64_t line_chunk(int rows, int cols) { return (int64_t(1) << 34) / ((int64_t)rows * cols); }

bool fast_shape(int r, int c) { return is_pow2(r) && is_pow2(c) && r >= 8 && r <= 256 && c >= 8 && c <= 256; }
// power-of-two shapes with an axis of 512 or 1024: two line passes (no workspace)
bool long_shape(int r, int c) { return is_pow2(r) && is_pow2(c) && r >= 8 && c >= 8 && r <= 1024 && c <= 1024 && (r > 256 || c > 256); }

int validate(int dir, const float* in, const float* out, int64_t batch, int rows, int cols, int64_t in_stride,
             int64_t out_stride)
{
    if (dir < DCT2D_FORWARD || dir > DCT2D_ROUNDTRIP || batch < 0) return DCT2D_ERR_ARG;
    if (rows < 8 || cols < 8 || rows > 1024 || cols > 1024 || (cols & 3)) return DCT2D_ERR_SIZE;
    const int64_t n = (int64_t)rows * cols;
    if (in_stride < n || out_stride < n) return DCT2D_ERR_STRIDE;
    if (batch == 0) return DCT2D_OK;
    if (!in || !out) return DCT2D_ERR_ARG;
    if ((reinterpret_cast<uintptr_t>(in) & 15u) || (reinterpret_cast<uintptr_t>(out) & 15u) || (in_stride & 3) ||
        (out_stride & 3))
        return DCT2D_ERR_ALIGN;
    if (in == out) {
        if (batch > 1 && in_stride != out_stride) return DCT2D_ERR_ARG;
    } else {
        const char* a0 = reinterpret_cast<const char*>(in);
        const char* a1 = a0 + ((batch - 1) * in_stride + n) * 4;
        const char* b0 = reinterpret_cast<const char*>(out);
        const char* b1 = b0 + ((batch - 1) * out_stride + n) * 4;
        if (a0 < b1 && b0 < a1) return DCT2D_ERR_ARG;
    }
    return DCT2D_OK;
}

// Cached dense Q_n of the current device (allocating entry point only).
const float* cached_q(int device, int n, int* err)
{
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_q.find({device, n});
    if (it != g_q.end()) return it->second;
    float* q = nullptr;
    if (hipMalloc(&q, (size_t)n * n * sizeof(float)) != hipSuccess) {
        *err = DCT2D_ERR_NOMEM;
        return nullptr;
    }
    // built on the null stream and completed before first use on any stream
    if (tables_dense_q(n, q, nullptr) != DCT2D_OK || hipDeviceSynchronize() != hipSuccess) {
        hipFree(q);
        *err = DCT2D_ERR_HIP;
        return nullptr;
    }
    g_q[{device, n}] = q;
    return q;
}

// Device address of `scratch` on the current device, resolved once per device.
float* scratch_ptr(int* err)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        *err = DCT2D_ERR_NOINIT;
        return nullptr;
    }
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (g_scratch[dev]) return g_scratch[dev];
    }
    const int rc = image_scratch_init(dev);
    if (rc != DCT2D_OK) {
        *err = rc;
        return nullptr;
    }
    std::lock_guard<std::mutex> lk(g_mu);
    return g_scratch[dev];
}

} // namespace

int dct::launch_image(const DeviceTables* t, const Job& j, float* ws, const float* q_rows)
{
    const int64_t n = (int64_t)j.rows * j.cols;
    const Addr in = j.addr();
    const Addr out{j.out, j.out, j.out_stride, j.out_stride, j.out_idx, j.out_idx, j.out_slot, j.out_slot};
    auto line = [&](const Addr& a, bool column_pass) {
        return launch_line_axis(t, a, j.batch, j.rows, j.cols, column_pass, j.dir, true, j.stream);
    };
    if (line_axis(j.rows)) {
        const int rc = line(in, false);
        return rc == DCT2D_OK ? line(out, true) : rc;
    }
    const Addr in_ws{j.in, ws, j.in_stride, n, j.in_idx, nullptr, j.in_slot, nullptr};
    const Addr ws_out{ws, j.out, n, j.out_stride, nullptr, j.out_idx, nullptr, j.out_slot};
    auto dense = [&](const Addr& a, bool inverse) {
        return launch_dense_columns(a, j.batch, j.rows, j.cols, inverse, q_rows, j.stream);
    };
    if (j.dir != DCT2D_ROUNDTRIP) {
        const int rc = line(in_ws, false);
        return rc == DCT2D_OK ? dense(ws_out, j.dir == DCT2D_INVERSE) : rc;
    }
    // round trip: the axes commute (Q_h^T Q_h X Q_w^T Q_w), the rows are one in-place pass
    int rc = dense(in_ws, false);
    if (rc == DCT2D_OK) rc = dense(ws_out, true);
    return rc == DCT2D_OK ? line(out, false) : rc;
}

namespace {

// launch_image on `per` images at a time.
int launch_chunks(const DeviceTables* t, const Job& job, int64_t per, float* ws, const float* q_rows)
{
    int rc = DCT2D_OK;
    for (int64_t b0 = 0; b0 < job.batch && rc == DCT2D_OK; b0 += per) {
        Job j = job;
        j.batch = job.batch - b0 < per ? job.batch - b0 : per;
        j.in = job.in + b0 * job.in_stride;
        j.out = job.out + b0 * job.out_stride;
        rc = launch_image(t, j, ws, q_rows);
    }
    return rc;
}

} // namespace

int dct::image_scratch_init(int device)
{
    if (device < 0 || device >= kMaxDevices) return DCT2D_ERR_NOINIT;
    std::lock_guard<std::mutex> lk(g_mu);
    if (g_scratch[device]) return DCT2D_OK;
    int prev = 0;
    if (hipGetDevice(&prev) != hipSuccess) return DCT2D_ERR_HIP;
    if (prev != device && hipSetDevice(device) != hipSuccess) return DCT2D_ERR_HIP;
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (prev != device) hipSetDevice(prev);
    if (e != hipSuccess || !p) return DCT2D_ERR_HIP;
    g_scratch[device] = static_cast<float*>(p);
    return DCT2D_OK;
}

void dct::image_release_all()
{
    std::lock_guard<std::mutex> lk(g_mu);
    int prev = 0;
    hipGetDevice(&prev);
    for (auto& kv : g_q) {
        hipSetDevice(kv.first.first);
        hipDeviceSynchronize();
        hipFree(kv.second);
    }
    g_q.clear();
    hipSetDevice(prev);
}

extern "C" {

int dct2d_image_transform(int dir, const float* in, float* out, int64_t batch, int32_t rows, int32_t cols,
                          int64_t in_stride, int64_t out_stride, void* stream)
{
    int rc = validate(dir, in, out, batch, rows, cols, in_stride, out_stride);
    if (rc != DCT2D_OK || batch == 0) return rc;
    const DeviceTables* t = tables_current(&rc);
    if (!t) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (fast_shape(rows, cols)) {
        Job j{dir, in, out, batch, rows, cols, in_stride, out_stride, s, 0};
        return dispatch(t, j, DCT2D_AUTO);
    }
    if (long_shape(rows, cols)) {
        Job j{dir, in, out, batch, rows, cols, in_stride, out_stride, s, 0};
        return launch_long(t, j);
    }
    Job j{dir, in, out, batch, rows, cols, in_stride, out_stride, s, 0};
    if (line_axis(rows)) return launch_chunks(t, j, line_chunk(rows, cols), nullptr, nullptr);
    const float* q_rows = cached_q(t->device, rows, &rc);
    if (!q_rows) return rc;
    const int64_t n = (int64_t)rows * cols;
    const int64_t per = batch < 65535 ? batch : 65535; // the dense grid's z extent
    float* ws = nullptr;
    if (hipMallocAsync(reinterpret_cast<void**>(&ws), (size_t)(per * n) * sizeof(float), s) != hipSuccess)
        return DCT2D_ERR_NOMEM;
    rc = launch_chunks(t, j, per, ws, q_rows);
    if (hipFreeAsync(ws, s) != hipSuccess && rc == DCT2D_OK) rc = DCT2D_ERR_HIP;
    return rc;
}

int dct2d_image_transform_noalloc(int dir, const float* in, float* out, int64_t batch, int32_t rows, int32_t cols,
                                  int64_t in_stride, int64_t out_stride, void* stream)
{
    int rc = validate(dir, in, out, batch, rows, cols, in_stride, out_stride);
    if (rc != DCT2D_OK || batch == 0) return rc;
    // the tables of dct2d_init; this entry point never builds them itself
    const DeviceTables* t = tables_ready(&rc);
    if (!t) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (fast_shape(rows, cols)) {
        Job j{dir, in, out, batch, rows, cols, in_stride, out_stride, s, 0};
        return dispatch(t, j, DCT2D_AUTO);
    }
    if (long_shape(rows, cols)) {
        Job j{dir, in, out, batch, rows, cols, in_stride, out_stride, s, 0};
        return launch_long(t, j);
    }
    Job j{dir, in, out, batch, rows, cols, in_stride, out_stride, s, 0};
    if (line_axis(rows)) return launch_chunks(t, j, line_chunk(rows, cols), nullptr, nullptr);
    float* base = scratch_ptr(&rc);
    if (!base) return rc;
    const size_t n = (size_t)rows * cols;
    const size_t ws_off = align256((size_t)rows * rows * sizeof(float));
    if (ws_off + n * sizeof(float) > kScratchBytes) return DCT2D_ERR_SIZE; // not reached for accepted shapes
    const int64_t fit = (int64_t)((kScratchBytes - ws_off) / (n * sizeof(float)));
    const int64_t per = fit < 65535 ? fit : 65535;
    char* b = reinterpret_cast<char*>(base);
    float* q_rows = reinterpret_cast<float*>(b);
    float* ws = reinterpret_cast<float*>(b + ws_off);
    // the table is rebuilt on the caller's stream every call: the scratch keeps whatever the previous
    // call on this device left in it
    rc = tables_dense_q(rows, q_rows, s);
    return rc == DCT2D_OK ? launch_chunks(t, j, per, ws, q_rows) : rc;
}

} // extern "C"
