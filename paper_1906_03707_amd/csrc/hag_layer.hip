// The dense parts of a GNN layer's training step on tall, narrow matrices: products with a weight matrix, the gradient of a weight matrix (a contraction
// over all nodes with a result of a few thousand elements) and the SoftMax cross-entropy over a few classes.
#include "hag_device_common.hpp"

namespace hag {

typedef float layer_f4_t __attribute__((ext_vector_type(4)));

// g_w [d, k] = x^T g for x [n, d], g [n, k].  Bound by reading x and g once.  A wavefront takes every (4 * wavefronts)-th group of four rows and 64 columns of x
// against up to 64 of g, accumulating with v_mfma_f32_16x16x4_f32: its k index is the row, so lane l supplies row l / 16 of both operands straight from
// memory, without LDS: of x four consecutive columns (one 16-byte load; column 4 m + t is row m of product t), of g column 16 j + l % 16.  The
// wavefronts of a workgroup are added up in LDS, the workgroups' parts by weight_grad_reduce_kernel in a fixed order.
// Called from Python, with the BLAS library's time: 65536 nodes, 64 x 16 14 us (that is the call: the kernels take about 8; library 82), 16 x 16 15 (174),
// 256 x 256 144 (217); 370000 nodes, 64 x 16 28 (284), 128 x 64 88 (609), 256 x 256 784 (878).  Error against 64 bits 2e-7 where the library has 2e-6.
constexpr int kWgradWaves = 4, kWgradAsk = 4;

// RELU: x is what a ReLU gets, and g_w = relu(x)^T g.
__device__ __forceinline__ float relu1(float v) { return v <= 0.f ? 0.f : v; }   // (a NaN stays)
__device__ __forceinline__ float4 relu4(float4 v) { return make_float4(relu1(v.x), relu1(v.y), relu1(v.z), relu1(v.w)); }

template <int NB, bool RELU>
__global__ __launch_bounds__(kWgradWaves * kWave) void weight_grad_kernel(const float *__restrict__ x, const float *__restrict__ g, int64_t n, int32_t d, int32_t k,
                                                                          float *__restrict__ partial) {
    __shared__ float part[kWgradWaves - 1][NB * 16][kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, q = lane >> 4, c = lane & 15;
    const int col = blockIdx.y * 64 + 4 * c, out0 = blockIdx.z * NB * 16;
    const bool col_ok = col < d;
    layer_f4_t acc[4][NB];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[t][j] = layer_f4_t{0.f, 0.f, 0.f, 0.f};
    const int64_t groups = (n + 3) / 4, step = (int64_t)gridDim.x * kWgradWaves;
    for (int64_t at = (int64_t)blockIdx.x * kWgradWaves + wave; at < groups; at += step * kWgradAsk) {
        float4 a[kWgradAsk];
        float b[kWgradAsk][NB];
#pragma unroll
        for (int u = 0; u < kWgradAsk; ++u) {
            const int64_t row = 4 * (at + u * step) + q;
            const bool ok = row < n;
            a[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (ok && col_ok) a[u] = ld4(x + (size_t)row * d + col);
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int o = out0 + 16 * j + c;
                b[u][j] = ok && o < k ? g[(size_t)row * k + o] : 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < kWgradAsk; ++u) {
            if (RELU) a[u] = relu4(a[u]);
            const float e[4] = {a[u].x, a[u].y, a[u].z, a[u].w};
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(e[t], b[u][j], acc[t][j], 0, 0, 0);
        }
    }
    if (wave > 0) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) part[wave - 1][(t * NB + j) * 4 + r][lane] = acc[t][j][r];
    }
    __syncthreads();
    if (wave > 0) return;
    float *out = partial + (size_t)blockIdx.x * ((size_t)d * k);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float sum = acc[t][j][r];
#pragma unroll
                for (int w = 0; w < kWgradWaves - 1; ++w) sum += part[w][(t * NB + j) * 4 + r][lane];
                const int row = blockIdx.y * 64 + 4 * (4 * q + r) + t, o = out0 + 16 * j + c;   // the result's lane l: column l % 16, rows 4 (l / 16) + r
                if (row < d && o < k) out[(size_t)row * k + o] = sum;
            }
}

// out[i] = sum over the groups of partial[group][i]: 32 outputs per workgroup, eight threads each, then those, in a fixed order
__global__ __launch_bounds__(kBlock) void weight_grad_reduce_kernel(const float *__restrict__ partial, int32_t groups, int64_t count, float *__restrict__ out) {
    __shared__ float part[8][32];
    const int o = threadIdx.x & 31, p = threadIdx.x >> 5;
    const int64_t i = (int64_t)blockIdx.x * 32 + o;
    float sum = 0.f;
    if (i < count) {
#pragma unroll 4
        for (int g = p; g < groups; g += 8) sum += partial[(size_t)g * count + i];
    }
    part[p][o] = sum;
    __syncthreads();
    if (p != 0 || i >= count) return;
#pragma unroll
    for (int w = 1; w < 8; ++w) sum += part[w][o];
    out[i] = sum;
}

// y [n, k] = x w for x [n, d] and a small w [d, k] (or the transpose of w [k, d]).  Bound by reading x and writing y once; a wavefront takes 32 rows and up to
// 64 columns of y, with v_mfma_f32_16x16x4_f32: lane l loads four consecutive columns 16 s + 4 (l / 16) + 0..3 of row l % 16, the k index of four
// products (any order of k will do, w is laid out in LDS to match, 16 bytes per lane and 16 columns of x).  RELU: relu(x) instead of x; MASK: elements of y
// where `mask` [n, k], what a ReLU got, is not positive are 0 (that ReLU's backward pass).
// 65536 nodes: 64 x 16 8.8 us (BLAS 9.4 and 20 us of host time a call, here 6), 16 x 16 with relu(x) 7.2 (6.1, and 6 for a ReLU of its own), transposed
// with a mask 6.4 (8.7, and 5.6).
constexpr int kProductRows = 32;           // per wavefront

template <int NB, bool RELU, bool MASK>
__global__ __launch_bounds__(kBlock) void product_kernel(const float *__restrict__ x, const float *__restrict__ w, int32_t transposed, int64_t n, int32_t d, int32_t k,
                                                         const float *__restrict__ mask, float *__restrict__ y) {
    extern __shared__ __align__(16) float ws[];            // [steps of 16 columns][NB][64 lanes][4]
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, q = lane >> 4, c = lane & 15;
    const int steps = (d + 15) / 16, out0 = blockIdx.y * NB * 16;
    for (int i = threadIdx.x; i < steps * NB * 256; i += kBlock) {
        const int e = i & 3, l = (i >> 2) & 63, j = (i >> 8) % NB, s = (i >> 8) / NB;
        const int row = 16 * s + 4 * (l >> 4) + e, col = out0 + 16 * j + (l & 15);
        ws[i] = row < d && col < k ? w[transposed ? (size_t)col * d + row : (size_t)row * k + col] : 0.f;
    }
    __syncthreads();
    const int64_t row0 = ((int64_t)blockIdx.x * (kBlock / kWave) + wave) * kProductRows;
    if (row0 >= n) return;
    constexpr int RT = kProductRows / 16;
    layer_f4_t acc[RT][NB];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[t][j] = layer_f4_t{0.f, 0.f, 0.f, 0.f};
    auto request = [&](int s, float4 (&a)[RT]) {
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const int64_t row = row0 + 16 * t + c;
            const int col = 16 * s + 4 * q;
            a[t] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (row < n && col < d) a[t] = ld4(x + (size_t)row * d + col);
        }
    };
    float4 next[RT];
    request(0, next);
    for (int s = 0; s < steps; ++s) {
        float4 a[RT];
#pragma unroll
        for (int t = 0; t < RT; ++t) a[t] = RELU ? relu4(next[t]) : next[t];
        if (s + 1 < steps) request(s + 1, next);
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const float4 b = *reinterpret_cast<const float4 *>(&ws[((s * NB + j) * 64 + lane) * 4]);
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].x, b.x, acc[t][j], 0, 0, 0);
                acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].y, b.y, acc[t][j], 0, 0, 0);
                acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].z, b.z, acc[t][j], 0, 0, 0);
                acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].w, b.w, acc[t][j], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t row = row0 + 16 * t + 4 * q + r;
                const int col = out0 + 16 * j + c;
                if (row >= n || col >= k) continue;
                const size_t at = (size_t)row * k + col;
                y[at] = MASK && mask[at] <= 0.f ? 0.f : acc[t][j][r];
            }
}

// Cross-entropy of softmax(z [n, classes]) with one label per row, mean over the rows whose label is not `ignore`, and its gradient.  A row is read once from
// memory: W lanes per row (16 up to 64 classes, else a wavefront), three passes over its columns (maximum, sum of exponentials, what is asked for), all
// but the first out of the caches; up to 4 columns per lane stay in registers.  A label that is neither a class nor `ignore` makes the loss NaN.
// Loss and gradient, called from Python: 65536 rows, 16 classes 27 us (torch 113), 300 classes 100 (234); 370000 rows, 16 classes 77 (561).
template <int W>
struct SoftRow {
    static constexpr int kHeld = 4;
    float v[kHeld], top, sum;
    __device__ __forceinline__ static float max_all(float a) {
#pragma unroll
        for (int off = 1; off < W; off <<= 1) a = fmaxf(a, __shfl_xor(a, off));
        return a;
    }
    __device__ __forceinline__ static float add_all(float a) {
#pragma unroll
        for (int off = 1; off < W; off <<= 1) a += __shfl_xor(a, off);
        return a;
    }
    __device__ __forceinline__ void read(const float *z, int classes, int l) {
        float m = -INFINITY;
        bool nan = false;
#pragma unroll
        for (int h = 0; h < kHeld; ++h) {
            v[h] = l + W * h < classes ? z[l + W * h] : -INFINITY;
            m = fmaxf(m, v[h]);
            nan |= v[h] != v[h];
        }
        for (int c = l + W * kHeld; c < classes; c += W) { m = fmaxf(m, z[c]); nan |= z[c] != z[c]; }
        top = max_all(nan ? INFINITY : m);                 // (a NaN among the logits: inf - inf below)
        float s = 0.f;
#pragma unroll
        for (int h = 0; h < kHeld; ++h)
            if (l + W * h < classes) s += expf(v[h] - top);
        for (int c = l + W * kHeld; c < classes; c += W) s += expf(z[c] - top);
        sum = add_all(s);
    }
};

template <int W>
__global__ __launch_bounds__(kBlock) void loss_kernel(const float *__restrict__ z, const int64_t *__restrict__ labels, int64_t n, int32_t classes, int64_t ignore,
                                                      double *__restrict__ partial) {
    __shared__ double sums[kBlock / kWave][2];
    const int l = threadIdx.x % W;
    double sum = 0., rows = 0.;
    for (int64_t base = (int64_t)blockIdx.x * (kBlock / W); base < n; base += (int64_t)gridDim.x * (kBlock / W)) {
        const int64_t row = base + threadIdx.x / W;
        const bool here = row < n;
        const float *p = z + (size_t)(here ? row : 0) * classes;
        SoftRow<W> s;
        s.read(p, classes, l);
        const int64_t label = here ? labels[row] : ignore;
        if (l == 0 && label != ignore) {
            const bool valid = label >= 0 && label < classes;
            sum += valid ? logf(s.sum) - (p[valid ? label : 0] - s.top) : NAN;
            rows += 1.;
        }
    }
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) { sum += __shfl_xor(sum, off); rows += __shfl_xor(rows, off); }
    if (threadIdx.x % kWave == 0) { sums[threadIdx.x / kWave][0] = sum; sums[threadIdx.x / kWave][1] = rows; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / kWave; ++w) { sum += sums[w][0]; rows += sums[w][1]; }
        partial[2 * blockIdx.x] = sum;
        partial[2 * blockIdx.x + 1] = rows;
    }
}

// mean, and the number of rows that count
__global__ __launch_bounds__(kBlock) void loss_reduce_kernel(const double *__restrict__ partial, int32_t groups, float *__restrict__ loss,
                                                         float *__restrict__ counted) {
    __shared__ double sums[kBlock / kWave][2];
    double sum = 0., rows = 0.;
    for (int g = threadIdx.x; g < groups; g += kBlock) { sum += partial[2 * g]; rows += partial[2 * g + 1]; }
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) { sum += __shfl_xor(sum, off); rows += __shfl_xor(rows, off); }
    if (threadIdx.x % kWave == 0) { sums[threadIdx.x / kWave][0] = sum; sums[threadIdx.x / kWave][1] = rows; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / kWave; ++w) { sum += sums[w][0]; rows += sums[w][1]; }
        *loss = (float)(sum / rows);                       // (no row that counts: 0 / 0)
        *counted = (float)rows;
    }
}

// g_z = g_loss * (softmax(z) - onehot) / rows, 0 in the rows whose label is `ignore`
template <int W>
__global__ __launch_bounds__(kBlock) void loss_grad_kernel(const float *__restrict__ z, const int64_t *__restrict__ labels, int64_t n, int32_t classes, int64_t ignore,
                                                           const float *__restrict__ counted, const float *__restrict__ g_loss, float *__restrict__ g_z) {
    const int l = threadIdx.x % W;
    const float scale = *g_loss / *counted;
    const int64_t row = (int64_t)blockIdx.x * (kBlock / W) + threadIdx.x / W;
    const bool here = row < n;
    const float *p = z + (size_t)(here ? row : 0) * classes;
    SoftRow<W> s;
    s.read(p, classes, l);
    if (!here) return;
    const int64_t label = labels[row];
    const float inv = 1.f / s.sum;
    float *out = g_z + (size_t)row * classes;
#pragma unroll
    for (int h = 0; h < SoftRow<W>::kHeld; ++h) {
        const int c = l + W * h;
        if (c < classes) out[c] = label == ignore ? 0.f : scale * (expf(s.v[h] - s.top) * inv - (c == label ? 1.f : 0.f));
    }
    for (int c = l + W * SoftRow<W>::kHeld; c < classes; c += W) out[c] = label == ignore ? 0.f : scale * (expf(p[c] - s.top) * inv - (c == label ? 1.f : 0.f));
}

constexpr int64_t kLossGroups = 512;

// workgroups along the rows: enough to fill the device, no more partial results than 16 M floats, at least eight groups of four rows per wavefront
static int64_t wgrad_groups(int64_t n, int64_t d, int64_t k) {
    const int64_t tiles = ((d + 63) / 64) * ((k + 63) / 64);
    const int64_t want = std::max<int64_t>(512 / tiles, 64), rows = (n + 4 * kWgradWaves * 8 - 1) / (4 * kWgradWaves * 8);
    return std::max<int64_t>(std::min({want, rows, ((int64_t)16 << 20) / (d * k)}), 1);
}

}  // namespace hag

using namespace hag;

extern "C" {

static bool wgrad_supported(int64_t n, int64_t d, int64_t k) { return n >= 0 && d > 0 && d % 4 == 0 && k > 0 && d <= 4096 && k <= 4096; }

size_t hag_weight_grad_workspace_bytes(int64_t n, int64_t d, int64_t k) {
    return wgrad_supported(n, d, k) ? (size_t)(wgrad_groups(n, d, k) * d * k) * sizeof(float) : 0;
}

int hag_weight_grad(int64_t n, int64_t d, int64_t k, const float *x, int32_t relu, const float *g, float *g_w, void *workspace, void *stream) {
    if (!wgrad_supported(n, d, k)) { set_error("d must be a multiple of 4, d and k at most 4096"); return HAG_EINVAL; }
    if (!g_w || !workspace || (n > 0 && (!x || !g))) { set_error("NULL pointer"); return HAG_EINVAL; }
    if ((uintptr_t)x & 15) { set_error("x must be 16-byte aligned"); return HAG_EINVAL; }
    hipStream_t s = (hipStream_t)stream;
    float *partial = (float *)workspace;
    const int64_t groups = wgrad_groups(n, d, k);
    const int nb = k <= 16 ? 1 : k <= 32 ? 2 : 4;
    const dim3 grid((unsigned)groups, (unsigned)((d + 63) / 64), (unsigned)((k + 16 * nb - 1) / (16 * nb))), block(kWgradWaves * kWave);
    typedef void (*kernel_t)(const float *, const float *, int64_t, int32_t, int32_t, float *);
    static const kernel_t kernels[3][2] = {{weight_grad_kernel<1, false>, weight_grad_kernel<1, true>}, {weight_grad_kernel<2, false>, weight_grad_kernel<2, true>},
                                           {weight_grad_kernel<4, false>, weight_grad_kernel<4, true>}};
    hipLaunchKernelGGL(kernels[nb / 2][relu != 0], grid, block, 0, s, x, g, n, (int32_t)d, (int32_t)k, partial);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(weight_grad_reduce_kernel, dim3((unsigned)((d * k + 31) / 32)), dim3(kBlock), 0, s, partial, (int32_t)groups, d * k, g_w);
    HIP_TRY(hipGetLastError());
    return HAG_OK;
}

int hag_narrow_product(int64_t n, int64_t d, int64_t k, const float *x, int32_t relu, const float *w, int32_t transposed, const float *mask, float *y, void *stream) {
    const int nb = k <= 16 ? 1 : k <= 32 ? 2 : 4;
    const int64_t lds = (d + 15) / 16 * nb * 1024;
    if (n < 0 || d <= 0 || d % 4 != 0 || k <= 0 || k > 4096 || lds > 64 * 1024) {
        set_error("d must be a multiple of 4 (at most 1024 for k <= 16, 512 for k <= 32, 256 beyond), k at most 4096");
        return HAG_EINVAL;
    }
    if (n == 0) return HAG_OK;
    if (!x || !w || !y) { set_error("NULL pointer"); return HAG_EINVAL; }
    if ((uintptr_t)x & 15) { set_error("x must be 16-byte aligned"); return HAG_EINVAL; }
    const int64_t per = kProductRows * (kBlock / kWave), groups = (n + per - 1) / per;
    if (groups > 0x7fffffffLL) { set_error("launch too large"); return HAG_EINVAL; }
    const dim3 grid((unsigned)groups, (unsigned)((k + 16 * nb - 1) / (16 * nb)));
    typedef void (*kernel_t)(const float *, const float *, int32_t, int64_t, int32_t, int32_t, const float *, float *);
    static const kernel_t kernels[3][2][2] = {{{product_kernel<1, false, false>, product_kernel<1, false, true>}, {product_kernel<1, true, false>, product_kernel<1, true, true>}},
                                              {{product_kernel<2, false, false>, product_kernel<2, false, true>}, {product_kernel<2, true, false>, product_kernel<2, true, true>}},
                                              {{product_kernel<4, false, false>, product_kernel<4, false, true>}, {product_kernel<4, true, false>, product_kernel<4, true, true>}}};
    hipLaunchKernelGGL(kernels[nb / 2][relu != 0][mask != nullptr], grid, dim3(kBlock), (size_t)lds, (hipStream_t)stream, x, w, transposed, n, (int32_t)d, (int32_t)k, mask, y);
    HIP_TRY(hipGetLastError());
    return HAG_OK;
}

size_t hag_softmax_loss_workspace_bytes(void) { return (size_t)kLossGroups * 2 * sizeof(double); }

int hag_softmax_loss(int64_t n, int64_t classes, const float *z, const int64_t *labels, int64_t ignore, float *loss, float *counted,
                     void *workspace, void *stream) {
    if (n < 0 || classes <= 0 || classes > (1 << 20)) { set_error("n < 0 or classes not in 1 .. 2^20"); return HAG_EINVAL; }
    if (!loss || !counted || !workspace || (n > 0 && (!z || !labels))) { set_error("NULL pointer"); return HAG_EINVAL; }
    if ((uintptr_t)workspace & 15) { set_error("workspace must be 16-byte aligned"); return HAG_EINVAL; }
    hipStream_t s = (hipStream_t)stream;
    const int64_t per = kBlock / (classes <= 64 ? 16 : 64), groups = std::max<int64_t>(std::min<int64_t>((n + per - 1) / per, kLossGroups), 1);
    if (classes <= 64)
        hipLaunchKernelGGL(loss_kernel<16>, dim3((unsigned)groups), dim3(kBlock), 0, s, z, labels, n, (int32_t)classes, ignore, (double *)workspace);
    else
        hipLaunchKernelGGL(loss_kernel<64>, dim3((unsigned)groups), dim3(kBlock), 0, s, z, labels, n, (int32_t)classes, ignore, (double *)workspace);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(kBlock), 0, s, (const double *)workspace, (int32_t)groups, loss, counted);
    HIP_TRY(hipGetLastError());
    return HAG_OK;
}

int hag_softmax_loss_grad(int64_t n, int64_t classes, const float *z, const int64_t *labels, int64_t ignore, const float *counted, const float *g_loss,
                          float *g_z, void *stream) {
    if (n < 0 || classes <= 0 || classes > (1 << 20)) { set_error("n < 0 or classes not in 1 .. 2^20"); return HAG_EINVAL; }
    if (n == 0) return HAG_OK;
    if (!z || !labels || !counted || !g_loss || !g_z) { set_error("NULL pointer"); return HAG_EINVAL; }
    hipStream_t s = (hipStream_t)stream;
    const int64_t per = kBlock / (classes <= 64 ? 16 : 64), groups = (n + per - 1) / per;
    if (groups > 0x7fffffffLL) { set_error("launch too large"); return HAG_EINVAL; }
    if (classes <= 64)
        hipLaunchKernelGGL(loss_grad_kernel<16>, dim3((unsigned)groups), dim3(kBlock), 0, s, z, labels, n, (int32_t)classes, ignore, counted, g_loss, g_z);
    else
        hipLaunchKernelGGL(loss_grad_kernel<64>, dim3((unsigned)groups), dim3(kBlock), 0, s, z, labels, n, (int32_t)classes, ignore, counted, g_loss, g_z);
    HIP_TRY(hipGetLastError());
    return HAG_OK;
}

}  // extern "C"
