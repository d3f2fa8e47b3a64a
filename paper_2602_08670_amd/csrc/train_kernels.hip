// Training helpers: the unrolled loss of eq 2.28 with its gradient, and Adam.
#include "cnn_internal.hpp"

namespace cnn {

__global__ __launch_bounds__(256) void loss_kernel(const float *pred, const float *tgt, const float *scale3, int B,
                                                   int plane, float *G, double *partials, int nvar)
{
    __shared__ double s[256];
    const size_t n = (size_t)B * nvar * plane;
    const double inv_n = 1.0 / (double)n;
    double acc = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        int v = (int)((i / plane) % nvar);
        float sv = scale3[v];
        float d = pred[i] - tgt[i];
        double r = (double)d / sv;
        acc += r * r * inv_n;
        G[i] += (float)(2.0 * (double)d / ((double)sv * sv) * inv_n);
    }
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partials[blockIdx.x] = s[0];
}

// loss_acc += sum of the block partials: thread i adds partials i, i + 256,
// ... in order, then a fixed tree over the 256 thread sums.
__global__ __launch_bounds__(256) void loss_final_kernel(const double *partials, int nblocks, double *loss_acc)
{
    __shared__ double s[256];
    double t = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += 256) t += partials[b];
    s[threadIdx.x] = t;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss_acc += s[0];
}

hipError_t launch_loss(const float *pred, const float *tgt, const float *scale3, int B, int nx, int ny, float *G,
                       double *partials, int max_blocks, double *loss_acc, hipStream_t st, int nvar)
{
    size_t n = (size_t)B * nvar * nx * ny;
    int blocks = (int)((n + 255) / 256);
    if (blocks > max_blocks) blocks = max_blocks;
    hipLaunchKernelGGL(loss_kernel, dim3(blocks), dim3(256), 0, st, pred, tgt, scale3, B, nx * ny, G, partials, nvar);
    hipLaunchKernelGGL(loss_final_kernel, dim3(1), dim3(256), 0, st, (const double *)partials, blocks, loss_acc);
    return hipGetLastError();
}

__global__ void scale_kernel(float *out, const float *in, float a, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        out[i] = a * in[i];
}

hipError_t launch_scale(float *out, const float *in, float a, size_t n, hipStream_t st)
{
    unsigned blocks = (unsigned)((n + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(scale_kernel, dim3(blocks), dim3(256), 0, st, out, in, a, n);
    return hipGetLastError();
}

// Adam (Kingma & Ba): m = b1 m + (1-b1) g; v = b2 v + (1-b2) g^2;
// p -= lr * (m / bc1) / (sqrt(v / bc2) + eps), bc_k = 1 - b_k^t.
__global__ void adam_kernel(float *p, const float *g, float *m, float *v, size_t n, float lr, float b1, float b2,
                            float eps, float bc1, float bc2)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        float gi = g[i];
        float mi = b1 * m[i] + (1.0f - b1) * gi;
        float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= lr * (mi / bc1) / (__builtin_sqrtf(vi / bc2) + eps);
    }
}

hipError_t launch_adam(float *p, const float *g, float *m, float *v, size_t n, float lr, float b1, float b2,
                       float eps, float bc1, float bc2, hipStream_t st)
{
    unsigned blocks = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(adam_kernel, dim3(blocks), dim3(256), 0, st, p, g, m, v, n, lr, b1, b2, eps, bc1, bc2);
    return hipGetLastError();
}

__global__ void flags_or_kernel(const int *flags, int B, int *any)
{
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B && flags[b]) atomicOr(any, 1);
}

hipError_t launch_flags_or(const int *flags, int B, int *any, hipStream_t st)
{
    hipLaunchKernelGGL(flags_or_kernel, dim3((B + 255) / 256), dim3(256), 0, st, flags, B, any);
    return hipGetLastError();
}

}  // namespace cnn

namespace cnn {

// Exact cell-average coarsening: coarse(I, J) = mean of the f x f fine block,
// accumulated in double precision in a fixed order.  Bound by reading the
// fine array once.  Below CO_BLOCK a thread sums a coarse cell's block by
// itself: a wave's lines are used whole within a few of its loads (3 x 2048^2
// at f = 2: 15 us, 41 as below; f = 4: 15 and 22; 3 x 2100^2 at f = 7: 16 and
// 18; 3 x 2048^2 at f = 8: 24 and 11).
constexpr int CO_BLOCK = 8;
__global__ void coarsen_cell_kernel(const float *__restrict__ fine, int nvar, int nx, int ny, int f,
                                    float *__restrict__ coarse)
{
    const int cx = nx / f, cy = ny / f;
    const size_t n = (size_t)nvar * cx * cy;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const size_t v = i / ((size_t)cx * cy);
        const int r = (int)(i - v * cx * cy), J = r / cx, I = r - J * cx;
        const float *src = fine + v * nx * ny + (size_t)J * f * nx + (size_t)I * f;
        double acc = 0.0;
        for (int a = 0; a < f; a++)
            for (int b = 0; b < f; b++) acc += (double)src[(size_t)a * nx + b];
        coarse[i] = (float)(acc / ((double)f * f));
    }
}
// From there on a workgroup takes
// 256 / f coarse cells of a row (one where f > 256): thread t sums column t of
// their fine cells down the f rows, so that a wave reads whole lines and has
// its rows' loads in flight together, then one thread per coarse cell adds its
// f column sums.  (One thread per coarse cell read f x f values in a strided
// serial chain: 157 us for 3 x 2048^2 at f = 32; now 14 us, 3.6 TB/s.)
constexpr int CO_TH = 256;
__global__ __launch_bounds__(CO_TH) void coarsen_kernel(const float *__restrict__ fine, int nvar, int nx, int ny, int f,
                                                        float *__restrict__ coarse)
{
    __shared__ double s[CO_TH];
    const int cx = nx / f, cy = ny / f;
    const int cb = f <= CO_TH ? CO_TH / f : 1, nb = (cx + cb - 1) / cb;
    const long total = (long)nvar * cy * nb;
    for (long w = blockIdx.x; w < total; w += gridDim.x) {
        const long row = w / nb;  // v * cy + J
        const int I0 = (int)(w - row * nb) * cb, nc = min(cb, cx - I0);
        const int J = (int)(row % cy);
        const float *src = fine + ((size_t)(row / cy) * ny + (size_t)J * f) * nx + (size_t)I0 * f;
        double acc = 0.0;
        for (int c = threadIdx.x; c < nc * f; c += CO_TH) {
            const float *p = src + c;
#pragma unroll 8
            for (int a = 0; a < f; a++) acc += (double)p[(size_t)a * nx];
        }
        s[threadIdx.x] = acc;
        __syncthreads();
        if ((int)threadIdx.x < nc) {
            const int n = f <= CO_TH ? f : CO_TH;
            double sum = 0.0;
            for (int b = 0; b < n; b++) sum += s[threadIdx.x * n + b];
            coarse[row * cx + I0 + threadIdx.x] = (float)(sum / ((double)f * f));
        }
        __syncthreads();
    }
}

hipError_t launch_coarsen(const float *fine, int nvar, int nx, int ny, int f, float *coarse, hipStream_t st)
{
    if (f < CO_BLOCK) {
        const size_t blocks = ((size_t)nvar * (nx / f) * (ny / f) + 255) / 256;
        hipLaunchKernelGGL(coarsen_cell_kernel, dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256), 0, st, fine,
                           nvar, nx, ny, f, coarse);
        return hipGetLastError();
    }
    const int cb = f <= CO_TH ? CO_TH / f : 1;
    const long total = (long)nvar * (ny / f) * ((nx / f + cb - 1) / cb);
    hipLaunchKernelGGL(coarsen_kernel, dim3((unsigned)(total < 1 << 20 ? total : 1 << 20)), dim3(CO_TH), 0, st, fine,
                       nvar, nx, ny, f, coarse);
    return hipGetLastError();
}

}  // namespace cnn
