// Small kernels around the path kernels: light-selection table, loss and
// adjoint image, block-partial gradient reduction, projected Adam.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ipt_internal.h"

namespace ipt {

__global__ void zero_u32_kernel(unsigned* p, int n) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

hipError_t launch_zero_u32(unsigned* p, int n, hipStream_t st) {
    hipLaunchKernelGGL(zero_u32_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Light-selection table.  The paper keeps light-sampling probabilities
// proportional to the current emission of each object in a Fenwick tree
// (Appendix E).  Here every call rebuilds the inclusive prefix sums of
// weight_j = area_j * max(lum(e_k), 1e-3 * max lum) over emitter triangles
// (area only if every emission is zero).
// ---------------------------------------------------------------------------
// Weight of light j: one rounding per operation, so that a sum of weights adds the
// rounded products wherever the compiler places them.
struct LightWeight {
    const int4* lights;
    const float* e;       // emissions
    float maxl;
    __device__ float operator()(int64_t j) const {
#pragma clang fp contract(off)
        const int4 L = lights[j];
        const float area = __int_as_float(L.z);
        if (!(maxl > 0.0f)) return area;
        const float* x = e + 3 * L.y;
        const float l = (x[0] + x[1] + x[2]) * (1.0f / 3.0f);
        return area * fmaxf(l, 1e-3f * maxl);
    }
};

// The table by one block: each of the 1024 threads scans a contiguous run, the run
// totals are scanned in LDS, and the runs are rescanned with their offsets.
__global__ __launch_bounds__(1024) void light_cdf_kernel(const int4* lights, int nlt, int S, int E, int nm,
                                                         const float* sp, float* cdf) {
    __shared__ float part[1024];
    __shared__ float maxl_sh;
    const int tid = threadIdx.x;
    if (tid == 0) {
        float m = 0.0f;
        for (int k = 0; k < E; ++k) {
            const float* e = sp + nm * S + 3 * k;
            m = fmaxf(m, (e[0] + e[1] + e[2]) * (1.0f / 3.0f));
        }
        maxl_sh = m;
    }
    __syncthreads();
    const float maxl = maxl_sh;
    const int per = (nlt + 1023) / 1024;
    const int b = tid * per, e_ = min(nlt, b + per);
    const LightWeight weight{lights, sp + nm * S, maxl};
    float s = 0.0f;
    for (int j = b; j < e_; ++j) s += weight(j);
    part[tid] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        float v = tid >= off ? part[tid - off] : 0.0f;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    float run = tid > 0 ? part[tid - 1] : 0.0f;
    for (int j = b; j < e_; ++j) {
        run += weight(j);
        cdf[j] = run;
    }
    // selection probabilities directly as w_j / total: a difference of two
    // prefix sums would lose digits when there are many lights
    const float rtot = 1.0f / part[1023];
    for (int j = b; j < e_; ++j) cdf[nlt + j] = weight(j) * rtot;
}

// The same table for many lights (more than kManyLights) by three kernels (500,582
// lights: 3455 -> 26 us; one block waits for its strided loads): a block per run computes the
// run's weights with all its threads and adds them with one, in the same order;
// one block scans the run totals; the blocks write their runs.  The same weights
// (LightWeight), summed in the same order as above: the same table bit for bit.
constexpr int kRuns = 1024;       // runs of the table
constexpr int kRunTile = 2048;    // lights of a run held in LDS at a time

// Largest emission luminance, over the block.
__device__ float block_max_lum(const float* e, int E) {
    __shared__ float red[256];
    float m = 0.0f;
    for (int k = threadIdx.x; k < E; k += 256) m = fmaxf(m, (e[3 * k] + e[3 * k + 1] + e[3 * k + 2]) * (1.0f / 3.0f));
    red[threadIdx.x] = m;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + off]);
        __syncthreads();
    }
    return red[0];
}

// WRITE = 0: sums[run] = total of the run; 1: the run's part of the table, sums
// being scanned.
template <int WRITE>
__global__ __launch_bounds__(256) void light_run_kernel(const int4* lights, int nlt, int E, const float* e, float* sums,
                                                        float* cdf) {
    __shared__ float w[kRunTile];
    const int tid = threadIdx.x;
    const LightWeight weight{lights, e, block_max_lum(e, E)};
    const int64_t per = (nlt + kRuns - 1) / kRuns;
    const int64_t b = blockIdx.x * per, end = min((int64_t)nlt, b + per);
    float run = WRITE && blockIdx.x > 0 ? sums[blockIdx.x - 1] : 0.0f;
    const float rtot = WRITE ? 1.0f / sums[kRuns - 1] : 0.0f;
    for (int64_t t = b; t < end; t += kRunTile) {
        const int m = (int)min((int64_t)kRunTile, end - t);
        for (int i = tid; i < m; i += 256) {
            const float x = weight(t + i);
            w[i] = x;
            if (WRITE) cdf[nlt + t + i] = x * rtot;
        }
        __syncthreads();
        if (tid == 0) {
#pragma unroll 8
            for (int i = 0; i < m; ++i) {
                run += w[i];
                if (WRITE) w[i] = run;
            }
        }
        __syncthreads();
        if (WRITE) {
            for (int i = tid; i < m; i += 256) cdf[t + i] = w[i];
            __syncthreads();
        }
    }
    if (!WRITE && tid == 0) sums[blockIdx.x] = run;
}

__global__ __launch_bounds__(kRuns) void light_scan_kernel(float* sums) {
    __shared__ float part[kRuns];
    const int tid = threadIdx.x;
    part[tid] = sums[tid];
    __syncthreads();
    for (int off = 1; off < kRuns; off <<= 1) {
        const float v = tid >= off ? part[tid - off] : 0.0f;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    sums[tid] = part[tid];
}

hipError_t launch_light_cdf(const SceneDev& sc, const float* sparams, float* cdf, float* sums, hipStream_t st) {
    if (sc.nlt <= 0) return hipSuccess;
    if (sc.nlt > kManyLights) {
        const float* e = sparams + sc.nm * sc.S;
        hipLaunchKernelGGL(light_run_kernel<0>, dim3(kRuns), dim3(256), 0, st, sc.lights, sc.nlt, sc.E, e, sums, cdf);
        hipLaunchKernelGGL(light_scan_kernel, dim3(1), dim3(kRuns), 0, st, sums);
        hipLaunchKernelGGL(light_run_kernel<1>, dim3(kRuns), dim3(256), 0, st, sc.lights, sc.nlt, sc.E, e, sums, cdf);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(light_cdf_kernel, dim3(1), dim3(1024), 0, st, sc.lights, sc.nlt, sc.S, sc.E, sc.nm,
                       sparams, cdf);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Loss and adjoint (Sec. 3.2 Eq. 3, Sec. 3.3 Eq. 4).  kind 0: E = mean (I-T)^2,
// w = 2 (I - T) / n; kind 1: E = mean |I - T|, w = sgn(I - T) / n.  (Eq. 4 as
// printed carries sgn(T - I), the descent direction; w here is dE/dI.)
// Block partial sums, then a one-block final sum: deterministic.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void loss_kernel(const float* img, const float* tgt, int64_t n3, int kind,
                                                   float* w, float* partials) {
    __shared__ float red[256];
    float acc = 0.0f;
    const float inv = 1.0f / (float)n3;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n3; i += (int64_t)gridDim.x * 256) {
        float r = img[i] - tgt[i];
        if (kind == 0) {
            acc += r * r;
            w[i] = 2.0f * r * inv;
        } else {
            acc += fabsf(r);
            w[i] = (r > 0.0f ? 1.0f : (r < 0.0f ? -1.0f : 0.0f)) * inv;
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) partials[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void loss_final_kernel(const float* partials, int n, int64_t n3, float* loss) {
    __shared__ double red[256];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) acc += (double)partials[i];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = (float)(red[0] / (double)n3);
}

hipError_t launch_loss_adjoint(const float* img, const float* target, int64_t n3, int kind, float* w,
                               float* partials, int nparts, float* loss, hipStream_t st) {
    nparts = (int)std::max<int64_t>(1, std::min<int64_t>(nparts, (n3 + 255) / 256));   // further sums are 0
    hipLaunchKernelGGL(loss_kernel, dim3(nparts), dim3(256), 0, st, img, target, n3, kind, w, partials);
    hipLaunchKernelGGL(loss_final_kernel, dim3(1), dim3(256), 0, st, partials, nparts, n3, loss);
    return hipGetLastError();
}

// Pixel means from the per-unit sample sums of a colour pass whose pixels were
// split over several lanes (fixed summation order: deterministic).
__global__ __launch_bounds__(256) void colour_reduce_kernel(const float* part, int nchunk, int64_t pix_count,
                                                            float inv_spp, float* image) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= 3 * pix_count) return;
    float s = 0.0f;
    for (int c = 0; c < nchunk; ++c) s += part[(size_t)c * 3 * pix_count + i];
    image[i] = s * inv_spp;
}

// The same for many units per pixel: a block stages kTileUnits units of 32 values
// in LDS with all its threads, and one thread per value adds them in order.
constexpr int kTileUnits = 128;
__global__ __launch_bounds__(256) void colour_reduce_tiled_kernel(const float* part, int nchunk, int64_t n, float inv_spp,
                                                                  float* image) {
    __shared__ float x[kTileUnits][33];
    const int tid = threadIdx.x, col = tid & 31;
    const int64_t i = (int64_t)blockIdx.x * 32 + col;
    float s = 0.0f;
    for (int c = 0; c < nchunk; c += kTileUnits) {
        const int m = min(kTileUnits, nchunk - c);
        if (i < n)
            for (int r = tid >> 5; r < m; r += 8) x[r][col] = part[(size_t)(c + r) * n + i];
        __syncthreads();
        if (tid < 32) {
#pragma unroll 8
            for (int r = 0; r < m; ++r) s += x[r][col];
        }
        __syncthreads();
    }
    if (tid < 32 && i < n) image[i] = s * inv_spp;
}

hipError_t launch_colour_reduce(const float* part, int nchunk, int64_t pix_count, int spp, float* image,
                                hipStream_t st) {
    int64_t n = 3 * pix_count;
    // long sums of few values wait for one load after the other (8 pixels x 512
    // units: 82 us, tiled 20 us); short ones are bandwidth
    if (nchunk >= kTileUnits) {
        hipLaunchKernelGGL(colour_reduce_tiled_kernel, dim3((unsigned)((n + 31) / 32)), dim3(256), 0, st, part, nchunk, n,
                           1.0f / (float)spp, image);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(colour_reduce_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, part, nchunk,
                       pix_count, 1.0f / (float)spp, image);
    return hipGetLastError();
}

constexpr int kFlatParams = 1 << 14;

// grad[i] (+)= sum_b part[b][i] in a fixed order (deterministic): 8 parameters
// per block, each summed by 32 threads over every 32nd row and a tree.  One
// thread per parameter waited for a load per row: 196 us for 1024 rows, now
// 5 us.
__global__ __launch_bounds__(256) void grad_reduce_kernel(const double* part, int nblocks, int P, float* grad,
                                                          int accumulate) {
    __shared__ double red[32][9];
    const int col = threadIdx.x & 7, row = threadIdx.x >> 3;
    const int i = blockIdx.x * 8 + col;
    double s = 0.0;
    if (i < P) {
#pragma unroll 8
        for (int b = row; b < nblocks; b += 32) s += part[(size_t)b * P + i];
    }
    red[row][col] = s;
    __syncthreads();
    for (int off = 16; off > 0; off >>= 1) {
        if (row < off) red[row][col] += red[row + off][col];
        __syncthreads();
    }
    if (row == 0 && i < P) grad[i] = accumulate ? (float)((double)grad[i] + red[0][col]) : (float)red[0][col];
}

// The same for many parameters, a thread each: the reads of a row are contiguous and
// there are threads enough to wait for them.
__global__ __launch_bounds__(256) void grad_reduce_flat_kernel(const double* part, int nblocks, int P, float* grad,
                                                               int accumulate) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= P) return;
    double s = 0.0;
#pragma unroll 8
    for (int b = 0; b < nblocks; ++b) s += part[(size_t)b * P + i];
    grad[i] = accumulate ? (float)((double)grad[i] + s) : (float)s;
}

hipError_t launch_grad_reduce(const double* part, int nblocks, int P, float* grad, int accumulate,
                              hipStream_t st) {
    // gradient of 8 pixels by rows of 32 threads / by one thread per parameter: 90 / 117 us
    // with 4203 parameters, 123 / 132 with 11903, 148 / 134 with 16383, 235 / 170 with
    // 350 thousand, 1063 / 208 with 14 million (two rows, which leave most of 32 threads idle)
    if (P >= kFlatParams) {
        hipLaunchKernelGGL(grad_reduce_flat_kernel, dim3((P + 255) / 256), dim3(256), 0, st, part, nblocks, P, grad,
                           accumulate);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(grad_reduce_kernel, dim3((P + 7) / 8), dim3(256), 0, st, part, nblocks, P, grad, accumulate);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Adam (Kingma & Ba; Sec. 4.5) on theta = p / scale, bias-corrected, then a
// clamp of theta to [lo, hi] (the material parameters live in [0, 1]).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void adam_kernel(float* params, const float* grad, float* m, float* v, int P,
                                                   float c1, float c2, float lr, float b1, float b2, float eps,
                                                   const float* scale, const float* lo, const float* hi,
                                                   const uint8_t* trainable) {
    int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= P) return;
    if (trainable && !trainable[i]) return;
    float sc = scale ? scale[i] : 1.0f;
    float g = grad[i] * sc;
    float mi = b1 * m[i] + (1.0f - b1) * g;
    float vi = b2 * v[i] + (1.0f - b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    float mh = mi / c1, vh = vi / c2;
    float th = params[i] / sc - lr * mh / (sqrtf(vh) + eps);
    if (lo) th = fmaxf(th, lo[i]);
    if (hi) th = fminf(th, hi[i]);
    params[i] = th * sc;
}

// L1 term: grad += w sgn(p); loss += sum w |p| (one wave-reduced atomic per wave).
__global__ __launch_bounds__(256) void l1_reg_kernel(const float* p, float* g, const float* w, int P, float* loss) {
    int i = blockIdx.x * 256 + threadIdx.x;
    float l = 0.0f;
    if (i < P && w[i] != 0.0f) {
        float x = p[i];
        float sg = x > 0.0f ? 1.0f : (x < 0.0f ? -1.0f : 0.0f);
        g[i] += w[i] * sg;
        l = w[i] * fabsf(x);
    }
    for (int o = 32; o >= 1; o >>= 1) l += __shfl_xor(l, o, 64);
    if ((threadIdx.x & 63) == 0 && l != 0.0f) atomicAdd(loss, l);
}

hipError_t launch_l1_reg(const float* p, float* g, const float* w, int P, float* loss, hipStream_t st) {
    hipLaunchKernelGGL(l1_reg_kernel, dim3((P + 255) / 256), dim3(256), 0, st, p, g, w, P, loss);
    return hipGetLastError();
}

hipError_t launch_adam(float* params, const float* grad, float* m, float* v, int P, int step, float lr,
                       float b1, float b2, float eps, const float* scale, const float* lo, const float* hi,
                       const uint8_t* trainable, hipStream_t st) {
    float c1 = (float)(1.0 - pow((double)b1, (double)step));
    float c2 = (float)(1.0 - pow((double)b2, (double)step));
    hipLaunchKernelGGL(adam_kernel, dim3((P + 255) / 256), dim3(256), 0, st, params, grad, m, v, P, c1, c2, lr,
                       b1, b2, eps, scale, lo, hi, trainable);
    return hipGetLastError();
}

}  // namespace ipt
