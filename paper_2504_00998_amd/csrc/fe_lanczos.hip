// The vector work of a Lanczos step with full reorthogonalisation (spectrum
// bounds of the filter, paper Sec. 2.3): w -= V (V^T w) twice and the next
// vector, on the device without a host read in between.
//
// Bound by reading V (n x (j+1), 8 B a value, from the last-level cache or HBM)
// four times a step.  The coefficients V^T w are fixed-order two-pass sums: each
// workgroup leaves its partial sums, and every workgroup of the next launch adds
// them up itself.  With a library call for each product and norm and a host read
// of each scalar a step of p = 4, 24x24x48 cells took 173 us beside the product,
// here 98 (ten steps with their products 1.96 -> 1.21 ms).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fe_internal.h"

namespace fe {

namespace {

constexpr int kThreads = 512, kWaves = kThreads / 64;
constexpr int kCols = 8;  // columns of V in flight at once

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) v += __shfl_xor(v, w);
    return v;
}

// part[c nb + blk] = sum over the workgroup's elements of V_c w, c < nc
__global__ __launch_bounds__(kThreads) void lanczos_dots_kernel(const double *__restrict__ V,
                                                                const double *__restrict__ w, int64_t n, int nc,
                                                                double *part) {
    __shared__ double lds[kWaves][kCols];
    const int lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    for (int c0 = 0; c0 < nc; c0 += kCols) {
        double acc[kCols];
#pragma unroll
        for (int c = 0; c < kCols; ++c) acc[c] = 0.0;
        for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
            const double wi = w[i];
#pragma unroll
            for (int c = 0; c < kCols; ++c)  // (past the last column: that one again)
                acc[c] += V[(int64_t)min(c0 + c, nc - 1) * n + i] * wi;
        }
#pragma unroll
        for (int c = 0; c < kCols; ++c) {
            const double s = wave_sum(acc[c]);
            if (lane == 0) lds[wave][c] = s;
        }
        __syncthreads();
        if ((int)threadIdx.x < kCols && c0 + (int)threadIdx.x < nc) {
            double s = lds[0][threadIdx.x];
            for (int k = 1; k < kWaves; ++k) s += lds[k][threadIdx.x];
            part[(int64_t)(c0 + threadIdx.x) * gridDim.x + blockIdx.x] = s;
        }
        __syncthreads();
    }
}

// h = the sums of part; w -= V h, and norm[blk] = the workgroup's share of w.w.
// alpha (may be null) = h of the last column.
__global__ __launch_bounds__(kThreads) void lanczos_project_kernel(const double *__restrict__ V,
                                                                   double *__restrict__ w, int64_t n, int nc,
                                                                   const double *__restrict__ part, double *norm,
                                                                   double *alpha) {
    __shared__ double h[kLanczosMost + kCols], lds[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    for (int c = wave; c < nc; c += kWaves) {
        double s = 0.0;
        for (int b = lane; b < (int)gridDim.x; b += 64) s += part[(int64_t)c * gridDim.x + b];
        s = wave_sum(s);
        if (lane == 0) h[c] = s;
    }
    if ((int)threadIdx.x < kCols) h[nc + threadIdx.x] = 0.0;
    __syncthreads();
    if (alpha && blockIdx.x == 0 && threadIdx.x == 0) *alpha = h[nc - 1];
    double sq = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
        double wi = w[i];
        for (int c0 = 0; c0 < nc; c0 += kCols) {
            double v[kCols];
#pragma unroll
            for (int c = 0; c < kCols; ++c) v[c] = V[(int64_t)min(c0 + c, nc - 1) * n + i];
#pragma unroll
            for (int c = 0; c < kCols; ++c) wi -= v[c] * h[c0 + c];
        }
        w[i] = wi;
        sq += wi * wi;
    }
    sq = wave_sum(sq);
    if (lane == 0) lds[wave] = sq;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < kWaves; ++k) sq += lds[k];
        norm[blockIdx.x] = sq;
    }
}

// beta = |w| from its nb partial sums; v = w / beta (zero where beta is)
__global__ __launch_bounds__(kThreads) void lanczos_next_kernel(double *__restrict__ v, const double *__restrict__ w,
                                                                int64_t n, const double *__restrict__ norm, int nb,
                                                                double *beta) {
    __shared__ double lds[kWaves];
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += kThreads) s += norm[b];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x / 64] = s;
    __syncthreads();
    s = lds[0];
    for (int k = 1; k < kWaves; ++k) s += lds[k];
    const double b = sqrt(s), inv = b == 0.0 ? 0.0 : 1.0 / b;
    if (blockIdx.x == 0 && threadIdx.x == 0) *beta = b;
    for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads)
        v[i] = w[i] * inv;
}

}  // namespace

// V: nc columns of n, w orthogonalised against them twice; v (null: not wanted)
// = w / |w|.  part: kLanczosMost + 1 rows of kLanczosBlocks.
hipError_t launch_lanczos(const double *V, double *w, int64_t n, int nc, double *v, double *part, double *alpha,
                          double *beta, hipStream_t s) {
    const int nb = (int)std::min<int64_t>(kLanczosBlocks, (n + kThreads - 1) / kThreads);
    double *norm = part + (int64_t)kLanczosMost * kLanczosBlocks;
    for (int pass = 0; pass < 2; ++pass) {
        hipLaunchKernelGGL(lanczos_dots_kernel, dim3(nb), dim3(kThreads), 0, s, V, w, n, nc, part);
        hipLaunchKernelGGL(lanczos_project_kernel, dim3(nb), dim3(kThreads), 0, s, V, w, n, nc, part, norm,
                           pass ? nullptr : alpha);
    }
    hipLaunchKernelGGL(lanczos_next_kernel, dim3(v ? nb : 1), dim3(kThreads), 0, s, v, w, v ? n : 0, norm, nb, beta);
    return hipGetLastError();
}

}  // namespace fe
