// Adjoint kernel instances, FP32, and the small helpers of the adjoint driver.
#include "adjoint2d.hpp"

namespace mp {
template int adj_launch<float>(const AdjLaunch&, const AdjCoef<float>&, hipStream_t);

__global__ void k_fill_f64(double* p, int64_t n, double v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Column sums of the per-block accumulator rows, each in row order.  The rows
// (256 on a filled chip) come in by the whole block; a lane reading its column
// from memory waited for a row at a time: 41.7 us, now 6.2.
constexpr int ADJ_RED_ROWS = 256;
__global__ void __launch_bounds__(256) k_adj_reduce(const double* __restrict__ acc, int nrows,
                                                    double* __restrict__ out) {
    __shared__ double buf[ADJ_RED_ROWS * ADJ_NPAR];
    const int t = threadIdx.x;
    double s = 0.0;
    for (int r0 = 0; r0 < nrows; r0 += ADJ_RED_ROWS) {
        const int n = min(ADJ_RED_ROWS, nrows - r0);
        for (int i = t; i < n * ADJ_NPAR; i += 256) buf[i] = acc[(size_t)r0 * ADJ_NPAR + i];
        __syncthreads();
        if (t < ADJ_NPAR) {
#pragma unroll 8
            for (int r = 0; r < n; ++r) s += buf[r * ADJ_NPAR + t];
        }
        __syncthreads();
    }
    if (t < ADJ_NPAR) out[t] = s;
}

void adj_fill(double* p, int64_t n, double v, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_f64, dim3(64), dim3(256), 0, s, p, n, v);
}

void adj_reduce(const double* acc, int nrows, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_adj_reduce, dim3(1), dim3(256), 0, s, acc, nrows, out);
}
}  // namespace mp
