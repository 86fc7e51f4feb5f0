// The start and the end of the symmetric product from one triangle (Sec. V: a
// symmetric matrix multiplied through one of its halves, without duplicated
// off-diagonal entries): sums = beta y + alpha d .* x in FP64, to which the
// off-diagonal halves add, and y = sums rounded.  FP64 needs no end: its sums
// are y.
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dtans {
namespace {

// (y and sums may be the same array)
template <typename VT, typename ST>
__global__ __launch_bounds__(256) void sym_start_kernel(const VT *d, const VT *x, const VT *y, ST *sums, int64_t n,
                                                        double alpha, double beta) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double t = d ? alpha * (double)d[i] * (double)x[i] : 0.0;
        sums[i] = (ST)(beta == 0.0 ? t : beta * (double)y[i] + t);
    }
}

__global__ __launch_bounds__(256) void sym_end_kernel(const double *__restrict__ sums, float *__restrict__ y,
                                                      int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = (float)sums[i];
}

unsigned vector_grid(int64_t n) { return (unsigned)(n / 256 + 1 < 65536 ? n / 256 + 1 : 65536); }

}  // namespace

hipError_t launch_sym_start(bool f64, const void *d, const void *x, void *y, double *sums, int64_t n, double alpha,
                            double beta, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const dim3 grid(vector_grid(n)), block(256);
    if (f64)
        hipLaunchKernelGGL((sym_start_kernel<double, double>), grid, block, 0, st, (const double *)d,
                           (const double *)x, (const double *)y, (double *)y, n, alpha, beta);
    else if (sums)
        hipLaunchKernelGGL((sym_start_kernel<float, double>), grid, block, 0, st, (const float *)d, (const float *)x,
                           (const float *)y, sums, n, alpha, beta);
    else
        hipLaunchKernelGGL((sym_start_kernel<float, float>), grid, block, 0, st, (const float *)d, (const float *)x,
                           (const float *)y, (float *)y, n, alpha, beta);
    return hipGetLastError();
}

hipError_t launch_sym_end(const double *sums, float *y, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(sym_end_kernel, dim3(vector_grid(n)), dim3(256), 0, st, sums, y, n);
    return hipGetLastError();
}

}  // namespace dtans
