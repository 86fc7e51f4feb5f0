// The start of the symmetric product from one triangle (Sec. V: a symmetric
// matrix multiplied through one of its halves, without duplicated off-diagonal
// entries): y = beta y + alpha d .* x, to which the off-diagonal halves add.
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dtans {
namespace {

template <typename VT>
__global__ __launch_bounds__(256) void sym_start_kernel(const VT *__restrict__ d, const VT *__restrict__ x,
                                                        VT *__restrict__ y, int64_t n, double alpha, double beta) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double t = d ? alpha * (double)d[i] * (double)x[i] : 0.0;
        y[i] = (VT)(beta == 0.0 ? t : beta * (double)y[i] + t);
    }
}

}  // namespace

hipError_t launch_sym_start(bool f64, const void *d, const void *x, void *y, int64_t n, double alpha, double beta,
                            hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const unsigned grid = (unsigned)(n / 256 + 1 < 65536 ? n / 256 + 1 : 65536);
    if (f64)
        hipLaunchKernelGGL(sym_start_kernel<double>, dim3(grid), dim3(256), 0, st, (const double *)d,
                           (const double *)x, (double *)y, n, alpha, beta);
    else
        hipLaunchKernelGGL(sym_start_kernel<float>, dim3(grid), dim3(256), 0, st, (const float *)d,
                           (const float *)x, (float *)y, n, alpha, beta);
    return hipGetLastError();
}

}  // namespace dtans
