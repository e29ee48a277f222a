// FP32 fast inverse x transforms (k_fft.h) of the refined path, walls in x (fields on cell
// centres), with their store and update epilogues,
// one instantiation per size.
#include "k_fft.h"

namespace ibs {

template <int R1, int R2, int AX>
static void go(const FftSet &js, int rows, int nz, int mode, double *red, int red_stride, const int *skip,
               const double *scale, hipStream_t s)
{
    typedef typename FftReal<R1 * R2, false>::type T;
    const dim3 grid(nz * rows / FFT_RW, js.n), blk(fft::Shape<R1, R2>::threads(AX, FFT_RW));
    switch (mode) {
    case 1: fft_x_kernel<float, float, T, R1, R2, true, AX, 1><<<grid, blk, 0, s>>>(js, nz, red, red_stride, skip, scale); break;
    case 2: fft_x_kernel<float, float, T, R1, R2, true, AX, 2><<<grid, blk, 0, s>>>(js, nz, red, red_stride, skip, scale); break;
    case 3: fft_x_kernel<float, float, T, R1, R2, true, AX, 3><<<grid, blk, 0, s>>>(js, nz, red, red_stride, skip, scale); break;
    default: fft_x_kernel<float, float, T, R1, R2, true, AX, 4><<<grid, blk, 0, s>>>(js, nz, red, red_stride, skip, scale); break;
    }
}

hipError_t launch_fft_x32_wall(const FftSet &js, int n, int rows, int nz, int mode, double *red, int red_stride, const int *skip,
                             const double *scale, hipStream_t s)
{
    if (js.n == 0) return hipSuccess;
    switch (n) {
#define IBS_CASE(N, R1, R2) case N: go<R1, R2, fft::AX_CENTRES>(js, rows, nz, mode, red, red_stride, skip, scale, s); break;
    IBS_FFT_SIZES_32(IBS_CASE)
#undef IBS_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace ibs
