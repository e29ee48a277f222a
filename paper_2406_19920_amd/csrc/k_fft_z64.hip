// FP64 fast z transforms (k_fft.h), one instantiation per size.
#include "k_fft.h"

namespace ibs {

template <int R1, int R2, typename Set>
static void go(const Set &js, int rows, int nx, bool inverse, bool walls, hipStream_t s)
{
    constexpr int CW = 128 / sizeof(double);
    const dim3 grid(rows * nx / CW, js.n), blk(fft::Shape<R1, R2>::threads(CW));
    if (inverse && walls) fft_z_kernel<double, double, R1, R2, true, true><<<grid, blk, 0, s>>>(js, nx, nullptr);
    else if (inverse) fft_z_kernel<double, double, R1, R2, true, false><<<grid, blk, 0, s>>>(js, nx, nullptr);
    else if (walls) fft_z_kernel<double, double, R1, R2, false, true><<<grid, blk, 0, s>>>(js, nx, nullptr);
    else fft_z_kernel<double, double, R1, R2, false, false><<<grid, blk, 0, s>>>(js, nx, nullptr);
}

template <typename Set>
static hipError_t by_size(const Set &js, int n, int rows, int nx, bool inverse, bool walls, hipStream_t s)
{
    if (js.n == 0) return hipSuccess;
    switch (n) {
#define IBS_CASE(N, R1, R2) case N: go<R1, R2>(js, rows, nx, inverse, walls, s); break;
    IBS_FFT_SIZES_32(IBS_CASE) IBS_FFT_SIZES_16(IBS_CASE)
#undef IBS_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_fft_z64(const FftSet &js, int n, int rows, int nx, bool inverse, bool walls, hipStream_t s)
{
    return by_size(js, n, rows, nx, inverse, walls, s);
}
hipError_t launch_fft_z64(const FftTable &js, int n, int rows, int nx, bool inverse, bool walls, hipStream_t s)
{
    return by_size(js, n, rows, nx, inverse, walls, s);
}

}  // namespace ibs
