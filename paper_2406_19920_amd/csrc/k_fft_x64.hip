// FP64 fast x transforms (k_fft.h), one instantiation per size.
#include "k_fft.h"

namespace ibs {

template <int R1, int R2, bool INV, int AX, typename Set>
static void one(const Set &js, int rows, int nz, hipStream_t s)
{
    const dim3 grid(nz * rows / FFT_RW, js.n), blk(fft::Shape<R1, R2>::threads(AX, FFT_RW));
    fft_x_kernel<double, double, double, R1, R2, INV, AX, 0><<<grid, blk, 0, s>>>(js, nz, nullptr, 0, nullptr, nullptr);
}

template <int R1, int R2, typename Set>
static void go(const Set &js, int rows, int nz, bool inverse, int ax, hipStream_t s)
{
    if (ax == fft::AX_FACES) one<R1, R2, true, fft::AX_FACES>(js, rows, nz, s);   // its own inverse
    else if (inverse && ax) one<R1, R2, true, fft::AX_CENTRES>(js, rows, nz, s);
    else if (inverse) one<R1, R2, true, fft::AX_PERIODIC>(js, rows, nz, s);
    else if (ax) one<R1, R2, false, fft::AX_CENTRES>(js, rows, nz, s);
    else one<R1, R2, false, fft::AX_PERIODIC>(js, rows, nz, s);
}

template <typename Set>
static hipError_t by_size(const Set &js, int n, int rows, int nz, bool inverse, int ax, hipStream_t s)
{
    if (js.n == 0) return hipSuccess;
    switch (n) {
#define IBS_CASE(N, R1, R2) case N: go<R1, R2>(js, rows, nz, inverse, ax, s); break;
    IBS_FFT_SIZES_32(IBS_CASE) IBS_FFT_SIZES_16(IBS_CASE)
#undef IBS_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_fft_x64(const FftSet &js, int n, int rows, int nz, bool inverse, int ax, hipStream_t s)
{
    return by_size(js, n, rows, nz, inverse, ax, s);
}
hipError_t launch_fft_x64(const FftTable &js, int n, int rows, int nz, bool inverse, int ax, hipStream_t s)
{
    return by_size(js, n, rows, nz, inverse, ax, s);
}

}  // namespace ibs
