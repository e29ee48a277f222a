// FP64 fast z transforms (k_fft.h), one instantiation per size.
#include "k_fft.h"

namespace ibs {

template <int R1, int R2, bool INV, int AX, typename Set>
static void one(const Set &js, int rows, int nx, hipStream_t s)
{
    constexpr int CW = 128 / sizeof(double);
    int runs;
    const dim3 grid(fft_z_tiles<double>(rows, nx, CW, runs), js.n), blk(fft::Shape<R1, R2>::threads(AX, CW));
    fft_z_kernel<double, double, R1, R2, INV, AX><<<grid, blk, 0, s>>>(js, nx, runs, nullptr);
}

template <int R1, int R2, typename Set>
static void go(const Set &js, int rows, int nx, bool inverse, int ax, hipStream_t s)
{
    if (ax == fft::AX_FACES) one<R1, R2, true, fft::AX_FACES>(js, rows, nx, s);   // its own inverse
    else if (inverse && ax) one<R1, R2, true, fft::AX_CENTRES>(js, rows, nx, s);
    else if (inverse) one<R1, R2, true, fft::AX_PERIODIC>(js, rows, nx, s);
    else if (ax) one<R1, R2, false, fft::AX_CENTRES>(js, rows, nx, s);
    else one<R1, R2, false, fft::AX_PERIODIC>(js, rows, nx, s);
}

template <typename Set>
static hipError_t by_size(const Set &js, int n, int rows, int nx, bool inverse, int ax, hipStream_t s)
{
    if (js.n == 0) return hipSuccess;
    switch (n) {
#define IBS_CASE(N, R1, R2) case N: go<R1, R2>(js, rows, nx, inverse, ax, s); break;
    IBS_FFT_SIZES_32(IBS_CASE) IBS_FFT_SIZES_16(IBS_CASE)
#undef IBS_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_fft_z64(const FftSet &js, int n, int rows, int nx, bool inverse, int ax, hipStream_t s)
{
    return by_size(js, n, rows, nx, inverse, ax, s);
}
hipError_t launch_fft_z64(const FftTable &js, int n, int rows, int nx, bool inverse, int ax, hipStream_t s)
{
    return by_size(js, n, rows, nx, inverse, ax, s);
}

}  // namespace ibs
