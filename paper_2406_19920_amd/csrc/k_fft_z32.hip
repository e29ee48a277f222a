// FP32 fast z transforms (k_fft.h), one instantiation per size.
#include "k_fft.h"

namespace ibs {

template <int R1, int R2, bool INV, int AX, bool EXACT>
static void one(const FftSet &js, int rows, int nx, const int *skip, hipStream_t s)
{
    typedef typename FftReal<R1 * R2, EXACT>::type T;
    constexpr int CW = fft_cw<float, T, R1 * R2>();
    int runs;
    const dim3 grid(fft_z_tiles<float>(rows, nx, CW, runs), js.n), blk(fft::Shape<R1, R2>::threads(AX, CW));
    fft_z_kernel<float, T, R1, R2, INV, AX><<<grid, blk, 0, s>>>(js, nx, runs, skip);
}

template <int R1, int R2>
static void go(const FftSet &js, int rows, int nx, bool inverse, int ax, bool exact, const int *skip, hipStream_t s)
{
    // the faces' transform is its own inverse, in the direction's arithmetic
    if (ax == fft::AX_FACES && exact && !inverse) one<R1, R2, true, fft::AX_FACES, true>(js, rows, nx, skip, s);
    else if (ax == fft::AX_FACES) one<R1, R2, true, fft::AX_FACES, false>(js, rows, nx, skip, s);
    else if (inverse && ax) one<R1, R2, true, fft::AX_CENTRES, false>(js, rows, nx, skip, s);
    else if (inverse) one<R1, R2, true, fft::AX_PERIODIC, false>(js, rows, nx, skip, s);
    else if (ax && exact) one<R1, R2, false, fft::AX_CENTRES, true>(js, rows, nx, skip, s);
    else if (ax) one<R1, R2, false, fft::AX_CENTRES, false>(js, rows, nx, skip, s);
    else if (exact) one<R1, R2, false, fft::AX_PERIODIC, true>(js, rows, nx, skip, s);
    else one<R1, R2, false, fft::AX_PERIODIC, false>(js, rows, nx, skip, s);
}

hipError_t launch_fft_z32(const FftSet &js, int n, int rows, int nx, bool inverse, int ax, bool exact, const int *skip,
                          hipStream_t s)
{
    if (js.n == 0) return hipSuccess;
    switch (n) {
#define IBS_CASE(N, R1, R2) case N: go<R1, R2>(js, rows, nx, inverse, ax, exact, skip, s); break;
    IBS_FFT_SIZES_32(IBS_CASE)
#undef IBS_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace ibs
