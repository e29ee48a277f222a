// FP32 fast forward x transforms (k_fft.h) of the refined path, one
// instantiation per size.
#include "k_fft.h"

namespace ibs {

template <int R1, int R2, int AX, bool EXACT>
static void go(const FftSet &js, int rows, int nz, bool in64, const int *skip, hipStream_t s)
{
    typedef typename FftReal<R1 * R2, EXACT>::type T;
    const dim3 grid(nz * rows / FFT_RW, js.n), blk(fft::Shape<R1, R2>::threads(AX, FFT_RW));
    if (in64) fft_x_kernel<double, float, T, R1, R2, false, AX, 0><<<grid, blk, 0, s>>>(js, nz, nullptr, 0, skip, nullptr);
    else fft_x_kernel<float, float, T, R1, R2, false, AX, 0><<<grid, blk, 0, s>>>(js, nz, nullptr, 0, skip, nullptr);
}

hipError_t launch_fft_x32_fwd(const FftSet &js, int n, int rows, int nz, int ax, bool exact, bool in64,
                              const int *skip,
                              hipStream_t s)
{
    if (js.n == 0) return hipSuccess;
    switch (n) {
#define IBS_CASE(N, R1, R2)                                                                       \
    case N:                                                                                       \
        if (ax == fft::AX_FACES && exact) go<R1, R2, fft::AX_FACES, true>(js, rows, nz, in64, skip, s);   \
        else if (ax == fft::AX_FACES) go<R1, R2, fft::AX_FACES, false>(js, rows, nz, in64, skip, s);      \
        else if (ax && exact) go<R1, R2, fft::AX_CENTRES, true>(js, rows, nz, in64, skip, s);     \
        else if (ax) go<R1, R2, fft::AX_CENTRES, false>(js, rows, nz, in64, skip, s);             \
        else if (exact) go<R1, R2, fft::AX_PERIODIC, true>(js, rows, nz, in64, skip, s);          \
        else go<R1, R2, fft::AX_PERIODIC, false>(js, rows, nz, in64, skip, s);                    \
        break;
    IBS_FFT_SIZES_32(IBS_CASE)
#undef IBS_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace ibs
