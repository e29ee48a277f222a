// Cyclic tridiagonal pencils of the triply periodic branch (Section 2.3.3,
// items S1 and S2 with y periodic too): the partitioned solve of
// tridiag.h with CYC = true, one shape per supported row count (the P
// chunks of M rows must hold the system exactly, since a cyclic system has
// no end at which padding rows could sit).
#include "tridiag.h"

namespace ibs {

template <typename T, typename R>
static hipError_t launch_cyclic(const TriSet &src, int n, hipStream_t s)
{
    switch (n) {
    case 48: return launch_pm<T, R, 12, 4, true>(src, s);
    case 64: return launch_pm<T, R, 16, 4, true>(src, s);
    case 80: return launch_pm<T, R, 20, 4, true>(src, s);
    case 96: return launch_pm<T, R, 12, 8, true>(src, s);
    case 128: return launch_pm<T, R, 16, 8, true>(src, s);
    case 160: return launch_pm<T, R, 20, 8, true>(src, s);
    case 192: return launch_pm<T, R, 16, 12, true>(src, s);
    case 256: return launch_pm<T, R, 16, 16, true>(src, s);
    case 320:
        if constexpr (sizeof(R) == 4) return launch_pm<T, R, 20, 16, true>(src, s);
        else return launch_pm<T, R, 32, 10, true>(src, s);
    case 384:
        if constexpr (sizeof(R) == 4) return launch_pm<T, R, 24, 16, true>(src, s);
        else return launch_pm<T, R, 32, 12, true>(src, s);
    case 512: return launch_pm<T, R, 32, 16, true>(src, s);
    default: return hipErrorInvalidValue;
    }
}

// cyclic_rows_supported() (the sizes above) is defined with the plan
// builder (host code).

hipError_t launch_cyclic_dd(const TriSet &src, int n, hipStream_t s)
{
    return launch_cyclic<double, double>(src, n, s);
}
hipError_t launch_cyclic_fd(const TriSet &src, int n, hipStream_t s)
{
    return launch_cyclic<float, double>(src, n, s);
}
hipError_t launch_cyclic_ff(const TriSet &src, int n, hipStream_t s)
{
    return launch_cyclic<float, float>(src, n, s);
}

}  // namespace ibs
