// x and z transforms of short periodic lines in one pass (k_fft.h's two, for
// both axes at once): one block per transform row y holds the plane [z][x] of
// that row in LDS, transforms its lines along the first axis, then along the
// second, and writes it back.
//
// Why: fields of short lines are small, and their passes are bound by launch
// latency (a 32^3 pass takes 3 us) or, many at a time, by the Infinity Cache;
// the fused pair saves a launch and a read and a write of the field per
// direction (63 fields of 64^3: 76 + 74 us where the four passes took 99 + 90;
// bound by FP64 issue, about 45 us of it, and the barriers).
// Lines as in k_fft.h, a work item per thread, 32 lines side by side in the
// lanes (row pitch odd, so x lines use different banks).  The exchange between
// the stages lies in the line itself: stage A's item n2 owns the R1 points n2 +
// R2 m, stage B's item k1 the blocks m = k1 and R1 - k1 of R2 points; k1 = 0
// and R1/2 need one block each, being real (up to R1/2's twiddle factors, which
// stage B applies).  So a 64 x 64 plane takes 33 KB and four blocks fit a CU
// (with an exchange buffer of its own: three, and 10% slower).
// All arithmetic and the plane in FP64.
#pragma once
#include "fft_line.h"
#include "fft_sizes.h"
#include "ibs_internal.h"

namespace ibs {

struct PlaneJob {
    const void *in;
    void *out;        // as FftJob's
    const void *xs;   // MODE 4: the stored FP32 iterate
    double *x0;       // MODE 3: the FP64 field whose wall rows are zeroed too
    const void *twx, *twz;
    int rows, skip;   // rows per plane; 1: the first row of a plane is left out
    int slot;         // job number in the call's state
};
struct PlaneSet {
    PlaneJob j[4];
    int n;
};
struct PlaneTable {   // any number of jobs in device memory
    const PlaneJob *j;
    int n;
};

// Planes of up to MAXN x MAXN points: row pitch in LDS, work items a line (x
// L lines at a time: a block).
template <int MAXN, int L> struct PlaneShape {
    static constexpr int PITCH = MAXN + 1, LANES = L, ITEMS = MAXN <= 48 ? 6 : 8, NT = ITEMS * LANES;
};

namespace fft {

// Every line of the plane along one axis.  The pitch is a constant: LDS
// offsets are immediates.
template <int R1, int R2, bool INV, bool Z, int MAXN, int L>
static __device__ __forceinline__ void plane_lines(double *P, int lines, const Cpx<double> *tw)
{
    typedef Shape<R1, R2> S;
    typedef PlaneShape<MAXN, L> B;
    static_assert(R2 <= B::ITEMS && S::K1 <= B::ITEMS, "items per line");
    constexpr int ls = Z ? 1 : B::PITCH, ps = Z ? B::PITCH : 1;
    const int lane = threadIdx.x % B::LANES, item = threadIdx.x / B::LANES;
    for (int l0 = 0; l0 < lines; l0 += B::LANES) {
        const bool on = l0 + lane < lines, onA = on && item < R2, onB = on && item < S::K1;
        double *const p = P + (l0 + lane) * ls;
        double *const own = p + item * ps;                            // stage A's points: + R2 m
        double *const lo = p + item * R2 * ps;                        // stage B's blocks: + n2
        double *const hi = p + (R1 - item) * R2 * ps;
        const bool mid = 2 * item == R1, ends = item == 0 || mid;
        double re[R2], im[R2];
        if constexpr (!INV) {
            if (onA) {
                double x[R1], yr[S::K1], yi[S::K1];
#pragma unroll
                for (int n1 = 0; n1 < R1; ++n1) x[n1] = own[R2 * n1 * ps];
                rdft<R1, double>(x, yr, yi);
                own[0] = yr[0] * tw[item].x;
                own[R2 * (R1 / 2) * ps] = yr[R1 / 2];
#pragma unroll
                for (int k1 = 1; k1 < R1 / 2; ++k1) {
                    const Cpx<double> w = tw[k1 * R2 + item];
                    own[R2 * k1 * ps] = w.x * yr[k1] - w.y * yi[k1];
                    own[R2 * (R1 - k1) * ps] = w.x * yi[k1] + w.y * yr[k1];
                }
            }
            __syncthreads();
            if (onB) {
#pragma unroll
                for (int q = 0; q < R2; ++q) re[q] = lo[q * ps];
                if (!ends) {
#pragma unroll
                    for (int q = 0; q < R2; ++q) im[q] = hi[q * ps];
                } else if (mid) {
#pragma unroll
                    for (int q = 0; q < R2; ++q) {
                        const Cpx<double> w = tw[(R1 / 2) * R2 + q];
                        im[q] = re[q] * w.y;
                        re[q] *= w.x;
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < R2; ++q) im[q] = 0.0;
                }
            }
            __syncthreads();
            if (onB) {
                cdft<R2, -1, double>(re, im);
                emit<R1, R2, false, double>(re, im, item, false, nullptr, [&](int a, double v) { p[a * ps] = v; });
            }
        } else {
            if (onB) {
                gather<R1, R2, false, double>(re, im, item, false, nullptr, [&](int a) { return p[a * ps]; });
                cdft<R2, 1, double>(re, im);
            }
            __syncthreads();
            if (onB) {
#pragma unroll
                for (int q = 0; q < R2; ++q) {
                    const Cpx<double> w = tw[item * R2 + q];
                    lo[q * ps] = w.x * re[q] - w.y * im[q];
                    if (!ends) hi[q * ps] = w.x * im[q] + w.y * re[q];
                }
            }
            __syncthreads();
            if (onA) {
                double x[R1], yr[S::K1], yi[S::K1];
                yr[0] = own[0];
                yr[R1 / 2] = own[R2 * (R1 / 2) * ps];
                yi[0] = yi[R1 / 2] = 0.0;
#pragma unroll
                for (int k1 = 1; k1 < R1 / 2; ++k1) {
                    yr[k1] = own[R2 * k1 * ps];
                    yi[k1] = own[R2 * (R1 - k1) * ps];
                }
                hdft<R1, double>(yr, yi, x);
#pragma unroll
                for (int n1 = 0; n1 < R1; ++n1) own[R2 * n1 * ps] = x[n1];
            }
        }
    }
    __syncthreads();
}

}  // namespace fft

// One plane per block: blockIdx.x the transform row, blockIdx.y the job.
// TIN: stored type of the input, TS: of the spectrum; MODE as fft_x_kernel's
// (INV, FP32 data).
template <typename TIN, typename TS, bool INV, int MODE, int MAXN, int L, typename Set>
__global__ __launch_bounds__((PlaneShape<MAXN, L>::NT), 4) void plane_kernel(Set js, int nx, int nz, double *red, int red_stride,
                                                         const int *skip, const double *scale)
{
    using namespace fft;
    typedef PlaneShape<MAXN, L> B;
    constexpr int NT = B::NT, pitch = B::PITCH;
    constexpr bool UPD = MODE == 2 || MODE == 4;
    typedef typename std::conditional<MODE == 1 || UPD, double, TS>::type Tout;
    __shared__ double P[MAXN * pitch];
    const PlaneJob &jb = js.j[blockIdx.y];
    if (skip && skip[jb.slot]) return;
    // this thread's pair of points: column 2 q, rows r0, r0 + step, ...
    const int vec = nx / 2, q = threadIdx.x % vec, r0 = threadIdx.x / vec, step = NT / vec;
    const int j = (int)blockIdx.x + jb.skip;
    const size_t ldp = (size_t)jb.rows * nx, base = (size_t)j * nx + 2 * q;
    constexpr int U = 8;   // loads in flight
    if (r0 < step) {
        typedef TIN vin __attribute__((ext_vector_type(2)));
        const TIN *in = static_cast<const TIN *>(jb.in);
        for (int k0 = r0; k0 < nz; k0 += U * step) {
            vin v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const vin *>(in + (size_t)min(k0 + u * step, nz - 1) * ldp + base);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k0 + u * step < nz) {
                    P[(k0 + u * step) * pitch + 2 * q] = (double)v[u][0];
                    P[(k0 + u * step) * pitch + 2 * q + 1] = (double)v[u][1];
                }
        }
    }
    __syncthreads();
    const Cpx<double> *twx = static_cast<const Cpx<double> *>(jb.twx), *twz = static_cast<const Cpx<double> *>(jb.twz);
    auto along = [&](auto zaxis) {
        constexpr bool Z = decltype(zaxis)::value;
        switch (Z ? nz : nx) {
#define IBS_CASE(N, R1, R2)                                                                              \
    case N:                                                                                              \
        if constexpr (N <= MAXN) plane_lines<R1, R2, INV, Z, MAXN, L>(P, Z ? nx : nz, Z ? twz : twx);    \
        break;
        IBS_PLANE_SIZES(IBS_CASE)
#undef IBS_CASE
        }
    };
    along(std::integral_constant<bool, INV>());   // forward x first, inverse z
    along(std::integral_constant<bool, !INV>());
    Tout *out = static_cast<Tout *>(jb.out);
    typedef Tout vout __attribute__((ext_vector_type(2)));
    double sd = 0.0, sx = 0.0;
    if (r0 < step) {
        if constexpr (UPD) {
            typedef typename std::conditional<MODE == 4, float, double>::type Told;
            typedef Told vold __attribute__((ext_vector_type(2)));
            const Told *xo = MODE == 4 ? static_cast<const Told *>(jb.xs) : static_cast<const Told *>(jb.out);
            const double isg = scale ? 1.0 / scale[jb.slot] : 1.0;
            for (int k0 = r0; k0 < nz; k0 += U * step) {
                vold v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const vold *>(xo + (size_t)min(k0 + u * step, nz - 1) * ldp + base);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (k0 + u * step < nz) {
                        vout o;
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const double d = P[(k0 + u * step) * pitch + 2 * q + e] * isg, xn = (double)v[u][e] + d;
                            o[e] = xn;
                            sd += d * d;
                            sx += xn * xn;
                        }
                        *reinterpret_cast<vout *>(out + (size_t)(k0 + u * step) * ldp + base) = o;
                    }
            }
        } else {
            for (int k = r0; k < nz; k += step) {
                vout o;
                o[0] = (Tout)P[k * pitch + 2 * q];
                o[1] = (Tout)P[k * pitch + 2 * q + 1];
                *reinterpret_cast<vout *>(out + (size_t)k * ldp + base) = o;
                if constexpr (MODE == 1 || MODE == 3)
                    if (jb.skip && blockIdx.x == 0) {   // the left-out wall row holds zeros in the result
                        const size_t w = (size_t)k * ldp + base - nx;
                        *reinterpret_cast<vout *>(out + w) = vout{};
                        if constexpr (MODE == 3) jb.x0[w] = jb.x0[w + 1] = 0.0;
                    }
            }
        }
    }
    if constexpr (UPD) {
        // block sums in a fixed order: butterflies, then the waves in turn
        constexpr int NW = NT / 64;
        __shared__ double ss[2][NW];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            sd += __shfl_xor(sd, d, 64);
            sx += __shfl_xor(sx, d, 64);
        }
        if ((threadIdx.x & 63) == 0) {
            ss[0][threadIdx.x >> 6] = sd;
            ss[1][threadIdx.x >> 6] = sx;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            double a = 0.0, b = 0.0;
            for (int w = 0; w < NW; ++w) {
                a += ss[0][w];
                b += ss[1][w];
            }
            const size_t at = 2 * ((size_t)jb.slot * red_stride + blockIdx.x);
            red[at] = a;
            red[at + 1] = b;
        }
    }
}

}  // namespace ibs
