// Host check of the fast transforms' lines: for every length and basis, the
// work items of a line run one after the other (the code the kernels run one
// per thread) against the plan's dense bases, forward and inverse, in double
// and float.  Prints "fft N basis T errors"; exits non-zero on a slot out of
// range, missed or written twice.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <string>
#include <vector>

#include "fft_line.h"
#include "fft_sizes.h"
#include "ibs_internal.h"

namespace ibs {
ibs_status build_plan(const ibs_grid_desc &d, Plan *&out);
void set_error(const std::string &msg) { std::fprintf(stderr, "%s\n", msg.c_str()); }
}  // namespace ibs
using namespace ibs;

static void fail(const char *what, int n)
{
    std::printf("FAIL %s at %d\n", what, n);
    std::exit(1);
}

template <int R1, int R2, bool WALL, typename T, typename TF = T>   // TF: forward
static void check(const Plan &p, int basis)
{
    typedef fft::Shape<R1, R2> S;
    constexpr int N = S::N;
    const bool sine = basis == XK_C;
    const fft::Cpx<TF> *twf = reinterpret_cast<const fft::Cpx<TF> *>(p.blob.data() + (sizeof(TF) == 4 ? p.lay.ftx_fwd32 : p.lay.ftx_fwd));
    const fft::Cpx<TF> *rf = reinterpret_cast<const fft::Cpx<TF> *>(p.blob.data() + (sizeof(TF) == 4 ? p.lay.frx_fwd32 : p.lay.frx_fwd));
    const fft::Cpx<T> *twi = reinterpret_cast<const fft::Cpx<T> *>(p.blob.data() + p.lay.ftx_inv);
    const fft::Cpx<T> *ri = reinterpret_cast<const fft::Cpx<T> *>(p.blob.data() + p.lay.frx_inv);
    const std::vector<double> &Q = *p.qx[basis < 0 ? 0 : basis];
    std::mt19937_64 g(N);
    std::normal_distribution<double> nd;
    double worst_f = 0, worst_i = 0;
    for (int rep = 0; rep < 4; ++rep) {
        std::vector<T> x(N), out(N, 0), back(N, 0);
        for (T &v : x) v = (T)nd(g);
        std::vector<T> re(S::K1 * R2), im(S::K1 * R2);
        std::vector<int> hit(N, 0);
        // forward
        std::vector<TF> fre(S::K1 * R2), fim(S::K1 * R2);
        for (int n2 = 0; n2 < R2; ++n2) {
            TF v[R1], yr[S::K1], yi[S::K1];
            for (int n1 = 0; n1 < R1; ++n1) {
                const int i = fft::line_index<R1, R2, WALL>(n2, n1);
                if (i < 0 || i >= N) fail("line index", N);
                ++hit[i];
                v[n1] = WALL && sine && 2 * n1 >= R1 ? -(TF)x[i] : (TF)x[i];
            }
            fft::rdft<R1, TF>(v, yr, yi);
            for (int k1 = 0; k1 < S::K1; ++k1) {
                const fft::Cpx<TF> w = twf[k1 * R2 + n2];
                fre[k1 * R2 + n2] = w.x * yr[k1] - w.y * yi[k1];
                fim[k1 * R2 + n2] = w.x * yi[k1] + w.y * yr[k1];
            }
        }
        for (int i = 0; i < N; ++i)
            if (hit[i] != 1) fail("input coverage", N);
        hit.assign(N, 0);
        for (int k1 = 0; k1 < S::K1; ++k1) {
            TF a[R2], b[R2];
            for (int q = 0; q < R2; ++q) { a[q] = fre[k1 * R2 + q]; b[q] = fim[k1 * R2 + q]; }
            fft::cdft<R2, -1, TF>(a, b);
            fft::emit<R1, R2, WALL, TF>(a, b, k1, sine, rf, [&](int s, TF v) {
                if (s < 0 || s >= N) fail("spectral slot", N);
                ++hit[s];
                out[s] = (T)v;
            });
        }
        for (int i = 0; i < N; ++i)
            if (hit[i] != 1) fail("spectral coverage", N);
        double d2 = 0, n2s = 0;
        for (int a = 0; a < N; ++a) {
            long double s = 0;
            for (int i = 0; i < N; ++i) s += (long double)Q[(size_t)i * N + a] * (long double)x[i];
            d2 += (double)((out[a] - s) * (out[a] - s));
            n2s += (double)(s * s);
        }
        worst_f = std::max(worst_f, std::sqrt(d2 / n2s));
        // inverse of x taken as a spectrum
        for (int k1 = 0; k1 < S::K1; ++k1) {
            T a[R2], b[R2];
            fft::gather<R1, R2, WALL, T>(a, b, k1, sine, ri, [&](int s) {
                if (s < 0 || s >= N) fail("inverse slot", N);
                return x[s];
            });
            fft::cdft<R2, 1, T>(a, b);
            for (int q = 0; q < R2; ++q) {
                const fft::Cpx<T> w = twi[k1 * R2 + q];
                re[k1 * R2 + q] = w.x * a[q] - w.y * b[q];
                im[k1 * R2 + q] = w.x * b[q] + w.y * a[q];
            }
        }
        for (int n2 = 0; n2 < R2; ++n2) {
            T v[R1], yr[S::K1], yi[S::K1];
            for (int k1 = 0; k1 < S::K1; ++k1) { yr[k1] = re[k1 * R2 + n2]; yi[k1] = im[k1 * R2 + n2]; }
            fft::hdft<R1, T>(yr, yi, v);
            for (int n1 = 0; n1 < R1; ++n1)
                back[fft::line_index<R1, R2, WALL>(n2, n1)] = WALL && sine && 2 * n1 >= R1 ? -v[n1] : v[n1];
        }
        d2 = n2s = 0;
        for (int i = 0; i < N; ++i) {
            long double s = 0;
            for (int a = 0; a < N; ++a) s += (long double)Q[(size_t)i * N + a] * (long double)x[a];
            d2 += (double)((back[i] - s) * (back[i] - s));
            n2s += (double)(s * s);
        }
        worst_i = std::max(worst_i, std::sqrt(d2 / n2s));
    }
    std::printf("fft %d %d %d %.3e %.3e\n", N, basis, (int)sizeof(T), worst_f, worst_i);
}

// the sine basis on the inner faces: its own inverse, so one direction
template <int R1, int R2, typename T>
static void check_faces(const Plan &p)
{
    typedef fft::Shape<R1, R2> S;
    constexpr int N = S::N, NA = R2 + 1;
    const fft::Cpx<T> *tw = reinterpret_cast<const fft::Cpx<T> *>(p.blob.data() + p.lay.ftx_face);
    const std::vector<double> &Q = *p.qx[XK_F];
    std::mt19937_64 g(N);
    std::normal_distribution<double> nd;
    double worst = 0;
    for (int rep = 0; rep < 4; ++rep) {
        std::vector<T> x(N), out(N, 0), re(S::K1 * NA), im(S::K1 * NA);
        for (T &v : x) v = (T)nd(g);
        std::vector<int> hit(N, 0);
        for (int n2 = 0; n2 < NA; ++n2) {
            T v[R1], yr[S::K1], yi[S::K1];
            for (int n1 = 0; n1 < R1; ++n1) {
                const int i = fft::face_slot<R1, R2>(n2, n1);
                if (i < 0 || i >= N) fail("face slot", N);
                ++hit[i];
                v[n1] = fft::face_value<R1, T>(x[i], n2, n1);
            }
            fft::rdft<R1, T>(v, yr, yi);
            for (int k1 = 0; k1 < S::K1; ++k1) {
                const fft::Cpx<T> w = tw[k1 * NA + n2];
                re[k1 * NA + n2] = w.x * yr[k1] - w.y * yi[k1];
                im[k1 * NA + n2] = w.x * yi[k1] + w.y * yr[k1];
            }
        }
        for (int i = 0; i < N; ++i)
            if (!hit[i]) fail("face coverage", N);
        hit.assign(N, 0);
        for (int k1 = 0; k1 < S::K1; ++k1) {
            T a[NA], b[NA];
            for (int q = 0; q < NA; ++q) { a[q] = re[k1 * NA + q]; b[q] = im[k1 * NA + q]; }
            fft::face_emit<R1, R2, T>(a, b, k1, [&](int s, T v) {
                if (s < 0 || s >= N) fail("face spectral slot", N);
                ++hit[s];
                out[s] = v;
            });
        }
        for (int i = 0; i < N; ++i)
            if (hit[i] != 1) fail("face spectral coverage", N);
        double d2 = 0, n2s = 0;
        for (int a = 0; a < N; ++a) {
            long double s = 0;
            for (int i = 0; i < N; ++i) s += (long double)Q[(size_t)i * N + a] * (long double)x[i];
            d2 += (double)((out[a] - s) * (out[a] - s));
            n2s += (double)(s * s);
        }
        worst = std::max(worst, std::sqrt(d2 / n2s));
    }
    std::printf("fft %d %d %d %.3e %.3e\n", N, XK_F, (int)sizeof(T), worst, worst);
}

template <int R1, int R2> static void size(int n, bool refined)
{
    for (int walls = 0; walls < 2; ++walls) {
        ibs_grid_desc d{};
        d.nx = n; d.ny = 4; d.nz = 32;
        d.bc_x = walls ? IBS_DIRICHLET : IBS_PERIODIC;
        d.bc_z = IBS_PERIODIC; d.bc_y_vel = IBS_DIRICHLET; d.bc_y_p = IBS_NEUMANN;
        d.precision = refined ? IBS_REFINED_BF16X3 : IBS_FP64;
        Plan *p = nullptr;
        if (build_plan(d, p) != IBS_OK) fail("plan", n);
        if (!p->fx) fail("kinds", n);
        if (refined && n > FFT_F64_ARITH_MAX) {
            if (walls) { check<R1, R2, true, float, double>(*p, XK_P); check<R1, R2, true, float>(*p, XK_C); check_faces<R1, R2, float>(*p); }
            else { check<R1, R2, false, float, double>(*p, -1); check<R1, R2, false, float>(*p, -1); }
        } else {
            if (walls) { check<R1, R2, true, double>(*p, XK_P); check<R1, R2, true, double>(*p, XK_C); check_faces<R1, R2, double>(*p); }
            else check<R1, R2, false, double>(*p, -1);
        }
        delete p;
    }
}

int main()
{
#define IBS_CASE(N, R1, R2) size<R1, R2>(N, false);
    IBS_FFT_SIZES_32(IBS_CASE) IBS_FFT_SIZES_16(IBS_CASE)
#undef IBS_CASE
#define IBS_CASE(N, R1, R2) size<R1, R2>(N, true);
    IBS_FFT_SIZES_32(IBS_CASE)
#undef IBS_CASE
    return 0;
}
