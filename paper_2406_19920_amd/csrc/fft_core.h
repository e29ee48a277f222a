// Small discrete Fourier transforms held in registers, the building blocks
// of the fast eigen-transforms (k_fft.h).  Every size is a compile-time
// constant and every loop unrolls, so the arrays live in vector registers
// and the roots of unity are literals.
//
//   cdft<R, SIGN>   R complex values in place, X_k = sum_n x_n e^{SIGN 2 pi i nk/R}
//   rdft<R>         R real values to X_0 .. X_{R/2} (SIGN = -1)
//   hdft<R>         X_0 .. X_{R/2} of a Hermitian X to the R real values
//                   sum_k X_k e^{+2 pi i nk/R}
//
// Composite sizes split by 4, 2, 3, 5, 7 (decimation in time); the odd
// sizes left (and primes) are summed directly over the pairs (n, R - n).
#pragma once
#include <hip/hip_runtime.h>

#include <utility>

// usable on both sides: the kernels run them, host checks call the same code
#define IBS_FFT_FN __host__ __device__ __forceinline__

namespace ibs {
namespace fft {

// cos and sin of 2 pi k / R at compile time: reduced exactly to the first
// octant, then Taylor series in double-double arithmetic (error below an
// ulp of double).
struct DD {
    double h, l;
};
constexpr DD two_sum(double a, double b)
{
    const double s = a + b, t = s - a;
    return {s, (a - (s - t)) + (b - t)};
}
constexpr DD two_prod(double a, double b)
{
    const double p = a * b;
    const double c = 134217729.0 * a, ah = c - (c - a), al = a - ah;
    const double d = 134217729.0 * b, bh = d - (d - b), bl = b - bh;
    return {p, ((ah * bh - p) + ah * bl + al * bh) + al * bl};
}
constexpr DD dd_add(DD a, DD b)
{
    const DD s = two_sum(a.h, b.h);
    return two_sum(s.h, s.l + a.l + b.l);
}
constexpr DD dd_mul(DD a, DD b)
{
    const DD p = two_prod(a.h, b.h);
    return two_sum(p.h, p.l + a.h * b.l + a.l * b.h);
}
constexpr DD dd_div(DD a, double b)
{
    const double q = a.h / b;
    const DD p = two_prod(q, b);
    return two_sum(q, ((a.h - p.h) - p.l + a.l) / b);
}
// series of cos (first = 0) or sin (first = 1) at angle x, |x| <= pi/4
constexpr double dd_series(DD x, int first)
{
    const DD x2 = dd_mul(x, x);
    DD term = first ? x : DD{1.0, 0.0}, sum = term;
    for (int n = first + 1; n < 28; n += 2) {
        term = dd_div(dd_mul(term, x2), -(double)(n * (n + 1)));
        sum = dd_add(sum, term);
    }
    return sum.h;
}
constexpr DD TWO_PI = {6.283185307179586232, 2.449293598294706414e-16};
// cos(2 pi k / R) for quarter = 0, sin for quarter = 1
constexpr double trig(int k, int R, int quarter)
{
    // angle in units of 2 pi / (8 R): a = 8 k (cos), sin(t) = cos(t - pi/2)
    int a = (8 * k - (quarter ? 2 * R : 0)) % (8 * R);
    if (a < 0) a += 8 * R;
    if (a > 4 * R) a = 8 * R - a;                 // cos is even
    const bool neg = a > 2 * R;
    if (neg) a = 4 * R - a;                       // 0 <= a <= 2 R (a quarter turn)
    const bool co = a > R;                        // past an eighth: the sine of the rest
    const int m = co ? 2 * R - a : a;
    const double v = dd_series(dd_div(dd_mul(TWO_PI, DD{(double)m, 0.0}), 8.0 * R), co ? 1 : 0);
    return neg ? -v : v;
}
template <int K, int R> struct Root {
    static constexpr double c = trig(K, R, 0), s = trig(K, R, 1);
};

template <int N, typename F, int... I>
IBS_FFT_FN void unroll_seq(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
// f(integral_constant 0 .. N-1)
template <int N, typename F> IBS_FFT_FN void unroll(F &&f)
{
    unroll_seq<N>(f, std::make_integer_sequence<int, N>{});
}

// (re, im) *= e^{SIGN 2 pi i K/R}
template <int K, int R, int SIGN, typename T> IBS_FFT_FN void rotate(T &re, T &im)
{
    constexpr int k = ((K % R) + R) % R;
    if constexpr (k == 0) {
    } else if constexpr (2 * k == R) {
        re = -re;
        im = -im;
    } else if constexpr (4 * k == R || 4 * k == 3 * R) {
        const T t = re;
        if constexpr ((4 * k == R) == (SIGN > 0)) { re = -im; im = t; }
        else { re = im; im = -t; }
    } else {
        constexpr T c = (T)Root<k, R>::c, s = (T)(SIGN * Root<k, R>::s);
        const T t = re;
        re = c * t - s * im;
        im = s * t + c * im;
    }
}

constexpr int split_of(int R)   // factor taken out first; R itself: summed directly
{
    return R % 4 == 0 && R > 4 ? 4 : R % 2 == 0 && R > 2 ? 2 : R % 3 == 0 && R > 3 ? 3 : R % 5 == 0 && R > 5 ? 5 : R;
}

template <int R, int SIGN, typename T> IBS_FFT_FN void cdft(T (&re)[R], T (&im)[R])
{
    if constexpr (R == 1) {
    } else if constexpr (R == 2) {
        const T a = re[0], b = im[0];
        re[0] = a + re[1];
        im[0] = b + im[1];
        re[1] = a - re[1];
        im[1] = b - im[1];
    } else if constexpr (R == 4) {
        const T ar = re[0] + re[2], ai = im[0] + im[2], br = re[0] - re[2], bi = im[0] - im[2];
        const T cr = re[1] + re[3], ci = im[1] + im[3], dr = re[1] - re[3], di = im[1] - im[3];
        re[0] = ar + cr;
        im[0] = ai + ci;
        re[2] = ar - cr;
        im[2] = ai - ci;
        // SIGN i (dr + i di) = SIGN (-di + i dr)
        if constexpr (SIGN > 0) {
            re[1] = br - di; im[1] = bi + dr;
            re[3] = br + di; im[3] = bi - dr;
        } else {
            re[1] = br + di; im[1] = bi - dr;
            re[3] = br - di; im[3] = bi + dr;
        }
    } else if constexpr (split_of(R) == R) {
        static_assert(R % 2 == 1, "odd sizes only");
        constexpr int H = (R - 1) / 2;
        T ar[H], ai[H], br[H], bi[H];
#pragma unroll
        for (int j = 0; j < H; ++j) {
            ar[j] = re[j + 1] + re[R - 1 - j];
            ai[j] = im[j + 1] + im[R - 1 - j];
            br[j] = re[j + 1] - re[R - 1 - j];
            bi[j] = im[j + 1] - im[R - 1 - j];
        }
        const T r0 = re[0], i0 = im[0];
#pragma unroll
        for (int j = 0; j < H; ++j) {
            re[0] += ar[j];
            im[0] += ai[j];
        }
        unroll<H>([&](auto kk) {
            constexpr int k = decltype(kk)::value + 1;
            T pr = r0, pi = i0, qr = 0, qi = 0;   // q: the sine part, times SIGN i
            unroll<H>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                constexpr T c = (T)Root<(k * (j + 1)) % R, R>::c, s = (T)Root<(k * (j + 1)) % R, R>::s;
                pr += c * ar[j];
                pi += c * ai[j];
                qr += s * br[j];
                qi += s * bi[j];
            });
            if constexpr (SIGN > 0) {
                re[k] = pr - qi; im[k] = pi + qr;
                re[R - k] = pr + qi; im[R - k] = pi - qr;
            } else {
                re[k] = pr + qi; im[k] = pi - qr;
                re[R - k] = pr - qi; im[R - k] = pi + qr;
            }
        });
    } else {
        constexpr int P = split_of(R), Q = R / P;
        T sr[P][Q], si[P][Q];
        unroll<P>([&](auto pp) {
            constexpr int p = decltype(pp)::value;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                sr[p][q] = re[P * q + p];
                si[p][q] = im[P * q + p];
            }
            cdft<Q, SIGN, T>(sr[p], si[p]);
        });
        unroll<Q>([&](auto qq) {
            constexpr int q = decltype(qq)::value;
            T tr[P], ti[P];
            unroll<P>([&](auto pp) {
                constexpr int p = decltype(pp)::value;
                tr[p] = sr[p][q];
                ti[p] = si[p][q];
                rotate<p * q, R, SIGN>(tr[p], ti[p]);
            });
            cdft<P, SIGN, T>(tr, ti);
#pragma unroll
            for (int p = 0; p < P; ++p) {
                re[q + Q * p] = tr[p];
                im[q + Q * p] = ti[p];
            }
        });
    }
}

// real input; outputs k = 0 .. R/2 (R odd: 0 .. (R-1)/2); im[0] and, R even,
// im[R/2] are zero
template <int R, typename T>
IBS_FFT_FN void rdft(const T (&x)[R], T (&re)[R / 2 + 1], T (&im)[R / 2 + 1])
{
    if constexpr (R == 1) {
        re[0] = x[0];
        im[0] = 0;
    } else if constexpr (R == 2) {
        re[0] = x[0] + x[1];
        re[1] = x[0] - x[1];
        im[0] = im[1] = 0;
    } else if constexpr (R % 2 == 1) {
        constexpr int H = (R - 1) / 2;
        T a[H], b[H];
#pragma unroll
        for (int j = 0; j < H; ++j) {
            a[j] = x[j + 1] + x[R - 1 - j];
            b[j] = x[j + 1] - x[R - 1 - j];
        }
        re[0] = x[0];
        im[0] = 0;
#pragma unroll
        for (int j = 0; j < H; ++j) re[0] += a[j];
        unroll<H>([&](auto kk) {
            constexpr int k = decltype(kk)::value + 1;
            T p = x[0], q = 0;
            unroll<H>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                p += (T)Root<(k * (j + 1)) % R, R>::c * a[j];
                q += (T)Root<(k * (j + 1)) % R, R>::s * b[j];
            });
            re[k] = p;
            im[k] = -q;
        });
    } else {
        constexpr int Q = R / 2, H = Q / 2;
        T e[Q], o[Q], er[H + 1], ei[H + 1], tr[H + 1], ti[H + 1];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            e[q] = x[2 * q];
            o[q] = x[2 * q + 1];
        }
        rdft<Q, T>(e, er, ei);
        rdft<Q, T>(o, tr, ti);
        unroll<H + 1>([&](auto kk) {
            constexpr int k = decltype(kk)::value;
            if constexpr (2 * k == Q) {   // both halves real: X = E - i O
                re[k] = er[k];
                im[k] = -tr[k];
            } else if constexpr (k == 0) {
                re[0] = er[0] + tr[0];
                re[Q] = er[0] - tr[0];
                im[0] = im[Q] = 0;
            } else {
                T a = tr[k], b = ti[k];
                rotate<k, R, -1>(a, b);
                re[k] = er[k] + a;
                im[k] = ei[k] + b;
                re[Q - k] = er[k] - a;
                im[Q - k] = b - ei[k];
            }
        });
    }
}

// Hermitian input (im[0] and, R even, im[R/2] taken as zero), real output
template <int R, typename T>
IBS_FFT_FN void hdft(const T (&re)[R / 2 + 1], const T (&im)[R / 2 + 1], T (&x)[R])
{
    if constexpr (R == 1) {
        x[0] = re[0];
    } else if constexpr (R == 2) {
        x[0] = re[0] + re[1];
        x[1] = re[0] - re[1];
    } else if constexpr (R % 2 == 1) {
        constexpr int H = (R - 1) / 2;
        T a[H], b[H];
        x[0] = re[0];
#pragma unroll
        for (int j = 0; j < H; ++j) {
            a[j] = re[j + 1] + re[j + 1];
            b[j] = im[j + 1] + im[j + 1];
            x[0] += a[j];
        }
        unroll<H>([&](auto nn) {
            constexpr int n = decltype(nn)::value + 1;
            T p = re[0], q = 0;
            unroll<H>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                p += (T)Root<(n * (j + 1)) % R, R>::c * a[j];
                q += (T)Root<(n * (j + 1)) % R, R>::s * b[j];
            });
            x[n] = p - q;
            x[R - n] = p + q;
        });
    } else {
        constexpr int Q = R / 2, H = Q / 2;
        T er[H + 1], ei[H + 1], tr[H + 1], ti[H + 1], e[Q], o[Q];
        unroll<H + 1>([&](auto kk) {
            constexpr int k = decltype(kk)::value;
            if constexpr (k == 0) {
                er[0] = re[0] + re[Q];
                tr[0] = re[0] - re[Q];
                ei[0] = ti[0] = 0;
            } else if constexpr (2 * k == Q) {   // X_{Q/2} and its conjugate: E = 2 Re, O = -2 Im
                er[k] = re[k] + re[k];
                tr[k] = -(im[k] + im[k]);
                ei[k] = ti[k] = 0;
            } else {
                er[k] = re[k] + re[Q - k];
                ei[k] = im[k] - im[Q - k];
                tr[k] = re[k] - re[Q - k];
                ti[k] = im[k] + im[Q - k];
                rotate<k, R, 1>(tr[k], ti[k]);
            }
        });
        hdft<Q, T>(er, ei, e);
        hdft<Q, T>(tr, ti, o);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            x[2 * q] = e[q];
            x[2 * q + 1] = o[q];
        }
    }
}

}  // namespace fft
}  // namespace ibs
