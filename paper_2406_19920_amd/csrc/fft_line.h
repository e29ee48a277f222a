// One line of a fast eigen-transform as work items (k_fft.h runs one item per
// thread; the arithmetic and the index maps here are shared with host checks).
#pragma once
#include "fft_core.h"

namespace ibs {
namespace fft {

// What an axis's transform is: the periodic Fourier basis, a basis of a walled
// axis on cell centres (cosine, sine), or the sine basis on its inner faces.
enum { AX_PERIODIC = 0, AX_CENTRES = 1, AX_FACES = 2 };

template <typename T> struct Cpx { T x, y; };

template <int R1, int R2> struct Shape {
    static constexpr int N = R1 * R2, H = N / 2, K1 = R1 / 2 + 1;   // K1 values of k1
    // stage A's items n2 (faces: one more), threads for the items of `lines`
    // lines, whole waves
    static constexpr int items(int ax) { return ax == AX_FACES ? R2 + 1 : R2; }
    static constexpr int threads(int ax, int lines)
    {
        return ((K1 > items(ax) ? K1 : items(ax)) * lines + 63) / 64 * 64;
    }
    static constexpr int LOW = (R2 + 1) / 2;                        // k2 < LOW: k <= N/2
    static_assert(R1 % 2 == 0, "stage A needs an even size");
};

// Slots of the coefficient pair (c, s) that X_kk, kk <= N/2, stands for.
// Periodic: c at kk, s at H + kk; kk = 0 and H have no sine
// and carry the basis's other normalisation.
// Walls: c at kk, s at N - kk (kk = 0 has no partner, kk = H is its own); the
// sine basis holds them in reverse order.
template <int N, bool WALL> IBS_FFT_FN int slot_c(int kk, bool sine) { return WALL && sine ? N - 1 - kk : kk; }
template <int N, bool WALL> IBS_FFT_FN int slot_s(int kk, bool sine)
{
    if (!WALL) return N / 2 + kk;
    return sine ? kk - 1 : N - kk;
}
constexpr double RSQRT2 = 0.70710678118654752440, SQRT2 = 1.41421356237309504880;

// X_kk -> (c, s); edge: kk = 0 or N/2
template <bool WALL, typename T>
IBS_FFT_FN void to_pair(T re, T im, int kk, bool edge, const Cpx<T> *rot, T &c, T &s)
{
    if constexpr (!WALL) {
        c = edge ? re * (T)RSQRT2 : re;
        s = -im;
    } else {
        const Cpx<T> w = rot[kk];   // (cos, -sin)
        c = w.x * re - w.y * im;
        s = -(w.x * im + w.y * re);
    }
}
template <bool WALL, typename T>
IBS_FFT_FN void from_pair(T c, T s, int kk, bool edge, const Cpx<T> *rot, T &re, T &im)
{
    if constexpr (!WALL) {
        re = edge ? c * (T)SQRT2 : c;
        im = edge ? (T)0 : -s;
    } else {
        const Cpx<T> w = rot[kk];   // (cos, +sin), kk = 0: (sqrt 2, 0); (c - i s) turned
        re = w.x * c + w.y * s;
        im = w.y * c - w.x * s;
    }
}

// Stage B's results of one work item (k1) to the line's coefficients:
// put(slot, value) for every coefficient the item owns.
template <int R1, int R2, bool WALL, typename T, typename F>
IBS_FFT_FN void emit(const T (&re)[R2], const T (&im)[R2], int k1, bool sine,
                                            const Cpx<T> *rot, F put)
{
    typedef Shape<R1, R2> S;
    const bool ends = k1 == 0 || 2 * k1 == R1;
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) {
        const int k = k1 + R1 * k2;
        T c, s;
        if (k2 < S::LOW) {
            const bool edge = k == 0 || k == S::H;
            to_pair<WALL, T>(re[k2], im[k2], k, edge, rot, c, s);
            put(slot_c<S::N, WALL>(k, sine), c);
            if (!edge) put(slot_s<S::N, WALL>(k, sine), s);
        } else {
            // conjugate partner N - k; k1 = 0 and R1/2 are their own partners
            const int kk = S::N - k;
            const bool mid = k1 == 0 && 2 * k2 == R2;   // k = N/2
            if (!ends || mid) {
                to_pair<WALL, T>(re[k2], -im[k2], kk, mid, rot, c, s);
                put(slot_c<S::N, WALL>(kk, sine), c);
                if (!mid) put(slot_s<S::N, WALL>(kk, sine), s);
            }
        }
    }
}
// The reverse: X_{k1 + R1 k2} of an item from the line's coefficients.
template <int R1, int R2, bool WALL, typename T, typename F>
IBS_FFT_FN void gather(T (&re)[R2], T (&im)[R2], int k1, bool sine, const Cpx<T> *rot, F get)
{
    typedef Shape<R1, R2> S;
    T c[R2], s[R2];
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) {   // all loads first
        const int k = k1 + R1 * k2, kk = k2 < S::LOW ? k : S::N - k;
        const bool edge = kk == 0 || kk == S::H;
        c[k2] = get(slot_c<S::N, WALL>(kk, sine));
        // an edge has no partner: any in-range slot, the value is not used
        // (walls, k = N/2: the pair is the coefficient itself twice)
        s[k2] = get(edge ? slot_c<S::N, WALL>(kk, sine) : slot_s<S::N, WALL>(kk, sine));
    }
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) {
        const int k = k1 + R1 * k2;
        const bool low = k2 < S::LOW;
        const int kk = low ? k : S::N - k;
        const bool edge = kk == 0 || kk == S::H;
        const T sv = WALL && kk == 0 ? (T)0 : s[k2];
        T a, b;
        from_pair<WALL, T>(c[k2], sv, kk, edge, rot, a, b);
        re[k2] = a;
        im[k2] = low ? b : -b;
    }
}

// line index of v_n, n = n2 + R2 n1: itself, or (walls) the even points up,
// then the odd points down
template <int R1, int R2, bool WALL> IBS_FFT_FN int line_index(int n2, int n1)
{
    const int n = n2 + R2 * n1;
    if (!WALL) return n;
    return 2 * n1 < R1 ? 2 * n : 2 * R1 * R2 - 1 - 2 * n;
}

// Sine basis on the inner faces 1 .. N-1 of a walled axis, its own inverse
// (slot 0, the wall face, counts as zero and becomes zero).  The line's odd
// extension e to length L = 2N = R1 (2 R2) has a purely imaginary spectrum,
// and stage A's results, twiddle included, are anti-Hermitian in n2: stage A
// runs for n2 = 0 .. R2 only and stage B is a Hermitian-to-real transform of
// length 2 R2, as much work as a periodic line of N.  Twiddle factors
// [k1][n2 <= R2] e^{-2 pi i k1 n2 / L} sqrt(2/N) / 2.
//
// e_n, n = n2 + 2 R2 n1, is the value of slot face_slot, negated for 2 n1 >=
// R1, times zero where face_wall (not left out: a NaN there stays one).
template <int R1> IBS_FFT_FN bool face_wall(int n2, int n1) { return n2 == 0 && (n1 == 0 || 2 * n1 == R1); }
template <int R1, int R2> IBS_FFT_FN int face_slot(int n2, int n1)
{
    const int n = n2 + 2 * R2 * n1;
    return face_wall<R1>(n2, n1) ? 0 : (2 * n1 < R1 ? n : 2 * R1 * R2 - n);
}
template <int R1, typename T> IBS_FFT_FN T face_value(T v, int n2, int n1)
{
    if (face_wall<R1>(n2, n1)) v *= (T)0;
    return 2 * n1 >= R1 ? -v : v;
}
// Stage B of item k1, re, im its R2 + 1 values: put(slot, value) for every
// coefficient the item owns.
template <int R1, int R2, typename T, typename F>
IBS_FFT_FN void face_emit(const T (&re)[R2 + 1], const T (&im)[R2 + 1], int k1, F put)
{
    T v[2 * R2];
    hdft<2 * R2, T>(im, re, v);   // anti-Hermitian: v the spectrum's imaginary part
    const bool ends = k1 == 0 || 2 * k1 == R1;
#pragma unroll
    for (int k2 = 0; k2 < 2 * R2; ++k2) {
        const int k = k1 + R1 * k2;
        if (k2 < R2) put(k, k ? -v[k2] : (T)0 * v[k2]);
        else if (!ends) put(2 * R1 * R2 - k, v[k2]);   // the odd partner
    }
}

}  // namespace fft
}  // namespace ibs
