// Fast eigen-transforms: x and z transforms of the separable solve (Section
// 2.3.3, items S1.1-S2.2; the paper's 2-D FFT) as two-stage fast Fourier
// transforms of real data, N = R1 R2 with R1 even, one pass over the field.
//
// Periodic axes (Appendix A's real Fourier basis).  With n = n2 + R2 n1 and
// k = k1 + R1 k2,
//   X_k = sum_{n2} e^{-2 pi i n2 k2/R2} e^{-2 pi i n2 k1/N}
//           [ sum_{n1} x_{n2 + R2 n1} e^{-2 pi i n1 k1/R1} ]:
// stage A, one thread per n2: the real R1-point transform in brackets (k1 =
// 0 .. R1/2 only: the rest are conjugates), times the twiddle factor; stage
// B, one thread per k1: the complex R2-point transform.  Between the stages
// the values cross threads through LDS.  The inverse runs B then A with the
// conjugate roots.  The basis's normalisation (sqrt(2/N)) is folded into the
// twiddle tables.  Spectral layout as for the dense transforms: index a <=
// N/2 the cosine modes, N/2 + k the sine mode k.
//
// Walls (uniform spacing).  The cosine basis of the pressure and the sine
// basis of the mirror-ghost components are the same transform of the
// reordered data v_n = x_{2n}, v_{N-1-n} = x_{2n+1} (the odd points negated
// for the sine basis), its result turned by e^{-i pi k/2N}: the real part is
// coefficient k, minus the imaginary part coefficient N - k (Makhoul, 1980);
// the sine coefficients come in reverse order.  The sine basis of the
// component on the axis's faces is the transform of the line's odd extension
// to 2N points, of which its symmetry leaves the work of N (fft_line.h).  As
// dense products those two launches each took 47-54 of a 160x128x160 duct
// step's 431 us; the step now takes 285 us, walls_x 256^3 refined 1920 -> 1717.
//
// Why this form: at 256 points it takes about 25 flops per value where the
// folded dense product takes 256, so the pass is bound by HBM (the dense
// FP64 transforms ran at 36 of 78.6 TFLOP/s and 2.2 of 5-7 TB/s).  Stage A's
// loads are R1 independent loads per thread and whole 128-byte lines, the
// tile is read completely before it is written (the transform may run in
// place), and about 39 KB of LDS per block leave four blocks per CU.
#pragma once
#include "fft_line.h"
#include "fft_sizes.h"
#include "ibs_internal.h"

namespace ibs {

// Arithmetic type of FP32 fields' transforms; EXACT: forward ones in FP64
// (fft_sizes.h).
template <int N, bool EXACT> struct FftReal {
    typedef typename std::conditional<(EXACT || N <= FFT_F64_ARITH_MAX), double, float>::type type;
};

struct FftJob {
    const void *in;
    void *out;        // spectrum; or (update and FP64 iterate modes) the iterate x
    const void *xs;   // MODE 4: the stored FP32 iterate
    double *x0;       // MODE 3: the FP64 field whose wall rows are zeroed too
    const void *tw;   // twiddle factors [k1][n2] (complex), normalisation included
    const void *rot;  // walls: e^{-+ i pi k/2N}, k = 0 .. N/2 (complex)
    int rows, skip;   // rows per plane; 1: the first row of a plane is left out
    int kind;         // XK_P / XK_C / XK_F (walls)
    int slot;         // job number in the call's state (flags, scale, partial sums)
};
struct FftSet {
    FftJob j[4];
    int n;
};

// The jobs of a launch as a table in device memory (any number of fields of
// one grid size).
struct FftTable {
    const FftJob *j;
    int n;
};

namespace fft {

static __device__ __forceinline__ double lanes_sum(double v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// The RW rows of a block to or from LDS lines (LR apart) by NT threads, 16
// bytes per lane and load.  In: every load is issued before the first value
// is stored to LDS (as one loop, each load waited for the one before: 221
// instead of 144 us for the inverse x transform of three 256^3 fields).
template <int NT, int RW, int N, int LR, typename TS, typename T>
static __device__ __forceinline__ void rows_in(const TS *in, const int *prow, T *lds)
{
    constexpr int V = 16 / sizeof(TS), CNT = RW * N / V, PER = (CNT + NT - 1) / NT;
    typedef TS vec __attribute__((ext_vector_type(V)));
    vec v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = (threadIdx.x + u * NT) * V;
        if (CNT % NT == 0 || i < RW * N) v[u] = *reinterpret_cast<const vec *>(in + (size_t)prow[i / N] * N + i % N);
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = (threadIdx.x + u * NT) * V;
        if (CNT % NT == 0 || i < RW * N) {
#pragma unroll
            for (int e = 0; e < V; ++e) lds[(i / N) * LR + i % N + e] = (T)v[u][e];
        }
    }
}
template <int NT, int RW, int N, int LR, typename T, typename TO>
static __device__ __forceinline__ void rows_out(const T *lds, const int *prow, TO *out)
{
    constexpr int V = 16 / sizeof(TO), CNT = RW * N / V, PER = (CNT + NT - 1) / NT;
    typedef TO vec __attribute__((ext_vector_type(V)));
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = (threadIdx.x + u * NT) * V;
        if (CNT % NT == 0 || i < RW * N) {
            vec v;
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = (TO)lds[(i / N) * LR + i % N + e];
            *reinterpret_cast<vec *>(out + (size_t)prow[i / N] * N + i % N) = v;
        }
    }
}

}  // namespace fft

// Columns of the z kernel's tile: 128 bytes of every plane; 64 for long FP32
// lines in FP64 arithmetic, whose exchange would leave two blocks per CU (256^3
// 37 us instead of 28).
template <typename TS, typename T, int N> constexpr int fft_cw()
{
    return sizeof(TS) == 4 && sizeof(T) == 8 && N > FFT_F64_ARITH_MAX ? 16 : 128 / (int)sizeof(TS);
}

// z transform of a tile of CW consecutive columns (128 bytes of every plane):
// lanes run along the columns, so every load and store is whole lines.
// Neighbouring tiles share DRAM pages, so each XCD (blocks are dealt to the 8
// of them in turn) takes a contiguous run of the columns, the runs started an
// eighth further in from XCD to XCD lest all meet in one channel.  Against
// tiles in turn: 384^3 FP64 2.75 -> 2.66 ms for three solves, 512x384x384
// 3.86 -> 3.73, refined 5.69 -> 5.46, 256^3 refined and FP64 equal.  FP64
// fields of a multiple of 256 rows take the tiles in turn (runs = 0); us for
// three solves, in turn / in runs: 512x256x256 1627 / 1661, 256x512x256 1609 /
// 1643, 128x256x512 723 / 730, 256^3 728 / 729 (v alone 221 / 228), but
// 400x256x400 2232 / 2204 and 128x512x384 1083 / 1064.  The pitch of a plane
// does not decide it: 512x128x384, its planes as long as 256 x 256 ones, takes
// 1153 / 1127.
// LDS [k1][n2][column], a pad line per k1 so that the two halves of a wave
// (k1 apart) use different banks.
// TS: stored type, T: arithmetic.
template <typename TS, typename T, int R1, int R2, bool INV, int AX, typename Set>
__global__ __launch_bounds__((fft::Shape<R1, R2>::threads(AX, fft_cw<TS, T, R1 * R2>()))) void fft_z_kernel(Set js, int nx, int runs,
                                                                                    const int *skip)
{
    using namespace fft;
    typedef Shape<R1, R2> S;
    constexpr bool WALL = AX == AX_CENTRES;
    constexpr int CW = fft_cw<TS, T, S::N>(), NA = S::items(AX), KZ = (NA | 1) * CW;
    __shared__ T sre[S::K1 * KZ], sim[S::K1 * KZ];
    const FftJob &jb = js.j[blockIdx.y];
    if (skip && skip[jb.slot]) return;
    const int Ncol = (jb.rows - jb.skip) * nx;
    const int xcd = blockIdx.x % 8, per = gridDim.x / 8;
    const int tile = runs ? xcd * per + (int)(blockIdx.x / 8 + per / 8 * xcd) % per : (int)blockIdx.x;
    if (tile * CW >= Ncol) return;   // whole block
    const int col = threadIdx.x % CW, item = threadIdx.x / CW;
    const size_t ldp = (size_t)jb.rows * nx;
    const size_t base = (size_t)jb.skip * nx + (size_t)tile * CW + col;
    const TS *in = static_cast<const TS *>(jb.in) + base;
    TS *out = static_cast<TS *>(jb.out) + base;
    const Cpx<T> *tw = static_cast<const Cpx<T> *>(jb.tw), *rot = static_cast<const Cpx<T> *>(jb.rot);
    const bool sine = jb.kind == XK_C;
    const T flip = WALL && sine ? (T)-1 : (T)1;
    if constexpr (AX == AX_FACES) {   // both directions
        if (item <= R2) {
            T x[R1], yr[S::K1], yi[S::K1];
#pragma unroll
            for (int n1 = 0; n1 < R1; ++n1) x[n1] = (T)in[(size_t)face_slot<R1, R2>(item, n1) * ldp];
#pragma unroll
            for (int n1 = 0; n1 < R1; ++n1) x[n1] = face_value<R1, T>(x[n1], item, n1);
            rdft<R1, T>(x, yr, yi);
#pragma unroll
            for (int k1 = 0; k1 < S::K1; ++k1) {
                const Cpx<T> w = tw[k1 * NA + item];
                const int o = k1 * KZ + item * CW + col;
                sre[o] = w.x * yr[k1] - w.y * yi[k1];
                sim[o] = w.x * yi[k1] + w.y * yr[k1];
            }
        }
        __syncthreads();
        if (item < S::K1) {
            T re[R2 + 1], im[R2 + 1];
#pragma unroll
            for (int n2 = 0; n2 <= R2; ++n2) {
                re[n2] = sre[item * KZ + n2 * CW + col];
                im[n2] = sim[item * KZ + n2 * CW + col];
            }
            face_emit<R1, R2, T>(re, im, item, [&](int a, T v) { out[(size_t)a * ldp] = (TS)v; });
        }
    } else if constexpr (!INV) {
        if (item < R2) {
            T x[R1], yr[S::K1], yi[S::K1];
#pragma unroll
            for (int n1 = 0; n1 < R1; ++n1) x[n1] = (T)in[(size_t)line_index<R1, R2, AX == AX_CENTRES>(item, n1) * ldp];
            if constexpr (WALL) {
#pragma unroll
                for (int n1 = R1 / 2; n1 < R1; ++n1) x[n1] *= flip;
            }
            rdft<R1, T>(x, yr, yi);
#pragma unroll
            for (int k1 = 0; k1 < S::K1; ++k1) {
                const Cpx<T> w = tw[k1 * R2 + item];
                const int o = k1 * KZ + item * CW + col;
                sre[o] = w.x * yr[k1] - w.y * yi[k1];
                sim[o] = w.x * yi[k1] + w.y * yr[k1];
            }
        }
        __syncthreads();
        if (item < S::K1) {
            T re[R2], im[R2];
#pragma unroll
            for (int n2 = 0; n2 < R2; ++n2) {
                re[n2] = sre[item * KZ + n2 * CW + col];
                im[n2] = sim[item * KZ + n2 * CW + col];
            }
            cdft<R2, -1, T>(re, im);
            emit<R1, R2, AX == AX_CENTRES, T>(re, im, item, sine, rot, [&](int a, T v) { out[(size_t)a * ldp] = (TS)v; });
        }
    } else {
        if (item < S::K1) {
            T re[R2], im[R2];
            gather<R1, R2, AX == AX_CENTRES, T>(re, im, item, sine, rot, [&](int a) { return (T)in[(size_t)a * ldp]; });
            cdft<R2, 1, T>(re, im);
#pragma unroll
            for (int n2 = 0; n2 < R2; ++n2) {
                const Cpx<T> w = tw[item * R2 + n2];
                sre[item * KZ + n2 * CW + col] = w.x * re[n2] - w.y * im[n2];
                sim[item * KZ + n2 * CW + col] = w.x * im[n2] + w.y * re[n2];
            }
        }
        __syncthreads();
        if (item < R2) {
            T x[R1], yr[S::K1], yi[S::K1];
#pragma unroll
            for (int k1 = 0; k1 < S::K1; ++k1) {
                yr[k1] = sre[k1 * KZ + item * CW + col];
                yi[k1] = sim[k1 * KZ + item * CW + col];
            }
            hdft<R1, T>(yr, yi, x);
#pragma unroll
            for (int n1 = 0; n1 < R1; ++n1) {
                const T v = WALL && 2 * n1 >= R1 ? flip * x[n1] : x[n1];
                out[(size_t)line_index<R1, R2, AX == AX_CENTRES>(item, n1) * ldp] = (TS)v;
            }
        }
    }
}

// x transform of RW rows.  Stage A's side is contiguous in global memory in
// runs of R2 values and goes straight to and from registers (walls: through
// LDS, the reordered points lying two apart); the spectral side goes through
// LDS rows so that global memory sees whole rows.
// MODE (INV): 0 out in TS; FP32 data: 1 x = result in FP64; 3 xs (out) =
// result in FP32; 2 x += result / sigma; 4 x = xs + result / sigma; 2 and 4
// also write the block's sums of (result / sigma)^2 and x^2 to red.  TIN:
// stored type of the forward input, TS of the spectrum, T: arithmetic.
template <typename TIN, typename TS, typename T, int R1, int R2, bool INV, int AX, int MODE, typename Set>
__global__ __launch_bounds__((fft::Shape<R1, R2>::threads(AX, FFT_RW))) void fft_x_kernel(Set js, int nz, double *red, int red_stride,
                                                                                 const int *skip, const double *scale)
{
    using namespace fft;
    typedef Shape<R1, R2> S;
    constexpr bool WALL = AX != AX_PERIODIC;   // the line goes through LDS on both sides
    constexpr int RW = FFT_RW, N = S::N, NT = S::threads(AX, RW), LR = N + 1;
    // LDS line of one row between the stages: odd strides against bank conflicts
    constexpr int NA = S::items(AX), KS = NA | 1, RS = (S::K1 * KS) | 1;
    constexpr int EX = RW * RS, RL = RW * LR;
    constexpr bool UPD = MODE == 2 || MODE == 4;
    typedef typename std::conditional<MODE == 1 || UPD, double, TS>::type Tout;
    __shared__ T sm[2 * EX > RL ? 2 * EX : RL];
    __shared__ int prow[RW];
    T *const sre = sm, *const sim = sm + EX;
    const FftJob &jb = js.j[blockIdx.y];
    if (skip && skip[jb.slot]) return;
    const int trows = jb.rows - jb.skip, M = nz * trows;
    const int row0 = blockIdx.x * RW;
    if (row0 >= M) return;   // whole block (M is a multiple of RW)
    const int tid = threadIdx.x;
    const bool sine = jb.kind == XK_C;
    const T flip = WALL && sine ? (T)-1 : (T)1;
    const Cpx<T> *tw = static_cast<const Cpx<T> *>(jb.tw), *rot = static_cast<const Cpx<T> *>(jb.rot);
    if (tid < RW) prow[tid] = (int)phys_row(row0 + tid, trows, jb.skip);
    // stage A: row ra, point n2; stage B: row rb, index k1
    const int ra = tid / NA, n2 = tid % NA;
    const int rb = tid % RW, k1b = tid / RW;
    const bool actA = tid < NA * RW, actB = k1b < S::K1;

    if constexpr (!INV && AX != AX_FACES) {
        const TIN *in = static_cast<const TIN *>(jb.in);
        T x[R1];
        if constexpr (WALL) {
            __syncthreads();
            rows_in<NT, RW, N, LR>(in, prow, sm);
            __syncthreads();
            if (actA) {
#pragma unroll
                for (int n1 = 0; n1 < R1; ++n1) {
                    const T v = sm[ra * LR + line_index<R1, R2, AX == AX_CENTRES>(n2, n1)];
                    x[n1] = 2 * n1 >= R1 ? flip * v : v;
                }
            }
            __syncthreads();
        } else if (actA) {
            const TIN *p = in + phys_row(row0 + ra, trows, jb.skip) * N + n2;
#pragma unroll
            for (int n1 = 0; n1 < R1; ++n1) x[n1] = (T)p[R2 * n1];
        }
        if (actA) {
            T yr[S::K1], yi[S::K1];
            rdft<R1, T>(x, yr, yi);
#pragma unroll
            for (int k1 = 0; k1 < S::K1; ++k1) {
                const Cpx<T> w = tw[k1 * R2 + n2];
                const int o = ra * RS + k1 * KS + n2;
                sre[o] = w.x * yr[k1] - w.y * yi[k1];
                sim[o] = w.x * yi[k1] + w.y * yr[k1];
            }
        }
        __syncthreads();
        T re[R2], im[R2];
        if (actB) {
#pragma unroll
            for (int q = 0; q < R2; ++q) {
                re[q] = sre[rb * RS + k1b * KS + q];
                im[q] = sim[rb * RS + k1b * KS + q];
            }
        }
        __syncthreads();
        if (actB) {
            cdft<R2, -1, T>(re, im);
            emit<R1, R2, AX == AX_CENTRES, T>(re, im, k1b, sine, rot, [&](int a, T v) { sm[rb * LR + a] = v; });
        }
        __syncthreads();
        rows_out<NT, RW, N, LR>(sm, prow, static_cast<TS *>(jb.out));
    } else {
        // the faces' forward transform is this one too, from TIN
        typedef typename std::conditional<INV, TS, TIN>::type Tsrc;
        const Tsrc *in = static_cast<const Tsrc *>(jb.in);
        Tout *out = static_cast<Tout *>(jb.out);
        T x[R1];
        __syncthreads();
        rows_in<NT, RW, N, LR>(in, prow, sm);
        __syncthreads();
        if constexpr (AX == AX_FACES) {
            if (actA) {
#pragma unroll
                for (int n1 = 0; n1 < R1; ++n1)
                    x[n1] = face_value<R1, T>(sm[ra * LR + face_slot<R1, R2>(n2, n1)], n2, n1);
            }
            __syncthreads();
            if (actA) {
                T yr[S::K1], yi[S::K1];
                rdft<R1, T>(x, yr, yi);
#pragma unroll
                for (int k1 = 0; k1 < S::K1; ++k1) {
                    const Cpx<T> w = tw[k1 * NA + n2];
                    const int o = ra * RS + k1 * KS + n2;
                    sre[o] = w.x * yr[k1] - w.y * yi[k1];
                    sim[o] = w.x * yi[k1] + w.y * yr[k1];
                }
            }
            __syncthreads();
            T re[NA], im[NA];
            if (actB) {
#pragma unroll
                for (int q = 0; q < NA; ++q) {
                    re[q] = sre[rb * RS + k1b * KS + q];
                    im[q] = sim[rb * RS + k1b * KS + q];
                }
            }
            __syncthreads();
            if (actB) face_emit<R1, R2, T>(re, im, k1b, [&](int a, T v) { sm[rb * LR + a] = v; });
        } else {
            T re[R2], im[R2];
            if (actB)
                gather<R1, R2, AX == AX_CENTRES, T>(re, im, k1b, sine, rot, [&](int a) { return sm[rb * LR + a]; });
            __syncthreads();
            if (actB) {
                cdft<R2, 1, T>(re, im);
#pragma unroll
                for (int q = 0; q < R2; ++q) {
                    const Cpx<T> w = tw[k1b * R2 + q];
                    const int o = rb * RS + k1b * KS + q;
                    sre[o] = w.x * re[q] - w.y * im[q];
                    sim[o] = w.x * im[q] + w.y * re[q];
                }
            }
        }
        // the iterate's old values of this thread's points, in flight under
        // the exchange
        typedef typename std::conditional<MODE == 4, float, double>::type Told;
        Told old[UPD ? R1 : 1];
        const size_t rowa = actA ? phys_row(row0 + ra, trows, jb.skip) * N : 0;
        if constexpr (UPD && !WALL) {
            const Told *xo = MODE == 4 ? static_cast<const Told *>(jb.xs) : static_cast<const Told *>(jb.out);
            if (actA) {
#pragma unroll
                for (int n1 = 0; n1 < R1; ++n1) old[n1] = xo[rowa + n2 + R2 * n1];
            }
        }
        if constexpr (AX != AX_FACES) {
            __syncthreads();
            if (actA) {
                T yr[S::K1], yi[S::K1];
#pragma unroll
                for (int k1 = 0; k1 < S::K1; ++k1) {
                    yr[k1] = sre[ra * RS + k1 * KS + n2];
                    yi[k1] = sim[ra * RS + k1 * KS + n2];
                }
                hdft<R1, T>(yr, yi, x);
            }
        }
        double sd = 0.0, sx = 0.0;
        const double isg = UPD && scale ? 1.0 / scale[jb.slot] : 1.0;
        if constexpr (WALL) {
            if constexpr (AX == AX_CENTRES) {
                __syncthreads();
                if (actA) {
#pragma unroll
                    for (int n1 = 0; n1 < R1; ++n1)
                        sm[ra * LR + line_index<R1, R2, true>(n2, n1)] = 2 * n1 >= R1 ? flip * x[n1] : x[n1];
                }
            }
            __syncthreads();
            if constexpr (UPD) {
                const Told *xo = MODE == 4 ? static_cast<const Told *>(jb.xs) : static_cast<const Told *>(jb.out);
                constexpr int PER = (RW * N + NT - 1) / NT, STEP = 8;   // old values: eight in flight at a time
#pragma unroll
                for (int u0 = 0; u0 < PER; u0 += STEP) {
                    Told o8[STEP];
#pragma unroll
                    for (int u = 0; u < STEP; ++u) {
                        const int i = tid + (u0 + u) * NT;
                        if (u0 + u < PER && i < RW * N) o8[u] = xo[(size_t)prow[i / N] * N + i % N];
                    }
#pragma unroll
                    for (int u = 0; u < STEP; ++u) {
                        const int i = tid + (u0 + u) * NT;
                        if (u0 + u < PER && i < RW * N) {
                            const double d = (double)sm[(i / N) * LR + i % N] * isg, xn = (double)o8[u] + d;
                            out[(size_t)prow[i / N] * N + i % N] = xn;
                            sd += d * d;
                            sx += xn * xn;
                        }
                    }
                }
            } else {
                rows_out<NT, RW, N, LR>(sm, prow, out);
            }
        } else if (actA) {
#pragma unroll
            for (int n1 = 0; n1 < R1; ++n1) {
                const size_t o = rowa + n2 + R2 * n1;
                if constexpr (UPD) {
                    const double d = (double)x[n1] * isg, xn = (double)old[n1] + d;
                    out[o] = xn;
                    sd += d * d;
                    sx += xn * xn;
                } else {
                    out[o] = (Tout)x[n1];
                }
            }
        }
        if constexpr (MODE == 1 || MODE == 3) {
            // the left-out wall row before a plane's first transform row
            // holds zeros in the result
            if (jb.skip)
                for (int r = 0; r < RW; ++r)
                    if ((row0 + r) % trows == 0)   // block-uniform
                        for (int i = tid; i < N; i += NT) {
                            const size_t o = (size_t)(prow[r] - 1) * N + i;
                            out[o] = 0;
                            if (MODE == 3) jb.x0[o] = 0.0;
                        }
        }
        if constexpr (UPD) {
            // block sums in a fixed order: butterflies, then the waves in turn
            constexpr int NW = NT / 64;
            __shared__ double ss[2][NW];
            sd = lanes_sum(sd);
            sx = lanes_sum(sx);
            if ((tid & 63) == 0) {
                ss[0][tid >> 6] = sd;
                ss[1][tid >> 6] = sx;
            }
            __syncthreads();
            if (tid == 0) {
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
}

// Grid and order of the z kernel's tiles (above); rows: transform rows, TS:
// stored type, cw: columns of a tile.
template <typename TS> inline int fft_z_tiles(int rows, int nx, int cw, int &runs)
{
    runs = sizeof(TS) == 4 || rows % 256 != 0;
    const int tiles = rows * nx / cw;
    return runs ? (tiles + 7) / 8 * 8 : tiles;
}

// One launch over the jobs of a set.  ax: form of their axis, the same for
// all jobs (AX_*); rows: transform rows per plane.  Sizes of the lists
// above only (fft_size()).
hipError_t launch_fft_z64(const FftTable &js, int n, int rows, int nx, bool inverse, int ax, hipStream_t s);
hipError_t launch_fft_x64(const FftTable &js, int n, int rows, int nz, bool inverse, int ax, hipStream_t s);
hipError_t launch_fft_z64(const FftSet &js, int n, int rows, int nx, bool inverse, int ax, hipStream_t s);
hipError_t launch_fft_z32(const FftSet &js, int n, int rows, int nx, bool inverse, int ax, bool exact,
                          const int *skip, hipStream_t s);
hipError_t launch_fft_x64(const FftSet &js, int n, int rows, int nz, bool inverse, int ax, hipStream_t s);
// mode as fft_x_kernel's; in64: the forward input is FP64; exact: FP64
// arithmetic
hipError_t launch_fft_x32_fwd(const FftSet &js, int n, int rows, int nz, int ax, bool exact, bool in64, const int *skip,
                              hipStream_t s);
hipError_t launch_fft_x32_inv(const FftSet &js, int n, int rows, int nz, int mode, double *red, int red_stride,
                              const int *skip, const double *scale, hipStream_t s);
hipError_t launch_fft_x32_wall(const FftSet &js, int n, int rows, int nz, int mode, double *red, int red_stride,
                               const int *skip, const double *scale, hipStream_t s);
hipError_t launch_fft_x32_face(const FftSet &js, int n, int rows, int nz, int mode, double *red, int red_stride,
                               const int *skip, const double *scale, hipStream_t s);

}  // namespace ibs
