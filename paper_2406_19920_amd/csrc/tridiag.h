// Tridiagonal solves along y, one system per (x-mode a, z-mode c) pencil.
//
// After the x and z transforms every pencil is decoupled (Section 2.3.3,
// items S1.1 and S2.1; Appendix B gives the matrices on a uniform grid).
// Row j of pencil (a, c), with T the y part of the Laplacian (lo, di, up)
// and s = lambda_x[a] + lambda_z[c] (minus the transverse modified
// wavenumber squared, Appendix A):
//   Poisson   : lo_j x_{j-1} + (di_j + s) x_j + up_j x_{j+1} = b_j
//   Helmholtz : -c lo_j x_{j-1} + (1 - c s - c di_j) x_j - c up_j x_{j+1} = r_j
// The Neumann (0,0) pressure pencil is singular: its right-hand side is
// first made compatible (its volume-weighted mean removed), its first point
// is pinned to zero (as in Section 2.3.3, item S2.1) and the rest follows by
// summing fluxes, and after the solve the weighted mean is removed, which
// fixes the null mode at zero mean.
//
// Layout and parallel scheme (an MI355X design, not the paper's
// thread-per-pencil Thomas sweep): a block solves a tile of TA consecutive
// x-modes (one 128-byte line of a row) of one z-plane, all rows.  Each pencil
// is split into P chunks of M consecutive rows, one thread per chunk, lanes
// along the pencils: a thread reads its M rows straight into registers (whole
// lines per row, all loads in flight together) and writes them back from
// there; no staging.  It eliminates its chunk with two local sweeps (down and
// up), leaving one equation that couples the last unknowns of neighbouring
// chunks.  The reduced tridiagonal system of P equations per pencil goes
// through LDS to two lanes per pencil, which eliminate it from both ends,
// meet in the middle and substitute back (P/2 dependent steps; cyclic
// systems: with a second right-hand side for the unknown the ring is cut
// at); then every thread back-substitutes its interior.  Rows beyond the
// system size are identity rows.
//
// Bound by memory (each value read and written once) and, where few blocks
// fit a CU, by a tile's own latency.  Measured, us per launch, against lanes
// along the rows with the tile staged through LDS and the reduced system by
// parallel cyclic reduction: FP64 three 256^3 fields 200 (228), one 61 (77);
// 512x384x384 three fields 733 (912), 4.9 TB/s; 176x101x208 three 35 (50);
// FP32 arithmetic, three 256^3 fields 75 (122).
// The arithmetic is FP64, or FP32 for Helmholtz launches whose pencil
// condition numbers are provably small (refined path).
#pragma once
#include "ibs_internal.h"

#include <algorithm>
#include <cmath>

namespace ibs {

// 1/d from the hardware reciprocal estimate refined by two Newton steps
// (d is a normal, finite FP64 number here: diagonally dominant pivots).
static __device__ __forceinline__ double rcp64(double d)
{
    double x = __builtin_amdgcn_rcp(d);
    double e = fma(-d, x, 1.0);
    x = fma(x, e, x);
    e = fma(-d, x, 1.0);
    return fma(x, e, x);
}

// 1/d in the arithmetic type: FP64 as above; FP32 from the hardware
// estimate and one Newton step.
static __device__ __forceinline__ double rcpr(double d) { return rcp64(d); }
static __device__ __forceinline__ float rcpr(float d)
{
    const float x = __builtin_amdgcn_rcpf(d);
    return fmaf(x, fmaf(-d, x, 1.0f), x);
}

// Largest pencil condition number solved in FP32 arithmetic (refined path).
constexpr double FP32_KAPPA = 16.0;

struct TriParams {
    const double *lam_x[NUM_XK], *lam_z[NUM_XK];   // per x / z kind of the job
    const double *lo[NUM_KINDS], *di[NUM_KINDS], *up[NUM_KINDS];
    const double *wy;   // Delta_j: weights of the pressure unknowns
    double *bmean;      // per job: weighted mean removed from the rhs (Poisson)
    const double *xsum; // per job: nxsum partial sums of Delta_j x (stride XSUM_SLOTS), or null
    int nxsum;
    int record_mean;    // write bmean (first pass of a solve)
    const int *skip;    // per job: refinement already stopped (later passes), or null
    double wsum_y;      // sum of Delta_j
    int nx, nz;
    int poisson;
    double inv_sqrt_nxnz;
    // pressure pencils of the refined path: the plan lists the 32-wide
    // x-tiles (per z-mode) holding a pencil too ill-conditioned for FP32
    // arithmetic (the FP64 lane).  lane_mode 0: every tile; 1: every tile
    // but the FP64-lane ones (FP32 arithmetic); 2: only the FP64-lane tiles.
    const unsigned *lane_mask;   // per z-mode: bit t = x-tile [32t, 32t+32) is in the FP64 lane
    const int *lane_list;        // FP64-lane tiles as (c << 8) | t
    int lane_len;
    int lane_mode;
    // refined path: the first pass's launches record the largest magnitude of
    // their pencil data per 16-wide x-tile and z-mode (bmax_slots() per job;
    // the FP64 lane's tiles by its own launch), from which the refinement
    // passes take the power of two sigma that scales their FP32 residuals;
    // those passes then steer the mean in sigma units
    float *bmax;           // first pass: the maxima, or null
    const double *scale;   // later passes: per job sigma, or null (1)
};

// Where a launch takes its fields from: a few jobs of one plan by value, or a
// table in device memory (fields of many plans, all of one grid size).
struct TriSet {
    JobSet js;
    TriParams tp;
    __device__ __forceinline__ const FieldJob &job(int q) const { return js.j[q]; }
    __device__ __forceinline__ const TriParams &params(int) const { return tp; }
    int count() const { return js.n; }
    int tiles(int TA) const { return tp.lane_mode == 2 ? tp.lane_len * (32 / TA) : tp.nx / TA * tp.nz; }
    int width() const { return tp.nx / 32 * tp.nz * js.n; }
};
struct TriEntry {
    FieldJob job;
    TriParams tp;
};
struct TriTable {
    const TriEntry *e;
    int n, nx, nz;
    __device__ __forceinline__ const FieldJob &job(int q) const { return e[q].job; }
    __device__ __forceinline__ const TriParams &params(int q) const { return e[q].tp; }
    int count() const { return n; }
    int tiles(int TA) const { return nx / TA * nz; }
    int width() const { return nx / 32 * nz * n; }
};

// The singular pressure pencil, in LDS, by one wave: y holds n right-hand
// side values on entry and the solution on return.  The volume-weighted mean
// of the right-hand side is removed (and returned); the rest is solved by
// summing fluxes, not by elimination (which loses digits with the square of
// the row count on a singular matrix): the flux through the face above row j
// is F_j = sum_{i <= j} Delta_i (b_i - mean), and x rises by delta_{j+1} F_j
// across it (wt: Delta_j, dl: delta_{j+1} = 1/(up_j Delta_j); 0 past the last
// row of a walled system), from x_0 = 0; cyclic: plus the constant flux that
// closes the ring.  Then the weighted mean of x is removed, and steer with it
// (refinement: so that x + d has zero weighted mean, in this pencil's
// normalisation).
template <int NR, bool CYC>
static __device__ __forceinline__ double singular_pencil(double *y, int n, const double *wt, const double *dl,
                                                         double steer)
{
    constexpr int RL = (NR + 63) / 64;   // rows per lane
    const int lane = threadIdx.x, j0 = lane * RL, j1 = min(n, j0 + RL);
    auto total = [](double v) {
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
        return v;
    };
    auto below = [&](double v) {   // sum over the lanes below this one
        double t = v;
        for (int d = 1; d < 64; d <<= 1) {
            const double o = __shfl_up(t, d, 64);
            if (lane >= d) t += o;
        }
        return t - v;
    };
    double sv = 0.0, sw = 0.0;
#pragma unroll 1
    for (int j = j0; j < j1; ++j) {
        sv += wt[j] * y[j];
        sw += wt[j];
    }
    sw = total(sw);
    const double mean = total(sv) / sw;
    double f = 0.0, d = 0.0, ds = 0.0;
#pragma unroll 1
    for (int j = j0; j < j1; ++j) f += wt[j] * (y[j] - mean);
    f = below(f);
#pragma unroll 1
    for (int j = j0; j < j1; ++j) {
        f += wt[j] * (y[j] - mean);
        y[j] = dl[j] * f;
        d += y[j];
        ds += dl[j];
    }
    const double f0 = CYC ? -total(d) / total(ds) : 0.0;
    double x = below(d) + f0 * below(ds), sx = 0.0;
#pragma unroll 1
    for (int j = j0; j < j1; ++j) {
        const double rise = y[j] + (CYC ? f0 * dl[j] : 0.0);
        y[j] = x;
        sx += wt[j] * x;
        x += rise;
    }
    const double mx = total(sx) / sw + steer;
#pragma unroll 1
    for (int j = j0; j < j1; ++j) y[j] -= mx;
    return mean;
}

// T: storage type of the field (double, or float on the refined path);
// R: arithmetic type (double; float only for well-conditioned Helmholtz
// systems of the refined path, whose refinement absorbs FP32 rounding).
// CYC: cyclic systems (periodic y: row 0 couples to row n-1 and row n-1 to
// row 0 through the operator's corner coefficients lo[0], up[n-1]); the
// system then fills the P chunks exactly (n = P M, no padding rows) and the
// reduced system of the chunk ends is itself cyclic.
// BMX: this launch records the maxima (the refined path's first pass).
// Waves per SIMD the registers are held to: what the three per-chunk arrays
// leave room for (16 rows: a dozen values spill, and the third 8-wave block
// per CU in FP32, the fourth 4-wave one in FP64, pays for them: 75 instead of
// 87 us for three 256^3 FP32 fields).  16-wave blocks: one per CU.
template <typename R, int P, int M, int TA> constexpr int tri_waves()
{
    if (P * TA > 512 && sizeof(R) == 4) return M >= 16 && P * TA <= 768 ? 6 : 4;
    return sizeof(R) == 4 ? (M <= 8 ? 8 : M <= 12 ? 7 : 6) : (M <= 4 ? 8 : M <= 6 ? 6 : M <= 8 ? 5 : 4);
}
template <typename T, typename R, int P, int M, int TA, bool CYC = false, bool BMX = false, typename Src = TriSet>
__global__ __launch_bounds__((TA * P + 63) / 64 * 64, (tri_waves<R, P, M, TA>())) void tridiag_kernel(Src src)
{
    static_assert(P % 2 == 0 && M >= 2 && 64 % TA == 0, "two solver lanes per pencil in one wave");
    constexpr int NT = (TA * P + 63) / 64 * 64, NW = NT / 64;
    struct alignas(4 * sizeof(R)) Row { R a, b, c, m; };   // row without the pencil shift; m: 1 if it takes one
    __shared__ Row rows_sm[P * M];
    __shared__ R ex[3][P][TA];    // chunk tops (lam, mu, sig); later z
    __shared__ R eq[4][P][TA];    // reduced equations
    __shared__ double xs_sm[NW];        // per-wave sums of the x-sum partials
    // the singular pencil: right-hand side, then solution; weights Delta_j;
    // distances delta_{j+1}
    __shared__ double pin_sm[P * M], wt_sm[P * M], dl_sm[P * M];

    const int tid = threadIdx.x, job = blockIdx.y;
    const TriParams &tp = src.params(job);
    const int nx = tp.nx;
    if (tp.skip && tp.skip[job]) return;   // converged (later refinement passes)
    int c, a0;
    if (tp.lane_mode == 2) {
        constexpr int per = 32 / TA;
        const int e = tp.lane_list[blockIdx.x / per];
        c = e >> 8;
        a0 = (e & 0xff) * 32 + (blockIdx.x % per) * TA;
    } else {
        const int ntx = nx / TA;
        c = blockIdx.x / ntx;
        a0 = (blockIdx.x - c * ntx) * TA;
        // tiles left to the FP64 lane
        if (tp.lane_mode == 1 && ((tp.lane_mask[c] >> (a0 >> 5)) & 1u)) return;
    }
    const FieldJob &jb = src.job(job);
    // the v systems leave out the first wall row (kept at zero below)
    const int kind = jb.kind, sys0 = skip_first_row(kind), n = jb.rows - sys0;
    const bool walls = kind == KIND_F, pois = tp.poisson != 0;
    const int p = tid % TA, k = tid / TA, s = k * M;
    const bool act = k < P;
    T *x = reinterpret_cast<T *>(jb.out) + ((size_t)c * jb.rows + sys0) * nx + a0 + p;
    T raw[M];
    if (act) {
#pragma unroll
        for (int t = 0; t < M; ++t) raw[t] = x[(size_t)min(s + t, n - 1) * nx];
    }
    const R cj = (R)jb.c;
    const R sh = (R)(tp.lam_x[jb.xk][a0 + p] + tp.lam_z[jb.zk][c]);
    const R sadd = pois ? sh : -cj * sh;               // pencil shift of the diagonal
    const bool pt = pois && a0 == 0 && c == 0;         // block-uniform: the tile of the singular pencil
    const bool pinned = pt && p == 0;
    // rows of the job's operator without the pencil shift: Poisson (lo, di,
    // up); Helmholtz (-c lo, 1 - c di, -c up); identity beyond the system
    for (int j = tid; j < P * M; j += NT) {
        Row w = {R(0), R(1), R(0), R(0)};
        if (j < n) {
            const R lo = (R)tp.lo[kind][j + sys0], di = (R)tp.di[kind][j + sys0], up = (R)tp.up[kind][j + sys0];
            w = pois ? Row{lo, di, up, R(1)} : Row{-cj * lo, R(1) - cj * di, -cj * up, R(1)};
        }
        rows_sm[j] = w;
        if (pt) {
            wt_sm[j] = j < n ? tp.wy[j] : 0.0;
            dl_sm[j] = j < (CYC ? n : n - 1) ? 1.0 / (tp.up[kind][j] * tp.wy[j]) : 0.0;
        }
    }
    if (pt && tp.xsum) {
        // refinement passes: the residual's partial sums of Delta_j x, summed
        // by the whole block for the pinned pencil (fixed order: strided per
        // thread, a butterfly per wave, the waves in order)
        const double *xsp = tp.xsum + (size_t)job * XSUM_SLOTS;
        double part = 0.0;
        for (int q = tid; q < tp.nxsum; q += NT) part += xsp[q];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) part += __shfl_xor(part, d, 64);
        if ((tid & 63) == 0) xs_sm[tid >> 6] = part;
    }
    R r[M];
#pragma unroll
    for (int t = 0; t < M; ++t) r[t] = act && s + t < (walls ? n - 1 : n) ? (R)raw[t] : R(0);
    if constexpr (BMX) {
        float m = 0.f;
#pragma unroll
        for (int t = 0; t < M; ++t) m = fmaxf(m, fabsf((float)r[t]));
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
        __shared__ float mx_sm[NW];
        if ((tid & 63) == 0) mx_sm[tid >> 6] = m;
        __syncthreads();
        if (tid < TA / 16) {
#pragma unroll
            for (int w = 0; w < NW; ++w) m = fmaxf(m, mx_sm[w]);
            tp.bmax[((size_t)job * tp.nz + c) * (nx / 16) + a0 / 16 + tid] = m;
        }
    }
    __syncthreads();
    if (pinned && act)
#pragma unroll
        for (int t = 0; t < M; ++t) pin_sm[s + t] = (double)r[t];
    auto coef = [&](int t, R &A, R &B, R &C) {
        const Row w = rows_sm[(act ? s : 0) + t];
        A = w.a;
        B = w.b + w.m * sadd;
        C = w.c;
    };

    // down-sweep: rows s+1 .. s+M-1 in the form al x_s + x_j + ga x_{j+1} = rho
    R al[M], ga[M];
    {
        R A, B, C;
        coef(1, A, B, C);
        R inv = rcpr(B);
        al[1] = A * inv; ga[1] = C * inv; r[1] = r[1] * inv;
#pragma unroll
        for (int t = 2; t < M; ++t) {
            coef(t, A, B, C);
            inv = rcpr(B - A * ga[t - 1]);
            al[t] = -A * al[t - 1] * inv;
            ga[t] = C * inv;
            r[t] = (r[t] - A * r[t - 1]) * inv;
        }
    }
    // interior rows in terms of the chunk ends, x_j = bp + bq x_s + br x_e,
    // by back-substitution (no divisions), then the top row
    //   lam x_{s-1} + x_s + mu x_e = sig
    R lam_u, mu_u, sig_u;
    {
        R A, B, C;
        coef(0, A, B, C);
        if (pinned && k == 0) { A = 0.0; B = 1.0; C = 0.0; }
        if constexpr (M == 2) {
            const R inv = rcpr(B);
            lam_u = A * inv;
            mu_u = C * inv;
            sig_u = r[0] * inv;
        } else {
            R bp = r[M - 2], bq = -al[M - 2], br = -ga[M - 2];
#pragma unroll
            for (int t = M - 3; t >= 1; --t) {
                bp = r[t] - ga[t] * bp;
                bq = -al[t] - ga[t] * bq;
                br = -ga[t] * br;
            }
            const R inv = rcpr(B + C * bq);
            lam_u = A * inv;
            mu_u = C * br * inv;
            sig_u = (r[0] - C * bp) * inv;
        }
    }
    if (act) { ex[0][k][p] = lam_u; ex[1][k][p] = mu_u; ex[2][k][p] = sig_u; }
    __syncthreads();
    if (act) {
        // reduced system in z_k = x_{last row of chunk k}
        R lam1 = 0.0, mu1 = 0.0, sig1 = 0.0;
        const int kn = k + 1 < P ? k + 1 : 0;   // cyclic: chunk 0 follows chunk P-1
        if (CYC || k + 1 < P) { lam1 = ex[0][kn][p]; mu1 = ex[1][kn][p]; sig1 = ex[2][kn][p]; }
        const R ae = al[M - 1], ge = ga[M - 1], re = r[M - 1];
        eq[0][k][p] = -ae * lam_u;
        eq[1][k][p] = R(1) - ae * mu_u - ge * lam1;
        eq[2][k][p] = -ge * mu1;
        eq[3][k][p] = re - ae * sig_u - ge * sig1;
    }
    __syncthreads();
    if (tid < 2 * TA) {
        // two lanes per pencil: side 0 eliminates downwards from chunk 0, side
        // 1 upwards from the last; in: the coefficient towards the side's own
        // end, out: towards the middle.  z_i + cp_i z_{i+1} = dp_i (+ qp_i w)
        const int side = tid / TA, q = tid % TA;
        constexpr int LEN = CYC ? P - 1 : P;          // cyclic: cut at w = z_{P-1}
        constexpr int H0 = (LEN + 1) / 2, H1 = LEN / 2;
        const int cnt = side ? H1 : H0;
        auto at = [&](int i) { return side ? LEN - 1 - i : i; };
        R cp = 0.0, dp = 0.0, qp = 1.0;               // "z_{-1} = w"
#pragma unroll 2
        for (int i = 0; i < H0; ++i) {
            if (H0 != H1 && i >= cnt) break;
            const int e = at(i);
            const R in = eq[side ? 2 : 0][e][q], out = eq[side ? 0 : 2][e][q];
            const R inv = rcpr(eq[1][e][q] - in * cp);
            cp = out * inv;
            dp = (eq[3][e][q] - in * dp) * inv;
            eq[side ? 0 : 2][e][q] = cp;
            eq[3][e][q] = dp;
            if constexpr (CYC) {
                qp = -in * qp * inv;
                ex[1][e][q] = qp;
            }
        }
        if (P == 2 && CYC && side) { cp = 0.0; dp = 0.0; qp = 0.0; }
        const R cpo = __shfl_xor(cp, TA, 64), dpo = __shfl_xor(dp, TA, 64), qpo = __shfl_xor(qp, TA, 64);
        const R det = rcpr(R(1) - cp * cpo);
        R z = (dp - cp * dpo) * det, g = CYC ? (qp - cp * qpo) * det : R(0);
        if (cnt > 0) {
            ex[0][at(cnt - 1)][q] = z;
            if (CYC) ex[1][at(cnt - 1)][q] = g;
        }
#pragma unroll 4
        for (int ii = 0; ii < H0 - 1; ++ii) {
            const int i = cnt - 2 - ii;
            if (i < 0) break;
            const int e = at(i);
            const R ci = eq[side ? 0 : 2][e][q];
            z = eq[3][e][q] - ci * z;
            ex[0][e][q] = z;
            if constexpr (CYC) {
                g = ex[1][e][q] - ci * g;
                ex[1][e][q] = g;
            }
        }
        if constexpr (CYC) {
            // z, g now stand for the chunk next to the cut on this side (0 or
            // P-2); the last equation gives w
            const R zo = __shfl_xor(z, TA, 64), go = __shfl_xor(g, TA, 64);
            const R EA = eq[0][P - 1][q], EB = eq[1][P - 1][q], EC = eq[2][P - 1][q], ED = eq[3][P - 1][q];
            const R z0 = side ? zo : z, zl = side ? z : zo, g0 = side ? go : g, gl = side ? g : go;
            const R w = (ED - EA * zl - EC * z0) * rcpr(EB + EA * gl + EC * g0);
            for (int i = 0; i < cnt; ++i) {
                const int e = at(i);
                ex[0][e][q] += ex[1][e][q] * w;
            }
            if (side == 0) ex[0][P - 1][q] = w;
        }
    }
    __syncthreads();
    if (act) {
        const R z = ex[0][k][p];
        const R zm = k > 0 ? ex[0][k - 1][p] : (CYC ? ex[0][P - 1][p] : R(0));
        const R xs = sig_u - lam_u * zm - mu_u * z;
        // interior back-substitution, in place: r[t] becomes x[t]
        r[M - 1] = z;
#pragma unroll
        for (int t = M - 2; t >= 1; --t) r[t] = r[t] - al[t] * xs - ga[t] * r[t + 1];
        r[0] = xs;
    }
    double removed = 0.0;
    if (pt) {
        double xpart = 0.0;
        if (tp.xsum)
            for (int w = 0; w < NW; ++w) xpart += xs_sm[w];
        const double steer = (tp.scale ? tp.scale[job] : 1.0) * xpart * tp.inv_sqrt_nxnz / tp.wsum_y;
        if (tid < 64) removed = singular_pencil<P * M, CYC>(pin_sm, n, wt_sm, dl_sm, steer);
        __syncthreads();
        if (pinned && act)
#pragma unroll
            for (int t = 0; t < M; ++t) r[t] = (R)pin_sm[s + t];
    }
    if (act) {
#pragma unroll
        for (int t = 0; t < M; ++t)
            if (s + t < n) x[(size_t)(s + t) * nx] = (T)r[t];
        if (sys0 && k == 0) *(x - nx) = T(0);   // the left-out wall row holds zeros
    }
    if (tid == 0 && a0 == 0 && c == 0) {
        const double rm = removed * tp.inv_sqrt_nxnz;
        if (pois && tp.record_mean) tp.bmean[job] = rm;
        if (jb.info) {
            ibs_solve_info *inf = static_cast<ibs_solve_info *>(jb.info);
            inf->iters = 1;
            inf->status = IBS_OK;
            inf->rel_residual = 0.0;
            inf->rel_correction = 0.0;
            inf->removed_mean = pois ? rm : 0.0;
        }
    }
}

template <typename T, typename R, int P, int M, bool CYC, bool BMX, typename Src>
static hipError_t launch_pm_k(const Src &src, hipStream_t s)
{
    // pencils per tile: one 128-byte line of a row of FP64 data, or of FP32
    // data in FP32 arithmetic; FP32 data in FP64 arithmetic (the few tiles of
    // the FP64 lane) take 16, so that their registers hold two blocks per CU
    constexpr int TA = sizeof(R) == 8 ? 16 : 32;
    const int tiles = src.tiles(TA);
    if (tiles == 0) return hipSuccess;
    tridiag_kernel<T, R, P, M, TA, CYC, BMX, Src>
        <<<dim3(tiles, src.count()), dim3((TA * P + 63) / 64 * 64), 0, s>>>(src);
    return hipGetLastError();
}

template <typename T, typename R, int P, int M, bool CYC = false, typename Src>
static hipError_t launch_pm(const Src &src, hipStream_t s)
{
    if constexpr (sizeof(T) == 4)
        if (src.tp.bmax) return launch_pm_k<T, R, P, M, CYC, true>(src, s);
    return launch_pm_k<T, R, P, M, CYC, false>(src, s);
}

}  // namespace ibs

namespace ibs {
// Cyclic launches (periodic y), k_tridiag_cyc.hip: n must be one of the
// sizes cyclic_rows_supported() accepts (n = P M exactly).
hipError_t launch_cyclic_dd(const TriSet &src, int n, hipStream_t s);
hipError_t launch_cyclic_fd(const TriSet &src, int n, hipStream_t s);
hipError_t launch_cyclic_ff(const TriSet &src, int n, hipStream_t s);
}  // namespace ibs
