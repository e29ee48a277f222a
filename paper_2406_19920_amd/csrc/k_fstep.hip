// Kernels of the Runge-Kutta sub-step around the linear solves (Section 2.1,
// eqs. a-e; kernels E1 and L1 of Section 2.3.2).
//
// explicit_kernel (E1): for every face of the three staggered grids,
//   u^e = u + dt [ (alpha+beta)/Re L u - (alpha+beta) G p
//                  - gamma N(u) - zeta N_prev ]                    (eq. a)
// together with the Helmholtz right-hand side without the forcing,
//   r = u^e - c L u,  c = beta dt / Re                             (eq. e)
// and N(u) itself (kept for the next stage's zeta term); u^e is written only
// when markers will interpolate it.  N is the
// convective term in divergence form, each product formed on the face or
// edge where its derivative needs it from arithmetic means of the
// neighbouring values; with walls, v = 0 on the wall faces and no product
// crosses them.  One thread per (i, j) of a block's tile, marching in z:
// the u and w faces of cell (i, j, k) and the v face j below it (rows
// 0..ny with walls: the wall faces get zeros); neighbours from an LDS ring
// of three planes.
//
// ibm_kernel (L1): 32 lanes per marker and component, 27 of them one point of
// the 3 x 3 x 3 support of the Roma three-point kernel on that component's
// grid: U^e(X) = sum u^e(x) w (eq. b), F = (U^d - U^e)/dt (eq. c), and
// r += dt F w dV / (hx hy hz) at each support point (eq. d, the spreading
// added straight into the Helmholtz right-hand side) by atomic adds, as
// the paper's L1 does.  Needs a uniform spacing in y (as the paper's grid).
#include "ibs_internal.h"

#include <algorithm>
#include <cmath>

namespace ibs {

struct FsGeo {
    int nx, ny, nz, py;
    double hx, hz, hy;           // hy: uniform y spacing (immersed boundary only)
    const double *dyc, *dyf;     // Delta_j [ny], delta_j [ny+1]
};

struct FsCoef {
    double ab;     // alpha + beta
    double gam, zet, dt, re, c;
};

// y rows of v: ny + 1 with walls, ny when periodic
static __device__ __forceinline__ int vrows(const FsGeo &g) { return g.py ? g.ny : g.ny + 1; }

// Tiling of the explicit kernel: a block owns ETX x ETY (x, y) points, one
// thread each, and marches through EKZ consecutive z planes.  The planes
// k-1, k, k+1 of u, v, w, p sit in LDS as a ring of three tiles with a
// one-point halo in x and y, so each plane of each field is read from HBM
// once per block (plus the halo, which the neighbouring tiles on the same
// XCD share in L2) instead of once per neighbour; the loads of plane k+2
// are in flight while plane k is computed.  Bound by HBM in 10 to 16 streams:
// 1.34 GB of a 256^3 stage in 316 us, with the previous N 1.75 GB in 368 us,
// with u^e for markers 1.75 GB in 377 us and both 2.15 GB in 437 us
// (368 was 430 with loads, stores and wall rows under branches, where every use
// waited for all loads in flight).  N is stored and read past the caches
// (non-temporal: the next use is a whole solve away), r is not.  With the
// waits for stores gone as well (loads a whole plane ahead of the ring's
// refill) it took as long.  (A four-slot ring with one
// barrier per plane needs 32 x 8 tiles to fit beside a second block and
// measured slower: three waves per SIMD instead of four.)
constexpr int ETX = 32, ETY = 16, ENT = ETX * ETY;
constexpr int EHX = ETX + 2, EHY = ETY + 2, EPL = EHX * EHY;
constexpr int EKZ = 16;                               // nz is a multiple of 16
constexpr int EPER = (4 * EPL + ENT - 1) / ENT;       // staged values per thread and plane

// UE: u^e is stored.
template <bool UE>
__global__ __launch_bounds__(ENT) void explicit_kernel(FsGeo g, FsCoef cf, const double *__restrict__ u,
                                                       const double *__restrict__ v,
                                                       const double *__restrict__ w,
                                                       const double *__restrict__ p,
                                                       const double *nu_prev, const double *nv_prev,
                                                       const double *nw_prev, double *ue, double *ve,
                                                       double *we, double *ru, double *rv, double *rw,
                                                       double *nu_out, double *nv_out, double *nw_out)
{
    __shared__ double sm[3][4 * EPL];   // ring slot, then field (u, v, w, p) x tile
    const int nx = g.nx, ny = g.ny, nz = g.nz, vr = vrows(g);
    // XCD-aware order: the hardware deals consecutive blocks to the 8 XCDs
    // in turn; block b takes tile (b % 8) * per + b / 8, so each XCD walks a
    // contiguous run of tiles (x fastest, then y, then z) and the halo lines
    // that neighbouring tiles share are fetched into its own L2 once
    const int gx = (nx + ETX - 1) / ETX, gy = (ny + ETY - 1) / ETY, ntile = gx * gy * (nz / EKZ);
    const int per = (ntile + 7) / 8;
    const int tile = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (tile >= ntile) return;   // whole block: before any barrier
    const int bx = tile % gx, by = (tile / gx) % gy, bz = tile / (gx * gy);
    const int tx = threadIdx.x % ETX, ty = threadIdx.x / ETX;
    const int i0 = bx * ETX, j0 = by * ETY, k0 = bz * EKZ;
    const int k1 = k0 + EKZ;
    const int i = i0 + tx, j = j0 + ty;

    // staging of one plane: this thread's EPER (field, tile point) values.
    // Points beyond a wall or the tile's overhang stage any value of the
    // plane: the formulas below never use them.  No load and no store of the
    // march sits in a branch: the compiler would then wait for all that are
    // in flight, not just for those it needs.
    const double *src[EPER];
    size_t pitch[EPER];   // of the field's planes
    bool wall[EPER];      // v on a wall face: staged as zero (the stored value is ignored)
#pragma unroll
    for (int e = 0; e < EPER; ++e) {
        const int idx = min((int)threadIdx.x + e * ENT, 4 * EPL - 1);
        const int f = idx / EPL, r = idx - f * EPL;
        const int hy = r / EHX, hx = r - hy * EHX;
        const int rows = f == 1 ? vr : ny;
        int gi = i0 - 1 + hx;
        gi = gi < 0 ? gi + nx : (gi >= nx ? min(gi - nx, nx - 1) : gi);
        int gj = j0 - 1 + hy;
        if (g.py) gj = gj < 0 ? gj + ny : (gj >= ny ? gj - ny : gj);
        wall[e] = f == 1 && !g.py && (gj <= 0 || gj >= ny);
        gj = min(max(gj, 0), rows - 1);
        src[e] = (f == 0 ? u : (f == 1 ? v : (f == 2 ? w : p))) + (size_t)gj * nx + gi;
        pitch[e] = (size_t)rows * nx;
    }
    double stg[EPER];
    auto fetch = [&](int kq) {
        const int kw = kq < 0 ? kq + nz : (kq >= nz ? kq - nz : kq);
#pragma unroll
        for (int e = 0; e < EPER; ++e) stg[e] = src[e][(size_t)kw * pitch[e]];
    };
    auto put = [&](int kq) {
        double *dst = sm[(kq - k0 + 1) % 3];
#pragma unroll
        for (int e = 0; e < EPER; ++e) {
            const int idx = threadIdx.x + e * ENT;
            if (idx < 4 * EPL) dst[idx] = wall[e] ? 0.0 : stg[e];
        }
    };
    // stores of a plane: offsets in the plane, out of range (dropped by the
    // bounds check) where a thread has nothing to store
    typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
    auto plane = [&](double *a, int k, int rows) {
        return __builtin_amdgcn_make_buffer_rsrc(a + (size_t)k * rows * nx, 0, (unsigned)(rows * nx * 8), 0x00027000);
    };
    auto store_nt = [&](double val, __amdgpu_buffer_rsrc_t to, unsigned at) {   // non-temporal
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, val), to, at, 0, 2);
    };
    auto store = [&](double val, __amdgpu_buffer_rsrc_t to, unsigned at) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, val), to, at, 0, 0);
    };
    constexpr unsigned NONE = 0xfffffff8u;

    const double ihx = 1.0 / g.hx, ihz = 1.0 / g.hz;
    const double vis = cf.ab / cf.re;
    const bool zprev = cf.zet != 0.0;

    // a thread keeps its (i, j) through the march: the y metric of its row
    // as reciprocals, once (cell rows: 1/Delta_j, 1/delta_j, 1/delta_{j+1},
    // and 2/Delta_j for the mirror-ghost flux; face rows: 1/delta_j and
    // 1/Delta of the cells above and below)
    const bool crow = i < nx && j < ny;
    const double iD = crow ? 1.0 / g.dyc[j] : 0.0;
    const double i2D = 2.0 * iD;
    const double idn = crow && (g.py || j + 1 < ny) ? 1.0 / g.dyf[j + 1] : 0.0;
    const double ids = crow && (g.py || j > 0) ? 1.0 / g.dyf[j] : 0.0;
    const bool frow = crow && (g.py || j > 0);
    const int jm = j > 0 ? j - 1 : ny - 1;   // the cell below a face (wraps when periodic)
    const double ifd = frow ? 1.0 / g.dyf[j] : 0.0;
    const double ifa = frow ? 1.0 / g.dyc[j] : 0.0;
    const double ifb = frow ? 1.0 / g.dyc[jm] : 0.0;

    const int oc = min(j, ny - 1) * nx + min(i, nx - 1);   // the thread's point in a plane, within the field
    const unsigned os = crow ? 8u * (unsigned)(j * nx + i) : NONE;
    const unsigned ow = crow && !g.py && j == ny - 1 ? 8u * (unsigned)(ny * nx + i) : NONE;   // the upper wall face
    fetch(k0 - 1);
    put(k0 - 1);
    fetch(k0);
    put(k0);
    fetch(k0 + 1);
    for (int k = k0; k < k1; ++k) {
        put(k + 1);   // into the slot of plane k-2
        // N_prev of this plane: before plane k+2's loads, which would
        // otherwise have to arrive first
        double pu = 0.0, pv = 0.0, pw = 0.0;
        if (zprev) {
            pu = __builtin_nontemporal_load(&nu_prev[(size_t)k * ny * nx + oc]);
            pw = __builtin_nontemporal_load(&nw_prev[(size_t)k * ny * nx + oc]);
            pv = __builtin_nontemporal_load(&nv_prev[(size_t)k * vr * nx + oc]);
        }
        __syncthreads();
        fetch(min(k + 2, k1));   // the last one is not used
        // field f at plane k + dk, row j + dj, column i + di (tile offsets)
        auto L = [&](int f, int dk, int dj, int di) {
            return sm[(k - k0 + 1 + dk) % 3][f * EPL + (ty + 1 + dj) * EHX + (tx + 1 + di)];
        };
        auto V = [&](int dk, int dj, int di) { return L(1, dk, dj, di); };
        {
            const bool hn = g.py || j + 1 < ny;   // a cell row above (else the wall)
            const bool hs = g.py || j > 0;        // a cell row below
            // y part of the Laplacian of a cell-height field at row j
            // (mirror ghost at a wall; fluxes over delta, delta_0 = delta_ny
            // across the periodic wrap)
            auto lapy = [&](int f) {
                const double fc = L(f, 0, 0, 0);
                const double in_u = (L(f, 0, 1, 0) - fc) * idn, in_l = (fc - L(f, 0, -1, 0)) * ids;
                const double fu = hn ? in_u : -fc * i2D;
                const double fl = hs ? in_l : fc * i2D;
                return (fu - fl) * iD;
            };
            // ---- u at x-face (i, j, k)
            {
                const double uc = L(0, 0, 0, 0);
                const double lap = (L(0, 0, 0, 1) - 2.0 * uc + L(0, 0, 0, -1)) * ihx * ihx +
                                   (L(0, 1, 0, 0) - 2.0 * uc + L(0, -1, 0, 0)) * ihz * ihz + lapy(0);
                const double gp = (L(3, 0, 0, 0) - L(3, 0, 0, -1)) * ihx;
                const double c1 = 0.5 * (uc + L(0, 0, 0, 1)), c0 = 0.5 * (L(0, 0, 0, -1) + uc);
                const double dxx = (c1 * c1 - c0 * c0) * ihx;
                // y fluxes v u on the faces j (below) and j+1 (above) at x-face i
                const double fb = 0.5 * (V(0, 0, 0) + V(0, 0, -1)) * 0.5 * (L(0, 0, -1, 0) + uc);
                const double ft = 0.5 * (V(0, 1, 0) + V(0, 1, -1)) * 0.5 * (uc + L(0, 0, 1, 0));
                const double dyy = ((hn ? ft : 0.0) - (hs ? fb : 0.0)) * iD;
                const double zb = 0.5 * (L(2, 0, 0, 0) + L(2, 0, 0, -1)) * 0.5 * (L(0, -1, 0, 0) + uc);
                const double zt = 0.5 * (L(2, 1, 0, 0) + L(2, 1, 0, -1)) * 0.5 * (uc + L(0, 1, 0, 0));
                const double N = dxx + dyy + (zt - zb) * ihz;
                double e = uc + cf.dt * (vis * lap - cf.ab * gp - cf.gam * N);
                if (zprev) e -= cf.dt * cf.zet * pu;
                if constexpr (UE) store(e, plane(ue, k, ny), os);
                store(e - cf.c * lap, plane(ru, k, ny), os);
                store_nt(N, plane(nu_out, k, ny), os);
            }
            // ---- w at z-face (i, j, k): the x <-> z mirror of u
            {
                const double wc = L(2, 0, 0, 0);
                const double lap = (L(2, 0, 0, 1) - 2.0 * wc + L(2, 0, 0, -1)) * ihx * ihx +
                                   (L(2, 1, 0, 0) - 2.0 * wc + L(2, -1, 0, 0)) * ihz * ihz + lapy(2);
                const double gp = (L(3, 0, 0, 0) - L(3, -1, 0, 0)) * ihz;
                const double c1 = 0.5 * (wc + L(2, 1, 0, 0)), c0 = 0.5 * (L(2, -1, 0, 0) + wc);
                const double dzz = (c1 * c1 - c0 * c0) * ihz;
                const double fb = 0.5 * (V(0, 0, 0) + V(-1, 0, 0)) * 0.5 * (L(2, 0, -1, 0) + wc);
                const double ft = 0.5 * (V(0, 1, 0) + V(-1, 1, 0)) * 0.5 * (wc + L(2, 0, 1, 0));
                const double dyy = ((hn ? ft : 0.0) - (hs ? fb : 0.0)) * iD;
                const double xb = 0.5 * (L(0, 0, 0, 0) + L(0, -1, 0, 0)) * 0.5 * (L(2, 0, 0, -1) + wc);
                const double xt = 0.5 * (L(0, 0, 0, 1) + L(0, -1, 0, 1)) * 0.5 * (wc + L(2, 0, 0, 1));
                const double N = (xt - xb) * ihx + dyy + dzz;
                double e = wc + cf.dt * (vis * lap - cf.ab * gp - cf.gam * N);
                if (zprev) e -= cf.dt * cf.zet * pw;
                if constexpr (UE) store(e, plane(we, k, ny), os);
                store(e - cf.c * lap, plane(rw, k, ny), os);
                store_nt(N, plane(nw_out, k, ny), os);
            }
        }
        // ---- v at y-face (i, j, k), zero on the walls; the last row's thread
        // has the upper one too
        {
            const bool in = g.py || j > 0;
            const double vc = V(0, 0, 0);
            const double lapy = ((V(0, 1, 0) - vc) * ifa - (vc - V(0, -1, 0)) * ifb) * ifd;
            const double lap = (V(0, 0, 1) - 2.0 * vc + V(0, 0, -1)) * ihx * ihx +
                               (V(1, 0, 0) - 2.0 * vc + V(-1, 0, 0)) * ihz * ihz + lapy;
            const double gp = (L(3, 0, 0, 0) - L(3, 0, -1, 0)) * ifd;
            const double c1 = 0.5 * (vc + V(0, 1, 0)), c0 = 0.5 * (V(0, -1, 0) + vc);
            const double dyy = (c1 * c1 - c0 * c0) * ifd;
            // x fluxes u v on the x-faces i and i+1 at y-face j
            const double xb = 0.5 * (L(0, 0, -1, 0) + L(0, 0, 0, 0)) * 0.5 * (vc + V(0, 0, -1));
            const double xt = 0.5 * (L(0, 0, -1, 1) + L(0, 0, 0, 1)) * 0.5 * (V(0, 0, 1) + vc);
            const double zb = 0.5 * (L(2, 0, -1, 0) + L(2, 0, 0, 0)) * 0.5 * (vc + V(-1, 0, 0));
            const double zt = 0.5 * (L(2, 1, -1, 0) + L(2, 1, 0, 0)) * 0.5 * (V(1, 0, 0) + vc);
            const double N = (xt - xb) * ihx + dyy + (zt - zb) * ihz;
            double e = vc + cf.dt * (vis * lap - cf.ab * gp - cf.gam * N);
            if (zprev) e -= cf.dt * cf.zet * pv;
            if constexpr (UE) {
                store(in ? e : 0.0, plane(ve, k, vr), os);
                store(0.0, plane(ve, k, vr), ow);
            }
            store(in ? e - cf.c * lap : 0.0, plane(rv, k, vr), os);
            store_nt(in ? N : 0.0, plane(nv_out, k, vr), os);
            store(0.0, plane(rv, k, vr), ow);
            store(0.0, plane(nv_out, k, vr), ow);
        }
        __syncthreads();   // the slot of plane k-1 is refilled next
    }
}

// Roma, Peskin and Berger's three-point regularised delta, grid units.
static __device__ __forceinline__ double roma3(double r)
{
    const double a = fabs(r);
    if (a <= 0.5) return (1.0 + sqrt(1.0 - 3.0 * a * a)) / 3.0;
    if (a <= 1.5) {
        const double t = 1.0 - a;
        return (5.0 - 3.0 * a - sqrt(fmax(0.0, 1.0 - 3.0 * t * t))) / 6.0;
    }
    return 0.0;
}

// The lanes of a marker share the three axes' divisions and weights: 35 us for
// 18 529 markers in 256^3 (one thread per marker: 76 us), bound by scattered
// accesses.  u^e is read as a field.  Recovering it at the support points from
// r + c L u would save the explicit kernel 62 to 69 us of stores, but loses
// up to c |L| roundings to the cancellation.
struct IbmFields {
    const double *ue[3];
    double *r[3];
};
constexpr int IBM_LANES = 32;
__global__ __launch_bounds__(256) void ibm_kernel(FsGeo g, double dt, int nm, const double *__restrict__ X,
                                                  const double *__restrict__ ud,
                                                  const double *__restrict__ dvol, IbmFields fd, double *force)
{
    const double vol = g.hx * g.hy * g.hz;
    const int lane = threadIdx.x % IBM_LANES;
    const int a = lane / 9, b = lane / 3 % 3, c = lane % 3;
    const int comp = blockIdx.y;
    const long groups = (long)gridDim.x * (256 / IBM_LANES);
    for (long m = (long)blockIdx.x * (256 / IBM_LANES) + threadIdx.x / IBM_LANES; m < nm; m += groups) {
        const int rows = comp == 1 ? vrows(g) : g.ny;
        // one axis's weight and index per lane, lanes 0-8 the x, y, z ones;
        // grid units, staggered by half a cell except along the component
        const int ax = lane / 3 % 3;
        const double at = X[3 * m + ax] / (ax == 0 ? g.hx : (ax == 1 ? g.hy : g.hz)) - (ax == comp ? 0.0 : 0.5);
        const int first = (int)floor(at + 0.5) - 1, pt = first + lane % 3;
        const int n = ax == 0 ? g.nx : (ax == 1 ? g.ny : g.nz);
        const double wt = roma3(pt - at);
        const int it = ax == 1 && !g.py ? pt : (pt % n + n) % n;
        const double w = __shfl(wt, 6 + a, IBM_LANES) * __shfl(wt, 3 + b, IBM_LANES) * __shfl(wt, c, IBM_LANES);
        const int ix = __shfl(it, c, IBM_LANES), iy = __shfl(it, 3 + b, IBM_LANES), iz = __shfl(it, 6 + a, IBM_LANES);
        const bool on = lane < 27 && iy >= 0 && iy < rows;
        const size_t o = ((size_t)iz * rows + iy) * g.nx + ix;
        double U = on ? fd.ue[comp][o] * w : 0.0;
#pragma unroll
        for (int d = IBM_LANES / 2; d >= 1; d >>= 1) U += __shfl_xor(U, d, IBM_LANES);
        const double F = (ud[3 * m + comp] - U) / dt;
        if (force && lane == 0) force[3 * m + comp] = F;
        if (on) atomicAdd(&fd.r[comp][o], F * w * (dt * dvol[m] / vol));
    }
}

static FsGeo fs_geo(const Plan &p)
{
    FsGeo g;
    g.nx = p.nx; g.ny = p.ny; g.nz = p.nz; g.py = p.py ? 1 : 0;
    g.hx = p.hx; g.hz = p.hz; g.hy = p.desc.ly / p.ny;
    g.dyc = blob_ptr(p, p.lay.dyc);
    g.dyf = blob_ptr(p, p.lay.dyf);
    return g;
}

hipError_t launch_explicit(const Plan &p, const FsStage &s, hipStream_t st)
{
    FsGeo g = fs_geo(p);
    FsCoef cf;
    cf.ab = s.alpha + s.beta;
    cf.gam = s.gamma;
    cf.zet = s.zeta;
    cf.dt = s.dt;
    cf.re = s.re;
    cf.c = s.beta * s.dt / s.re;
    const int ntile = ((p.nx + ETX - 1) / ETX) * ((p.ny + ETY - 1) / ETY) * (p.nz / EKZ);
    dim3 grid(8 * ((ntile + 7) / 8));   // a whole number of blocks per XCD
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(ENT), 0, st, g, cf, s.u, s.v, s.w, s.p, s.nu, s.nv, s.nw,
                           s.ue, s.ve, s.we, s.ru, s.rv, s.rw, s.nu, s.nv, s.nw);
    };
    s.nmarkers > 0 ? go(explicit_kernel<true>) : go(explicit_kernel<false>);
    return hipGetLastError();
}

hipError_t launch_ibm(const Plan &p, const FsStage &s, hipStream_t st)
{
    if (s.nmarkers <= 0) return hipSuccess;
    const FsGeo g = fs_geo(p);
    const IbmFields f{{s.ue, s.ve, s.we}, {s.ru, s.rv, s.rw}};
    constexpr int PER = 256 / IBM_LANES, MOST = 1 << 20;   // groups of lanes per block, blocks
    const dim3 grid(std::min(MOST, s.nmarkers / PER + (s.nmarkers % PER != 0)), 3), blk(256);
    hipLaunchKernelGGL(ibm_kernel, grid, blk, 0, st, g, s.dt, s.nmarkers, s.markers, s.ud, s.dvol, f, s.force);
    return hipGetLastError();
}

}  // namespace ibs
