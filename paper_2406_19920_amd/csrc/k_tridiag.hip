// Tridiagonal solves along y: launch-shape selection and the entry points
// (the kernel and its per-shape launcher are in tridiag.h; the cyclic
// shapes of the triply periodic branch are instantiated in
// k_tridiag_cyc.hip).
#include "tridiag.h"

namespace ibs {

template <typename T, typename R, typename Src>
static hipError_t launch_by_rows(const Src &src, int n, hipStream_t s)
{
    // chunks per pencil and rows per chunk: up to 16 chunks while the rows of
    // one fit the registers (64 rows: 8 x 8 takes 61 us for 63 fields of 64^3,
    // 16 x 4 70).  Beyond: FP32 more chunks of 16 rows; FP64 32 chunks,
    // whose 12 or fewer rows leave two 8-wave blocks per CU (384 rows of
    // 512x384x384: 733 us for three fields, 24 chunks of 16 rows 1069).
    if (n <= 32) return launch_pm<T, R, 8, 4>(src, s);
    if (n <= 64) return launch_pm<T, R, 8, 8>(src, s);
    if (n <= 96) return launch_pm<T, R, 16, 6>(src, s);
    if (n <= 128) return launch_pm<T, R, 16, 8>(src, s);
    if (n <= 160) return launch_pm<T, R, 16, 10>(src, s);
    if (n <= 192) return launch_pm<T, R, 16, 12>(src, s);
    if constexpr (sizeof(R) == 4) {
        // at most one tile per CU: nothing else hides a tile's own latency,
        // so shorter chunks
        if (n <= 256 && src.width() <= 256) return launch_pm<T, R, 32, 8>(src, s);
        if (n <= 256) return launch_pm<T, R, 16, 16>(src, s);
        if (n <= 320) return launch_pm<T, R, 20, 16>(src, s);
        if (n <= 384) return launch_pm<T, R, 24, 16>(src, s);
        if (n <= 512) return launch_pm<T, R, 32, 16>(src, s);
        if (n <= 768) return launch_pm<T, R, 32, 24>(src, s);
    } else {
        if (n <= 224) return launch_pm<T, R, 16, 14>(src, s);
        if (n <= 256) return launch_pm<T, R, 16, 16>(src, s);
        if (n <= 320) return launch_pm<T, R, 32, 10>(src, s);
        if (n <= 384) return launch_pm<T, R, 32, 12>(src, s);
        if (n <= 512) return launch_pm<T, R, 32, 16>(src, s);
        if (n <= 768) return launch_pm<T, R, 48, 16>(src, s);
    }
    return hipErrorInvalidValue;
}

// Upper bound on the condition number of every Helmholtz pencil matrix
// (1 - c s) I - c T_kind of the jobs: its eigenvalues lie in
// [1, 1 + c (max|s| + Gershgorin bound of -T)].
static double helmholtz_kappa(const JobSet &js, const Plan &p)
{
    double smax = 0.0;
    for (int xk = 0; xk < NUM_XK; ++xk)
        for (double v : p.lam_x[xk]) smax = std::max(smax, -v);
    double szmax = 0.0;
    for (int zk = 0; zk < NUM_XK; ++zk)
        for (double v : p.lam_z[zk]) szmax = std::max(szmax, -v);
    double kap = 1.0;
    for (int q = 0; q < js.n; ++q) {
        const int kd = js.j[q].kind;
        double g = 0.0;
        for (size_t j = 0; j < p.di[kd].size(); ++j)
            g = std::max(g, std::fabs(p.lo[kd][j]) + std::fabs(p.di[kd][j]) + std::fabs(p.up[kd][j]));
        kap = std::max(kap, 1.0 + std::fabs(js.j[q].c) * (smax + szmax + g));
    }
    return kap;
}

bool fp32_pencils(const JobSet &js, const Plan &p) { return helmholtz_kappa(js, p) <= FP32_KAPPA; }

// Launch shape by system size: padded partitions, or (periodic y) the
// cyclic shapes, which need the exact row count.
template <typename T, typename R>
static hipError_t launch_rows(const Plan &p, const JobSet &js, const TriParams &tp, int n, hipStream_t s)
{
    const TriSet src{js, tp};
    if (p.py) {
        if constexpr (sizeof(T) == 8) return launch_cyclic_dd(src, n, s);
        else if constexpr (sizeof(R) == 8) return launch_cyclic_fd(src, n, s);
        else return launch_cyclic_ff(src, n, s);
    }
    return launch_by_rows<T, R>(src, n, s);
}

// What every launch on a plan shares: its tables and sizes, no state.
static TriParams tri_params(const Plan &p, bool poisson)
{
    TriParams tp;
    for (int xk = 0; xk < NUM_XK; ++xk) tp.lam_x[xk] = blob_ptr(p, p.lay.lam_x[xk]);
    for (int zk = 0; zk < NUM_XK; ++zk) tp.lam_z[zk] = blob_ptr(p, p.lay.lam_z[zk]);
    for (int kd = 0; kd < NUM_KINDS; ++kd) {
        tp.lo[kd] = blob_ptr(p, p.lay.lo[kd]);
        tp.di[kd] = blob_ptr(p, p.lay.di[kd]);
        tp.up[kd] = blob_ptr(p, p.lay.up[kd]);
    }
    tp.wy = blob_ptr(p, p.lay.wy);
    tp.bmean = nullptr;
    tp.xsum = nullptr;
    tp.record_mean = 1;
    tp.skip = nullptr;
    tp.wsum_y = 0.0;
    for (int j = 0; j < p.ny; ++j) tp.wsum_y += p.dyc[j];
    tp.nx = p.nx;
    tp.nz = p.nz;
    tp.poisson = poisson ? 1 : 0;
    tp.nxsum = 0;
    tp.inv_sqrt_nxnz = 1.0 / std::sqrt((double)p.nx * (double)p.nz);
    tp.lane_mask = nullptr;
    tp.lane_list = nullptr;
    tp.lane_len = 0;
    tp.lane_mode = 0;
    tp.bmax = nullptr;
    tp.scale = nullptr;
    return tp;
}

template <typename T>
static hipError_t launch_tridiag(const JobSet &js, const Plan &p, const State &st, bool poisson, int pass,
                                 hipStream_t s)
{
    TriParams tp = tri_params(p, poisson);
    tp.bmean = st.bmean;
    tp.nxsum = residual_tiles(p);
    if (pass > 0) {
        tp.record_mean = 0;
        tp.xsum = st.xsum;
    }
    if (pass >= 2) tp.skip = st.done;
    // refined path (FP32 data): the first pass records the partial maxima
    // the residual scale is taken from; later passes steer in its units
    tp.bmax = (sizeof(T) == 4 && pass == 0) ? st.bmax : nullptr;
    tp.scale = (sizeof(T) == 4 && pass > 0) ? st.scale : nullptr;
    int n = 0;
    for (int q = 0; q < js.n; ++q) {
        const int rows = js.j[q].rows - skip_first_row(js.j[q].kind);   // system rows
        n = rows > n ? rows : n;
    }
    // FP32 arithmetic where its rounding is far below what refinement
    // removes anyway: FP32 data (refined path), Helmholtz, and pencil
    // condition numbers bounded by FP32_KAPPA.
    if constexpr (sizeof(T) == 4) {
        if (!poisson && fp32_pencils(js, p)) return launch_rows<T, float>(p, js, tp, n, s);
        // few tiles: FP64 arithmetic on all of them in one launch costs less
        // than the lane's launch on top of the FP32 one (us per pass, one
        // launch against both: 64^3 7 / 13, 128^3 15 / 17, 192x128x192 23 / 26,
        // 192x256x192 32 / 33, 256^3 49 / 42; side by side with other
        // work, where only the throughput counts, the larger ones do not gain)
        constexpr int ONE_LAUNCH_TILES = 4 * 256;   // 16-wide tiles, four per CU
        if (poisson && p.lane_len > 0 && p.nx / 16 * p.nz * js.n > ONE_LAUNCH_TILES) {
            // pressure pencils: FP32 arithmetic on every tile but the FP64
            // lane's, then FP64 arithmetic on the lane's tiles (disjoint
            // pencils; the lane holds the singular (0,0) pencil and every
            // pencil whose condition bound exceeds LANE64_KAPPA)
            tp.lane_mask = reinterpret_cast<const unsigned *>(blob_ptr(p, p.lay.lane_mask));
            tp.lane_list = reinterpret_cast<const int *>(blob_ptr(p, p.lay.lane_list));
            tp.lane_len = p.lane_len;
            tp.lane_mode = 1;
            hipError_t e = launch_rows<T, float>(p, js, tp, n, s);
            if (e != hipSuccess) return e;
            tp.lane_mode = 2;
            return launch_rows<T, double>(p, js, tp, n, s);
        }
    }
    return launch_rows<T, double>(p, js, tp, n, s);
}

size_t tri_entry_bytes() { return sizeof(TriEntry); }

void tri_entry_fill(void *to, const Plan &p, const FieldJob &job, bool poisson)
{
    TriEntry &e = *static_cast<TriEntry *>(to);
    e.job = job;
    e.tp = tri_params(p, poisson);
    e.tp.record_mean = 0;
}

hipError_t launch_tridiag_table(const void *entries, int n, int nx, int ny, int nz, hipStream_t s)
{
    return launch_by_rows<double, double>(TriTable{static_cast<const TriEntry *>(entries), n, nx, nz}, ny, s);
}

hipError_t launch_tridiag_f64(const JobSet &js, const Plan &p, const State &st, bool poisson, hipStream_t s)
{
    return launch_tridiag<double>(js, p, st, poisson, 0, s);
}

hipError_t launch_tridiag_f32(const JobSet &js, const Plan &p, const State &st, bool poisson, int pass,
                              hipStream_t s)
{
    return launch_tridiag<float>(js, p, st, poisson, pass, s);
}

}  // namespace ibs
