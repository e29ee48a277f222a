// Launches of the fused x-z transforms (k_plane.h).
#include <algorithm>

#include "k_plane.h"

namespace ibs {

template <typename TIN, typename TS, bool INV, int MODE, typename Set>
static hipError_t go(const Set &js, const int nx, int ny, int nz, hipStream_t s, double *red = nullptr,
                     int red_stride = 0, const int *skip = nullptr, const double *scale = nullptr)
{
    auto run = [&](auto kernel, int threads) {
        kernel<<<dim3(ny, js.n), dim3(threads), 0, s>>>(js, nx, nz, red, red_stride, skip, scale);
    };
#define IBS_RUN(MAXN, L) run(plane_kernel<TIN, TS, INV, MODE, MAXN, L, Set>, PlaneShape<MAXN, L>::NT)
    const int side = std::max(nx, nz);
    // 64 lines at a time where the planes fill the chip at most a few times and
    // a plane's own time counts (64^3 FP64 Poisson 19.7 us, 32 lines 23.8; three
    // 64x512x64 Helmholtz 82.6 / 84.1); where they queue, smaller blocks
    // overlap better (96 small grids as chains 585 / 557)
    const bool wide = (size_t)ny * js.n <= 8 * 256;
    if (side <= 32) IBS_RUN(32, 32);
    else if (side <= 48) wide ? IBS_RUN(48, 64) : IBS_RUN(48, 32);
    else wide ? IBS_RUN(64, 64) : IBS_RUN(64, 32);
#undef IBS_RUN
    return hipGetLastError();
}

static PlaneJob plane_job(const Plan &p, bool inverse, int rows, int kind, int slot)
{
    PlaneJob j{};
    j.twx = blob_ptr(p, inverse ? p.lay.ftx_inv : p.lay.ftx_fwd);
    j.twz = blob_ptr(p, inverse ? p.lay.ftz_inv : p.lay.ftz_fwd);
    j.rows = rows;
    j.skip = skip_first_row(kind);
    j.slot = slot;
    return j;
}

hipError_t launch_plane_f64(const JobSet &js, const Plan &p, bool inverse, hipStream_t s)
{
    PlaneSet f{};
    f.n = js.n;
    for (int q = 0; q < js.n; ++q) {
        f.j[q] = plane_job(p, inverse, js.j[q].rows, js.j[q].kind, q);
        f.j[q].in = js.j[q].in;
        f.j[q].out = js.j[q].out;
    }
    return inverse ? go<double, double, true, 0>(f, p.nx, p.ny, p.nz, s) : go<double, double, false, 0>(f, p.nx, p.ny, p.nz, s);
}

size_t plane_entry_bytes() { return sizeof(PlaneJob); }

void plane_entry_fill(void *to, const Plan &p, const FieldJob &job, bool inverse)
{
    PlaneJob &j = *static_cast<PlaneJob *>(to);
    j = plane_job(p, inverse, job.rows, job.kind, 0);
    j.in = job.in;
    j.out = job.out;
}

hipError_t launch_plane_table(const void *entries, int n, int nx, int ny, int nz, bool inverse, hipStream_t s)
{
    const PlaneTable t{static_cast<const PlaneJob *>(entries), n};
    return inverse ? go<double, double, true, 0>(t, nx, ny, nz, s) : go<double, double, false, 0>(t, nx, ny, nz, s);
}

hipError_t launch_plane_f32(const SplitSet &ss, const Plan &p, const State &st, bool inverse, bool in64, int mode,
                            int pass, hipStream_t s)
{
    const int *skip = pass >= 2 ? st.done : nullptr;
    PlaneSet f{};
    f.n = ss.n;
    for (int q = 0; q < ss.n; ++q) {
        const SplitJob &j = ss.j[q];
        f.j[q] = plane_job(p, inverse, j.rows, j.kind, j.slot);
        f.j[q].in = j.in;
        f.j[q].out = !inverse ? static_cast<void *>(j.out) : (mode == 3 ? j.xs : static_cast<void *>(j.x));
        f.j[q].xs = j.xs;
        f.j[q].x0 = j.x;
    }
    if (!inverse)
        return in64 ? go<double, float, false, 0>(f, p.nx, p.ny, p.nz, s, nullptr, 0, skip)
                    : go<float, float, false, 0>(f, p.nx, p.ny, p.nz, s, nullptr, 0, skip);
    const bool upd = mode == 2 || mode == 4;
    double *red = upd ? st.upd : nullptr;
    const double *scale = upd ? st.scale : nullptr;
    const int stride = (int)update_slots(p);
    switch (mode) {
    case 1: return go<float, float, true, 1>(f, p.nx, p.ny, p.nz, s, red, stride, skip, scale);
    case 2: return go<float, float, true, 2>(f, p.nx, p.ny, p.nz, s, red, stride, skip, scale);
    case 3: return go<float, float, true, 3>(f, p.nx, p.ny, p.nz, s, red, stride, skip, scale);
    default: return go<float, float, true, 4>(f, p.nx, p.ny, p.nz, s, red, stride, skip, scale);
    }
}

}  // namespace ibs
