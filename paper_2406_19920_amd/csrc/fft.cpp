// Fast transforms: job sets of the solve stages to launches (k_fft.h).
#include "k_fft.h"

namespace ibs {

static const void *table(const Plan &p, size_t off) { return blob_ptr(p, off); }

static FftJob fft_job(const Plan &p, bool z_axis, bool inverse, int rows, int ykind, int kind, int slot)
{
    const BlobLayout &L = p.lay;
    FftJob f{};
    f.tw = table(p, z_axis ? (inverse ? L.ftz_inv : L.ftz_fwd) : (inverse ? L.ftx_inv : L.ftx_fwd));
    f.rot = table(p, z_axis ? (inverse ? L.frz_inv : L.frz_fwd) : (inverse ? L.frx_inv : L.frx_fwd));
    f.rows = rows;
    f.skip = skip_first_row(ykind);
    f.kind = kind;
    f.slot = slot;
    return f;
}

// every component has ny transform rows per plane
hipError_t launch_fft_f64(const JobSet &js, const Plan &p, bool z_axis, bool inverse, hipStream_t s)
{
    FftSet f{};
    f.n = js.n;
    for (int q = 0; q < js.n; ++q) {
        const FieldJob &j = js.j[q];
        f.j[q] = fft_job(p, z_axis, inverse, j.rows, j.kind, z_axis ? j.zk : j.xk, q);
        f.j[q].in = j.in;
        f.j[q].out = j.out;
    }
    return z_axis ? launch_fft_z64(f, p.nz, p.ny, p.nx, inverse, p.wz, s)
                  : launch_fft_x64(f, p.nx, p.ny, p.nz, inverse, p.wx, s);
}

size_t fft_entry_bytes() { return sizeof(FftJob); }

void fft_entry_fill(void *to, const Plan &p, const FieldJob &job, bool z_axis, bool inverse)
{
    FftJob &f = *static_cast<FftJob *>(to);
    f = fft_job(p, z_axis, inverse, job.rows, job.kind, z_axis ? job.zk : job.xk, 0);
    f.in = job.in;
    f.out = job.out;
}

hipError_t launch_fft_table(const void *entries, int n, int nx, int ny, int nz, bool z_axis, bool inverse, bool walls,
                            hipStream_t s)
{
    const FftTable t{static_cast<const FftJob *>(entries), n};
    return z_axis ? launch_fft_z64(t, nz, ny, nx, inverse, walls, s) : launch_fft_x64(t, nx, ny, nz, inverse, walls, s);
}

hipError_t launch_fft_x32(const SplitSet &ss, const Plan &p, const State &st, bool inverse, bool in64, int mode,
                          int pass, hipStream_t s)
{
    const int *skip = pass >= 2 ? st.done : nullptr;
    FftSet f{};
    f.n = ss.n;
    for (int q = 0; q < ss.n; ++q) {
        const SplitJob &j = ss.j[q];
        f.j[q] = fft_job(p, false, inverse, j.rows, j.kind, j.xk, j.slot);
        f.j[q].in = j.in;
        f.j[q].out = !inverse ? static_cast<void *>(j.out) : (mode == 3 ? j.xs : static_cast<void *>(j.x));
        f.j[q].xs = j.xs;
        f.j[q].x0 = j.x;
    }
    if (!inverse) return launch_fft_x32_fwd(f, p.nx, p.ny, p.nz, p.wx, in64, skip, s);
    const bool upd = mode == 2 || mode == 4;
    double *red = upd ? st.red + (size_t)(pass - 1) * st.upd_region : nullptr;
    const double *scale = upd ? st.scale : nullptr;
    const int stride = (int)update_slots(p);
    return p.wx ? launch_fft_x32_wall(f, p.nx, p.ny, p.nz, mode, red, stride, skip, scale, s)
                : launch_fft_x32_inv(f, p.nx, p.ny, p.nz, mode, red, stride, skip, scale, s);
}

hipError_t launch_fft_z32(const SplitSet &ss, const Plan &p, const State &st, bool inverse, int pass, hipStream_t s)
{
    FftSet f{};
    f.n = ss.n;
    for (int q = 0; q < ss.n; ++q) {
        const SplitJob &j = ss.j[q];
        f.j[q] = fft_job(p, true, inverse, j.rows, j.kind, j.zk, j.slot);
        f.j[q].in = j.in;
        f.j[q].out = j.out;
    }
    return launch_fft_z32(f, p.nz, p.ny, p.nx, inverse, p.wz, pass >= 2 ? st.done : nullptr, s);
}

}  // namespace ibs
