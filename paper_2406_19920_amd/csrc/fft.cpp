// Fast transforms: job sets of the solve stages to launches (k_fft.h).
#include "k_fft.h"

namespace ibs {

static const void *table(const Plan &p, size_t off) { return blob_ptr(p, off); }

// form of an axis's transform for a field of kind xk along it
static int axis_form(bool walls, int xk)
{
    return !walls ? fft::AX_PERIODIC : (xk == XK_F ? fft::AX_FACES : fft::AX_CENTRES);
}

// f32: forward in FP32 arithmetic
static FftJob fft_job(const Plan &p, bool z_axis, bool inverse, int rows, int ykind, int kind, int slot,
                      bool f32 = false)
{
    const BlobLayout &L = p.lay;
    FftJob f{};
    const bool faces = axis_form(z_axis ? p.wz : p.wx, kind) == fft::AX_FACES;
    if (faces) f.tw = table(p, f32 || inverse ? (z_axis ? L.ftz_face : L.ftx_face) : (z_axis ? L.ftz_face64 : L.ftx_face64));
    else if (f32 && !inverse) f.tw = table(p, z_axis ? L.ftz_fwd32 : L.ftx_fwd32);
    else f.tw = table(p, z_axis ? (inverse ? L.ftz_inv : L.ftz_fwd) : (inverse ? L.ftx_inv : L.ftx_fwd));
    if (f32 && !inverse) f.rot = table(p, z_axis ? L.frz_fwd32 : L.frx_fwd32);
    else f.rot = table(p, z_axis ? (inverse ? L.frz_inv : L.frz_fwd) : (inverse ? L.frx_inv : L.frx_fwd));
    f.rows = rows;
    f.skip = skip_first_row(ykind);
    f.kind = kind;
    f.slot = slot;
    return f;
}

// every component has ny transform rows per plane
hipError_t launch_fft_f64(const JobSet &js, const Plan &p, bool z_axis, bool inverse, hipStream_t s)
{
    for (int ax = 0; ax < 3; ++ax) {   // the jobs by form: at most two launches
        FftSet f{};
        for (int q = 0; q < js.n; ++q) {
            const FieldJob &j = js.j[q];
            const int kind = z_axis ? j.zk : j.xk;
            if (axis_form(z_axis ? p.wz : p.wx, kind) != ax) continue;
            FftJob &to = f.j[f.n++];
            to = fft_job(p, z_axis, inverse, j.rows, j.kind, kind, q);
            to.in = j.in;
            to.out = j.out;
        }
        const hipError_t e = z_axis ? launch_fft_z64(f, p.nz, p.ny, p.nx, inverse, ax, s)
                                    : launch_fft_x64(f, p.nx, p.ny, p.nz, inverse, ax, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
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
                            int kind, hipStream_t s)
{
    const FftTable t{static_cast<const FftJob *>(entries), n};
    const int ax = axis_form(walls, kind);
    return z_axis ? launch_fft_z64(t, nz, ny, nx, inverse, ax, s) : launch_fft_x64(t, nx, ny, nz, inverse, ax, s);
}

hipError_t launch_fft_x32(const SplitSet &ss, const Plan &p, const State &st, bool inverse, bool exact, bool in64,
                          int mode, int pass, hipStream_t s)
{
    const int *skip = pass >= 2 ? st.done : nullptr;
    const bool upd = mode == 2 || mode == 4;
    double *red = upd ? st.upd : nullptr;
    const double *scale = upd ? st.scale : nullptr;
    const int stride = (int)update_slots(p);
    for (int ax = 0; ax < 3; ++ax) {
        FftSet f{};
        for (int q = 0; q < ss.n; ++q) {
            const SplitJob &j = ss.j[q];
            if (axis_form(p.wx, j.xk) != ax) continue;
            FftJob &to = f.j[f.n++];
            to = fft_job(p, false, inverse, j.rows, j.kind, j.xk, j.slot, !exact && p.nx > FFT_F64_ARITH_MAX);
            to.in = j.in;
            to.out = !inverse ? static_cast<void *>(j.out) : (mode == 3 ? j.xs : static_cast<void *>(j.x));
            to.xs = j.xs;
            to.x0 = j.x;
        }
        hipError_t e;
        if (!inverse) e = launch_fft_x32_fwd(f, p.nx, p.ny, p.nz, ax, exact, in64, skip, s);
        else if (ax == fft::AX_FACES) e = launch_fft_x32_face(f, p.nx, p.ny, p.nz, mode, red, stride, skip, scale, s);
        else if (ax) e = launch_fft_x32_wall(f, p.nx, p.ny, p.nz, mode, red, stride, skip, scale, s);
        else e = launch_fft_x32_inv(f, p.nx, p.ny, p.nz, mode, red, stride, skip, scale, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_fft_z32(const SplitSet &ss, const Plan &p, const State &st, bool inverse, bool exact, int pass,
                          hipStream_t s)
{
    for (int ax = 0; ax < 3; ++ax) {
        FftSet f{};
        for (int q = 0; q < ss.n; ++q) {
            const SplitJob &j = ss.j[q];
            if (axis_form(p.wz, j.zk) != ax) continue;
            FftJob &to = f.j[f.n++];
            to = fft_job(p, true, inverse, j.rows, j.kind, j.zk, j.slot, !exact && p.nz > FFT_F64_ARITH_MAX);
            to.in = j.in;
            to.out = j.out;
        }
        if (hipError_t e = launch_fft_z32(f, p.nz, p.ny, p.nx, inverse, ax, exact,
                                          pass >= 2 ? st.done : nullptr, s); e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

}  // namespace ibs
