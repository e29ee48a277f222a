"""Precision of the markers' interpolated velocity at a large viscous number,
where the Helmholtz right-hand side r = u^e - c L u is 17 times u: u^e must
not be recovered from it."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

NX, NY, NZ = 32, 32, 16
AB, DT, C = 2.0 ** -10, 2.0 ** -10, 1.7e-3   # c |L| = 15.7
# Roundings against the exact interpolation, in eps rms for values below 1: u^e
# 0.14, five factors and products of a term 0.14 each, on 27 terms whose weights
# have the root sum square 0.35 at most; the sum's levels 0.1: below 0.2 in all.
# r lies between 8 and 17, so its own rounding alone leaves 0.8.
TOL = 0.4 * 2.0 ** -52


def _fields(rng):
    shape = {0: (NZ, NY, NX), 1: (NZ, NY + 1, NX), 2: (NZ, NY, NX)}
    out = []
    for comp in range(3):
        k, j, i = np.indices(shape[comp])
        f = (1.0 - 2.0 * ((i + j + k) % 2)) * rng.uniform(0.5, 1.0, shape[comp])
        if comp == 1:
            f[:, 0] = f[:, NY] = 0.0
        out.append(f)
    return out


def _ue(f, c):
    """u^e = u + (alpha + beta) c L u in extended precision, away from the walls."""
    f = f.astype(np.longdouble)
    lap = np.zeros_like(f)
    for axis, n in ((2, NX), (1, NY), (0, NZ)):
        lap += (np.roll(f, 1, axis) - 2 * f + np.roll(f, -1, axis)) * np.longdouble(n) ** 2
    return f + np.longdouble(AB) * c * lap


def _weight(r):
    a = np.abs(np.longdouble(r))
    if a <= 0.5:
        return (1 + np.sqrt(1 - 3 * a * a)) / 3
    return (5 - 3 * a - np.sqrt(1 - 3 * (1 - a) ** 2)) / 6 if a < 1.5 else np.longdouble(0)


def _interpolate(f, comp, m):
    at = [m[ax] - (0.0 if ax == comp else 0.5) for ax in range(3)]   # grid units
    first = [int(np.floor(a + 0.5)) - 1 for a in at]
    U = np.longdouble(0)
    for k in range(3):
        for j in range(3):
            for i in range(3):
                w = _weight(first[0] + i - at[0]) * _weight(first[1] + j - at[1]) * _weight(first[2] + k - at[2])
                U += w * f[(first[2] + k) % NZ, first[1] + j, (first[0] + i) % NX]
    return U


def test_marker_velocity_keeps_its_digits():
    assert torch.cuda.is_available()
    from paper_2406_19920_amd import ibsolve as ibs
    print("case ibm precision", flush=True)
    rng = np.random.default_rng(11)
    vel = _fields(rng)
    # on the grid points of u and halfway between v's and w's: exact distances
    nm = 300
    m = np.stack([rng.integers(0, NX, nm), rng.integers(4, NY - 4, nm) + 0.5, rng.integers(0, NZ, nm) + 0.5], 1)
    X = m / np.array([NX, NY, NZ])
    re = DT / C
    c = np.longdouble(DT) / np.longdouble(re)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).to("cuda") for a in vel]
    p = torch.zeros((NZ, NY, NX), dtype=torch.float64, device="cuda")
    n = [torch.zeros_like(t) for t in dev]
    force = torch.zeros((nm, 3), dtype=torch.float64, device="cuda")
    S = ibs.Solver(NX, NY, NZ)
    S.rk_stage(*dev, p, *n, dict(alpha=AB - 1.0, beta=1.0, gamma=0.0, zeta=0.0, dt=DT, re=re),
               torch.from_numpy(X).to("cuda"), torch.zeros((nm, 3), dtype=torch.float64, device="cuda"),
               torch.full((nm,), 1e-5, dtype=torch.float64, device="cuda"), force=force)
    U = -force.cpu().numpy() * DT   # F = (0 - U) / dt, dt a power of two
    for comp in range(3):
        ref = _ue(vel[comp], c)
        err = np.array([float(U[q, comp] - _interpolate(ref, comp, m[q])) for q in range(nm)])
        rms = np.sqrt(np.mean(err ** 2))
        print("component", comp, "rms error", rms / 2.0 ** -52, "eps", flush=True)
        assert rms < TOL, (comp, rms)
