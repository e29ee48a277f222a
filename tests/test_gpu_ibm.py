"""The immersed boundary's two ways to u^e, against the oracle's stage: formed
from the right-hand side (with F kept in the workspace), and, at a large
viscous number, as a field."""
import numpy as np
import pytest

import oracle
from oracle import OP_P, OP_U, OP_V, OP_W, fstep
from paper_2406_19920_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("py", [False, True])
@pytest.mark.parametrize("re,keep", [(150.0, False), (0.05, False), (0.05, True)])
def test_marker_paths(re, keep, py):
    assert torch.cuda.is_available()
    from paper_2406_19920_amd import ibsolve as ibs
    nx, ny, nz, nm = 32, 48, 16, 70
    print("case ibm", re, keep, py, flush=True)
    g = oracle.Grid(nx, ny, nz, periodic_y=py)
    S = ibs.Solver(nx, ny, nz, **(dict(bc_y_vel=ibs.IBS_PERIODIC, bc_y_p=ibs.IBS_PERIODIC) if py else {}))
    rng = np.random.default_rng(5)
    vel = [rng.standard_normal(g.shape(op)) for op in (OP_U, OP_V, OP_W)]
    if not py:
        vel[1][:, 0, :] = 0
        vel[1][:, ny, :] = 0
    p = rng.standard_normal(g.shape(OP_P))
    # a shell that leaves the box at every side: supports wrap, or end at a wall
    X = synth.sphere_markers(nm, 0.55, centre=(0.5, 0.5, 0.5))
    ud, dvol = 0.3 * rng.standard_normal((nm, 3)), np.full(nm, (1.0 / nx) ** 3)
    coef = dict(alpha=4 / 15, beta=4 / 15, gamma=8 / 15, zeta=0.0, dt=2e-3, re=re)
    ref = fstep.stage(g, *vel, p, coef, n_prev=None, markers=X, ud=ud, dvol=dvol)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).to("cuda") for a in (*vel, p, X, ud, dvol)]
    n = [torch.zeros_like(t) for t in dev[:3]]
    force = torch.zeros((nm, 3), dtype=torch.float64, device="cuda") if keep else None
    S.rk_stage(*dev[:4], *n, coef, *dev[4:], force=force)
    torch.cuda.synchronize()
    # the sides' FP64 roundings: of r, up to 1 + c |L| = 154 of |u| (re 0.05),
    # and of the solves; 1e-12 is what the other stages' tests allow
    for got, want in zip(dev[:4], (ref["u"], ref["v"], ref["w"], ref["p"])):
        err = np.linalg.norm(got.cpu().numpy() - want) / np.linalg.norm(want)
        assert err < (1e-12 if re > 1 else 1e-10), err
    if keep:
        err = np.linalg.norm(force.cpu().numpy() - ref["force"]) / np.linalg.norm(ref["force"])
        assert err < 1e-12, err
