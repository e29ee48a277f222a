"""y pencils on the GPU: row counts at the edges of every launch shape, walls
and periodic y, both precisions, through the solve of known fields (r = A x
formed by the stencil of residual())."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# first and last row count of each shape (chunks x rows per chunk), and odd
# ones between; the smallest and largest a plan takes
WALL_ROWS = [2, 3, 31, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 256, 257, 320, 321, 384, 385,
             512, 513, 768]
CYCLIC_ROWS = [48, 64, 80, 96, 128, 160, 192, 256, 320, 384, 512]
# Helmholtz: condition number of the pencils below 10, see TOL of the transforms' test
TOL = {False: 1e-13, True: 1e-10}


@pytest.fixture(scope="module")
def ibs():
    from paper_2406_19920_amd import ibsolve
    assert torch.cuda.is_available()
    return ibsolve


def _field(S, op, ny, walls, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.randn(S.shape(op), generator=g, dtype=torch.float64, device="cuda")
    if op == 2 and walls:
        x[:, 0] = 0
        x[:, ny] = 0
    return x


@pytest.mark.parametrize("refined", [False, True])
@pytest.mark.parametrize("ny,walls", [(n, True) for n in WALL_ROWS] + [(n, False) for n in CYCLIC_ROWS])
def test_every_shape(ibs, ny, walls, refined):
    kw = {} if walls else dict(bc_y_vel=ibs.IBS_PERIODIC, bc_y_p=ibs.IBS_PERIODIC)
    for nx, nz in ((32, 32), (96, 160)):    # few tiles (shorter chunks), and many
        print("case pencils", nx, ny, nz, walls, refined, flush=True)
        S = ibs.Solver(nx, ny, nz, beta=0.5 if walls else 0.0,
                       precision=ibs.IBS_REFINED_BF16X3 if refined else ibs.IBS_FP64, **kw)
        c = 0.125 / max(nx, ny, nz) ** 2
        xs = [_field(S, q, ny, walls, 7 * ny + q) for q in (1, 2, 3)]
        rs = [-S.residual(q, c, x, torch.zeros_like(x)) for q, x in zip((1, 2, 3), xs)]
        for got, x in zip(S.helmholtz([0, 1, 2], [c] * 3, rs), xs):
            err = float((got - x).norm() / x.norm())
            assert err < TOL[refined], err
        # the pressure's singular pencil: a field of y alone, zero weighted
        # mean, solved by sums of fluxes.  Its right-hand side, formed by the
        # stencil, is off by an ulp of the largest term; summed back twice
        # over ny rows: about eps ny^2 of the field
        x = _field(S, 0, ny, walls, 5)
        x[:] = x[:1, :, :1]
        w = torch.diff(torch.tensor(ibs.ibs_plan_export(S.plan, 0), device="cuda"))[None, :, None]
        x -= (x * w).sum() / (w.sum() * nx * nz)
        b = -S.residual(0, 0.0, x, torch.zeros_like(x))
        err = float((S.poisson(b) - x).norm() / x.norm())
        assert err < max(1e-13, 2.0 ** -52 * ny ** 2) if not refined else err < 1e-10, err
