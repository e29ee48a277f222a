"""Fast transforms on the GPU: every line length along x and z, periodic and
walled, both precisions, through Helmholtz solves of known fields (r = A x
formed by the stencil of residual(), which shares no code with the solve)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

SIZES_32 = list(range(32, 513, 32))
SIZES_16 = [16, 48, 80, 112, 144, 176, 208, 240, 336, 400, 432]
# c |lambda| <= 2 at the smallest cell: condition number below 10.  FP64: five
# stages of at most 4 ulps each and the stencil's own rounding, times that
# condition: under 1e-13; refined: the solve's own tolerance
TOL = {False: 1e-13, True: 1e-10}


@pytest.fixture(scope="module")
def ibs():
    from paper_2406_19920_amd import ibsolve
    assert torch.cuda.is_available()
    return ibsolve


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("refined", [False, True])
@pytest.mark.parametrize("n", SIZES_32 + SIZES_16)
def test_every_length(ibs, n, refined, walls):
    if refined and n % 32:
        pytest.skip("the refined path takes multiples of 32")
    kw = dict(bc_x=ibs.IBS_DIRICHLET, bc_z=ibs.IBS_DIRICHLET) if walls else {}
    for nx, nz in ((n, 32), (32, n)):
        print("case fft", nx, nz, refined, walls, flush=True)
        S = ibs.Solver(nx, 5, nz, beta=0.5, precision=ibs.IBS_REFINED_BF16X3 if refined else ibs.IBS_FP64, **kw)
        c = 0.125 / max(nx, nz) ** 2
        xs, rs = [], []
        for comp in range(3):
            g = torch.Generator(device="cuda")
            g.manual_seed(10 * n + comp)
            x = torch.randn(S.shape(comp + 1), generator=g, dtype=torch.float64, device="cuda")
            if comp == 1:
                x[:, 0] = 0
                x[:, 5] = 0
            if walls and comp == 0:
                x[:, :, 0] = 0
            if walls and comp == 2:
                x[0] = 0
            xs.append(x)
            rs.append(-S.residual(comp + 1, c, x, torch.zeros_like(x)))
        got = S.helmholtz([0, 1, 2], [c] * 3, rs)
        for comp in range(3):
            err = float((got[comp] - xs[comp]).norm() / xs[comp].norm())
            assert err < TOL[refined], (nx, nz, comp, err)


def test_solutions_over_other_right_hand_sides(ibs):
    """FP64 jobs work in place on their solutions: solutions that lie on another
    component's right-hand side, or one plane into their own, end bitwise as
    apart."""
    print("case fft overlap", flush=True)
    n = 64
    S = ibs.Solver(n, n, n, beta=0.5)
    c = [0.125 / n ** 2] * 3
    flat = [torch.randn((n + 1) * n * n, generator=torch.Generator(device="cuda").manual_seed(q),
                        dtype=torch.float64, device="cuda") for q in range(3)]
    u, w = flat[0][:n ** 3].view(n, n, n), flat[1][:n ** 3].view(n, n, n)
    want = S.helmholtz([0, 2], c[:2], [u.clone(), w.clone()])
    S.helmholtz([0, 2], c[:2], [u, w], [w, u])
    assert torch.equal(w, want[0]) and torch.equal(u, want[1])
    b = flat[2][n * n:].view(n, n, n)
    phi = flat[2][:n ** 3].view(n, n, n)
    want = S.poisson(b.clone())
    S.poisson(b, phi)
    assert torch.equal(phi, want)


# 104 MB is half a group: two components and one, and one by one
@pytest.mark.parametrize("ny", [192, 212])
def test_component_groups(ibs, ny):
    print("case fft groups", ny, flush=True)
    S = ibs.Solver(256, ny, 256, beta=0.5)
    c = [1e-6, 2e-6, 3e-6]
    rs = [torch.randn(S.shape(op), generator=torch.Generator(device="cuda").manual_seed(op),
                      dtype=torch.float64, device="cuda") for op in (1, 2, 3)]
    got = S.helmholtz([0, 1, 2], c, rs)
    for q in range(3):
        assert torch.equal(got[q], S.helmholtz([q], c[q:q + 1], rs[q:q + 1])[0])
        assert S.read_info(0).status == 0


# both classes of blocks (few planes, and above 2048), every size of the fused
# x-z transforms beside another one
@pytest.mark.parametrize("refined", [False, True])
@pytest.mark.parametrize("nx,ny,nz", [(16, 17, 64), (64, 9, 48), (48, 700, 32), (32, 700, 64), (64, 700, 64), (64, 17, 64)])
def test_planes(ibs, nx, ny, nz, refined):
    if refined and (nx % 32 or nz % 32):
        pytest.skip("the refined path takes multiples of 32")
    print("case planes", nx, ny, nz, refined, flush=True)
    S = ibs.Solver(nx, ny, nz, beta=0.5, precision=ibs.IBS_REFINED_BF16X3 if refined else ibs.IBS_FP64)
    c = 0.125 / max(nx, ny, nz) ** 2
    xs, rs = [], []
    for comp in range(3):
        g = torch.Generator(device="cuda")
        g.manual_seed(comp)
        x = torch.randn(S.shape(comp + 1), generator=g, dtype=torch.float64, device="cuda")
        if comp == 1:
            x[:, 0] = 0
            x[:, ny] = 0
        xs.append(x)
        rs.append(-S.residual(comp + 1, c, x, torch.zeros_like(x)))
    got = S.helmholtz([0, 1, 2], [c] * 3, rs)
    for comp in range(3):
        assert float((got[comp] - xs[comp]).norm() / xs[comp].norm()) < TOL[refined]
        assert S.read_info(comp).status == 0
