"""Multi-grid batches whose fields run as chains of the fast kernels (groups of
8 MB and more): against the single-grid solves, which run the same arithmetic,
with walls (the face-normal components in chains of their own, or too few for
one and so in the stage kernels), and the batch
whose fields overlap, which keeps the order every right-hand side before any
solution."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ibs():
    from paper_2406_19920_amd import ibsolve
    assert torch.cuda.is_available()
    return ibsolve


def _randn(shape, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, dtype=torch.float64, device="cuda")


# 17 rows: the fewest a chain takes; 96x64x64: several fields of a chain; the
# last one beside a group of its own size class too small for a chain
@pytest.mark.parametrize("shape,walls,count", [((256, 17, 112), False, 1), ((96, 64, 64), True, 2),
                                                ((96, 64, 64), True, 3), ((64, 33, 48), False, 3)])
def test_chains_match_single_solves(ibs, shape, walls, count):
    nx, ny, nz = shape
    print("case chains", shape, walls, count, flush=True)
    kw = dict(bc_x=ibs.IBS_DIRICHLET, bc_z=ibs.IBS_DIRICHLET) if walls else {}
    recs, keep = [], []
    for q in range(count):
        S = ibs.Solver(nx, ny, nz, beta=0.4 * q, **kw)
        r = [_randn(S.shape(op), 10 * q + op) for op in (1, 2, 3)]
        b = _randn(S.shape(0), 10 * q)
        x = [S.empty(op) for op in (1, 2, 3)] + [S.empty(0)]
        work = torch.empty(S.work_p, dtype=torch.uint8, device="cuda")
        recs += [S.helmholtz_job([0, 1, 2], [1e-3] * 3, r, x[:3]), S.poisson_job(b, x[3], info_slot=3, work=work)]
        keep.append((S, r, b, x, work))
    h = ibs.ibs_batch_build_multigrid(recs)
    try:
        for _ in range(2):
            ibs.ibs_batch_launch(h, torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            for S, r, b, x, _w in keep:
                infos = [S.read_info(q) for q in range(4)]
                ref = S.helmholtz([0, 1, 2], [1e-3] * 3, r, info_slot=4) + [S.poisson(b, info=S.new_info(1))]
                for got, want in zip(x, ref):
                    # fast kernels: the same arithmetic; dense ones round differently
                    assert float((got - want).norm() / want.norm()) < 1e-13
                assert all(i.status == 0 and i.iters == 1 for i in infos)
    finally:
        ibs.ibs_batch_destroy(h)


def test_overlapping_fields_keep_their_order(ibs):
    print("case chains overlap", flush=True)
    n = 64
    S = [ibs.Solver(n, n, n, beta=b) for b in (0.0, 1.0)]
    b0, x0, x1 = _randn(S[0].shape(0), 1), _randn(S[0].shape(0), 2), S[0].empty(0)
    work = [torch.empty(s.work_p, dtype=torch.uint8, device="cuda") for s in S]
    old = x0.clone()
    # the second job's right-hand side is the buffer the first one's solution goes to
    h = ibs.ibs_batch_build_multigrid([S[0].poisson_job(b0, x0, work=work[0]),
                                       *[s.poisson_job(x0, x1, work=w) for s, w in zip(S[1:], work[1:])]])
    try:
        ibs.ibs_batch_launch(h, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        ibs.ibs_batch_destroy(h)
    for got, s, b in ((x0, S[0], b0), (x1, S[1], old)):
        want = s.poisson(b)
        assert float((got - want).norm() / want.norm()) < 1e-11
