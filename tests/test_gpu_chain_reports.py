"""Reports of a multi-grid batch whose pressure fields run as chains: the mean
removed from each right-hand side, against the single solves' reports."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# fields of 3.9 and 3.1 MB, the first at the fewest rows a chain takes: three
# plans of each make a group large enough
@pytest.mark.parametrize("shape", [(256, 17, 112), (96, 64, 64)])
def test_removed_means(shape):
    from paper_2406_19920_amd import ibsolve as ibs
    assert torch.cuda.is_available()
    print("case chain reports", shape, flush=True)
    recs, keep = [], []
    for q in range(3):
        S = ibs.Solver(*shape, beta=0.5 * q)
        g = torch.Generator(device="cuda").manual_seed(q)
        b = torch.randn(S.shape(), generator=g, dtype=torch.float64, device="cuda") + (q + 2.0)
        x = S.empty()
        recs.append(S.poisson_job(b, x))
        keep.append((S, b, x))
    h = ibs.ibs_batch_build_multigrid(recs)
    try:
        ibs.ibs_batch_launch(h, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        ibs.ibs_batch_destroy(h)
    for q, (S, b, x) in enumerate(keep):
        got = S.read_info(0)
        S.poisson(b, info=S.info[1:2])
        want = S.read_info(1)
        assert got.status == want.status == 0 and got.iters == 1
        # a mean near q + 2 of unit noise; the same arithmetic on both sides
        assert abs(want.removed_mean - (q + 2.0)) < 0.1
        assert abs(got.removed_mean - want.removed_mean) < 1e-14 * (q + 2.0)
