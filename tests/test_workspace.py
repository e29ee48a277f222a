"""Workspace sizes of the refined path: the call's state takes the same small
room on every grid, so grids at the limit of the fixed scratch array are served."""
import numpy as np
import pytest
import torch   # before the library, whose HIP runtime is torch's

ibs = pytest.importorskip("paper_2406_19920_amd.ibsolve", exc_type=ImportError)

# three FP32 fields of these take all but 262 KB or less of the array's 64 MB
AT_THE_LIMIT = [(416, 26, 512), (512, 26, 416), (32, 676, 256), (32, 541, 320)]


@pytest.mark.parametrize("shape", AT_THE_LIMIT)
@pytest.mark.parametrize("max_iter", [0, 8])
def test_grids_at_the_limit_fit(shape, max_iter):
    plan = ibs.solver_plan(ibs.make_desc(*shape, precision=ibs.IBS_REFINED_BF16X3, max_iter=max_iter))
    try:
        assert ibs.solver_plan_bytes(plan, ibs.IBS_OP_POISSON)[1] <= ibs.IBS_NOALLOC_SCRATCH_BYTES
    finally:
        ibs.solver_plan_destroy(plan)


@pytest.mark.parametrize("refined", [False, True])
@pytest.mark.parametrize("shape", [(32, 2, 32), (32, 768, 512), (512, 2, 512), (512, 768, 512), (96, 75, 64)])
def test_state_is_small_on_every_grid(shape, refined):
    nx, ny, nz = shape
    faces = np.linspace(0, 1, nx + 1) ** 1.1
    for kw in ({}, dict(bc_x=ibs.IBS_DIRICHLET, x_faces=faces)):
        plan = ibs.solver_plan(ibs.make_desc(*shape, precision=ibs.IBS_REFINED_BF16X3 if refined else ibs.IBS_FP64, **kw))
        per = 12 if refined else 8
        try:
            for op, ncomp, rows in ((ibs.IBS_OP_POISSON, 1, ny), (ibs.IBS_OP_HELMHOLTZ_U, 3, ny + 1)):
                fields = per * ncomp * nx * rows * nz
                assert 0 < ibs.solver_plan_bytes(plan, op, ncomp)[1] - fields <= 256 << 10
        finally:
            ibs.solver_plan_destroy(plan)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", AT_THE_LIMIT[1:3])
def test_solves_at_the_limit_without_workspace(shape):
    assert torch.cuda.is_available()
    print("case workspace", shape, flush=True)
    S = ibs.Solver(*shape, beta=1.0, precision=ibs.IBS_REFINED_BF16X3)
    b = torch.randn(S.shape(), generator=torch.Generator(device="cuda").manual_seed(3), dtype=torch.float64, device="cuda")
    want, phi = S.poisson(b), S.empty()
    report = S.read_info(0)
    ibs.solve_poisson_noalloc(S.plan, b.data_ptr(), phi.data_ptr(), S.info[1].data_ptr(), S.stream())
    assert torch.equal(phi, want)
    got = S.read_info(1)
    assert got.status == report.status == 0 and got.iters == report.iters and got.rel_residual == report.rel_residual
