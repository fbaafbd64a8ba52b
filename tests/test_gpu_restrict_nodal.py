"""3D residual and full weighting of a grid with nodal coefficients as a
single-level call, which forms the faces it needs as it marches: every column
height, chunks of coarse planes that divide the grid or not, bit for bit against
the oracle; and no scratch beyond a launch descriptor."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 17, 33, 129])  # 1, 7, 15 and 63 inner coarse nodes an edge
@pytest.mark.parametrize("by", [0, 8, 16, 32])
@pytest.mark.parametrize("zc", [1, 3, 8, 64])
@pytest.mark.parametrize("dt", [np.float64, np.float32])
def test_restrict_with_nodal_coefficients(n, by, zc, dt, dev_ok):
    import torch

    import paper_1406_5369_amd as m

    dev = lambda a: torch.from_numpy(a).to("cuda")  # noqa: E731
    u, f = inputs.random_guess(3, n, 70 + n).astype(dt), inputs.uniform_rhs(3, n, 71 + n).astype(dt)
    k = inputs.varcoef_k(n, 72 + n).astype(dt)
    expect = oracle.restrict(oracle.residual(u, f, k=k))
    fc = torch.full(expect.shape, 7.0, dtype=getattr(torch, np.dtype(dt).name), device="cuda")
    m.mg_level_residual_restrict(dev(u), dev(f), fc, k=dev(k), by=by, zchunk=zc)
    torch.cuda.synchronize()
    got, inner = fc.cpu().numpy(), (slice(1, -1),) * 3
    assert np.array_equal(got[inner], expect[inner])
    got[inner] = 7.0  # the boundary is not written
    assert (got == 7.0).all()


def test_no_scratch(dev_ok):
    """257^3 FP64 with 256 MiB of device memory left: three face arrays would take 407 MB."""
    import torch

    import paper_1406_5369_amd as m

    n = 257
    u, f = (torch.rand((n,) * 3, dtype=torch.float64, device="cuda") for _ in range(2))
    k = torch.rand((n,) * 3, dtype=torch.float64, device="cuda") + 1.0
    first, second = (torch.zeros((129,) * 3, dtype=torch.float64, device="cuda") for _ in range(2))
    m.mg_level_residual_restrict(u, f, first, k=k)
    torch.cuda.empty_cache()
    held = []
    try:
        while (free := torch.cuda.mem_get_info()[0]) > (288 << 20):
            held.append(torch.empty(min(free - (256 << 20), 32 << 30), dtype=torch.uint8, device="cuda"))
        m.mg_level_residual_restrict(u, f, second, k=k)
        torch.cuda.synchronize()
    finally:
        held.clear()
        torch.cuda.empty_cache()
    assert torch.equal(first, second)
