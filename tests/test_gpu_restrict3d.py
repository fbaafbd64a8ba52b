"""3D residual and full weighting at the edges of its columns: 30 coarse nodes
along x, 2, 3, 4 or 6 along y by tile rows and type, chunks of coarse planes that
divide the grid or not; bit for bit against the oracle."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 9, 65, 129])  # 1, 3, 31 and 63 inner coarse nodes an edge
@pytest.mark.parametrize("by", [8, 16, 32])
@pytest.mark.parametrize("zc", [1, 4, 31, 64])
@pytest.mark.parametrize("dt,varcoef", [(np.float64, False), (np.float32, False), (np.float16, False),
                                        (np.float64, True), (np.float32, True)])
def test_restrict_columns(n, by, zc, dt, varcoef, dev_ok):
    import torch

    import paper_1406_5369_amd as m

    u, f = inputs.random_guess(3, n, 40 + n), inputs.uniform_rhs(3, n, 41 + n)
    if dt == np.float16:
        u = u * (8.0 / (n - 1) ** 2)
    u, f = u.astype(dt), f.astype(dt)
    k = inputs.varcoef_k(n, 6).astype(dt) if varcoef else None
    expect = oracle.restrict(oracle.residual(u, f, k=k), **({"out_dtype": dt} if dt == np.float16 else {}))
    fc = torch.full(expect.shape, 7.0, dtype=getattr(torch, np.dtype(dt).name), device="cuda")
    dev = lambda a: torch.from_numpy(a).to("cuda")  # noqa: E731
    m.mg_level_residual_restrict(dev(u), dev(f), fc, k=dev(k) if varcoef else None, by=by, zchunk=zc)
    torch.cuda.synchronize()
    got, inner = fc.cpu().numpy(), (slice(1, -1),) * 3
    assert np.array_equal(got[inner], expect[inner])
    got[inner] = 7.0  # the boundary is not written
    assert (got == 7.0).all()
