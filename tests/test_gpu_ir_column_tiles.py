"""The refinement pass with one wavefront per column as a single-level call: both
column heights, chunks of one plane, dividing the grid or not, and longer than
the grid, from a nonzero iterate and correction, with and without coefficients;
u and r bit for bit against the oracle, and the tile that a solver reports is one
that the call takes."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


def run(n, varcoef, noalloc, **tile):
    import torch

    import paper_1406_5369_amd as m

    dev = lambda a: torch.from_numpy(a).to("cuda")  # noqa: E731
    u, f = inputs.random_guess(3, n, 61), inputs.uniform_rhs(3, n, 62)
    e = (inputs.random_guess(3, n, 63) * 1e-3).astype(np.float32)
    k = inputs.varcoef_k(n, 64) if varcoef else None
    ue, re, rho = oracle.ir_update(u, e, f, k=k)
    uo = torch.full(u.shape, 7.0, dtype=torch.float64, device="cuda")
    r = torch.full(u.shape, 7.0, dtype=torch.float32, device="cuda")
    got = m.mg_level_ir_update(dev(u), dev(e), dev(f), uo, r, k=dev(k) if varcoef else None, noalloc=noalloc, **tile)
    torch.cuda.synchronize()
    inner = (slice(1, -1),) * 3
    for a, expect in ((uo.cpu().numpy(), ue), (r.cpu().numpy(), re)):
        assert np.array_equal(a[inner], expect[inner])
        a[inner] = 7.0  # the boundary is not written
        assert (a == 7.0).all()
    # two sums of N squares in different orders differ by at most (N - 1) 2^-53 relative each
    assert got == pytest.approx(rho, rel=max(1e-14, 2.0 * f.size * 2.0**-53))


@pytest.mark.parametrize("n", [5, 9, 65, 129])
@pytest.mark.parametrize("by", [6, 8])
@pytest.mark.parametrize("zchunk", [1, 3, 8, 200])
@pytest.mark.parametrize("varcoef", [False, True])
def test_column_pass(n, by, zchunk, varcoef, dev_ok):
    run(n, varcoef, zchunk == 3, by=by, zchunk=zchunk, waves=1)


@pytest.mark.parametrize("varcoef", [False, True])
def test_reported_tile_is_accepted(varcoef, dev_ok, monkeypatch):
    import torch

    import paper_1406_5369_amd as m

    monkeypatch.setenv("MG_AUTOTUNE", "0")
    n = 65
    par = dict(op=m.OP_VARCOEF_NODAL, k=torch.from_numpy(inputs.varcoef_k(n, 64)).to("cuda")) if varcoef else {}
    with m.Solver(m.Params(dim=3, n=n, precision=m.PREC_FP32_IR, **par)) as s:
        by, zchunk, prefetch, waves, _, pairs = m.mg_tile_config(s.ctx, 0, 2, with_order=True)
    assert waves == 1
    run(n, varcoef, False, by=by, zchunk=zchunk, prefetch=prefetch, waves=waves, pairs=pairs)


@pytest.mark.parametrize("tile", [dict(), dict(by=12), dict(by=16), dict(by=8, prefetch=2), dict(by=8, pairs=1)])
def test_other_columns_are_refused(tile, dev_ok):
    import paper_1406_5369_amd as m

    with pytest.raises(m.MGError) as ei:
        run(9, False, False, zchunk=4, waves=1, **tile)
    assert ei.value.code == m.MG_EINVAL
