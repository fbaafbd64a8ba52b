"""3D refinement pass with one wavefront per column (the built-in geometry of
FP32 refinement), through whole untuned solves: ragged columns, chunks of one
plane and more, with and without coefficients, single grids and batches; fields
bit for bit against the oracle, norms up to the order of their sums."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 9, 17, 33, 65, 129])
@pytest.mark.parametrize("varcoef", [False, True])
def test_refinement_columns(n, varcoef, dev_ok, monkeypatch):
    import torch

    import paper_1406_5369_amd as m

    monkeypatch.setenv("MG_AUTOTUNE", "0")
    f = inputs.uniform_rhs(3, n, 21)
    k = inputs.varcoef_k(n, 7) if varcoef else None
    ue, he, _ = oracle.solve_ir_f32(np.zeros_like(f), f, tol=0.0, max_cycles=4, k=k)
    par = dict(op=m.OP_VARCOEF_NODAL, k=torch.from_numpy(k).to("cuda")) if varcoef else {}
    with m.Solver(m.Params(dim=3, n=n, precision=m.PREC_FP32_IR, **par)) as s:
        assert m.mg_tile_config(s.ctx, 0, 2)[3] == 1
        fd = torch.from_numpy(f).to("cuda")
        u = torch.zeros_like(fd)
        _, cyc, h = s.solve(u, fd, tol=0.0, max_cycles=4)
        norm = s.residual_norm(u, fd)
        torch.cuda.synchronize()
    assert cyc == len(he) - 1
    assert np.array_equal(u.cpu().numpy(), ue)
    # two sums of N squares in different orders differ by at most (N - 1) 2^-53 relative each
    tol = max(1e-14, 2.0 * f.size * 2.0**-53)
    np.testing.assert_allclose(h, he, rtol=tol)
    np.testing.assert_allclose(norm, he[-1], rtol=tol)
