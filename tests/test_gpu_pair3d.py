"""3D red-black levels whose sweeps run two to a launch: 56 x 24 owned nodes per
box and chunks of planes, with the correction, with the residual norm of the
incoming iterate, from an iterate and from zero, for each constant operator.
Whole solves on the built-in tiles (no tuning) against the oracle: fields bit
for bit."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu

RB, SYM = 0, 2
V, W = 0, 1
SKEW = (7.0, -1.2, -0.8, -1.3, -1.2, -1.4, -1.1)


# one grid with enough boxes: several boxes and chunks along each axis, ragged last ones
@pytest.mark.parametrize("op,precision,smoother,nu1,nu2", [
    ("laplace", 0, RB, 2, 2), ("laplace", 0, SYM, 4, 3), ("laplace", 0, RB, 3, 1), ("laplace", 1, RB, 2, 2),
    ("laplace", 1, SYM, 3, 4), ("laplace", 2, SYM, 2, 2), ("stencil", 0, SYM, 2, 2), ("stencil", 0, RB, 5, 3),
    ("cells", 0, RB, 2, 2), ("cells", 0, RB, 4, 3)])
def test_pairs_of_one_grid(op, precision, smoother, nu1, nu2, dev_ok, monkeypatch):
    import torch

    import paper_1406_5369_amd as m

    monkeypatch.setenv("MG_AUTOTUNE", "0")
    n = 256 if op == "cells" else 257
    kw = dict(tol=0.0, max_cycles=2, smoother=smoother, nu1=nu1, nu2=nu2)
    par = dict(dim=3, n=n, smoother=smoother, nu1=nu1, nu2=nu2, precision=precision)
    f = inputs.random_cells(3, n, 4) if op == "cells" else inputs.uniform_rhs(3, n, 4)
    if op == "cells":
        f = f - f.mean()
    z = np.zeros_like(f)
    if op == "stencil":
        ue, he, _ = oracle.st_solve(z, f, SKEW, **kw)
        par.update(op=m.OP_CONST_STENCIL, stencil=SKEW)
    elif op == "cells":
        ue, he, *_ = oracle.cc_solve(z, f, **kw)
        par.update(bc=m.BC_NEUMANN_CC)
    else:
        ue, he, *_ = (oracle.solve, oracle.solve_ir_f32, oracle.solve_ir_f16)[precision](z, f, **kw)
    with m.Solver(m.Params(**par)) as s:
        u, fd = torch.zeros(f.shape, dtype=torch.float64, device="cuda"), torch.from_numpy(f).to("cuda")
        _, cyc, h = s.solve(u, fd, tol=0.0, max_cycles=2)
        torch.cuda.synchronize()
    assert cyc == len(he) - 1
    assert np.array_equal(u.cpu().numpy(), ue)
    # two sums of N squares in different orders differ by at most (N - 1) 2^-53 relative each
    np.testing.assert_allclose(h, he, rtol=2.0 * f.size * 2.0**-53)


# many grids: boxes larger than the grid, one box, ragged boxes, one chunk or several
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 3), (3, 2)])
def test_pairs_of_a_batch(nu1, nu2, dev_ok, monkeypatch):
    import torch

    import paper_1406_5369_amd as m

    monkeypatch.setenv("MG_AUTOTUNE", "0")
    monkeypatch.setenv("MG_NO_TAIL", "1")
    edges = [5] * 4 + [9] * 60 + [17] * 60 + [33] * 90 + [65] * 15 + [129] * 3
    fs = [inputs.uniform_rhs(3, n, 500 + i) for i, n in enumerate(edges)]
    ctx = m.mg_batch_setup([m.Params(dim=3, n=n, precision=m.PREC_FP32_IR, nu1=nu1, nu2=nu2) for n in edges])
    try:
        us = [torch.zeros((n,) * 3, dtype=torch.float64, device="cuda") for n in edges]
        m.mg_batch_solve(ctx, us, [torch.from_numpy(f).to("cuda") for f in fs], tol=1e-3, max_cycles=4)
        torch.cuda.synchronize()
        for f, u in zip(fs, us):
            ue, *_ = oracle.solve_ir_f32(np.zeros_like(f), f, tol=1e-3, max_cycles=4, nu1=nu1, nu2=nu2)
            assert np.array_equal(u.cpu().numpy(), ue)
    finally:
        m.mg_destroy(ctx)
