"""2D red-black cycles whose levels run each leg in one launch (sweeps with
residual and restriction, correction with sweeps), at the edges of its boxes:
26 x 10 (26 x 26 on many) coarse nodes going down, 56 x 24 (56 x 56) nodes going
up.  Whole solves against the oracle: fields bit for bit."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu

RB, SYM = 0, 2
V, W, F = 0, 1, 2
SKEW = (4.5, -1.1, -0.9, -1.4, -1.1)


def run(op, precision, n, smoother, cycle, nu1, nu2, steps=3):
    import torch

    import paper_1406_5369_amd as m

    f = inputs.uniform_rhs(2, n, 11)
    kw = dict(tol=0.0, max_cycles=steps, smoother=smoother, nu1=nu1, nu2=nu2, cycle=cycle)
    z = np.zeros_like(f)
    par = dict(dim=2, n=n, smoother=smoother, cycle=cycle, nu1=nu1, nu2=nu2, precision=precision)
    if op == "stencil":
        ue, he, _ = oracle.st_solve(z, f, SKEW, **kw)
        par.update(op=m.OP_CONST_STENCIL, stencil=SKEW)
    else:
        k = inputs.varcoef_k(n, 5, dim=2) if op == "varcoef" else None
        solve = (oracle.solve, oracle.solve_ir_f32, oracle.solve_ir_f16)[precision]
        ue, he, *_ = solve(z, f, k=k, **kw)
        if k is not None:
            par.update(op=m.OP_VARCOEF_NODAL, k=torch.from_numpy(k).to("cuda"))
    with m.Solver(m.Params(**par)) as s:
        u, fd = torch.zeros(f.shape, dtype=torch.float64, device="cuda"), torch.from_numpy(f).to("cuda")
        _, cyc, h = s.solve(u, fd, tol=0.0, max_cycles=steps)
        torch.cuda.synchronize()
    assert cyc == len(he) - 1
    assert np.array_equal(u.cpu().numpy(), ue)
    # two sums of N squares in different orders differ by at most (N - 1) 2^-53 relative each
    np.testing.assert_allclose(h, he, rtol=max(1e-14, 2.0 * f.size * 2.0**-53))


# every level a leg (no tail): boxes larger than the grid, one box, ragged boxes
@pytest.mark.parametrize("n", [5, 9, 17, 33, 65, 129, 257])
@pytest.mark.parametrize("op,precision", [("laplace", 0), ("laplace", 1), ("laplace", 2), ("varcoef", 0),
                                          ("varcoef", 1), ("stencil", 0)])
@pytest.mark.parametrize("smoother,cycle,nu1,nu2", [(RB, V, 2, 2), (RB, V, 1, 1), (SYM, V, 2, 1), (RB, V, 3, 3),
                                                    (SYM, W, 1, 2), (RB, F, 4, 1)])
def test_legs_on_every_level(n, op, precision, smoother, cycle, nu1, nu2, dev_ok, monkeypatch):
    monkeypatch.setenv("MG_NO_TAIL", "1")
    run(op, precision, n, smoother, cycle, nu1, nu2)


# one grid that the taller boxes cover (from 1025), with the levels below
@pytest.mark.parametrize("op,precision", [("laplace", 0), ("laplace", 1), ("laplace", 2), ("varcoef", 1),
                                          ("stencil", 0)])
@pytest.mark.parametrize("smoother,nu1,nu2", [(RB, 2, 2), (SYM, 1, 3)])
def test_legs_of_a_large_grid(op, precision, smoother, nu1, nu2, dev_ok):
    run(op, precision, 1025, smoother, V, nu1, nu2, steps=2)


# many grids of a few boxes each: the taller boxes at small edges
def test_legs_of_a_batch(dev_ok, monkeypatch):
    import torch

    import paper_1406_5369_amd as m

    monkeypatch.setenv("MG_NO_TAIL", "1")
    edges = [33, 65, 129] * 90
    fs = [inputs.uniform_rhs(2, n, 300 + i) for i, n in enumerate(edges)]
    ctx = m.mg_batch_setup([m.Params(dim=2, n=n, precision=m.PREC_FP32_IR) for n in edges])
    try:
        us = [torch.zeros((n, n), dtype=torch.float64, device="cuda") for n in edges]
        m.mg_batch_solve(ctx, us, [torch.from_numpy(f).to("cuda") for f in fs], tol=1e-6, max_cycles=20)
        torch.cuda.synchronize()
        for f, u in zip(fs, us):
            ue, *_ = oracle.solve_ir_f32(np.zeros_like(f), f, tol=1e-6, max_cycles=20)
            assert np.array_equal(u.cpu().numpy(), ue)
    finally:
        m.mg_destroy(ctx)
