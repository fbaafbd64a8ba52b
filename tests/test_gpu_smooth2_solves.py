"""2D solves and batches whose levels run the two-sweep launches (from zero, and
with the correction) instead of whole legs, as levels above the legs' largest edge
do: every level, or only those above an edge with legs below; forced on, off, and
as tuned.  Fields bit for bit against the oracle."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu

RB, SYM = 0, 2
V, W, F = 0, 1, 2
FORCED = {"MG_FUSED_SMOOTH2": "1", "MG_FUSED_POST2": "1"}


def solve(n, precision, smoother=RB, cycle=V, nu1=2, nu2=2, steps=4, prof=False):
    import torch

    import paper_1406_5369_amd as m

    f = inputs.uniform_rhs(2, n, 5)
    ref = oracle.solve_ir_f32 if precision == 1 else oracle.solve_ir_f16
    ue, he, *_ = ref(np.zeros_like(f), f, tol=0.0, max_cycles=steps, smoother=smoother, cycle=cycle, nu1=nu1, nu2=nu2)
    with m.Solver(m.Params(dim=2, n=n, precision=precision, smoother=smoother, cycle=cycle, nu1=nu1, nu2=nu2)) as s:
        pair = [m.mg_tile_config(s.ctx, 0, family)[1] > 0 for family in (7, 8)]
        fd = torch.from_numpy(f).to("cuda")
        u = torch.zeros_like(fd)
        m.mg_prof_enable(s.ctx, prof)
        _, cyc, h = s.solve(u, fd, tol=0.0, max_cycles=steps)
        sweeps = m.mg_prof_read(s.ctx, 0)[0]
    assert cyc == len(he) - 1
    assert np.array_equal(u.cpu().numpy(), ue)
    # two sums of N squares in different orders differ by at most (N - 1) 2^-53 relative each
    np.testing.assert_allclose(h, he, rtol=max(1e-14, 2.0 * f.size * 2.0**-53))
    return pair, sweeps


@pytest.mark.parametrize("edge", ["0", "129"])  # no legs; legs on the levels up to 129
@pytest.mark.parametrize("n,precision", [(257, 2), (513, 1), (1025, 1)])
@pytest.mark.parametrize("env", [{}, FORCED, {"MG_NO_FUSED_SMOOTH2": "1"}, {"MG_NO_FUSED_POST2": "1"},
                                 {"MG_FUSED_POST2": "1", "MG_NO_FUSED_SMOOTH2": "1"}])
def test_solves_with_and_without_the_pairs(edge, n, precision, env, dev_ok, monkeypatch):
    monkeypatch.setenv("MG_LEG_MAX_EDGE", edge)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    pair, _ = solve(n, precision)
    if env == FORCED:
        assert pair == [True, True]


# every parity of the sweeps around the pairs, black first after the correction, second visits of a level
@pytest.mark.parametrize("edge", ["0", "129"])
@pytest.mark.parametrize("smoother,cycle", [(RB, V), (SYM, V), (SYM, W), (RB, F)])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (2, 3), (3, 2), (3, 3), (2, 4), (1, 2), (2, 1), (4, 5)])
def test_sweep_counts_around_the_pairs(edge, smoother, cycle, nu1, nu2, dev_ok, monkeypatch):
    monkeypatch.setenv("MG_LEG_MAX_EDGE", edge)
    for k, v in FORCED.items():
        monkeypatch.setenv(k, v)
    solve(257, 1, smoother, cycle, nu1, nu2, steps=3)


# plain finest-level sweeps a step: all but the pair from zero and the pair with the correction
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (2, 3), (3, 3), (2, 4), (2, 5), (4, 3)])
def test_pairs_run_whatever_the_sweep_counts(nu1, nu2, dev_ok, monkeypatch):
    for k, v in dict(FORCED, MG_LEG_MAX_EDGE="0").items():
        monkeypatch.setenv(k, v)
    pair, sweeps = solve(257, 1, nu1=nu1, nu2=nu2, steps=3, prof=True)
    assert pair == [True, True]
    assert sweeps == 3 * (nu1 - 2 + nu2 - 2)


def test_batch_with_the_pairs(dev_ok, monkeypatch):
    import torch

    import paper_1406_5369_amd as m

    for k, v in dict(FORCED, MG_LEG_MAX_EDGE="65").items():
        monkeypatch.setenv(k, v)
    edges = [65, 129, 33, 257, 65, 9, 129, 513]
    fs = [inputs.uniform_rhs(2, n, 730 + i) for i, n in enumerate(edges)]
    ctx = m.mg_batch_setup([m.Params(dim=2, n=n, precision=m.PREC_FP32_IR) for n in edges])
    try:
        us = [torch.zeros((n, n), dtype=torch.float64, device="cuda") for n in edges]
        m.mg_batch_solve(ctx, us, [torch.from_numpy(f).to("cuda") for f in fs], tol=1e-8, max_cycles=40)
        torch.cuda.synchronize()
        for f, u in zip(fs, us):
            ue, *_ = oracle.solve_ir_f32(np.zeros_like(f), f, tol=1e-8, max_cycles=40)
            assert np.array_equal(u.cpu().numpy(), ue)
    finally:
        m.mg_destroy(ctx)
