"""Cell-centred solves at the edges of their kernels: grids that are all tail,
one level above it, ragged tiles; every cycle and smoother, sweep counts of
zero (no sweep to subtract the mean and sum the norm in), starting guesses with
a mean, two right-hand sides through one context, solves of zero cycles.  The
iterates bit for bit against the oracle."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu

RB, JAC = 0, 1
V, W, F = 0, 1, 2


@pytest.mark.parametrize("dim,n", [(2, 2), (2, 4), (2, 32), (2, 64), (2, 128), (2, 256), (2, 2048), (3, 2), (3, 4), (3, 8),
                                   (3, 16), (3, 32), (3, 64)])
@pytest.mark.parametrize("smoother,cycle,nu1,nu2,cycles", [(RB, V, 2, 2, 3), (JAC, W, 1, 2, 2), (RB, F, 1, 1, 3),
                                                           (RB, W, 0, 2, 2), (RB, V, 3, 0, 2), (JAC, V, 2, 1, 2),
                                                           (RB, V, 2, 2, 0)])
def test_cc_solve_levels(dim, n, smoother, cycle, nu1, nu2, cycles):
    import torch

    import paper_1406_5369_amd as m

    omega = 0.8 if smoother == JAC else 1.0
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")  # noqa: E731
    with m.Solver(m.Params(dim=dim, n=n, bc=m.BC_NEUMANN_CC, smoother=smoother, cycle=cycle, nu1=nu1, nu2=nu2)) as s:
        for seed in (1, 2):
            f, u0 = inputs.random_cells(dim, n, seed) + 0.25, inputs.random_cells(dim, n, seed + 7) + 0.5
            ue, he, _, _ = oracle.cc_solve(u0, f, tol=0.0, max_cycles=cycles, smoother=smoother, omega=omega, nu1=nu1,
                                           nu2=nu2, cycle=cycle)
            u = dev(u0)
            _, cyc, h = s.solve(u, dev(f), tol=0.0, max_cycles=cycles)
            torch.cuda.synchronize()
            assert cyc == len(he) - 1
            assert np.array_equal(u.cpu().numpy(), ue)
            # two sums of N squares in different orders differ by at most (N - 1) 2^-53 relative each
            np.testing.assert_allclose(h, he, rtol=max(1e-13, 2.0 * f.size * 2.0**-53))


@pytest.mark.parametrize("dim,n", [(2, 2), (2, 128), (2, 1024), (2, 8192), (3, 2), (3, 64), (3, 256)])
def test_cc_mean_order(dim, n):
    import torch

    import paper_1406_5369_amd as m

    v = inputs.random_cells(dim, n, 3) * 1e3 + 0.1
    vd = torch.from_numpy(v).to("cuda")
    mean = m.mg_level_cc_remove_mean(vd)
    assert mean == oracle.cc_sum(v) / v.size
    assert np.array_equal(vd.cpu().numpy(), v - mean)
