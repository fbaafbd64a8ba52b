"""Constant-stencil solves at the edges of their kernels' tiles: grids that are
all tail, one level above it, ragged tiles; sweep counts of zero (no sweep to
sum the norm in), every cycle and smoother, two right-hand sides through one
context.  Fields bit for bit against the oracle."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu

RB, JAC, SYM = 0, 1, 2
V, W, F = 0, 1, 2
SKEW = {2: (4.5, -1.1, -0.9, -1.4, -1.1), 3: (7.0, -1.2, -0.8, -1.3, -1.2, -1.4, -1.1)}


@pytest.mark.parametrize("dim,n", [(2, 3), (2, 5), (2, 65), (2, 129), (2, 257), (3, 3), (3, 5), (3, 17), (3, 33), (3, 65)])
@pytest.mark.parametrize("smoother,cycle,nu1,nu2", [(RB, V, 2, 2), (SYM, W, 2, 1), (JAC, F, 1, 2), (RB, V, 0, 2),
                                                    (SYM, V, 3, 0)])
def test_stencil_solve_levels(dim, n, smoother, cycle, nu1, nu2):
    import torch

    import paper_1406_5369_amd as m

    omega = 0.8 if smoother == JAC else 1.0
    with m.Solver(m.Params(dim=dim, n=n, op=m.OP_CONST_STENCIL, stencil=SKEW[dim], smoother=smoother, cycle=cycle,
                           nu1=nu1, nu2=nu2)) as s:
        for seed in (1, 2):
            f = inputs.uniform_rhs(dim, n, seed)
            ue, he, _ = oracle.st_solve(np.zeros_like(f), f, SKEW[dim], tol=0.0, max_cycles=3, smoother=smoother,
                                        omega=omega, nu1=nu1, nu2=nu2, cycle=cycle)
            u, fd = torch.zeros(f.shape, dtype=torch.float64, device="cuda"), torch.from_numpy(f).to("cuda")
            _, cyc, h = s.solve(u, fd, tol=0.0, max_cycles=3)
            torch.cuda.synchronize()
            assert cyc == len(he) - 1
            assert np.array_equal(u.cpu().numpy(), ue)
            # two sums of N squares in different orders differ by at most (N - 1) 2^-53 relative each
            np.testing.assert_allclose(h, he, rtol=max(1e-14, 2.0 * f.size * 2.0**-53))
            norm = s.residual_norm(u, fd)
            np.testing.assert_allclose(norm, he[-1], rtol=max(1e-14, 2.0 * f.size * 2.0**-53))
