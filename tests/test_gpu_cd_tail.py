"""Complex diffusion on the levels that run in one launch and just above them:
FAS cycles bit for bit against the oracle (every edge the tail takes, both
smoothers, sweep counts down to zero), and equal to the levels launched apart."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu

RB, JAC = 0, 1


def fas(dim, n, u0, f, tau, smoother, nu):
    import math

    import torch

    import paper_1406_5369_amd as m

    ctx = m.mg_cdiff_setup(dim, n, tau, math.pi / 30, 0.1, smoother, 0.0, *nu)
    u, fd = torch.from_numpy(u0).to("cuda"), torch.from_numpy(f).to("cuda")
    for _ in range(2):
        m.mg_cdiff_fas(ctx, u, fd)
    torch.cuda.synchronize()
    m.mg_destroy(ctx)
    return u.cpu().numpy()


@pytest.mark.parametrize("dim,n", [(2, 2), (2, 4), (2, 8), (2, 16), (2, 32), (2, 64), (3, 2), (3, 4), (3, 8), (3, 16)])
@pytest.mark.parametrize("smoother,nu", [(RB, (2, 2)), (JAC, (2, 1)), (RB, (0, 1)), (JAC, (1, 0)), (RB, (3, 0))])
def test_cd_tail(dim, n, smoother, nu, monkeypatch):
    tau = 10.0 / n**2
    u0 = inputs.noisy_image(dim, n, 4) + 1j * inputs.random_cells(dim, n, 5, 0.2)
    f = u0 / tau
    P = oracle.CD(tau=tau, k=0.1)
    exp = u0
    for _ in range(2):
        exp = oracle.cd_fas(exp, f, P, smoother=smoother, omega=0.8 if smoother == JAC else 1.0, nu1=nu[0], nu2=nu[1])
    got = fas(dim, n, u0, f, tau, smoother, nu)
    assert np.array_equal(got, exp)
    monkeypatch.setenv("MG_NO_TAIL", "1")
    assert np.array_equal(fas(dim, n, u0, f, tau, smoother, nu), got)
