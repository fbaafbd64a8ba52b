"""3D red-black sweeps with one wavefront per tile and nodes held by colour:
every box height, chunks of one plane up to more than the grid, grids smaller
than a tile and with ragged last tiles, both colour orders, block orders, with
the correction and from a zero iterate; bit for bit against the oracle."""

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 9, 17, 33, 65, 129])
@pytest.mark.parametrize("dt,by", [(np.float64, 8), (np.float32, 8), (np.float32, 12), (np.float16, 8), (np.float16, 12)])
@pytest.mark.parametrize("zchunk", [1, 3, 8, 200])
@pytest.mark.parametrize("form", ["plain", "black", "correct", "black_correct", "zero"])
def test_pair_sweep_bitwise(n, dt, by, zchunk, form):
    import torch

    import paper_1406_5369_amd as m

    c = float((n - 1) ** 2)
    su, sf = (8.0 / c, 12.0) if dt == np.float16 else (1.0, 50.0)
    u = np.zeros((n,) * 3, dt) if form == "zero" else (inputs.random_guess(3, n, n) * su).astype(dt)
    f = (inputs.uniform_rhs(3, n, n + 1) * sf).astype(dt)
    ec = (inputs.random_guess(3, (n - 1) // 2 + 1, n + 2) * su).astype(dt) if "correct" in form else None
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")  # noqa: E731
    ue = oracle.prolong_correct(u.copy(), ec) if ec is not None else u
    if "black" in form:
        exp = oracle.smooth(ue, f, smoother=oracle.SMOOTH_RBGS_SYM)
    else:
        exp = oracle.smooth(ue, f)
    out = torch.zeros((n,) * 3, dtype=dev(u).dtype, device="cuda")
    m.mg_level_smooth(None if form == "zero" else dev(u), dev(f), out, smoother=2 if "black" in form else 0,
                      ec=None if ec is None else dev(ec), zero_guess=form == "zero", by=by, zchunk=zchunk, waves=1,
                      order=zchunk & 1)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    bits = np.uint16 if dt == np.float16 else (np.uint32 if dt == np.float32 else np.uint64)
    assert np.array_equal((got + dt(0)).view(bits), (exp + dt(0)).view(bits))
