"""mg_norm_launch names the launch that a solve's event brackets time: its form by
operator, size and sweep counts, with the workgroups of the kernel traces."""

import pytest


pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("par,form,sweeps,blocks", [
    (dict(dim=2, n=129), "leg", 2, 3 * 7),            # 64 coarse columns and rows in boxes of 26 x 10
    (dict(dim=2, n=129, nu1=1), "leg", 1, 3 * 7),
    (dict(dim=2, n=1025), "leg", 2, 20 * 20),         # boxes of 26 x 26
    (dict(dim=2, n=129, nu1=3), "sweep", 1, None),
    (dict(dim=2, n=129, nu2=0), "sweep", 1, None),
    (dict(dim=3, n=257), "pair", 2, 5 * 11 * 4),      # 255 nodes in boxes of 56 x 24, chunks of 64 planes
    (dict(dim=3, n=257, nu1=1), "sweep", 1, None),
    (dict(dim=3, n=65), "sweep", 1, None),
    (dict(dim=3, n=65, nu1=0), "pass", 0, None),
    (dict(dim=3, n=65, precision=1), "pass", 0, None),
    (dict(dim=2, n=128, cells=True), "sweep", 1, None),
])
def test_norm_launch(par, form, sweeps, blocks, dev_ok, monkeypatch):
    import torch

    import paper_1406_5369_amd as m

    monkeypatch.setenv("MG_AUTOTUNE", "0")
    par = dict(par)
    if par.pop("cells", False):
        par["bc"] = m.BC_NEUMANN_CC
    with m.Solver(m.Params(**par)) as s:
        got = m.mg_norm_launch(s.ctx)
        assert (got["form"], got["sweeps"]) == (form, sweeps)
        assert got["blocks"] == blocks if blocks else got["blocks"] > 0
        if form == "pass" and par.get("precision"):
            assert (got["by"], got["zchunk"], got["prefetch"], got["waves"]) == m.mg_tile_config(s.ctx, 0, 2)
        if form == "sweep" and "bc" not in par:
            assert (got["by"], got["zchunk"], got["prefetch"], got["waves"]) == m.mg_tile_config(s.ctx, 0, 6)
    ctx = m.mg_cdiff_setup(2, 16, 0.1)
    try:
        with pytest.raises(m.MGError):
            m.mg_norm_launch(ctx)
    finally:
        m.mg_destroy(ctx)
