"""mg_vcycle of constant-stencil and cell-centred contexts is launches only: a
program may capture it in a HIP graph, with arrays the context has not seen, and
each replay works on the captured arrays while eager calls in between work on
theirs.  Every result bit for bit against cycles of a context of its own."""

import numpy as np
import pytest

import inputs

pytestmark = pytest.mark.gpu

RB, JAC = 0, 1
SKEW = {2: (4.5, -1.1, -0.9, -1.4, -1.1), 3: (7.0, -1.2, -0.8, -1.3, -1.2, -1.4, -1.1)}


@pytest.mark.parametrize("kind,dim,n", [("stencil", 2, 3), ("stencil", 2, 129), ("stencil", 3, 33), ("cells", 2, 128),
                                        ("cells", 3, 32)])
@pytest.mark.parametrize("smoother,nu1,nu2", [(RB, 2, 2), (JAC, 2, 1)])
def test_captured_vcycle(kind, dim, n, smoother, nu1, nu2, dev_ok):
    import torch

    import paper_1406_5369_amd as m

    side = torch.cuda.Stream()
    par = dict(dim=dim, n=n, smoother=smoother, nu1=nu1, nu2=nu2)
    par.update(dict(op=m.OP_CONST_STENCIL, stencil=SKEW[dim]) if kind == "stencil" else dict(bc=m.BC_NEUMANN_CC))
    make = inputs.random_cells if kind == "cells" else inputs.uniform_rhs
    fs = [torch.from_numpy(make(dim, n, 50 + i)).to("cuda") for i in range(2)]
    with torch.cuda.stream(side):
        expect = []  # iterates after 1, 2, 3 cycles of each right-hand side
        with m.Solver(m.Params(**par)) as ref:
            for f in fs:
                u, got = torch.zeros_like(f), []
                for _ in range(3):
                    ref.vcycle(u, f)
                    got.append(u.clone())
                expect.append(got)
        with m.Solver(m.Params(**par)) as s:
            us = [torch.zeros_like(f) for f in fs]
            side.synchronize()
            graph = torch.cuda.CUDAGraph()
            graph.capture_begin()
            s.vcycle(us[0], fs[0])
            graph.capture_end()
            for i in range(3):
                graph.replay()
                s.vcycle(us[1], fs[1])
                side.synchronize()
                for u, e in zip(us, expect):
                    assert np.array_equal(u.cpu().numpy(), e[i].cpu().numpy())
            del graph
