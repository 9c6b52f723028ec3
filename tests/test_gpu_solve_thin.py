"""Flexible CG on grids whose inference runs in few or many blocks for their
size (one column of planes, one plane, one row): its dot partials have room
whatever their number, and the solution is the one of Jacobi-PCG."""
import numpy as np
import pytest

from paper_1301_3925_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(5, 4, 900), (300, 210, 1), (17, 3, 40), (1000, 3), (3, 700),
                                  (400, 330)], ids=lambda d: "x".join(map(str, d)))
def test_learned_solve_matches_jacobi(dims):
    import torch
    import paper_1301_3925_amd as adlbr
    D = (synth.tensor2d_field(4, *dims, 10.0) if len(dims) == 2
         else synth.tensor3d_field(4, dims, 10.0))
    off, w, _ = adlbr.build_stencils(torch.from_numpy(D).cuda(), dims)
    op = adlbr.Operator(dims, off, w)
    dt = 20.0 * op.dt_cfl()
    net = adlbr.Net(op, seed=1)
    net.prepare(dt)
    b = torch.from_numpy(synth.uniform(6, op.N)).float().cuda()
    x, rep = op.solve(b, dt, tol=1e-6)
    y, rep2 = op.solve(b, dt, method="fcg", net=net, tol=1e-6)
    assert rep["converged"] and rep2["converged"]
    # |K^-1| <= 1: either is within its residual of the solution, and FP32's rounding
    assert (x - y).norm() <= (2e-6 + 2.0 ** -22) * b.norm()
