"""The training loss of a small merged operator against the same operator
without merged pairs (2D, where a workspace that holds only the plain layout
keeps every edge listed), for grids of one block and more, of one row, folded
edges and wide offsets.  A row has at most some twenty FP32 products, so the
gradients agree to 20 units of 2^-24 (1.2e-6); the losses sum at least 40
such rows in FP64 (2e-7)."""
import ctypes

import pytest

from paper_1301_3925_amd import capi, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,kappa,periodic,wide", [
    ((64, 67), 20.0, False, False), ((40, 1), 3.0, False, False), ((33, 31), 200.0, True, False),
    ((96, 50), 50.0, False, True), ((150, 101), 5.0, True, True)])
def test_loss_matches_plain(dims, kappa, periodic, wide):
    import torch
    import paper_1301_3925_amd as adlbr
    D = synth.tensor2d_field(7, *dims, kappa)
    off, w, _ = adlbr.build_stencils(torch.from_numpy(D).cuda(), dims)
    out = []
    for plain in (False, True):
        ws = None
        if plain:
            nb = ctypes.c_size_t()
            g = adlbr.grid(dims, periodic, False)
            capi.check(capi.load().adlbr_operator_workspace(ctypes.byref(g), capi.F32,
                                                            capi.OP_WIDE if wide else 0, ctypes.byref(nb)))
            ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
        op = adlbr.Operator(dims, off, w, storage=torch.float32, periodic=periodic, wide=wide, workspace=ws)
        assert (op.workspace is ws) == plain
        dt = 50.0 * op.dt_cfl() if not out else dt
        net = adlbr.Net(op, seed=2)
        net.prepare(dt)
        r = torch.from_numpy(synth.uniform(8, op.N) - 0.5).float().cuda()
        z = torch.from_numpy(synth.uniform(9, op.N) - 0.5).float().cuda()
        gz, loss = torch.empty_like(z), torch.zeros(1, dtype=torch.float64, device="cuda")
        net.loss_grad(dt, r, z, gz, loss)
        out.append((gz, loss.item()))
    (g0, l0), (g1, l1) = out
    assert (g0 - g1).norm() <= 1.2e-6 * g1.norm()
    assert abs(l0 - l1) <= 2e-7 * abs(l1)
