"""Training kernels at the edges of their tiles against the FP64 oracle.

The convolutions walk tiles of 64 x 4 (2D) and 32 x 4 x 4 (3D) points, the
weight gradients 64 x 4 and 32 x 4 x 2, the gate net 256 points: one point,
exactly one tile, one more in each direction, and more tiles than blocks (so
that blocks walk several).  Tolerances as for the network's parity: forward
1e-5, gradients 1e-4 relative L2 (FP32 sums against FP64).
"""
import numpy as np
import pytest

import oracle
from oracle import solvers
from paper_1301_3925_amd import synth

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(np.ravel(a) - np.ravel(b)) / max(np.linalg.norm(np.ravel(b)), 1e-300))


@pytest.mark.parametrize("dims", [(2, 1), (64, 4), (65, 5), (63, 9), (700, 300),
                                  (32, 4, 4), (33, 5, 3), (31, 9, 5), (100, 64, 48)],
                         ids=lambda d: "x".join(map(str, d)))
def test_forward_and_gradients(dims):
    import torch
    import paper_1301_3925_amd as adlbr
    dim = len(dims)
    D = synth.tensor2d_field(3, *dims, 20.0) if dim == 2 else synth.tensor3d_field(4, dims, 20.0)
    off, w, _ = adlbr.build_stencils(torch.from_numpy(D).cuda(), dims)
    op = adlbr.Operator(dims, off, w, storage=torch.float32)
    w32 = w.float().double().cpu().numpy()
    diag = op.diagonal().cpu().numpy()
    dt = 50.0 / float(diag.max())
    flat = solvers.net_pack(solvers.net_init(5, dim), dim).astype(np.float32)
    P = solvers.net_unpack(flat.astype(np.float64), dim)
    F = solvers.net_features(dims, off.cpu().numpy(), w32, diag, dt)
    net = adlbr.Net(op, params=torch.from_numpy(flat))
    net.prepare(dt)
    rng = np.random.default_rng(7)
    r = rng.normal(size=op.N).astype(np.float32)
    gz = rng.normal(size=op.N).astype(np.float32)
    G = solvers.net_gates(P, F)
    q = np.rint(255.0 * G.reshape(32, -1)).T
    assert np.abs(net.gates8.cpu().numpy().astype(float) - q).max() <= 1  # a tie either way
    saved = torch.empty((49, op.N), device="cuda")
    rt = torch.from_numpy(r).cuda()
    z = net.forward(rt, saved=saved)
    ref = solvers.net_precondition(P, G, r.astype(np.float64), 1.0 + dt * diag)
    assert _rel(z.double().cpu().numpy(), ref) <= 1e-5
    # both gradients are added to what is there
    gp = torch.full((net.nparams,), 0.5, device="cuda")
    gg = torch.zeros((49, op.N), device="cuda")
    net.backward(rt, torch.from_numpy(gz).cuda(), saved, gp, gg)
    net.gates_backward(gg, gp)
    got = solvers.net_unpack(gp.double().cpu().numpy() - 0.5, dim)
    want = solvers.net_backward(P, F, r.astype(np.float64), gz.astype(np.float64))
    # the start of 0.5 leaves its rounding on every parameter
    for name in want:
        err = np.linalg.norm(got[name] - want[name])
        assert err <= 1e-4 * np.linalg.norm(want[name]) + 6e-8 * np.sqrt(got[name].size), name
