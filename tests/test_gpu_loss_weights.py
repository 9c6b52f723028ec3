"""The training loss sums rows of K z with every weight as it was given, in
one order, at every size.

First a z with K z = r in numbers that FP32 rows hold exactly, with weights 1
and k 2^-24 whose pair sums FP32 does not hold: the gradient must be 0.  Then,
in 2D, loss and gradient of a merged operator against one that lists every
edge (a workspace of the plain size): the same bits.  Sizes below and above
2^16 points.
"""
import ctypes

import numpy as np
import pytest

from paper_1301_3925_amd import capi, synth

pytestmark = pytest.mark.gpu


def _loss(op, dt, r, z):
    import torch
    import paper_1301_3925_amd as adlbr
    net = adlbr.Net(op)
    gz, loss = torch.empty_like(z), torch.zeros(1, dtype=torch.float64, device="cuda")
    net.loss_grad(dt, r, z, gz, loss)
    return gz, loss.item()


@pytest.mark.parametrize("boundary", ["neumann", "periodic", "reflect"])
@pytest.mark.parametrize("dims", [(48, 5), (64, 1032), (48, 5, 4), (48, 40, 36)],
                         ids=lambda d: "x".join(map(str, d)))
def test_exact_solution_has_no_gradient(dims, boundary):
    import torch
    import paper_1301_3925_amd as adlbr
    nx, d = dims[0], len(dims)
    n = int(np.prod(dims))
    k = np.random.default_rng(5).integers(1, 4, nx).astype(np.float64)
    a, p, c = 6, 22, 38  # a tent of slope 1 on [a, c], its kinks on edges of k = 2
    k[[a + 1, p - 1, p + 1, c - 1]] = 2.0
    wx = np.where(np.arange(nx) % 2 == 0, 1.0, k * 2.0 ** -24)
    e = wx[:-1] + wx[1:]
    u = np.maximum(0.0, (p - a) - abs(np.arange(nx) - float(p)))
    Au = np.zeros(nx)
    Au[:-1] += e * (u[:-1] - u[1:])
    Au[1:] += e * (u[1:] - u[:-1])
    dt = 2.0 ** 24
    b = u + dt * Au
    S = 3 if d == 2 else 6
    off = np.zeros((S, d, n), dtype=np.int16)
    o = np.eye(d, dtype=np.int16)
    off[:] = np.stack([o[0], o[1], -o[0] - o[1]] if d == 2 else
                      [o[0], o[1], o[2], -(o[0] + o[1]), o[0] - o[2], o[1] + o[2]])[:, :, None]
    w = np.zeros((S, n))
    w[0] = np.tile(wx, n // nx)
    op = adlbr.Operator(dims, torch.from_numpy(off).cuda(), torch.from_numpy(w).float().cuda(),
                        periodic=boundary == "periodic", reflect=boundary == "reflect")
    z, r = np.tile(u, n // nx), np.tile(b, n // nx)
    gz, loss = _loss(op, dt, torch.from_numpy(r).float().cuda(), torch.from_numpy(z).float().cuda())
    assert not gz.any()
    ref = -0.5 * (z @ r) / (r @ r)
    assert abs(loss - ref) <= 1e-12 * abs(ref)


@pytest.mark.parametrize("dims,kappa,boundary,wide", [
    ((64, 67), 20.0, "neumann", False), ((33, 31), 200.0, "periodic", True),
    ((256, 256), 50.0, "neumann", False), ((257, 300), 50.0, "reflect", False),
    ((301, 250), 10.0, "periodic", False)])
def test_same_bits_as_complete_lists(dims, kappa, boundary, wide):
    import torch
    import paper_1301_3925_amd as adlbr
    kw = {"periodic": boundary == "periodic", "reflect": boundary == "reflect"}
    off, w, _ = adlbr.build_stencils(
        torch.from_numpy(synth.tensor2d_field(7, *dims, kappa)).cuda(), dims)
    nb = ctypes.c_size_t()
    capi.check(capi.load().adlbr_operator_workspace(ctypes.byref(adlbr.grid(dims, **kw)), capi.F32,
                                                    capi.OP_WIDE if wide else 0, ctypes.byref(nb)))
    ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
    merged = adlbr.Operator(dims, off, w, wide=wide, **kw)
    plain = adlbr.Operator(dims, off, w, wide=wide, workspace=ws, **kw)
    assert plain.workspace is ws and merged.workspace.numel() > nb.value
    r = torch.from_numpy(synth.uniform(8, plain.N) - 0.5).float().cuda()
    z = torch.from_numpy(synth.uniform(9, plain.N) - 0.5).float().cuda()
    dt = 50.0 * plain.dt_cfl()
    (g0, l0), (g1, l1) = _loss(merged, dt, r, z), _loss(plain, dt, r, z)
    assert torch.equal(g0, g1) and l0 == l1
