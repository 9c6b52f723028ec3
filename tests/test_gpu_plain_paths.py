"""2D operators without merged pairs (a workspace of the plain size) on every
path that takes them: steps of several components, batches with and without
merged operators beside them, the Jacobi-PCG solve, the residual, the loss.
Against the FP64 oracle, and bit for bit against the single calls where those
share the arithmetic."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1301_3925_amd import capi, synth

pytestmark = pytest.mark.gpu

CASES = [((70, 45), "neumann", False), ((64, 32), "neumann", True), ((33, 90), "periodic", False),
         ((52, 41), "reflect", True)]


def _operator(dims, boundary, wide, td, plain=True, seed=7):
    import torch
    import paper_1301_3925_amd as adlbr
    kw = {"periodic": boundary == "periodic", "reflect": boundary == "reflect"}
    off, w, _ = adlbr.build_stencils(
        torch.from_numpy(synth.tensor2d_field(seed, *dims, 15.0)).cuda(), dims)
    w = w.to(td)
    ws = None
    if plain:
        nb = ctypes.c_size_t()
        capi.check(capi.load().adlbr_operator_workspace(
            ctypes.byref(adlbr.grid(dims, **kw)), capi.F64 if td == torch.float64 else capi.F32,
            capi.OP_WIDE if wide else 0, ctypes.byref(nb)))
        ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
    op = adlbr.Operator(dims, off, w, storage=td, wide=wide, workspace=ws, **kw)
    assert (op.workspace is ws) == plain
    A = oracle.operator_matrix(dims, off.cpu().numpy(), w.double().cpu().numpy(), **kw)
    return op, A


def _image(td, op, seed=3):
    import torch
    return torch.from_numpy(synth.uniform(seed, op.N)).to(td).cuda()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("dims,boundary,wide", CASES)
def test_components_and_oracle(dims, boundary, wide, dtype):
    import torch
    td = torch.float64 if dtype == "f64" else torch.float32
    op, A = _operator(dims, boundary, wide, td)
    u = torch.stack([_image(td, op, s) for s in (3, 4, 5, 6, 7)])
    dt, steps = 0.8 * op.dt_cfl(), 7
    single = [c.clone() for c in u]
    for c in single:
        op.step(c, dt, steps)
    got = op.step_multi(u.clone(), dt, steps)
    assert torch.equal(got, torch.stack(single))
    # a step maps [0, 1] into itself and rounds its dozen terms: at most some
    # 40 units of the last place each
    eps = 40 * steps * (2.0 ** -53 if dtype == "f64" else 2.0 ** -24)
    for c, g in zip(u, got):
        ref = oracle.explicit_steps(A, c.double().cpu().numpy(), dt, steps)
        assert np.abs(g.double().cpu().numpy() - ref).max() <= eps


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_batch_of_plain_and_merged(dtype, graph):
    import torch
    import paper_1301_3925_amd as adlbr
    td = torch.float64 if dtype == "f64" else torch.float32
    ops = [_operator(dims, bnd, wide, td, plain=k % 2 == 0, seed=20 + k)[0]
           for k, (dims, bnd, wide) in enumerate(CASES + CASES[1:])]
    us = [_image(td, op, 30 + k) for k, op in enumerate(ops)]
    ref = [u.clone() for u in us]
    for op, u in zip(ops, ref):
        op.step(u, 0.9, 12, cfl_fraction=True)
    b = adlbr.Batch(ops, us, dt=0.9, dt_mode="cfl")
    assert {v["class"] // 10000 for v in b.variants()} == {0, 2}
    b.run(5, graph=graph)
    b.run(5, graph=graph)
    b.run(2, graph=graph)
    torch.cuda.synchronize()
    for u, r in zip(us, ref):
        assert torch.equal(u, r)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("dims,boundary,wide", CASES)
def test_solve_and_residual(dims, boundary, wide, dtype):
    import torch
    import scipy.sparse as sp
    from scipy.sparse.linalg import spsolve
    import paper_1301_3925_amd as adlbr
    td = torch.float64 if dtype == "f64" else torch.float32
    op, A = _operator(dims, boundary, wide, td)
    dt = 30.0 * op.dt_cfl()
    K = (sp.identity(op.N) + dt * A).tocsc()
    b = _image(td, op)
    bh = b.double().cpu().numpy()
    tol = 1e-11 if dtype == "f64" else 1e-6
    x, rep = op.solve(b, dt, tol=tol)
    assert rep["converged"] and rep["rel_res"] <= tol
    ref = spsolve(K, bh)
    eps = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    xh = x.double().cpu().numpy()
    # |K^-1| <= 1, so x is within its residual of the solution; FP32 rounds it
    assert np.linalg.norm(xh - ref) <= 2 * tol * np.linalg.norm(bh) + eps * np.linalg.norm(ref)
    r = adlbr.residual(op, b, x, dt).double().cpu().numpy()
    # dt, then a product, a difference and an addition for each of up to 255 + 6 edges;
    # the sums stay within a tenth of them on these fields
    mag = abs(bh) + abs(K) @ abs(xh)
    assert np.all(abs(r - (bh - K @ xh)) <= 32 * eps * mag)


@pytest.mark.parametrize("dims,boundary,wide", CASES)
def test_loss_and_gradient(dims, boundary, wide):
    import torch
    import paper_1301_3925_amd as adlbr
    op, A = _operator(dims, boundary, wide, torch.float32)
    dt = 30.0 * op.dt_cfl()
    net = adlbr.Net(op)
    r, z = _image(torch.float32, op, 8) - 0.5, _image(torch.float32, op, 9) - 0.5
    gz, loss = torch.empty_like(z), torch.zeros(1, dtype=torch.float64, device="cuda")
    net.loss_grad(dt, r, z, gz, loss)
    rh, zh = r.double().cpu().numpy(), z.double().cpu().numpy()
    Kz, rr = zh + dt * (A @ zh), rh @ rh
    eps = 32 * 2.0 ** -24
    mag = (abs(zh) + dt * (abs(A) @ abs(zh)) + abs(rh)) / rr
    assert np.all(abs(gz.double().cpu().numpy() - (Kz - rh) / rr) <= eps * mag)
    ref = (0.5 * zh @ Kz - zh @ rh) / rr
    assert abs(loss.item() - ref) <= eps * (abs(zh) @ mag)
