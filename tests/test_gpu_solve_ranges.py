"""The solver's update over its block ranges, and its stops.

Jacobi-PCG against the same recurrence in torch FP64 on the operator's own
apply and diagonal, after a fixed number of iterations: grids of one block,
of ragged ranges (fewer and more than one step of a block's threads, one and
two blocks a CU, a second step of a few points).  Both run in FP64 and differ
in the order of sums alone, so a relative 1e-9 after 12 iterations leaves
three decades over their rounding.
"""
import pytest

from paper_1301_3925_amd import capi, synth

pytestmark = pytest.mark.gpu


def _operator(dims, kappa=20.0):
    import torch
    import paper_1301_3925_amd as adlbr
    D = synth.tensor2d_field(3, *dims, kappa) if len(dims) == 2 else synth.tensor3d_field(3, dims, kappa)
    off, w, _ = adlbr.build_stencils(torch.from_numpy(D).cuda(), dims)
    return adlbr.Operator(dims, off, w, storage=torch.float64)


@pytest.mark.parametrize("dims", [(3, 1), (31, 33), (37, 29, 1), (511, 514), (1031, 1019), (1449, 1451)],
                         ids=lambda d: "x".join(map(str, d)))
def test_update_ranges(dims):
    import torch
    op = _operator(dims)
    dt = 20.0 * op.dt_cfl()
    b = torch.from_numpy(synth.uniform(4, op.N)).cuda()
    iters = 12 if op.N > 3 else 2
    x, rep = op.solve(b, dt, tol=1e-30, max_iter=iters, check_every=5)
    kd = 1.0 + dt * op.diagonal()
    xr, r = torch.zeros_like(b), b.clone()
    z = r / kd
    p, rz = z.clone(), r @ z
    done = 0
    while done < iters and r @ r > 1e-60 * (b @ b):  # the tiniest grid's K is solved exactly
        done += 1
        q = p + dt * op.apply(p)
        a = rz / (p @ q)
        xr += a * p
        r -= a * q
        z = r / kd
        rz, old = r @ z, rz
        p = z + (rz / old) * p
    assert rep["iters"] == done and rep["converged"] == (done < iters)
    assert (x - xr).norm() <= 1e-9 * xr.norm()
    res = (b - x - dt * op.apply(x)).norm() / b.norm()
    assert abs(rep["rel_res"] - res.item()) <= 1e-9


def test_stops():
    """A solve that ends within a batch counts its own iterations whatever the
    batch; a zero right-hand side breaks down at once and leaves x zero."""
    import torch
    op = _operator((96, 80))
    dt = 20.0 * op.dt_cfl()
    b = torch.from_numpy(synth.uniform(4, op.N)).cuda()
    runs = [op.solve(b, dt, tol=1e-6, check_every=c) for c in (1, 7, 200)]
    assert len({r["iters"] for _, r in runs}) == 1 and all(r["converged"] for _, r in runs)
    assert all(torch.equal(runs[0][0], x) for x, _ in runs)
    for c in (1, 10):
        x, rep = op.solve(torch.zeros_like(b), dt, tol=1e-6, max_iter=30, check_every=c)
        assert rep["iters"] == 0 and not rep["converged"] and not x.any()
