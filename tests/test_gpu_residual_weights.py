"""The true residual that a solve reports is that of the weights as given.

x solves (I + dt A) x = b exactly, with every number a small multiple of a
power of two, so the residual of x is 0 in FP64, in any order of its sums.
Along x the weights are 1 at even points and k 2^-24 at odd ones (k = 1, 2,
3); neighbours' edges meet, and 1 + k 2^-24 is an FP32 number only for k = 2:
a residual of pair weights rounded to FP32 is far from 0.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("boundary", ["neumann", "periodic", "reflect"])
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("dims", [(48, 1), (64, 4), (70, 5), (48, 5, 4), (129, 3, 2)],
                         ids=lambda d: "x".join(map(str, d)))
def test_exact_solution_has_no_residual(dims, storage, wide, boundary):
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
    assert np.array_equal(b, b.astype(np.float32).astype(np.float64))  # FP32 numbers
    S = 3 if d == 2 else 6
    off = np.zeros((S, d, n), dtype=np.int16)
    o = np.eye(d, dtype=np.int16)
    slots = [o[0], o[1], -o[0] - o[1]] if d == 2 else \
        [o[0], o[1], o[2], -(o[0] + o[1]), o[0] - o[2], o[1] + o[2]]
    off[:] = np.stack(slots)[:, :, None]
    w = np.zeros((S, n))
    w[0] = np.tile(wx, n // nx)
    td = torch.float32 if storage == "f32" else torch.float64
    op = adlbr.Operator(dims, torch.from_numpy(off).cuda(), torch.from_numpy(w).to(td).cuda(),
                        storage=td, wide=wide, periodic=boundary == "periodic",
                        reflect=boundary == "reflect")
    x = torch.from_numpy(np.tile(u, n // nx)).to(td).cuda()
    rhs = torch.from_numpy(np.tile(b, n // nx)).to(td).cuda()
    # a residual of 0 leaves no direction: the solve ends at once, with x as it was
    got, rep = op.solve(rhs, dt, x=x.clone(), tol=1e-12, max_iter=1)
    assert torch.equal(got, x)
    assert rep["rel_res"] == 0.0
