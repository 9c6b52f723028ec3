"""Non-finite values of u in A u and in a step: where they reach.

Every edge in the grid carries its difference, also one of weight 0
(0 times infinity is NaN); an edge that leaves the grid or folds onto the
point has the difference of the point to itself.  The classes (finite, NaN,
+inf, -inf) of all rows are those of the definition taken term by term.
"""
import ctypes

import numpy as np
import pytest

from paper_1301_3925_amd import synth

pytestmark = pytest.mark.gpu


def _apply(dims, off, w, u, boundary):
    """A u term by term, in FP64."""
    idx, d, nd = np.arange(u.size), len(dims), np.array(dims)[:, None]
    p = np.stack([(idx // int(np.prod(dims[:c]))) % dims[c] for c in range(d)])
    out = np.zeros(u.size)
    for q in range(w.shape[0]):
        for s in (-1, 1):
            t = p + s * off[q].astype(np.int64)
            if boundary == "periodic":
                t %= nd
            elif boundary == "reflect":
                t %= 2 * nd
                t = np.where(t < nd, t, 2 * nd - 1 - t)
            ok = np.all((t >= 0) & (t < nd), axis=0)
            lin = np.where(ok, sum(t[c] * int(np.prod(dims[:c])) for c in range(d)), idx)
            ok &= lin != idx
            out += w[q] * (u - u[lin])
            ok &= w[q] > 0
            np.add.at(out, lin[ok], (w[q] * (u[lin] - u))[ok])
    return out


def _classes(a):
    return np.where(np.isnan(a), 1, np.where(np.isposinf(a), 2, np.where(np.isneginf(a), 3, 0)))


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16", "f16"])
@pytest.mark.parametrize("boundary", ["neumann", "periodic", "reflect"])
@pytest.mark.parametrize("dims,plain", [((70, 45), False), ((70, 45), True), ((64, 8), False),
                                        ((64, 8), True), ((20, 17, 15), False)])
def test_classes_of_rows(dims, plain, boundary, dtype):
    import torch
    import paper_1301_3925_amd as adlbr
    from paper_1301_3925_amd import capi
    n, d = int(np.prod(dims)), len(dims)
    td = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16,
          "f16": torch.float16}[dtype]
    D = np.zeros((3 if d == 2 else 6, n))  # half the slots of a diagonal tensor weigh 0
    D[0], D[2 if d == 2 else 3] = 1.0, 2.0
    if d == 3:
        D[5] = 3.0
    off, w, _ = adlbr.build_stencils(torch.from_numpy(D).cuda(), dims)
    assert (w == 0).any() and (w > 0).any()
    kw = {"periodic": boundary == "periodic", "reflect": boundary == "reflect"}
    ws = None
    if plain:
        nb = ctypes.c_size_t()
        code = {"f64": capi.F64, "f32": capi.F32, "bf16": capi.BF16, "f16": capi.F16}[dtype]
        capi.check(capi.load().adlbr_operator_workspace(ctypes.byref(adlbr.grid(dims, **kw)), code,
                                                        0, ctypes.byref(nb)))
        ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
    op = adlbr.Operator(dims, off, w, storage=td, workspace=ws, **kw)
    u = torch.from_numpy(synth.uniform(3, n)).to(td).cuda()
    u[n // 2], u[n // 3], u[0], u[n - 1] = np.nan, np.inf, np.inf, -np.inf
    h, uh = off.cpu().numpy(), u.double().cpu().numpy()
    with np.errstate(invalid="ignore"):
        ref = _apply(dims, h, w.cpu().numpy(), uh, boundary)
        step = uh - 0.01 * ref
    assert np.array_equal(_classes(op.apply(u).double().cpu().numpy()), _classes(ref))
    got = op.step(u.clone(), 0.01, 1)
    assert np.array_equal(_classes(got.double().cpu().numpy()), _classes(step))
    um = torch.stack([u, u.flip(0), u])
    multi = op.step_multi(um, 0.01, 1)
    assert np.array_equal(_classes(multi[2].double().cpu().numpy()), _classes(step))
