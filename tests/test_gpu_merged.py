"""Merged pairs of opposite edges against the oracle's operator.

Random stencils of short offsets, drawn per point from few vectors, so that
about half of the edges meet their opposite at the target; equal and zero
slots, zero weights and edges that leave the grid are among them.  The same
operator without merging (a workspace that only holds the plain lists) must
agree as well.
"""
import ctypes

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _stencils(dims, seed):
    """int16 offsets [S, d, N] with the superbase relations, weights [S, N];
    each component -2..2, few distinct vectors, a fifth of the weights 0."""
    rng = np.random.default_rng(seed)
    n, d = int(np.prod(dims)), len(dims)
    base = rng.integers(-2, 3, size=(5, 3, d))
    base[0] = 0                                            # zero offsets
    base[1, 1] = base[1, 0]                                # two equal slots
    # runs of points share their stencil, so that neighbours often agree
    pick = base[np.repeat(rng.integers(0, 5, n // 6 + 1), 6)[:n]]
    a, b, c = pick[:, 0], pick[:, 1], pick[:, 2]
    o = [a, b, -a - b] if d == 2 else [a, b, c, -(a + b), a - c, b + c]
    off = np.stack(o).transpose(0, 2, 1).astype(np.int16)  # [S, d, N]
    w = rng.uniform(0.1, 1.0, (off.shape[0], n)) * (rng.random((off.shape[0], n)) > 0.2)
    w[:, (off == 0).all(1).any(0)] *= rng.random() > 0.5   # zero offsets with and without weight
    return np.ascontiguousarray(off), w


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16", "f16"])
@pytest.mark.parametrize("boundary", ["neumann", "periodic", "reflect"])
@pytest.mark.parametrize("dims", [(5, 3), (64, 4), (65, 9), (129, 70), (7, 5, 3), (64, 4, 2),
                                  (33, 17, 9)], ids=lambda d: "x".join(map(str, d)))
def test_merged_operator_against_oracle(dims, boundary, dtype):
    import torch
    import paper_1301_3925_amd as adlbr
    from paper_1301_3925_amd import capi
    td = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16,
          "f16": torch.float16}[dtype]
    kw = {"periodic": boundary == "periodic", "reflect": boundary == "reflect"}
    off, w = _stencils(dims, 7 + len(dims))
    og, wg = torch.from_numpy(off).cuda(), torch.from_numpy(w).cuda()
    u = torch.from_numpy(np.random.default_rng(3).uniform(-1, 1, w.shape[1])).to(td).cuda()
    if dtype != "f64":
        wg = wg.float()  # one rounding to the storage type
    # the weights and u as the operator holds them
    held = wg.to(td).double().cpu().numpy()
    # a zero offset's edge joins a point to itself and adds nothing; the oracle
    # would add and subtract its weight on the diagonal, and keep the rounding
    A = oracle.operator_matrix(dims, off, held * ~(off == 0).all(1), **kw)
    uh = u.double().cpu().numpy()
    ref, mag = A @ uh, abs(A) @ abs(uh)
    # at most 12 own terms and the row's list, each with a product, a
    # difference, a weight sum and an addition rounded; then the storage
    eps = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    out = {"f64": 0.0, "f32": 0.0, "bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype]
    terms = np.diff(A.indptr) * 2 + 8
    tol = 4 * terms * eps * mag + out * (abs(ref) + 4 * terms * eps * mag) + \
        (2.0 ** -24 if dtype == "f16" else 0.0)
    ops = [adlbr.Operator(dims, og, wg, storage=td, **kw)]
    if len(dims) == 2:
        g, nb = adlbr.grid(dims, **kw), ctypes.c_size_t()
        code = {"f64": capi.F64, "f32": capi.F32, "bf16": capi.BF16, "f16": capi.F16}[dtype]
        capi.check(capi.load().adlbr_operator_workspace(ctypes.byref(g), code, 0,
                                                        ctypes.byref(nb)))
        ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
        ops.append(adlbr.Operator(dims, og, wg, storage=td, workspace=ws, **kw))
        assert ops[1].workspace is ws and ops[0].workspace.numel() > nb.value
    for op in ops:
        got = op.apply(u).double().cpu().numpy()
        assert np.all(abs(got - ref) <= tol), float((abs(got - ref) - tol).max())
        d = op.diagonal().cpu().numpy()
        da = np.zeros(w.shape[1])
        src, tgt, wt = _edge_weights(dims, off, held, **kw)
        np.add.at(da, src, wt)
        # a 2D list leaves out a zero offset's edge: it counts at its source only
        lists = (src != tgt) | (len(dims) == 3)
        np.add.at(da, tgt[lists], wt[lists])
        assert np.all(abs(d - da) <= (2e-14 if dtype == "f64" else 1.2e-7) * da)


def _edge_weights(dims, off, w, periodic=False, reflect=False):
    """Directed edges (source, target, weight) of positive weight that the
    operator counts in its diagonal."""
    nd = np.array(dims)
    d, n = len(dims), w.shape[1]
    idx = np.arange(n)
    p = np.stack([(idx // int(np.prod(dims[:c]))) % dims[c] for c in range(d)])
    src, tgt, wt = [], [], []
    for q in range(w.shape[0]):
        for s in (-1, 1):
            t = p + s * off[q].astype(np.int64)
            ok = w[q] > 0
            if periodic:
                t %= nd[:, None]
            elif reflect:
                t %= 2 * nd[:, None]
                t = np.where(t < nd[:, None], t, 2 * nd[:, None] - 1 - t)
            else:
                ok = ok & np.all((t >= 0) & (t < nd[:, None]), axis=0)
            lin = sum(t[c] * int(np.prod(dims[:c])) for c in range(d))
            if periodic or reflect:
                ok = ok & (lin != idx)
            src.append(idx[ok])
            tgt.append(lin[ok])
            wt.append(w[q][ok])
    return np.concatenate(src), np.concatenate(tgt), np.concatenate(wt)


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("spread", [1, 6])
def test_unpaired_edges_fill_the_bins(dtype, spread):
    """Every point its own random offsets: nearly nothing merges, and bins of
    1024 targets receive up to 12 entries a target, more than a block holds in
    LDS (spread 6) or about as many (spread 1: short offsets often meet)."""
    import torch
    import paper_1301_3925_amd as adlbr
    dims = (40, 16, 8)
    n = int(np.prod(dims))
    td = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    rng = np.random.default_rng(spread)
    a, b, c = rng.integers(-spread, spread + 1, size=(3, n, 3))
    off = np.stack([a, b, c, -(a + b), a - c, b + c]).transpose(0, 2, 1).astype(np.int16)
    off = np.ascontiguousarray(off)
    w = torch.from_numpy(rng.uniform(0.1, 1.0, (6, n)).astype(np.float32)).cuda()
    u = torch.from_numpy(rng.uniform(-1, 1, n)).to(td).cuda()
    op = adlbr.Operator(dims, torch.from_numpy(off).cuda(), w, storage=td)
    held = w.to(td).double().cpu().numpy() * ~(off == 0).all(1)
    A = oracle.operator_matrix(dims, off, held)
    uh = u.double().cpu().numpy()
    ref, mag = A @ uh, abs(A) @ abs(uh)
    eps = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    out = 2.0 ** -8 if dtype == "bf16" else 0.0
    tol = 4 * (np.diff(A.indptr) * 2 + 8) * eps * mag * (1 + out) + out * abs(ref)
    got = op.apply(u).double().cpu().numpy()
    assert np.all(abs(got - ref) <= tol), float((abs(got - ref) - tol).max())
