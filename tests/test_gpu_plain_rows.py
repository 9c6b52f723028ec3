"""Rows of a 2D operator without merged pairs (a workspace of the plain size).

A slot's two differences are added before they meet its weight: on a linear
image they cancel exactly, whatever the weight's digits, and so do the two
listed edges of the slot.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("boundary", ["neumann", "periodic", "reflect"])
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("dims", [(33, 3), (64, 4), (70, 45)])
def test_linear_image_is_exact(dims, wide, boundary, dtype):
    import torch
    import paper_1301_3925_amd as adlbr
    from paper_1301_3925_amd import capi
    kw = {"periodic": boundary == "periodic", "reflect": boundary == "reflect"}
    td = torch.float64 if dtype == "f64" else torch.float32
    nb = ctypes.c_size_t()
    capi.check(capi.load().adlbr_operator_workspace(
        ctypes.byref(adlbr.grid(dims, **kw)), capi.F64 if dtype == "f64" else capi.F32,
        capi.OP_WIDE if wide else 0, ctypes.byref(nb)))
    ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
    n = int(np.prod(dims))
    off = np.zeros((3, 2, n), dtype=np.int16)
    off[:] = np.array([[1, 0], [0, 1], [-1, -1]])[:, :, None]
    w = np.zeros((3, n))
    w[0] = 0.3
    op = adlbr.Operator(dims, torch.from_numpy(off).cuda(), torch.from_numpy(w).to(td).cuda(),
                        storage=td, wide=wide, workspace=ws, **kw)
    assert op.workspace is ws
    u = torch.from_numpy(np.tile(7.0 * np.arange(dims[0]), dims[1])).to(td).cuda()
    rows = op.apply(u).reshape(dims[1], dims[0])
    assert not rows[:, 1:-1].any()
