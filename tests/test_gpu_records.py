"""ADLBR_OP_RECORDS without merged pairs: the entries' weights are stored
beside them for the batch, and nothing else changes.  Results are those of a
plain operator, bit for bit: the single calls', and a batch's in every way of
launching it; a batch of plain and records operators has a class for each.
(The binding asks for merged pairs as well, unless the caller's workspace is
of the size without them.)"""
import ctypes

import numpy as np
import pytest

from paper_1301_3925_amd import capi, synth

# A process that had run 402 other GPU tests aborted on the host in this one
# (no fault of the GPU was reported; the test alone had passed twice).  No cause
# is known, so the layout it tests was taken out again: ADLBR_OP_RECORDS implies
# merged pairs.
pytestmark = [pytest.mark.gpu, pytest.mark.skip(
    reason="records without merged pairs were taken out: one run aborted on the host, cause unknown")]


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16", "f16"])
@pytest.mark.parametrize("boundary,wide", [("neumann", False), ("periodic", False),
                                           ("reflect", True), ("neumann", True)])
def test_same_bits_as_plain(boundary, wide, dtype):
    import torch
    import paper_1301_3925_amd as adlbr
    code = {"f64": capi.F64, "f32": capi.F32, "bf16": capi.BF16, "f16": capi.F16}[dtype]
    td = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16,
          "f16": torch.float16}[dtype]
    kw = {"periodic": boundary == "periodic", "reflect": boundary == "reflect"}

    def size(dims, flags):
        nb = ctypes.c_size_t()
        capi.check(capi.load().adlbr_operator_workspace(
            ctypes.byref(adlbr.grid(dims, **kw)), code, flags | (capi.OP_WIDE if wide else 0),
            ctypes.byref(nb)))
        return nb.value

    ops, us = [], []
    for records in (True, False):
        for k, dims in enumerate([(70, 45), (33, 90), (128, 64), (5, 3), (64, 4)]):
            off, w, _ = adlbr.build_stencils(
                torch.from_numpy(synth.tensor2d_field(100 + k, *dims, 20.0)).cuda(), dims)
            flags = capi.OP_RECORDS if records else 0
            # the plain layout: less than the binding's, that with records the more
            assert size(dims, 0) < size(dims, capi.OP_RECORDS) < size(dims, flags | capi.OP_MERGED)
            ws = torch.empty(size(dims, flags), dtype=torch.uint8, device="cuda")
            ops.append(adlbr.Operator(dims, off, w, storage=td, wide=wide, workspace=ws,
                                      records=records, **kw))
            assert ops[-1].workspace is ws
            us.append(torch.from_numpy(synth.uniform(200 + k, int(np.prod(dims)))).to(td).cuda())
    half = len(ops) // 2
    for rec, plain, u in zip(ops[:half], ops[half:], us):
        assert torch.equal(rec.apply(u), plain.apply(u))
        assert torch.equal(rec.diagonal(), plain.diagonal()) and rec.dt_cfl() == plain.dt_cfl()
    ref = [u.clone() for u in us]
    for op, u in zip(ops, ref):
        op.step(u, 0.9, 5, cfl_fraction=True)
    for a, b in zip(ref[:half], ref[half:]):
        assert torch.equal(a, b)
    for variant, chunk in ((1, 300_000), (0, 0), (4, 0), (9, 1)):
        state = [u.clone() for u in us]
        b = adlbr.Batch(ops, state, dt=0.9, dt_mode="cfl")
        keys = [v["class"] for v in b.variants()]
        assert len(keys) == 2 and keys[0] == 100000 + keys[1]
        for cls in (0, 1):
            b.set_variant(cls, variant, chunk)
        b.run(2)
        b.run(3)
        torch.cuda.synchronize()
        for u, r in zip(state, ref):
            assert torch.equal(u, r)
