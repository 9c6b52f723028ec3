"""Operators with and without merged pairs run different kernels: a batch of
both has a class key for each, and the tuner's cache and file an entry for
each.  Entries saved for plain lists do not serve merged operators."""
import ctypes
import json

import numpy as np
import pytest

from paper_1301_3925_amd import capi, synth

pytestmark = pytest.mark.gpu


def _ops(plain):
    """The same two images, twice the points apart at most."""
    import torch
    import paper_1301_3925_amd as adlbr
    out = []
    for k, dims in enumerate([(70, 45), (64, 48)]):
        off, w, _ = adlbr.build_stencils(
            torch.from_numpy(synth.tensor2d_field(50 + k, *dims, 10.0)).cuda(), dims)
        ws = None
        if plain:
            nb = ctypes.c_size_t()
            capi.check(capi.load().adlbr_operator_workspace(ctypes.byref(adlbr.grid(dims)),
                                                            capi.F32, 0, ctypes.byref(nb)))
            ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
        out.append(adlbr.Operator(dims, off, w, workspace=ws))
        assert (out[-1].workspace is ws) == plain
    return out


def test_merged_and_plain_classes_are_told_apart(tmp_path):
    import torch
    import paper_1301_3925_amd as adlbr
    adlbr.tune_cache_clear()
    ops = _ops(False) + _ops(True)
    us = [torch.from_numpy(synth.uniform(60 + k % 2, op.N)).float().cuda() for k, op in enumerate(ops)]
    ref = [u.clone() for u in us]
    for op, u in zip(ops, ref):
        op.step(u, 0.9, 5, cfl_fraction=True)
    b = adlbr.Batch(ops, us, dt=0.9, dt_mode="cfl")
    keys = [v["class"] for v in b.variants()]
    assert len(keys) == 2 and keys[0] != keys[1]
    assert keys[1] == 2000 + capi.F32 and keys[0] == 20000 + keys[1]  # merged first
    tuned = b.tune(steps=1, use_cache=False)
    points = sum(op.N for op in ops[:2])
    for v in tuned:
        assert adlbr.tune_cache_lookup(v["class"], points, 2) == (v["variant"], v["chunk_bytes"])
    path = tmp_path / "tune.json"
    adlbr.tune_cache_save(path)
    assert sorted(e["class"] for e in json.loads(path.read_text())["entries"]) == sorted(keys)
    b.run(5)
    torch.cuda.synchronize()
    for u, r in zip(us, ref):
        assert torch.equal(u, r)
    # an entry of the plain lists alone: only the plain class takes it
    adlbr.tune_cache_clear()
    lg = int(np.floor(np.log2(points)))
    path.write_text(json.dumps({"format": "adlbr-batch-tune", "version": 1, "entries": [
        {"class": keys[1], "log2_points": lg, "problems": 2, "variant": 6, "chunk_bytes": 4096}]}))
    adlbr.tune_cache_load(path)
    got = {v["class"]: v["variant"] for v in adlbr.Batch(ops, us, dt=0.9, dt_mode="cfl").variants()}
    assert got == {keys[0]: 1, keys[1]: 6}
    adlbr.tune_cache_clear()
