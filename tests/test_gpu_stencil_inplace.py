"""Weights written where the tensor was: a caller without room for both passes
the tensor's planes as the weights'.  Each point's tensor is read before its
weights are written, also where a point is reduced a second time in 64-bit
integers (extreme anisotropy)."""
import numpy as np
import pytest

from paper_1301_3925_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kappa", [10.0, 1e8, 1e12])
@pytest.mark.parametrize("dims", [(65, 33), (33, 17, 9)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_weights_in_the_tensors_place(dims, kappa, dtype):
    import torch
    import paper_1301_3925_amd as adlbr
    D = (synth.tensor2d_field(3, *dims, kappa) if len(dims) == 2
         else synth.tensor3d_field(3, dims, kappa))
    D = torch.from_numpy(np.ascontiguousarray(D)).cuda()
    D = D if dtype == "f64" else D.float()
    off, w, st = adlbr.build_stencils(D, dims)
    o2, s2 = torch.empty_like(off), torch.empty_like(st)
    adlbr.build_stencils(D, dims, out=(o2, D, s2))
    assert torch.equal(o2, off) and torch.equal(D, w) and torch.equal(s2, st)
