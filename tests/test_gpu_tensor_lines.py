"""The blurs' four-output lines and the 3D eigen map at their edges.

Lines shorter than the Gaussian's radius, of 1 to 9 values (every remainder of
four), in each direction, and images so faint that squares of J vanish in FP32,
against the FP64 oracle: 1e-12 (FP64) and 1e-5 (FP32) relative L2, the bounds
of the tensor's parity.
"""
import numpy as np
import pytest

import oracle
from paper_1301_3925_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eig_map", ["ced", "eed"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("dims", [(1, 1, 1), (5, 3, 2), (4, 4, 4), (9, 6, 7), (2, 8, 5), (33, 1, 3),
                                  (7, 9), (65, 5)], ids=lambda d: "x".join(map(str, d)))
def test_short_lines(dims, dtype, eig_map):
    import torch
    import paper_1301_3925_amd as adlbr
    td = torch.float64 if dtype == "f64" else torch.float32
    n = int(np.prod(dims))
    for scale in (1.0, 1e-12):
        u = torch.from_numpy(scale * synth.uniform(5, n)).to(td).cuda()
        D = adlbr.structure_tensor(u, dims, 1.5, 2.0, 1e-2, 1e-3, eig_map=eig_map)
        ref = oracle.structure_tensor_d(u.double().cpu().numpy(), dims, 1.5, 2.0, 1e-2, 1e-3,
                                        oracle.CED if eig_map == "ced" else oracle.EED)
        got = D.double().cpu().numpy()
        tol = 1e-12 if dtype == "f64" else 1e-5
        assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref), scale
