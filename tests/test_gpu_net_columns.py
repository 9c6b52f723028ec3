"""The 3D inference's columns at their edges against the FP32 forward pass.

Grids of one point, of one row or plane in each direction, one point short of
and beyond the 16 x 8 column, the 16 x 16 x 8 box of the last layer and the
planes that a block walks.  The inference holds activations and the inner
weights in BF16 and gates in 8 bits, the forward pass all in FP32: 3 % of
relative L2 (1 % with the diagonal part), the bounds of the inference's
parity; a lost or doubled tap at an edge of these grids is worth more.
"""
import pytest

from paper_1301_3925_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(1, 1, 1), (40, 1, 1), (1, 40, 1), (1, 1, 40), (15, 7, 3), (16, 8, 4),
                                  (17, 9, 5), (33, 17, 9), (16, 16, 8), (18, 15, 17)],
                         ids=lambda d: "x".join(map(str, d)))
def test_columns(dims):
    import torch
    import paper_1301_3925_amd as adlbr
    D = synth.tensor3d_field(9, dims, 50.0)
    off, w, _ = adlbr.build_stencils(torch.from_numpy(D).cuda(), dims)
    op = adlbr.Operator(dims, off, w, storage=torch.float32)
    dt = 50.0 * op.dt_cfl()
    net = adlbr.Net(op, seed=3)
    net.prepare(dt)
    r = torch.from_numpy(synth.uniform(12, op.N) - 0.5).float().cuda()
    z32, z16 = net.forward(r), net.precondition(r)
    n32, n16 = z32 - r * net.features[0], z16 - r * net.features[0]
    assert float((n16 - n32).norm() / n32.norm()) <= 3e-2
    assert float((z16 - z32).norm() / z32.norm()) <= 1e-2
