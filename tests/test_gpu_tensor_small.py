"""Small grids blur with one output per thread, larger ones with four: the
tensors are the same bits.  A volume extruded along its last axis has the
tensor of one of its planes on every plane, whatever their number, so grids on
both sides of the change (200000 points) and a short one agree bit for bit."""
import numpy as np
import pytest

from paper_1301_3925_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("sigma,rho", [(0.5, 2.0), (1.0, 4.0), (3.0, 9.5)])
@pytest.mark.parametrize("base,lengths", [((60, 60), (3, 50, 55, 56, 61)),
                                          ((450,), (5, 444, 445, 500)),
                                          ((7, 331), (1, 85, 87))],
                         ids=lambda d: "x".join(map(str, d)))
def test_extruded_images_agree(base, lengths, sigma, rho, dtype):
    import torch
    import paper_1301_3925_amd as adlbr
    td = torch.float64 if dtype == "f64" else torch.float32
    n = int(np.prod(base))
    plane = torch.from_numpy(synth.uniform(5, n)).to(td).cuda()
    ref = None
    for m in lengths:
        if len(base) == 1 and sigma <= 1.0 and dtype == "f32":
            continue  # the tiled 2D kernels
        D = adlbr.structure_tensor(plane.repeat(m), base + (m,), sigma, rho, 1e-2, 1e-3)
        D = D.reshape(D.shape[0], m, n)
        ref = D[:, :1].clone() if ref is None else ref
        assert torch.equal(D, ref.expand_as(D)), m
