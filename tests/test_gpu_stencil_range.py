"""Stencils at the edges of the reduction's exact range.

Sheared integer tensors whose reduction needs one coefficient of 2^14, 2^23
(components held exactly as doubles) or 2^25 + 1 (beyond the exact range: the
64-bit integer pass), between ordinary points of the same wavefronts, against
the oracle: offsets, status and weights.  Every product of the sheared forms
is an integer below 2^53, so both sides decide on exact numbers.
"""
import numpy as np
import pytest

import oracle
from paper_1301_3925_amd import synth

pytestmark = pytest.mark.gpu


def _field(dim, n, shears, seed):
    D = synth.random_spd2(seed, n, 50.0) if dim == 2 else synth.random_spd3(seed, n, 50.0)
    for i, a in zip(range(5, n, 7), np.resize(shears, n)):
        a = float(a)
        D[:, i] = [a * a + 1, a, 1] if dim == 2 else [1, -a, 0, a * a + 1, 0, 1]
    return D


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("shears", [(2 ** 14,), (2 ** 23,), (2 ** 25 + 1,),
                                    (3, -2 ** 14, 2 ** 25 + 1, -2 ** 24 - 1)], ids=str)
@pytest.mark.parametrize("n", [1, 64, 1000])
def test_sheared_tensors(dim, shears, n):
    import torch
    import paper_1301_3925_amd as adlbr
    dims = (n, 1) if dim == 2 else (n, 1, 1)
    D = _field(dim, n, shears, 3)
    off, w, st = adlbr.build_stencils(torch.from_numpy(D).cuda(), dims)
    ro, rw, rst = oracle.stencil(D)
    assert np.array_equal(off.cpu().numpy(), ro)
    bad = np.where(rst & 7)[0]
    assert st.cpu().tolist() == [bad[0] if bad.size else -1, np.bitwise_or.reduce(rst)]
    # ordinary points: the bound of the stencil builder's parity; sheared
    # ones: sums of exact integers, halved
    r2 = np.maximum(1.0, (ro.astype(float) ** 2).sum(1).max(0))
    if dim == 3:
        r2 = np.maximum(r2, np.abs(oracle.superbase3d(D)[0].astype(float)).sum(1).max(0) ** 2)
    assert np.all(np.abs(w.cpu().numpy() - rw) <= 1e-14 * np.abs(D).max(0) * r2)
