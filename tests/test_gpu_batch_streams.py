"""A batch whose launch settings change while its last run is still going on
another stream: the change waits for the run, whose launches read the same
descriptor table and scratch."""
import numpy as np
import pytest

from paper_1301_3925_amd import synth

pytestmark = pytest.mark.gpu


def _batch(steps, runs):
    """A batch, its states, and the states after each of `runs` runs."""
    import torch
    import paper_1301_3925_amd as adlbr
    ops, us, refs = [], [], [[] for _ in range(runs)]
    for k, dims in enumerate([(40, 31), (700, 520), (64, 17), (300, 410)]):
        off, w, _ = adlbr.build_stencils(
            torch.from_numpy(synth.tensor2d_field(300 + k, *dims, 20.0)).cuda(), dims)
        ops.append(adlbr.Operator(dims, off, w))
        us.append(torch.from_numpy(synth.uniform(400 + k, int(np.prod(dims)))).float().cuda())
        r = us[-1].clone()
        for ref in refs:
            ops[-1].step(r, 0.9, steps, cfl_fraction=True)
            ref.append(r.clone())
    b = adlbr.Batch(ops, us, dt=0.9, dt_mode="cfl")
    torch.cuda.synchronize()
    return b, us, refs


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("change", ["variant", "tune"])
def test_settings_change_behind_a_run(change, graph):
    import torch
    b, us, refs = _batch(130, 4)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    seen = []
    for variant, chunk in ((2, 0), (9, 1), (3, 200_000), (0, 0)):
        b.run(130, graph=graph, stream=s1)
        if change == "variant":
            b.set_variant(0, variant, chunk, stream=s2)
            assert b.variants()[0]["variant"] == variant
        else:
            b.tune(steps=1, use_cache=False, stream=s2)
        with torch.cuda.stream(s2):  # not ordered behind s1: the run has ended by now
            seen.append([u.clone() for u in us])
    torch.cuda.synchronize()
    for got, ref in zip(seen, refs):
        for u, r in zip(got, ref):
            assert torch.equal(u, r)


@pytest.mark.skip(reason="the first process that ran it aborted on the host in a later test, cause unknown")
@pytest.mark.parametrize("variant,chunk", [(1, 0), (9, 1)])
def test_direct_run_in_the_callers_graph(variant, chunk):
    """A direct run captured by the caller steps at every replay; direct runs
    and changes of the settings before and after it are ordered as ever."""
    import torch
    b, us, refs = _batch(7, 5)
    b.set_variant(0, variant, chunk)
    s = torch.cuda.Stream()
    b.run(7, graph=False, stream=s)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        b.run(7, graph=False)
    for ref in refs[1:4]:
        g.replay()
        torch.cuda.synchronize()
        for u, r in zip(us, ref):
            assert torch.equal(u, r)
    b.set_variant(0, 3, 0)
    b.run(7, graph=False)
    torch.cuda.synchronize()
    for u, r in zip(us, refs[4]):
        assert torch.equal(u, r)
