"""GPU: probe records read back in the caller's [batch, steps, width] layout.

A probed input node records its feed unchanged, so every read must equal the
feed bit for bit.  The batch sizes lie at the edges of the read's two forms (large
records a 64 x 64 transposition tile from 16 batch columns on, others one thread
per value), the widths and step counts make (step, value) pairs cross tile
boundaries, and two probes put the second one at an offset in the record."""
import numpy as np
import pytest
import torch

import paper_1805_11144_amd as M
from synth.spec import ModelSpec, Node, Probe

pytestmark = pytest.mark.gpu


# records on the transposition tiles: 1,179,648 values, twice that below 32
# columns; the first two lie on both sides of the line
LARGE = [(64, 96, 96), (64, 96, 95), (16, 128, 576), (17, 101, 688), (33, 77, 233), (65, 1, 9085), (130, 130, 36),
         (1100, 541, 1), (257, 63, 37)]


@pytest.mark.parametrize("batch,width,steps", LARGE)
def test_large_record_is_the_feed(batch, width, steps):
    test_record_is_the_feed(batch, width, steps)


@pytest.mark.parametrize("batch", [1, 15, 16, 63, 65, 130])
@pytest.mark.parametrize("width,steps", [(1, 3), (7, 29), (70, 5), (64, 2)])
def test_record_is_the_feed(batch, width, steps):
    spec = ModelSpec(dt=0.001)
    a, b = spec.add_node(Node(size=3)), spec.add_node(Node(size=width))
    for n in (a, b):
        spec.probe(Probe(target=n))
    rng = np.random.default_rng(batch * 1000 + width)
    feeds = {i: rng.standard_normal((batch, 2 * steps, s)).astype(np.float32) for i, s in ((a[1], 3), (b[1], width))}
    with M.Simulator(M.model_from_spec(spec), minibatch=batch, probe_capacity_steps=steps) as sim:
        for h in (0, 1):
            sim.run_steps(steps, {k: np.ascontiguousarray(f[:, h * steps:(h + 1) * steps]) for k, f in feeds.items()})
        for p, n in enumerate((a, b)):
            want = feeds[n[1]]
            np.testing.assert_array_equal(sim.data(p), want)
            np.testing.assert_array_equal(sim.data_static(p), want)
            dev = torch.full(want.shape, float("nan"), device="cuda")
            torch.cuda.synchronize()   # the fill is on torch's stream, the read on the simulator's
            ptr = M.mergesim.C.cast(dev.data_ptr(), M.mergesim._fp)
            assert M.load_library().ms_sim_probe_read(sim.handle, p, ptr, dev.numel(), 1) == 0
            np.testing.assert_array_equal(dev.cpu().numpy(), want)
