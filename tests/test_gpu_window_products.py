"""GPU: the window driver's fp32 products at the edges of their tiles.

A product's tiles (128 x 128, 64 x 64, slices of 16 or 32 k, packed weights
padded to whole tiles) add every sum over k in order into one accumulator, as
the time-major driver's one-thread-per-row products do, so rate-neuron layers
fed by them must agree with that driver bit for bit.  Sizes: rows and inputs
one below, at and one above a tile or slice edge; minibatches with and without
16-byte aligned columns; few and many column tiles.  On 256 CUs the large shapes
run on 128 x 128 tiles: with aligned columns, and without them 279 tiles (the
last columns on 64 x 64 tiles), 256 (none left over) and 1144 (past four a CU,
where the last columns stay on large tiles); none of them whole multiples of a
tile or slice in every direction."""
import numpy as np
import pytest

import paper_1805_11144_amd as M
from synth import make_workload
from synth.spec import Connection, ModelSpec, Node, Probe, Workload
from tests.test_gpu_parity import run_gpu

pytestmark = pytest.mark.gpu

SHAPES = [(n_in, hidden, batch, 6) for n_in in (15, 16, 31, 33) for hidden in (63, 65) for batch in (5, 8)]
SHAPES += [(129, 128, 7, 9), (130, 129, 12, 11), (257, 193, 12, 5), (1000, 64, 5, 3), (144, 1100, 12, 320)]
SHAPES += [(255, 65, 5, 6), (256, 65, 8, 6)]   # where slices of 16 k end and those of 32 begin
SHAPES += [(145, 1100, 13, 300), (145, 1024, 7, 585), (145, 1300, 13, 1024)]


@pytest.mark.parametrize("n_in,hidden,batch,steps", SHAPES)
def test_products_equal_time_major(n_in, hidden, batch, steps):
    w = make_workload("c3", neuron_type="relu", n_steps=steps, minibatch=batch, n_hidden=hidden, n_in=n_in, n_out=3)
    got, ref = run_gpu(w, driver=M.DRIVER_WINDOW), run_gpu(w, driver=M.DRIVER_STEPS)
    for p in (1, 2):   # the two hidden layers
        assert np.abs(ref[p]).max() > 0
        assert np.array_equal(got[p], ref[p]), (p, np.abs(got[p] - ref[p]).max())


@pytest.mark.parametrize("rows,cols", [(1, 16), (8, 48), (17, 33), (65, 16), (16, 255)])
@pytest.mark.parametrize("batch", [5, 8])
def test_many_small_products(rows, cols, batch):
    """Seven products of one group, of few rows and short sums."""
    rng = np.random.default_rng(rows * cols)
    spec, ops, steps = ModelSpec(dt=0.001), 7, 9
    u, o = spec.add_node(Node(size=cols * ops)), spec.add_node(Node(size=rows * ops, passthrough=True))
    for k in range(ops):
        spec.connect(Connection(pre=u, post=o, transform=rng.standard_normal((rows, cols)),
                                pre_slice=(cols * k, cols * k + cols), post_slice=(rows * k, rows * k + rows)))
    spec.probe(Probe(target=o))
    feed = rng.standard_normal((batch, steps, cols * ops)).astype(np.float32)
    w = Workload("products", spec, batch, steps, {u[1]: feed})
    got, ref = run_gpu(w, driver=M.DRIVER_WINDOW), run_gpu(w, driver=M.DRIVER_STEPS)
    assert np.array_equal(got[0], ref[0])
    x = feed.astype(np.float64).reshape(batch, steps, ops, cols)
    W = np.stack([np.float32(c.transform).astype(np.float64) for c in spec.connections])
    exp, mag = (np.einsum("btoc,orc->btor", f(x), f(W)).reshape(got[0].shape) for f in (np.asarray, np.abs))
    assert (np.abs(got[0] - exp) <= cols * 2.0 ** -24 * mag).all()   # cols roundings, each half an ulp of a partial sum
