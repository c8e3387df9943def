"""GPU: which driver a recurrent model gets that would run as launches without
its resident program: the faster one of the two, by the plan's estimate; the
outputs are the same bits on both."""
import numpy as np
import pytest

import paper_1805_11144_amd as M
from tests.test_resident_plan import CHOICE, ring_spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,minibatch,faster", CHOICE)
def test_the_faster_driver(model, minibatch, faster):
    spec, steps = ring_spec(**model), 30
    feeds = {0: np.random.default_rng(0).uniform(-1, 1, (minibatch, steps, 1)).astype(np.float32)}
    out = []
    for kw in ({}, dict(driver=M.DRIVER_STEPS)):
        with M.Simulator(M.model_from_spec(spec), minibatch=minibatch, **kw) as sim:
            if not kw:
                assert sim.info()["driver"] == (M.DRIVER_PERSISTENT if faster else M.DRIVER_GRAPH)
            sim.run_steps(steps, feeds)
            out.append(sim.data(0))
    assert np.abs(out[1]).max() > 0
    np.testing.assert_array_equal(*out)
