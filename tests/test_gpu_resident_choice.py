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


@pytest.mark.parametrize("E,n", [(20, 250), (84, 50)])
def test_any_voltage_at_the_longest_step(E, n):
    """Voltages far above threshold at dt = tau_rc / 16, the longest step that the
    program takes: where the overshoot ratio is past 1/16 the crossing lies before
    the step, so its polynomial and the launch drivers' log1pf give the same."""
    dt, B = 0.00125, 2
    spec = ring_spec(E, n=n, dt=dt)
    V = np.concatenate([np.full(16, np.nextafter(np.float32(1), np.float32(2))), np.geomspace(1.01, 1e30, n - 16)])
    V = np.stack([V, V[::-1]]).astype(np.float32)
    out = []
    for kw in ({}, dict(driver=M.DRIVER_STEPS)):
        with M.Simulator(M.model_from_spec(spec), minibatch=B, dt=dt, **kw) as sim:
            assert sim.info()["driver"] == kw.get("driver", M.DRIVER_PERSISTENT)
            for e in range(E):
                sim.set_state(M.mergesim.STATE_VOLTAGE, e, V)
            sim.run_steps(1)
            out.append([sim.get_state(k, e, n) for e in range(E)
                        for k in (M.mergesim.STATE_VOLTAGE, M.mergesim.STATE_REFRACTORY)])
    assert max(np.abs(x).max() for x in out[1][1::2]) > 0
    np.testing.assert_array_equal(*out)
