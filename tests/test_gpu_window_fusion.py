"""GPU: window phases that took over others' work (dropped resets and copies,
neuron phases that compute their input current and run its filter).

Every value is formed by the same operations in the same order as in the
separate phases, so: a run split into windows of 1, 7 and 12 steps equals the
whole run bit for bit, with the carried filter and neuron state; rate layers
equal the time-major driver bit for bit; a model built without simplification
(whose copies all stay, since it can be trained) equals one built with it."""
import numpy as np
import pytest

import paper_1805_11144_amd as M
from synth import make_workload
from tests.test_launch_plan_mixed_inputs import passthrough_model

pytestmark = pytest.mark.gpu
MS = M.mergesim


def run(w, splits, **opts):
    with M.Simulator(M.model_from_spec(w.spec), minibatch=w.minibatch, probe_capacity_steps=4, **opts) as sim:
        t = 0
        for n in splits:
            sim.run_steps(n, {k: np.ascontiguousarray(f[:, t:t + n]) for k, f in w.feeds.items()})
            t += n
        out = [sim.data(p) for p in range(len(w.spec.probes))]
        state = [sim.get_state(MS.STATE_SYNAPSE, 1, w.spec.ensembles[1].n_neurons),
                 sim.get_state(MS.STATE_VOLTAGE, 1, w.spec.ensembles[1].n_neurons)] \
            if w.name == "c3" and w.spec.ensembles[0].neuron_type == "lif" else []
    return out + state


@pytest.mark.parametrize("tau_rc", [0.02, 0.01])   # dt / tau_rc below and above 1/16: both LIF updates
@pytest.mark.parametrize("minibatch", [3, 8])
@pytest.mark.parametrize("simplify", [True, False])
def test_spiking_layers_split_runs(tau_rc, minibatch, simplify):
    w = make_workload("c3", n_steps=20, minibatch=minibatch, n_in=20, n_hidden=70)
    for e in w.spec.ensembles:
        e.tau_rc = tau_rc
    whole = run(w, [20], driver=M.DRIVER_WINDOW, simplify=simplify)
    assert all(np.abs(o).max() > 0 for o in whole[:3])
    for a, b in zip(whole, run(w, [1, 7, 12], driver=M.DRIVER_WINDOW, simplify=simplify)):
        np.testing.assert_array_equal(a, b)
    for a, b in zip(whole, run(w, [20], driver=M.DRIVER_WINDOW, simplify=not simplify)):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("neuron_type", ["relu", "softlif_rate"])
@pytest.mark.parametrize("minibatch", [5, 8])
def test_rate_layers_equal_time_major(neuron_type, minibatch):
    w = make_workload("c3", neuron_type=neuron_type, n_steps=9, minibatch=minibatch, n_in=20, n_hidden=70)
    for a, b in zip(run(w, [9], driver=M.DRIVER_WINDOW)[1:], run(w, [9], driver=M.DRIVER_STEPS)[1:]):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("minibatch", [2, 4])
def test_copies_through_passthrough_nodes(minibatch):
    """Copies whose readers read the source instead (in pieces, in another order,
    one step earlier behind a filter), and the copy of a probed row, which stays."""
    w = passthrough_model(minibatch)
    whole = run(w, [12], driver=M.DRIVER_WINDOW)
    for a, b in zip(whole, run(w, [1, 11], driver=M.DRIVER_WINDOW)):
        np.testing.assert_array_equal(a, b)
    for k, (a, b) in enumerate(zip(whole, run(w, [12], driver=M.DRIVER_STEPS))):
        assert np.abs(b).max() > 0, k
        np.testing.assert_allclose(a, b, rtol=0, atol=2e-6 * np.abs(b).max(), err_msg=str(k))
