"""CPU: what the window driver makes of its phases (the `run` entry of the
plan's JSON): which of them others take over, and which stay.  The GPU tests of
the fused phases compare results; these say that there is something fused."""
import pytest

import paper_1805_11144_amd as M
from synth import make_workload
from tests.test_launch_plan_mixed_inputs import passthrough_model


def phases(w, **opts):
    ph = M.Plan(M.model_from_spec(w.spec), minibatch=w.minibatch, **opts).json()["window"]["phases"]
    return [(p["group"]["type"], p["run"]) for p in ph]


def kinds(ph, *types):
    return [r for t, r in ph if t in types]


@pytest.mark.parametrize("simplify", [True, False])
@pytest.mark.parametrize("neuron_type", ["lif", "relu"])
def test_classifier(neuron_type, simplify):
    """Resets and parameter copies go, products are stored, neurons compute their
    currents; spiking neurons run the filter before them, unless the model can be
    trained (simplify = False), whose signals all stay."""
    ph = phases(make_workload("c3", neuron_type=neuron_type, n_steps=5, minibatch=8, n_in=20, n_hidden=70),
                simplify=simplify)
    init = 1 if simplify else 2   # the bias: a constant, or the parameter's rows
    assert all(r["skip"] for r in kinds(ph, "Reset", "Copy", "ElementwiseInc"))
    assert [r["init"] for r in kinds(ph, "DotInc")] == [1, 1, 1]
    neurons = kinds(ph, "SimLIF", "SimLIFRate")
    fold = neuron_type == "lif" and simplify
    assert [(r["skip"], r["init"], r["current"]) for r in neurons] == [(False, init, 1), (False, init, 2 if fold else 1)]
    assert [r["skip"] for r in kinds(ph, "Lowpass")] == [fold, False]   # the second is the readout's


@pytest.mark.parametrize("simplify", [True, False])
def test_copies(simplify):
    """Whole-row copies whose readers can read the source go; the copy of a probed
    row, increments of several sources and (simplify = False) every copy stay."""
    ph = kinds(phases(passthrough_model(2), simplify=simplify), "CopyInc")
    gone = sum(r["skip"] for r in ph)
    assert gone == (4 if simplify else 0) and gone < len(ph)
    assert sum(r["init"] == 0 for r in ph) == 1   # adds to what another started
