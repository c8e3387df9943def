"""CPU: which models have a resident program, and why not, from the plan's JSON.

The GPU tests of the resident program compare it with the driver that would run
the model without it; they mean something only where the program exists, which
is checked here for each of their models and options (and that the reference has
none).  The refusals are tried at their limits: one step inside and one past."""
import numpy as np
import pytest

import paper_1805_11144_amd as M
from synth.configs import lif_ensemble
from synth.spec import Connection, ModelSpec, Node, Probe
from tests import test_gpu_resident as gpu
from tests.test_gpu_set_params import RESIDENT as SET_PARAMS


def resident(w, **opts):
    return M.Plan(M.model_from_spec(w.spec), minibatch=w.minibatch, **opts).json()["launch"]["resident"]


@pytest.mark.parametrize("ns,d,n_feed,K,minibatch", gpu.PERSISTENT_ORDER)
def test_models_in_the_persistent_kernels_order(ns, d, n_feed, K, minibatch):
    r = resident(gpu.recurrent(ns, d, minibatch, n_feed, K))
    assert r["persistent_order"]["ok"], r
    r = resident(gpu.recurrent(ns, d, minibatch, n_feed, K, rate=True))
    assert not r["persistent_order"]["ok"] and not r["launch_order"]["ok"]


@pytest.mark.parametrize("ns,fill,d,n_feed,K,minibatch", gpu.LAUNCH_ORDER + gpu.ANY_VOLTAGE)
def test_models_in_the_launch_drivers_order(ns, fill, d, n_feed, K, minibatch):
    r = resident(gpu.recurrent(ns, d, minibatch, n_feed, K, fill=fill))
    assert r["launch_order"]["ok"], r


@pytest.mark.parametrize("ns,fill,d,n_feed,K,minibatch", SET_PARAMS)
def test_models_whose_parameters_are_set(ns, fill, d, n_feed, K, minibatch):
    r = resident(gpu.recurrent(ns, d, minibatch, n_feed, K, fill=fill))
    assert r["launch_order" if fill else "persistent_order"]["ok"], r


@pytest.mark.parametrize("opts", gpu.OPTIONS)
def test_plan_options(opts):
    r = resident(gpu.option_model(0), **opts)
    assert r["persistent_order"]["ok"], r
    r = resident(gpu.option_model(90), **opts)
    assert r["launch_order"]["ok"], r


def ring_spec(E, n=50, d=1, n_feed=1, tau_rc=(0.02,), dt=0.001, K=0, neuron="lif", spikes=False):
    """E ensembles in a ring, the first one fed; K: a K x K product over them."""
    rng = np.random.default_rng(E)
    spec = ModelSpec(dt=dt)
    u = spec.add_node(Node(size=n_feed))
    ids = []
    for i in range(E):
        e = lif_ensemble(rng, n, d, 20 + n, neuron)
        e.tau_rc = tau_rc[i % len(tau_rc)]
        ids.append(spec.add_ensemble(e))
    for i, e in enumerate(ids):
        spec.connect(Connection(pre=("ens", e), post=("ens", ids[(i + 1) % E]), transform=0.7, synapse=0.02))
    spec.connect(Connection(pre=u, post=("ens", ids[0]), transform=rng.standard_normal((d, n_feed)), synapse=0.01))
    if K:
        a, b = spec.add_node(Node(size=K, passthrough=True)), spec.add_node(Node(size=K, passthrough=True))
        spec.connect(Connection(pre=("ens", ids[0]), post=a, post_slice=(0, d)))
        spec.connect(Connection(pre=a, post=b, transform=rng.standard_normal((K, K))))
        spec.connect(Connection(pre=b, post=("ens", ids[0]), transform=0.1, pre_slice=(0, d), synapse=0.01))
    spec.probe(Probe(target=("ens", ids[0]), synapse=0.01))
    if spikes:
        spec.probe(Probe(target=("neurons", ids[0])))
    return spec


def ring(E, minibatch=1, dt=0.001, planner=M.mergesim.PLANNER_GREEDY, **kw):
    return M.Plan(M.model_from_spec(ring_spec(E, dt=dt, **kw)), minibatch=minibatch, planner=planner,
                  dt=dt).json()["launch"]["resident"]


# (inside the limit, past it, a word of the reason, order)
LIMITS = [
    # 8 wavefronts of 40 chunks; 106 ensembles of 3 chunks are 318, but 42 in a wavefront
    (dict(E=320), dict(E=321), "registers", "launch_order"),
    (dict(E=104, n=150), dict(E=106, n=150), "registers", "launch_order"),
    (dict(E=128, d=2), dict(E=129, d=2), "registers", "launch_order"),
    (dict(E=3, d=2), dict(E=3, d=3), "dimensions", "persistent_order"),
    (dict(E=2, n=256), dict(E=2, n=257), "256 neurons", "launch_order"),
    (dict(E=2, n=257), dict(E=2, neuron="lif_rate"), "rate", "persistent_order"),
    (dict(E=2), dict(E=2, tau_rc=(0.02, 0.03)), "parameters differ", "persistent_order"),
    (dict(E=2, dt=0.00125), dict(E=2, dt=0.00126), "tau_rc / 16", "persistent_order"),
    (dict(E=2, n_feed=128), dict(E=2, n_feed=129), "feed rows", "persistent_order"),
    (dict(E=2, K=128), dict(E=2, K=129), "long product", "launch_order"),
    (dict(E=2, K=129), dict(E=2, K=1025), "one workgroup", "persistent_order"),
    (dict(E=2, minibatch=7), dict(E=2, minibatch=8), "one workgroup", "launch_order"),
    (dict(E=60, n=64, K=250), dict(E=60, n=64, K=300), "k_persistent", "persistent_order"),   # 66 k weights
    (dict(E=12, n=150, K=90, minibatch=300), dict(E=12, n=150, K=91, minibatch=300), "k_persistent", "persistent_order"),
    (dict(E=12, n=150, K=91, minibatch=256), dict(E=12, n=150, K=91, minibatch=257), "k_persistent", "persistent_order"),
]


@pytest.mark.parametrize("inside,past,why,order", LIMITS)
def test_limits(inside, past, why, order):
    r = ring(**inside)[order]
    assert r["ok"], r
    r = ring(**past)[order]
    assert not r["ok"] and why in r["why"], r


# (model, minibatch, whether the program was measured faster than the launch drivers)
CHOICE = [
    # a ring's step is two launches
    (dict(E=160), 1, True), (dict(E=320), 1, False), (dict(E=320), 4, True), (dict(E=80, n=250), 1, False),
    (dict(E=80, n=250), 7, False), (dict(E=20, n=250), 1, True), (dict(E=128, d=2), 1, True),
    (dict(E=240, spikes=True), 1, False), (dict(E=160, spikes=True), 7, True),
    # twelve with a product
    (dict(E=300, K=64), 1, True), (dict(E=80, n=250, K=64), 4, True)]


@pytest.mark.parametrize("model,minibatch,faster", CHOICE)
def test_choice_against_the_launch_drivers(model, minibatch, faster):
    r = ring(**model, minibatch=minibatch, planner=M.mergesim.PLANNER_TREE)["launch_order"]
    assert r["ok"] and r["faster"] == faster, r


@pytest.mark.parametrize("model,waves", [
    (dict(E=1), 1), (dict(E=4), 1), (dict(E=5), 2), (dict(E=40), 8),                       # four chunks a wavefront
    (dict(E=1, K=40), 3), (dict(E=1, K=200), 8), (dict(E=1, n_feed=128), 2)])              # rows, columns of a product
def test_wavefronts(model, waves):
    assert ring(**model)["persistent_order"]["waves"] == waves
