"""GPU: parameters set on a simulator reach everything its driver reads.

Each simulator is built from one model, then every trained parameter of a second
model of the same shape is written to it; its runs must equal, bit for bit, those
of a simulator built from the second model.  Drivers keep parameters in other
forms beside the parameter bases: the resident program's tables, transposed
products (persistent kernel) and encoders, neuron-major decoders (event
decoding), packed fp32 and bf16 weights (window driver)."""
import copy

import numpy as np
import pytest

import paper_1805_11144_amd as M
from synth import make_workload
from synth.spec import Connection, ModelSpec, Node, Probe
from tests.test_gpu_resident import recurrent

pytestmark = pytest.mark.gpu
MS = M.mergesim


def other(w, scalars, ensembles):
    """The same model with other encoders, biases, decoders and matrix
    transforms, and (scalars) other scalar transforms where they are not 1."""
    w = copy.deepcopy(w)
    rng = np.random.default_rng(5)
    for e in w.spec.ensembles if ensembles else []:
        e.encoders = -np.asarray(e.encoders)
        e.intercepts = np.asarray(e.intercepts) * 0.8
        e.max_rates = np.asarray(e.max_rates) * 1.1
    for c in w.spec.connections:
        t = np.asarray(c.transform, np.float64)
        if t.ndim == 2:
            c.transform = t * rng.uniform(0.5, 1.5, t.shape)
        elif scalars and t != 1.0:
            c.transform = float(t) * 0.75
    return w


def params(sim, w):
    keys = [(MS.TRAIN_ENCODERS, e, 0) for e in range(len(w.spec.ensembles))]
    keys += [(MS.TRAIN_BIASES, e, 0) for e in range(len(w.spec.ensembles))]
    keys += [(MS.TRAIN_DECODERS, e, 0) for e in range(len(w.spec.ensembles))]
    keys += [(MS.TRAIN_TRANSFORM, c, 0) for c in range(len(w.spec.connections))]
    got = {}
    for k in keys:
        try:
            got[k] = sim.train_param(*k)
        except MS.MergesimError:
            pass   # the model has no such parameter
    assert len({k[0] for k in got}) > 1
    return got


def check(w, scalars=True, ensembles=True, driver=None, auto=False, **opts):
    w2 = other(w, scalars, ensembles)
    probes = range(len(w.spec.probes))
    requested = M.DRIVER_AUTO if auto else driver

    def run(sim):
        sim.reset()
        sim.run_steps(w.n_steps, w.feeds)
        return [sim.data(p) for p in probes]

    def make(v):
        return M.Simulator(M.model_from_spec(v.spec), minibatch=v.minibatch, probe_capacity_steps=v.n_steps,
                           driver=requested, **opts)

    with make(w2) as sim:
        assert sim.info()["driver"] == driver
        new, exp = params(sim, w2), run(sim)
    with make(w) as sim:
        first = run(sim)
        for k, v in new.items():
            sim.set_train_param(k[0], k[1], v, k[2])
        got = run(sim)
    assert any(np.abs(a - b).max() > 0 for a, b in zip(first, exp))
    for a, b in zip(got, exp):
        np.testing.assert_array_equal(a, b)


RESIDENT = [
    ((65, 64), 0, 1, 3, 70, 2), ((200, 30), 0, 2, 4, 9, 9),           # the persistent kernel's order
    ((65, 256), 100, 1, 300, 70, 4), ((130, 200), 85, 2, 30, 33, 3)]  # the launch drivers' order


@pytest.mark.parametrize("ns,fill,d,n_feed,K,minibatch", RESIDENT)
def test_resident_program(ns, fill, d, n_feed, K, minibatch):
    check(recurrent(ns, d, minibatch, n_feed, K, fill=fill), driver=M.DRIVER_PERSISTENT, auto=True)


def test_interpreting_kernel():
    check(recurrent((65, 64), 1, 2, 3, 70, rate=True), driver=M.DRIVER_PERSISTENT)


# (the fused synapse launch takes scalar transforms as constants)
@pytest.mark.parametrize("decode", ["dense", "event"])
@pytest.mark.parametrize("d", [1, 2])
def test_launch_drivers(decode, d):
    check(recurrent((65, 256, 30), d, 3, 4, 9, n_steps=20), scalars=False, driver=M.DRIVER_STEPS, decode=decode)


def test_launch_driver_many_neurons():
    check(make_workload("pes", n_steps=20, minibatch=2, D=12, neurons_per_dim=50), scalars=False,
          driver=M.DRIVER_STEPS)


@pytest.mark.parametrize("gemm_dtype", ["f32", "bf16"])
def test_window_products(gemm_dtype):
    w = make_workload("c3", neuron_type="relu", n_steps=10, minibatch=8, n_hidden=72, n_in=24, n_out=3)
    check(w, scalars=False, ensembles=False, driver=M.DRIVER_WINDOW, gemm_dtype=gemm_dtype)   # gains are not set


SIZES = [(17, 16), (33, 40), (64, 100), (65, 31), (130, 33), (1, 64)]


def test_packed_weights_of_many_products():
    """Products of six shapes, their weights packed by one launch, and by a launch
    of its own where one transform is set."""
    rng, B, steps = np.random.default_rng(3), 5, 4
    spec = ModelSpec(dt=0.001)
    u = spec.add_node(Node(size=100))
    for rows, cols in SIZES:
        o = spec.add_node(Node(size=rows, passthrough=True))
        spec.connect(Connection(pre=u, post=o, transform=rng.standard_normal((rows, cols)), pre_slice=(0, cols)))
        spec.probe(Probe(target=o))
    feeds = {u[1]: rng.standard_normal((B, steps, 100)).astype(np.float32)}
    model = M.model_from_spec(spec)
    with M.Simulator(model, minibatch=B, driver=M.DRIVER_WINDOW) as win, \
            M.Simulator(model, minibatch=B, driver=M.DRIVER_STEPS) as ref:
        for k in range(-1, len(SIZES)):
            for s in (win, ref):
                if k >= 0:
                    s.set_train_param(MS.TRAIN_TRANSFORM, k, np.random.default_rng(k).standard_normal(SIZES[k]))
                s.reset()
                s.run_steps(steps, feeds)
            for p in range(len(SIZES)):
                assert np.abs(ref.data(p)).max() > 0
                np.testing.assert_array_equal(win.data(p), ref.data(p))
