"""GPU: recurrent models small enough to run as a resident program (one
workgroup per batch column, neurons in registers).

Its sums are taken in the order of the driver that would run the model
without it, so every probe and the carried voltages equal that driver's bit
for bit: the launch drivers for models of more than 8,192 rows and fewer than
eight batch columns, the interpreting persistent kernel otherwise.  A model
with one unconnected rate ensemble more has no resident program; requested on
the persistent driver it is that reference (test_resident_plan checks on the CPU
that each model here has a program and each reference none).  Sizes: ensembles around the 64
lanes of a wavefront, of one and two dimensions, with one and several chunks;
fed rows fewer and more than a workgroup's threads; products of 63 to 128
columns and rows that are no multiple of eight; runs in pieces."""
import numpy as np
import pytest

import paper_1805_11144_amd as M
from synth.configs import lif_ensemble
from synth.spec import Connection, ModelSpec, Node, Probe, Workload

pytestmark = pytest.mark.gpu
MS = M.mergesim


def recurrent(ns, d, minibatch, n_feed, K, rate=False, n_steps=40, fill=0) -> Workload:
    """Ensembles of ns neurons in a ring behind filters, each fed, filtered and
    unfiltered; a product of K columns over what they decode; `fill` ensembles
    of 50 neurons more."""
    rng = np.random.default_rng(len(ns) * 100 + d)
    spec = ModelSpec(dt=0.001)
    u = spec.add_node(Node(size=n_feed))
    mid = spec.add_node(Node(size=K, passthrough=True))
    out = spec.add_node(Node(size=13, passthrough=True))
    ids = [spec.add_ensemble(lif_ensemble(rng, n, d, 60, "lif")) for n in list(ns) + [50] * fill]
    for i, e in enumerate(ids):
        k = i % (n_feed - d + 1)
        spec.connect(Connection(pre=u, post=("ens", e), transform=0.5, pre_slice=(k, k + d),
                                synapse=0.005 if i % 2 else None))
        spec.connect(Connection(pre=("ens", e), post=("ens", ids[(i + 1) % len(ids)]), transform=0.7, synapse=0.02))
        j = d * i % (K - d + 1)
        spec.connect(Connection(pre=("ens", e), post=mid, transform=1.0, post_slice=(j, j + d)))
    spec.connect(Connection(pre=mid, post=out, transform=rng.standard_normal((13, K)) / np.sqrt(K)))
    spec.connect(Connection(pre=out, post=("ens", ids[0]), transform=0.1, pre_slice=(13 - d, 13), synapse=0.01))
    spec.probe(Probe(target=("ens", ids[0]), synapse=0.01))
    spec.probe(Probe(target=out))
    spec.probe(Probe(target=mid, synapse=0.005))
    if not fill:
        spec.probe(Probe(target=("neurons", ids[-1])))
    feed = rng.uniform(-1, 1, (minibatch, n_steps, n_feed)).astype(np.float32)
    if rate:
        r = spec.add_ensemble(lif_ensemble(rng, 3, 1, 20, "relu"))
        spec.probe(Probe(target=("ens", r)))
    return Workload("recurrent", spec, minibatch, n_steps, {u[1]: feed})


def run(w, splits, n_probes, state=None, **opts):
    with M.Simulator(M.model_from_spec(w.spec), minibatch=w.minibatch, probe_capacity_steps=64, **opts) as sim:
        n = w.spec.ensembles[0].n_neurons
        if state is not None:
            sim.set_state(MS.STATE_VOLTAGE, 0, state)
        t = 0
        for k in splits:
            sim.run_steps(k, {i: np.ascontiguousarray(f[:, t:t + k]) for i, f in w.feeds.items()})
            t += k
        return [sim.data(p) for p in range(n_probes)] + [sim.get_state(MS.STATE_VOLTAGE, 0, n),
                                                         sim.get_state(MS.STATE_REFRACTORY, 0, n)]


def same(got, ref):
    assert all(np.abs(r).max() > 0 for r in ref[:-1])
    for a, b in zip(got, ref):
        np.testing.assert_array_equal(a, b)


PERSISTENT_ORDER = [
    ((1,), 1, 1, 3, 1), ((63, 64), 1, 3, 5, 2), ((65, 128, 129), 1, 2, 63, 3), ((100,) * 9, 1, 40, 64, 1),
    ((64,) * 33, 2, 130, 70, 2), ((200, 30), 2, 4, 9, 9), ((60,) * 40, 1, 6, 90, 8)]


@pytest.mark.parametrize("ns,d,n_feed,K,minibatch", PERSISTENT_ORDER)
def test_order_of_the_persistent_kernel(ns, d, n_feed, K, minibatch):
    got = run(recurrent(ns, d, minibatch, n_feed, K), [40], 4, driver=M.DRIVER_PERSISTENT)
    same(got, run(recurrent(ns, d, minibatch, n_feed, K, rate=True), [40], 4, driver=M.DRIVER_PERSISTENT))


LAUNCH_ORDER = [
    ((64, 1, 63), 90, 1, 5, 64, 1), ((65, 256), 100, 1, 300, 70, 4), ((65, 64), 300, 1, 7, 128, 2), ((64,), 310, 1, 7, 120, 1),
    ((130, 200), 85, 2, 30, 127, 3), ((50,), 90, 2, 600, 63, 5),
    # two decoded sums over up to four chunks, exchanged between lanes, at every place in a block of eight slots
    ((256, 193, 255, 129, 256), 75, 2, 3, 64, 2)]


@pytest.mark.parametrize("ns,fill,d,n_feed,K,minibatch", LAUNCH_ORDER)
def test_order_of_the_launch_drivers(ns, fill, d, n_feed, K, minibatch):
    w = recurrent(ns, d, minibatch, n_feed, K, fill=fill)
    same(run(w, [1, 2, 37], 3), run(w, [40], 3, driver=M.DRIVER_STEPS))


def test_voltage_above_threshold_then_resident_again():
    """Voltages above threshold, which only a caller can set, in the order of the
    persistent kernel."""
    ns = (65, 64)
    V = np.random.default_rng(0).uniform(0.5, 1.5, (2, 65)).astype(np.float32)
    a = recurrent(ns, 1, 2, 3, 5)
    same(run(a, [3, 37], 4, state=V, driver=M.DRIVER_PERSISTENT),
         run(recurrent(ns, 1, 2, 3, 5, rate=True), [40], 4, state=V, driver=M.DRIVER_PERSISTENT))


ANY_VOLTAGE = [((64,), 90, 1, 7, 64, 1), ((130, 200), 85, 2, 7, 64, 3), ((65, 256), 100, 1, 7, 64, 4),
               ((64,), 310, 1, 7, 64, 2)]


@pytest.mark.parametrize("ns,fill,d,n_feed,K,minibatch", ANY_VOLTAGE)
@pytest.mark.parametrize("splits", [[1, 39], [40]])
def test_any_voltage_in_the_launch_drivers_order(ns, fill, d, n_feed, K, minibatch, splits):
    """Voltages that a caller set, far above threshold, infinite and negative
    ones among them, in models that would run on the launch drivers."""
    w = recurrent(ns, d, minibatch, n_feed, K, fill=fill)
    V = np.random.default_rng(1).uniform(-1.0, 3.0, (minibatch, ns[0])).astype(np.float32)
    V[0, :6] = np.inf, -np.inf, 1e30, 1.0, np.nextafter(np.float32(1), np.float32(2)), 40.0
    same(run(w, splits, 3, state=V), run(w, splits, 3, state=V, driver=M.DRIVER_STEPS))


OPTIONS = [dict(planner_depth=1), dict(planner=MS.PLANNER_GREEDY), dict(sort=False), dict(simplify=False),
           dict(merge=False)]


def option_model(fill, rate=False):
    return recurrent((65, 64), 1, 2, 3, 5, rate=rate, fill=fill)


@pytest.mark.parametrize("opts", OPTIONS)
def test_plan_options(opts):
    w = option_model(0)
    same(run(w, [40], 4, driver=M.DRIVER_PERSISTENT, **opts),
         run(option_model(0, rate=True), [40], 4, driver=M.DRIVER_PERSISTENT, **opts))
    w = option_model(90)
    same(run(w, [3, 37], 3, **opts), run(w, [40], 3, driver=M.DRIVER_STEPS, **opts))


def test_the_program_is_what_runs(monkeypatch, capfd):
    monkeypatch.setenv("MS_LOG", "1")
    for w, word in ((option_model(0), "mergesim: resident program"), (option_model(90), "mergesim: resident program"),
                    (option_model(0, rate=True), "mergesim: no resident program: rate neurons")):
        with M.Simulator(M.model_from_spec(w.spec), minibatch=w.minibatch) as sim:
            assert sim.info()["driver"] == M.DRIVER_PERSISTENT
        assert word in capfd.readouterr().err
