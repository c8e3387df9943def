"""The time-major step program (no GPU) of a model whose ensembles get filtered
and unfiltered connections: the fused synapse group leaves the filtered sum in
the post input at the end of a step, and the copies that add the unfiltered
values in the next step have to stay in the program (they once went with the
post input's reset, so the ensembles saw the filtered part alone)."""
import numpy as np
import pytest

import paper_1805_11144_amd as M
from oracle.sim import OracleSim
from synth.configs import lif_ensemble
from synth.spec import Connection, ModelSpec, Node, Probe, Workload
from tests.plan_exec import LaunchExecutor


def passthrough_model(minibatch, n_steps=12) -> Workload:
    """Passthrough nodes whose rows are read in pieces, in another order, by two
    readers, by filters, and by a probe; ensembles with a filtered and an
    unfiltered input each."""
    rng = np.random.default_rng(3)
    spec = ModelSpec(dt=0.001)
    u = spec.add_node(Node(size=4))
    p, q, r = (spec.add_node(Node(size=4, passthrough=True)) for _ in range(3))
    spec.connect(Connection(pre=u, post=p, transform=1.0, synapse=0.005))
    spec.connect(Connection(pre=p, post=q, transform=1.0, pre_slice=(2, 4), post_slice=(0, 2)))
    spec.connect(Connection(pre=p, post=q, transform=1.0, pre_slice=(0, 2), post_slice=(2, 4)))
    spec.connect(Connection(pre=q, post=r, transform=1.0))
    for s in ((0, 2), (1, 3), (2, 4)):
        e = spec.add_ensemble(lif_ensemble(rng, 30, 2, 50, "lif_rate"))
        spec.connect(Connection(pre=q, post=("ens", e), transform=1.0, pre_slice=s))
        spec.connect(Connection(pre=q, post=("ens", e), transform=rng.standard_normal((2, 4)), synapse=0.01))
        spec.probe(Probe(target=("ens", e)))
    spec.probe(Probe(target=r, synapse=0.005))
    spec.probe(Probe(target=q))
    feed = rng.standard_normal((minibatch, n_steps, 4)).astype(np.float32)
    return Workload("passthrough", spec, minibatch, n_steps, {u[1]: feed})


@pytest.mark.parametrize("fuse", [True, M.mergesim.FUSE_ENSEMBLES, M.mergesim.FUSE_SYNAPSES, False])
def test_filtered_and_unfiltered_inputs(fuse):
    w = passthrough_model(2)
    plan = M.Plan(M.model_from_spec(w.spec), minibatch=2, fuse=fuse)
    ref = OracleSim(w.spec, minibatch=2, param_dtype=np.float32)
    ex = LaunchExecutor(plan, w.spec, 2, params_from=ref)
    ex.run(5, {k: f[:, :5] for k, f in w.feeds.items()})
    ex.run(7, {k: f[:, 5:] for k, f in w.feeds.items()})
    ref.run_steps(12, w.feeds)
    for p in range(len(w.spec.probes)):
        np.testing.assert_allclose(ex.data(p), ref.data(p), rtol=0, atol=1e-11)
