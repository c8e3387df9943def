"""GPU: parameters set between the replays of a captured run.  A replay reads
what the eager run would: the weights as they are, in every form that the
kernels read them."""
import numpy as np
import pytest
import torch   # before the library, which then runs on the same HIP runtime

import paper_1805_11144_amd as M
from synth import make_workload
from tests.test_gpu_resident import recurrent

pytestmark = pytest.mark.gpu
MS = M.mergesim


@pytest.mark.parametrize("kind", ["packed", "bf16", "resident"])
def test_replays_read_the_parameters_as_they_are(kind):
    if kind == "resident":
        w, which, opts = recurrent((65, 64), 1, 2, 3, 70), (MS.TRAIN_BIASES, 0), {}
    else:
        w = make_workload("c3", neuron_type="relu", n_steps=10, minibatch=8, n_hidden=72, n_in=24, n_out=3)
        which, opts = (MS.TRAIN_TRANSFORM, 1), dict(gemm_dtype="bf16" if kind == "bf16" else "f32")
    n, model, probes = 10, M.model_from_spec(w.spec), range(len(w.spec.probes))
    feeds = {i: torch.from_numpy(np.ascontiguousarray(f[:, :n])).cuda() for i, f in w.feeds.items()}
    opts.update(minibatch=w.minibatch, probe_capacity_steps=64)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with M.Simulator(model, **opts) as eager, M.Simulator(model, stream=stream.cuda_stream, **opts) as sim:
        sim.run_steps(n, feeds)   # (the window driver sizes its signals in the first run)
        sim.reset()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sim.run_steps(n, feeds)
        p0 = eager.train_param(*which)
        for k, scale in enumerate((1.0, 0.5, 0.5, -1.0)):
            for s in (eager, sim):
                s.set_train_param(*which, p0 * np.float32(scale))
            eager.run_steps(n, feeds)
            with torch.cuda.stream(stream):
                graph.replay()
            torch.cuda.synchronize()
            for p in probes:
                np.testing.assert_array_equal(sim.data(p), eager.data(p)[:, k * n:])
