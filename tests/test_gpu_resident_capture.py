"""GPU: a run of a resident program captured into a graph."""
import numpy as np
import pytest
import torch   # before the library, which then runs on the same HIP runtime

import paper_1805_11144_amd as M
from tests.test_gpu_resident import recurrent

pytestmark = pytest.mark.gpu
MS = M.mergesim


def test_voltages_set_between_replays_of_a_captured_run():
    """A run captured into a graph, replayed with voltages below and above
    threshold set before each replay, against eager runs."""
    w = recurrent((65, 64), 1, 2, 3, 5)
    n, model = 10, M.model_from_spec(w.spec)
    feeds = {i: torch.from_numpy(np.ascontiguousarray(f[:, :n])).cuda() for i, f in w.feeds.items()}
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with M.Simulator(model, minibatch=2, probe_capacity_steps=64, driver=M.DRIVER_PERSISTENT) as eager, \
            M.Simulator(model, minibatch=2, probe_capacity_steps=64, driver=M.DRIVER_PERSISTENT,
                        stream=stream.cuda_stream) as sim:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sim.run_steps(n, feeds)
        for k, top in enumerate((0.9, 1.7, 0.9, 2.5)):
            V = np.random.default_rng(k).uniform(0.0, top, (2, 65)).astype(np.float32)
            for s in (eager, sim):
                s.set_state(MS.STATE_VOLTAGE, 0, V)
            eager.run_steps(n, feeds)
            with torch.cuda.stream(stream):
                graph.replay()
            torch.cuda.synchronize()
            for p in range(4):
                np.testing.assert_array_equal(sim.data(p), eager.data(p)[:, k * n:])


def test_voltages_set_before_a_capture():
    """A run captured but not replayed leaves the voltages to the next eager run."""
    w = recurrent((65, 64), 1, 2, 3, 5)
    n, model = 10, M.model_from_spec(w.spec)
    feeds = {i: torch.from_numpy(np.ascontiguousarray(f[:, :n])).cuda() for i, f in w.feeds.items()}
    V = np.random.default_rng(2).uniform(0.5, 2.5, (2, 65)).astype(np.float32)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with M.Simulator(model, minibatch=2, probe_capacity_steps=64, driver=M.DRIVER_PERSISTENT) as eager, \
            M.Simulator(model, minibatch=2, probe_capacity_steps=64, driver=M.DRIVER_PERSISTENT,
                        stream=stream.cuda_stream) as sim:
        for s in (eager, sim):
            s.set_state(MS.STATE_VOLTAGE, 0, V)
        with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=stream):
            sim.run_steps(n, feeds)
        eager.run_steps(n, feeds)
        sim.run_steps(n, feeds)
        for k in (MS.STATE_VOLTAGE, MS.STATE_REFRACTORY):
            np.testing.assert_array_equal(sim.get_state(k, 0, 65), eager.get_state(k, 0, 65))
        for p in range(4):
            np.testing.assert_array_equal(sim.data(p)[:, n:], eager.data(p))
