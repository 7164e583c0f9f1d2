"""Runs captured into a HIP graph and replayed (needs an MI355X): a replay takes
the captured steps (their indices are fixed) from the state and the protocols
that the context holds when it runs, as launches of the same calls would."""
import numpy as np
import pytest

from parity_util import gpu_available
from workloads import BF16X2, FP32, PHI_FIXED, Physics, constant

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _sim(ph, rails, sites, mode="auto", ea=None):
    """A simulator on a stream of its own (a capture needs one)."""
    import torch
    from paper_2511_09413_amd import Simulator
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sim = Simulator(ph, rails, sites, mode=mode, ea=ea)
        sim.fill_random([0.3] * len(rails))
    return sim


def _capture(sim, steps):
    """(graph, tallies of its replays) of run_steps(steps)."""
    import torch
    from paper_2511_09413_amd import run_steps
    torch.cuda.synchronize()
    net = torch.zeros((steps, sim.n_devices), dtype=torch.int32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=sim.stream):
        run_steps(sim.ctx, steps, net.data_ptr())
    return graph, net


def _load(sim, occ):
    import torch
    with torch.cuda.stream(sim.stream):
        sim.load_occupancy(occ)
    torch.cuda.synchronize()


def _replay(sim, graph):
    import torch
    with torch.cuda.stream(sim.stream):
        graph.replay()
    torch.cuda.synchronize()


def _eager(sim, steps):
    import torch
    with torch.cuda.stream(sim.stream):
        net = sim.run_steps(steps, tallies=True)[0]
    torch.cuda.synchronize()
    return net.cpu().numpy()


def test_a_replay_uses_the_protocols_installed_when_it_runs():
    """The protocol of one device of several is installed by its call, not by
    the next run (which is captured)."""
    ph = Physics(precision=FP32, seed=8, ea_ev=0.1)
    rails, sites = [30, 30], [64, 64]
    sim, ref = (_sim(ph, rails, sites, mode="half_step") for _ in range(2))
    start = sim.read_occupancy().copy()
    sim.set_bias_protocol(*constant(3.0), device=0)
    graph, net = _capture(sim, 4)
    sim.set_bias_protocol(*constant(-3.0), device=0)
    ref.set_bias_protocol(*constant(-3.0), device=0)
    expect = _eager(ref, 4)
    for _ in range(3):
        _load(sim, start)
        _replay(sim, graph)
        assert np.array_equal(net.cpu().numpy(), expect)
        assert np.array_equal(sim.read_occupancy(), ref.read_occupancy())
