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


LONG_RANGE = [(BF16X2, [40, 40], 96), (PHI_FIXED, [40, 40], 96)]


def _long_range(precision, sites):
    return Physics(precision=precision, seed=6, ea_ev=0.2, screening_sites=0.0, cutoff_sites=sites - 1, rail_range=2)


@pytest.mark.parametrize("precision,rails,sites", LONG_RANGE)
def test_a_replay_starts_from_the_state_loaded_before_it(precision, rails, sites):
    """Captured after a run (when both planes of the low-draw half-steps are
    alike), replayed after loads and runs."""
    ph = _long_range(precision, sites)
    sim, ref = (_sim(ph, rails, [sites] * 2) for _ in range(2))
    states = [sim.read_occupancy().copy()]
    for s in (sim, ref):
        s.set_bias_protocol(*constant(1.0))
        _eager(s, 10)
    states.append(sim.read_occupancy().copy())
    graph, net = _capture(sim, 12)
    expect = []
    for occ in states:
        twin = _sim(ph, rails, [sites] * 2)
        twin.set_bias_protocol(*constant(1.0))
        _eager(twin, 10)
        _load(twin, occ)
        expect.append((_eager(twin, 12), twin.read_occupancy()))
        twin.close()
    for k in (0, 1, 0, 1):
        _load(sim, states[k])
        _replay(sim, graph)
        assert np.array_equal(net.cpu().numpy(), expect[k][0])
        assert np.array_equal(sim.read_occupancy(), expect[k][1])
        if k == 1:                       # a replay, then a run from its state
            step = sim.step
            got = _eager(sim, 12)
            twin = _sim(ph, rails, [sites] * 2)
            twin.set_bias_protocol(*constant(1.0))
            _eager(twin, step)
            _load(twin, expect[k][1])
            assert np.array_equal(got, _eager(twin, 12))
            assert np.array_equal(sim.read_occupancy(), twin.read_occupancy())
            twin.close()
    sim.close()
    ref.close()


@pytest.mark.parametrize("precision,rails,sites", LONG_RANGE)
def test_a_captured_first_run_changes_nothing_until_it_is_replayed(precision, rails, sites):
    ph = _long_range(precision, sites)
    sim, ref = (_sim(ph, rails, [sites] * 2) for _ in range(2))
    start = sim.read_occupancy().copy()
    for s in (sim, ref):
        s.set_bias_protocol(*constant(1.0))
    graph, _ = _capture(sim, 12)
    _eager(ref, 12)
    _load(ref, start)
    # (the second plane still holds whatever it held before the load)
    assert np.array_equal(_eager(sim, 12), _eager(ref, 12))
    assert np.array_equal(sim.read_occupancy(), ref.read_occupancy())
    sim.close()
    ref.close()


def test_captured_open_electrodes_replay():
    ph = Physics(precision=FP32, seed=6, ea_ev=0.12)
    sim, ref = (_sim(ph, [24, 24], [80, 80]) for _ in range(2))
    start = sim.read_occupancy().copy()
    for s in (sim, ref):
        s.set_bias_protocol(*constant(1.0))
        s.set_electrodes(0.12, 0.08, 0.12, -0.08)
    graph, net = _capture(sim, 9)
    expect = _eager(ref, 9)
    for _ in range(3):
        _load(sim, start)
        _replay(sim, graph)
        assert np.array_equal(net.cpu().numpy(), expect)
        assert np.array_equal(sim.read_occupancy(), ref.read_occupancy())
    sim.close()
    ref.close()


@pytest.mark.parametrize("gate", [100000, 0])
def test_captured_zone_runs_replay(gate):
    """(constant bias: the table of a loaded state is that of the captured steps)"""
    import torch
    from paper_2511_09413_amd import lib
    from test_gpu_zone import _pair
    with torch.cuda.stream(torch.cuda.Stream()):
        sim, p, X = _pair(601, 50, 21, 10, 0.7, 1e-3, seed=11)
        sim.set_bias_protocol(*constant(2.0))
    sim.set_gate_limit(gate)
    start = sim.read_occupancy().copy()
    import oracle
    out = oracle.zone_run(p, constant(2.0), X, 0, 25)
    net = torch.zeros(25, dtype=torch.int32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=sim.stream):
        assert lib().kmc_zone_run_steps(sim.ctx, 25, net.data_ptr(), None) == 0
    for _ in range(3):
        _load(sim, start)
        _replay(sim, graph)
        assert np.array_equal(net.cpu().numpy(), out["net"])
        assert np.array_equal(sim.read_positions(), X)
    sim.close()
