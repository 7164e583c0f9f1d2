"""Wave tiles of 64 sites per lane, the automatic choice for long rails that the
persistent kernel does not hold, and the queue of half-steps that takes a
launch's steps when it leaves at its gate (needs an MI355X).  The reference is
the half-step strategy, which the parity tests hold against the oracle: all
strategies take bit-identical decisions, so tallies and states are equal."""
import math

import numpy as np
import pytest

from parity_util import gpu_available
from workloads import FP32, FP64, Physics, constant, gaussian_barriers, triangle

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _barrier(ph, sites, words):
    """Barrier at which about `words` words of a rail pass their threshold per half-step."""
    reach = math.exp(-1.0 / ph.screening_sites) if ph.cutoff_sites >= 1 else 0.0
    bound = ph.coulomb_kappa_v * (reach + 2 * ph.rail_range * math.exp(-1.0 / ph.screening_sites))
    return ph.kT_ev * math.log(sites / (2 * words)) + bound / 2


def _make(rails, sites, cut, precision, words=1.5, sigma=0.004):
    """(simulator with the automatic strategy, one with half-steps)."""
    from paper_2511_09413_amd import KMC_EUNSUPPORTED, KmcError, Simulator
    ph = Physics(precision=precision, seed=5, cutoff_sites=cut)
    ph = ph.replace(ea_ev=_barrier(ph, max(sites), words))
    n = sum(r * l for r, l in zip(rails, sites))
    ea = gaussian_barriers((n,), ph.ea_ev, sigma, seed=3, dtype=np.float32 if precision == FP32 else np.float64)
    sim, ref = Simulator(ph, rails, sites, ea=ea), Simulator(ph, rails, sites, ea=ea, mode="half_step")
    with pytest.raises(KmcError) as e:                 # the persistent kernel does not hold it
        sim.set_launch_mode("persistent")
    assert e.value.status == KMC_EUNSUPPORTED and sim.launch_mode == "wave"
    for s in (sim, ref):
        s.fill_random([0.35] * len(rails))
        s.set_protocols([triangle(2.0, 60e-12), constant(-0.8)][:len(rails)])
    return sim, ref


def _same(sim, ref, steps):
    net, dec = sim.run_steps(steps, tallies=True)
    net_ref, dec_ref = ref.run_steps(steps, tallies=True)
    assert np.array_equal(net.cpu().numpy(), net_ref.cpu().numpy())
    assert np.array_equal(dec.cpu().numpy(), dec_ref.cpu().numpy())
    assert np.array_equal(sim.read_occupancy(), ref.read_occupancy())
    assert np.array_equal(sim.read_current()[1], ref.read_current()[1])
    return int(np.abs(net_ref.cpu().numpy()).sum())


# the shortest such rails, odd lengths, the longest; a window wider than a
# wavefront; a short device beside the long one; from the launch itself and,
# with no time at the gate, from the queue
@pytest.mark.parametrize("gate", [100000, 0])
@pytest.mark.parametrize("rails,sites,cut,precision", [
    ([640], [2049], 16, FP32), ([515], [4096], 16, FP64), ([514], [3001], 31, FP32), ([641], [2064], 40, FP64),
    ([640, 40], [2177, 100], 16, FP32), ([1100], [2100], 16, FP32)])
def test_long_rails(rails, sites, cut, precision, gate):
    sim, ref = _make(rails, sites, cut, precision, words=0.9 if cut > 31 else 1.5)
    sim.set_gate_limit(gate)
    # (calls of less than four steps go by half-steps)
    hops = sum(_same(sim, ref, steps) for steps in (14, 3, 4, 1, 40))
    assert hops > 100
    # a new state and a new protocol
    occ = sim.read_occupancy()[::-1].copy()
    for s in (sim, ref):
        s.load_occupancy(occ)
        s.set_bias_protocol(*constant(-1.5))
    _same(sim, ref, 20)
    sim.close()
    ref.close()


# lattices that the persistent kernel holds too, which takes the calls of less
# than 20 steps: words on both sides of the rule's line, per-site barriers and one
@pytest.mark.parametrize("gate", [100000, 0])
@pytest.mark.parametrize("rails,sites,cut,precision,words,sigma", [
    ([26], [2351], 16, FP32, 0.03, 0.0), ([8], [4096], 16, FP64, 0.03, 0.004), ([64], [2049], 40, FP32, 0.02, 0.004),
    ([40, 30], [3001, 2100], 16, FP64, 0.03, 0.0), ([64], [2500], 16, FP32, 0.3, 0.0)])
def test_long_rails_that_the_persistent_kernel_holds(rails, sites, cut, precision, words, sigma, gate):
    from paper_2511_09413_amd import Simulator
    ph = Physics(precision=precision, seed=5, cutoff_sites=cut)
    ph = ph.replace(ea_ev=_barrier(ph, max(sites), words))
    ea = None
    if sigma:
        n = sum(r * l for r, l in zip(rails, sites))
        ea = gaussian_barriers((n,), ph.ea_ev, sigma, seed=3, dtype=np.float32 if precision == FP32 else np.float64)
    sim, ref = Simulator(ph, rails, sites, ea=ea), Simulator(ph, rails, sites, ea=ea, mode="half_step")
    sim.set_launch_mode("persistent")
    sim.set_launch_mode("auto")
    for s in (sim, ref):
        s.fill_random([0.35] * len(rails))
        s.set_protocols([triangle(2.0, 60e-12), constant(-0.8)][:len(rails)])
    sim.set_gate_limit(gate)
    assert sum(_same(sim, ref, steps) for steps in (20, 19, 1500, 3, 21)) > 0
    sim.close()
    ref.close()


def test_which_calls_wait_for_neighbours():
    """With no polls a neighbour wait is declared hung: the calls in wave tiles
    report it, those in half-steps have no such wait."""
    from paper_2511_09413_amd import KMC_EHIP, KmcError
    for words, steps, waits in ((1.5, 3, False), (1.5, 8, True), (40.0, 8, False)):
        sim, ref = _make([514], [3001], 16, FP32, words=words)
        sim.set_wait_limit(0)
        sim.run_steps(steps)
        if waits:
            with pytest.raises(KmcError) as e:
                sim.read_occupancy()
            assert e.value.status == KMC_EHIP
        else:
            ref.run_steps(steps)
            assert np.array_equal(sim.read_occupancy(), ref.read_occupancy())
        sim.close()
        ref.close()


def test_steps_from_the_queue_are_recorded():
    """More steps than one launch takes, recorded for the replay, whose terms are
    those of decisions drawn again, summed in another order."""
    sim, ref = _make([640], [2100], 16, FP32, words=0.8, sigma=0.0)
    sim.set_gate_limit(0)
    start = sim.snapshot()
    sim.record_hops(1030, cap=2048)
    assert _same(sim, ref, 1030) > 1000
    w = np.ones((1030, 1))
    recorded = sim.score_replay(start, 0, w).cpu().numpy()
    sim.record_hops(0)
    drawn = sim.score_replay(start, 0, w).cpu().numpy()
    assert np.all(np.abs(recorded - drawn) <= 1e-6 * np.abs(drawn))
    sim.close()
    ref.close()


def test_captured_long_rails_replay():
    """A captured run of long rails, replayed after loads (its launches publish
    nothing that the next replay could mistake for its own)."""
    import torch
    from test_gpu_capture import _capture, _load, _replay
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sim, ref = _make([514], [3001], 16, FP32)
    start = sim.read_occupancy().copy()
    graph, net = _capture(sim, 12)
    with torch.cuda.stream(stream):
        expect = ref.run_steps(12, tallies=True)[0].cpu().numpy()
    for _ in range(3):
        _load(sim, start)
        _replay(sim, graph)
        assert np.array_equal(net.cpu().numpy(), expect)
        assert np.array_equal(sim.read_occupancy(), ref.read_occupancy())
    sim.close()
    ref.close()
