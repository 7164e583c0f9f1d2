"""Set-up kernels at the sizes where they can go wrong (needs an MI355X): the
random placement (the last ion's word found bit by bit) against the oracle's
ranking, the replay's starting Coulomb parts (table sums over window bits)
through the replay against the oracle's, and protocols installed device by
device."""
import numpy as np
import pytest

import oracle
from parity_util import gpu_available
from workloads import FP32, FP64, Physics, constant, step_then_relax

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# piece boundaries of 256 sites, every instance of the kernel, lengths that are
# not a multiple of four, fillings 0 and 1
@pytest.mark.parametrize("rails,sites,fill", [
    ([5, 3], [2, 3], [0.5, 0.34]), ([4, 4, 4], [255, 256, 257], [0.3, 0.0, 1.0]), ([3, 2], [512, 513], [0.05, 0.95]),
    ([3, 2], [1023, 1025], [0.5, 0.3]), ([2, 2], [2048, 2049], [0.3, 0.3]), ([3], [4095], [0.999])])
def test_placement_equals_ranking(rails, sites, fill):
    from paper_2511_09413_amd import Simulator
    for seed in (0, 0xC0FFEE1234):
        ph = Physics(precision=FP32, seed=seed)
        sim = Simulator(ph, rails, sites)
        sim.fill_random(fill)
        assert np.array_equal(sim.read_occupancy(), oracle.fill(oracle.OracleParams(ph, rails, sites), fill))
        sim.close()


# windows of 2 cut + 2 bits: within a byte, at byte edges, 64 bits, and wider
# (the other start-up kernel); rails shorter than the window, rings of 1, 2 and
# 3 rails, a device of more than sixteen rails with a remainder
@pytest.mark.parametrize("cut", [0, 2, 3, 16, 30, 31, 32])
@pytest.mark.parametrize("rails,sites,m", [([1, 2, 3], [20, 70, 33], 2), ([37], [129], 1), ([18, 16], [64, 40], 4)])
def test_replay_from_the_start_state(rails, sites, m, cut):
    """One-step replays: every term comes from the starting Coulomb parts and
    the first half-step's update.  Tolerance: binary64 sums of the same terms in
    another order, 1e-9 of the terms' magnitude (as in test_gpu_score.py)."""
    from paper_2511_09413_amd import Simulator
    ph = Physics(precision=FP64, seed=cut + 3, ea_ev=0.12, coulomb_kappa_v=0.04, cutoff_sites=cut, rail_range=m)
    D = len(rails)
    sim = Simulator(ph, rails, sites)
    sim.fill_random([0.4] * D)
    protos = [constant(0.7)] * D
    sim.set_protocols(protos)
    occ0 = sim.read_occupancy()
    w = np.random.default_rng(1).normal(size=(1, D))
    grad = sim.score_replay(occ0, 0, w).cpu().numpy()
    ref = oracle.score_replay(oracle.OracleParams(ph, rails, sites), protos, occ0, 0, w)
    g, mag = ref["grad"], ref["mag"]
    assert np.all(np.abs(grad - g) <= 1e-9 * mag + 1e-300), (grad, g)
    sim.close()


def test_protocols_set_device_by_device():
    """Runs of equal and different protocols, set in and out of order and again
    after steps, give the trajectories of devices that each had theirs alone."""
    from paper_2511_09413_amd import Simulator
    rails, sites = [6] * 7, [48] * 7
    ph = Physics(precision=FP64, seed=4, ea_ev=0.12)
    p_or = oracle.OracleParams(ph, rails, sites)
    a, b, c = constant(1.5), step_then_relax(-2.0, 15e-12), constant(-0.7)
    sim = Simulator(ph, rails, sites)
    occ = oracle.fill(p_or, [0.35] * 7)
    sim.load_occupancy(occ)
    first = [a, a, a, b, b, a, c]
    for d in (0, 1, 2, 3, 4, 6, 5):
        sim.set_bias_protocol(*first[d], device=d)
    net = sim.run_steps(20, tallies=True)[0].cpu().numpy()
    out = oracle.run(p_or, first, occ, 0, 20)
    assert out["n_log"] > 0 or np.array_equal(net, out["net"])
    for d in (2, 3):                                  # an incomplete run, then the steps
        sim.set_bias_protocol(*b, device=d)
    second, n_set = list(first), [0] * 7
    second[2] = second[3] = b
    n_set[2] = n_set[3] = 20
    net = sim.run_steps(20, tallies=True)[0].cpu().numpy()
    out = oracle.run(p_or, second, occ, 20, 20, n_set=n_set)
    assert out["n_log"] > 0 or np.array_equal(net, out["net"])
    assert np.array_equal(sim.read_occupancy(), occ)
    sim.close()
