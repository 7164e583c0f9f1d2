"""The score replay's starting Coulomb parts from table sums, on lattices of
several devices (needs an MI355X).  One-step replays, every term from the starting
parts and the first half-step's update, against the oracle's; tolerance: binary64
sums of the same terms in another order, 1e-9 of the terms' magnitude (as in
test_gpu_score.py)."""
import numpy as np
import pytest

import oracle
from parity_util import gpu_available
from workloads import FP64, Physics, constant

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# ragged devices, more than the 64 that a workgroup looks up at a time; units of
# four rails with a remainder; rails no longer than the window; the widest
# window and range; units of sixteen rails (32768 rails or more)
@pytest.mark.parametrize("rails,sites,m,cut", [
    ([1, 2, 3] * 24, [20, 70, 33] * 24, 2, 0), ([1, 2, 3] * 24, [20, 70, 33] * 24, 2, 16), ([7, 4, 9, 13], [129] * 4, 1, 3),
    ([7, 4, 9, 13], [129] * 4, 1, 31), ([18, 9] * 5, [64, 40] * 5, 4, 31), ([18, 9] * 5, [64, 40] * 5, 4, 2),
    ([6] * 12, [33, 2] * 6, 4, 30), ([520] * 64, [20] * 64, 1, 8)])
def test_replay_of_several_devices(rails, sites, m, cut):
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
    assert np.all(np.abs(grad - ref["grad"]) <= 1e-9 * ref["mag"] + 1e-300)
    sim.close()
