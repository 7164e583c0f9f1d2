"""Zone-model runs whose workgroups cannot wait for one another (needs an MI355X).

* A wait that is declared hung (the limit is set to no polls on the host; every
  kernel ends normally): each reader reports it and nothing goes on from the
  invalid state.
* A launch that leaves at its gate (the limit is set to no time): its steps are
  taken from the queue of tiles, with the oracle's trajectory."""
import numpy as np
import pytest

import oracle
from parity_util import gpu_available
from test_gpu_zone import _pair
from workloads import constant, step_then_relax, triangle

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

NO_TALLY = -2 ** 31


# (a single step of the larger lattice is a launch of its own kind)
@pytest.mark.parametrize("reader,rails,steps", [("positions", 601, 5), ("occupancy", 601, 1), ("load", 601, 5),
                                                ("occupancy", 16387, 1)])
def test_a_hung_wait_is_reported(reader, rails, steps):
    from paper_2511_09413_amd import KMC_EHIP, KMC_ESTATE, KmcError
    sim, _, X = _pair(rails, 50, 21, 10, 0.7, 1e-3, seed=3)
    sim.set_bias_protocol(*constant(2.0))
    before = sim.read_occupancy().copy()
    sim.set_wait_limit(0)
    net, zones = sim.run_steps(12, tallies=True)
    sim.set_wait_limit(1 << 22)
    later, zones_later = sim.run_steps(steps, tallies=True)      # enqueued before anyone looked
    for t in (net, zones, later, zones_later):
        assert bool((t == NO_TALLY).all())
    with pytest.raises(KmcError) as e:
        {"positions": sim.read_positions, "occupancy": sim.read_occupancy,
         "load": lambda: sim.load_occupancy(before)}[reader]()
    assert e.value.status == KMC_EHIP
    with pytest.raises(KmcError) as e:
        sim.run_steps(1)
    assert e.value.status == KMC_ESTATE
    sim.close()


# one tile and two; a tile's last pair without its second rail; a workgroup per
# compute unit with one and with two rail pairs per wavefront, most rails; more
# steps than a launch takes; every lane and zone
@pytest.mark.parametrize("rails,sites,ions,zones,steps", [
    (33, 24, 9, 5, 40), (35, 24, 9, 5, 40), (601, 50, 21, 10, 4100), (4097, 24, 9, 5, 12), (12345, 70, 64, 64, 12),
    (131072, 24, 9, 5, 6)])
def test_steps_from_the_queue(rails, sites, ions, zones, steps):
    sim, p, X = _pair(rails, sites, ions, zones, 0.8, 1e-5, seed=rails)
    proto = triangle(4.0, 0.06) if zones > 5 else step_then_relax(4.0, 0.004)
    sim.set_bias_protocol(*proto)
    for limit, chunk in ((0, steps), (100000, 3), (0, 2)):
        sim.set_gate_limit(limit)
        net, zon = sim.run_steps(chunk, tallies=True)
        out = oracle.zone_run(p, proto, X, sim.step - chunk, chunk)
        assert np.array_equal(net.cpu().numpy(), out["net"])
        assert np.array_equal(zon.cpu().numpy(), out["zones"])
        assert np.array_equal(sim.read_positions(), X)
    sim.close()
