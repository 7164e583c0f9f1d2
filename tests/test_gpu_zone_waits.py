"""A zone-model run whose workgroups' wait for one another is declared hung (the
limit is set to no polls on the host; every kernel ends normally): each reader
reports it and nothing goes on from the invalid state (needs an MI355X)."""
import numpy as np
import pytest

from parity_util import gpu_available
from test_gpu_zone import _pair
from workloads import constant

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

NO_TALLY = -2 ** 31


@pytest.mark.parametrize("reader", ["positions", "occupancy", "load"])
def test_a_hung_wait_is_reported(reader):
    from paper_2511_09413_amd import KMC_EHIP, KMC_ESTATE, KmcError
    sim, _, X = _pair(601, 50, 21, 10, 0.7, 1e-3, seed=3)
    sim.set_bias_protocol(*constant(2.0))
    before = sim.read_occupancy().copy()
    sim.set_wait_limit(0)
    net, zones = sim.run_steps(12, tallies=True)
    sim.set_wait_limit(1 << 22)
    later, zones_later = sim.run_steps(5, tallies=True)       # enqueued before anyone looked
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
