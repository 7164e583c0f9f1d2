"""Random placement on short rails (needs an MI355X): the sites with the smallest
(word, site) keys, the oracle's ranking, at the sizes where a lane holds one and
two sites and beyond."""
import numpy as np
import pytest

import oracle
from parity_util import gpu_available
from workloads import FP32, Physics

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("rails,sites,fill", [
    ([5, 3, 2], [2, 3, 64], [0.5, 0.34, 0.3]), ([9, 4], [63, 17], [0.0, 1.0]), ([3, 2, 2], [65, 127, 128], [0.05, 0.95, 0.5]),
    ([2, 7], [129, 64], [0.3, 0.3])])
def test_placement_on_short_rails(rails, sites, fill):
    from paper_2511_09413_amd import Simulator
    for seed in (1, 0xC0FFEE5678):
        ph = Physics(precision=FP32, seed=seed)
        sim = Simulator(ph, rails, sites)
        sim.fill_random(fill)
        assert np.array_equal(sim.read_occupancy(), oracle.fill(oracle.OracleParams(ph, rails, sites), fill))
        sim.close()
