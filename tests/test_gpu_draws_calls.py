"""Calls of the fixed-point path of all lengths in turn: short ones go by the
decision and update launches, longer ones by low draws, and the state and the
potential pass from one form to the other (needs an MI355X).  Trajectories in
lockstep with the binary64 oracle, the kept potential equal to its recomputation."""
import numpy as np
import pytest

import oracle
from parity_util import gpu_available, lockstep
from workloads import FP64, PHI_FIXED, Physics, constant, gaussian_barriers

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("calls", [[1, 2, 3, 9, 1, 1, 1, 1, 12, 3, 20], [30, 1, 30, 1, 1, 1, 4, 2], [7, 7, 1, 1, 1, 8]])
def test_calls_of_all_lengths(calls):
    from paper_2511_09413_amd import Simulator
    rails, sites = [40, 7, 3], [96, 200, 33]
    ph = Physics(precision=PHI_FIXED, seed=12, ea_ev=0.2, screening_sites=0.0, cutoff_sites=60, rail_range=2)
    ea = gaussian_barriers((sum(r * l for r, l in zip(rails, sites)),), 0.2, 0.01, seed=2, dtype=np.float64)
    sim = Simulator(ph, rails, sites, ea=ea)
    p_or = oracle.OracleParams(ph.replace(precision=FP64), rails, sites, ea)
    protos = [constant(1.0), constant(-0.8), constant(0.4)]
    n_set, hops = [0] * 3, 0
    sim.set_protocols(protos)
    for state in (0.35, 0.2):                          # the calls, then again from a new state
        occ = oracle.fill(p_or, [state] * 3)
        sim.load_occupancy(occ)
        for n in calls:
            st = lockstep(sim, p_or, protos, occ, n, n, n_set=n_set)
            occ, hops = st["occ"], hops + st["hops"]
            kept, _ = sim.fixed_potential()
            fresh, _ = sim.fixed_potential(recompute=True)
            assert bool((kept == fresh).all())
    assert hops > 0
    sim.close()
