"""Open electrodes in wave tiles (a device's tiles in one workgroup) and in
half-step launches, against the oracle in lockstep (needs an MI355X): integers
equal outside the logged near-threshold draws."""
import numpy as np
import pytest

import oracle
from parity_util import gpu_available, lockstep
from workloads import FP32, FP64, Physics, constant, gaussian_barriers, triangle

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

EL = (0.12, 0.08, 0.12, -0.08)


# one tile; sixteen tiles (the most in one workgroup) and seventeen; a rail of
# one lane with its end on every place of a lane; 32 sites per lane; windows
# shorter than eight sites, wider than a rail and than a wavefront; rails that
# read none or two neighbours; unequal devices (half-step launches); certain
# and nearly impossible transfers; a closed device among open ones
@pytest.mark.parametrize("mode", [None, "half_step"])
@pytest.mark.parametrize("precision", [FP32, FP64])
@pytest.mark.parametrize("rails,sites,cut,reach,els", [
    ([64, 64], [200, 200], 16, 1, [EL, EL]),
    ([65], [200], 16, 1, [EL]),
    ([2], [2], 3, 1, [EL]),
    ([5], [15], 31, 1, [EL]), ([5], [16], 16, 2, [EL]), ([5], [17], 0, 1, [EL]), ([6], [33], 7, 0, [EL]),
    ([4], [1500], 16, 1, [EL]), ([3], [1025], 40, 1, [EL]),
    ([1], [70], 60, 1, [EL]),
    ([7, 30], [50, 300], 16, 1, [EL, EL]),
    ([9, 9, 9], [64, 64, 64], 16, 1, [(-0.2, 5.0, 0.9, 900.0), None, (0.3, -1500.0, 0.05, 0.0)])])
def test_open_tiles_follow_oracle(mode, precision, rails, sites, cut, reach, els):
    from paper_2511_09413_amd import Simulator
    ph = Physics(precision=precision, seed=cut + 2, ea_ev=0.12, coulomb_kappa_v=0.03, cutoff_sites=cut,
                 rail_range=reach)
    n = sum(r * l for r, l in zip(rails, sites))
    ea = gaussian_barriers((n,), 0.12, 0.01, seed=4, dtype=np.float32 if precision == FP32 else np.float64)
    sim = Simulator(ph, rails, sites, ea=ea)
    if mode:
        sim.set_launch_mode(mode)
    for d, el in enumerate(els):
        if el is not None:
            sim.set_electrodes(*el, device=d)
    p_or = oracle.OracleParams(ph, rails, sites, ea)
    occ0 = oracle.fill(p_or, [0.35] * len(rails))
    sim.load_occupancy(occ0)
    protos = [triangle(2.0, 30e-12), constant(-0.8), constant(0.4)][:len(rails)]
    sim.set_protocols(protos)
    st = lockstep(sim, p_or, protos, occ0, 24, 12, electrodes=els)
    assert sim.launch_mode == "half_step" and st["steps"] == 24 and st["hops"] > 0
    sim.close()
