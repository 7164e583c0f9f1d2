"""The wave kernel's survivor groups and its 64-sites-per-lane tiles against the
oracle (needs an MI355X): trajectories, tallies and occupancy in lockstep, as
in test_gpu_parity.py (integers equal outside the logged near-threshold
draws)."""
import numpy as np
import pytest

import oracle
from parity_util import gpu_available, lockstep
from workloads import FP32, FP64, Physics, constant, gaussian_barriers, triangle

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _run(ph, rails, sites, ea, steps, chunk, mode, fill=0.35):
    from paper_2511_09413_amd import Simulator
    sim = Simulator(ph, rails, sites, ea=ea)
    if mode:
        sim.set_launch_mode(mode)
    p_or = oracle.OracleParams(ph, rails, sites, ea)
    occ0 = oracle.fill(p_or, [fill] * len(rails))
    sim.load_occupancy(occ0)
    protos = [triangle(2.0, 60e-12), constant(-0.8), constant(0.4)][:len(rails)]
    sim.set_protocols(protos)
    st = lockstep(sim, p_or, protos, occ0, steps, chunk)
    assert sim.launch_mode == "wave" and st["steps"] == steps
    return st


# windows of 2 cut + 2 sites: one site, just under and at a wavefront's width,
# and wider (one survivor at a time); rails shorter than the window; a
# barrier at which a tile has several survivors per half-step (more than one
# group round) and one at which nearly every candidate survives
@pytest.mark.parametrize("precision", [FP32, FP64])
@pytest.mark.parametrize("cut", [0, 1, 15, 30, 31, 32])
@pytest.mark.parametrize("ea_ev", [0.1, 0.02])
def test_survivor_groups(precision, cut, ea_ev):
    ph = Physics(precision=precision, seed=cut + 1, ea_ev=ea_ev, coulomb_kappa_v=0.03, cutoff_sites=cut)
    rails, sites = [33, 2, 7], [40, 333, 1024]
    ea = gaussian_barriers((sum(r * l for r, l in zip(rails, sites)),), ea_ev, ea_ev / 10, seed=9,
                           dtype=np.float32 if precision == FP32 else np.float64)
    st = _run(ph, rails, sites, ea, 24, 12, "wave")
    assert st["hops"] > 100


# 64 sites per lane: the shortest such rails, odd lengths, the longest; one
# rail, rails on several tiles, a short device beside a long one; a window
# wider than a wavefront
@pytest.mark.parametrize("rails,sites,cut,precision", [
    ([5], [2049], 16, FP32), ([1], [4096], 16, FP64), ([12], [3001], 16, FP32), ([3], [2064], 40, FP64),
    ([6, 40], [4095, 100], 16, FP32), ([2, 9], [2177, 64], 31, FP64)])
def test_long_rails_in_wave_tiles(rails, sites, cut, precision):
    ph = Physics(precision=precision, seed=5, ea_ev=0.14, cutoff_sites=cut)
    n = sum(r * l for r, l in zip(rails, sites))
    ea = gaussian_barriers((n,), 0.14, 0.01, seed=3, dtype=np.float32 if precision == FP32 else np.float64)
    st = _run(ph, rails, sites, ea, 60, 30, None)
    assert st["hops"] > 20
    from paper_2511_09413_amd import KMC_EUNSUPPORTED, KmcError, Simulator
    with pytest.raises(KmcError) as e:                 # an explicit request is refused for such rails
        Simulator(ph, rails, sites, ea=ea, mode="wave")
    assert e.value.status == KMC_EUNSUPPORTED
