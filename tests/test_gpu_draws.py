"""Half-steps of the long-range paths driven by their low Philox draws (needs an
MI355X).

* Fixed-point potential: trajectories in lockstep with the binary64 oracle, and
  the potential kept hop by hop equal to its recomputation, as in
  test_gpu_phifix.py.
* Dense potential: such a half-step evaluates the potential of the few sites
  that a decision needs with the products of the full potential, so a decision
  made from kmc_dense_potential of the same state with the same arithmetic
  agrees; here every accepted hop of a step is compared with that decision,
  taken in numpy in binary32 with the operations in the same order.  The two
  exponentials may differ in their last bits (2 ulp each, 5e-7 of p in all):
  the inputs have no word within 1e-6 p of its probability.
"""
import numpy as np
import pytest

import oracle
from parity_util import gpu_available, lockstep
from workloads import BF16X2, FP64, PHI_FIXED, Physics, constant, gaussian_barriers, step_then_relax, triangle

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# (rails, sites, filling, rail range, cutoff, barrier): partial and odd column
# blocks and rails; small rings whose rails meet (also at half the ring); the
# longest rails (products of 16 survivors); ragged devices (fixed only); a
# barrier with many draws per half-step, and one with none for many steps
DENSE = [([40, 40, 7], 96, 0.3, 4, 95, 0.2), ([5, 8, 1, 2, 3], 130, 0.5, 4, 129, 0.19), ([64] * 4, 512, 0.3, 4, 511, 0.22),
         ([24], 1000, 0.4, 2, 999, 0.2), ([300], 33, 0.45, 0, 20, 0.17), ([3, 260], 64, 0.5, 1, 16, 0.16),
         ([60], 256, 0.3, 4, 255, 0.4)]


def _philox_hop_words(seed, d, n, h, R, L):
    s = np.arange(h, L - 1, 2)
    return s, np.array([[oracle.hop_word(seed, d, n, r, int(x)) for x in s] for r in range(R)], dtype=np.uint64)


@pytest.mark.parametrize("rails,L,fill,m,cut,ea", DENSE)
@pytest.mark.parametrize("barriers", [False, True])
def test_dense_half_steps_decide_from_the_potential(rails, L, fill, m, cut, ea, barriers):
    from paper_2511_09413_amd import Simulator
    D, steps = len(rails), 6
    ph = Physics(precision=BF16X2, seed=17 + L, ea_ev=ea, screening_sites=0.0, cutoff_sites=cut, rail_range=m)
    n_sites = sum(rails) * L
    field = gaussian_barriers((n_sites,), ea, 0.01, seed=2, dtype=np.float32) if barriers else None
    sim = Simulator(ph, rails, [L] * D, ea=field)
    sim.fill_random([fill] * D)
    proto = step_then_relax(1.5, 3 * ph.dt_s)
    sim.set_protocols([proto] * D)
    # the same lattice stepped half by half in numpy, its potential from the
    # product over every site (a second context holding the state)
    twin = Simulator(ph, rails, [L] * D, ea=field)
    occ = sim.read_occupancy().copy()
    f32 = np.float32
    c0, beta, k10 = f32(ph.nu0_hz * ph.dt_s), f32(1.0 / ph.kT_ev), f32(ph.coulomb_kappa_v if cut >= 1 else 0.0)
    hops = 0
    for n in range(steps):
        V = f32(oracle.protocol_voltage(*proto, n * ph.dt_s))
        net_ref = np.zeros(D, dtype=np.int64)
        for h in (0, 1):
            twin.load_occupancy(occ)
            phi = twin.dense_potential().cpu().numpy()
            off = 0
            for d, R in enumerate(rails):
                o2 = occ[off:off + R * L].reshape(R, L)
                p2 = phi[off:off + R * L].reshape(R, L)
                s, w = _philox_hop_words(ph.seed, d, n, h, R, L)
                a, b = o2[:, s].astype(bool), o2[:, s + 1].astype(bool)
                up = a
                po, pt = np.where(up, p2[:, s], p2[:, s + 1]), np.where(up, p2[:, s + 1], p2[:, s])
                e = ((f32(ph.field_coupling) * V) * np.where(up, f32(1), f32(-1))) / f32(L) + ((pt - k10) - po)
                if barriers:
                    e2 = field[off:off + R * L].reshape(R, L)
                    bar = np.where(up, e2[:, s], e2[:, s + 1])
                else:
                    bar = f32(ea)
                p = np.minimum(c0 * np.exp(-beta * (bar + f32(0.5) * e)), f32(1)).astype(f32)
                u = (w.astype(np.float32) * f32(2.0 ** -32)).astype(f32)
                cand = a ^ b
                assert not np.any(cand & (np.abs(u.astype(np.float64) - p) < 1e-6 * p)), "a word at its threshold"
                acc = cand & (u < p)
                net_ref[d] += int((acc & ~up).sum()) - int((acc & up).sum())
                hops += int(acc.sum())
                o2[:, s] ^= acc.astype(np.int8)
                o2[:, s + 1] ^= acc.astype(np.int8)
                off += R * L
        net, _ = sim.run_steps(1, tallies=True)
        assert np.array_equal(net.cpu().numpy()[0], net_ref), f"step {n}"
        assert np.array_equal(sim.read_occupancy(), occ), f"step {n}"
    assert hops > 0 or ea > 0.3
    # one call of several steps takes the same steps
    one = Simulator(ph, rails, [L] * D, ea=field)
    one.fill_random([fill] * D)
    one.set_protocols([proto] * D)
    net, dec = one.run_steps(steps, tallies=True)
    assert np.array_equal(one.read_occupancy(), occ)
    edges = (np.arange(L) * 10) // L
    off = 0
    for d, R in enumerate(rails):
        o2 = occ[off:off + R * L].reshape(R, L)
        assert np.array_equal(dec[-1, d].cpu().numpy(), [int(o2[:, edges == k].sum()) for k in range(10)])
        off += R * L
    for x in (sim, twin, one):
        x.close()


@pytest.mark.parametrize("rails,sites,m,cut,ea", [
    ([40, 7, 3], [96, 200, 33], 4, 60, 0.2), ([64] * 4, [512] * 4, 4, 511, 0.22), ([2, 5], [2048, 1500], 2, 700, 0.2),
    ([30], [65], 0, 64, 0.17), ([33, 33], [128, 64], 1, 16, 0.4)])
def test_fixed_half_steps_follow_the_oracle(rails, sites, m, cut, ea):
    from paper_2511_09413_amd import Simulator
    D = len(rails)
    ph = Physics(precision=PHI_FIXED, seed=5, ea_ev=ea, screening_sites=0.0, cutoff_sites=cut, rail_range=m)
    n = sum(r * l for r, l in zip(rails, sites))
    field = gaussian_barriers((n,), ea, 0.01, seed=2, dtype=np.float64)
    sim = Simulator(ph, rails, sites, ea=field)
    p_or = oracle.OracleParams(ph.replace(precision=FP64), rails, sites, field)
    occ0 = oracle.fill(p_or, [0.35] * D)
    sim.load_occupancy(occ0)
    protos = [triangle(2.0, 40e-12), constant(-0.8), constant(0.4), constant(1.0)][:D]
    sim.set_protocols(protos)
    st = lockstep(sim, p_or, protos, occ0, 30, 10)
    assert st["steps"] == 30 and (st["hops"] > 0 or ea > 0.3)
    kept, _ = sim.fixed_potential()
    fresh, _ = sim.fixed_potential(recompute=True)
    assert bool((kept == fresh).all())
    # a new state, then single steps
    occ1 = oracle.fill(p_or, [0.2] * D)
    sim.load_occupancy(occ1)
    sim.set_protocols(protos)
    before = sim.step
    for k in range(4):
        net, _ = sim.run_steps(1, tallies=True)
        out = oracle.run(p_or, protos, occ1, before + k, 1, n_set=[before] * D)
        assert out["n_log"] > 0 or np.array_equal(net.cpu().numpy(), out["net"])
    kept, _ = sim.fixed_potential()
    fresh, _ = sim.fixed_potential(recompute=True)
    assert bool((kept == fresh).all())
    sim.close()
