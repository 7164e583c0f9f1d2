"""Half-steps of the dense path driven by low Philox draws: a resolving
workgroup's tile where more survivors share it than one turn of its threads
stages (needs an MI355X).

One turn of the 1024 threads stages 16-site pieces of the survivors' rails, so
rails of more than 512 sites (more than 32 pieces) take a second turn for the
tile's last rows.  Lattices are chosen so that column blocks have more survivors
than one turn holds; the decisions are those of numpy in binary32 on the
potential of every site, as in test_gpu_draws.py (no word within 1e-6 p of its
probability), so tallies and states are compared for equality."""
import math

import numpy as np
import pytest

from parity_util import gpu_available
from workloads import BF16X2, Physics, constant

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

VOLT = 1.0


def hop_words(seed, d, n, h, R, L):
    """Philox4x32-10 words of device d's bonds of parity h at step n, [R, bonds]."""
    mask = np.uint64(0xFFFFFFFF)
    blocks, rails = (L + 7) // 8, np.arange(R, dtype=np.uint64)[:, None]
    x = [np.broadcast_to(np.arange(blocks, dtype=np.uint64), (R, blocks)), np.broadcast_to(rails, (R, blocks)),
         np.full((R, blocks), n, dtype=np.uint64), np.full((R, blocks), 16 * d + h, dtype=np.uint64)]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        m0, m1 = x[0] * np.uint64(0xD2511F53), x[2] * np.uint64(0xCD9E8D57)
        x = [(m1 >> np.uint64(32)) ^ x[1] ^ np.uint64(k0), m1 & mask,
             (m0 >> np.uint64(32)) ^ x[3] ^ np.uint64(k1), m0 & mask]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return np.stack(x, axis=-1).reshape(R, -1)[:, :len(range(h, L - 1, 2))]


def coulomb_bound(ph):
    """The exact bound of a hop's Coulomb part: K(1, 0) and K(0, dist) of the
    neighbour rails (rings of more than 2 rail_range rails)."""
    return ph.coulomb_kappa_v * (1.0 + 2.0 * sum(1.0 / k for k in range(1, ph.rail_range + 1)))


def barrier_for(ph, n_bonds, L, mean):
    """Barrier at which `mean` of n_bonds words pass the lattice's stage 0."""
    return (ph.kT_ev * math.log(ph.nu0_hz * ph.dt_s * n_bonds / mean)
            + 0.5 * (abs(ph.field_coupling * VOLT) / L + coulomb_bound(ph)))


def low_word(ph, L):
    """Largest word that may pass stage 0 (no less the library's by its widening)."""
    p = ph.nu0_hz * ph.dt_s * math.exp(-(ph.ea_ev - 0.5 * (VOLT / L + coulomb_bound(ph))) / ph.kT_ev)
    return p * 2.0 ** 32


def dense_half_step(ph, occ, phi, rails, L, n, h):
    """One half-step of `occ` in place, decided in numpy from the potential phi.
    Returns the net hops per device and the survivors of stage 0 per column block."""
    f32 = np.float32
    c0, beta, k10 = f32(ph.nu0_hz * ph.dt_s), f32(1.0 / ph.kT_ev), f32(ph.coulomb_kappa_v)
    s = np.arange(h, L - 1, 2)
    net, per_block = np.zeros(len(rails), dtype=np.int64), np.zeros((L - 1 - h) // 32 + 1, dtype=np.int64)
    off = 0
    for d, R in enumerate(rails):
        o2, p2 = occ[off:off + R * L].reshape(R, L), phi[off:off + R * L].reshape(R, L)
        off += R * L
        w = hop_words(ph.seed, d, n, h, R, L)
        up, b = o2[:, s].astype(bool), o2[:, s + 1].astype(bool)
        po, pt = np.where(up, p2[:, s], p2[:, s + 1]), np.where(up, p2[:, s + 1], p2[:, s])
        e = ((f32(ph.field_coupling) * f32(VOLT)) * np.where(up, f32(1), f32(-1))) / f32(L) + ((pt - k10) - po)
        p = np.minimum(c0 * np.exp(-beta * (f32(ph.ea_ev) + f32(0.5) * e)), f32(1)).astype(f32)
        u = (w.astype(f32) * f32(2.0 ** -32)).astype(f32)
        cand = up ^ b
        assert not np.any(cand & (np.abs(u.astype(np.float64) - p) < 1e-6 * p)), "a word at its threshold"
        np.add.at(per_block, np.broadcast_to((s - h) // 32, w.shape)[cand & (w <= low_word(ph, L))], 1)
        acc = cand & (u < p)
        net[d] += int((acc & ~up).sum()) - int((acc & up).sum())
        o2[:, s] ^= acc.astype(np.int8)
        o2[:, s + 1] ^= acc.astype(np.int8)
    return net, per_block


# sites, rail range, survivors of a tile that one turn of the threads stages
# (1024 // pieces): 20, 24, 28 and 32 column blocks; tiles of 32 rows (whose
# rails fit the LDS) and, at rail ranges 3 and 4, of 16, which one turn always
# holds
@pytest.mark.parametrize("L,m,staged", [(520, 0, 25), (640, 3, 25), (700, 1, 21), (768, 3, 21), (896, 2, 18), (1000, 1, 16),
                                        (1024, 0, 16), (1024, 2, 16), (800, 3, 16), (640, 4, 16), (1000, 4, 16)])
def test_tiles_of_long_rails(L, m, staged):
    from paper_2511_09413_amd import Simulator
    blocks = (L - 2) // 32 + 1
    # about 45 draws in every column block, one resolving workgroup each, and no
    # more than one draw per 128 sites
    mean = 45.0 * blocks
    rails = [-(-int(mean * 128 * 1.1 / L) // 2)] * 2
    ph = Physics(precision=BF16X2, seed=100 + L + m, screening_sites=0.0, cutoff_sites=L - 1, rail_range=m)
    ph = ph.replace(ea_ev=barrier_for(ph, sum(rails) * L / 2, L, mean))
    sim, twin = (Simulator(ph, rails, [L] * 2) for _ in range(2))
    sim.fill_random([0.5] * 2)
    sim.set_bias_protocol(*constant(VOLT))
    occ = sim.read_occupancy().copy()
    most = 0
    for n in range(3):
        net = np.zeros(2, dtype=np.int64)
        for h in (0, 1):
            twin.load_occupancy(occ)
            moved, per_block = dense_half_step(ph, occ, twin.dense_potential().cpu().numpy(), rails, L, n, h)
            net += moved
            most = max(most, int(per_block.max()))
        got, _ = sim.run_steps(1, tallies=True)
        assert np.array_equal(got.cpu().numpy()[0], net), f"step {n}"
        assert np.array_equal(sim.read_occupancy(), occ), f"step {n}"
    assert most > staged, "no tile with more survivors than one turn stages"
    sim.close()
    twin.close()


# rails that fill a few of their padded column blocks, many of them, with close
# to one draw per 128 sites: the first block's resolving workgroups take nearly
# all draws (33 sites or fewer), half of them, or a third
@pytest.mark.parametrize("L,devices", [(20, 51), (33, 31), (40, 26), (65, 16), (129, 8), (140, 7)])
def test_draws_of_short_rails_fit_their_workgroups(L, devices):
    from paper_2511_09413_amd import Simulator
    rails = [1024] * devices
    n_sites = 1024 * devices * L
    ph = Physics(precision=BF16X2, seed=9 + L, screening_sites=0.0, cutoff_sites=L - 1, rail_range=1)
    ph = ph.replace(ea_ev=barrier_for(ph, n_sites / 2, L, 0.985 * min(8192, n_sites / 128)))
    sim, twin = (Simulator(ph, rails, [L] * devices) for _ in range(2))
    sim.fill_random([0.3] * devices)
    sim.set_bias_protocol(*constant(VOLT))
    occ = sim.read_occupancy().copy()
    for n in range(2):
        net = np.zeros(devices, dtype=np.int64)
        for h in (0, 1):
            twin.load_occupancy(occ)
            net += dense_half_step(ph, occ, twin.dense_potential().cpu().numpy(), rails, L, n, h)[0]
        got, _ = sim.run_steps(1, tallies=True)
        assert np.array_equal(got.cpu().numpy()[0], net), f"step {n}"
        assert np.array_equal(sim.read_occupancy(), occ), f"step {n}"
    # (an overfull list is reported by the next read)
    sim.run_steps(1000)
    sim.read_occupancy()
    sim.close()
    twin.close()
