"""The zone model's multi-step launch (one launch for a call's steps, ions in
registers, the zone sums exchanged between workgroups) against the oracle's zone
model, at the sizes where its shape changes (needs an MI355X).  Both sides
evaluate the same binary64 table and draw the same words, so everything is
compared for equality, as in test_gpu_zone.py."""
import numpy as np
import pytest

import oracle
from parity_util import gpu_available
from test_gpu_zone import _occ, _pair
from workloads import step_then_relax, triangle

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# 256 compute units: up to 2048 rails four wavefronts per workgroup and one rail
# pair each; then sixteen, with 1, 2, 4, 8, 16 pairs up to 8192 x those; beyond
# 131072 rails one launch per step.
@pytest.mark.parametrize("rails", [8, 9, 2047, 2048, 2049, 8192, 8193, 16385, 32770, 65537, 131072, 131073])
def test_multi_step_launch_shapes(rails):
    sites, ions = 24, 9
    sim, p, X = _pair(rails, sites, ions, 5, 0.8, 1e-5, seed=rails)
    proto = step_then_relax(4.0, 0.004)
    sim.set_bias_protocol(*proto)
    for chunk in (1, 6):
        net_g, zon_g = sim.run_steps(chunk, tallies=True)
        out = oracle.zone_run(p, proto, X, sim.step - chunk, chunk)
        assert np.array_equal(net_g.cpu().numpy(), out["net"])
        assert np.array_equal(zon_g.cpu().numpy(), out["zones"])
        assert np.array_equal(sim.read_positions(), X)
    assert np.abs(out["net"]).sum() > 0
    sim.close()


@pytest.mark.parametrize("rails,sites,ions,zones", [(40, 70, 64, 64), (300, 3000, 64, 10), (5, 65534, 3, 3), (1, 64, 63, 2)])
def test_multi_step_launch_wide(rails, sites, ions, zones):
    """Every zone and lane in use, long rails (a large column table), more than
    one launch per call."""
    sim, p, X = _pair(rails, sites, ions, zones, 0.9, 1e-3, seed=rails + zones)
    proto = triangle(5.0, 0.05)
    sim.set_bias_protocol(*proto)
    steps = 4100 if rails == 1 else 90
    net_g, zon_g = sim.run_steps(steps, tallies=True)
    out = oracle.zone_run(p, proto, X, 0, steps)
    assert np.array_equal(net_g.cpu().numpy(), out["net"])
    assert np.array_equal(zon_g.cpu().numpy(), out["zones"])
    assert np.array_equal(sim.read_positions(), X)
    assert np.array_equal(sim.read_occupancy(), _occ(X, rails, sites))
    sim.close()


def test_steps_left_to_one_workgroup():
    """With a gate limit of 0 the workgroups leave at once and one workgroup runs
    the steps; a later call with the default limit goes on from there."""
    sim, p, X = _pair(601, 50, 21, 10, 0.7, 1e-3, seed=11)
    proto = triangle(4.0, 0.06)
    sim.set_bias_protocol(*proto)
    for limit in (0, 100000, 0):
        sim.set_gate_limit(limit)
        net_g, zon_g = sim.run_steps(25, tallies=True)
        out = oracle.zone_run(p, proto, X, sim.step - 25, 25)
        assert np.array_equal(net_g.cpu().numpy(), out["net"])
        assert np.array_equal(zon_g.cpu().numpy(), out["zones"])
        assert np.array_equal(sim.read_positions(), X)
    sim.close()
