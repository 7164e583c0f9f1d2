"""Performance cases of the rail-KMC library: the work that a program using it
has done, through its public entry points, at the sizes of the repository's own
workloads, benchmark and tests.

A case is a dict of plain values; `kind` selects the path:

* steps:    Simulator.run_steps with tallies (binary64 or binary32 hop step, one
            device or a batch, with or without per-site barriers, traps or open
            electrodes); the outputs are the per-step net hops and deciles and
            the occupancy.
* dense:    the same with the long-range potential of every site (BF16 hi/lo
            products), and the potential after the steps.
* fixed:    the same with the potential kept in fixed point.
* gradient: one training step of autograd.observables: the forward with its
            observables, and the backward pass (score replay).
* zone:     ZoneSimulator.run_steps with tallies (the paper's own model).

exact() computes the floating outputs in binary64 with torch alone.
"""
import math

import numpy as np
import torch

import paper_2511_09413_amd as kmc
from paper_2511_09413_amd import autograd
from workloads import Physics, c3_batched, constant, gaussian_barriers, sparse_traps, step_then_relax, triangle

KT = 0.0259          # eV
DT = 1e-12           # s
NU0 = 1e12           # Hz
E_CHARGE = 1.602176634e-19


def listed():
    return [
        # the plain validation lattice of the reference model: far too small to
        # fill the GPU, so a step's latency and the call's launches count
        dict(name="small_fp64", kind="steps", precision="fp64", devices=1, rails=64, sites=128, filling=0.2,
             ea=0.3, barriers="one", protocol="constant", volt=0.5, steps=1000),
        # a large device stepped in short calls, as by a program that looks at
        # the current or changes the bias every few steps
        dict(name="large_call_20", kind="steps", precision="fp32", devices=1, rails=4096, sites=1024, filling=0.3,
             ea=0.3, barriers="gaussian", protocol="triangle", volt=2.0, steps=20),
        # the same device in a long run (an I-V sweep)
        dict(name="large_chunk", kind="steps", precision="fp32", devices=1, rails=4096, sites=1024, filling=0.3,
             ea=0.3, barriers="gaussian", protocol="triangle", volt=2.0, steps=1024),
        # a heterogeneous ensemble advanced by one call, every shape ragged
        dict(name="batch_ragged", kind="steps", precision="fp32", devices=256, shape_seed=3, rails=1024, sites=2048,
             filling=0.0, ea=0.3, barriers="one", protocol="mixed", volt=1.0, steps=256),
        # thick devices: rails of more than 2048 sites, an odd count
        dict(name="long_rails", kind="steps", precision="fp32", devices=1, rails=512, sites=3001, filling=0.3,
             ea=0.3, barriers="gaussian", protocol="triangle", volt=2.0, steps=256),
        # deep traps in a soft matrix: a barrier at which hops are common
        dict(name="traps_soft", kind="steps", precision="fp32", devices=1, rails=128, sites=1024, filling=0.3,
             ea=0.15, barriers="traps", protocol="constant", volt=1.0, steps=512),
        # open electrodes on a few replicas of a soft lattice (binary64, as the
        # grand-canonical checks use it)
        dict(name="electrodes", kind="steps", precision="fp64", devices=4, rails=64, sites=200, filling=0.3,
             ea=0.15, barriers="one", protocol="constant", volt=1.0, steps=100, electrodes=True),
        # the long-range interaction of every ion over the whole rail and +-4
        # rails, the potential of every site from the matrix product
        dict(name="dense_mfma", kind="dense", precision="bf16x2", devices=64, rails=1024, sites=512, filling=0.3,
             ea=0.3, steps=10, volt=1.0),
        # the same lattice with the potential kept hop by hop
        dict(name="dense_fixed", kind="fixed", precision="phi_fixed", devices=64, rails=1024, sites=512, filling=0.3,
             ea=0.3, steps=50, volt=1.0),
        # one training step: 512 replicas, forward with observables and the
        # score-function gradient of four parameters
        dict(name="gradient", kind="gradient", devices=512, rails=256, sites=512, filling=0.3, ea=0.3, volt=1.0,
             steps=64),
        # the paper's own zone model, smallest and largest table sizes
        dict(name="zone_500", kind="zone", rails=500, sites=200, zones=10, fraction=0.3, steps=500),
        dict(name="zone_128k", kind="zone", rails=128_000, sites=200, zones=10, fraction=0.3, steps=100),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["steps", "steps", "steps", "open", "dense", "fixed", "gradient", "zone"])
    filling = round(rng.uniform(0.05, 0.4), 3)
    volt = round(rng.uniform(-2.0, 2.0), 3)
    if kind == "steps":
        precision = rng.choice(["fp32", "fp32", "fp64"])
        if rng.random() < 0.2:
            return dict(kind="steps", precision=precision, devices=_log(rng, 4, 64), shape_seed=rng.randrange(1000),
                        rails=_log(rng, 64, 1024), sites=_log(rng, 96, 2048), filling=0.0, ea=0.3, barriers="one",
                        protocol="mixed", volt=1.0, steps=_log(rng, 16, 256))
        soft = rng.random() < 0.3
        rails, sites = _log(rng, 16, 512 if soft else 4096), _log(rng, 40, 1024 if soft else 4096)
        steps = max(8, min(1200, int((3e7 if soft else 2e9) / (rails * sites)), _log(rng, 16, 1200)))
        return dict(kind="steps", precision=precision, devices=1, rails=rails, sites=sites, filling=filling,
                    ea=0.15 if soft else 0.3, barriers=rng.choice(["one", "gaussian", "traps"]),
                    protocol=rng.choice(["constant", "triangle", "relax"]), volt=volt, steps=steps)
    if kind == "open":
        return dict(kind="steps", precision=rng.choice(["fp64", "fp32"]), devices=rng.randint(1, 8),
                    rails=_log(rng, 8, 256), sites=_log(rng, 33, 800), filling=filling, ea=0.15,
                    barriers=rng.choice(["one", "gaussian"]), protocol="constant", volt=volt,
                    steps=_log(rng, 16, 150), electrodes=True)
    if kind in ("dense", "fixed"):
        return dict(kind=kind, precision="bf16x2" if kind == "dense" else "phi_fixed", devices=_log(rng, 1, 64),
                    rails=_log(rng, 32, 1024), sites=rng.choice([512, 128, 200, 333, 401, 256]), filling=filling,
                    ea=0.3 if kind == "dense" else rng.choice([0.3, 0.2]), steps=rng.randint(4, 20), volt=volt)
    if kind == "gradient":
        ea = rng.choice([0.3, 0.15])
        return dict(kind="gradient", devices=_log(rng, 32, 512) if ea == 0.3 else _log(rng, 32, 128),
                    rails=_log(rng, 8, 256) if ea == 0.3 else _log(rng, 8, 32),
                    sites=_log(rng, 32, 512) if ea == 0.3 else _log(rng, 32, 200), filling=filling, ea=ea, volt=volt,
                    steps=_log(rng, 16, 64))
    rails = _log(rng, 500, 128_000)
    return dict(kind="zone", rails=rails, sites=rng.choice([200, 100, 317, 64]), zones=rng.choice([10, 10, 7]),
                fraction=round(rng.uniform(0.1, 0.4), 3), steps=max(16, min(400, 10_000_000 // rails)))


# ------------------------------------------------------------------- inputs
def _physics(case, seed):
    long_range = case["kind"] in ("dense", "fixed")
    return Physics(precision=case.get("precision", "fp32"), seed=seed, ea_ev=case["ea"], kT_ev=KT, dt_s=DT, nu0_hz=NU0,
                   screening_sites=0.0 if long_range else 4.0,
                   cutoff_sites=case["sites"] - 1 if long_range else 16, rail_range=4 if long_range else 1)


def _protocol(case):
    kind, v = case.get("protocol", "constant"), case["volt"]
    if kind == "triangle":
        return triangle(v, 100_000 * DT)
    if kind == "relax":
        return step_then_relax(v, 200 * DT)
    return constant(v)


def _batch(case):
    return c3_batched(n_steps=100_000, n_devices=case["devices"], seed=case["shape_seed"], max_rails=case["rails"],
                      max_sites=case["sites"])


def _simulator(case, seed):
    """A simulator with its barriers, placement, protocols and electrodes set."""
    ph = _physics(case, seed)
    D, shape = case["devices"], (case["devices"], case["rails"], case["sites"])
    if case.get("protocol") == "mixed":
        wl = _batch(case)
        sim = kmc.Simulator(ph, wl.rails, wl.sites)
        sim.fill_random(wl.filling)
        sim.set_protocols(wl.protocols)
        return sim
    dtype = np.float64 if ph.precision == "fp64" else np.float32
    ea = None
    if case.get("barriers") == "gaussian":
        ea = gaussian_barriers(shape, case["ea"], case["ea"] / 15, seed=seed, dtype=dtype)
    elif case.get("barriers") == "traps":
        ea = sparse_traps(shape, case["ea"], 0.005, 0.25, seed + 1, dtype=dtype,
                          field=gaussian_barriers(shape, case["ea"], 0.01, seed=seed, dtype=dtype))
    sim = kmc.Simulator(ph, [case["rails"]] * D, [case["sites"]] * D, ea=ea)
    sim.fill_random([case["filling"]] * D)
    sim.set_bias_protocol(*_protocol(case))
    if case.get("electrodes"):
        sim.set_electrodes(0.12, 0.08, 0.12, -0.08)
    return sim


def _loss_weights(case, seed):
    """Weights of the observables of a training step: of the decile curve
    (per step) and of the mean current."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(case["steps"], dtype=torch.float64, device="cuda", generator=g) / case["steps"], 1e6


def prepare(case, seed):
    if case["kind"] == "zone":
        ions = max(1, int(round(case["fraction"] * case["sites"])))
        g = torch.Generator(device="cuda").manual_seed(seed)
        keys = torch.rand((case["rails"], case["sites"]), device="cuda", generator=g)
        occ = torch.zeros((case["rails"], case["sites"]), dtype=torch.int8, device="cuda")
        occ.scatter_(1, keys.argsort(dim=1)[:, :ions], 1)
        sim = kmc.ZoneSimulator(case["rails"], case["sites"], ions, zones=case["zones"], dt_s=0.016, seed=seed,
                                occ=occ.cpu().numpy())
        sim.set_bias_protocol(*step_then_relax(5.0, 5.0))
        return {"kind": "zone", "sim": sim, "steps": case["steps"]}
    if case["kind"] == "gradient":
        D = case["devices"]
        spec = autograd.ObservableSpec(
            physics=_physics(case, seed), rails=[case["rails"]] * D, sites=[case["sites"]] * D,
            filling=[case["filling"]] * D, protocols=[step_then_relax(case["volt"], (case["steps"] // 2) * DT)] * D,
            n_steps=case["steps"])
        theta = torch.tensor([case["ea"], NU0, 0.025, 1.0], dtype=torch.float64, device="cuda")
        wf, wi = _loss_weights(case, seed)
        return {"kind": "gradient", "spec": spec, "theta": theta, "wf": wf, "wi": wi}
    return {"kind": case["kind"], "sim": _simulator(case, seed), "steps": case["steps"]}


def run(state):
    kind = state["kind"]
    if kind == "gradient":
        theta = state["theta"].clone().requires_grad_(True)
        f, cur = autograd.observables(theta, state["spec"])
        loss = (f.mean(dim=1) * state["wf"]).sum() + state["wi"] * cur.mean()
        loss.backward()
        return {"f": f.detach(), "current": cur.detach(), "grad": theta.grad}
    sim = state["sim"]
    counts, populations = sim.run_steps(state["steps"], tallies=True)
    out = {"net": counts, "populations": populations, "occ": sim.occ}
    if kind == "dense":
        out["phi"] = sim.dense_potential()
    elif kind == "fixed":
        out["phi"] = sim.fixed_potential()[0]
    return out


def work(case):
    """One pass: the state read and written once, the inputs of the path read
    once, the tallies written; the operations are those of the random stream
    (40 per Philox block, one word per ion and trial or per bond and half-step),
    of one potential of every site in the dense kind, and of the terms of every
    candidate in the gradient kind."""
    if case["kind"] == "zone":
        ions = case["rails"] * max(1, int(round(case["fraction"] * case["sites"])))
        return {"bytes": 2 * case["rails"] * case["sites"] + 4 * case["steps"] * (1 + case["zones"]),
                "flops": 20 * ions * case["steps"]}
    if case.get("protocol") == "mixed":
        n = _batch(case).n_sites
    else:
        n = case["devices"] * case["rails"] * case["sites"]
    b = 2 * n + 44 * case["devices"] * case["steps"]
    ops = 10 * n * case["steps"]
    if case.get("barriers", "one") != "one":
        b += n * (8 if case["precision"] == "fp64" else 4)
    if case["kind"] == "dense":
        b += 4 * n
        ops += 2 * n * case["sites"] * 5
    elif case["kind"] == "fixed":
        b += 8 * n
    elif case["kind"] == "gradient":
        # every candidate bond (half-filled bonds of the placement) has one term
        c = 2 * case["filling"] * (1 - case["filling"])
        ops += 12 * c * n * case["steps"]
        b += n * case["steps"] // 4
    return {"bytes": b, "flops": ops}


# ------------------------------------------------------- binary64 in torch
_M0, _M1, _W0, _W1 = 0xD2511F53, 0xCD9E8D57, 0x9E3779B9, 0xBB67AE85
_MASK = 0xFFFFFFFF


def _mul(m, x):
    """(high, low) 32 bits of m * x in int64 tensors."""
    lo16, hi16 = (x & 0xFFFF) * m, (x >> 16) * m
    return (hi16 + (lo16 >> 16)) >> 16, (lo16 + ((hi16 & 0xFFFF) << 16)) & _MASK


def _philox(c0, c1, c2, c3, seed):
    x = list(torch.broadcast_tensors(c0, c1, c2, c3))
    k0, k1 = seed & _MASK, (seed >> 32) & _MASK
    for _ in range(10):
        h0, l0 = _mul(_M0, x[0])
        h1, l1 = _mul(_M1, x[2])
        x = [h1 ^ x[1] ^ k0, l1, h0 ^ x[3] ^ k1, l0]
        k0, k1 = (k0 + _W0) & _MASK, (k1 + _W1) & _MASK
    return torch.stack(x, dim=-1)


class _Exact:
    """The hop model of `devices` equal devices in binary64: checkerboard
    half-steps, potentials by the convolution theorem."""

    def __init__(self, case, seed):
        self.D, self.R, self.L = case["devices"], case["rails"], case["sites"]
        self.seed, ph = seed, _physics(case, seed)
        R, L = self.R, self.L
        i64 = dict(dtype=torch.int64, device="cuda")
        self.d = torch.arange(self.D, **i64).view(-1, 1, 1)
        self.r = torch.arange(R, **i64).view(1, -1, 1)
        self.N = 2 * L
        ds = torch.arange(self.N, **i64)
        ds = torch.minimum(ds, self.N - ds).double()
        dr = torch.arange(R, **i64)
        dr = torch.minimum(dr, R - dr).double()
        dist = (ds.view(1, -1) ** 2 + dr.view(-1, 1) ** 2).sqrt()
        K = ph.coulomb_kappa_v / dist
        if ph.screening_sites > 0:
            K = K * torch.exp(-dist / ph.screening_sites)
        K = torch.where((dist == 0) | (ds.view(1, -1) > ph.cutoff_sites) | (dr.view(-1, 1) > ph.rail_range),
                        torch.zeros_like(K), K)
        self.K10, self.Khat, self.ph = float(K[0, 1]), torch.fft.rfft2(K), ph
        words = _philox(torch.arange((L + 3) // 4, **i64).view(1, 1, -1), self.r, self.d * 0, 16 * self.d + 2, seed)
        ions = int(math.floor(case["filling"] * L + 0.5))
        first = words.flatten(2)[..., :L].argsort(dim=2, stable=True)[..., :ions]
        self.occ = torch.zeros((self.D, R, L), dtype=torch.bool, device="cuda").scatter_(2, first, True)

    def potential(self):
        out = torch.empty((self.D, self.R, self.L), dtype=torch.float64, device="cuda")
        step = max(1, (1 << 25) // (self.R * self.N))
        for a in range(0, self.D, step):
            x = torch.fft.rfft2(self.occ[a:a + step].double(), s=(self.R, self.N)) * self.Khat
            out[a:a + step] = torch.fft.irfft2(x, s=(self.R, self.N))[..., :self.L]
        return out

    def half_step(self, n, h, volt):
        """Takes the half-step; (candidates, accepted, p, Coulomb part, t - o)."""
        L, ph = self.L, self.ph
        blocks = torch.arange((L + 7) // 8, dtype=torch.int64, device="cuda").view(1, 1, -1)
        w = _philox(blocks, self.r, torch.full_like(self.d, n), 16 * self.d + h, self.seed).flatten(2)
        s = torch.arange(h, L - 1, 2, device="cuda")
        a, b = self.occ[..., s], self.occ[..., s + 1]
        phi = self.potential()
        diff = phi[..., s + 1] - phi[..., s]
        cand = a ^ b
        sign = torch.where(a, 1.0, -1.0).double()
        coul = sign * diff - self.K10
        dE = ph.field_coupling * volt * sign / L + coul
        p = (ph.nu0_hz * ph.dt_s * torch.exp(-(ph.ea_ev + 0.5 * dE) / ph.kT_ev)).clamp(max=1.0)
        y = cand & (w[..., :len(s)].double() * 2.0 ** -32 < p)
        self.occ[..., s] = a ^ y
        self.occ[..., s + 1] = b ^ y
        return cand, y, p, coul, sign


def exact(case, seed):
    if case["kind"] == "dense":
        m = _Exact(case, seed)
        for n in range(case["steps"]):
            for h in (0, 1):
                m.half_step(n, h, case["volt"])
        return {"net": None, "populations": None, "occ": None, "phi": m.potential().reshape(-1)}
    if case["kind"] != "gradient":
        return None                      # whole numbers alone
    m = _Exact(case, seed)
    n_steps, D, L = case["steps"], case["devices"], case["sites"]
    f64 = dict(dtype=torch.float64, device="cuda")
    f, cur, scores = torch.empty((n_steps, D), **f64), torch.empty((n_steps, D), **f64), torch.empty((n_steps, D, 4), **f64)
    first = torch.arange(L, device="cuda") * 10 // L == 0
    ions = m.occ.sum(dim=(1, 2)).double().clamp(min=1.0)
    for n in range(n_steps):
        volt = case["volt"] if n < n_steps // 2 else 0.0
        net, sc = torch.zeros(D, **f64), torch.zeros((D, 4), **f64)
        for h in (0, 1):
            cand, y, p, coul, sign = m.half_step(n, h, volt)
            net -= (y * sign).sum(dim=(1, 2))
            t = torch.where(cand & (p < 1.0), (y.double() - p) / (1.0 - p), torch.zeros_like(p))
            sc[:, 0] += t.sum(dim=(1, 2)) * (-1.0 / KT)
            sc[:, 1] += t.sum(dim=(1, 2)) / NU0
            sc[:, 2] += (t * coul).sum(dim=(1, 2)) * (-0.5 / (KT * m.ph.coulomb_kappa_v))
            sc[:, 3] += (t * sign).sum(dim=(1, 2)) * (-0.5 * volt / (L * KT))
        f[n] = m.occ[..., first].sum(dim=(1, 2)).double() / ions
        cur[n] = net * (E_CHARGE / DT / L)
        scores[n] = sc

    def deviation(x):
        return x if D < 2 else x - (x.sum(dim=1, keepdim=True) - x) / (D - 1)

    wf, wi = _loss_weights(case, seed)
    contrib = deviation(f) * (wf.view(-1, 1) / D) + deviation(cur) * (wi / (n_steps * D))
    future = torch.flip(torch.cumsum(torch.flip(contrib, [0]), 0), [0])
    return {"f": f, "current": cur, "grad": (future.unsqueeze(-1) * scores).sum(dim=(0, 1))}
