"""Measured cases of the framework: the calls its users make, over their real range.

A particle set is drawn from the seed with the repository's own generators, the tree
(or the simulation, the network) is what a program has in hand, and one pass is one
call through the Python binding:

* ``forces``   ``Tree.forces`` on a resident tree (opening angle, or the learned criterion)
* ``oneshot``  ``Tree(..., device_build=True)`` from host arrays, then ``forces``
* ``sim``      ``Sim.run`` of some leapfrog steps (tree rebuilt every step), then the
               state and the energies
* ``direct``   ``Tree.direct``, the reference sum, for sampled targets or for all particles
* ``train``    one mini-batch step of the network: ``Mlp.loss_grad`` and ``Mlp.adam``
"""
import math

import numpy as np
import torch

from paper_1005_5384_amd import learned as L
from paper_1005_5384_amd import octgrav as og
from paper_1005_5384_amd import workloads as W

# The learned criterion where the benchmark uses it: theta* = 0.5625 with the band
# (theta* - 0.015, theta* + 0.25), the threshold calibrated there, a budget of 30 thresholds.
MAC_LO, MAC_HI, MAC_TAU = 0.5475, 0.8125, 3.46e-4


def listed():
    return [
        # A star cluster of a thousand bodies: latency and launches are everything.
        {"name": "forces_cluster_1k", "kind": "forces", "gen": "plummer", "n": 1000, "theta": 0.5,
         "eps": 0.01, "n_leaf": 16, "n_group": 64, "mac": "theta"},
        # The small benchmark workload; fewer work items than the chip holds waves.
        {"name": "forces_plummer_16k", "kind": "forces", "gen": "plummer", "n": 16384, "theta": 0.5,
         "eps": 0.01, "n_leaf": 16, "n_group": 64, "mac": "theta"},
        # A mid-size galaxy at a ragged size and a wide opening angle: short lists.
        {"name": "forces_galaxy_200k_wide", "kind": "forces", "gen": "milky_way", "n": 200003,
         "theta": 0.75, "eps": 1e-3, "n_leaf": 16, "n_group": 64, "mac": "theta"},
        # The headline workload.
        {"name": "forces_plummer_1m", "kind": "forces", "gen": "plummer", "n": 1 << 20, "theta": 0.5,
         "eps": 1e-3, "n_leaf": 16, "n_group": 64, "mac": "theta"},
        # The clustered workload with larger leaves, the largest force call.
        {"name": "forces_clumps_4m", "kind": "forces", "gen": "plummer_clumps", "n": 1 << 22,
         "theta": 0.5, "eps": 1e-3, "n_leaf": 32, "n_group": 64, "mac": "theta"},
        # The headline set under the learned criterion at its operating point.
        {"name": "forces_learned_1m", "kind": "forces", "gen": "plummer", "n": 1 << 20,
         "theta": 0.5625, "eps": 1e-3, "n_leaf": 16, "n_group": 64, "mac": "learned"},
        # Forces of a snapshot that is in host memory: build on the GPU, one evaluation.
        {"name": "oneshot_plummer_250k", "kind": "oneshot", "gen": "plummer", "n": 250007,
         "theta": 0.5, "eps": 1e-3, "n_leaf": 16, "n_group": 64},
        # A small cluster advanced many steps: each is a rebuild and a force call.
        {"name": "sim_cluster_5k", "kind": "sim", "gen": "plummer", "n": 5003, "theta": 0.5,
         "eps": 0.01, "dt": 1.0 / 256, "steps": 16, "n_leaf": 16, "n_group": 64},
        # The size of the merger runs.
        {"name": "sim_plummer_256k", "kind": "sim", "gen": "plummer", "n": 1 << 18, "theta": 0.5,
         "eps": 1e-3, "dt": 1.0 / 64, "steps": 16, "n_leaf": 16, "n_group": 64},
        # The accuracy check: 4096 sampled particles against the direct sum.
        {"name": "direct_sampled_1m", "kind": "direct", "gen": "plummer", "n": 1 << 20,
         "targets": 4096, "eps": 1e-3},
        # The direct sum of every particle, the training labels' reference.
        {"name": "direct_all_64k", "kind": "direct", "gen": "two_plummer", "n": 1 << 16,
         "targets": 0, "eps": 1e-3},
        # The trainer's mini-batch.
        {"name": "train_batch_4096", "kind": "train", "batch": 4096},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forces", "forces", "forces", "learned", "oneshot", "sim", "direct", "train"])
    gens = ["plummer", "two_plummer", "plummer_clumps", "milky_way", "galaxy_mix"]
    if kind in ("forces", "learned"):
        n = _log_int(rng, 300, 1.2e6)
        theta = round(rng.uniform(0.4 if n > 300000 else 0.3, 0.9), 3)
        if kind == "learned":
            n, theta = max(n, 2000), 0.5625
        return {"kind": "forces", "gen": rng.choice(gens), "n": n, "theta": theta,
                "eps": rng.choice([1e-3, 5e-4, 0.01]), "n_leaf": rng.choice([8, 16, 32]),
                "n_group": rng.choice([32, 64, 64, 128]),
                "mac": "learned" if kind == "learned" else "theta"}
    if kind == "oneshot":
        return {"kind": "oneshot", "gen": rng.choice(gens), "n": _log_int(rng, 2000, 600000),
                "theta": round(rng.uniform(0.4, 0.8), 3), "eps": 1e-3,
                "n_leaf": rng.choice([8, 16, 32]), "n_group": 64}
    if kind == "sim":
        return {"kind": "sim", "gen": "plummer", "n": _log_int(rng, 1000, 200000),
                "theta": round(rng.uniform(0.4, 0.8), 3), "eps": 0.01, "dt": 1.0 / 256,
                "steps": rng.randint(3, 16), "n_leaf": 16, "n_group": 64}
    if kind == "direct":
        n = _log_int(rng, 1000, 500000)
        # sampled targets, or (0) every particle of a small set
        return {"kind": "direct", "gen": rng.choice(gens), "n": n,
                "targets": 0 if n < 50000 and rng.random() < 0.5 else min(n, _log_int(rng, 100, 8192)),
                "eps": rng.choice([1e-3, 0.01])}
    return {"kind": "train", "batch": _log_int(rng, 256, 20000)}


def _particles(case, seed):
    n, gen = case["n"], case["gen"]
    if gen == "two_plummer":
        pos, m = W.two_plummer(n, seed, 4.0)
    else:
        pos, m = getattr(W, gen)(n, seed)
    # a mild mass spectrum, the total kept at 1
    f = np.random.default_rng(seed + 1).uniform(0.5, 1.5, n)
    return pos, (f / f.sum()).astype(np.float32)


def _train_inputs(case, seed):
    """Features as the band pairs have them (order one, non-negative) and log10 errors."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    b = case["batch"]
    x = torch.rand((b, 12), generator=g, device="cuda") * 2.0
    y = -4.0 + torch.randn(b, generator=g, device="cuda") - 0.5 * x[:, 0]
    return x, y


def prepare(case, seed):
    s = dict(case)
    if s["kind"] == "train":
        s["x"], s["y"] = _train_inputs(case, seed)
        s["params"] = L.init_params(seed)
        s["net"] = og.Mlp(s["params"])
        s["step"] = 0
        return s
    if s["kind"] == "sim":
        pos, vel, m = W.plummer_with_velocities(case["n"], seed)
        s["sim"] = og.Sim(pos, vel, m, case["n_leaf"], case["n_group"])
        s["sim"].run(case["theta"], case["eps"], case["dt"], 0)  # the first forces
        return s
    pos, m = _particles(case, seed)
    if s["kind"] == "oneshot":
        s["pos"], s["m"] = pos, m
        return s
    s["tree"] = og.Tree(pos, m, case.get("n_leaf", 16), case.get("n_group", 64))
    if s["kind"] == "forces" and case["mac"] == "learned":
        s["net"] = og.Mlp(L.load_params())
        s["tree"].set_mac(s["net"], MAC_LO, MAC_HI, MAC_TAU, 30 * MAC_TAU)
    if s["kind"] == "direct":
        s["idx"] = torch.from_numpy(W.sample_indices(case["n"], case["targets"], seed).astype(np.int32)).cuda() \
            if case["targets"] else None
    return s


def run(s):
    kind = s["kind"]
    if kind == "forces":
        return s["tree"].forces(s["theta"], s["eps"])
    if kind == "oneshot":
        tree = og.Tree(s["pos"], s["m"], s["n_leaf"], s["n_group"], device_build=True)
        return tree.forces(s["theta"], s["eps"])
    if kind == "sim":
        s["sim"].run(s["theta"], s["eps"], s["dt"], s["steps"])
        pos, vel, acc = s["sim"].state()
        e = s["sim"].energy()
        return {"pos": pos, "vel": vel, "acc": acc, "K": float(e["K"]), "W": float(e["W"])}
    if kind == "direct":
        return s["tree"].direct(s["eps"], s["idx"])
    s["step"] += 1
    loss, grad = s["net"].loss_grad(s["x"], s["y"], L.PINBALL_TAU)
    s["net"].adam(s["step"])
    return {"loss": loss, "grad": grad, "params": s["net"].params()}


def _interactions(case):
    """(particle-cell, particle-particle) interactions per particle: a fit to the lists' lengths
    (groups of 64; within a third of the counts from 10^3 to 10^6 particles, theta 0.3 to 0.75)."""
    n, th = case["n"], max(case["theta"], 0.3)
    leaf = max(1.0, case.get("n_leaf", 16) / 16.0)
    pp = min(0.6 * n, 700 * (0.5 / th) ** 2.5 * leaf)
    pc = max(120.0, 960 + 190 * math.log2(n / 16384.0)) * (0.5 / th) ** 2.4 / leaf ** 0.4
    pc = min(pc, 0.12 * n)
    if case.get("mac") == "learned":
        pc, pp = 0.55 * pc, 0.9 * pp
    return pc, pp


def work(case):
    kind = case["kind"]
    if kind == "train":
        b, p = case["batch"], og.N_PARAMS
        # forward, and backward for the weights and the hidden layer
        return {"bytes": 52.0 * b + 28.0 * p, "flops": b * 2.0 * (12 * 64 + 64 * 64 + 64) * 3.0}
    n = case["n"]
    if kind == "direct":
        nt = case["targets"] or n
        return {"bytes": 16.0 * n + 20.0 * nt, "flops": 38.0 * n * nt}
    pc, pp = _interactions(case)
    flops = n * (70.0 * pc + 38.0 * pp)
    cells = n / (4.0 if case["n_leaf"] <= 16 else 7.0)
    nbytes = 16.0 * n + 16.0 * n + 96.0 * cells
    if kind == "oneshot":
        nbytes += 16.0 * n
    if kind == "sim":
        flops *= case["steps"]
        nbytes = case["steps"] * (nbytes + 72.0 * n)
    return {"bytes": nbytes, "flops": flops}


def _direct64(pos, m, eps, idx=None):
    """FP64 direct sum (acc [nt, 3], pot [nt]) over all particles, the target itself left out."""
    x = torch.as_tensor(pos, device="cuda").double()
    m = torch.as_tensor(m, device="cuda").double()
    nt = x.shape[0] if idx is None else idx.shape[0]
    acc = torch.empty((nt, 3), dtype=torch.float64, device="cuda")
    pot = torch.empty(nt, dtype=torch.float64, device="cuda")
    step = max(1, (1 << 26) // x.shape[0])
    own = torch.arange(nt, device="cuda") if idx is None else idx.long()
    xt = x.t().contiguous()
    for a in range(0, nt, step):
        t = own[a:a + step]
        r2 = torch.full((t.shape[0], x.shape[0]), float(eps) ** 2, dtype=torch.float64, device="cuda")
        for k in range(3):
            d = xt[k][None, :] - xt[k][t][:, None]
            r2.addcmul_(d, d)
        ri = r2.rsqrt_()
        ri[torch.arange(t.shape[0], device="cuda"), t] = 0.0
        w = ri * m[None, :]
        pot[a:a + step] = -w.sum(1)
        w.mul_(ri).mul_(ri)
        ws = w.sum(1)
        for k in range(3):
            acc[a:a + step, k] = w @ xt[k] - ws * xt[k][t]
    return acc, pot


def _mlp64(params, x, y, tau):
    """Loss and gradient in FP64 with the network's BF16 rounding points (inputs, weights and
    hidden activations before each product, activation gradients in the weight gradients)."""
    bf = lambda v: v.float().bfloat16().double()
    p = torch.as_tensor(np.asarray(params), device="cuda").double()
    w1, b1 = p[:768].view(64, 12), p[768:832]
    w2, b2 = p[832:4928].view(64, 64), p[4928:4992]
    w3, b3 = p[4992:5056], p[5056]
    xr = bf(x)
    a1 = xr @ bf(w1).t() + b1
    h1 = bf(a1.clamp(min=0))
    a2 = h1 @ bf(w2).t() + b2
    h2 = bf(a2.clamp(min=0))
    out = h2 @ bf(w3) + b3
    r = y.double() - out
    b = x.shape[0]
    loss = torch.where(r > 0, tau * r, (tau - 1.0) * r).sum() / b
    dy = torch.where(r > 0, -tau, 1.0 - tau) / b
    d2 = (a2 > 0) * dy[:, None] * bf(w3)[None, :]
    d2r = bf(d2)
    d1 = (a1 > 0) * (d2r @ bf(w2))
    d1r = bf(d1)
    grad = torch.cat([(d1r.t() @ xr).reshape(-1), d1.sum(0), (d2r.t() @ h1).reshape(-1),
                      d2.sum(0), (dy[:, None] * h2).sum(0), dy.sum().reshape(1)])
    return loss, grad


def exact(case, seed):
    """The sums themselves in FP64: the direct sum over all particles for every kind of force
    (what the opening angle leaves out is part of the error then), the network's loss and gradient
    with its rounding points.  None where that takes too long or has no such value."""
    kind = case["kind"]
    if kind == "train":
        x, y = _train_inputs(case, seed)
        loss, grad = _mlp64(L.init_params(seed), x, y, L.PINBALL_TAU)
        return {"loss": float(loss), "grad": grad.cpu().numpy(), "params": None}
    if kind == "direct":
        pos, m = _particles(case, seed)
        idx = torch.from_numpy(W.sample_indices(case["n"], case["targets"], seed)).cuda() \
            if case["targets"] else None
        return _direct64(pos, m, case["eps"], idx)
    if kind in ("forces", "oneshot") and case["n"] <= 300000:
        pos, m = _particles(case, seed)
        return _direct64(pos, m, case["eps"])
    if kind == "sim" and case["n"] <= 20000:
        pos, vel, m = W.plummer_with_velocities(case["n"], seed)
        x = torch.as_tensor(pos, device="cuda").double()
        v = torch.as_tensor(vel, device="cuda").double()
        a, pot = _direct64(x, m, case["eps"])
        for _ in range(case["steps"]):
            v = v + 0.5 * case["dt"] * a
            x = x + case["dt"] * v
            a, pot = _direct64(x, m, case["eps"])
            v = v + 0.5 * case["dt"] * a
        md = torch.as_tensor(m, device="cuda").double()
        return {"pos": x.cpu().numpy(), "vel": v.cpu().numpy(), "acc": a.cpu().numpy(),
                "K": float((0.5 * md * (v * v).sum(1)).sum()), "W": float((0.5 * md * pot).sum())}
    return None
