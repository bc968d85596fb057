"""Timed cases of the fire library: the work its users have it do, through its public entry points.

Every case names a kind of work (``kind``) and its sizes. ``prepare`` makes what a program has in hand
before the call (a context with its landscapes and reference maps loaded, device buffers, a network with
its weights), ``run`` is one pass, ``work`` the bytes and operations the pass cannot do without and
``exact`` the binary64 values of the network's outputs. Simulation results are integers and correctly
rounded quotients of integers, so they have no other exact value than themselves.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_1701_03549_amd import autotune, fire, ga, mc, nn, scan, synth

#: parameter vectors of the workloads: fires that stay on their hillside (the calibration vector), fires
#: that fill their forest stand (the ignition scan's), fires that spread everywhere, and even odds per edge
BETAS = {"slope": (-3.0, -0.5, 6.0, 1.0, 2.0), "forest": synth.SCAN_BETA,
         "open": (0.0, 0.0, 0.0, 0.5, 0.5), "even": (0.0, 0.0, 0.0, 0.0, 0.0)}
#: about what share of the lattice a fire burns under them (box: uniform over the search box)
SHARE = {"slope": 0.035, "forest": 0.03, "open": 0.85, "even": 0.85, "box": 0.15, "prior": 0.05}
#: the lattices of the uneven batch: side lengths and landscape seeds
UNEVEN = ((128, 128, 101), (256, 256, 102), (512, 512, 103), (1024, 768, 104))


def listed():
    return [
        # one simulation, scored against the reference fire: what a program that looks at a single fire, or
        # evaluates a search one simulation at a time, waits for
        {"name": "one_fire_512", "kind": "replicates", "width": 512, "height": 512, "land": 102, "wind": "uniform",
         "fires": "slope", "n": 1, "entry": "device", "maps": False, "turn_off": False},
        # a small lattice with its burn maps, from host descriptors: the plain small workload
        {"name": "maps_64", "kind": "replicates", "width": 64, "height": 64, "land": 101, "wind": "uniform",
         "fires": "even", "n": 200, "entry": "host", "maps": True, "turn_off": False},
        # the calibration batch: Eq. 1 table on the device, then 1280 scored replicates
        {"name": "calibration_512", "kind": "replicates", "width": 512, "height": 512, "land": 102, "wind": "uniform",
         "fires": "slope", "n": 1280, "entry": "table", "maps": False, "turn_off": False},
        # the same batch with turn-off times per vegetation
        {"name": "turn_off_512", "kind": "replicates", "width": 512, "height": 512, "land": 102, "wind": "uniform",
         "fires": "slope", "n": 1280, "entry": "device", "maps": False, "turn_off": True},
        # fires that cross a lattice of the paper's size study, whose burn bitset does not fit LDS, with maps
        {"name": "crossing_1600", "kind": "replicates", "width": 1600, "height": 1600, "land": 105, "wind": "uniform",
         "fires": "open", "n": 32, "entry": "host", "maps": True, "turn_off": False},
        # a whole GA calibration and its accepted ensemble
        {"name": "ga_512", "kind": "ga", "width": 512, "height": 512, "land": 102, "pop": 64, "reps": 20,
         "generations": 50, "ignition": False},
        # a GA with the ignition point estimated, on a lattice whose sides are no multiple of 32
        {"name": "ga_ignition_300", "kind": "ga", "width": 300, "height": 250, "land": 105, "pop": 32, "reps": 10,
         "generations": 20, "ignition": True},
        # a Monte Carlo fit: one simulation per parameter vector drawn from the search box
        {"name": "monte_carlo_512", "kind": "mc", "width": 512, "height": 512, "land": 102, "n": 8192},
        # lattices of four sizes and a parameter vector per simulation in one call
        {"name": "uneven_2000", "kind": "uneven", "lattices": 4, "each": 500},
        # an ignition-point scan: 256 candidates x 32 replicates and the reduction
        {"name": "scan_1024", "kind": "scan", "width": 1024, "height": 1024, "land": 103, "half": 8, "reps": 32},
        # one training batch of the surrogate with burn maps, forward and backward
        {"name": "surrogate_grad_512", "kind": "gradients", "batch": 512, "maps": True, "side": 256},
        # the candidates of one screened generation through the surrogate
        {"name": "surrogate_score_498", "kind": "score", "batch": 498, "maps": False, "side": 256},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["replicates", "replicates", "replicates", "replicates", "ga", "mc", "uneven", "scan",
                       "gradients", "score"])
    if kind == "replicates":
        if rng.random() < 0.2:  # beyond the LDS: fires across the lattice
            w = rng.randrange(1300, 1900)
            h = rng.randrange(1100, 1500)
            return {"kind": kind, "width": w, "height": h, "land": rng.randrange(1000), "wind": "smooth",
                    "fires": "open", "n": rng.randrange(2, 33), "entry": rng.choice(["host", "device"]),
                    "maps": rng.random() < 0.5, "turn_off": False}
        fires, turn_off = rng.choice(["slope", "forest", "forest", "even"]), rng.random() < 0.25
        top = 400 if fires == "even" and turn_off else 1024
        w, h = _log_int(rng, 40, top), _log_int(rng, 40, top)
        most = max(1, min(1280, 40_000_000 // (w * h))) if fires == "even" else 1280
        return {"kind": kind, "width": w, "height": h, "land": rng.randrange(1000),
                "wind": rng.choice(["uniform", "smooth"]), "fires": fires, "n": _log_int(rng, 1, most),
                "entry": rng.choice(["host", "device", "table"]), "maps": rng.random() < 0.3, "turn_off": turn_off}
    if kind == "ga":
        return {"kind": kind, "width": _log_int(rng, 64, 512), "height": _log_int(rng, 64, 512),
                "land": rng.randrange(1000), "pop": rng.randrange(12, 65), "reps": rng.randrange(8, 21),
                "generations": rng.randrange(4, 40), "ignition": rng.random() < 0.5}
    if kind == "mc":
        return {"kind": kind, "width": _log_int(rng, 64, 512), "height": _log_int(rng, 64, 512),
                "land": rng.randrange(1000), "n": _log_int(rng, 256, 8192)}
    if kind == "uneven":
        return {"kind": kind, "lattices": rng.randrange(2, 5), "each": _log_int(rng, 40, 500)}
    if kind == "scan":
        return {"kind": kind, "width": rng.randrange(300, 1025), "height": rng.randrange(300, 1025),
                "land": rng.randrange(1000), "half": rng.randrange(2, 9), "reps": rng.randrange(8, 33)}
    if kind == "gradients":
        return {"kind": kind, "batch": _log_int(rng, 16, 512), "maps": rng.random() < 0.6,
                "side": rng.choice([128, 256, 512])}
    return {"kind": kind, "batch": _log_int(rng, 1, 1500), "maps": rng.random() < 0.3,
            "side": rng.choice([128, 256, 512])}


# -- inputs ------------------------------------------------------------------

@functools.lru_cache(maxsize=24)
def _landscape(w, h, land, wind="uniform"):
    return synth.make_landscape(w, h, land, wind=wind)


def _context():
    g = fire.FireGPU(0)
    autotune.apply_cache(g)
    return g


def _ignition(ls, fires):
    """Where the fires start: on the driest exposure, or in the forest stand nearest the centre."""
    h, w = ls["veg"].shape
    if fires == "forest" and (ls["veg"] == 1).any():
        return synth.nearest_of_class(ls["veg"], 1, w // 2, h // 2)
    return synth.ignition_site(ls)


def _reference(g, lid, ign, beta, seed):
    """Load the reference map: of 32 replicates the one whose fire is of the middle size."""
    w, h = g.dims[lid]
    res, maps = g.run(np.array([beta]), fire.make_sims(32, lid, -1, ign), seed ^ 0x7A26E7, want_maps=True)
    g.sync()
    k = int(np.argsort(fire.results_to_numpy(res)["burnt"], kind="stable")[16])
    ref = maps[k].cpu().numpy().view(np.uint32)[:h * ((w + 31) // 32)].reshape(h, -1)
    return g.load_target(lid, ref), ref


def _device_sims(sims):
    return torch.from_numpy(sims.view(np.uint8).copy()).cuda()


def _weights(seed):
    """The network's parameters in their flat order (fp32): weights uniform in +-sqrt(6 / (fan in + fan
    out)), small biases."""
    rng = np.random.default_rng(seed)
    out = []
    for shape, fan, used in (((16, 256), (7, 256), 7), ((256, 256), (256, 256), 256), ((256, 256), (256, 256), 256),
                             ((256, 1), (256, 1), 256), ((256, 2048), (256, 2048), 256), ((8, 8, 3, 3), (72, 72), 8),
                             ((8, 8, 3, 3), (72, 72), 8), ((1, 8, 3, 3), (72, 9), 1)):
        lim = math.sqrt(6.0 / sum(fan))
        w = rng.uniform(-lim, lim, size=shape)
        w[used:] = 0.0
        bias = shape[1] if len(shape) == 2 else shape[0]
        out += [w.reshape(-1), rng.uniform(-0.05, 0.05, size=bias)]
    return np.concatenate(out).astype(np.float32)


def _batch(case, seed):
    """Rows as the simulator gives them: parameters from the search prior, an ignition, log(1 + delta) and
    the burnt cells around the ignition on the 128 x 128 grid."""
    rng = np.random.default_rng([seed, 1])
    b, side = case["batch"], case["side"]
    x = np.empty((b, 7), dtype=np.float32)
    x[:, :5] = np.clip(rng.normal(0.0, 5.0, size=(b, 5)), -30.0, 30.0)
    x[:, 5:] = rng.integers(0, side, size=(b, 2))
    y = np.log1p(np.abs(rng.normal(0.5, 0.4, size=b))).astype(np.float32)
    radius = rng.uniform(1.0, 40.0, size=b).astype(np.float32)
    return x, y, radius


def _map_targets(x, radius, side):
    """Burnt discs around the ignitions, uint8 [B][128][128]."""
    c = torch.arange(128, dtype=torch.float32, device=x.device) + 0.5
    cx, cy = (x[:, 5 + k] * (128.0 / side) for k in (0, 1))
    d2 = (c[None, None, :] - cx[:, None, None]) ** 2 + (c[None, :, None] - cy[:, None, None]) ** 2
    return (d2 < (radius * radius)[:, None, None]).to(torch.uint8).contiguous()


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "seed": 0x5EED0001 + 7919 * seed}
    if kind in ("gradients", "score"):
        x, y, radius = (torch.from_numpy(a).cuda() for a in _batch(case, seed))
        s["net"] = nn.Surrogate(max_batch=512, lattice=(case["side"], case["side"]), w_map=1.0, seed=1)
        s["net"].set_params(torch.from_numpy(_weights(seed)))
        s["x"], s["y"] = x, y
        s["map"] = _map_targets(x, radius, case["side"]) if case["maps"] and kind == "gradients" else None
        return s
    g = s["g"] = _context()
    rng = np.random.default_rng([seed, 2])
    if kind == "uneven":
        sims, n = [], case["each"]
        for k, (w, h, land) in enumerate(UNEVEN[:case["lattices"]]):
            ls = _landscape(w, h, land)
            lid = g.load_landscape(ls)
            index = np.arange(n * k, n * (k + 1), dtype=np.uint32)
            sims.append(fire.make_sims(n, lid, -1, synth.ignition_site(ls), param_index=index, sim_index=index))
        s["sims"] = np.concatenate(sims)
        s["betas"] = rng.uniform(-30.0, 30.0, size=(len(s["sims"]), 5))
        return s
    w, h = case["width"], case["height"]
    wind = case.get("wind", "smooth" if kind == "scan" else "uniform")
    fires = case.get("fires", "forest" if kind == "scan" else "slope")
    ls = _landscape(w, h, case["land"], wind)
    lid = s["lid"] = g.load_landscape(ls)
    ign = s["ign"] = _ignition(ls, fires)
    beta = s["beta"] = BETAS[fires]
    s["tid"], ref = _reference(g, lid, ign, beta, s["seed"])
    if kind == "ga":
        if case["ignition"]:
            s["pop0"] = ga.initial_population_ignition(ref, w, h, case["pop"], seed=seed)
        else:
            s["pop0"] = np.clip(rng.normal(0.0, 5.0, size=(case["pop"], 5)), -30.0, 30.0)
    elif kind == "mc":
        s["draws"] = int(rng.integers(1 << 30))
    elif kind == "scan":
        s["cands"] = scan.candidate_grid(ign, w, h, spacing=4, half=case["half"])
    else:
        n = case["n"]
        if case["turn_off"]:
            steps = np.full(256, 3, dtype=np.uint8)
            steps[1] = 2
            g.set_burn_steps(lid, steps)
        s["sims"] = fire.make_sims(n, lid, s["tid"], ign)
        s["betas"] = np.array([beta], dtype=np.float64)
        if case["entry"] != "host":
            s["d_sims"] = _device_sims(s["sims"])
            s["d_beta"] = torch.from_numpy(s["betas"]).cuda()
            s["out"] = torch.empty((n, 24), dtype=torch.uint8, device="cuda")
            s["words"] = h * ((w + 31) // 32)
            s["out_maps"] = torch.empty((n, s["words"]), dtype=torch.int32, device="cuda") if case["maps"] else None
            if case["entry"] == "table":
                s["table"] = torch.empty((h, w, 8), dtype=torch.int32, device="cuda")
    return s


# -- one pass ----------------------------------------------------------------

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "gradients":
        loss, grads = s["net"].gradients(s["x"], s["y"], s["map"])
        return {"loss": loss, "grads": grads}
    if kind == "score":
        if case["maps"]:  # forward() takes at most the handle's batch
            parts = [s["net"].forward(s["x"][i:i + 512], want_map=True) for i in range(0, case["batch"], 512)]
            return {"t": [p[0] for p in parts], "map": [p[1] for p in parts]}
        return {"t": s["net"].predict(s["x"])}
    g = s["g"]
    if kind == "uneven":
        return g.run(s["betas"], s["sims"], s["seed"])[0]
    if kind == "ga":
        common = dict(R=case["reps"], generations=case["generations"], sim_seed=s["seed"], ga_seed=s["seed"] + 1)
        if case["ignition"]:
            pop, fit = ga.run_ignition(g, s["lid"], s["tid"], s["pop0"], **common)
        else:
            pop, fit = ga.run_batched(g, s["lid"], s["tid"], s["ign"], s["pop0"], **common)
        best = g.ensemble(pop.reshape(-1, pop.shape[2]), fit.reshape(-1, case["reps"]), 1.5 if case["ignition"] else 0.3)
        return {"pop": pop, "fit": fit, "ensemble": best}
    if kind == "mc":
        out = mc.run_mc(g, s["lid"], s["tid"], s["ign"], case["n"], s["draws"], s["seed"])
        return {k: out[k] for k in ("deltas", "trials", "best_index", "n_accepted", "accepted_mean", "accepted_sd")}
    if kind == "scan":
        return scan.run_scan(g, s["lid"], s["tid"], s["beta"], s["cands"], R=case["reps"], seed=s["seed"])
    if case["entry"] == "host":
        res, maps = g.run(s["betas"], s["sims"], s["seed"], want_maps=case["maps"])
        return [res, maps] if case["maps"] else [res]
    table = None
    if case["entry"] == "table":
        table = g.thresholds_dev(s["lid"], s["d_beta"], out=s["table"])
    g.run_dev(s["d_beta"], s["d_sims"], case["n"], s["seed"], s["out"], maps=s["out_maps"],
              map_words=s["words"] if case["maps"] else 0, override=table)
    return [s["out"], s["out_maps"]] if case["maps"] else [s["out"]]


# -- what a pass cannot do without --------------------------------------------

def _fires(cells, n, share):
    """Bytes and operations of n simulations on one lattice: its layers read once (17 B a cell), a
    descriptor and a result each; two generator calls (ten rounds of two 32-bit products, their upper halves
    and six other operations) and about four tried edges (a comparison, Eq. 1's five products and sums) a
    burnt cell."""
    return 17 * cells + 52 * n, n * cells * share * (2 * 100 + 4 * 12)


def work(case):
    kind = case["kind"]
    if kind in ("gradients", "score"):
        b, passes = case["batch"], 3 if kind == "gradients" else 1
        dense = 16 * 256 + 2 * 256 * 256 + 256
        macs, params = dense, dense + 3 * 256 + 1
        byts = b * 7 * 4 + b * 4
        if case["maps"]:
            macs += 256 * 2048 + 72 * (8 * 32 * 32 + 8 * 64 * 64 + 128 * 128)
            params += 257 * 2048 + 2 * 584 + 73
            byts += b * 128 * 128 * (1 if kind == "gradients" else 4)
        if kind == "gradients":
            byts += 4 * b + 4 * 663770  # targets, every parameter's gradient
        return {"bytes": byts + 4 * params, "flops": 2 * passes * b * macs}
    if kind == "uneven":
        parts = [_fires(w * h, case["each"], SHARE["box"]) for w, h, _ in UNEVEN[:case["lattices"]]]
        return {"bytes": sum(p[0] for p in parts) + 40 * case["each"] * len(parts), "flops": sum(p[1] for p in parts)}
    cells = case["width"] * case["height"]
    if kind == "ga":
        n = case["pop"] * case["reps"] * case["generations"]
        byts, ops = _fires(cells, n, SHARE["prior"])
        return {"bytes": byts + 8 * n + 8 * case["pop"] * case["generations"] * 7, "flops": ops}
    if kind == "mc":
        byts, ops = _fires(cells, case["n"], SHARE["box"])
        return {"bytes": byts + 40 * case["n"], "flops": ops}
    if kind == "scan":
        byts, ops = _fires(cells, (2 * case["half"]) ** 2 * case["reps"], SHARE["forest"])
        return {"bytes": byts, "flops": ops}
    byts, ops = _fires(cells, case["n"], SHARE[case["fires"]])
    if case["turn_off"]:
        ops *= 2.5
    if case["maps"]:
        byts += case["n"] * case["height"] * ((case["width"] + 31) // 32) * 4
    if case["entry"] == "table":
        byts += 32 * cells
    return {"bytes": byts, "flops": ops}


# -- binary64 values ------------------------------------------------------------

def _network(p, x, side, want_map):
    """The surrogate in binary64: (t, map logits or None) of rows x under the parameters p (one tensor
    each, in their flat order)."""
    w1, c1, w2, c2, w3, c3, wf, cf, wd, cd, k1, b1, k2, b2, k3, b3 = p
    xs = torch.cat([x[:, :5] / 30.0, 2.0 * x[:, 5:] / side - 1.0, torch.zeros(len(x), 9, dtype=x.dtype)], dim=1)
    h = torch.relu(xs @ w1 + c1)
    h = torch.relu(h @ w2 + c2)
    h = torch.relu(h @ w3 + c3)
    t = (h @ wf + cf)[:, 0]
    if not want_map:
        return t, None
    up = lambda v: v.repeat_interleave(2, dim=2).repeat_interleave(2, dim=3)  # noqa: E731
    conv = torch.nn.functional.conv2d
    d = torch.relu(h @ wd + cd).reshape(-1, 8, 16, 16)
    d = torch.relu(conv(up(d), k1, b1, padding=1))
    d = torch.relu(conv(up(d), k2, b2, padding=1))
    return t, conv(up(d), k3, b3, padding=1)[:, 0]


def _parameters(seed):
    flat, out, at = torch.from_numpy(_weights(seed)).double(), [], 0
    for shape in ((16, 256), (256,), (256, 256), (256,), (256, 256), (256,), (256, 1), (1,), (256, 2048), (2048,),
                  (8, 8, 3, 3), (8,), (8, 8, 3, 3), (8,), (1, 8, 3, 3), (1,)):
        n = math.prod(shape)
        out.append(flat[at:at + n].reshape(shape).clone().requires_grad_(True))
        at += n
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("gradients", "score"):
        return None
    x, y, radius = (torch.from_numpy(a) for a in _batch(case, seed))
    p, side, b = _parameters(seed), case["side"], case["batch"]
    if kind == "score":
        with torch.no_grad():
            parts = [_network(p, v.double(), side, case["maps"]) for v in x.split(512)]
        if case["maps"]:
            return {"t": [q[0] for q in parts], "map": [torch.sigmoid(q[1]) for q in parts]}
        return {"t": torch.cat([q[0] for q in parts])}
    target = _map_targets(x, radius, side).double() if case["maps"] else None
    loss = torch.zeros(2, dtype=torch.float64)
    for i in range(0, b, 32):
        t, z = _network(p, x[i:i + 32].double(), side, case["maps"])
        fit = ((t - y[i:i + 32].double()) ** 2).sum() / b
        total = fit
        if z is not None:
            part = torch.nn.functional.binary_cross_entropy_with_logits(z, target[i:i + 32], reduction="sum") / (b * 128 * 128)
            total = total + part
            loss[1] += part.detach()
        loss[0] += fit.detach()
        total.backward()
    return {"loss": loss, "grads": torch.cat([(v.grad if v.grad is not None else torch.zeros_like(v)).reshape(-1) for v in p])}
