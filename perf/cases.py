"""Workloads that time the library through its public entry points.

A case is a dict of plain values.  `prepare` builds what a program has in hand
before the call (problem, handle, device workspace, input tensors), `run` makes
one pass and returns everything the call gives back, `work` counts what the
pass cannot do without, and `exact` computes the same outputs in 64 bits with
plain torch and numpy where they have such a value.

Kinds of case:
  run       one protocol run (ppp_run and ppp_get_result): parallel, sequential or
            with the unrestrained ensemble; 1-D model or bead-spring chain
  oneshot   the same through the one-call convenience ppp.run
  chunked   begin, advances, finalize, result: how a long run is driven
  forces    ppp_eval_forces on a batch of configurations
  batch     an uneven batch of chains in one captured graph
  adaptive  exploration, surrogate training, placement and production run
"""
import math

import numpy as np
import torch

import paper_1105_4840_amd as ppp

# What a chain of the workloads is made of: harmonic bonds, cosine angles,
# Lennard-Jones cut at 2.5 sigma beyond second neighbours, BAOAB at dt = 0.005.
FORCE_FIELD = {"k_bond": 100.0, "r0": 1.0, "k_angle": 5.0, "lj_eps": 1.0, "lj_sigma": 1.0, "lj_rc": 2.5,
               "rc_mode": 0, "mass": 1.0, "gamma": 1.0}


# most windows a placement may ask for
MAX_PLACED = 128


def listed():
    return [
        # the smallest call: energies and forces of a few hundred short-chain
        # configurations; latency and launches are all there is
        {"name": "forces_chain10", "kind": "forces", "beads": 10, "configs": 256, "precision": "fp32"},
        # a small run of the turn-on study: a particle in a harmonic well, few
        # windows, the unrestrained ensemble beside them, fp32, no work histogram
        {"name": "harmonic_turn_on", "kind": "run", "model": "harmonic", "windows": 8, "replicas": 256, "steps": 2000,
         "lo": -1.0, "hi": 0.4, "k": 2.0, "precision": "fp32", "integrator": 0, "bins": 4096, "half_bins": 0,
         "free": True},
        # the 1-D workload at its full size (parity, smoke and quadrature runs)
        {"name": "double_well", "kind": "run", "model": "double_well", "windows": 21, "replicas": 256, "steps": 20000,
         "lo": -1.5, "hi": 1.5, "k": 50.0, "precision": "fp64", "integrator": 0, "bins": 4096, "half_bins": 15000,
         "free": False},
        # the 1-D model with enough replicas to fill the chip (variance pins use
        # 4096 replicas a window), Euler-Maruyama
        {"name": "double_well_wide", "kind": "run", "model": "double_well", "windows": 21, "replicas": 4096,
         "steps": 2000, "lo": -1.5, "hi": 1.5, "k": 50.0, "precision": "fp64", "integrator": 1, "bins": 4096,
         "half_bins": 15000, "free": False},
        # a look at a new system: the 10-bead chain with few replicas and steps,
        # through the one-call entry point
        {"name": "chain10_short", "kind": "oneshot", "model": "chain", "beads": 10, "windows": 21, "replicas": 64,
         "steps": 1000, "lo": 1.5, "hi": 8.5, "k": 20.0, "pull": False, "precision": "fp32", "bins": 4096,
         "half_bins": 15000, "free": False},
        # the 10-bead workload at its full size
        {"name": "chain10", "kind": "run", "model": "chain", "beads": 10, "windows": 21, "replicas": 1024,
         "steps": 40000, "lo": 1.5, "hi": 8.5, "k": 20.0, "pull": False, "precision": "fp32", "bins": 4096,
         "half_bins": 15000, "free": False},
        # the 32-bead workload's grid of windows and replicas, a slice of its steps
        {"name": "chain32", "kind": "run", "model": "chain", "beads": 32, "windows": 21, "replicas": 4096,
         "steps": 1500, "lo": 9.0, "hi": 17.0, "k": 20.0, "pull": True, "precision": "fp32", "bins": 4096,
         "half_bins": 45000, "free": False},
        # the 256-bead workload's grid, driven in advances as its long run is
        {"name": "chain256", "kind": "chunked", "model": "chain", "beads": 256, "windows": 41, "replicas": 4096,
         "steps": 100, "chunks": 2, "lo": 96.0, "hi": 106.0, "k": 20.0, "pull": True, "precision": "fp32",
         "bins": 8192, "half_bins": 45000, "free": False},
        # work distributions at the resolution the paper prints (x bins of 0.001
        # over [0, 50], work bins of 0.01 over +-450) in fp64, with the
        # unrestrained ensemble: a ragged 70 replicas a window
        {"name": "chain10_fine_grid", "kind": "run", "model": "chain", "beads": 10, "windows": 5, "replicas": 70,
         "steps": 600, "lo": 3.2, "hi": 6.0, "k": 20.0, "pull": False, "precision": "fp64", "bins": 50000,
         "half_bins": 45000, "free": True},
        # the sequential protocol: the same replicas taken through the windows in turn
        {"name": "chain10_sequential", "kind": "run", "model": "chain", "beads": 10, "windows": 21, "replicas": 256,
         "steps": 500, "lo": 1.5, "hi": 8.5, "k": 20.0, "pull": False, "precision": "fp32", "bins": 4096,
         "half_bins": 15000, "free": False, "sequential": True},
        # uneven batch: chain lengths, windows, replicas and steps all differ
        {"name": "batch", "kind": "batch", "chains": 12, "beads_lo": 8, "beads_hi": 128, "windows_lo": 11,
         "windows_hi": 41, "replicas_max": 512, "steps_lo": 400, "steps_hi": 2000, "half_bins": 15000, "mix": 3},
        # learned placement on the double well: exploration rounds, training, production
        {"name": "adaptive_double_well", "kind": "adaptive", "budget_steps": 4000, "replicas": 256, "windows": 21,
         "k": 50.0, "initial_windows": 11, "rounds": 4, "train_iters": 600},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forces", "1d", "1d", "1d", "chain", "chain", "chain", "chain", "batch", "adaptive"])
    if kind == "forces":
        return {"kind": "forces", "beads": _log(rng, 2, 256), "configs": _log(rng, 16, 4096),
                "precision": rng.choice(["fp32", "fp64"])}
    if kind == "1d":
        model = rng.choice(["double_well", "harmonic"])
        c = {"kind": rng.choice(["run", "run", "oneshot"]), "model": model, "windows": rng.randint(3, 41),
             "replicas": _log(rng, 16, 4096), "steps": _log(rng, 400, 20000), "lo": -1.5 if model == "double_well" else -1.0,
             "hi": rng.uniform(0.4, 1.5), "k": rng.choice([2.0, 20.0, 50.0]) if model == "harmonic" else rng.choice([20.0, 50.0, 100.0]),
             "precision": rng.choice(["fp32", "fp64", "fp64"]), "integrator": rng.choice([0, 0, 1]),
             "bins": rng.choice([500, 1024, 4096, 4096, 20000]), "half_bins": rng.choice([0, 2000, 15000, 15000]),
             "free": rng.random() < 0.3}
        most = 21 * 4096 * 2000 * 2
        c["steps"] = max(100, min(c["steps"], most // (c["windows"] * c["replicas"])))
        return c
    if kind == "chain":
        n = _log(rng, 5, 256)
        mid, w = 0.395 * (n - 1), min(0.1 * (n - 1) + 1.0, 5.0)
        c = {"kind": rng.choice(["run", "run", "oneshot", "chunked"]), "model": "chain", "beads": n,
             "windows": rng.randint(3, 41), "replicas": _log(rng, 32, 4096), "steps": _log(rng, 100, 20000),
             "lo": max(0.8, mid - w * rng.uniform(0.5, 1.0)), "hi": mid + w * rng.uniform(0.5, 1.0), "k": 20.0,
             "pull": True, "precision": "fp32" if rng.random() < 0.85 else "fp64", "bins": rng.choice([1024, 4096, 4096, 8192]),
             "half_bins": rng.choice([0, 6000, 15000, 45000]), "free": rng.random() < 0.2}
        most = 2.5e12 * (0.15 if c["precision"] == "fp64" else 1.0)
        c["steps"] = int(max(40, min(c["steps"], most / (_chain_flops(n) * c["windows"] * c["replicas"]))))
        c["replicas"] = int(max(8, min(c["replicas"], most / (_chain_flops(n) * c["windows"] * c["steps"]))))
        if c["precision"] == "fp64":
            c["steps"] = min(c["steps"], 400)      # chaotic beyond: two correct runs part
        if c["kind"] == "chunked":
            c["chunks"] = rng.randint(2, 5)
        elif not c["free"] and rng.random() < 0.25:
            c["sequential"] = True
            c["steps"] = max(40, min(c["steps"], 20000 // c["windows"]))
            c["pull"] = False
        return c
    if kind == "batch":
        return {"kind": "batch", "chains": rng.randint(2, 12), "beads_lo": rng.randint(5, 16), "beads_hi": rng.randint(24, 128),
                "windows_lo": 5, "windows_hi": rng.randint(11, 31), "replicas_max": rng.choice([64, 128, 256]),
                "steps_lo": 200, "steps_hi": rng.randint(400, 1500), "half_bins": rng.choice([0, 6000, 15000]),
                "mix": rng.randint(0, 10 ** 6)}
    return {"kind": "adaptive", "budget_steps": _log(rng, 2000, 8000), "replicas": rng.choice([64, 128, 256]),
            "windows": rng.randint(11, 21), "k": rng.choice([50.0, 100.0]), "initial_windows": rng.randint(9, 13),
            "rounds": rng.randint(2, 4), "train_iters": _log(rng, 100, 600)}


# ----------------------------------------------------------------------------- problems

def _linspace(lo, hi, n):
    return [float(x) for x in np.linspace(lo, hi, n)]


def _problem(case, seed):
    """The problem dict of one run case; the seed moves the noise and, a little, the windows."""
    jit = np.random.default_rng(seed).uniform(-0.01, 0.01, 2)
    steps = case["steps"]
    p = {"lambda": _linspace(case["lo"] + jit[0], case["hi"] + jit[1], case["windows"]), "k": case["k"], "kT": 1.0,
         "n_steps": steps, "n_equil": steps // 10, "sample_every": 10, "n_replicas": case["replicas"], "seed": int(seed),
         "init_coords": None, "n_blocks": 32, "w_bin": 0.01, "w_half_bins": case["half_bins"],
         "precision": case["precision"], "xi_bound": 1.0e4, "free_ensemble": bool(case.get("free", False)),
         "sequential": bool(case.get("sequential", False))}
    if case["model"] == "chain":
        n = case["beads"]
        p.update(FORCE_FIELD, model="chain", n_beads=n, dt=0.005)
        if case["pull"]:
            p["n_equil"] = p["n_pull"] = steps // 2
        if n > 64:
            p["w_bin"] = 0.05
        # the fine grid is the printed one; the others span the chain's reach
        lo, hi = (0.0, 50.0) if case["bins"] == 50000 else (0.0, max(n + 1.0, case["hi"] + 3.0))
    else:
        p.update(model="1d", pot_kind=0 if case["model"] == "double_well" else 1, pot_a=5.0, pot_b=1.0,
                 pot_kappa=4.0 if case["model"] == "harmonic" else 0.0, mobility=1.0,
                 integrator_1d=case["integrator"], dt=1e-3)
        lo, hi = -2.5, 2.5
    p.update(xi_min=lo, xi_bin=(hi - lo) / case["bins"], xi_nbins=case["bins"])
    return p


def _batch_problems(case, seed):
    """The batch's shapes come from the case; the seed moves the noise."""
    r = np.random.default_rng(case["mix"])
    out = []
    for i in range(case["chains"]):
        n = int(r.integers(case["beads_lo"], case["beads_hi"] + 1))
        s = int(r.integers(case["windows_lo"], case["windows_hi"] + 1))
        reps = int(r.choice([x for x in (32, 64, 128, 256, 512) if x <= case["replicas_max"]]))
        steps = int(round(math.exp(r.uniform(math.log(case["steps_lo"]), math.log(case["steps_hi"])))))
        mid, w = 0.395 * (n - 1), min(0.1 * (n - 1) + 1.0, 5.0)
        out.append(_problem({"model": "chain", "beads": n, "windows": s, "replicas": reps, "steps": steps,
                             "lo": max(0.8, mid - w), "hi": mid + w, "k": 20.0, "pull": True, "precision": "fp32",
                             "bins": 4096, "half_bins": case["half_bins"]}, 1000 * int(seed) + i))
    return out


def _adaptive_problem(case, seed):
    base = _problem({"model": "double_well", "windows": case["windows"], "replicas": case["replicas"], "steps": 4000,
                     "lo": -1.5, "hi": 1.5, "k": case["k"], "precision": "fp64", "integrator": 0, "bins": 4096,
                     "half_bins": 0}, seed)
    base["n_blocks"] = 16
    return base, {"budget_replica_steps": case["windows"] * case["replicas"] * case["budget_steps"],
                  "initial_windows": case["initial_windows"], "max_rounds": case["rounds"], "max_windows": MAX_PLACED,
                  "target_dl_over_sigma": 1.0, "train_iters": case["train_iters"], "lr": 3e-3, "init_seed": 3,
                  "explore_replicas": 32, "explore_steps": 500, "min_production_steps": 200}


def _helix(n, r0=1.0):
    """The chain's shared start state: unit bonds, 100 degrees of turn and 0.395 of rise a bead."""
    th, rise = 100.0 * math.pi / 180.0, 0.395 * r0
    rho = math.sqrt((r0 * r0 - rise * rise) / (2.0 * (1.0 - math.cos(th))))
    j = np.arange(n)
    return np.stack([rho * (np.cos(j * th) - 1.0), rho * np.sin(j * th), j * rise], axis=1)


def _configs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    n = case["beads"]
    x = torch.from_numpy(_helix(n)).cuda()[None] + 0.05 * torch.randn(case["configs"], n, 3, generator=g, device="cuda",
                                                                       dtype=torch.float64)
    x[:, 0] = 0.0
    return x.reshape(case["configs"], 3 * n).contiguous()


def _forces_problem(case):
    n = case["beads"]
    return _problem({"model": "chain", "beads": n, "windows": 2, "replicas": 1, "steps": 10, "lo": 0.3 * n, "hi": 0.5 * n,
                     "k": 20.0, "pull": False, "precision": case["precision"], "bins": 64, "half_bins": 0}, 0)


class _Handle:
    """A library handle that goes with the state it belongs to."""

    def __init__(self, h):
        self.h = h

    def __del__(self):
        ppp.ppp_destroy(self.h)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "kind": kind}
    if kind == "adaptive":
        s["base"], s["adaptive"] = _adaptive_problem(case, seed)
        return s
    if kind == "batch":
        s["probs"] = _batch_problems(case, seed)
        s["handle"] = _Handle(ppp.ppp_batch_create(s["probs"]))
    else:
        s["prob"] = _forces_problem(case) if kind == "forces" else _problem(case, seed)
        if kind == "oneshot":
            return s
        s["handle"] = _Handle(ppp.ppp_create(s["prob"]))
    s["ws"] = ppp.workspace(s["handle"].h)
    if kind == "forces":
        s["coords"], s["lam"] = _configs(case, seed), 0.4 * case["beads"]
    return s


# ----------------------------------------------------------------------------- one pass

def _outputs(res):
    out = {}
    for key, v in res.items():
        if key == "turn_on":
            out[key] = np.array(list(v.values()))
        elif isinstance(v, np.ndarray):
            out[key] = v.view(np.int64) if v.dtype == np.uint64 else v
        else:
            out[key] = int(v)
    return out


def _padded(v, n):
    if not isinstance(v, np.ndarray) or v.shape[0] not in (n, n - 1):
        return v
    out = np.full((MAX_PLACED,) + v.shape[1:], np.nan if v.dtype.kind == "f" else -1, dtype=v.dtype)
    out[:v.shape[0]] = v
    return out


def run(state):
    kind = state["kind"]
    if kind == "adaptive":
        res, lam, used = ppp.ppp_adaptive_run(state["base"], state["adaptive"])
        # how many windows are placed is part of the answer: records of one fixed size
        out = {key: _padded(v, lam.size) for key, v in _outputs(res).items()}
        return dict(out, windows=_padded(lam, lam.size), used=used)
    if kind == "oneshot":
        return _outputs(ppp.run(state["prob"])[0])
    h, ws = state["handle"].h, state["ws"]
    if kind == "forces":
        f, e = ppp.ppp_eval_forces(h, ws, state["coords"], state["lam"])
        return {"forces": f, "energy": e}
    if kind == "batch":
        ppp.ppp_run(h, ws)
        each = [_outputs(ppp.ppp_batch_get_result(h, p, i)) for i, p in enumerate(state["probs"])]
        return {key: np.concatenate([np.ravel(r[key]) for r in each if key in r]) for key in each[0]}
    if kind == "chunked":
        steps, chunks = state["case"]["steps"], state["case"]["chunks"]
        ppp.ppp_begin(h, ws)
        for _ in range(chunks):
            ppp.ppp_advance(h, -(-steps // chunks))
        ppp.ppp_finalize(h)
    else:
        ppp.ppp_run(h, ws)
    return _outputs(ppp.ppp_get_result(h, state["prob"]))


# ----------------------------------------------------------------------------- what a pass cannot do without

def _chain_flops(n):
    """Per replica-step: 24 per Lennard-Jones pair beyond second neighbours, 21 per bond,
    45 per angle, 11 per mobile degree of freedom, 15 for the restraint."""
    return 24 * ((n - 3) * (n - 2) // 2 if n > 3 else 0) + 21 * (n - 1) + 45 * max(0, n - 2) + 33 * (n - 1) + 15


def _run_work(p):
    s, r = len(p["lambda"]), p["n_replicas"]
    sw = s + (1 if p["free_ensemble"] else 0)
    per = _chain_flops(p["n_beads"]) if p["model"] == "chain" else 12
    out = 8 * s * (40 + p["xi_nbins"] + 2 * (2 * p["w_half_bins"] + 1 if p["w_half_bins"] else 0))
    return {"bytes": out + 8 * sw + 24 * p.get("n_beads", 1), "flops": float(per) * sw * r * p["n_steps"]}


def work(case):
    kind = case["kind"]
    if kind == "forces":
        n, c = case["beads"], case["configs"]
        return {"bytes": c * (6 * n + 5) * 8, "flops": float(c) * _chain_flops(n)}
    if kind == "batch":
        each = [_run_work(p) for p in _batch_problems(case, 0)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    if kind == "adaptive":
        base, ad = _adaptive_problem(case, 0)
        w = _run_work(base)
        # the budget of replica-steps, and per training step 36 points of a 64x64 layer
        # (two paths forward, about three times that back)
        return {"bytes": w["bytes"], "flops": 12.0 * ad["budget_replica_steps"] +
                case["train_iters"] * case["rounds"] * 36 * 4.0 * 16384}
    return _run_work(_problem(case, 0))


# ----------------------------------------------------------------------------- the same in 64 bits

M32 = 0xFFFFFFFF


def _philox(seed, c0, c1, c2):
    """Philox4x32-10 words of counters (c0, c1, c2, 0) as int64 tensors."""
    k0, k1 = seed & M32, (seed >> 32) & M32
    c0, c1, c2 = torch.broadcast_tensors(c0, c1, c2)
    c3 = torch.zeros_like(c0)
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & M32) ^ c1 ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ c3 ^ k1, p0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def _box_muller(u, v):
    r = torch.sqrt(-2.0 * torch.log(u))
    return r * torch.cos(2.0 * math.pi * v), r * torch.sin(2.0 * math.pi * v)


def _noise_1d(p, gid, b0, nb):
    """Normals of blocks b0 .. b0+nb-1 of every replica: [4 nb, replicas]."""
    blk = torch.arange(b0, b0 + nb, device=gid.device)[:, None]
    w = _philox(p["seed"], gid[None, :], blk, torch.zeros_like(blk))
    if p["precision"] == "fp64":
        u = [(x.double() + 0.5) * 2.0 ** -32 for x in w]
    else:
        u = [((x >> 9).double() + 0.5) * 2.0 ** -23 for x in w]
    z = torch.stack([*_box_muller(u[0], u[1]), *_box_muller(u[2], u[3])], dim=1)
    return z.reshape(4 * nb, -1)


def _centre(p, lam, start, n):
    np_ = p.get("n_pull", 0)
    return lam if np_ <= 0 or n >= np_ else start + (lam - start) * (n / np_)


def _sampled(p, n):
    return n > p["n_equil"] and (n - p["n_equil"]) % p["sample_every"] == 0


def _samples_1d(p, dev):
    """Sampled xi [windows (+ the unrestrained), replicas, samples]."""
    lam = list(p["lambda"])
    s, r = len(lam), p["n_replicas"]
    sw = s + int(p["free_ensemble"])
    gid = torch.arange(sw * r, device=dev)
    cen = torch.tensor(lam + [lam[0]] * (sw - s), dtype=torch.float64, device=dev).repeat_interleave(r)
    k = torch.tensor([p["k"]] * s + [0.0] * (sw - s), dtype=torch.float64, device=dev).repeat_interleave(r)
    x = torch.full((sw * r,), lam[0], dtype=torch.float64, device=dev)
    lm = p["integrator_1d"] == 0
    mu_dt = p["mobility"] * p["dt"]
    amp = math.sqrt((0.5 if lm else 2.0) * p["mobility"] * p["kT"] * p["dt"])
    nb = max(1, min(256, (1 << 22) // (sw * r)))
    out, prev, z, at = [], None, None, -1
    for n in range(p["n_steps"] + 1):
        if n >> 2 >= at + nb or z is None:
            at = n >> 2
            z = _noise_1d(p, gid, at, nb)
        e = z[n - 4 * at].clone()
        if n:
            f = -4.0 * p["pot_a"] * x * (x * x - p["pot_b"]) if p["pot_kind"] == 0 else -p["pot_kappa"] * x
            x = x + mu_dt * (f - k * (x - cen)) + amp * (prev + e if lm else e)
            if _sampled(p, n):
                out.append(x)
        prev = e
    return torch.stack(out, dim=1).reshape(sw, r, -1) if out else x.new_zeros(sw, r, 0)


def _chain_forces(p, x, centre, k):
    """Forces and energy parts (bond, angle, Lennard-Jones, restraint) of x [n, N, 3]."""
    n_b = x.shape[1]
    f = torch.zeros_like(x)
    b = x[:, 1:] - x[:, :-1]
    ln = b.norm(dim=2, keepdim=True)
    u = b / ln
    fb = p["k_bond"] * (ln - p["r0"]) * u
    f[:, :-1] += fb
    f[:, 1:] -= fb
    e_bond = (0.5 * p["k_bond"] * (ln - p["r0"]) ** 2).sum(dim=(1, 2))
    e_ang = torch.zeros_like(e_bond)
    if n_b > 2:
        u0, u1 = u[:, :-1], u[:, 1:]
        c = (u0 * u1).sum(dim=2, keepdim=True)
        ga = p["k_angle"] * (c * u0 - u1) / ln[:, :-1]       # dU/d(first bond)
        gb = p["k_angle"] * (c * u1 - u0) / ln[:, 1:]
        f[:, :-2] += ga
        f[:, 1:-1] += gb - ga
        f[:, 2:] -= gb
        e_ang = (p["k_angle"] * (1.0 - c)).sum(dim=(1, 2))
    e_lj = torch.zeros_like(e_bond)
    if n_b > 3:
        i, j = torch.triu_indices(n_b, n_b, offset=3, device=x.device)
        d = x[:, i] - x[:, j]
        r2 = (d * d).sum(dim=2)
        rc = p["lj_rc"] * p["lj_sigma"]
        ok = r2 < rc * rc
        s6 = (p["lj_sigma"] ** 2 / r2) ** 3
        q = (p["lj_sigma"] / rc) ** 6
        e_lj = torch.where(ok, 4.0 * p["lj_eps"] * (s6 * s6 - s6 - (q * q - q)), 0.0).sum(dim=1)
        g = torch.where(ok, 24.0 * p["lj_eps"] * (2.0 * s6 * s6 - s6) / r2, 0.0)[..., None] * d
        f.index_add_(1, i, g)
        f.index_add_(1, j, -g)
    e = x[:, -1] - x[:, 0]
    xi = e.norm(dim=1)
    f[:, -1] -= (k * (xi - centre) / xi)[:, None] * e
    return f, e_bond, e_ang, e_lj, 0.5 * k * (xi - centre) ** 2


def _noise_chain(p, gid, n):
    n_b = p["n_beads"]
    m = torch.arange((n_b + 1) // 2, device=gid.device)[None, :]
    r = _philox(p["seed"], gid[:, None], torch.full_like(m, n), m)
    a = [w >> 11 for w in r] + [((r[0] & 0x7FF) << 10) | (r[1] & 0x3FF), ((r[2] & 0x7FF) << 10) | (r[3] & 0x3FF)]
    u = [(v.double() + 0.5) * 2.0 ** -21 for v in a]
    z = [v for q in range(3) for v in _box_muller(u[2 * q], u[2 * q + 1])]
    return torch.stack(z, dim=2).reshape(gid.numel(), -1, 3)[:, :n_b]


def _samples_chain(p, dev):
    lam = list(p["lambda"])
    s, r = len(lam), p["n_replicas"]
    sw = s + int(p["free_ensemble"])
    gid = torch.arange(sw * r, device=dev)
    lam_w = torch.tensor(lam + [lam[0]] * (sw - s), dtype=torch.float64, device=dev).repeat_interleave(r)
    k = torch.tensor([p["k"]] * s + [0.0] * (sw - s), dtype=torch.float64, device=dev).repeat_interleave(r)
    x = torch.from_numpy(_helix(p["n_beads"], p["r0"])).to(dev).repeat(sw * r, 1, 1)
    start = float((x[0, -1] - x[0, 0]).norm())
    sd = math.sqrt(p["kT"] / p["mass"])
    c1 = math.exp(-p["gamma"] * p["dt"])
    c2 = math.sqrt(1.0 - c1 * c1) * sd
    v = sd * _noise_chain(p, gid, 0)
    v[:, 0] = 0.0
    h, hm = 0.5 * p["dt"], 0.5 * p["dt"] / p["mass"]
    f = _chain_forces(p, x, _centre(p, lam_w, start, 0), k)[0]
    out = []
    for n in range(1, p["n_steps"] + 1):
        v[:, 1:] += hm * f[:, 1:]
        x[:, 1:] += h * v[:, 1:]
        v[:, 1:] = c1 * v[:, 1:] + c2 * _noise_chain(p, gid, n)[:, 1:]
        x[:, 1:] += h * v[:, 1:]
        f = _chain_forces(p, x, _centre(p, lam_w, start, n), k)[0]
        v[:, 1:] += hm * f[:, 1:]
        if _sampled(p, n):
            out.append((x[:, -1] - x[:, 0]).norm(dim=1))
    return torch.stack(out, dim=1).reshape(sw, r, -1)


def _estimates(p, xi):
    """Window statistics, profiles, jackknife errors and the work distribution from samples [S, R, T]."""
    dev = xi.device
    lam = torch.tensor(p["lambda"], dtype=torch.float64, device=dev)
    s, r = lam.numel(), p["n_replicas"]
    beta, k, kT = 1.0 / p["kT"], p["k"], p["kT"]
    x = xi[:s]
    n = float(x[0].numel())
    d = x - lam[:, None, None]
    dl = lam[1:] - lam[:-1]
    mean, std = lam + d.mean(dim=(1, 2)), d.reshape(s, -1).std(dim=1)
    var = std ** 2
    af = beta * k * dl[:, None, None] * (d[:-1] - 0.5 * dl[:, None, None])
    ar = -beta * k * dl[:, None, None] * (d[1:] + 0.5 * dl[:, None, None])
    lf, lr = torch.logsumexp(af, dim=(1, 2)), torch.logsumexp(ar, dim=(1, 2))
    lf2 = torch.logsumexp(2.0 * af, dim=(1, 2))
    nan = lf.new_full((1,), math.nan)

    def profile(step):
        return torch.cat([torch.zeros_like(step[..., :1]), torch.cumsum(step, dim=-1)], dim=-1)

    je = profile(-kT * (lf - math.log(n)))
    fl_step = k * dl * (lam[:-1] - mean[:-1])
    fl = profile(fl_step)
    ga = profile(fl_step + 0.5 * k * dl * dl * (1.0 - k * var[:-1] / kT))
    res = {"xi_mean": mean, "xi_std": std, "gamma2": k * var / kT, "xi_min_sample": x.amin(dim=(1, 2)),
           "xi_max_sample": x.amax(dim=(1, 2)), "lse_fwd": torch.cat([lf, nan]), "lse_rev": torch.cat([nan, lr]),
           "dF_je": je, "dF_fluct": fl, "dF_gauss": ga, "dF_com": 0.5 * (je + fl), "dF_unc": 0.5 * (je - fl),
           "dF_rev": profile(kT * (lr - math.log(n))), "kish_frac": torch.exp(2.0 * lf - lf2) / n,
           "dlambda_over_sigma": dl.abs() / std[:-1]}
    # jackknife over replica blocks, one block left out of every window at once
    nb = min(p["n_blocks"], r)
    blk = torch.arange(r, device=dev) * nb // r
    je_b, fl_b = [], []
    for b in range(nb):
        keep = blk != b
        if not bool(keep.any()):
            return {key: v.cpu().numpy() for key, v in res.items()}
        m = float(int(keep.sum()) * x.shape[2])
        je_b.append(profile(-kT * (torch.logsumexp(af[:, keep], dim=(1, 2)) - math.log(m))))
        fl_b.append(profile(-k * dl * d[:-1, keep].mean(dim=(1, 2))))
    if nb > 1:
        for key, v in (("dF_je_se", torch.stack(je_b)), ("dF_fluct_se", torch.stack(fl_b))):
            res[key] = torch.sqrt((nb - 1.0) / nb * ((v - v.mean(dim=0)) ** 2).sum(dim=0))
    # histograms, their overlap, and the work distribution folded step by step
    bins = torch.floor((x - p["xi_min"]) / p["xi_bin"]).long()
    hist = []
    for w in range(s):
        q = bins[w].reshape(-1)
        hist.append(torch.bincount(q[(q >= 0) & (q < p["xi_nbins"])], minlength=p["xi_nbins"]).double() / n)
    rho = torch.stack(hist)
    res["overlap_ovl"] = torch.minimum(rho[:-1], rho[1:]).sum(dim=1)
    m = p["w_half_bins"]
    if m > 0 and p["precision"] == "fp64":
        om = torch.zeros(s, 2 * m + 1, dtype=torch.float64, device=dev)
        om[0, m] = 1.0
        xb = p["xi_min"] + (torch.arange(p["xi_nbins"], device=dev, dtype=torch.float64) + 0.5) * p["xi_bin"]
        for j in range(1, s):
            dw = 0.5 * k * ((xb - lam[j]) ** 2 - (xb - lam[j - 1]) ** 2)
            shift = torch.floor(dw / p["w_bin"]).long()
            on = rho[j - 1] > 0
            u, where = torch.unique(shift[on], return_inverse=True)
            pr = torch.zeros(u.numel(), dtype=torch.float64, device=dev).index_add_(0, where, rho[j - 1][on])
            for c, q in zip(u.tolist(), pr.tolist()):
                if c >= 0 and c <= 2 * m:
                    om[j, c:] += q * om[j - 1, :2 * m + 1 - c]
                elif -2 * m <= c < 0:
                    om[j, :c] += q * om[j - 1, -c:]
        res["work_hist"] = om
        w = (torch.arange(2 * m + 1, device=dev, dtype=torch.float64) - m) * p["w_bin"]
        tot = om.sum(dim=1)
        res["dF_je_hist"] = -kT * (torch.logsumexp(torch.log(om) - beta * w, dim=1) - torch.log(tot))
    return {key: v.cpu().numpy() for key, v in res.items()}


def exact(case, seed):
    """64-bit values of what `run` returns, None where there is none: fp32 chain runs and
    what is placed or trained on the way depend chaotically on every rounding, so their
    trajectories have no 64-bit counterpart; fp64 chain runs are kept short enough to."""
    kind = case["kind"]
    if kind == "forces":
        p = _forces_problem(case)
        x = _configs(case, seed).reshape(case["configs"], -1, 3)
        f, *e = _chain_forces(p, x, 0.4 * case["beads"], p["k"])
        return {"forces": f.reshape(case["configs"], -1), "energy": torch.stack([sum(e), *e], dim=1)}
    if kind in ("batch", "adaptive"):
        return None
    p = _problem(case, seed)
    if p["model"] == "chain" and (p["precision"] == "fp32" or p["sequential"]):
        return None
    sw = len(p["lambda"]) + 1
    if p["model"] == "chain" and float(p["n_steps"]) * sw * p["n_replicas"] * p["n_beads"] ** 2 > 2e10:
        return None
    xi = _samples_chain(p, "cuda") if p["model"] == "chain" else _samples_1d(p, "cuda")
    if xi.shape[2] == 0:
        return None
    return _estimates(p, xi)
