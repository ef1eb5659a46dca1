"""Performance cases of the sampler: what its users have it do, at the sizes they do it.

A case is a dict of plain values. ``listed()`` gives the fixed ones, ``draw(rng)`` one more of
the same ranges, ``prepare(case, seed)`` what a program holds before the call, ``run(state)`` one
pass through the public entry points, ``work(case)`` the bytes and operations of one pass that no
implementation can do without, and ``exact(case, seed)`` the outputs in 64 bits where they are
computed numbers that follow from the inputs in a few lines of numpy.

Kinds:
  iterate  rounds of the weight iteration: sweeps, the device update, the training targets
  produce  sweeps under fixed production weights, round-trip times and histograms read back
  pt       parallel tempering sweeps, slots, exchanges and walkers read back, temperatures adapted
  update   the weight update alone, from histograms the program hands over
  samples  a new batch: couplings, spins, energies and the couplings' statistics
  train    Adam steps of the weight-seeding network, minibatch by minibatch
  infer    its BF16 inference
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2011_08560_amd import nfm

SEED = 20110856
F_TOL = 0.5


def listed():
    return [
        # a first look at one sample: one wave of walkers, a few sweeps, everything read back
        {"name": "look L8x1", "kind": "iterate", "mix": "8:1", "walkers": 64, "sweeps": 10, "profile": 0,
         "dE": 1.0, "alpha": 0.0, "schedule": 0, "chunk": 0},
        # the smallest batch of the benchmark: L = 4, 32 realizations, flat target
        {"name": "iterate L4x32", "kind": "iterate", "mix": "4:32", "walkers": 64, "sweeps": 500, "profile": 0,
         "dE": 1.0, "alpha": 0.0, "schedule": 0, "chunk": 0},
        # its L = 6 batch: one wave of walkers per SIMD
        {"name": "iterate L6x1024", "kind": "iterate", "mix": "6:1024", "walkers": 64, "sweeps": 1000, "profile": 1,
         "dE": 1.0, "alpha": -1.0, "schedule": 0, "chunk": 1000},
        # its L = 8 batch: production under the paper's power law, several waves per SIMD
        {"name": "produce L8x4096", "kind": "produce", "mix": "8:4096", "walkers": 64, "sweeps": 500, "profile": 1,
         "dE": 96.0, "alpha": -3.6, "schedule": 0, "chunk": 0},
        # its default workload: five sizes in one batch under the launch the autotuner picks for it
        {"name": "iterate mixed", "kind": "iterate", "mix": "4:4096,6:2048,8:1024,10:512,12:256", "walkers": 64,
         "sweeps": 256, "profile": 1, "dE": 1.0, "alpha": -1.0, "schedule": 2, "chunk": 256},
        # the largest lattice alone, two waves of walkers per sample: long serial chains
        {"name": "produce L12x200", "kind": "produce", "mix": "12:200", "walkers": 128, "sweeps": 60, "profile": 0,
         "dE": 1.0, "alpha": 0.0, "schedule": 0, "chunk": 0},
        # tempering with 32 fixed temperatures, two sets per wave
        {"name": "pt L8x2048 M32", "kind": "pt", "mix": "8:2048", "walkers": 64, "sweeps": 400, "M": 32,
         "t0": 0.2, "t1": 2.0, "adapt": False},
        # the paper's tempering protocol at L = 6: 14 temperatures, adapted after each round
        {"name": "pt L6x500 M14 adapt", "kind": "pt", "mix": "6:500", "walkers": 64, "sweeps": 500, "M": 14,
         "t0": 0.2, "t1": 3.2, "adapt": True},
        # the update of a batch's estimates between two rounds
        {"name": "update L8x1024", "kind": "update", "L": 8, "real": 1024, "profile": 1, "dE": 1.0, "alpha": -1.0},
        # the start of a campaign
        {"name": "samples L10x1024", "kind": "samples", "mix": "10:1024", "walkers": 64},
        # the seeding network: training minibatches, inference over an evaluation set (odd size)
        {"name": "train B256", "kind": "train", "batch": 256, "steps": 8},
        {"name": "infer B1000", "kind": "infer", "batch": 1000},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.999)))))))


def draw(rng):
    kind = rng.choice(["iterate", "iterate", "produce", "produce", "mixed", "pt", "pt", "update", "samples", "train",
                       "infer"])
    if kind == "train":
        return {"kind": kind, "batch": _log_int(rng, 1, 1024), "steps": rng.randint(1, 12)}
    if kind == "infer":
        return {"kind": kind, "batch": _log_int(rng, 1, 8192)}
    if kind == "mixed":
        sizes = sorted(rng.sample([2, 4, 6, 8, 10, 12], rng.randint(2, 4)))
        mix = ",".join(f"{L}:{_log_int(rng, 1, max(8, 2 ** 18 // L ** 3))}" for L in sizes)
        walkers, kind = 64, "iterate"
    else:
        L = rng.choice([2, 4, 6, 8, 10, 12])
        mix = f"{L}:{_log_int(rng, 1, max(16, min(4096, 2 ** 21 // L ** 3)))}"
        walkers = rng.choice([64, 64, 128, 192])
        if kind == "update":
            L = max(L, 4)
            return {"kind": kind, "L": L, "real": _log_int(rng, 1, min(2048, 2 ** 19 // L ** 3)),
                    "profile": rng.choice([0, 1, 2]), "dE": rng.choice([1.0, 24.0, 96.0]),
                    "alpha": rng.choice([-1.0, -2.0, -3.6])}
        if kind == "samples":
            return {"kind": kind, "mix": mix, "walkers": walkers}
    sizes = _mix(mix)
    # at most the work of the largest listed case, and chains no longer than 20 ms or so
    per_sweep = walkers * sum(L ** 3 * r for L, r in sizes)
    cap = min(4e10 / per_sweep, 2.5e5 / max(L for L, _ in sizes) ** 3)
    sweeps = _log_int(rng, 1, max(2, int(cap)))
    if kind == "pt":
        M = rng.choice([2, 7, 12, 14, 20, 32, 64, rng.randint(2, 64)])
        return {"kind": kind, "mix": mix, "walkers": walkers, "sweeps": max(sweeps, 2), "M": M, "t0": 0.2,
                "t1": rng.choice([2.0, 3.2]), "adapt": rng.random() < 0.5}
    profile = rng.choice([0, 1, 1, 2])
    return {"kind": kind, "mix": mix, "walkers": walkers, "sweeps": sweeps, "profile": profile,
            "dE": rng.choice([1.0, 24.0, 96.0]), "alpha": rng.choice([-1.0, -2.0, -3.6]),
            "schedule": rng.choice([0, 1, 2]) if len(sizes) > 1 else rng.choice([0, 0, 1]),
            "chunk": rng.choice([0, 64, 256])}


def _mix(text):
    return [tuple(int(v) for v in part.split(":")) for part in text.split(",")]


def _batch(case, seed):
    Ls = [L for L, r in _mix(case["mix"]) for _ in range(r)]
    b = nfm.Batch(Ls, [case["walkers"]] * len(Ls), disorder_seed=SEED + seed, walker_seed=SEED + 7919 * seed + 1)
    b.init_couplings()
    b.init_spins()
    b.compute_energies()
    return b


def _warm(b, case, rounds, sweeps):
    """A few rounds of the weight iteration, so that tables, bounds and walkers are those of a run."""
    b.rec_init(case["profile"], case["dE"], case["alpha"])
    for _ in range(rounds):
        b.run_sweeps(sweeps)
        b.rec_update(F_TOL)


# ------------------------------------------------------------------ the update's inputs (numpy)

def _update_inputs(case, seed):
    """Couplings (ABI words) and, per realization, a weight-iteration state on the way to
    convergence: steps b near 4 beta(E) of a Gaussian density of states with noise, accumulated
    weights, the weights of the target profile, and a histogram near flat with counting noise, in
    every other realization with a few levels not visited this round."""
    L, R = case["L"], case["real"]
    N = L ** 3
    cap = 3 * N // 2 + 1
    rng = np.random.default_rng([seed, L, R])
    jw = (N + 31) // 32
    J = rng.integers(0, 2 ** 32, size=(R, 3, jw), dtype=np.uint64).astype(np.uint32)
    if N % 32:
        J[:, :, -1] &= np.uint32((1 << (N % 32)) - 1)
    n_minus = np.unpackbits(J.reshape(R, -1).view(np.uint8), axis=1).sum(axis=1).astype(np.int64)
    out = []
    for r in range(R):
        e_base = -3 * N + 2 * int(n_minus[r] % 2)
        k_top = (-e_base + 3) // 4
        k_lo = -(-(int(-rng.uniform(1.60, 1.72) * N) - e_base) // 4)
        k = np.arange(cap)
        E = e_base + 4.0 * k
        b = np.where((k >= k_lo) & (k < k_top), 4.0 * np.maximum(-E, 0.0) / (2.2 * N) + rng.normal(0, 0.02, cap), 0.0)
        p = np.where((k >= k_lo) & (k < k_top), rng.uniform(50.0, 2000.0, cap), 0.0)
        visited = ((k >= k_lo) & (k <= k_top)).astype(np.uint8)
        S, lnP, lnW = _weights(e_base, k_lo, k_top, b, case["profile"], case["dE"], case["alpha"])
        lam = 64 * 200.0 / (k_top - k_lo + 1) * np.exp(rng.normal(0, 0.3, cap))
        H = np.where((k >= k_lo) & (k <= k_top + 8), rng.poisson(lam), 0).astype(np.uint64)
        if r % 2:   # levels known from earlier rounds that this one missed
            H[k_lo + rng.integers(0, max(1, k_top - k_lo), 3)] = 0
        out.append((e_base, k_lo, k_top, b, p, lnP, lnW, visited, H))
    return J.reshape(R, -1), out


def _weights(e_base, k_lo, k_top, b, profile, dE, alpha):
    """S, ln P and ln W on [k_lo, k_top] (zero elsewhere) from the steps b."""
    n = len(b)
    S, lnP = np.zeros(n), np.zeros(n)
    S[k_lo:k_top] = -np.cumsum(b[k_lo:k_top][::-1])[::-1]
    E = e_base + 4.0 * np.arange(k_lo, k_top + 1)
    if profile == 1:
        lnP[k_lo:k_top + 1] = alpha * np.log(E / (dE - E[0]) + 1.0)
    elif profile == 2:
        lnP[k_lo:k_top + 1] = S[k_lo:k_top + 1] - np.logaddexp.accumulate(S[k_lo:k_top + 1])
    lnW = np.zeros(n)
    lnW[k_lo:k_top + 1] = -S[k_lo:k_top + 1] + lnP[k_lo:k_top + 1]
    return S, lnP, lnW


# ------------------------------------------------------------------ the network's inputs

N_PARAM = 78464
LAYERS = ((96, 128), (128, 128), (128, 128), (128, 256))


def _net_inputs(case, seed, rows, batches=1):
    """Parameters (uniform +-sqrt(6 / (in + out)), small biases), inputs with the spread of the
    features, targets and masks shaped like the training set's."""
    rng = np.random.default_rng([seed, rows, 5])
    parts = []
    for i, (n_in, n_out) in enumerate(LAYERS):
        fan = 81 if i == 0 else n_in
        W = rng.uniform(-1, 1, (n_in, n_out)) * math.sqrt(6.0 / (fan + n_out))
        if i == 0:
            W[81:] = 0.0
        parts += [W.ravel(), rng.normal(0, 0.05, n_out)]
    theta = np.concatenate(parts).astype(np.float32)
    norm = np.stack([rng.uniform(0.0, 0.6, 81), rng.uniform(0.01, 0.2, 81)]).astype(np.float32)
    X = (norm[0] + norm[1] * rng.normal(0, 1, (batches, rows, 81))).astype(np.float32)
    e = -2.0 + 2.0 * np.arange(256) / 255.0
    T = (-0.45 * e * e * rng.uniform(0.9, 1.1, (batches, rows, 1)) + rng.normal(0, 0.01, (batches, rows, 256)))
    mask = (e >= rng.uniform(-1.78, -1.55, (batches, rows, 1)))
    return theta, norm, X, (T * mask).astype(np.float32), mask.astype(np.float32)


# ------------------------------------------------------------------ prepare and run

def prepare(case, seed):
    kind = case["kind"]
    if kind in ("iterate", "produce"):
        b = _batch(case, seed)
        if case["schedule"] or case["chunk"]:
            b.set_tuning(schedule=case["schedule"], sweeps_per_launch=case["chunk"])
        _warm(b, case, 4, max(10, min(150, case["sweeps"])))
        if kind == "produce":
            b.rec_production(case["profile"], case["dE"], case["alpha"])
            b.reset_round_trips()
        b.sync()
        return {"case": case, "b": b}
    if kind == "pt":
        b = _batch(case, seed)
        M = case["M"]
        b.pt_init([case["t0"] * (case["t1"] / case["t0"]) ** (s / (M - 1)) for s in range(M)])
        for r in range(b.n_real):
            N = int(b.Ls[r]) ** 3
            b.set_rt_bounds(r, int(-1.66 * N), int(-1.40 * N))
        b.pt_run_sweeps(50)
        b.reset_round_trips()
        b.sync()
        return {"case": case, "b": b}
    if kind == "update":
        L, R = case["L"], case["real"]
        J, reals = _update_inputs(case, seed)
        b = nfm.Batch([L] * R, [64] * R, disorder_seed=SEED, walker_seed=SEED + seed)
        b.set_couplings(0, J)
        b.init_spins()
        b.compute_energies()
        b.rec_init(case["profile"], case["dE"], case["alpha"])
        for r, (_, k_lo, k_top, bs, p, lnP, lnW, vis, _) in enumerate(reals):
            b.rec_set_state(r, bs, p, lnP, lnW, vis, k_lo, k_top, case["profile"], case["dE"], case["alpha"])
        return {"case": case, "b": b, "H": np.concatenate([x[8] for x in reals])}
    if kind == "samples":
        Ls = [L for L, r in _mix(case["mix"]) for _ in range(r)]
        b = nfm.Batch(Ls, [case["walkers"]] * len(Ls), disorder_seed=SEED + seed, walker_seed=SEED + 7919 * seed + 1)
        b.reset_histograms()
        return {"case": case, "b": b}
    theta, norm, X, T, mask = _net_inputs(case, seed, case["batch"], case.get("steps", 1))
    net = nfm.Mlp(batch_max=case["batch"])
    net.set_params(theta, norm)
    net.to_bf16()
    dev = net.device
    return {"case": case, "net": net, "x": [torch.tensor(v, device=dev) for v in X],
            "t": [torch.tensor(v, device=dev) for v in T], "m": [torch.tensor(v, device=dev) for v in mask]}


def _fields(a, skip=("pad", "reserved")):
    return {k: np.ascontiguousarray(a[k]) for k in a.dtype.names if k not in skip}


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "iterate":
        b = state["b"]
        b.run_sweeps(case["sweeps"])
        real = _fields(b.read_realizations())
        info = _fields(b.rec_update(F_TOL))
        y, m = b.rec_targets()
        out = {"real": real, "info": info, "y": y, "mask": m}
        if b.n_walkers <= 4096:   # a small batch: its walkers as well
            out["walkers"] = _fields(b.read_walkers())
        return out
    if kind == "produce":
        b = state["b"]
        b.run_sweeps(case["sweeps"])
        tau, summ = b.rt_stats(min_trips=1)
        return {"tau": tau, "trips": int(summ["trips"]), "used": int(summ["n_used"]),
                "real": _fields(b.read_realizations()), "hist": b.read_histograms()}
    if kind == "pt":
        b, M = state["b"], case["M"]
        b.pt_run_sweeps(case["sweeps"])
        out = {"slots": b.pt_slots(), "acc": b.pt_exchanges(M), "walkers": _fields(b.read_walkers())}
        if case["adapt"]:
            out["rates"], out["outside"] = b.pt_adapt(M)
        return out
    if kind == "update":
        b = state["b"]
        b.set_histograms(state["H"])
        info = b.rec_update(F_TOL)
        y, m = b.rec_targets()
        return {"flatness": info["flatness"].copy(), "k_lo": info["k_lo"].copy(), "k_top": info["k_top"].copy(),
                "converged": info["converged"].copy(), "y": y, "mask": m}
    if kind == "samples":
        b = state["b"]
        b.init_couplings()
        b.init_spins()
        b.compute_energies()
        x = b.features()
        J = [b.get_couplings(0, b.n_real)]
        return {"x": x, "J": J, "real": _fields(b.read_realizations())}
    net = state["net"]
    if kind == "infer":
        return {"y": net.infer_bf16(state["x"][0])}
    for x, t, m in zip(state["x"], state["t"], state["m"]):
        net.train_step(x, t, m, lr=1e-3)
    return {"loss": net.last_loss(), "params": net.get_params()[0], "grads": net.get_grads()}


# ------------------------------------------------------------------ the least work of a pass

# integer operations of one spin-flip attempt with word-parallel neighbour counts: the share of a
# Philox4x32-10 call 10, neighbour count 1, table address 2, acceptance 2, update 2, bookkeeping 1
OPS_PER_ATTEMPT = 18


def work(case):
    kind = case["kind"]
    if kind in ("train", "infer"):
        B, macs = case["batch"], sum(i * o for i, o in LAYERS)
        if kind == "infer":
            return {"bytes": 4 * B * (81 + 256) + 2 * N_PARAM, "flops": 2 * B * macs}
        return {"bytes": case["steps"] * (4 * B * (81 + 2 * 256) + 4 * 6 * N_PARAM),
                "flops": case["steps"] * 2 * B * (3 * macs - LAYERS[0][0] * LAYERS[0][1])}
    if kind == "update":
        levels = case["real"] * (3 * case["L"] ** 3 // 2 + 1)
        # histogram in and cleared; b, p in and out; lnW, lnP in and out, S out; table out, over
        # the levels between the ground state and E = 0
        used = case["real"] * int(1.66 * case["L"] ** 3 / 4)
        return {"bytes": 2 * 8 * levels + used * (8 * 9 + 32), "flops": used * 100}
    sizes, W = _mix(case["mix"]), case["walkers"]
    spins = sum(W * r * L ** 3 / 8 for L, r in sizes)
    bonds = sum(r * 3 * L ** 3 / 8 for L, r in sizes)
    walkers = sum(W * r for _, r in sizes)
    if kind == "samples":
        return {"bytes": spins + bonds + 40 * walkers, "flops": sum(W * r * L ** 3 for L, r in sizes) * 8}
    attempts = case["sweeps"] * sum(W * r * L ** 3 for L, r in sizes)
    table = sum(r * 32 * 1.66 * L ** 3 / 4 for L, r in sizes)
    return {"bytes": 2 * spins + bonds + 2 * 40 * walkers + 2 * table, "flops": attempts * OPS_PER_ATTEMPT}


# ------------------------------------------------------------------ the same in 64 bits

def exact(case, seed):
    kind = case["kind"]
    if kind == "update":
        return _exact_update(case, seed)
    if kind in ("train", "infer"):
        return _exact_net(case, seed)
    return None   # whole numbers and what follows from them: the chains have no short form


def _exact_update(case, seed):
    _, reals = _update_inputs(case, seed)
    N = case["L"] ** 3
    e = -2.0 + 2.0 * np.arange(256) / 255.0
    flat, ys, ms = [], [], []
    for e_base, k_lo, k_top, b, p, lnP, lnW, vis, H in reals:
        H = H.astype(np.float64)
        b, p, vis = b.copy(), p.copy(), vis.copy()
        k = k_lo + np.flatnonzero(H[k_lo:k_top + 1])
        lo, hi = k[:-1], k[1:]
        c = np.concatenate([[0.0], np.cumsum(b)])
        est = (np.log(H[hi]) - lnW[hi]) - (np.log(H[lo]) - lnW[lo])
        g0 = H[lo] * H[hi] / (H[lo] + H[hi])
        p[lo] += g0
        b[lo] += g0 / p[lo] * (est - (c[hi] - c[lo]))
        vis[k] = 1
        kv = k_lo + np.flatnonzero(vis[k_lo:k_top + 1])
        v = H[kv] / np.exp(lnP[kv])
        flat.append(v.min() / v.mean() if v.sum() > 0 else 0.0)
        S, _, _ = _weights(e_base, k_lo, k_top, b, case["profile"], case["dE"], case["alpha"])
        E = e * N
        t = (E - e_base) / 4.0
        f = np.clip(np.floor(t).astype(int), k_lo, k_top - 1)
        y = np.where(E >= e_base + 4 * k_top, S[k_top], S[f] + (t - f) * (S[f + 1] - S[f])) / N
        m = E >= e_base + 4 * k_lo
        ys.append(np.where(m, y, 0.0))
        ms.append(m.astype(np.float64))
    return {"flatness": np.array(flat), "k_lo": None, "k_top": None, "converged": None, "y": np.stack(ys),
            "mask": np.stack(ms)}


def _exact_net(case, seed):
    theta, norm, X, T, mask = _net_inputs(case, seed, case["batch"], case.get("steps", 1))
    th = torch.tensor(theta, dtype=torch.float64, requires_grad=True)
    nm = torch.tensor(norm, dtype=torch.float64)

    def forward(x):
        h = torch.nn.functional.pad((torch.tensor(x, dtype=torch.float64) - nm[0]) / nm[1], (0, 15))
        o = 0
        for i, (n_in, n_out) in enumerate(LAYERS):
            W, o = th[o:o + n_in * n_out].reshape(n_in, n_out), o + n_in * n_out
            h, o = h @ W + th[o:o + n_out], o + n_out
            if i < 3:
                h = 0.5 * h * (1.0 + torch.erf(h / math.sqrt(2.0)))
        return h

    if case["kind"] == "infer":
        return {"y": forward(X[0]).detach()}
    am, av = torch.zeros(N_PARAM, dtype=torch.float64), torch.zeros(N_PARAM, dtype=torch.float64)
    for s in range(case["steps"]):
        m = torch.tensor(mask[s], dtype=torch.float64)
        loss = (m * (forward(X[s]) - torch.tensor(T[s], dtype=torch.float64)) ** 2).sum() / m.sum()
        (g,) = torch.autograd.grad(loss, th)
        am, av = 0.9 * am + 0.1 * g, 0.999 * av + 0.001 * g * g
        with torch.no_grad():
            th -= 1e-3 * (am / (1 - 0.9 ** (s + 1))) / ((av / (1 - 0.999 ** (s + 1))).sqrt() + 1e-8)
    return {"loss": float(loss.detach()), "params": th.detach(), "grads": g}
