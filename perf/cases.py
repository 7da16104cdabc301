"""The library's workloads as timed cases: what a program that uses it calls, over the sizes it calls it with.

Every case goes through the public entry points of ``paper_2401_02852_amd``. Instances are random k-NAE-SAT (or
3-SAT) clauses at the clause densities of the repository's own workloads, with one planted solution, since runs are
made on satisfiable instances. Results that the library returns as Python floats are returned as they are; arrays of
results and of gradients come back as float32, which is what the complex64 state behind them carries and what an
optimiser with float32 parameters takes.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2401_02852_amd as q

# Clause densities m / n of the workloads: near the NAE threshold for k = 3, 5 and 9, near the 3-SAT threshold.
DENSITY = {("nae", 3): 2.1, ("nae", 5): 9.0, ("nae", 9): 176.9, ("sat", 3): 4.2}


def listed():
    return [
        # One small instance with its cost resident, as an angle search over one instance calls it: latency.
        {"name": "solve_n12", "kind": "solve", "n": 12, "k": 3, "pred": "nae", "p": 3, "build": False, "state": False, "tuned": False},
        # An ordinary small instance solved once, cost build included; the first sizes above one workgroup.
        {"name": "solve_n17", "kind": "solve", "n": 17, "k": 5, "pred": "nae", "p": 8, "build": True, "state": False, "tuned": False},
        # Plain 3-SAT (no flip symmetry), the final state kept for sampling.
        {"name": "sat_n22_state", "kind": "solve", "n": 22, "k": 3, "pred": "sat", "p": 12, "build": False, "state": True, "tuned": False},
        # A state about as large as the last-level cache, on the tile shape that a tuned program loads for it.
        {"name": "solve_n24_tuned", "kind": "solve", "n": 24, "k": 3, "pred": "nae", "p": 10, "build": False, "state": False, "tuned": True},
        # The benchmark's headline step: cost build and a ten-layer run at n = 30 (8 GiB state).
        {"name": "solve_n30", "kind": "solve", "n": 30, "k": 3, "pred": "nae", "p": 10, "build": True, "state": False, "tuned": False},
        # The half-state entry point, odd n, half state kept.
        {"name": "half_n27", "kind": "half", "n": 27, "k": 3, "p": 10, "state": True},
        # The ragged batch of the benchmark: 512 instances, n 10..20, cost build and run of a fixed set.
        {"name": "batch_512", "kind": "batch", "count": 512, "n_lo": 10, "n_hi": 20, "p": 5, "half": False},
        # One angle-training step on one instance (the benchmark's gradient workload).
        {"name": "grad_n22", "kind": "grad", "n": 22, "k": 3, "p": 12, "w_energy": 0.0},
        # The same beyond the last-level cache, energy term included, odd n.
        {"name": "grad_n25", "kind": "grad", "n": 25, "k": 3, "p": 10, "w_energy": 0.05},
        # One epoch of fixed-angle pretraining: 100 instances, k = 9 (16-bit costs).
        {"name": "pretrain_n12", "kind": "pretrain", "count": 100, "n": 12, "k": 9, "p": 8},
        # A large cost diagonal alone, 16-bit (m = 261).
        {"name": "cost_n29_u16", "kind": "cost", "n": 29, "k": 5},
        # Measuring a final state: 100 000 draws with their costs.
        {"name": "sample_n26", "kind": "sample", "n": 26, "k": 3, "count": 100000},
    ]


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "half", "batch", "grad", "grad", "pretrain", "cost", "sample"])
    if kind == "solve":
        pred = rng.choice(["nae", "nae", "nae", "sat"])
        n = rng.randint(10, 29)
        return {"kind": kind, "n": n, "k": 3 if pred == "sat" else rng.choice([3, 3, 5]), "pred": pred, "p": rng.randint(2, 12 if n < 26 else 8),
                "build": rng.random() < 0.5, "state": rng.random() < 0.3, "tuned": False}
    if kind == "half":
        return {"kind": kind, "n": rng.randint(16, 28), "k": rng.choice([3, 5]), "p": rng.randint(2, 12), "state": rng.random() < 0.5}
    if kind == "batch":
        return {"kind": kind, "count": int(math.exp(rng.uniform(math.log(8), math.log(512)))), "n_lo": rng.randint(8, 12), "n_hi": rng.randint(13, 20),
                "p": rng.randint(2, 8), "half": rng.random() < 0.3}
    if kind == "grad":
        return {"kind": kind, "n": rng.randint(10, 25), "k": rng.choice([3, 3, 5]), "p": rng.randint(3, 12), "w_energy": rng.choice([0.0, 0.05])}
    if kind == "pretrain":
        return {"kind": kind, "count": rng.randint(20, 100), "n": rng.randint(10, 13), "k": rng.choice([3, 5, 9]), "p": rng.randint(2, 8)}
    if kind == "cost":
        k = rng.choice([3, 5, 9])
        return {"kind": kind, "n": rng.randint(12, 20 if k == 9 else 29), "k": k}
    return {"kind": kind, "n": rng.randint(14, 27), "k": 3, "count": int(math.exp(rng.uniform(math.log(1000), math.log(200000))))}


# --------------------------------------------------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------------------------------------------------

def _clauses(n, k, pred, rng):
    m = int(DENSITY[(pred, k)] * n + 0.5)
    v = np.argsort(rng.random((m, n)), axis=1)[:, :k]
    neg = rng.integers(0, 2, (m, k))
    val = rng.integers(0, 2, n)[v] ^ neg  # the literals at the planted solution
    bad = val.sum(axis=1) == 0
    if pred == "nae":
        bad |= val.sum(axis=1) == k
    neg[bad, 0] ^= 1
    return np.where(neg == 1, -(v + 1), v + 1).astype(np.int32)


def _ramp(p, rng):
    """Linear-ramp angles that lower the cost, as the start of a training or as a fixed schedule."""
    l = np.arange(1, p + 1, dtype=np.float64)
    s, t = rng.uniform(0.4, 0.6, 2)
    return s * l / p, -t * (1.0 - l / (p + 1.0))


def _single(case, seed):
    rng = np.random.default_rng([seed, case["n"], case["k"], case.get("p", 0)])
    cl = _clauses(case["n"], case["k"], case.get("pred", "nae"), rng)
    return cl, _ramp(case.get("p", 4), rng), rng


def _many(case, seed):
    rng = np.random.default_rng([seed, case["count"], case["p"]])
    if case["kind"] == "pretrain":
        ns = [case["n"]] * case["count"]
        cls = [_clauses(n, case["k"], "nae", rng) for n in ns]
        return ns, cls, _ramp(case["p"], rng)
    ns = [case["n_lo"] + i % (case["n_hi"] - case["n_lo"] + 1) for i in range(case["count"])]
    rng.shuffle(ns)
    cls = [_clauses(n, int(rng.choice([3, 5])), "nae", rng) for n in ns]
    angles = rng.uniform(0.0, math.pi, (2, case["count"], case["p"]))
    return ns, cls, (angles[0], angles[1])


def _halves(case, ns):
    return [case["half"] and n > 14 for n in ns]


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("batch", "pretrain"):
        ns, cls, (g, b) = _many(case, seed)
        if kind == "pretrain":
            return dict(case, ns=ns, ms=[c.shape[0] for c in cls], g=g, b=b, costs=q.build_cost_diagonals(cls, ns))
        half = _halves(case, ns)
        size = [1 << (n - h) for n, h in zip(ns, half)]
        flat = torch.empty(sum(size), dtype=torch.uint8, device="cuda")
        outs = list(torch.split(flat, size))
        build = q.PreparedCostBuild(cls, ns, outs=outs, half=half)
        return dict(case, flat=flat, make=build, solve=q.PreparedBatch(outs, ns, [c.shape[0] for c in cls], [case["p"]] * len(ns), half=half), g=g, b=b)
    cl, (g, b), rng = _single(case, seed)
    n = case["n"]
    s = dict(case, cl=cl, g=g, b=b, m=cl.shape[0], psi=None)
    if kind == "half":
        s["cost"] = q.build_cost_diagonal_z2(cl, n)
        if case["state"]:
            s["psi"] = torch.empty(1 << (n - 1), dtype=torch.complex64, device="cuda")
        return s
    s["cost"] = q.build_cost_diagonal(cl, n, predicate=case.get("pred", "nae"))
    if kind == "solve":
        if n > 14:
            shape = {"tile_bits": 14, "low_run_bits": 4, "page_bit": 18, "split": 0}
            q.default_context().set_tune(n, shape if case["tuned"] else None)
        if case["state"]:
            s["psi"] = torch.empty(1 << n, dtype=torch.complex64, device="cuda")
    elif kind == "sample":
        s["psi"] = torch.empty(1 << n, dtype=torch.complex64, device="cuda")
        q.qaoa_run(s["cost"], n, s["m"], g, b, state=s["psi"])
        s["u"] = rng.random(case["count"])
    return s


# --------------------------------------------------------------------------------------------------------------------
# One pass
# --------------------------------------------------------------------------------------------------------------------

def _plain(cost):
    """16-bit costs (all far below 2^15) as int16, which every torch operation takes."""
    return cost.view(torch.int16) if cost.dtype == torch.uint16 else cost


def run(s):
    kind = s["kind"]
    if kind == "solve":
        if s["build"]:
            q.build_cost_diagonal(s["cl"], s["n"], out=s["cost"], predicate=s["pred"])
        r = q.qaoa_run(s["cost"], s["n"], s["m"], s["g"], s["b"], state=s["psi"])
        return [r, s["psi"], _plain(s["cost"]) if s["build"] else None]
    if kind == "half":
        return [q.qaoa_run_z2(s["cost"], s["n"], s["m"], s["g"], s["b"], state=s["psi"]), s["psi"]]
    if kind == "batch":
        s["make"].build()
        r = torch.from_numpy(s["solve"].run(s["g"], s["b"])).float()
        return [r[:, 0], r[:, 1], r[:, 2], s["flat"]]
    if kind == "grad":
        dg, db, r = q.qaoa_grad(s["cost"], s["n"], s["m"], s["g"], s["b"], w_psucc=1.0, w_energy=s["w_energy"])
        return [torch.from_numpy(dg).float(), torch.from_numpy(db).float(), r]
    if kind == "pretrain":
        c = s["count"]
        dg, db, r = q.qaoa_grad_batched(s["costs"], s["ns"], s["ms"], [s["g"]] * c, [s["b"]] * c, w_psucc=1.0 / c)
        return [torch.from_numpy(np.stack(dg)).float(), torch.from_numpy(np.stack(db)).float(), torch.tensor([x.p_success for x in r])]
    if kind == "cost":
        return [_plain(q.build_cost_diagonal(s["cl"], s["n"], out=s["cost"]))]
    x, c = q.sample(s["psi"], s["n"], s["u"], cost=s["cost"])
    return [x.view(np.int64), c]


def work(case):
    """Inputs read once, outputs written once; a layer costs a complex product and n butterflies of 4 operations an amplitude."""
    kind = case["kind"]
    if kind in ("batch", "pretrain"):
        ns = _many(case, 1)[0]
        h = _halves(case, ns) if kind == "batch" else [False] * len(ns)
        amps = [2.0 ** (n - x) for n, x in zip(ns, h)]
        reps = 1 if kind == "batch" else 4  # forward; forward, and two states backward
        cb = 2 if kind == "pretrain" and DENSITY[("nae", case["k"])] * case["n"] > 255 else 1
        return {"bytes": cb * sum(amps), "flops": reps * case["p"] * sum(a * (4.0 * n + 6.0) for a, n in zip(amps, ns))}
    n, k = case["n"], case["k"]
    m = int(DENSITY[(case.get("pred", "nae"), k)] * n + 0.5)
    cb = 1 if m <= 255 else 2
    amps = 2.0 ** (n - 1 if kind == "half" else n)
    layer = amps * (4.0 * n + 6.0)
    if kind == "cost":
        return {"bytes": cb * amps, "flops": 0}
    if kind == "sample":
        return {"bytes": 8.0 * amps + 20.0 * case["count"], "flops": 3.0 * amps}
    if kind == "grad":
        return {"bytes": cb * amps, "flops": 4 * case["p"] * layer}
    return {"bytes": cb * amps * (2 if case.get("build") else 1) + (8.0 * amps if case["state"] else 0.0), "flops": case["p"] * layer}


# --------------------------------------------------------------------------------------------------------------------
# The same in 64 bits, in plain torch
# --------------------------------------------------------------------------------------------------------------------

def _cost64(cl, n, pred, top=None):
    """Violated clauses at every x < 2^n (or < top), by evaluating every literal."""
    top = top or 1 << n
    var = torch.from_numpy(np.abs(cl).astype(np.int64) - 1).cuda()
    neg = torch.from_numpy((cl < 0).astype(np.int64)).cuda()
    out = torch.empty(top, dtype=torch.int16, device="cuda")
    step = min(top, 1 << 20)
    rows = max(1, (1 << 26) // (step * cl.shape[1]))
    for x0 in range(0, top, step):
        x = torch.arange(x0, x0 + step, device="cuda")
        tot = torch.zeros(step, dtype=torch.int32, device="cuda")
        bits = torch.stack([((x >> v) & 1).to(torch.uint8) for v in range(n)])
        for c in range(0, cl.shape[0], rows):
            true = bits[var[c:c + rows]] ^ neg[c:c + rows, :, None].to(torch.uint8)  # [rows, k, step]
            cnt = true.sum(dim=1, dtype=torch.uint8)
            tot += ((cnt == 0) | (cnt == cl.shape[1]) if pred == "nae" else cnt == 0).sum(dim=0, dtype=torch.int32)
        out[x0:x0 + step] = tot.to(torch.int16)
    return out


def _mix64(psi, n, beta):
    """exp(-i beta X) on every qubit: the lowest five (or what is left) as a dense 2^w x 2^w product over rows of 2^w
    amplitudes, whose bits then go to the top."""
    c, s = torch.cos(beta), torch.sin(beta)
    left = n
    while left:
        w = min(5, left)
        i = torch.arange(1 << w, device="cuda")
        d = i[:, None] ^ i[None, :]
        pop = sum((d >> j) & 1 for j in range(w))
        phase = torch.tensor([1, -1j, -1, 1j], dtype=torch.complex128, device="cuda")[pop % 4]
        m = phase * (c ** (w - pop) * s ** pop)
        rows = psi.view(-1, 1 << w)
        if rows.shape[0] <= 1 << 22:
            psi = torch.mm(rows, m).t().contiguous().view(-1)
        else:
            out = torch.empty(1 << w, rows.shape[0], dtype=torch.complex128, device="cuda")
            for r in range(0, rows.shape[0], 1 << 22):
                out[:, r:r + (1 << 22)] = torch.mm(rows[r:r + (1 << 22)], m).t()
            psi = out.view(-1)
        left -= w
    return psi


def _state64(cost, n, g, b):
    psi = torch.full((1 << n,), 2.0 ** (-n / 2), dtype=torch.complex128, device="cuda")
    for l in range(len(g)):
        if torch.is_tensor(g):
            psi = psi * torch.exp(-1j * (g[l] * cost.to(torch.float64)))
            psi = _mix64(psi, n, b[l])
        else:
            t = torch.exp(-1j * float(g[l]) * torch.arange(int(cost.max()) + 1, dtype=torch.float64, device="cuda"))
            for x in range(0, 1 << n, 1 << 26):
                psi[x:x + (1 << 26)] *= t[cost[x:x + (1 << 26)].long()]
            psi = _mix64(psi, n, torch.tensor(float(b[l]), dtype=torch.float64, device="cuda"))
    return psi


def _readout64(psi, cost):
    ps = e = nn = 0.0
    for x in range(0, psi.numel(), 1 << 26):
        pr = torch.view_as_real(psi[x:x + (1 << 26)]).square().sum(dim=1)
        c = cost[x:x + (1 << 26)]
        ps, e, nn = ps + pr[c == 0].sum(), e + (pr * c).sum(), nn + pr.sum()
    return ps, e, nn


def _grad64(cost, n, g, b, w_p, w_e):
    g = torch.tensor(g, dtype=torch.float64, device="cuda", requires_grad=True)
    b = torch.tensor(b, dtype=torch.float64, device="cuda", requires_grad=True)
    r = _readout64(_state64(cost, n, g, b), cost)
    dg, db = torch.autograd.grad(w_p * r[0] + w_e * r[1], [g, b])
    return dg, db, [x.item() for x in r]


def exact(case, seed):
    kind = case["kind"]
    if kind in ("cost", "sample"):
        return None  # integers
    if kind in ("batch", "pretrain"):
        ns, cls, (g, b) = _many(case, seed)
        if kind == "pretrain":
            got = [_grad64(_cost64(c, n, "nae"), n, g, b, 1.0 / case["count"], 0.0) for n, c in zip(ns, cls)]
            return [torch.stack([x[0] for x in got]), torch.stack([x[1] for x in got]), torch.tensor([x[2][0] for x in got], dtype=torch.float64)]
        r = []
        for n, c, gi, bi in zip(ns, cls, g, b):
            cost = _cost64(c, n, "nae")
            r.append(torch.stack(_readout64(_state64(cost, n, gi, bi), cost)))
        r = torch.stack(r)
        return [r[:, 0], r[:, 1], r[:, 2], None]
    cl, (g, b), _ = _single(case, seed)
    n = case["n"]
    cost = _cost64(cl, n, case.get("pred", "nae"))
    if kind == "grad":
        dg, db, r = _grad64(cost, n, g, b, 1.0, case["w_energy"])
        return [dg, db, _wide(r)]
    psi = _state64(cost, n, g, b)
    r = _wide([x.item() for x in _readout64(psi, cost)])
    if kind == "half":
        return [r, psi[:1 << (n - 1)] if case["state"] else None]
    return [r, psi if case["state"] else None, None]


def _wide(values):
    return [torch.tensor(v, dtype=torch.float64) for v in values]
