"""Timed cases of the library's public entry points: each is a whole
multi-start search (``Handle.solve``: random starts, sweeps or passes, best
restart) on one of the instance families of ``instances``, with what a caller
reads back after it.

``listed`` holds the fixed cases, ``draw`` draws further ones of the same
ranges, ``prepare`` builds a case's instances from a seed and binds them to
the GPU, ``run`` is one search and its readout, ``work`` the bytes and integer
operations a search cannot do without, and ``exact`` the result of the sweeps
on the smaller lattices in plain numpy.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import instances as gen
import paper_0912_3912_amd as sg
from paper_0912_3912_amd import factoring

RULES = {"greedy": sg.GREEDY, "tie": sg.GREEDY_TIE, "fm": sg.FM}

# Sweeps (or passes) of a search that runs until it converges, per replica, as
# the work model counts them (means over random instances of each family).
TYPICAL = {"lattice": 6, "chimera": 5, "er": 9, "regular3": 7, "factoring": 3, "fm": 6}


def listed():
    return [
        # One small lattice, 64 starts: the smallest call a program makes,
        # usually in a loop over instances; latency and launches count.
        _lattice("square16_greedy", "16x16", "pm1", 64, "greedy"),
        # The 50x50 quality benchmark of the pass-based search with ln^2 n
        # starts, bimodal couplings.
        _lattice("square50_fm", "50x50", "pm1", 62, "fm"),
        # The same with Gaussian couplings, rounded to integers that need 32
        # bits: the distribution that benchmark is quoted on.
        _lattice("square50_gauss_fm", "50x50", "gauss32", 62, "fm"),
        # The paper's 164x164 bimodal grid: four passes from 64 starts.
        _lattice("square164_fm", "164x164", "pm1", 64, "fm", sweeps=4),
        # 10^6 spins in three dimensions with fields, 1000 sweeps with tie
        # moves from one start: the benchmark's headline, the largest case.
        _lattice("cubic100_tie", "100x100x100", "pm1", 1, "tie", hmax=2, sweeps=1000),
        # A large lattice with couplings of several magnitudes and a fixed
        # number of sweeps.
        _lattice("cubic64_j3_tie", "64x64x64", "j3", 1, "tie", hmax=2, sweeps=300),
        # Batches of small annealer graphs, many restarts each, under the
        # three rules: descent, descent with tie moves, pass-based search.
        _chimera("chimera_greedy", 8, 1024, 256, "greedy"),
        _chimera("chimera_tie", 8, 1024, 256, "tie", sweeps=50, energies=True),
        _chimera("chimera_fm", 8, 1024, 256, "fm", energies=True),
        # An uneven batch: random graphs with three-spin terms, sizes
        # log-uniform over three decades, a few restarts each.
        {"name": "er_greedy", "family": "er", "count": 96, "n_lo": 100, "n_hi": 100000, "restarts": 8,
         "rule": "greedy", "sweeps": 10000, "converge": True, "energies": True},
        # One large sparse graph without a lattice's structure.
        {"name": "regular3_greedy", "family": "regular3", "n": 500000, "restarts": 1, "rule": "greedy",
         "sweeps": 10000, "converge": True},
        # Factoring 612171 with 10 + 10 free bits from 15000 random starts.
        {"name": "factoring_fm", "family": "factoring", "N": 612171, "nx": 10, "ny": 10, "restarts": 15000,
         "rule": "fm", "sweeps": 1000, "converge": True, "energies": True},
    ]


def _lattice(name, dims, couplings, restarts, rule, hmax=0, sweeps=None):
    return {"name": name, "family": "lattice", "dims": dims, "couplings": couplings, "hmax": hmax,
            "restarts": restarts, "rule": rule, "sweeps": sweeps or 10000, "converge": sweeps is None}


def _chimera(name, side, count, restarts, rule, sweeps=None, energies=False):
    return {"name": name, "family": "chimera", "side": side, "count": count, "restarts": restarts, "rule": rule,
            "sweeps": sweeps or 10000, "converge": sweeps is None, "energies": energies}


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_lattice(rng):
    kind = rng.choice(["small", "fm", "fm", "large_fm", "large", "large"])
    if kind == "small":  # one workgroup per replica
        L = 2 * int(_log(rng, 3, 120))
        c = _lattice("", "%dx%d" % (L, L), rng.choice(["pm1", "j3"]), int(_log(rng, 1, 300)),
                     rng.choice(["greedy", "greedy", "tie"]), hmax=rng.choice([0, 2]))
        if c["rule"] == "tie":
            c.update(sweeps=100, converge=False)
        return c
    if kind == "fm":  # sides of either parity, one wavefront per replica
        return _lattice("", "%dx%d" % (rng.randint(33, 64), rng.randint(33, 63)),
                        rng.choice(["pm1", "gauss32", "j3"]), int(_log(rng, 16, 400)), "fm",
                        hmax=rng.choice([0, 1]))
    if kind == "large_fm":
        L = int(_log(rng, 66, 250))
        return _lattice("", "%dx%d" % (L, L + rng.randint(0, 3)), rng.choice(["pm1", "pm1", "j3", "gauss32"]),
                        int(_log(rng, 1, 200)), "fm", sweeps=max(1, min(8, 4 * 164 * 164 // (L * (L + 3)))))
    L = 2 * rng.randint(30, 48)
    if rng.random() < 0.4:  # a two-dimensional lattice until nothing improves
        L = 2 * rng.randint(200, 500)
        return _lattice("", "%dx%d" % (L, L), "pm1", 1, "greedy")
    return _lattice("", "%dx%dx%d" % (L, L - 4, L + 2), rng.choice(["pm1", "j3"]), 1, rng.choice(["greedy", "tie"]),
                    hmax=rng.choice([0, 2]), sweeps=int(_log(rng, 50, 500)))


def draw(rng):
    family = rng.choice(["lattice", "lattice", "lattice", "chimera", "chimera", "er", "regular3", "factoring"])
    if family == "lattice":
        c = _draw_lattice(rng)
    elif family == "chimera":
        side = rng.randint(3, 11)
        restarts = int(_log(rng, 32, 300))
        count = int(min(1024, 1024 * 256 * 64 // (side * side * restarts)) * rng.uniform(0.1, 0.7)) + 1
        rule = rng.choice(["greedy", "tie", "fm"])
        c = _chimera("", side, count, restarts, rule, sweeps=rng.randint(10, 50) if rule == "tie" else None,
                     energies=rule != "greedy")
    elif family == "er":
        n_hi = int(_log(rng, 2000, 100000))
        c = {"family": "er", "count": rng.randint(32, 96), "n_lo": 100, "n_hi": n_hi, "restarts": rng.randint(1, 8),
             "rule": rng.choice(["greedy", "greedy", "tie"]), "sweeps": 10000, "converge": True, "energies": True}
        if c["rule"] == "tie":
            c.update(sweeps=20, converge=False)
    elif family == "regular3":
        c = {"family": "regular3", "n": 2 * int(_log(rng, 500, 250000)), "restarts": int(_log(rng, 1, 5)),
             "rule": rng.choice(["greedy", "tie"]), "sweeps": 10000, "converge": True}
        if c["rule"] == "tie":
            c.update(sweeps=30, converge=False)
    else:
        bits = rng.randint(5, 10)
        p = (1 << bits) + 2 * rng.randint(0, (1 << (bits - 1)) - 1) + 1
        q = (1 << bits) + 2 * rng.randint(0, (1 << (bits - 1)) - 1) + 1
        c = {"family": "factoring", "N": p * q, "nx": bits, "ny": bits, "restarts": int(_log(rng, 200, 15000)),
             "rule": "fm", "sweeps": 1000, "converge": True, "energies": True}
    c.pop("name", None)
    return c


def _dims(case):
    return tuple(int(v) for v in case["dims"].split("x"))


def _instances(case, seed):
    fam, R = case["family"], case["restarts"]
    if fam == "lattice":
        dims = _dims(case)
        inst = gen.lattice(dims, periodic=True, seed=seed,
                           h_range=(-case["hmax"], case["hmax"]) if case["hmax"] else None,
                           j_values=(-3, -2, -1, 1, 2, 3) if case["couplings"] == "j3" else (-1, 1), restarts=R,
                           hint=True)
        if case["couplings"] == "gauss32":  # Gaussian couplings to six digits
            J = np.random.default_rng(seed + 1).standard_normal(inst.m)
            inst = inst.replace(J=np.round(J * 1e6).astype(np.int32))
        return [inst]
    if fam == "chimera":
        seeds = np.random.SeedSequence(seed).spawn(case["count"])
        return [gen.chimera(case["side"], case["side"], seed=s, instance_id=i, restarts=R)
                for i, s in enumerate(seeds)]
    if fam == "er":
        u = np.random.default_rng(seed).uniform(math.log(case["n_lo"]), math.log(case["n_hi"]), case["count"])
        u[0] = math.log(case["n_hi"])
        sizes = np.round(np.exp(u)).astype(np.int64)
        return [i.replace(restarts=R) for i in gen.cfg4_uneven_batch(seed=seed, sizes=sizes)]
    if fam == "regular3":
        return [gen.random_regular3(case["n"], seed=seed, restarts=R)]
    return [factoring.factoring_instance(case["N"], case["nx"], case["ny"], restarts=R, instance_id=seed & 0xFFFF)]


def prepare(case, seed):
    insts = _instances(case, seed)
    h = sg.load_dense(insts) if case["family"] == "factoring" else sg.load_instance(insts)
    if case["rule"] == "fm" and max(i.n for i in insts) > 4096:
        h.tune("fm_slots", min(512, case["restarts"]))  # scratch for the searches that run at once
    h.bind()
    return {"h": h, "seed": seed * 7 + 1, "rule": RULES[case["rule"]], "sweeps": case["sweeps"],
            "converge": case["converge"], "energies": case.get("energies", False)}


def run(state):
    """One multi-start search; the best energy and restart of every instance,
    the call's totals, the configuration of the best instance's best restart,
    and where the program looks at the distribution over its starts, every
    replica's energy."""
    h = state["h"]
    stats, E, r = h.solve(state["seed"], rule=state["rule"], max_sweeps=state["sweeps"],
                          until_converged=state["converge"])
    k = int(E.argmin())
    out = {"energies": h.energy()} if state["energies"] else {}
    return {**out, "E": E, "r": r, "spins": h.spins_out(k, int(r[k])), "attempts": stats["attempts"],
            "flips": stats["flips"], "sweeps": stats["sweeps_max"], "unconverged": stats["n_unconverged"]}


def work(case):
    """Bytes: couplings (4-byte partner and coefficient each way, 1 byte per
    axis on a lattice), fields and hyper-couplings read once, every replica's
    spins written once.  Operations: per examined spin a multiply and an add
    per coupling, three operations per hyper-coupling, and four for the field,
    the energy change and the comparison; under the pass-based search the
    updates of the partners' gains and log2 n for the selection."""
    fam, R = case["family"], case["restarts"]
    tau = 0.0
    if fam == "lattice":
        n, deg = math.prod(_dims(case)), 2 * len(_dims(case))
        total, struct = n, n * (deg // 2 + 1) * (4 if case["couplings"] == "gauss32" else 1)
    elif fam == "chimera":
        s = case["side"]
        n, deg, tau = 8 * s * s, 2 * (16 * s * s + 8 * s * (s - 1)) / (8 * s * s), 0.15
        total = n * case["count"]
        struct = total * (4 * deg + 8 * tau + 1)
    elif fam == "er":
        lo, hi = case["n_lo"], case["n_hi"]
        n, deg, tau = (hi - lo) / math.log(hi / lo), 6, 1.5
        total = n * case["count"]
        struct = total * (4 * deg + 8 * tau + 1)
    elif fam == "regular3":
        n, deg = case["n"], 3
        total, struct = n, n * (4 * deg + 1)
    else:
        n = case["nx"] + case["ny"]
        terms = 0.15 * n * n * n  # terms of up to four spins of the squared product
        total, struct, deg = n, 16 * terms, 4 * terms / n
    fm = case["rule"] == "fm"
    sweeps = case["sweeps"] if not case["converge"] else TYPICAL["fm" if fm and fam != "factoring" else fam]
    per_spin = 2 * deg + 3 * tau + 4 + (math.log2(n) if fm else 0)
    return {"bytes": struct + total * R + (8 * R * case.get("count", 1) if case.get("energies") else 0),
            "flops": total * R * sweeps * per_spin}


# ---------------------------------------------------------------------------
# The sweeps on an even lattice in numpy.


def _philox_bit(seed, spin, word1, inst, restart):
    """Bit 0 of word 0 of Philox4x32-10 (Salmon et al., SC'11)."""
    m32 = np.uint64(0xFFFFFFFF)
    c = [spin.astype(np.uint64), np.uint64(word1), np.uint64(inst), np.uint64(restart)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32 & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [p1 >> np.uint64(32) ^ c[1] ^ np.uint64(k0), p1 & m32, p0 >> np.uint64(32) ^ c[3] ^ np.uint64(k1), p0 & m32]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return (c[0] & np.uint64(1)).astype(bool)


def exact(case, seed):
    if case["family"] != "lattice" or case["rule"] == "fm":
        return None
    dims = _dims(case)
    cost = math.prod(dims) * case["restarts"] * (30 if case["converge"] else case["sweeps"])
    if any(L % 2 for L in dims) or cost > 1e8:
        return None
    inst = _instances(case, seed)[0]
    n, d, key = inst.n, len(dims), seed * 7 + 1
    J = inst.J.reshape(dims + (d,)).astype(np.int64)
    h = (inst.h if inst.h is not None else np.zeros(n)).reshape(dims).astype(np.int64)
    site = np.arange(n, dtype=np.int64).reshape(dims)
    colour = np.indices(dims).sum(axis=0) % 2
    best, totals = None, {"attempts": 0, "flips": 0, "sweeps": 0, "unconverged": 0}
    for r in range(case["restarts"]):
        s = np.where(_philox_bit(key, site, 0xFFFFFFFF, inst.instance_id, r), -1, 1).astype(np.int64)
        sweeps, converged = 0, False
        while sweeps < case["sweeps"] and not converged:
            moved = 0
            for c in (0, 1):
                f = h.copy()
                for ax in range(d):
                    f += J[..., ax] * np.roll(s, -1, ax) + np.roll(J[..., ax] * s, 1, ax)
                dE = 2 * s * f
                flip = (dE < 0) & (colour == c)
                if case["rule"] == "tie":
                    tie = (dE == 0) & (colour == c)
                    flip[tie] = _philox_bit(key, site[tie], sweeps, inst.instance_id, r)
                s[flip] *= -1
                moved += int(flip.sum())
            sweeps += 1
            totals["flips"] += moved
            converged = case["converge"] and not moved
        totals["attempts"] += sweeps * n
        totals["sweeps"] = max(totals["sweeps"], sweeps)
        totals["unconverged"] += int(case["converge"] and not converged)
        E = -int((h * s).sum()) - sum(int((J[..., ax] * s * np.roll(s, -1, ax)).sum()) for ax in range(d))
        if best is None or E < best[0]:
            best = (E, r, s.reshape(-1).astype(np.int8))
    return {"E": np.array([best[0]], np.int64), "r": np.array([best[1]], np.int32), "spins": best[2], **totals}
