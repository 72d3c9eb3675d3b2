"""GPU parity of the sweeps of one instance in one launch, a team of
workgroups per replica (SG_SCHED_AUTO on few replicas of an irregular graph):
one workgroup, forced and chosen team sizes, one colour and many, colours
smaller than the team, hyper-couplings, rows longer than what is loaded at
once, both rules, resumed runs with frozen replicas.  Results are integers and
equal the oracle's bit for bit."""
import numpy as np
import pytest

import instances as gen
import oracle
from parity import compare, log

pytestmark = pytest.mark.gpu

GREEDY, TIE = 0, 1


def _lone():
    rng = np.random.default_rng(3)
    e = np.zeros(0, np.int32)
    return gen.Instance(700, e, e, e, rng.integers(-3, 4, 700), restarts=3, instance_id=4, name="fields700")


CASES = {
    "one": lambda: gen.chain(1, seed=1).replace(h=np.array([2], np.int32)),
    "fields": _lone,
    "regular": lambda: gen.random_regular3(6002, seed=2, instance_id=3, restarts=2),
    "triples": lambda: gen.erdos_renyi_triples(5000, seed=4, restarts=3),
    "dense": lambda: gen.random_small(400, seed=5, p_edge=0.08, n_triples=900, j_range=(-100, 100), h_range=(-9, 9),
                                      k_range=(-50, 50)).replace(restarts=2),
}


@pytest.mark.parametrize("rule,uc,runs", [(GREEDY, True, [1000]), (TIE, False, [7]), (TIE, True, [2, 3, 9]),
                                          (GREEDY, False, [1, 3])])
@pytest.mark.parametrize("name", list(CASES))
def test_team(gpu, name, rule, uc, runs):
    import paper_0912_3912_amd as sg
    inst = CASES[name]()
    st = None
    for r in runs:
        st, _ = oracle.run(inst, seed=3, rule=rule, max_sweeps=r, until_converged=uc, state=st, threads=8)
    for wgs in (1, 2, 7):
        log(f"team case: {name} n={inst.n} restarts={inst.restarts} rule={rule} uc={uc} runs={runs} wgs={wgs}")
        h = sg.load_instance([inst])
        h.tune("team_wgs", wgs)
        h.bind()
        h.init_spins(3)
        for r in runs:
            s = h.run_sweeps(seed=3, rule=rule, max_sweeps=r, until_converged=uc)
        assert s["schedule_used"] == sg.SCHED_PHASE and 1 <= h.query("last_team") <= wgs
        compare(h, [inst], [st])
        h.free()


@pytest.mark.parametrize("rule,uc", [(GREEDY, True), (TIE, False)])
def test_chosen_teams(gpu, rule, uc):
    """Sizes where SG_SCHED_AUTO splits a replica by itself, a small instance
    beside it, and the per-phase launches asked for."""
    import paper_0912_3912_amd as sg
    insts = [gen.random_regular3(70000, seed=6, instance_id=1, restarts=2),
             gen.erdos_renyi_triples(900, seed=7, instance_id=2, restarts=2)]
    log(f"chosen teams: rule={rule} uc={uc}")
    ref = [oracle.run(i, seed=5, rule=rule, max_sweeps=12, until_converged=uc, threads=8)[0] for i in insts]
    for wgs, want in ((0, (1,)), (-1, (0,))):
        h = sg.load_instance(insts)
        h.tune("team_wgs", wgs)
        h.bind()
        h.init_spins(5)
        h.run_sweeps(seed=5, rule=rule, max_sweeps=12, until_converged=uc)
        assert h.query("last_team") in want
        compare(h, insts, ref)
        h.free()
    h = sg.load_instance(insts[:1]).bind()
    h.init_spins(5)
    h.run_sweeps(seed=5, rule=rule, max_sweeps=12, until_converged=uc)
    assert h.query("last_team") >= 2
    compare(h, insts[:1], ref[:1])
    assert np.array_equal(h.spins_out(0, 1), ref[0].spins[1])  # beyond the pinned buffer
    h.free()


def _wide_rows():
    """Rows of about 16 couplings (more than are loaded ahead), a few spins in
    many triples, fields."""
    rng = np.random.default_rng(8)
    n = 26001
    e = rng.integers(0, n, (8 * n, 2))
    e = np.unique(np.sort(e[e[:, 0] != e[:, 1]], axis=1), axis=0)
    t = np.unique(np.sort(np.stack([rng.integers(0, 300, 900), rng.integers(300, 600, 900), rng.integers(600, 900, 900)], 1),
                          axis=1), axis=0)
    return gen.Instance(n, e[:, 0], e[:, 1], rng.integers(1, 128, len(e)) * rng.choice([-1, 1], len(e)),
                        rng.integers(-127, 128, n), tri=t, K=rng.integers(1, 100, len(t)), restarts=2, instance_id=6)


@pytest.mark.parametrize("rule,uc,runs", [(GREEDY, True, [1000]), (TIE, False, [3, 4])])
@pytest.mark.parametrize("name", ["triples", "wide rows"])
def test_split_replicas(gpu, name, rule, uc, runs):
    """Teams whose replicas hold the spins as bits, with hyper-couplings."""
    import paper_0912_3912_amd as sg
    inst = gen.erdos_renyi_triples(40003, seed=4, restarts=2) if name == "triples" else _wide_rows()
    log(f"split replicas: {name} rule={rule} uc={uc} runs={runs}")
    st = None
    for r in runs:
        st, _ = oracle.run(inst, seed=3, rule=rule, max_sweeps=r, until_converged=uc, state=st, threads=8)
    for wgs in (0, 2, 33):
        h = sg.load_instance([inst])
        h.tune("team_wgs", wgs)
        h.bind()
        h.init_spins(3)
        for r in runs:
            h.run_sweeps(seed=3, rule=rule, max_sweeps=r, until_converged=uc)
        log(f"  team of {h.query('last_team')}")
        assert h.query("last_team") >= (2 if name == "triples" else 1)
        compare(h, [inst], [st])
        h.free()


@pytest.mark.parametrize("first", ["run", "capped", "fixed", "phase", "energy", "best"])
def test_start_energies_left_out(gpu, first):
    """The start energies that the team kernel makes unnecessary, read or needed
    in every other way first: a run that converges, one that the sweep cap ends,
    a fixed number of sweeps, per-phase launches, and the readers."""
    import paper_0912_3912_amd as sg
    inst = gen.erdos_renyi_triples(6001, seed=9, restarts=2)
    log(f"start energies left out: {first}")
    h = sg.load_instance([inst]).bind()
    h.init_spins(3)
    assert h.query("energy_pending") == 1
    n, uc = {"run": (1000, True), "capped": (2, True), "fixed": (3, False)}.get(first, (1000, True))
    if first == "energy":
        assert np.array_equal(h.energy(), h.energy(recompute=True))
    elif first == "best":
        E, _ = h.best()
        assert E[0] == h.energy(recompute=True).min()
    h.run_sweeps(seed=3, rule=GREEDY, max_sweeps=n, until_converged=uc,
                 schedule=sg.SCHED_PHASE if first == "phase" else sg.SCHED_AUTO)
    assert h.query("energy_pending") == 0
    compare(h, [inst], [oracle.run(inst, seed=3, rule=GREEDY, max_sweeps=n, until_converged=uc, threads=8)[0]])
    h.free()
