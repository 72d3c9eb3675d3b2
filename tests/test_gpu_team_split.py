"""GPU parity of replicas split over a given number of workgroups (team_wgs),
where that many really run: one colour and many, colours with fewer slices than
the team has members, rows of few, up to twelve and more couplings, with and
without hyper-couplings, a lattice under the stopping rule with tie moves,
replicas frozen by an earlier run under the other rule.  Results are integers
and equal the oracle's bit for bit."""
import numpy as np
import pytest

import instances as gen
import oracle
from parity import compare, log

pytestmark = pytest.mark.gpu

GREEDY, TIE = 0, 1


def _fields():
    e = np.zeros(0, np.int32)
    return gen.Instance(700, e, e, e, np.random.default_rng(3).integers(-3, 4, 700), restarts=3, instance_id=4)


def _wheel():
    """One spin coupled to 1500 others, which are not coupled: a colour of one
    slice beside one of 24."""
    j = np.arange(1, 1501, dtype=np.int32)
    rng = np.random.default_rng(5)
    return gen.Instance(1501, np.zeros(1500, np.int32), j, rng.choice([-1, 1], 1500).astype(np.int32),
                        rng.integers(-1, 2, 1501), restarts=2, instance_id=5)


CASES = {
    "fields": _fields,
    "wheel": _wheel,
    "regular": lambda: gen.random_regular3(6002, seed=2, instance_id=3, restarts=2),
    "rows of 8": lambda: gen.erdos_renyi_triples(9001, seed=3, mean_degree=3, triples_per_spin=0.0, restarts=2),
    "rows of 20": lambda: gen.erdos_renyi_triples(12003, seed=4, mean_degree=14, triples_per_spin=0.0, restarts=2),
    "triples": lambda: gen.erdos_renyi_triples(5000, seed=4, restarts=3),
    "many triples": lambda: gen.erdos_renyi_triples(4000, seed=6, mean_degree=4, triples_per_spin=3.0, restarts=2),
    "lattice": lambda: gen.lattice((30, 32, 34), seed=6, h_range=(-2, 2), j_values=(-3, -1, 2), restarts=2, hint=True),
}


@pytest.mark.parametrize("rule,uc,runs", [([GREEDY], True, [1000]), ([TIE], False, [7]), ([TIE], True, [2, 3, 9]),
                                          ([GREEDY, TIE], True, [6, 5])])
@pytest.mark.parametrize("name", list(CASES))
def test_split(gpu, name, rule, uc, runs):
    import paper_0912_3912_amd as sg
    inst = CASES[name]()
    if name == "lattice" and rule != [TIE]:
        pytest.skip("partly on the lattice kernels")
    rules = rule * (len(runs) // len(rule))
    st = None
    for r, rl in zip(runs, rules):
        st, _ = oracle.run(inst, seed=3, rule=rl, max_sweeps=r, until_converged=uc, state=st, threads=8)
    for wgs in (2, 7, 40):
        h = sg.load_instance([inst])
        h.tune("team_wgs", wgs)
        h.tune("lattice_wg_max_n", 0)
        h.bind()
        slices = (int(np.bincount(h.info(0)["colour"]).max()) + 63) // 64
        log(f"split: {name} n={inst.n} rule={rule} uc={uc} runs={runs} wgs={wgs} slices={slices}")
        h.init_spins(3)
        for r, rl in zip(runs, rules):
            h.run_sweeps(seed=3, rule=rl, max_sweeps=r, until_converged=uc)
            if name != "lattice" or uc:
                assert h.query("last_team") == min(wgs, slices) > 1
        compare(h, [inst], [st])
        h.free()


def test_no_room(gpu):
    """Where the workspace has no room for the exchange, a large instance is not
    forced on one workgroup per replica."""
    import paper_0912_3912_amd as sg
    inst = gen.random_regular3(900000, seed=2, restarts=42)
    for wgs, team in ((33, 0), (0, 0), (1, 1)):
        h = sg.load_instance([inst])
        h.tune("team_wgs", wgs)
        assert h.workspace_bytes() <= 64 << 20
        h.bind()
        h.init_spins(3)
        h.run_sweeps(seed=3, rule=GREEDY, max_sweeps=4, until_converged=False)
        assert h.query("last_team") == team
        E = h.energy()
        assert np.array_equal(E, h.energy(recompute=True))
        h.free()
