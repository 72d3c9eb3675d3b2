"""Calls of few phases on instances that are otherwise split over several
workgroups: SG_SCHED_AUTO keeps them on per-phase launches, one sweep at a time
or under a low cap, with start energies left out or not, and a longer call that
follows goes to the team; equal to the oracle throughout."""
import pytest

import instances as gen
import oracle
from parity import compare, log

pytestmark = pytest.mark.gpu

GREEDY, TIE = 0, 1


@pytest.mark.parametrize("rule,uc,runs", [(GREEDY, False, [1, 1, 8]), (TIE, False, [2, 9]), (GREEDY, True, [1, 2, 100]),
                                          (TIE, True, [1, 12])])
def test_short_calls(gpu, rule, uc, runs):
    import paper_0912_3912_amd as sg
    inst = gen.random_regular3(70000, seed=6, instance_id=1, restarts=2)
    st = None
    h = sg.load_instance([inst]).bind()
    h.init_spins(3)
    for r in runs:
        log(f"short calls: rule={rule} uc={uc} sweeps={r}")
        st, _ = oracle.run(inst, seed=3, rule=rule, max_sweeps=r, until_converged=uc, state=st, threads=8)
        h.run_sweeps(seed=3, rule=rule, max_sweeps=r, until_converged=uc)
        assert (h.query("last_team") > 1) == (r >= 8) and h.query("last_team") != 1
        compare(h, [inst], [st])
    h.free()


@pytest.mark.parametrize("rule,runs", [(GREEDY, [(6, False), (30, True)]), (TIE, [(3, False), (12, True)])])
def test_two_colours(gpu, rule, runs):
    """A chain: two phases a sweep, and rows that cost a launch little."""
    import paper_0912_3912_amd as sg
    inst = gen.chain(40000, seed=1, periodic=True).replace(restarts=3)
    st = None
    h = sg.load_instance([inst]).bind()
    h.init_spins(5)
    for r, team in runs:
        log(f"short calls on a chain: rule={rule} sweeps={r}")
        st, _ = oracle.run(inst, seed=5, rule=rule, max_sweeps=r, until_converged=False, state=st, threads=8)
        h.run_sweeps(seed=5, rule=rule, max_sweeps=r, until_converged=False)
        assert (h.query("last_team") > 1) == team
        compare(h, [inst], [st])
    h.free()


def test_given_team(gpu):
    """A given number of workgroups is used in calls of any length."""
    import paper_0912_3912_amd as sg
    inst = gen.random_regular3(70000, seed=6, instance_id=1)
    h = sg.load_instance([inst])
    h.tune("team_wgs", 5)
    h.bind()
    h.init_spins(3)
    h.run_sweeps(seed=3, rule=TIE, max_sweeps=1, until_converged=False)
    assert h.query("last_team") == 5
    h.free()


@pytest.mark.parametrize("rule", [GREEDY, TIE])
def test_few_sweeps(gpu, rule):
    """One or two sweeps until converged on one workgroup per replica: from random
    starts and from where nothing moves."""
    import paper_0912_3912_amd as sg
    inst = gen.chain(289, seed=1, periodic=True).replace(restarts=5)
    log(f"few sweeps until converged: rule={rule}")
    h = sg.load_instance([inst]).bind()
    h.init_spins(5)
    st = None
    for r in (1, 2, 40, 1, 2):
        st, _ = oracle.run(inst, seed=5, rule=rule, max_sweeps=r, until_converged=True, state=st, threads=8)
        h.run_sweeps(seed=5, rule=rule, max_sweeps=r, until_converged=True)
        assert h.query("last_team") == 1 and h.query("energy_pending") == 0
        compare(h, [inst], [st])
    h.free()


@pytest.mark.parametrize("rule,uc", [(GREEDY, True), (TIE, False)])
def test_no_couplings(gpu, rule, uc):
    import numpy as np
    import paper_0912_3912_amd as sg
    e = np.zeros(0, np.int32)
    inst = gen.Instance(70001, e, e, e, np.random.default_rng(1).integers(-1, 2, 70001))
    log(f"no couplings: rule={rule} uc={uc}")
    st, _ = oracle.run(inst, seed=5, rule=rule, max_sweeps=25, until_converged=uc, threads=8)
    h = sg.load_instance([inst]).bind()
    h.init_spins(5)
    h.run_sweeps(seed=5, rule=rule, max_sweeps=25, until_converged=uc)
    assert h.query("last_team") == 0
    compare(h, [inst], [st])
    h.free()
