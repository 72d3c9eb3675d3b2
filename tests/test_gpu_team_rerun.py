"""GPU parity of runs whose teams of workgroups give up: a limit of one look
makes every wait between workgroups that is not over at once end the team, a
limit of none stands for a launch that the runtime refuses.  The replicas
concerned run from where they stood without teams, with the results of a run
that had no such trouble: spins, energies (left out at the
start or read before), counters, call totals, and replicas frozen earlier."""
import copy

import pytest

import instances as gen
import oracle
from parity import compare, expected_stats, log

pytestmark = pytest.mark.gpu

GREEDY, TIE = 0, 1


def _ref(insts, rule, uc, runs):
    """States after the first runs and after the last."""
    before, after = [], []
    for i in insts:
        st = None
        for r in runs[:-1]:
            st, _ = oracle.run(i, seed=3, rule=rule, max_sweeps=r, until_converged=uc, state=st, threads=8)
        before.append(copy.deepcopy(st))
        after.append(oracle.run(i, seed=3, rule=rule, max_sweeps=runs[-1], until_converged=uc, state=st, threads=8)[0])
    return before, after


def _check(insts, rule, uc, runs, pending, schedule, polls):
    before, ref = _ref(insts, rule, uc, runs)
    import paper_0912_3912_amd as sg
    h = sg.load_instance(insts)
    h.tune("lattice_wg_max_n", 0)
    h.bind()
    h.init_spins(3)
    if not pending:
        h.energy()
    for r in runs[:-1]:
        h.run_sweeps(seed=3, rule=rule, max_sweeps=r, until_converged=uc, schedule=schedule)
    assert h.query("last_team_reruns") == 0
    h.tune("team_polls", polls)
    s = h.run_sweeps(seed=3, rule=rule, max_sweeps=runs[-1], until_converged=uc, schedule=schedule)
    assert (h.query("last_team_reruns") > 0) == (polls > 0)
    assert polls > 0 or (h.query("last_team") <= 1 and h.query("last_queue_teams") == 0)
    compare(h, insts, ref)
    assert (s["attempts"], s["flips"]) == expected_stats(insts, before, ref)
    assert s["n_unconverged"] == (sum(int((st.converged == 0).sum()) for st in ref) if uc else 0)
    # the flags of that call do not outlive it
    h.tune("team_polls", 1 << 22)
    for _ in range(2):
        h.init_spins(3)
        h.run_sweeps(seed=3, rule=rule, max_sweeps=2, until_converged=False, schedule=schedule)
        assert h.query("last_team_reruns") == 0
    h.free()


CASES = [(GREEDY, True, [1000], True), (GREEDY, True, [1000], False), (GREEDY, True, [4], True),
         (TIE, False, [12], False), (TIE, True, [2, 3, 9], False)]


@pytest.mark.parametrize("polls", [1, 0])
@pytest.mark.parametrize("name,rule,uc,runs,pending", [("regular", *c) for c in CASES] + [("lattice", *CASES[-1])])
def test_team(gpu, name, rule, uc, runs, pending, polls):
    """A replica split by itself beside one that a workgroup takes; a lattice
    that only the stopping rule under TIE gives to the team kernel."""
    import paper_0912_3912_amd as sg
    if name == "lattice":
        insts = [gen.lattice((40, 40, 42), seed=6, h_range=(-2, 2), j_values=(-3, -1, 2), restarts=2, hint=True)]
    else:
        insts = [gen.random_regular3(70002, seed=6, instance_id=1, restarts=2),
                 gen.erdos_renyi_triples(900, seed=7, instance_id=2, restarts=2)]
    log(f"team rerun: {name} rule={rule} uc={uc} runs={runs} pending={pending} polls={polls}")
    _check(insts, rule, uc, runs, pending, sg.SCHED_AUTO, polls)


@pytest.mark.parametrize("polls", [1, 0])
@pytest.mark.parametrize("rule,uc,runs,pending", CASES)
def test_queue(gpu, rule, uc, runs, pending, polls):
    import paper_0912_3912_amd as sg
    insts = [gen.erdos_renyi_triples(60011, seed=1, restarts=3, instance_id=1),
             gen.random_regular3(90002, seed=2, restarts=2, instance_id=2)]
    insts += [gen.erdos_renyi_triples(700 + 37 * i, seed=10 + i, restarts=8, instance_id=10 + i) for i in range(12)]
    log(f"queue rerun: rule={rule} uc={uc} runs={runs} pending={pending} polls={polls}")
    _check(insts, rule, uc, runs, pending, sg.SCHED_QUEUE, polls)


def test_limits(gpu):
    import paper_0912_3912_amd as sg
    h = sg.load_instance([gen.random_regular3(100, seed=1)])
    for v in (-1, (1 << 30) + 1):
        with pytest.raises(sg.SGError):
            h.tune("team_polls", v)
    assert h.query("team_polls") == 1 << 22
    h.free()
