"""GPU parity of the queue schedule's whole-workgroup items: rows of no, few
and many couplings and hyper-couplings (more than are loaded ahead), more
colours than the kernel's tables hold, sizes that leave the last slice and the
last sixteen spins part filled, both rules, resumed runs with frozen replicas.
Results are integers and equal the oracle's bit for bit."""
import numpy as np
import pytest

import instances as gen
import oracle
from parity import compare, log

pytestmark = pytest.mark.gpu

GREEDY, TIE = 0, 1


def _fields():
    e = np.zeros(0, np.int32)
    return gen.Instance(1037, e, e, e, np.random.default_rng(3).integers(-3, 4, 1037), restarts=3, instance_id=4)


def _clique():
    """80 spins coupled in all pairs among 333: at least 80 colours."""
    rng = np.random.default_rng(4)
    i, j = np.triu_indices(80, 1)
    return gen.Instance(333, i.astype(np.int32), j.astype(np.int32), rng.integers(1, 128, i.size) * rng.choice([-1, 1], i.size),
                        rng.integers(-127, 128, 333), restarts=3, instance_id=5)


CASES = {
    "one": lambda: gen.chain(1, seed=1).replace(h=np.array([2], np.int32)),
    "fields": _fields,
    "regular": lambda: gen.random_regular3(6002, seed=2, instance_id=3, restarts=2),
    "triples": lambda: gen.erdos_renyi_triples(20011, seed=4, restarts=2),
    "dense": lambda: gen.random_small(401, seed=5, p_edge=0.08, n_triples=900, j_range=(-100, 100), h_range=(-9, 9),
                                      k_range=(-50, 50)).replace(restarts=2),
    "clique": _clique,
}


@pytest.mark.parametrize("rule,uc,runs", [(GREEDY, True, [1000]), (TIE, False, [7]), (TIE, True, [2, 3, 9])])
def test_queue_items(gpu, rule, uc, runs):
    """All cases in one launch, whole-workgroup items only and with the small
    ones on wavefronts."""
    import paper_0912_3912_amd as sg
    insts = [make() for make in CASES.values()]
    ref = []
    for i in insts:
        st = None
        for r in runs:
            st, _ = oracle.run(i, seed=3, rule=rule, max_sweeps=r, until_converged=uc, state=st, threads=8)
        ref.append(st)
    for small in (0, 512):
        log(f"queue items: rule={rule} uc={uc} runs={runs} queue_wave_max_n={small}")
        h = sg.load_instance(insts)
        h.tune("queue_wave_max_n", small)
        h.bind()
        h.init_spins(3)
        for r in runs:
            s = h.run_sweeps(seed=3, rule=rule, max_sweeps=r, until_converged=uc, schedule=sg.SCHED_QUEUE)
        assert s["schedule_used"] == sg.SCHED_QUEUE
        compare(h, insts, ref)
        h.free()


@pytest.mark.parametrize("rule,uc,runs", [(GREEDY, True, [1000]), (TIE, False, [5]), (TIE, True, [2, 4])])
def test_queue_teams(gpu, rule, uc, runs):
    """Batches whose largest items outlast the rest run on teams of workgroups:
    with and without hyper-couplings, start energies pending or read, replicas
    frozen by an earlier run; and the same batch without teams."""
    import paper_0912_3912_amd as sg
    insts = [gen.erdos_renyi_triples(60011, seed=1, restarts=3, instance_id=1),
             gen.random_regular3(90002, seed=2, restarts=2, instance_id=2)]
    insts += [gen.erdos_renyi_triples(700 + 37 * i, seed=10 + i, restarts=8, instance_id=10 + i) for i in range(12)]
    ref = []
    for i in insts:
        st = None
        for r in runs:
            st, _ = oracle.run(i, seed=3, rule=rule, max_sweeps=r, until_converged=uc, state=st, threads=8)
        ref.append(st)
    for wgs, pending in ((0, False), (0, True), (-1, True)):
        log(f"queue teams: rule={rule} uc={uc} runs={runs} team_wgs={wgs} pending={pending}")
        h = sg.load_instance(insts)
        h.tune("team_wgs", wgs)
        h.bind()
        h.init_spins(3)
        if not pending:
            h.energy()
        for r in runs:
            h.run_sweeps(seed=3, rule=rule, max_sweeps=r, until_converged=uc, schedule=sg.SCHED_QUEUE)
            assert (h.query("last_queue_teams") > 0) == (wgs == 0)
        compare(h, insts, ref)
        h.free()
