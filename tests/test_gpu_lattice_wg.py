"""GPU parity of the whole-lattice workgroup mode at the edges of its
variants: fewer sites of a colour than a wavefront, one, two and four sites a
thread in registers (up to 1024, 2048 and 4096 sites of a colour), and more
than that; two and three dimensions, full int8 couplings and fields, both
rules, resumed runs with frozen replicas, and the one-call solve.  Results are
integers and equal the oracle's bit for bit."""
import numpy as np
import pytest

import instances as gen
from parity import compare, log, oracle_run

pytestmark = pytest.mark.gpu

GREEDY, TIE = 0, 1
SCHED_LATTICE = 3

DIMS = [(4, 4), (8, 16), (16, 18), (32, 64), (46, 46), (64, 64), (64, 66), (64, 128), (92, 92), (94, 130), (4, 6, 8), (12, 14, 16),
        (16, 16, 16), (20, 20, 20), (22, 22, 18), (6, 100, 130), (130, 64)]


def _inst(dims, jm, hm):
    return gen.lattice(dims, seed=4, h_range=(-hm, hm) if hm else None, j_values=[v for v in range(-jm, jm + 1) if v],
                       restarts=3, instance_id=9)


@pytest.mark.parametrize("rule,uc,runs", [(GREEDY, True, [1000]), (TIE, False, [5]), (TIE, True, [2, 40])])
@pytest.mark.parametrize("dims", DIMS)
def test_workgroup_mode(gpu, dims, rule, uc, runs):
    import paper_0912_3912_amd as sg
    for jm, hm in ((1, 0), (127, 127)):
        inst = _inst(dims, jm, hm)
        log(f"lattice workgroup case: {dims} J<={jm} h<={hm} rule={rule} uc={uc} runs={runs}")
        h = sg.load_instance([inst], lattice_dims=[dims]).bind()
        h.init_spins(7)
        for ms in runs:
            s = h.run_sweeps(seed=7, rule=rule, max_sweeps=ms, until_converged=uc, schedule=SCHED_LATTICE)
        assert s["schedule_used"] == SCHED_LATTICE
        ref = oracle_run(inst, 7, rule, runs[0], uc, runs)
        compare(h, [inst], [ref])
        if len(runs) == 1:
            _, E, r = h.solve(7, rule=rule, max_sweeps=runs[0], until_converged=uc)
            assert E[0] == ref.energy.min() and r[0] == int(np.argmin(ref.energy))
            compare(h, [inst], [ref])
        h.free()


@pytest.mark.parametrize("rule", [GREEDY, TIE])
@pytest.mark.parametrize("dims", [(24, 20, 16), (40, 72)])
def test_byte_tiles(gpu, dims, rule):
    """The tile kernel's byte form at full int8 couplings and fields; odd
    numbers of phases between exchanges."""
    import paper_0912_3912_amd as sg
    for jm, hm in ((1, 2), (127, 127)):
        inst = _inst(dims, jm, hm)
        log(f"byte tiles case: {dims} J<={jm} h<={hm} rule={rule}")
        h = sg.load_instance([inst], lattice_dims=[dims])
        for k, v in {"lattice_wg_max_n": 0, "lattice_msc": 0, "lattice_k": 3}.items():
            h.tune(k, v)
        h.bind()
        h.init_spins(7)
        for ms in (7, 2):
            s = h.run_sweeps(seed=7, rule=rule, max_sweeps=ms, until_converged=False, schedule=SCHED_LATTICE)
        assert s["schedule_used"] == SCHED_LATTICE
        compare(h, [inst], [oracle_run(inst, 7, rule, 7, False, [7, 2])])
        h.free()
