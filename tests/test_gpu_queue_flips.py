"""The queue schedule counts a replica's flips in 64 bits: 150000 free spins
flip more than 2^31 times in 29500 sweeps of tie moves, and the call's total and
the replica's counter equal those of the per-phase launches."""
import numpy as np
import pytest

import instances as gen
from parity import log

pytestmark = pytest.mark.gpu


def test_flips_beyond_32_bits(gpu):
    import paper_0912_3912_amd as sg
    e = np.zeros(0, np.int32)
    inst = gen.Instance(150000, e, e, e, None, restarts=1, instance_id=4)
    got = []
    for schedule in (sg.SCHED_QUEUE, sg.SCHED_PHASE):
        log(f"flips beyond 32 bits: schedule {schedule}")
        h = sg.load_instance([inst]).bind()
        h.init_spins(3)
        s = h.run_sweeps(seed=3, rule=sg.GREEDY_TIE, max_sweeps=29500, until_converged=False, schedule=schedule)
        got.append((s["flips"], int(h.counters()[1][0]), h.spins_out(0, 0).tobytes()))
        h.free()
    assert got[0] == got[1]
    assert got[0][0] == got[0][1] > 2 ** 31
