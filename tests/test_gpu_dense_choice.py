"""When the pass-based search on dense instances goes by a table of energies:
in calls of as many passes as pay for it, in rounds, beside instances too large
for one; equal to the oracle either way."""
import pytest

import instances as gen
import oracle
from parity import compare, log

pytestmark = pytest.mark.gpu

FM = 2


def _dense(n, terms, count, restarts):
    return [gen.random_dense(n, terms, max_order=3, coef_range=(-9, 9), seed=k, restarts=restarts, instance_id=k)
            for k in range(count)]


@pytest.mark.parametrize("make,runs,tables", [
    (lambda: _dense(3, 7, 1, 70), [1000], [0]),
    (lambda: _dense(22, 44, 1, 64), [1, 1000], [0, 1]),
    (lambda: _dense(12, 24, 500, 10), [1, 3], [0, 500]),
    (lambda: _dense(16, 300, 2, 100), [1, 1, 1000], [2, 2, 2]),
    (lambda: _dense(21, 200, 6, 20) + _dense(30, 60, 1, 20), [4], [6]),
])
def test_choice(gpu, make, runs, tables):
    import paper_0912_3912_amd as sg
    ds = make()
    log(f"dense choice: {ds[0].n} spins, {ds[0].masks.shape[0]} terms, {len(ds)} instances, runs={runs}")
    h = sg.load_dense(ds).bind()
    h.init_spins(5)
    states = [None] * len(ds)
    for r, t in zip(runs, tables):
        uc = r > 100
        h.run_sweeps(seed=5, rule=FM, max_sweeps=r, until_converged=uc)
        assert h.query("last_dense_tables") == t
        states = [oracle.dense_fm(d, seed=5, max_passes=r, until_converged=uc, state=st)[0] for d, st in zip(ds, states)]
    compare(h, ds, states)
    h.run_sweeps(seed=5, rule=0, max_sweeps=1, until_converged=False)
    assert h.query("last_dense_tables") == 0
    h.free()
