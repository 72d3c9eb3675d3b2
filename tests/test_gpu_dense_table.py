"""GPU parity of the dense pass-based search by energy tables (at most 22
spins): sizes around the tile of the transform, several instances to a round
and several rounds, larger instances among them, resumed and fixed pass
counts.  Results are integers and equal the oracle's bit for bit."""
import pytest

import instances as gen
import oracle
from parity import compare, log

pytestmark = pytest.mark.gpu

FM = 2


def _check(ds, seed, runs, uc, tables):
    import paper_0912_3912_amd as sg
    log(f"dense table case: {[(d.n, d.masks.shape[0], d.restarts) for d in ds][:4]} runs={runs} uc={uc}")
    h = sg.load_dense(ds)
    if tables:
        assert h.workspace_bytes() > (8 << max(d.n for d in ds if d.n <= 22))
    h.bind()
    h.init_spins(seed)
    for r in runs:
        h.run_sweeps(seed=seed, rule=FM, max_sweeps=r, until_converged=uc)
    states = []
    for d in ds:
        st = None
        for r in runs:
            st, _ = oracle.dense_fm(d, seed=seed, max_passes=r, until_converged=uc, state=st)
        states.append(st)
    compare(h, ds, states)
    h.free()


@pytest.mark.parametrize("n,nterms", [(10, 300), (11, 400), (12, 400), (17, 500), (22, 600), (23, 600)])
def test_sizes(gpu, n, nterms):
    d = gen.random_dense(n, nterms, max_order=4, coef_range=(-3, 3), seed=n, restarts=100, instance_id=n)
    _check([d], n, [1000], True, n <= 22)
    _check([d], n, [1, 2], False, n <= 22)


def test_rounds_and_larger_instances(gpu):
    """21-spin tables come two to a round; a 30-spin instance runs between."""
    ds = [gen.random_dense(n, 300, max_order=3, coef_range=(-9, 9), seed=k, restarts=70 + k, instance_id=k)
          for k, n in enumerate((21, 9, 21, 30, 15, 21, 21, 21))]
    _check(ds, 5, [1, 0, 1000], True, True)
