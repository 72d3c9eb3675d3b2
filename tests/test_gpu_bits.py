"""GPU parity of the bit-sliced block kernel under both sweep rules: rows of
every width around its column sums (3, 4, 6 couplings and further ones three
at a time, hyper-couplings), per-spin sums up to the limit of 255, instances
full of ties (queues that fill within a slice), resumed runs.  Results are
integers and equal the oracle's bit for bit."""
import numpy as np
import pytest

import instances as gen
import oracle
from parity import compare, log

pytestmark = pytest.mark.gpu

GREEDY, TIE, SCHED_BLOCK = 0, 1, 4


def _ring(n, reach, seed, j_range, **kw):
    """n spins on a ring, each coupled to the next `reach` ones: rows of 2 reach couplings."""
    rng = np.random.default_rng(seed)
    i = np.repeat(np.arange(n), reach)
    j = (i + np.tile(np.arange(1, reach + 1), n)) % n
    J = rng.integers(j_range[0], j_range[1] + 1, i.size)
    return gen.Instance(n, i, j, J, rng.integers(-2, 3, n), name=f"ring{n}x{reach}", **kw)


def _star():
    """A centre of 17 couplings of 15 (sum 255), leaves with odd and even sums."""
    h = np.arange(18) % 3 - 1
    h[0] = 0
    return gen.Instance(18, np.zeros(17, int), np.arange(1, 18), np.where(np.arange(17) % 2, 15, -15), h,
                        restarts=100, instance_id=9, name="star")


CASES = {
    "chain": lambda: gen.chain(300, seed=1, j_range=(-1, 1)).replace(restarts=90),
    "deg4": lambda: _ring(130, 2, 2, (-1, 1), restarts=100),
    "deg6": lambda: _ring(257, 3, 3, (-15, 15), restarts=64),
    "deg8": lambda: _ring(100, 4, 4, (-3, 3), restarts=70),
    "deg14": lambda: _ring(200, 7, 5, (-15, 15), restarts=40),
    "star": _star,
    "ties": lambda: gen.lattice((36, 38), seed=2, restarts=64),  # 1368 spins, +-1 couplings, no field
    "triples": lambda: gen.random_small(200, seed=7, p_edge=0.02, n_triples=300, j_range=(-2, 2), h_range=(-1, 1),
                                        k_range=(-2, 2)).replace(restarts=96),
}


@pytest.mark.parametrize("rule,uc,runs", [(GREEDY, True, [1000]), (TIE, False, [9]), (TIE, True, [2, 1, 12]),
                                          (GREEDY, False, [1, 4])])
@pytest.mark.parametrize("name", list(CASES))
def test_bit_sliced_block(gpu, name, rule, uc, runs):
    import paper_0912_3912_amd as sg
    inst = CASES[name]()
    log(f"bits case: {name} n={inst.n} restarts={inst.restarts} rule={rule} uc={uc} runs={runs}")
    st = None
    for r in runs:
        st, _ = oracle.run(inst, seed=3, rule=rule, max_sweeps=r, until_converged=uc, state=st, threads=8)
    for ng in (2, 8):
        h = sg.load_instance([inst])
        h.tune("bits_groups", ng)
        h.bind()
        h.init_spins(3)
        for r in runs:
            h.run_sweeps(seed=3, rule=rule, max_sweeps=r, until_converged=uc, schedule=SCHED_BLOCK)
        assert h.query("last_bits") == 1
        compare(h, [inst], [st])
        h.free()
