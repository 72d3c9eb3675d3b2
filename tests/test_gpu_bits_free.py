"""Bit-sliced block kernel on rows without couplings: fields alone (up to the
largest coefficient, also zero), hyper-couplings without couplings, and such
rows beside others, against the oracle."""
import numpy as np
import pytest

import instances as gen
import oracle
from parity import compare, log

pytestmark = pytest.mark.gpu

GREEDY, TIE = 0, 1


def _inst(name, k):
    e = np.zeros(0, np.int32)
    r = np.random.default_rng(k)
    if name == "fields":
        return gen.Instance(130, e, e, e, r.integers(-15, 16, 130))
    if name == "triples":  # 70 spins of 200 in one triple each, the others free
        i = gen.random_small(200, seed=k, p_edge=0.0, n_triples=60, h_range=(-2, 2))
        assert i.m == 0
        return i
    return gen.erdos_renyi_triples(300, seed=k, mean_degree=1, triples_per_spin=0.1)


@pytest.mark.parametrize("restarts", [33, 256])
@pytest.mark.parametrize("rule,uc", [(GREEDY, True), (GREEDY, False), (TIE, False)])
@pytest.mark.parametrize("name", ["fields", "triples", "mixed"])
def test_free_rows(gpu, name, rule, uc, restarts):
    import paper_0912_3912_amd as sg
    insts = [_inst(name, k).replace(instance_id=k, restarts=restarts) for k in range(3)]
    log(f"rows without couplings: {name} rule={rule} uc={uc} restarts={restarts}")
    h = sg.load_instance(insts).tune("bits_groups", 8).bind()
    h.init_spins(3)
    h.run_sweeps(seed=3, rule=rule, max_sweeps=7, until_converged=uc)
    assert h.query("last_bits") == 1
    compare(h, insts, [oracle.run(i, seed=3, rule=rule, max_sweeps=7, until_converged=uc, threads=8)[0] for i in insts])
    h.free()
