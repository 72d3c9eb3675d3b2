"""The pass kernels for instances of more than 4096 spins (SG_RULE_FM with
fm_slots): half-gains in LDS as bytes or int32, or in device memory, at the
edges of their leaves-per-lane steps and of their ranges.  Coefficients scaled
by a common factor order every move alike, so an instance in bytes, the same
one scaled (int32, or beyond LDS) and the oracle give one trajectory; results
are integers and equal bit for bit."""
import numpy as np
import pytest

import instances as gen
import oracle
from parity import compare, log

pytestmark = pytest.mark.gpu

FM = 2


def _run(inst, seed, passes, slots=2):
    import paper_0912_3912_amd as sg
    log(f"fm mid case: {inst.name} n={inst.n} restarts={inst.restarts} passes={passes}")
    h = sg.load_instance([inst])
    h.tune("fm_slots", slots)
    h.bind()
    h.init_spins(seed)
    for p in passes:
        h.run_sweeps(seed=seed, rule=FM, max_sweeps=p, until_converged=False)
    assert h.query("last_fm_big") == inst.restarts
    return h


@pytest.mark.parametrize("dims", [(128, 128), (128, 129), (180, 183), (300, 301)])
def test_scaled_lattice(gpu, dims):
    """16384 and 16512 spins (one and two leaves per lane), 32940 (four) in
    bytes and int32; 90300 spins in bytes (eight) and in device memory."""
    inst = gen.lattice(dims, seed=6, h_range=(-1, 1), restarts=3)
    a = _run(inst, 4, [1, 1])
    b = _run(inst.replace(J=inst.J * 1000, h=inst.h * 1000), 4, [2])
    assert b.query("wide_instances") == 1
    assert np.array_equal(a.spins_out_batch(0), b.spins_out_batch(0))
    assert np.array_equal(a.energy() * 1000, b.energy())
    assert np.array_equal(a.energy(), a.energy(recompute=True))
    assert all(np.array_equal(x, y) for x, y in zip(a.counters(), b.counters()))
    if inst.n < 17000:
        ref, _ = oracle.fm(inst, seed=4, max_passes=2, until_converged=False, threads=8)
        compare(a, [inst], [ref])
    a.free()
    b.free()


@pytest.mark.parametrize("scale", [1, 1000])
def test_scaled_hyper_couplings(gpu, scale):
    """16500 spins with hyper-couplings (several lanes change one spin, and
    four byte half-gains share a word)."""
    inst = gen.erdos_renyi_triples(16500, seed=3, restarts=2)
    inst = inst.replace(J=inst.J * scale, K=inst.K * scale)
    ref, _ = oracle.fm(inst, seed=9, max_passes=1, until_converged=False, threads=8)
    h = _run(inst, 9, [1])
    compare(h, [inst], [ref])
    h.free()


def test_hyper_couplings_beyond_lds(gpu):
    """40000 spins, one with 100 couplings more than the others: int32
    half-gains beyond LDS against the same instance in bytes."""
    inst = gen.erdos_renyi_triples(40000, seed=5, restarts=2)
    have = set(zip(np.minimum(inst.ei, inst.ej).tolist(), np.maximum(inst.ei, inst.ej).tolist()))
    extra = [j for j in range(20001, 20140) if (7, j) not in have][:100]
    inst = inst.replace(ei=np.concatenate([inst.ei, np.full(100, 7)]), ej=np.concatenate([inst.ej, extra]),
                        J=np.concatenate([inst.J, np.where(np.arange(100) % 2, 1, -1)]))
    a = _run(inst, 2, [2])
    b = _run(inst.replace(J=inst.J * 1000, K=inst.K * 1000), 2, [2])
    assert np.array_equal(a.spins_out_batch(0), b.spins_out_batch(0))
    assert np.array_equal(a.energy() * 1000, b.energy())
    a.free()
    b.free()
