"""Pass-based search on handles whose instances need different kernels: few
replicas share the launch that the largest or densest needs, where a launch of
their own would only come on top of it; equal to the oracle."""
import pytest

import instances as gen
import oracle
from parity import compare, log

pytestmark = pytest.mark.gpu

FM = 2


def _run(insts, knobs, passes, seed=5):
    import paper_0912_3912_amd as sg
    h = sg.load_instance(insts)
    for k, v in knobs.items():
        h.tune(k, v)
    h.bind()
    h.init_spins(seed)
    h.run_sweeps(seed=seed, rule=FM, max_sweeps=passes, until_converged=False)
    launches = h.query("hot_launches")
    compare(h, insts, [oracle.fm(i, seed=seed, max_passes=passes, until_converged=False, threads=8)[0] for i in insts])
    h.free()
    return launches


@pytest.mark.parametrize("sizes,launches", [((39300, 6000), 1), ((39300, 39200), 1), ((6000, 5000), 2)])
def test_beyond_4096(gpu, sizes, launches):
    """The first instance in the wide form (beyond 39168 spins only the
    device-memory kernel takes it), the second not."""
    wide = gen.erdos_renyi_triples(sizes[0], seed=1, mean_degree=3, triples_per_spin=0.1, instance_id=1)
    insts = [wide.replace(J=wide.J * 1000),
             gen.erdos_renyi_triples(sizes[1], seed=2, mean_degree=3, triples_per_spin=0.1, instance_id=2)]
    log(f"pass kernels beyond 4096 spins: {sizes}")
    assert _run(insts, {"fm_slots": 4}, 1) == launches


@pytest.mark.parametrize("dense,sparse,launches", [(400, 300, 1), (400, 3000, 2), (0, 3000, 1)])
def test_up_to_4096(gpu, dense, sparse, launches):
    """A complete graph too large for row tables beside sparse graphs: these get
    a row-table launch of their own only if they are much the longer."""
    insts = [gen.lattice((sparse // 50, 50), seed=k, instance_id=k, j_values=(-90, 80), restarts=2) for k in range(2)]
    if dense:
        insts.append(gen.complete_graph(dense, seed=1).replace(instance_id=9, restarts=2))
    log(f"pass kernels up to 4096 spins: complete graph of {dense} beside {sparse}")
    assert _run(insts, {"fm_lanes": 0}, 2) == launches


@pytest.mark.parametrize("hub,passes,restarts,waves", [(150, 3, 4, False), (50, 3, 4, True), (110, 3, 4, True),
                                                       (110, 1, 4, False)])
def test_wide_rows(gpu, hub, passes, restarts, waves):
    """One spin coupled to many others makes every row of a table as wide; the
    table is left out where that costs more than the sliced rows (waves: the
    launch has a row table's few wavefronts, one for few replicas)."""
    import numpy as np
    import paper_0912_3912_amd as sg
    r = np.random.default_rng(3)
    n = 200
    j = np.arange(1, hub + 1, dtype=np.int32)
    ring = np.arange(1, n - 1, dtype=np.int32)
    e = np.concatenate([np.stack([np.zeros_like(j), j], 1), np.stack([ring, ring + 1], 1)])
    if hub == 110:  # dense beside it: the sliced rows are long too
        a, b = np.triu_indices(100, 2)
        e = np.concatenate([e, np.stack([a + 1, b + 1], 1)]).astype(np.int32)
    inst = gen.Instance(n, e[:, 0].copy(), e[:, 1].copy(), r.integers(-3, 4, len(e)), None).replace(restarts=restarts)
    log(f"row tables: hub={hub} passes={passes}")
    h = sg.load_instance([inst]).tune("fm_lanes", 0).bind()
    h.init_spins(5)
    h.run_sweeps(seed=5, rule=FM, max_sweeps=passes, until_converged=False)
    assert (h.query("last_fm_waves") == 1) == waves
    compare(h, [inst], [oracle.fm(inst, seed=5, max_passes=passes, until_converged=False, threads=8)[0]])
    h.free()
