"""GPU parity of the pass kernel with LDS row tables (SG_RULE_FM, at most 4096
spins): sizes at the edges of its leaves and of its range, rows longer than a
wavefront, both storage forms, one and several wavefronts per workgroup.
Results are integers and equal the oracle's bit for bit."""
import numpy as np
import pytest

import instances as gen
import oracle
from parity import compare, log

pytestmark = pytest.mark.gpu

FM = 2


def _case(name):
    if name.startswith("square"):  # the largest lattices; odd extents
        a, b = {"square64x64": (64, 64), "square63x65": (63, 65)}[name]
        return gen.lattice((a, b), seed=3, h_range=(-1, 1), restarts=2)
    if name.startswith("sparse"):  # around one and two leaves; more replicas than wavefronts of a workgroup
        n = int(name[6:])
        return gen.random_small(n, seed=n, p_edge=min(1.0, 5.0 / n), n_triples=n // 3, j_range=(-40, 40),
                                h_range=(-9, 9), k_range=(-30, 30)).replace(restarts=37, instance_id=n)
    if name == "complete150":  # rows of 149 couplings: three rounds of 64 per move
        return gen.complete_graph(150, seed=2, j_range=(-9, 9)).replace(restarts=5)
    # 100 hyper-couplings on one spin beside few elsewhere
    rng = np.random.default_rng(4)
    base = gen.random_small(400, seed=4, p_edge=0.01, n_triples=50, j_range=(-50, 50), h_range=(-9, 9))
    pairs = rng.permutation(np.arange(1, 201)).reshape(100, 2)
    tri = np.concatenate([base.tri[~(base.tri == 0).any(axis=1)], np.column_stack([np.zeros(100, int), pairs])])
    return base.replace(tri=tri, K=rng.integers(1, 9, tri.shape[0]), restarts=3)


@pytest.mark.parametrize("scale", [1, 100000])
@pytest.mark.parametrize("name", ["sparse63", "sparse64", "sparse65", "sparse129", "complete150", "triples", "square63x65",
                                  "square64x64"])
def test_row_table_kernel(gpu, name, scale):
    import paper_0912_3912_amd as sg
    inst = _case(name)
    inst = inst.replace(J=inst.J * scale, K=inst.K * scale)
    log(f"fm rows case: {name} n={inst.n} scale={scale} restarts={inst.restarts}")
    ref, _ = oracle.fm(inst, seed=5, max_passes=3, until_converged=True, threads=8)
    for waves in (1, 16) if name.startswith("sparse") else (0,):
        h = sg.load_instance([inst])
        h.tune("fm_waves", waves)
        h.tune("fm_lanes", 0)
        h.bind()
        h.init_spins(5)
        h.run_sweeps(seed=5, rule=FM, max_sweeps=3, until_converged=True)
        assert h.query("wide_instances") == (1 if scale > 1 else 0)
        compare(h, [inst], [ref])
        h.free()
