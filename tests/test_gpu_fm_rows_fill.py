"""The pass kernel with LDS row tables on graphs whose slices have few rows (a
complete graph has a colour, and so a slice, per spin): equal to the oracle, and
building the tables costs less than the other wavefront kernel's passes."""
import time

import pytest

import instances as gen
import oracle
from parity import compare, log

pytestmark = pytest.mark.gpu

FM = 2


@pytest.mark.parametrize("scale", [1, 100000])
@pytest.mark.parametrize("n,restarts", [(2, 3), (65, 1), (120, 20)])
def test_complete_graphs(gpu, n, restarts, scale):
    """Packed and wide form, with zero couplings in the rows and triples."""
    import paper_0912_3912_amd as sg
    inst = gen.random_small(n, seed=n, p_edge=1.0, n_triples=2 * n if n > 2 else 0, j_range=(-3, 3), h_range=(-2, 2))
    inst = inst.replace(J=inst.J * scale, K=inst.K * scale, restarts=restarts)
    log(f"rows of a complete graph: n={n} restarts={restarts} scale={scale}")
    ref, _ = oracle.fm(inst, seed=5, max_passes=3, until_converged=True, threads=8)
    for lanes in (0, 1):
        h = sg.load_instance([inst])
        h.tune("fm_lanes", lanes)
        h.bind()
        h.init_spins(5)
        h.run_sweeps(seed=5, rule=FM, max_sweeps=3, until_converged=True)
        compare(h, [inst], [ref])
        h.free()


def test_building_the_rows_is_cheap(gpu):
    """Two passes of one replica of a complete graph of 200 spins: the tables
    once took five times as long as the whole call on 64-bit keys."""
    import paper_0912_3912_amd as sg
    inst = gen.complete_graph(200, seed=1)
    ms = []
    for key32 in (1, 0):
        h = sg.load_instance([inst])
        h.tune("fm_key32", key32)
        h.bind()
        best = 1e9
        for _ in range(6):
            h.init_spins(5)
            h.energy()
            t0 = time.perf_counter()
            h.run_sweeps(seed=5, rule=FM, max_sweeps=2, until_converged=False)
            best = min(best, time.perf_counter() - t0)
        ms.append(best * 1e3)
        h.free()
    log(f"complete graph of 200 spins: row tables {ms[0]:.2f} ms, 64-bit keys {ms[1]:.2f} ms")
    assert ms[0] < 1.5 * ms[1]
