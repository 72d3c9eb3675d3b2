"""Which of the two block kernels takes a batch under GREEDY_TIE: small batches
of small instances the byte kernel, large ones the bit-sliced kernel, a given
bits_groups the bit-sliced kernel, under either schedule request and beside
instances that only the byte kernel can take; the results are those of the
oracle, with start energies left out or not."""
import pytest

import instances as gen
import oracle
from parity import compare, log

pytestmark = pytest.mark.gpu

TIE = 1


def _er(n, count, restarts):
    return [gen.erdos_renyi_triples(n, seed=k, mean_degree=5, triples_per_spin=0.2, restarts=restarts, instance_id=k)
            for k in range(count)]


CASES = {  # instances, knobs, whether the bit-sliced kernel runs under TIE
    "one": (lambda: _er(32, 1, 64), {}, 0),
    "few": (lambda: _er(200, 8, 256), {}, 0),
    "given": (lambda: _er(200, 2, 64), {"bits_groups": 8}, 1),
    "many": (lambda: _er(72, 500, 256), {}, 1),
    "chimera": (lambda: [gen.chimera(8, 8, seed=k, instance_id=k, restarts=64) for k in range(4)], {}, 1),
    # one launch for every number of groups per workgroup: two in turn lose
    "chimera, lattices": (lambda: [gen.chimera(11, 11, seed=1, instance_id=1, restarts=117)] +
                          [gen.lattice((20, 20), seed=2, instance_id=2, restarts=58)], {}, 0),
    "lattice with fields": (lambda: [gen.lattice((22, 24), seed=3, h_range=(-2, 2), instance_id=1, restarts=113)], {}, 0),
    "chimera of 968": (lambda: [gen.chimera(11, 11, seed=1, instance_id=1, restarts=117)], {}, 1),
    "mixed": (lambda: _er(64, 2, 64) + [gen.random_regular3(300, seed=5, j_range=(-40, 40), instance_id=9, restarts=64)],
              {}, 0),
}


@pytest.mark.parametrize("uc", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_choice(gpu, name, uc):
    import paper_0912_3912_amd as sg
    make, knobs, bits = CASES[name]
    insts = make()
    schedules = (sg.SCHED_AUTO, sg.SCHED_BLOCK) if name != "many" else (sg.SCHED_AUTO,)
    ref = [oracle.run(i, seed=3, rule=TIE, max_sweeps=20, until_converged=uc, threads=8)[0] for i in insts[:40]]
    for schedule in schedules:
        log(f"block kernel under TIE: {name} schedule={schedule} uc={uc}")
        h = sg.load_instance(insts)
        for k, v in knobs.items():
            h.tune(k, v)
        h.bind()
        h.init_spins(3)
        h.run_sweeps(seed=3, rule=TIE, max_sweeps=20, until_converged=uc, schedule=schedule)
        assert h.query("last_bits") == bits
        if name == "many":
            E = h.energy()
            assert (E == h.energy(recompute=True)).all()
            for k, st in enumerate(ref):
                assert (E[k * 256:(k + 1) * 256] == st.energy).all() and (h.spins_out_batch(k) == st.spins).all()
        else:
            compare(h, insts, ref)
        h.free()


def test_sparse_full_device(gpu):
    """Many ties on a device full of workgroups, where both kernels come close."""
    import paper_0912_3912_amd as sg
    insts = [gen.erdos_renyi_triples(400, seed=k, mean_degree=2, triples_per_spin=0.0, restarts=256, instance_id=k)
             for k in range(256)]
    log("block kernel under TIE: 256 sparse graphs, 50 sweeps")
    h = sg.load_instance(insts).bind()
    h.init_spins(3)
    h.run_sweeps(seed=3, rule=TIE, max_sweeps=50, until_converged=False)
    assert h.query("last_bits") == 1
    E = h.energy()
    assert (E == h.energy(recompute=True)).all()
    for k in (0, 255):
        st = oracle.run(insts[k], seed=3, rule=TIE, max_sweeps=50, until_converged=False, threads=8)[0]
        assert (E[k * 256:(k + 1) * 256] == st.energy).all() and (h.spins_out_batch(k) == st.spins).all()
    h.free()


def test_autotuner_leaves_the_choice(gpu):
    """Applying a setting that changes nothing does not ask for a kernel."""
    import paper_0912_3912_amd as sg
    from paper_0912_3912_amd import autotune as at
    h = sg.load_instance(_er(100, 2, 64)).bind()
    at.apply(h, {}, {k: h.query(k) for k in at._DEFAULTS})
    h.init_spins(3)
    h.run_sweeps(seed=3, rule=TIE, max_sweeps=5, until_converged=False)
    assert h.query("last_bits") == 0
    h.free()
