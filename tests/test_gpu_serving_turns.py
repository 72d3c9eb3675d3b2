"""Solo requests of the serving loop take turns only where a run may hold the
device with workgroups that wait for one another: which handles say so, and the
turns that a server takes."""
import threading

import pytest

import instances as gen
from parity import log

pytestmark = pytest.mark.gpu

GREEDY, TIE, FM = 0, 1, 2


def _wide():
    i = gen.random_regular3(70000, seed=3, instance_id=4)
    return i.replace(J=i.J * 1000)


@pytest.mark.parametrize("make,knobs,want", [
    (lambda: gen.random_regular3(6000, seed=1, instance_id=1), {}, 0),
    (lambda: gen.random_regular3(6000, seed=1, instance_id=1), {"team_wgs": 4}, 1),
    (lambda: gen.random_regular3(70000, seed=2, instance_id=2), {}, 1),
    (lambda: gen.random_regular3(70000, seed=2, instance_id=2), {"team_wgs": -1}, 0),
    (lambda: gen.random_regular3(70000, seed=2, instance_id=2), {"team_wgs": 1}, 0),
    (lambda: gen.random_regular3(70000, seed=2, instance_id=2, restarts=64), {}, 1),
    (_wide, {}, 0),
])
def test_may_team(gpu, make, knobs, want):
    import paper_0912_3912_amd as sg
    h = sg.load_instance([make()])
    for k, v in knobs.items():
        h.tune(k, v)
    h.bind()
    assert h.query("may_team") == want
    h.free()


class _Counting:
    def __init__(self):
        self.lock, self.taken = threading.Lock(), 0

    def __enter__(self):
        self.lock.acquire()
        self.taken += 1

    def __exit__(self, *a):
        self.lock.release()


def test_turns(gpu):
    from paper_0912_3912_amd.serve import Request, Server
    server = Server(budget_bytes=1 << 28, slots=2, ingest_workers=2, shared=False)
    server.coop_lock = turn = _Counting()
    fixed = dict(max_sweeps=5, until_converged=False)
    reqs = [Request(rid=0, instance=gen.random_regular3(6000, seed=1, instance_id=1), rule=TIE, **fixed),
            Request(rid=1, instance=_wide(), rule=GREEDY, **fixed),
            Request(rid=2, instance=gen.random_regular3(12000, seed=2, instance_id=2), rule=GREEDY),
            Request(rid=3, instance=gen.lattice((64, 64), seed=4, instance_id=3), rule=TIE, **fixed),
            Request(rid=4, instance=gen.lattice((44, 40), seed=4, instance_id=5), rule=FM, **fixed)]
    for r in reqs:
        server.submit(r)
    res = server.wait([r.rid for r in reqs])
    log(f"turns: {[r.status for r in res]}")
    assert all(r.status == "ok" for r in res) and turn.taken == 0
    server.submit(Request(rid=5, instance=gen.random_regular3(70000, seed=2, instance_id=2), rule=TIE, **fixed))
    server.submit(Request(rid=6, instance=gen.lattice((64, 64, 64), seed=4, instance_id=6), rule=TIE, **fixed))
    res = server.wait([5, 6])
    server.close()
    assert res[0].status == res[1].status == "ok" and turn.taken == 2
