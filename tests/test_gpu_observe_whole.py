"""E and M of a batch's lattices at the line between those that one workgroup takes
whole (up to 4096 words: L = 292 has 4088) and those that several share (294:
4116), alone and beside small ones, read after each of two calls; and of a
server's.  All equal the oracle's."""
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


@pytest.mark.parametrize("Ls", [[292], [294], [4, 292, 64], [294, 4, 292, 64]])
def test_batch_observables_at_the_line(Ls):
    print(f"observables of a batch {Ls}", flush=True)
    states = [oracle.init(L, i, True) for i, L in enumerate(Ls)]
    b = ising.Batch(Ls, list(range(len(Ls))), hot=True)
    try:
        for t in (0, 3):
            b.sweep([2.1] * len(Ls), 3)
            r = b.results()
            for i, s in enumerate(states):
                oracle.sweep(s, i, t, 3, 2.1)
                assert (int(r["E"][i]), int(r["M"][i])) == oracle.observables(s), (t, Ls[i])
    finally:
        b.close()


@pytest.mark.parametrize("Ls", [[292], [294], [4, 64, 292], [294, 4]])
def test_served_observables_at_the_line(Ls):
    print(f"observables of a server {Ls}", flush=True)
    srv = ising.Server(hbm_budget=1 << 24, max_slots=8, quantum_sweeps=4)
    got = {}
    try:
        for rid, L in enumerate(Ls):
            srv.submit(rid, L, 2.4, 4)
        while len(got) < len(Ls):
            srv.step()
            got.update({r["req_id"]: r for r in srv.poll()})
    finally:
        srv.close()
    for rid, L in enumerate(Ls):
        s = oracle.init(L, rid, True)
        oracle.sweep(s, rid, 0, 4, 2.4)
        assert (got[rid]["E"], got[rid]["M"]) == oracle.observables(s), L
