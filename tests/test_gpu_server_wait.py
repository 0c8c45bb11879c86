"""A served large lattice whose resident-tile launches are abandoned (forced from the
host: every wait bounded to one tick, so the launches stop early and end): its
request is run again without tiles and ends with the oracle's E and M, and a small
request beside it, which retires earlier, keeps its own."""
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


@pytest.mark.parametrize("L,sweeps,quantum", [(1024, 120, 50), (4096, 60, 25)])
def test_abandoned_request_is_served_all_the_same(L, sweeps, quantum):
    print(f"served L={L} with a one-tick wait bound", flush=True)
    reqs = {1: (L, 2.2, sweeps), 2: (64, 2.0, quantum // 2)}
    srv = ising.Server(hbm_budget=1 << 30, max_slots=16, quantum_sweeps=quantum)
    got = {}
    try:
        srv.set_resident_wait(1)
        for rid, (n, T, k) in reqs.items():
            srv.submit(rid, n, T, k)
        for _ in range(1000):
            srv.step()
            got.update({r["req_id"]: r for r in srv.poll()})
            if len(got) == len(reqs):
                break
    finally:
        srv.close()
    for rid, (n, T, k) in reqs.items():
        s = oracle.init(n, rid, True)
        oracle.sweep(s, rid, 0, k, T)
        assert (got[rid]["E"], got[rid]["M"]) == oracle.observables(s) and got[rid]["status"] == ising.ISING_OK, rid
    # it was abandoned: admitted once more after the small one was through
    assert got[1]["t_admit_s"] >= got[2]["t_done_s"]


def test_resident_wait_is_checked():
    srv = ising.Server(hbm_budget=1 << 20, max_slots=1)
    try:
        with pytest.raises(ising.IsingError) as e:
            srv.set_resident_wait(60 * 100000000 + 1)
        assert e.value.code == ising.ISING_EINVAL
        srv.set_resident_wait(0)
    finally:
        srv.close()


def test_served_beside_a_captured_lattice():
    """A lattice's resident tiles, captured by the caller and replayed on one stream while a server advances a large
    lattice on another: both give the oracle's results."""
    import torch

    L, seed, T = 1024, 9, 2.269
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(a):
        lat = ising.Lattice(L, seed, hot=True, stream=a)
        assert lat.resident_tiles()[0] > 0
        lat.sweep(T, 2)
        start = lat.spins()
        graph = torch.cuda.CUDAGraph()
        a.synchronize()
        with torch.cuda.graph(graph, stream=a):
            lat.sweep(T, 60)
    srv = ising.Server(hbm_budget=1 << 28, max_slots=8, quantum_sweeps=40, stream=b)
    got = {}
    print("captured tiles beside a server", flush=True)
    try:
        s = start.copy()
        oracle.sweep(s, seed, 2, 60, T)
        for rid in range(3):
            srv.submit(rid, 2048, 2.0 + 0.2 * rid, 80)
            with torch.cuda.stream(a):
                lat.set_spins(start)
                graph.replay()
            while len(got) <= rid:
                srv.step()
                got.update({r["req_id"]: r for r in srv.poll()})
            assert (lat.spins() == s).all(), rid
            lat.synchronize()
        for rid in range(3):
            s = oracle.init(2048, rid, True)
            oracle.sweep(s, rid, 0, 80, 2.0 + 0.2 * rid)
            assert (got[rid]["E"], got[rid]["M"]) == oracle.observables(s), rid
    finally:
        srv.close()
        lat.close()
