"""E and M of the replicas from their words: runs of words that end inside a
thread's four, inside a row and in the last workgroup, and repeated
observations (the counters are left zero).  Equal to the oracle's observables of
the unpacked spins."""
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


# 16, 1764, 2116 (just above a run of 2048), 65536, 66564 and 1052676 (runs of 2304) words
@pytest.mark.parametrize("L", [4, 42, 46, 256, 258, 1026])
def test_replica_observables(L):
    print(f"replica observables L={L}", flush=True)
    T = [1.5 + 0.1 * k for k in range(ising.REPLICAS)]
    r = ising.Replicas(L, 19, hot=True)
    try:
        r.sweep(T, 2)
        E, M = (x.cpu().numpy() for x in r.sweep_measure(T, 2, 1))
        want = [oracle.observables(r.spins(k)) for k in range(ising.REPLICAS)]
        for _ in range(2):
            e, m = r.observables()
            assert [(int(a), int(b)) for a, b in zip(e, m)] == want
        assert [(int(a), int(b)) for a, b in zip(E.reshape(-1, ising.REPLICAS)[-1], M.reshape(-1, ising.REPLICAS)[-1])] == want
    finally:
        r.close()
