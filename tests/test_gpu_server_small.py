"""Served small lattices: sizes from one wavefront to two words per thread in one
quantum, alone and beside large ones, with different numbers of sweeps left; more
lattices than compute units; and more words than the codes of one group, whose
sweeps are then drawn in several parts.  Every E, M equals the oracle's."""
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


def _serve(reqs, quantum):
    srv = ising.Server(hbm_budget=1 << 30, max_slots=1024, quantum_sweeps=quantum)
    try:
        for rid, (L, T, sweeps) in enumerate(reqs):
            srv.submit(rid, L, T, sweeps)
        out, steps = {}, 0
        while len(out) < len(reqs):
            srv.step()
            out.update({r["req_id"]: r for r in srv.poll()})
            steps += 1
            assert steps < 10000
        return out
    finally:
        srv.close()


def _check(out, reqs, ids):
    for rid in ids:
        L, T, sweeps = reqs[rid]
        s = oracle.init(L, rid, True)
        oracle.sweep(s, rid, 0, sweeps, T)
        assert (out[rid]["E"], out[rid]["M"]) == oracle.observables(s), (rid, L)


@pytest.mark.parametrize("large", [[], [514, 300]])
def test_served_small_sizes(large):
    print(f"served small sizes beside {large}", flush=True)
    Ls = [4, 42, 64, 100, 204, 206, 256] + large
    reqs = [(L, 1.8 + 0.1 * i, 7 * i % 23) for i, L in enumerate(Ls)]
    _check(_serve(reqs, 9), reqs, range(len(reqs)))


@pytest.mark.parametrize("L,n", [(64, 300), (256, 340)])
def test_served_many_small(L, n):
    print(f"served {n} of L={L}", flush=True)
    reqs = [(L, 2.0 + 0.001 * i, 20 - i % 3) for i in range(n)]
    _check(_serve(reqs, 20), reqs, [0, 1, 255, 256, 299, n - 27, n - 26, n - 25, n - 24, n - 1])


@pytest.mark.parametrize("Ls,quantum", [
    ([294], 30),                 # bands of 8 columns
    ([1024], 40), ([1026], 40),  # bands of 4 columns; of 6, the last one narrower
    ([2048, 64], 40),            # beside a small lattice
    ([700, 2048, 1008], 100),    # one after the other, with different numbers of sweeps left
])
def test_served_few_large(Ls, quantum):
    """Few large lattices: they go through a quantum in resident tiles, and results, retired in turn, are those of
    half-sweep launches."""
    print(f"served few large {Ls}", flush=True)
    reqs = [(L, 2.1 + 0.1 * i, 130 + 17 * i) for i, L in enumerate(Ls)]
    _check(_serve(reqs, quantum), reqs, range(len(reqs)))
