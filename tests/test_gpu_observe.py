"""GPU parity of E and M taken from the words: one lattice by workgroups of 256
and of 2048 words, batches whose lattices take one workgroup, several, and
more runs of words than workgroups, and repeated observations (the sums are
left zero for the next one).  Equal to the oracle's exactly."""
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


# 4, 292, 520, 193536, 1048000 and 1055700 words
@pytest.mark.parametrize("L", [4, 74, 104, 2016, 4678, 4692])
def test_single_observables_match_oracle(L):
    print(f"observables L={L}", flush=True)
    lat = ising.Lattice(L, 3, hot=True)
    try:
        s = oracle.init(L, 3, True)
        for _ in range(2):
            assert tuple(lat.observables()) == tuple(oracle.observables(s))
        lat.sweep(1.5, 1)
        oracle.sweep(s, 3, 0, 1, 1.5)
        assert tuple(lat.observables()) == tuple(oracle.observables(s))
    finally:
        lat.close()


@pytest.mark.parametrize("Ls", [[4], [194], [196, 210, 1008, 6], [1008] + [4, 6, 8, 42] * 600], ids=["one", "run", "mixed", "many"])
def test_batch_observables_match_oracle(Ls):
    print(f"batch observables n={len(Ls)}", flush=True)
    seeds = [9 + i for i in range(len(Ls))]
    b = ising.Batch(Ls, seeds, hot=True)
    try:
        want = [oracle.observables(oracle.init(L, seed, True)) for L, seed in zip(Ls, seeds)]
        for _ in range(3):
            res = b.results()
            got = list(zip((int(x) for x in res["E"]), (int(x) for x in res["M"])))
            assert got == [tuple(w) for w in want]
    finally:
        b.close()
