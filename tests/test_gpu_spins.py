"""Spins set from host bytes: lattices that go to the device whole and in pieces
(above L = 4096), with dead slots in the last word rows and without, any nonzero
byte up; words set over an earlier state, read back and swept on as the oracle."""
import numpy as np
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


@pytest.mark.parametrize("L", [4, 22, 42, 130, 1008, 4096, 4098])
def test_set_spins_roundtrip(L):
    print(f"set spins L={L}", flush=True)
    rng = np.random.default_rng(L)
    s = rng.integers(0, 2, (L, L), dtype=np.uint8)
    lat = ising.Lattice(L, 5, hot=True)
    try:
        lat.set_spins(s * rng.integers(1, 256, (L, L), dtype=np.uint8))
        assert (lat.spins() == s).all()
        assert tuple(lat.observables()) == tuple(oracle.observables(s))
        lat.sweep(2.1, 2)
        oracle.sweep(s, 5, 0, 2, 2.1)
        assert (lat.spins() == s).all()
    finally:
        lat.close()


# rows that fill, just miss and just exceed a wavefront's and a workgroup's run
@pytest.mark.parametrize("L", [4, 62, 64, 66, 254, 256, 258, 1022, 1024, 1026, 2058])
@pytest.mark.parametrize("hot", [True, False])
def test_initial_state_matches_oracle(L, hot):
    print(f"initial state L={L} hot={hot}", flush=True)
    lat = ising.Lattice(L, 77 + (3 << 32), hot=hot)
    try:
        assert (lat.spins() == oracle.init(L, 77 + (3 << 32), hot)).all()
    finally:
        lat.close()
