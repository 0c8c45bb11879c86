"""Sweeps applied from drawn codes in passes of the most sweeps there are, with a
sample after each, which take the most LDS there is.  Equal to the oracle."""
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


@pytest.mark.parametrize("L,S", [(64, 4096), (204, 4096)])
def test_long_passes_match_oracle(L, S):
    print(f"long passes L={L} S={S}", flush=True)
    T, seed = 2.2, 4
    b = ising.Batch([L], [seed], hot=True)
    try:
        b.set_plan(resident_max_L=L, resident_block=256, words_per_thread=1, tiled_block=64, sweeps_per_graph=S,
                   draw_sweeps=S)
        E, M = (x.cpu().numpy() for x in b.sweep([T], S, every=1, series=True))
        s = oracle.init(L, seed, True)
        Es, Ms = oracle.sweep(s, seed, 0, S, T, every=1)
        assert E[0].tolist() == Es.tolist() and M[0].tolist() == Ms.tolist()
        assert (b.spins(0) == s).all()
    finally:
        b.close()
