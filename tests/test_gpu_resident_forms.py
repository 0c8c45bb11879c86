"""GPU parity of resident tiles whose lattices hold their words in different
ways: one word per thread, two, and formed in every half-sweep, alone and side by
side in one batch (which then runs the kernel that holds all three), with a
narrower last band and with a whole lattice in one band.  Equal to the oracle."""
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


# bands of 20 columns, 64 threads: 50 words of a colour per band (L = 100), 110 (222), 240 (500: formed), 5 x 10 whole (20)
@pytest.mark.parametrize("Ls", [[100], [222], [500], [20], [100, 222, 500, 20], [104, 100], [224, 500]], ids=str)
def test_forms_match_oracle(Ls):
    print(f"resident forms L={Ls}", flush=True)
    seeds, Ts = [11 + i for i in range(len(Ls))], [2.0 + 0.2 * i for i in range(len(Ls))]
    b = ising.Batch(Ls, seeds, hot=True)
    try:
        b.set_plan(resident_max_L=0, resident_block=64, words_per_thread=1, tiled_block=64, sweeps_per_graph=6,
                   tile_max_L=1024, tile_sweeps=1, tile_cols=20, tile_block=64, tile_exchange=1)
        for n, every in ((6, 1), (9, 3)):
            t = b.sweep_count(0)
            E, M = (x.cpu().numpy() for x in b.sweep(Ts, n, every=every, series=True))
            for i, (L, seed, T) in enumerate(zip(Ls, seeds, Ts)):
                s = oracle.init(L, seed, True)
                oracle.sweep(s, seed, 0, t, T)
                Es, Ms = oracle.sweep(s, seed, t, n, T, every=every)
                assert E[i].tolist() == Es.tolist() and M[i].tolist() == Ms.tolist(), L
                assert (b.spins(i) == s).all(), L
    finally:
        b.close()
