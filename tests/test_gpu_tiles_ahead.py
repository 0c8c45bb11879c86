"""GPU parity of batches whose resident tiles run beside the other launches (at
most half of what a compute unit holds, of each) or ahead of them (more), with
half-sweeps and a small lattice, over several replays of a chunk.  Equal to the
oracle."""
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


# lattices of 30 tiles of 512 threads, two of which a compute unit holds: 240 and 270 of the 256 that may run beside
@pytest.mark.parametrize("tiled", [8, 9])
def test_tiles_beside_and_ahead_match_oracle(tiled):
    print(f"tiles ahead tiled={tiled}", flush=True)
    Ls = [300] * tiled + [302, 40, 504]
    seeds, Ts = [31 + i for i in range(len(Ls))], [2.0 + 0.05 * i for i in range(len(Ls))]
    b = ising.Batch(Ls, seeds, hot=True)
    try:
        b.set_plan(resident_max_L=64, resident_block=64, words_per_thread=2, tiled_block=64, sweeps_per_graph=4,
                   tile_max_L=300, tile_sweeps=1, tile_cols=10, tile_block=512, tile_exchange=1)
        E, M = (x.cpu().numpy() for x in b.sweep(Ts, 14, every=2, series=True))
        for i, (L, seed, T) in enumerate(zip(Ls, seeds, Ts)):
            s = oracle.init(L, seed, True)
            Es, Ms = oracle.sweep(s, seed, 0, 14, T, every=2)
            assert E[i].tolist() == Es.tolist() and M[i].tolist() == Ms.tolist(), (i, L)
            assert (b.spins(i) == s).all(), (i, L)
    finally:
        b.close()
