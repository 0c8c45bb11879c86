"""Half-sweep launches over a table of small lattices: sizes with few live positions
a word (2 at L = 4 to 16 at L = 64 and 128) and with 17 or more (42, 84, 100, 130), in
tables that are mostly of the first kind, mostly of the second, and of one kind
alone.  Series, sums and states equal the oracle's."""
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


@pytest.mark.parametrize("wpt,block", [(1, 64), (1, 256), (2, 128), (4, 256)])
@pytest.mark.parametrize("Ls", [[4, 6, 8, 16, 32, 44, 64, 86, 96, 128], [4, 16, 64, 128, 42, 130], [42, 84, 100, 130, 64],
                                [64, 64, 300]])
def test_table_of_small_lattices(Ls, wpt, block):
    print(f"half-sweep table {Ls} words_per_thread={wpt} block={block}", flush=True)
    seeds, Ts = [5 + i for i in range(len(Ls))], [1.6 + 0.15 * i for i in range(len(Ls))]
    b = ising.Batch(Ls, seeds, hot=True)
    try:
        b.set_plan(resident_max_L=0, resident_block=256, words_per_thread=wpt, tiled_block=block, sweeps_per_graph=3)
        E, M = (x.cpu().numpy() for x in b.sweep(Ts, 8, every=2, series=True))
        for i, (L, seed, T) in enumerate(zip(Ls, seeds, Ts)):
            s = oracle.init(L, seed, True)
            Es, Ms = oracle.sweep(s, seed, 0, 8, T, every=2)
            assert E[i].tolist() == Es.tolist() and M[i].tolist() == Ms.tolist(), L
            assert (b.spins(i) == s).all(), L
    finally:
        b.close()
