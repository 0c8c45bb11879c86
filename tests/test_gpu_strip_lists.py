"""GPU parity of the strip dynamics by lists of picks per word at the edges of its
shapes: one, two and four wavefronts per strip, two words per lane, one column and
several, phases of different widths, strips that do not fill the last workgroup,
picks in several chunks, the first shape with too many words, and a run over
several calls.  State and series equal the oracle's bit for bit."""
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


@pytest.mark.parametrize("L,S", [
    (4, 2), (6, 3), (8, 4),      # the smallest lattices: neighbours that coincide
    (1010, 2),                   # 50 words, 505 strips (four to a workgroup)
    (1344, 2), (1346, 2),        # 64 words; 66 words in 673 strips (two to a workgroup)
    (1010, 5),                   # 100 and 150 words: phases of two and of three columns
    (2688, 2), (2690, 2),        # 128 words; 130 words, four wavefronts
    (990, 9),                    # 192 and 240 words
    (2016, 8),                   # 384 words, two per lane, 3840 picks
    (1344, 16),                  # 512 words, 5120 picks
    (5418, 2),                   # 258 words of one column in chunks of picks
    (1386, 18),                  # 594 words: by windows of picks
])
def test_strip_lists_match_oracle(L, S):
    print(f"strip lists L={L} S={S}", flush=True)
    seed, T = 13, 2.25
    n = 3 if L < 2000 else 1
    s = oracle.init(L, seed, True)
    lat = ising.Lattice(L, seed, hot=True)
    try:
        t = 0
        for n, every in ((n, 2), (1, 1), (1, 0)):
            out = lat.random_iterations(T, S, n, every)
            want = oracle.random_iterations(s, seed, t, n, T, S, every=every)
            t += n
            if every:
                assert out[0].cpu().numpy().tolist() == want[0].tolist() and out[1].cpu().numpy().tolist() == want[1].tolist()
            assert (lat.spins() == s).all() and lat.t == t
    finally:
        lat.close()
