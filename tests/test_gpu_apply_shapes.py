"""GPU parity of the sweeps applied from drawn codes at the edges of their
workgroup shapes: one to four words of a colour per thread, one to four
wavefronts, slots past the last word, and lattices of one batch that need
different shapes.  Series and state equal the oracle's bit for bit."""
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


# words of a colour: 42, 66, 128, 225, 250, 260, 378, 592, 774, 1020
@pytest.mark.parametrize("Ls", [[42], [44], [64], [90], [100], [104], [126], [148], [172], [204], [204, 4, 64, 168]],
                         ids=str)
@pytest.mark.parametrize("block", [64, 192, 256])
def test_applied_codes_match_oracle(Ls, block):
    print(f"apply shapes L={Ls} block={block}", flush=True)
    seeds = [71 + i for i in range(len(Ls))]
    Ts = [1.9 + 0.3 * i for i in range(len(Ls))]
    b = ising.Batch(Ls, seeds, hot=True)
    try:
        b.set_plan(resident_max_L=204, resident_block=block, words_per_thread=1, tiled_block=64, sweeps_per_graph=20,
                   draw_sweeps=11)
        E1, M1 = (x.cpu().numpy() for x in b.sweep(Ts, 20, every=1, series=True))
        E2, M2 = (x.cpu().numpy() for x in b.sweep(Ts, 9, every=4, series=True))
        for i, (L, seed, T) in enumerate(zip(Ls, seeds, Ts)):
            s = oracle.init(L, seed, True)
            Es1, Ms1 = oracle.sweep(s, seed, 0, 20, T, every=1)
            Es2, Ms2 = oracle.sweep(s, seed, 20, 9, T, every=4)
            assert E1[i].tolist() == Es1.tolist() and M1[i].tolist() == Ms1.tolist(), L
            assert E2[i].tolist() == Es2.tolist() and M2[i].tolist() == Ms2.tolist(), L
            assert (b.spins(i) == s).all(), L
    finally:
        b.close()
