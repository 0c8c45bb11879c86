"""Resident tiles where the library's default runs drawn codes instead (L <= 292),
set explicitly, in the shapes that ising_get_resident_tiles gives for these
lattices; and thresholds at both ends of their range in every form of a tile
(one word per thread, two, formed in every half-sweep; bands and whole
lattices).  Series and state equal the oracle's bit for bit."""
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


def _run(L, shape, T, seed=8, n=6):
    print(f"resident tiles L={L} {shape} T={T}", flush=True)
    lat = ising.Lattice(L, seed, hot=True)
    try:
        lat.set_resident_tiles(*(shape or lat.resident_tiles()))
        E, M = lat.sweep_measure(T, n, 2)
        lat.sweep(T, 3)
        got, gE, gM = lat.spins(), E.cpu().numpy().tolist(), M.cpu().numpy().tolist()
    finally:
        lat.close()
    s = oracle.init(L, seed, True)
    Es, Ms = oracle.sweep(s, seed, 0, n, T, every=2)
    oracle.sweep(s, seed, n, 3, T)
    assert gE == Es.tolist() and gM == Ms.tolist()
    assert (got == s).all()


@pytest.mark.parametrize("L", [4, 6, 42, 64, 130, 192, 194, 256, 292])
def test_default_shapes_of_small_lattices(L):
    _run(L, None, 2.269)


# kept words per thread: one, two, none; bands, then whole lattices
@pytest.mark.parametrize("L,shape", [(300, (8, 512, 1000)), (1008, (64, 1024, 1000)), (512, (64, 256, 1000)),
                                     (64, (64, 128, 1000)), (64, (64, 64, 1000)), (128, (128, 128, 1000))])
@pytest.mark.parametrize("T", [0.05, 1e9])
def test_thresholds_at_both_ends_in_tiles(L, shape, T):
    """T = 0.05: both thresholds 0, no uphill move; T = 1e9: both 2^32 - 1."""
    _run(L, shape, T)
