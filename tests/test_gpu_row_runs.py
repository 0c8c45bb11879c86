"""GPU parity of the half-sweep kernels' runs of words (64 words of a colour
of one row per wavefront and run, one to four runs) at the edges of their
rules: rows that fill, just miss and just exceed a run, a wavefront or a
workgroup; word rows in bands per XCD (from 256 rows) whose number is and is
not a multiple of 8; a word buffer that is aligned to eight bytes only; and
thresholds at both ends of their range.  Series and state equal the oracle's
bit for bit."""
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


# 63, 64, 65, 128, 129, 255, 256 and 257 words of a colour per row; 256 and 258 word rows
@pytest.mark.parametrize("L", [126, 128, 130, 256, 258, 510, 512, 514, 5376, 5400])
def test_runs_match_oracle(L):
    seed, n = 31, 4
    s = oracle.init(L, seed, True)
    Es, Ms = oracle.sweep(s, seed, 0, n, 2.269, every=1)
    for wpt, block in ((1, 64), (1, 256), (2, 128), (4, 64), (4, 192), (4, 256)):
        print(f"runs L={L} words_per_thread={wpt} block={block}", flush=True)
        lat = ising.Lattice(L, seed, hot=True)
        try:
            lat.set_resident_tiles(0)
            lat.set_plan(wpt, block)
            E, M = lat.sweep_measure(2.269, n, 1)
            assert E.cpu().numpy().tolist() == Es.tolist() and M.cpu().numpy().tolist() == Ms.tolist(), (wpt, block)
            assert (lat.spins() == s).all(), (wpt, block)
        finally:
            lat.close()


@pytest.mark.parametrize("L", [126, 130, 256, 258])
def test_replica_runs_match_oracle(L):
    seed, Ts = 5, [1.5 + 0.1 * ((k * 7) % 21) for k in range(21)]
    s = oracle.replica_init(L, seed, True)
    oracle.replica_sweep(s, seed, 0, 3, Ts)
    for wpt in (1, 2, 4):
        rep = ising.Replicas(L, seed, hot=True)
        rep.set_plan(wpt)
        rep.sweep(Ts, 3)
        got = [rep.spins(k) for k in range(21)]
        rep.close()
        assert all(np.array_equal(got[k], s[k]) for k in range(21)), wpt


def test_buffer_aligned_to_eight_bytes():
    import torch

    L, seed = 258, 3
    n = ising.ising_required_bytes(L) // 8
    buf = torch.zeros(n + 2, dtype=torch.int64, device="cuda")
    h = ising.ising_create_in(L, seed, ising.ISING_HOT, buf.data_ptr() + 8, 8 * n)
    try:
        ising.ising_set_resident_tiles(h, 0)
        ising.ising_sweep(h, 2.0, 3)
        got = ising.ising_get_spins(h, L)
    finally:
        ising.ising_destroy(h)
    s = oracle.init(L, seed, True)
    oracle.sweep(s, seed, 0, 3, 2.0)
    assert (got == s).all()
    assert int(buf[0]) == 0 and int(buf[n + 1]) == 0


@pytest.mark.parametrize("T", [0.05, 1e9])
def test_thresholds_at_both_ends(T):
    """T = 0.05: both thresholds 0, no uphill move; T = 1e9: both 2^32 - 1."""
    L, seed = 258, 8
    s = oracle.init(L, seed, True)
    oracle.sweep(s, seed, 0, 5, T)
    for resident in (False, True):
        lat = ising.Lattice(L, seed, hot=True)
        try:
            if not resident:
                lat.set_resident_tiles(0)
            lat.sweep(T, 5)
            assert (lat.spins() == s).all(), resident
        finally:
            lat.close()


@pytest.mark.parametrize("wpt,block", [(1, 64), (1, 256), (2, 64), (4, 256)])
def test_batch_table_in_runs_per_xcd(wpt, block):
    """A batch's table of wavefronts dealt to the XCDs in runs, with workgroups left over behind the last whole
    round of runs."""
    print(f"batch table words_per_thread={wpt} block={block}", flush=True)
    Ls = [1008, 256, 2048, 130, 514]
    seeds, Ts = [3, 4, 5, 6, 7], [2.0, 2.3, 2.6, 1.8, 3.0]
    b = ising.Batch(Ls, seeds, hot=True)
    try:
        b.set_plan(resident_max_L=0, resident_block=256, words_per_thread=wpt, tiled_block=block, sweeps_per_graph=3)
        E, M = (x.cpu().numpy() for x in b.sweep(Ts, 6, every=3, series=True))
        for i, (L, seed, T) in enumerate(zip(Ls, seeds, Ts)):
            s = oracle.init(L, seed, True)
            Es, Ms = oracle.sweep(s, seed, 0, 6, T, every=3)
            assert E[i].tolist() == Es.tolist() and M[i].tolist() == Ms.tolist(), L
            assert (b.spins(i) == s).all(), L
    finally:
        b.close()
