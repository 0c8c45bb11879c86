"""GPU parity of a single small lattice whose sweeps are applied from codes
drawn by the launch before: workgroups of one wavefront, of 64 to 1024 threads and
of two words per thread, the first lattice that is too large for them, more
sweeps than one launch takes, samples that cross launches, scans (whose
temperatures follow one another without a gap), graph capture and a change of
shape between calls.  Series, moments and state equal the oracle's bit for bit."""
import pytest

import oracle
import paper_1811_04384_amd as ising

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ising.load()


# words of a colour: 2, 8, 42, 63, 66, 128, 225, 260, 990, 1020, 1030, 2044 and (half-sweeps or tiles) 2058
@pytest.mark.parametrize("L", [4, 8, 42, 44, 64, 90, 104, 198, 204, 206, 292, 294])
def test_drawn_sweeps_match_oracle(L):
    print(f"drawn sweeps L={L}", flush=True)
    seed, T = 5, 2.3
    s = oracle.init(L, seed, True)
    lat = ising.Lattice(L, seed, hot=True)
    try:
        for n, every in ((1, 0), (7, 1), (1, 1), (20, 3)):
            t = lat.t
            if every:
                E, M = (x.cpu().numpy().tolist() for x in lat.sweep_measure(T, n, every))
                Es, Ms = oracle.sweep(s, seed, t, n, T, every=every)
                assert E == Es.tolist() and M == Ms.tolist(), (n, every)
            else:
                lat.sweep(T, n)
                oracle.sweep(s, seed, t, n, T)
            assert (lat.spins() == s).all() and lat.t == t + n, (n, every)
        # another shape, then none
        for shape in ((8, 256, 3), (0,)):
            lat.set_resident_tiles(*shape)
            t = lat.t
            lat.sweep(T, 4)
            oracle.sweep(s, seed, t, 4, T)
            assert (lat.spins() == s).all(), shape
    finally:
        lat.close()


@pytest.mark.parametrize("L,n", [(16, 600), (64, 257), (204, 300), (290, 140)])
def test_drawn_sweeps_across_launches(L, n):
    """More sweeps than a launch takes, the sampling interval no divisor of a launch's sweeps."""
    print(f"drawn sweeps across launches L={L}", flush=True)
    seed, T, every = 6, 2.1, 7
    s = oracle.init(L, seed, True)
    Es, Ms = oracle.sweep(s, seed, 0, n, T, every=every)
    lat = ising.Lattice(L, seed, hot=True)
    try:
        E, M = lat.sweep_measure(T, n, every)
        assert E.cpu().numpy().tolist() == Es.tolist() and M.cpu().numpy().tolist() == Ms.tolist()
        assert (lat.spins() == s).all()
    finally:
        lat.close()


@pytest.mark.parametrize("therm,meas", [(0, 5), (30, 0), (4, 6), (270, 9)])
def test_drawn_scan_matches_oracle(therm, meas):
    print(f"drawn scan {therm} {meas}", flush=True)
    L, seed, Ts = 64, 8, [1.7, 2.2, 2.9]
    lat = ising.Lattice(L, seed, hot=True)
    try:
        got = lat.scan(Ts, therm, meas, 2)
        want, s, t = oracle.scan(L, seed, True, Ts, therm, meas, 2)
        assert got == want and lat.t == t
        assert (lat.spins() == s).all()
        lat.sweep(2.0, 3)
        oracle.sweep(s, seed, t, 3, 2.0)
        assert (lat.spins() == s).all()
    finally:
        lat.close()


def test_drawn_sweeps_in_a_graph():
    """Captured sweeps replay at the captured sweep index: replayed on a restored state, with eager work between
    the replays, each gives the oracle's state."""
    import torch

    L, seed, T = 64, 9, 2.269
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        lat = ising.Lattice(L, seed, hot=True, stream=stream)
        try:
            lat.sweep(T, 3)
            start = lat.spins()
            graph = torch.cuda.CUDAGraph()
            stream.synchronize()
            with torch.cuda.graph(graph, stream=stream):
                lat.sweep(T, 600)
            s = start.copy()
            oracle.sweep(s, seed, 3, 600, T)
            for _ in range(3):
                lat.set_spins(start)
                graph.replay()
                assert (lat.spins() == s).all()
                lat.sweep(T, 2)
        finally:
            lat.close()
