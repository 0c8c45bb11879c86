"""What the library's host code does when something fails, without a GPU: its
sources are compiled with a stand-in HIP runtime (host_stub.cpp) that runs work
late and whose allocations and launches can be made to fail."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1811_04384_amd", "csrc")


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("stub") / "host_stub")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w",
                    "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    os.path.join(ROOT, "tests", "host_stub.cpp"), os.path.join(CSRC, "ising_server.cpp"),
                    os.path.join(CSRC, "ising_lattice.cpp"), os.path.join(CSRC, "ising_batch.cpp"), "-Wl,--unresolved-symbols=ignore-all", "-o", exe], check=True)

    def run(*args):
        out = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True, timeout=60)
        assert out.returncode == 0, out.stdout + out.stderr
        return out.stdout.split("\n")[:-1]

    return run


@pytest.mark.parametrize("sweeps", [
    (400, 50, 250),   # the small request, valid, is read back before either abandoned one
    (100, 100, 100),  # all of one quantum: valid and abandoned in one read-back, nothing left afterwards
    (400, 0, 0),
])
def test_server_runs_abandoned_requests_again(stub, sweeps):
    """A resident-tile launch whose waits expire leaves a state that is not its lattice's: that request, and no
    other, is run again without tiles, and a caller who stops when nothing is resident or queued has every result."""
    got = stub("abandon", *sweeps, 1)
    assert got[:3] == ["right 1", "right 2", "right 3"], got
    assert got[3].startswith("again 1 persist ") and not got[3].startswith("again 1 persist 0 "), got
    assert got[4] == "rewritten 0 wrong 0"
    # with the default bound nothing expires and nothing is run again
    plain = stub("abandon", *sweeps, 0)
    assert plain[:3] == ["right 1", "right 2", "right 3"] and plain[3].startswith("again 0 "), plain


@pytest.mark.parametrize("most", [1 << 30, (64 << 20) - 1, 1 << 20, 100000, 65536, 32768, 1024])
def test_server_serves_small_lattices_with_little_memory_left(stub, most):
    """However little memory is left for the codes of small lattices, no quantum fails, no group draws past the
    buffer (an address sanitizer watches) and every sweep is applied from its own codes."""
    got = stub("tight", most)
    assert got[:61] == [f"right {k}" for k in range(61)], got
    assert got[62] == "rewritten 0 wrong 0"


@pytest.mark.parametrize("quantum,first", [(100, 40), (20, 100)])  # large lattices in tiles; in half-sweep launches
def test_server_step_that_fails_half_way_leaves_no_staging_in_use(stub, quantum, first):
    """After a launch that fails anywhere in a step, copies enqueued before it have not run yet: the caller's next
    steps must not rewrite the host buffers they read, nor report a request twice."""
    for n in range(1, first):
        got = stub("halfway", n, quantum)
        assert got[-1] == "rewritten 0 wrong 0" and got[-2] == "failed 1" and "a result twice" not in got, (n, got)


def test_server_keeps_off_tiles_while_captured_ones_may_be_replayed(stub):
    """Tiles in a caller's graph are replayed in no order with the server's: none are launched while a handle holds
    such a graph's tiles, and they are again once it is gone or has set others."""
    assert stub("captured", 0) == ["captures 1", "right 1", "again 0 persist 0 halfsweeps 200", "captures 0", "right 2",
                                   "again 0 persist 1 halfsweeps 200", "rewritten 0 wrong 0"]
    assert stub("captured", 1) == ["captures 1", "right 1", "again 0 persist 1 halfsweeps 0", "captures 0", "right 2",
                                   "again 0 persist 2 halfsweeps 0", "rewritten 0 wrong 0"]


@pytest.mark.parametrize("plain", [0, 1])
def test_drawn_sweeps_that_fail_leave_the_counter_with_the_state(stub, plain):
    """A launch of drawn sweeps that fails: the sweep counter names the first sweep that the state lacks, and the
    calls after it go on from there."""
    for n in range(1, 5 if plain else 8):
        assert stub("drawn", plain, n) == ["ok t right", "failed t right", "ok t right", "rewritten 0 wrong 0"], n
    assert stub("drawn", plain, 0) == ["ok t right"] * 3 + ["rewritten 0 wrong 0"]


# L, strip columns of two kinds in turn: few words per strip and in all (lists), more (windows), or too many for either
@pytest.mark.parametrize("L,a,b,forms", [
    (84, 2, 12, (0, 0, 1)), (1008, 2, 36, (0, 1, 1)), (1008, 36, 2, (0, 1, 1)), (4200, 2, 4, (0, 0, 1)),
    (8064, 2, 2, (0, 0, 1)), (9072, 2, 2, (0, 1, 0)), (1008, 504, 2, (1, 0, 1)),
])
def test_strip_dynamics_with_little_memory_left(stub, L, a, b, forms):
    """Both forms that draw picks ahead use one buffer (48 MiB, allocated once, within which all they draw lies); and
    where the device has no room for it the form that needs none runs every shape."""
    names = ("phase", "draws", "lists")
    got = stub("strips", L, a, b, 1 << 30)
    assert got == ["allocations 1 " + " ".join(f"{n} {f}" for n, f in zip(names, forms)), "rewritten 0 wrong 0"]
    assert stub("strips", L, a, b, 48 << 20) == got
    assert stub("strips", L, a, b, (48 << 20) - 1) == ["allocations 0 phase 1 draws 0 lists 0", "rewritten 0 wrong 0"]


def test_samples_of_a_launch_at_any_interval(stub):
    """A sampling interval near 2^31 sweeps, and launches just before and over its end."""
    assert stub("samples") == ["bad 0 none 0 0", "rewritten 0 wrong 0"]


# tiles that a compute unit holds alone, lattices in 32 tiles each, whether they may run beside the half-sweeps
@pytest.mark.parametrize("per_cu,tiled,together", [
    (1, 8, 1), (2, 8, 1), (2, 9, 0), (2, 16, 0), (3, 16, 1), (3, 17, 0), (4, 16, 1), (4, 17, 0), (4, 32, 0),
])
def test_batch_runs_tiles_that_may_find_no_room_ahead_of_the_half_sweeps(stub, per_cu, tiled, together):
    """Tiles wait for each other, so all of a launch have to find room: beside other kernels no more than half of
    what a compute unit holds is sure to.  More run alone."""
    assert stub("beside", per_cu, tiled + 2, tiled) == [f"tiles 1 halfsweeps 20 beside {together}", "rewritten 0 wrong 0"]
