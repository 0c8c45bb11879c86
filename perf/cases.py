"""The work this library is used for, as cases that can be timed and checked.

Every case goes through the public Python entry points (``Lattice``,
``Batch``, ``Replicas``, ``Server``).  The listed cases are the library's own
workloads (``bench.py``, the README's examples) cut to a fraction of a second
and, between them, the smallest calls, ragged sizes (L not a multiple of 21),
hot and cold starts, sampled and unsampled sweeps, and lattices that are
written from and read back to the host.  ``draw`` gives more of the same
kinds over the same ranges.

One pass advances the lattices it is given, so a second pass on the same state
continues the chain.  All results are whole numbers fixed by the inputs
(L, seed, start, temperatures, sweeps).
"""
import math

import numpy as np
import torch

import paper_1811_04384_amd as ising

# the plan the autotuner settles on for mixed batches that fill the chip
TILED_PLAN = dict(resident_max_L=0, resident_block=256, words_per_thread=2, tiled_block=64, sweeps_per_graph=10)


def _resident_plan(L):
    """The heating scan's plan: resident tiles of 64 word columns, 200 sweeps per chunk."""
    return dict(resident_max_L=0, resident_block=256, words_per_thread=1, tiled_block=64, sweeps_per_graph=200,
                tile_max_L=L, tile_sweeps=1, tile_cols=64, tile_block=1024, tile_exchange=1)


def listed():
    return [
        # the smallest call a program makes: a few sampled sweeps of one small
        # lattice (a plot that is updated live, a step of a caller's own loop)
        {"name": "call_L64", "kind": "single", "L": 64, "hot": False, "T": 2.0, "sweeps": 20, "every": 1},
        # the README's temperature scan of one L = 64 lattice, shortened
        {"name": "scan_L64", "kind": "scan", "L": 64, "hot": True, "T0": 1.5, "T1": 3.5, "n_T": 5, "therm": 200,
         "meas": 200, "every": 1},
        # a checkpointed run of a mid-size lattice (N = 48): spins from the
        # host, a sampled run, spins back to the host
        {"name": "restart_L1008", "kind": "restart", "L": 1008, "T": 2.269, "sweeps": 200, "every": 1},
        # the plain single-lattice workload: E/M every 10 sweeps at T_c
        {"name": "plain_L4096", "kind": "single", "L": 4096, "hot": True, "T": 2.269, "sweeps": 300, "every": 10},
        # a large ragged lattice (L = 21 * 476 + 2), sampled
        {"name": "ragged_L9998", "kind": "single", "L": 9998, "hot": True, "T": 2.6, "sweeps": 20, "every": 5},
        # the headline: fresh hot start of L = 32768, unsampled sweeps, final E and M
        {"name": "headline_L32768", "kind": "fresh", "L": 32768, "T": 2.269, "sweeps": 20},
        # the small-lattice temperature scan as one batch: 8 temperatures, the whole series kept
        {"name": "batch_8xL64", "kind": "batch", "L0": 64, "L1": 64, "n": 8, "hot": False, "sweeps": 500, "every": 1,
         "series": True, "plan": "default"},
        # the heating scan: 16 replicas of L = 1008 carried over the temperatures, exact moments
        {"name": "heating_16xL1008", "kind": "heating", "L": 1008, "n": 16, "T0": 2.2, "T1": 2.3, "n_T": 2, "therm": 50,
         "meas": 100, "every": 1},
        # the mixed batch: L = 256 ... 2048, 32 temperatures, E/M every 10
        {"name": "mixed_batch", "kind": "batch", "L0": 256, "L1": 2048, "n": 256, "hot": True, "sweeps": 20, "every": 10,
         "series": False, "plan": "tiled"},
        # the paper's own dynamics on its Table 2 lattice (N = 96), the energy after every iteration
        {"name": "strips_L2016", "kind": "strips", "L": 2016, "cols": 2, "T": 2.269, "iterations": 20, "every": 1},
        # 21 temperatures in one word lattice, sampled
        {"name": "replicas_L2048", "kind": "replicas", "L": 2048, "sweeps": 20, "every": 5},
        # a served burst of requests of mixed sizes and lengths
        {"name": "served_16", "kind": "served", "n": 16, "p0": 7, "p1": 12, "sweeps0": 50, "sweeps1": 500,
         "quantum": 100},
    ]


# Largest number of spin-flip attempts of a drawn case (the headline's).
MOST_ATTEMPTS = 20 * 32768 ** 2


def _even(rng, lo, hi):
    """An even size, spread over the logarithm of [lo, hi]."""
    L = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, L - L % 2))


def _count(rng, lo, hi, cap):
    return max(1, min(int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))), int(cap)))


def draw(rng):
    kind = rng.choice(["single", "single", "single", "scan", "restart", "fresh", "batch", "batch", "heating", "strips",
                       "replicas", "served"])
    T = round(rng.uniform(1.2, 3.5), 3)
    if kind == "single":
        L = _even(rng, 16, 16384)
        sweeps = _count(rng, 10, 1000, 4e9 / L ** 2)
        return {"kind": kind, "L": L, "hot": rng.random() < 0.5, "T": T, "sweeps": sweeps,
                "every": rng.choice([1, 1, 3, 10])}
    if kind == "scan":
        L = _even(rng, 16, 512)
        return {"kind": kind, "L": L, "hot": rng.random() < 0.5, "T0": 1.5, "T1": 3.5, "n_T": rng.randint(2, 4),
                "therm": rng.choice([0, 50, 100]), "meas": _count(rng, 20, 200, 200), "every": rng.choice([1, 5])}
    if kind == "restart":
        L = _even(rng, 64, 2048)
        return {"kind": kind, "L": L, "T": T, "sweeps": _count(rng, 10, 300, 1e9 / L ** 2), "every": rng.choice([1, 5])}
    if kind == "fresh":
        L = _even(rng, 2048, 32768)
        return {"kind": kind, "L": L, "T": T, "sweeps": _count(rng, 5, 500, MOST_ATTEMPTS / L ** 2)}
    if kind == "batch":
        if rng.random() < 0.5:  # small lattices
            L0 = _even(rng, 16, 128)
            return {"kind": kind, "L0": L0, "L1": L0, "n": _count(rng, 2, 256, 256), "hot": rng.random() < 0.5,
                    "sweeps": _count(rng, 50, 1000, 600), "every": rng.choice([1, 10]),
                    "series": rng.random() < 0.5, "plan": "default"}
        return {"kind": kind, "L0": rng.choice([64, 128, 256]), "L1": rng.choice([512, 1024, 2048]),
                "n": rng.randint(16, 256), "hot": True, "sweeps": rng.choice([10, 20, 30]), "every": 10,
                "series": rng.random() < 0.5, "plan": rng.choice(["default", "tiled"])}
    if kind == "heating":
        L = _even(rng, 256, 1008)
        return {"kind": kind, "L": L, "n": rng.randint(2, 16), "T0": 1.5, "T1": 3.5, "n_T": rng.randint(2, 3),
                "therm": rng.choice([0, 20, 50]), "meas": rng.randint(20, 100), "every": rng.choice([1, 5])}
    if kind == "strips":
        cols = rng.choice([2, 2, 4, 6])
        L = 12 * rng.randint(7, 168)
        return {"kind": kind, "L": L, "cols": cols, "T": T, "iterations": rng.randint(2, 12), "every": rng.choice([1, 2])}
    if kind == "replicas":
        L = _even(rng, 64, 4096)
        return {"kind": kind, "L": L, "sweeps": _count(rng, 5, 100, 2e8 / L ** 2), "every": rng.choice([1, 5])}
    n, p1 = rng.randint(4, 24), rng.choice([10, 11, 12])
    return {"kind": "served", "n": n, "p0": rng.choice([6, 7, 8]), "p1": p1, "sweeps0": 20,
            "sweeps1": _count(rng, 50, 500, MOST_ATTEMPTS / (n * 4 ** p1)), "quantum": rng.choice([50, 100, 200])}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _temperatures(case):
    return [case["T0"] + (case["T1"] - case["T0"]) * j / max(1, case["n_T"] - 1) for j in range(case["n_T"])]


def _batch_lattices(case, seed):
    """Sizes, seeds and temperatures of a batch: L doubling from L0 to L1 in
    turn, 32 temperatures over [1.5, 3.5]."""
    sizes = [case["L0"]]
    while sizes[-1] * 2 <= case["L1"]:
        sizes.append(sizes[-1] * 2)
    n = case["n"]
    steps = min(32, max(2, n // len(sizes)))
    Ls = [sizes[i % len(sizes)] for i in range(n)]
    Ts = [1.5 + 2.0 * ((i // len(sizes)) % steps) / (steps - 1) for i in range(n)]
    return Ls, [1000 * seed + i for i in range(n)], Ts


def _host_spins(L, seed):
    """A checkpoint's spins: domains of 8 x 8 with 5 % noise."""
    r = np.random.default_rng(seed)
    b = (L + 7) // 8
    s = np.repeat(np.repeat(r.integers(0, 2, (b, b), dtype=np.uint8), 8, axis=0), 8, axis=1)[:L, :L]
    return np.ascontiguousarray(s ^ (r.random((L, L)) < 0.05).astype(np.uint8))


def _requests(case, seed):
    r = np.random.default_rng(seed)
    return [(i, int(2 ** r.integers(case["p0"], case["p1"] + 1)), float(r.uniform(1.5, 3.5)),
             int(r.integers(case["sweeps0"], case["sweeps1"] + 1)), 1000 * seed + i) for i in range(case["n"])]


def _replica_temperatures():
    return [round(1.5 + 0.1 * k, 10) for k in range(ising.REPLICAS)]


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("single", "scan"):
        return case, ising.Lattice(case["L"], seed, hot=case["hot"])
    if kind == "fresh":
        return case, ising.Lattice(case["L"], seed, hot=True), seed
    if kind == "restart":
        return case, ising.Lattice(case["L"], seed, hot=False), _host_spins(case["L"], seed)
    if kind == "batch":
        Ls, seeds, Ts = _batch_lattices(case, seed)
        b = ising.Batch(Ls, seeds, hot=case["hot"])
        if case["plan"] == "tiled":
            b.set_plan(**TILED_PLAN)
        return case, b, Ts
    if kind == "heating":
        b = ising.Batch([case["L"]] * case["n"], [1000 * seed + i for i in range(case["n"])], hot=False)
        b.set_plan(**_resident_plan(case["L"]))
        return case, b
    if kind == "strips":
        return case, ising.Lattice(case["L"], seed, hot=True)
    if kind == "replicas":
        return case, ising.Replicas(case["L"], seed, hot=True)
    return case, ising.Server(hbm_budget=1 << 30, max_slots=128, quantum_sweeps=case["quantum"]), _requests(case, seed)


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

_MOMENTS = ("n_samples", "sum_E", "sum_E2", "sum_absM", "sum_M2", "sum_M4")


def _moments(rows):
    """Exact moment sums as signed 64-bit numbers: each wide sum in limbs of 62 bits."""
    low = (1 << 62) - 1
    return np.array([[[m[k] & low if k not in ("n_samples", "sum_E", "sum_absM") else m[k] for k in _MOMENTS] +
                      [m[k] >> 62 & low for k in ("sum_E2", "sum_M2", "sum_M4")] + [m["sum_M4"] >> 124]
                      for m in row] for row in rows], dtype=np.int64)


def run(state):
    case = state[0]
    kind = case["kind"]
    if kind == "single":
        lat = state[1]
        E, M = lat.sweep_measure(case["T"], case["sweeps"], case["every"])
        return {"words": lat.words, "E": E, "M": M}
    if kind == "scan":
        lat = state[1]
        rows = lat.scan(_temperatures(case), case["therm"], case["meas"], case["every"])
        return {"words": lat.words, "moments": _moments([rows])}
    if kind == "fresh":
        lat = state[1]
        lat.reset(state[2], hot=True)
        lat.sweep(case["T"], case["sweeps"])
        E, M = lat.observables()
        return {"words": lat.words, "E": E, "M": M}
    if kind == "restart":
        lat = state[1]
        lat.set_spins(state[2])
        lat.t = 0
        E, M = lat.sweep_measure(case["T"], case["sweeps"], case["every"])
        return {"spins": lat.spins(), "E": E, "M": M}
    if kind == "batch":
        b = state[1]
        if case["series"]:
            E, M = b.sweep(state[2], case["sweeps"], case["every"], series=True)
            return {"E": E, "M": M}
        b.sweep(state[2], case["sweeps"], case["every"])
        return b.results()
    if kind == "heating":
        return _moments(state[1].scan(_temperatures(case), case["therm"], case["meas"], case["every"]))
    if kind == "strips":
        lat = state[1]
        E, M = lat.random_iterations(case["T"], case["cols"], case["iterations"], case["every"])
        return {"words": lat.words, "E": E, "M": M}
    if kind == "replicas":
        return state[1].sweep_measure(_replica_temperatures(), case["sweeps"], case["every"])
    srv = state[1]
    for rid, L, T, sweeps, lattice_seed in state[2]:
        srv.submit(rid, L, T, sweeps, seed=lattice_seed)
    got = []
    while len(got) < len(state[2]):
        srv.step()
        got += srv.poll()
    got.sort(key=lambda r: r["req_id"])
    return np.array([[r["req_id"], r["E"], r["M"]] for r in got], dtype=np.int64)


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _word_bytes(L):
    return ising.ising_required_bytes(L)


def _attempts(case):
    kind = case["kind"]
    if kind in ("single", "fresh", "restart"):
        return case["L"] ** 2 * case["sweeps"]
    if kind == "scan":
        return case["L"] ** 2 * case["n_T"] * (case["therm"] + case["meas"])
    if kind == "batch":
        return sum(L * L for L in _batch_lattices(case, 0)[0]) * case["sweeps"]
    if kind == "heating":
        return case["n"] * case["L"] ** 2 * case["n_T"] * (case["therm"] + case["meas"])
    if kind == "strips":
        return 10 * case["L"] ** 2 * case["iterations"]
    if kind == "replicas":
        return ising.REPLICAS * case["L"] ** 2 * case["sweeps"]
    return sum(L * L * sweeps for _, L, _, sweeps, _ in _requests(case, 0))


def work(case):
    """Bytes: the packed lattices read once and written once, the samples
    written.  Operations: 18 integer lane operations per spin-flip attempt (a
    quarter of a ten-round Philox4x32 block, two comparisons, the bit-sliced
    neighbour count)."""
    kind = case["kind"]
    if kind == "batch":
        Ls = _batch_lattices(case, 0)[0]
        moved = 2 * sum(map(_word_bytes, Ls)) + 16 * len(Ls) * (case["sweeps"] // case["every"])
    elif kind == "heating":
        moved = 2 * case["n"] * _word_bytes(case["L"])
    elif kind == "replicas":
        moved = 2 * 8 * case["L"] ** 2 + 16 * ising.REPLICAS * (case["sweeps"] // case["every"])
    elif kind == "served":
        moved = sum(_word_bytes(L) for _, L, _, _, _ in _requests(case, 0))
    elif kind == "restart":
        moved = 2 * case["L"] ** 2 + 2 * _word_bytes(case["L"]) + 16 * (case["sweeps"] // case["every"])
    elif kind == "fresh":
        moved = _word_bytes(case["L"])
    else:
        moved = 2 * _word_bytes(case["L"]) + (16 * (case["sweeps"] // case["every"]) if kind == "single" else 0)
    return {"bytes": moved, "flops": 18.0 * _attempts(case)}


# ---------------------------------------------------------------------------
# the same results from plain numpy, site by site
# ---------------------------------------------------------------------------

def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 (Salmon et al., SC'11) on arrays of counters."""
    c = [np.asarray(x, dtype=np.uint64) for x in np.broadcast_arrays(c0, c1, c2, c3)]
    m32 = np.uint64(0xFFFFFFFF)
    s32 = np.uint64(32)
    for r in range(10):
        a = c[0] * np.uint64(0xD2511F53)
        b = c[2] * np.uint64(0xCD9E8D57)
        k = [np.uint64((k0 + r * 0x9E3779B9) & 0xFFFFFFFF), np.uint64((k1 + r * 0xBB67AE85) & 0xFFFFFFFF)]
        c = [(b >> s32) ^ c[1] ^ k[0], b & m32, (a >> s32) ^ c[3] ^ k[1], a & m32]
    return np.stack(c)


class _Sites:
    """The counters of every site of an L x L lattice: word row and position
    of its row, and which output of which block serves it."""

    def __init__(self, L):
        self.L = L
        self.N = ising.ising_word_rows(L)
        r, c = np.indices((L, L))
        self.I, p = r % self.N, r // self.N
        shared = p == 20  # position 20 of four words of a colour shares block 5
        self.col = np.where(shared, 8 * (c // 8) + c % 2, c)
        self.block = np.where(shared, 5, p // 4)
        self.out = np.where(shared, (c // 2) % 4, p % 4)
        self.colour = (self.I + c) % 2

    def uniforms(self, mask, t, stream, seed):
        u = _philox(t & 0xFFFFFFFF, self.I[mask] * self.L + self.col[mask], t >> 32, self.block[mask] + 8 * stream,
                    seed & 0xFFFFFFFF, seed >> 32)
        return np.take_along_axis(u, self.out[mask][None], axis=0)[0]

    def start(self, seed, hot):
        s = np.ones((self.L, self.L), dtype=bool)
        if hot:
            s[:] = self.uniforms(s, 0, 0, seed).reshape(self.L, self.L) < 1 << 31
        return s

    def sweep(self, s, seed, t, T):
        t4, t8 = (min((1 << 32) - 1, int(math.exp(-d / T) * 4294967296.0)) for d in (4.0, 8.0))
        for colour in (0, 1):
            mask = self.colour == colour
            u = self.uniforms(mask, t, 1, seed)
            n = sum((s != np.roll(s, k, axis=a)).astype(int) for k in (1, -1) for a in (0, 1))[mask]
            s[mask] ^= (n >= 2) | ((n == 1) & (u < t4)) | ((n == 0) & (u < t8))

    def energy(self, s):
        anti = int((s != np.roll(s, 1, axis=0)).sum()) + int((s != np.roll(s, 1, axis=1)).sum())
        return 2 * anti - 2 * self.L ** 2, 2 * int(s.sum()) - self.L ** 2

    def words(self, s):
        w = np.zeros((self.N, self.L), dtype=np.int64)
        for r in range(self.L):
            w[r % self.N] |= s[r].astype(np.int64) << (3 * (20 - r // self.N))
        return w.reshape(-1)


def _series(sites, s, seed, t, T, sweeps, every):
    E, M = [], []
    for k in range(1, sweeps + 1):
        sites.sweep(s, seed, t + k - 1, T)
        if every and k % every == 0:
            e, m = sites.energy(s)
            E.append(e)
            M.append(m)
    return E, M


def _moments_of(E, M):
    return {"n_samples": len(E), "sum_E": sum(E), "sum_E2": sum(e * e for e in E), "sum_absM": sum(map(abs, M)),
            "sum_M2": sum(m * m for m in M), "sum_M4": sum(m ** 4 for m in M)}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("strips", "replicas", "served") or _attempts(case) > 1.2e7:
        return None
    if kind == "batch":
        Ls, seeds, Ts = _batch_lattices(case, seed)
        got = []
        for L, own, T in zip(Ls, seeds, Ts):
            sites = _Sites(L)
            s = sites.start(own, case["hot"])
            got.append(_series(sites, s, own, 0, T, case["sweeps"], case["every"]) + (sites.energy(s),))
        if case["series"]:
            return {"E": np.array([g[0] for g in got]), "M": np.array([g[1] for g in got])}
        return {"E": np.array([g[2][0] for g in got]), "M": np.array([g[2][1] for g in got]),
                "sum_E": np.array([sum(g[0]) for g in got]), "sum_absM": np.array([sum(map(abs, g[1])) for g in got]),
                "n_samples": np.array([len(g[0]) for g in got])}
    if kind == "heating":
        sites = _Sites(case["L"])
        lattices = [sites.start(1000 * seed + i, False) for i in range(case["n"])]
        rows, t = [], 0
        for T in _temperatures(case):
            row = []
            for i, s in enumerate(lattices):
                _series(sites, s, 1000 * seed + i, t, T, case["therm"], 0)
                row.append(_moments_of(*_series(sites, s, 1000 * seed + i, t + case["therm"], T, case["meas"],
                                                case["every"])))
            rows.append(row)
            t += case["therm"] + case["meas"]
        return _moments(rows)
    sites = _Sites(case["L"])
    if kind == "scan":
        s = sites.start(seed, case["hot"])
        row, t = [], 0
        for T in _temperatures(case):
            _series(sites, s, seed, t, T, case["therm"], 0)
            row.append(_moments_of(*_series(sites, s, seed, t + case["therm"], T, case["meas"], case["every"])))
            t += case["therm"] + case["meas"]
        return {"words": sites.words(s), "moments": _moments([row])}
    if kind == "restart":
        s = _host_spins(case["L"], seed).astype(bool)
        E, M = _series(sites, s, seed, 0, case["T"], case["sweeps"], case["every"])
        return {"spins": s.astype(np.uint8), "E": np.array(E), "M": np.array(M)}
    s = sites.start(seed, case.get("hot", True))
    E, M = _series(sites, s, seed, 0, case["T"], case["sweeps"], case.get("every", 0))
    if kind == "fresh":
        E, M = sites.energy(s)
        return {"words": sites.words(s), "E": E, "M": M}
    return {"words": sites.words(s), "E": np.array(E, dtype=np.int64), "M": np.array(M, dtype=np.int64)}
