// Continuous-batching server: requests of different L, T and sweep counts
// share the GPU.  Their packed lattices and sweep counters stay resident in
// one device arena; every quantum advances all resident lattices together
// (large lattices in shared half-sweep launches, or one after the other in
// resident tiles where they are few; small ones one workgroup each from codes
// drawn by the whole chip), and requests join and leave between quanta.  Admission is by
// memory footprint (first-fit in the arena) and free slots, in arrival order.
//
// Pipelining: the host plans, uploads and enqueues quantum q+1 while quantum
// q runs (at most two quanta in flight).  Bookkeeping counts sweeps when they
// are enqueued; a request whose last quantum has been enqueued has its E/M
// reduction and read-back enqueued right behind it into a pinned ring entry,
// and its slot and arena range are reused at once (stream order puts any
// later use after the read-back).  Results are harvested when their event
// has completed.
//
// A resident-tile launch can be abandoned (its tiles wait for each other, at
// most a second, and something else may hold the device for longer).  It then
// marks its own lattice's state, and nothing else; the mark comes back with the
// lattice's E and M, and its request goes through the queue once more, from its
// start and without tiles.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <deque>
#include <new>
#include <vector>

#include "ising_host.hpp"
#include "ising_launch.hpp"
#include "ising_sched.hpp"

using namespace ising;

namespace {

// Acceptance codes of the small lattices held at once (a device buffer, made when
// first needed): small lattices go in groups of which it holds at least eight
// sweeps (about 300 of L = 256, and 157 sweeps of 16 of them).  Where the device has
// no 64 MB left the buffer and the groups are smaller, down to a sweep of one
// lattice (3584 words at L = 256), whose room a server has from its creation on: a
// quantum never fails for want of it.
constexpr int64_t kServerCodeWords = int64_t(8) << 20;
constexpr int64_t kServerCodeWordsLeast = 4096;
constexpr int64_t kServerGroupWords = kServerCodeWords / 8;

// Large lattices in resident tiles, one after the other, in a quantum: at most so
// many, of so many columns, and the tiles of each.
constexpr int32_t kServerTiled = 8;
constexpr int32_t kServerTiledMaxL = 4096;
constexpr int32_t kServerTiles = 256;
constexpr int32_t kServerTileSweeps = 4096;  // of one launch

// us of `sweeps` sweeps of a lattice in resident tiles (2.3 a sweep at L = 300, 2.6 at
// 1024, 3.5 at 2048, 5.6 at 3072, 7.6 at 4096, and 50 to set a launch up), and of
// a half-sweep launch of n wavefronts of one word per thread (3.3 with 100, 3.7
// with 392, 4.7 with 1568, 8.6 with 6272, 17 with 24232 in half as many of two).
double tiled_us(int32_t L, int64_t sweeps) { return 50.0 + (double)sweeps * (2.2 + (double)L * L / 3.1e6); }
double halfsweep_us(int64_t n) {
    return 3.3 + 0.0008 * (double)std::min<int64_t>(n, 8192) + 0.0005 * (double)std::max<int64_t>(n - 8192, 0);
}

// A group: entries [begin, end) of the quantum's table of small lattices.
struct SmallGroup {
    int32_t begin, end;
    int64_t words;       // of its lattices
    int32_t max_NL, max_words, max_draws, K;  // the largest lattice's words, words of a colour, draw items; sweeps
};
constexpr int kServerTiledBlock = 64;  // threads of a half-sweep workgroup
constexpr uint64_t kWaitTicks = 100000000;  // one second of the 100 MHz clock
constexpr int kStages = 2;     // quanta in flight = staging buffer sets
constexpr int kRing = 4;       // read-back ring entries

double now_s() {
    return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

// Host staging of one quantum's tables (pinned), reusable once `done` fired.
struct Stage {
    LatticeDesc* desc = nullptr;
    WaveItem* waves = nullptr;
    int64_t waves_cap = 0;
    DrawLat* draw = nullptr;
    PersistTile* tiles = nullptr;
    hipEvent_t done = nullptr;  // recorded after the quantum's kernels
    bool used = false;
};

// A finished request, and when it was admitted.
struct Finished {
    Request req;
    double t_admit;
};

// One batch of finished requests whose E/M read-back is in flight.
struct Readback {
    int32_t* ids = nullptr;  // pinned: slot ids uploaded for the reduction
    int64_t* em = nullptr;   // pinned: kObservedWords per listed slot
    hipEvent_t done = nullptr;
    bool pending = false;
    std::vector<Finished> requests;
};

}  // namespace

struct ising_server {
    Scheduler sched;
    hipStream_t stream = nullptr;
    hipStream_t side = nullptr;  // resident (small-lattice) work runs beside the tiled launches
    hipEvent_t fork_ev = nullptr, join_ev = nullptr;
    int device = 0;
    uint8_t* arena = nullptr;
    LatticeDesc* d_desc = nullptr;
    LatticeState* d_state = nullptr;
    WaveItem* d_waves = nullptr;
    int64_t d_waves_cap = 0;
    DrawLat* d_draw = nullptr;  // small lattices of the current quantum
    // their acceptance codes: the buffer of kServerCodeWordsLeast words, and the one in use
    uint64_t* d_codes_least = nullptr;
    uint64_t* d_codes = nullptr;
    int64_t code_words = 0;
    int cus = 0;
    // resident tiles (set up when first wanted): the quantum's tables; one word
    // per tile and the exchange buffer
    enum { kTilesUnknown, kTilesUsable, kTilesNot } tiles = kTilesUnknown;
    PersistTile* d_tiles = nullptr;
    uint64_t* d_exch = nullptr;
    uint64_t wait_ticks = kWaitTicks;  // bound of each wait of the tiles, 100 MHz clock ticks
    int32_t* d_fin = nullptr;  // ids of a read-back batch
    int64_t* d_em = nullptr;   // kObservedWords per lattice of a read-back batch
    Stage stage[kStages];
    int next_stage = 0;
    std::deque<hipEvent_t> inflight;  // quantum events, oldest first
    Readback ring[kRing];
    int next_ring = 0;  // entry the next batch uses = oldest entry
    size_t lds_limit = 0;
    int32_t resident_max_L = 256;
    std::vector<ising_result> done;

    ising_server(size_t budget, int32_t slots, int32_t quantum) : sched(budget, slots, quantum) {}
};

namespace {

void release(ising_server* s) {
    if (!s) return;
    if (s->arena) (void)hipFree(s->arena);
    if (s->d_desc) (void)hipFree(s->d_desc);
    if (s->d_state) (void)hipFree(s->d_state);
    if (s->d_waves) (void)hipFree(s->d_waves);
    if (s->d_draw) (void)hipFree(s->d_draw);
    if (s->d_codes && s->d_codes != s->d_codes_least) (void)hipFree(s->d_codes);
    if (s->d_codes_least) (void)hipFree(s->d_codes_least);
    if (s->d_tiles) (void)hipFree(s->d_tiles);
    if (s->d_exch) (void)hipFree(s->d_exch);
    if (s->d_fin) (void)hipFree(s->d_fin);
    if (s->d_em) (void)hipFree(s->d_em);
    for (Stage& st : s->stage) {
        if (st.desc) (void)hipHostFree(st.desc);
        if (st.waves) (void)hipHostFree(st.waves);
        if (st.draw) (void)hipHostFree(st.draw);
        if (st.tiles) (void)hipHostFree(st.tiles);
        if (st.done) (void)hipEventDestroy(st.done);
    }
    for (Readback& r : s->ring) {
        if (r.ids) (void)hipHostFree(r.ids);
        if (r.em) (void)hipHostFree(r.em);
        if (r.done) (void)hipEventDestroy(r.done);
    }
    for (hipEvent_t e : s->inflight) (void)hipEventDestroy(e);
    if (s->fork_ev) (void)hipEventDestroy(s->fork_ev);
    if (s->join_ev) (void)hipEventDestroy(s->join_ev);
    if (s->side) (void)hipStreamDestroy(s->side);
    delete s;
}

// Move a completed read-back batch into the finished list (an abandoned request
// back into the queue).  wait: block on its event; otherwise only if it has
// already completed.
int harvest(ising_server* s, Readback& r, bool wait) {
    if (!r.pending) return ISING_OK;
    if (wait) {
        ISING_HIP(hipEventSynchronize(r.done));
    } else {
        const hipError_t e = hipEventQuery(r.done);
        if (e == hipErrorNotReady) return ISING_OK;
        if (e != hipSuccess) return hip_fail(e, "hipEventQuery");
    }
    const double t = now_s();
    std::vector<Request> again;
    for (size_t k = 0; k < r.requests.size(); ++k) {
        const Request& q = r.requests[k].req;
        const int64_t* em = r.em + kObservedWords * k;
        if (em[2]) {
            again.push_back(q);
            again.back().no_tiles = true;
            continue;
        }
        ising_result res;
        res.req_id = q.id;
        res.L = q.L;
        res.status = ISING_OK;
        res.T = q.T;
        res.sweeps = q.sweeps;
        res.E = em[0];
        res.M = em[1];
        res.t_submit_s = q.t_submit;
        res.t_admit_s = r.requests[k].t_admit;
        res.t_done_s = t;
        s->done.push_back(res);
    }
    s->sched.requeue(again);
    r.requests.clear();
    r.pending = false;
    return ISING_OK;
}

// Harvest in submission order (oldest ring entry first); stop at the first
// batch that is not ready unless `wait`.
int harvest_all(ising_server* s, bool wait) {
    for (int k = 0; k < kRing; ++k) {
        Readback& r = s->ring[(s->next_ring + k) % kRing];
        int rc = harvest(s, r, wait);
        if (rc != ISING_OK) return rc;
        if (r.pending) break;
    }
    return ISING_OK;
}

int grow_waves(ising_server* s, Stage& st, int64_t need) {
    if (need > st.waves_cap) {
        const int64_t cap = std::max<int64_t>(need, 2 * st.waves_cap);
        if (st.waves) (void)hipHostFree(st.waves);
        st.waves = nullptr;
        st.waves_cap = 0;
        ISING_HIP(hipHostMalloc(&st.waves, sizeof(WaveItem) * cap, hipHostMallocDefault));
        st.waves_cap = cap;
    }
    if (need > s->d_waves_cap) {
        // earlier quanta read the device table: let them finish before replacing it
        ISING_HIP(hipStreamSynchronize(s->stream));
        const int64_t cap = std::max<int64_t>(need, 2 * s->d_waves_cap);
        if (s->d_waves) (void)hipFree(s->d_waves);
        s->d_waves = nullptr;
        s->d_waves_cap = 0;
        ISING_HIP(hipMalloc(&s->d_waves, sizeof(WaveItem) * cap));
        s->d_waves_cap = cap;
    }
    return ISING_OK;
}

int admit_queued(ising_server* s) {
    const std::vector<int32_t> adm = s->sched.admit(now_s());
    for (int32_t i : adm) {
        const Slot& sl = s->sched.slots()[i];
        const Geometry g = make_geometry(sl.req.L);
        ISING_HIP(launch_init(reinterpret_cast<uint64_t*>(s->arena + sl.off), g, sl.req.seed, sl.req.init, s->stream));
        ISING_HIP(hipMemsetAsync(s->d_state + i, 0, sizeof(LatticeState), s->stream));
    }
    return ISING_OK;
}

// (at most 27 KB of LDS, which every launch may use)
bool is_resident(const ising_server* s, const Geometry& g) {
    return g.L <= s->resident_max_L && (size_t)g.N * g.L * 8 <= s->lds_limit;
}

// Whether resident tiles can be used: the device holds those of the largest
// lattice at once and the buffers could be had.
bool tiles_usable(ising_server* s) {
    if (s->tiles != ising_server::kTilesUnknown) return s->tiles == ising_server::kTilesUsable;
    s->tiles = ising_server::kTilesNot;
    const Geometry big = make_geometry(kServerTiledMaxL);
    int32_t w, block;
    default_resident_shape(big, &w, &block);
    const size_t lds = persist_lds_bytes(big.L, big.N, w, block);
    int64_t capacity = 0;
    if (lds > persist_lds_limit(s->device)) return false;
    // (smaller lattices need less than the largest one, and no leave)
    hipError_t e = allow_persist_lds(s->device, persist_form(big.L, big.N, w, block), lds);
    if (e == hipSuccess) e = persist_capacity(block, lds, s->device, &capacity);
    if (e == hipSuccess && capacity >= kServerTiles) {
        e = hipMalloc(&s->d_tiles, sizeof(PersistTile) * kServerTiled * kServerTiles);
        if (e == hipSuccess)
            e = hipMalloc(&s->d_exch, sizeof(uint64_t) * (kServerTiles + (size_t)kServerTiles * 4 * (size_t)big.N));
        for (Stage& st : s->stage)
            if (e == hipSuccess)
                e = hipHostMalloc(&st.tiles, sizeof(PersistTile) * kServerTiled * kServerTiles, hipHostMallocDefault);
        if (e == hipSuccess) s->tiles = ising_server::kTilesUsable;
    }
    if (e != hipSuccess) (void)hipGetLastError();
    return s->tiles == ising_server::kTilesUsable;
}

// Sweeps of a group whose codes are drawn together.
int32_t group_sweeps(const ising_server* s, const SmallGroup& gr) {
    return (int32_t)std::min<int64_t>(gr.K, s->code_words / gr.words);
}

// The buffer of the small lattices' codes, once: the largest that can be had.
void code_buffer(ising_server* s) {
    if (s->d_codes) return;
    for (int64_t words = kServerCodeWords; words > kServerCodeWordsLeast; words /= 2) {
        if (hipMalloc(&s->d_codes, sizeof(uint64_t) * (size_t)words) == hipSuccess) {
            s->code_words = words;
            return;
        }
        (void)hipGetLastError();
    }
    s->d_codes = s->d_codes_least;
    s->code_words = kServerCodeWordsLeast;
}

// Words of a group of small lattices, at most (of more than one lattice).
int64_t group_words(const ising_server* s) {
    return std::min(kServerGroupWords, std::max(s->code_words / 8, kServerCodeWordsLeast));
}

// Plan the next quantum, upload its tables through a staging set and enqueue
// its kernels.  Descriptors cover every active slot (those already done with
// zero sweeps, so the read-back that follows can use them).
int enqueue_quantum(ising_server* s) {
    Scheduler& sc = s->sched;
    sc.plan_quantum();
    const int32_t slots = (int32_t)sc.slots().size();
    Stage& st = s->stage[s->next_stage];
    s->next_stage = (s->next_stage + 1) % kStages;
    if (st.used) ISING_HIP(hipEventSynchronize(st.done));  // its previous copies have been read
    int64_t n_waves = 0;
    for (int32_t i = 0; i < slots; ++i) {
        const Slot& sl = sc.slots()[i];
        if (!sl.active || sl.planned <= 0) continue;
        const Geometry g = make_geometry(sl.req.L);
        if (!is_resident(s, g)) n_waves += waves_per_colour(g, 1);
    }
    // Few large lattices leave a launch per half-sweep mostly waiting for the next:
    // then they go through the quantum one after the other in resident tiles.  The
    // estimates above say which is less; us for 300 sweeps in quanta of 100, half-sweeps /
    // tiles: L = 512 2001/878, 2048 2813/1317, 4096 5181/2665, 2048 and 1024 and 512
    // 3091/2776; three of 1024 2544/2633, four of 512 2171/2156.
    double tiled = 0.0, swept = 0.0;
    int32_t n_large = 0;
    for (int32_t i = 0; i < slots; ++i) {
        const Slot& sl = sc.slots()[i];
        if (!sl.active || sl.planned <= 0) continue;
        const Geometry g = make_geometry(sl.req.L);
        if (is_resident(s, g)) continue;
        n_large += 1;
        tiled += g.L <= kServerTiledMaxL && !sl.req.no_tiles ? tiled_us(g.L, sl.planned) : 1e300;
        swept = std::max(swept, 2.0 * (double)sl.planned * halfsweep_us(n_waves));
    }
    // Not while a caller's graph may replay a lattice's resident tiles beside them, in
    // no order with these: each could wait for compute units that the other holds.
    const bool tiles = n_large > 0 && n_large <= kServerTiled && tiled < swept && resident_captures(s->device) == 0 &&
                       tiles_usable(s);
    if (tiles) n_waves = 0;
    struct Tiled {
        int32_t lattice, first, count, w, block, K;
    };
    std::vector<Tiled> large;
    // two words per thread where one would be more wavefronts than the device holds
    // at once (bursts of 16 requests of L = 128 ... 4096, six seeds: 16.3 / 17.1, 20.1
    // / 21.1, 12.7 / 13.3 ms and three within 1 %; the line at 12288 or 16384
    // wavefronts is no better); below, more wavefronts fill it better
    const int wpt = n_waves > 8192 ? 2 : 1;
    int rc = grow_waves(s, st, std::max<int64_t>(n_waves, 1));
    if (rc != ISING_OK) return rc;
    int32_t n_res = 0, K = 0;
    std::vector<SmallGroup> groups;
    int64_t filling = 0;  // wavefronts of rows that fill the XCDs evenly
    n_waves = 0;
    for (int32_t i = 0; i < slots; ++i) {
        const Slot& sl = sc.slots()[i];
        LatticeDesc& d = st.desc[i];
        d = LatticeDesc{};
        if (!sl.active) continue;
        const Geometry g = make_geometry(sl.req.L);
        d.W = reinterpret_cast<uint64_t*>(s->arena + sl.off);
        d.L = g.L;
        d.N = g.N;
        d.istar = g.istar;
        d.sh_star = g.sh_star;
        d.k0 = (uint32_t)sl.req.seed;
        d.k1 = (uint32_t)(sl.req.seed >> 32);
        thresholds_of(sl.req.T, &d.t4, &d.t8);
        d.pstar = (g.L - 1) / g.N;
        d.sweep_limit = (int32_t)sl.planned;
        if (sl.planned <= 0) continue;
        K = std::max<int32_t>(K, (int32_t)sl.planned);
        if (is_resident(s, g)) {
            code_buffer(s);
            d.resident = 1;
            st.draw[n_res] = {i, 2 * g.N * ((g.L + 7) / 8), 0};
            const int64_t words = (int64_t)g.N * g.L;
            if (groups.empty() || groups.back().words + words > group_words(s))
                groups.push_back({n_res, n_res, 0, 0, 0, 0, 0});
            SmallGroup& gr = groups.back();
            gr.end = n_res + 1;
            gr.words += words;
            gr.max_NL = std::max(gr.max_NL, g.N * g.L);
            gr.max_words = std::max(gr.max_words, g.N * (g.L / 2));
            gr.max_draws = std::max(gr.max_draws, st.draw[n_res].n_draw);
            gr.K = std::max<int32_t>(gr.K, (int32_t)sl.planned);
            ++n_res;
        } else if (tiles) {
            Tiled t = {i, large.empty() ? 0 : large.back().first + large.back().count, 0, 0, 0, (int32_t)sl.planned};
            default_resident_shape(g, &t.w, &t.block);
            const std::vector<PersistTile> table = resident_tile_table(i, g.L, t.w, 0);
            t.count = (int32_t)table.size();
            std::copy(table.begin(), table.end(), st.tiles + t.first);
            large.push_back(t);
        } else {
            d.part_begin = (int32_t)n_waves;
            for (int32_t I = 0; I < g.N; ++I)
                for (int32_t w0 = 0; w0 < g.L / 2; w0 += 64 * wpt) st.waves[n_waves++] = {i, I, w0};
            d.part_count = (int32_t)(n_waves - d.part_begin);
            if (rows_fill_xcds(g, wpt, kServerTiledBlock)) filling += d.part_count;
        }
    }
    const bool wave_runs = 2 * filling <= n_waves;
    for (const SmallGroup& gr : groups) {
        int64_t base = 0;
        const int64_t S = group_sweeps(s, gr);
        for (int32_t k = gr.begin; k < gr.end; ++k) {
            const LatticeDesc& d = st.desc[st.draw[k].lat];
            st.draw[k].base = base;
            base += S * d.N * d.L;
        }
    }
    bool forked = false;
    auto enqueue = [&]() -> int {
        ISING_HIP(hipMemcpyAsync(s->d_desc, st.desc, sizeof(LatticeDesc) * slots, hipMemcpyHostToDevice, s->stream));
        if (n_waves)
            ISING_HIP(hipMemcpyAsync(s->d_waves, st.waves, sizeof(WaveItem) * n_waves, hipMemcpyHostToDevice, s->stream));
        if (!large.empty())
            ISING_HIP(hipMemcpyAsync(s->d_tiles, st.tiles,
                                     sizeof(PersistTile) * (size_t)(large.back().first + large.back().count),
                                     hipMemcpyHostToDevice, s->stream));
        if (n_res) ISING_HIP(hipMemcpyAsync(s->d_draw, st.draw, sizeof(DrawLat) * n_res, hipMemcpyHostToDevice, s->stream));
        if (K > 0) {
            const int block = kServerTiledBlock;
            if (n_res) {
                // The small lattices (one workgroup each) run on the side stream,
                // beside the tiled launches of the other lattices if there are any; as in
                // a batch, a word per thread where each has a compute unit to itself.  us
                // for requests of 300 to 500 sweeps in quanta of 100, with workgroups that
                // draw their own codes / these: 8 of L = 64 1379/775, 16 of L = 256
                // 5261/836, 300 of L = 128 and 256 8519/3663; 100 of L = 16 in quanta of
                // one sweep, where launches and the join of two streams are all there is,
                // 1852/1369.
                if (n_large) {
                    ISING_HIP(hipEventRecord(s->fork_ev, s->stream));
                    ISING_HIP(hipStreamWaitEvent(s->side, s->fork_ev, 0));
                    forked = true;
                }
                const hipStream_t on = n_large ? s->side : s->stream;
                for (const SmallGroup& gr : groups) {
                    const int32_t n = gr.end - gr.begin, S = group_sweeps(s, gr);
                    const int wmax = n <= s->cus || gr.max_words > 1024 ? (gr.max_words + 1023) / 1024
                                                                        : (gr.max_words + 255) / 256;
                    for (int32_t done = 0; done < gr.K; done += S) {
                        const int32_t k = std::min(S, gr.K - done);
                        ISING_HIP(launch_draw_codes(s->d_desc, s->d_state, s->d_draw + gr.begin, n, gr.max_draws,
                                                    s->d_codes, done, k, on));
                        ISING_HIP(launch_wave_apply(wmax, wave_apply_block(gr.max_words, wmax), s->d_desc, s->d_state,
                                                    s->d_draw + gr.begin, n, s->d_codes, done, k, 0,
                                                    wave_apply_lds_bytes(gr.max_NL, 0), on));
                    }
                }
                if (n_large) ISING_HIP(hipEventRecord(s->join_ev, s->side));
            }
            for (const Tiled& t : large) {
                const Geometry g = make_geometry(sc.slots()[t.lattice].req.L);
                // the tags of the lattice before
                ISING_HIP(launch_zero_words(s->d_exch, kServerTiles + (uint64_t)t.count * 4 * g.N, s->stream));
                PersistLaunch a = {};
                a.tiles = s->d_tiles + t.first;
                a.descs = s->d_desc;
                a.states = s->d_state;
                a.n_tiles = t.count;
                a.flags = s->d_exch;
                a.exch = s->d_exch + kServerTiles;
                a.exch_tile_words = 4 * (int64_t)g.N;
                a.error = &s->d_state[t.lattice].abandoned;
                a.wait_ticks = s->wait_ticks;
                for (int32_t done = 0; done < t.K; done += kServerTileSweeps) {
                    a.sweep_off = (uint32_t)done;
                    a.K = std::min(kServerTileSweeps, t.K - done);
                    ISING_HIP(resident_gate(s->device, s->stream, [&] {
                        return launch_persist(a, persist_form(g.L, g.N, t.w, t.block), t.count, t.block,
                                              persist_lds_bytes(g.L, g.N, t.w, t.block), s->stream);
                    }));
                }
            }
            for (int32_t k = 0; k < K && n_waves; ++k) {
                ISING_HIP(launch_halfsweep_multi(wpt, block, s->d_desc, s->d_state, s->d_waves, n_waves, wave_runs, false, 0,
                                                 (uint32_t)k, nullptr, nullptr, 0, s->stream));
                ISING_HIP(launch_halfsweep_multi(wpt, block, s->d_desc, s->d_state, s->d_waves, n_waves, wave_runs, false, 1,
                                                 (uint32_t)k, nullptr, nullptr, 0, s->stream));
            }
            if (n_res && n_large) ISING_HIP(hipStreamWaitEvent(s->stream, s->join_ev, 0));
            ISING_HIP(launch_chunk_end(s->d_desc, s->d_state, slots, nullptr, 0, (uint32_t)K, s->stream));
        }
        return ISING_OK;
    };
    rc = enqueue();
    // also after a failure half way: what was enqueued still reads this set and the device's tables
    if (rc != ISING_OK && forked) {
        (void)hipEventRecord(s->join_ev, s->side);
        (void)hipStreamWaitEvent(s->stream, s->join_ev, 0);
    }
    const hipError_t e = hipEventRecord(st.done, s->stream);
    st.used = true;
    if (rc == ISING_OK && e != hipSuccess) rc = hip_fail(e, "hipEventRecord");
    if (rc != ISING_OK) return rc;
    sc.complete_quantum();
    return ISING_OK;
}

// Enqueue E/M and read-back of every request whose sweeps are all enqueued,
// then free their slots and memory.
int enqueue_retirements(ising_server* s) {
    const std::vector<int32_t> fin = s->sched.finished();
    if (fin.empty()) return ISING_OK;
    Readback& r = s->ring[s->next_ring];
    int rc = harvest(s, r, true);  // the entry's previous batch must have landed
    if (rc != ISING_OK) return rc;
    s->next_ring = (s->next_ring + 1) % kRing;
    const int32_t nf = (int32_t)fin.size();
    int64_t max_words = 0;
    for (int32_t k = 0; k < nf; ++k) {
        const Slot& sl = s->sched.slots()[fin[k]];
        r.ids[k] = fin[k];
        max_words = std::max<int64_t>(max_words, (int64_t)(ising_required_bytes(sl.req.L) / 8));
        r.requests.push_back({sl.req, sl.t_admit});
    }
    auto enqueue = [&]() -> int {
        ISING_HIP(hipMemcpyAsync(s->d_fin, r.ids, sizeof(int32_t) * nf, hipMemcpyHostToDevice, s->stream));
        ISING_HIP(launch_observe_multi(s->d_desc, s->d_state, s->d_fin, nf, max_words, s->d_em, s->stream));
        ISING_HIP(hipMemcpyAsync(r.em, s->d_em, sizeof(int64_t) * kObservedWords * nf, hipMemcpyDeviceToHost, s->stream));
        return ISING_OK;
    };
    rc = enqueue();
    const hipError_t e = hipEventRecord(r.done, s->stream);
    if (rc == ISING_OK && e != hipSuccess) rc = hip_fail(e, "hipEventRecord");
    r.pending = true;  // also after a failure half way: what was enqueued still uses the entry
    if (rc != ISING_OK) {
        r.requests.clear();  // read back with the next step's
        return rc;
    }
    for (int32_t i : fin) s->sched.retire(i);
    return ISING_OK;
}

// Admit what fits and enqueue a quantum of all resident lattices, the read-back
// of those that it finishes behind it.
int run_quantum(ising_server* s) {
    int rc = admit_queued(s);
    if (rc != ISING_OK || s->sched.active() == 0) return rc;
    rc = enqueue_quantum(s);
    if (rc == ISING_OK) rc = enqueue_retirements(s);
    if (rc != ISING_OK) return rc;
    hipEvent_t e = nullptr;
    hipError_t he = hipEventCreateWithFlags(&e, hipEventDisableTiming);
    if (he == hipSuccess) he = hipEventRecord(e, s->stream);
    if (he != hipSuccess) {
        if (e) (void)hipEventDestroy(e);
        return hip_fail(he, "quantum event");
    }
    s->inflight.push_back(e);
    return ISING_OK;
}

int wait_idle(ising_server* s) {
    while (!s->inflight.empty()) {
        hipEvent_t e = s->inflight.front();
        s->inflight.pop_front();
        const hipError_t he = hipEventSynchronize(e);
        (void)hipEventDestroy(e);
        if (he != hipSuccess) return hip_fail(he, "hipEventSynchronize");
    }
    return harvest_all(s, true);
}

}  // namespace

extern "C" {

int ising_server_create(size_t hbm_budget, int32_t max_slots, int32_t quantum_sweeps, void* stream,
                        ising_server** out) {
    if (!out) return fail(ISING_EINVAL, "ising_server_create: null output");
    *out = nullptr;
    if (hbm_budget < 256) return fail(ISING_EINVAL, "ising_server_create: budget too small");
    if (max_slots < 1 || max_slots > (1 << 20)) return fail(ISING_EINVAL, "ising_server_create: max_slots in [1, 2^20]");
    if (quantum_sweeps < 1 || quantum_sweeps > 100000)
        return fail(ISING_EINVAL, "ising_server_create: quantum_sweeps in [1, 100000]");
    ising_server* s = new (std::nothrow) ising_server(hbm_budget, max_slots, quantum_sweeps);
    if (!s) return fail(ISING_ENOMEM, "ising_server_create: host allocation failed");
    s->stream = (hipStream_t)stream;
    hipError_t e = hipGetDevice(&s->device);
    if (e == hipSuccess) e = hipMalloc(&s->arena, s->sched.budget());
    if (e != hipSuccess) {
        s->arena = nullptr;
        release(s);
        return fail(ISING_ENOMEM, "ising_server_create: arena of %zu bytes: %s", hbm_budget, hipGetErrorString(e));
    }
    e = hipMalloc(&s->d_desc, sizeof(LatticeDesc) * max_slots);
    if (e == hipSuccess) e = hipMalloc(&s->d_state, sizeof(LatticeState) * max_slots);
    if (e == hipSuccess) e = hipMalloc(&s->d_draw, sizeof(DrawLat) * max_slots);
    if (e == hipSuccess) e = hipMalloc(&s->d_codes_least, sizeof(uint64_t) * kServerCodeWordsLeast);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&s->cus, hipDeviceAttributeMultiprocessorCount, s->device);
    if (e == hipSuccess) e = hipMalloc(&s->d_fin, sizeof(int32_t) * max_slots);
    if (e == hipSuccess) e = hipMalloc(&s->d_em, sizeof(int64_t) * kObservedWords * max_slots);
    for (Stage& st : s->stage) {
        if (e == hipSuccess) e = hipHostMalloc(&st.desc, sizeof(LatticeDesc) * max_slots, hipHostMallocDefault);
        if (e == hipSuccess) e = hipHostMalloc(&st.draw, sizeof(DrawLat) * max_slots, hipHostMallocDefault);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&st.done, hipEventDisableTiming);
    }
    for (Readback& r : s->ring) {
        if (e == hipSuccess) e = hipHostMalloc(&r.ids, sizeof(int32_t) * max_slots, hipHostMallocDefault);
        if (e == hipSuccess) e = hipHostMalloc(&r.em, sizeof(int64_t) * kObservedWords * max_slots, hipHostMallocDefault);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&r.done, hipEventDisableTiming);
    }
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&s->side, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&s->fork_ev, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&s->join_ev, hipEventDisableTiming);
    if (e == hipSuccess) e = hipMemsetAsync(s->d_state, 0, sizeof(LatticeState) * max_slots, s->stream);
    if (e != hipSuccess) {
        release(s);
        return hip_fail(e, "ising_server_create");
    }
    s->lds_limit = resident_lds_limit(s->device);
    *out = s;
    return ISING_OK;
}

int ising_server_submit(ising_server* s, uint64_t req_id, int32_t L, double T, int64_t sweeps, uint64_t seed,
                        int32_t init) {
    if (!s) return fail(ISING_EINVAL, "ising_server_submit: null handle");
    if (!valid_L(L)) return fail(ISING_EINVAL, "ising_server_submit: L = %d invalid", L);
    if (!valid_T(T)) return fail(ISING_EINVAL, "ising_server_submit: T must be finite and > 0");
    if (sweeps < 0 || sweeps > 0x7FFFFFFF) return fail(ISING_EINVAL, "ising_server_submit: sweeps out of range");
    if (init != ISING_COLD && init != ISING_HOT) return fail(ISING_EINVAL, "ising_server_submit: init must be 0 or 1");
    Request r;
    r.id = req_id;
    r.L = L;
    r.T = T;
    r.sweeps = sweeps;
    r.seed = seed;
    r.init = init;
    r.bytes = ising_required_bytes(L);
    r.t_submit = now_s();
    if (!s->sched.submit(r))
        return fail(ISING_EINVAL, "ising_server_submit: lattice of %zu bytes exceeds the budget", r.bytes);
    return ISING_OK;
}

int ising_server_step(ising_server* s, int32_t* active) {
    if (!s) return fail(ISING_EINVAL, "ising_server_step: null handle");
    int rc = harvest_all(s, false);
    // at most kStages quanta in flight: wait for the oldest before adding one
    while (rc == ISING_OK && (int)s->inflight.size() >= kStages) {
        hipEvent_t e = s->inflight.front();
        s->inflight.pop_front();
        const hipError_t he = hipEventSynchronize(e);
        (void)hipEventDestroy(e);
        if (he != hipSuccess) rc = hip_fail(he, "hipEventSynchronize");
        if (rc == ISING_OK) rc = harvest_all(s, false);
    }
    if (rc == ISING_OK) rc = run_quantum(s);
    // nothing resident or queued: let every pending read-back land; one that brings
    // an abandoned request back to the queue has the next quantum follow, so that a
    // caller who stops when nothing is resident or queued has every result
    while (rc == ISING_OK && s->sched.active() == 0 && s->sched.queued() == 0) {
        rc = wait_idle(s);
        if (s->sched.queued() == 0) break;
        if (rc == ISING_OK) rc = run_quantum(s);
    }
    if (active) *active = s->sched.active();
    return rc;
}

int ising_server_set_resident_wait(ising_server* s, uint64_t ticks) {
    if (!s) return fail(ISING_EINVAL, "ising_server_set_resident_wait: null handle");
    if (ticks > kWaitTicks * 60)
        return fail(ISING_EINVAL, "ising_server_set_resident_wait: at most %llu ticks (one minute)",
                    (unsigned long long)(kWaitTicks * 60));
    s->wait_ticks = ticks ? ticks : kWaitTicks;
    return ISING_OK;
}

int ising_server_poll(ising_server* s, ising_result* out, int32_t cap, int32_t* n) {
    if (!s || !n || (cap > 0 && !out)) return fail(ISING_EINVAL, "ising_server_poll: null argument");
    int rc = harvest_all(s, false);
    if (rc != ISING_OK) return rc;
    const int32_t k = std::max<int32_t>(0, std::min<int32_t>(cap, (int32_t)s->done.size()));
    for (int32_t i = 0; i < k; ++i) out[i] = s->done[i];
    s->done.erase(s->done.begin(), s->done.begin() + k);
    *n = k;
    return ISING_OK;
}

int ising_server_stats(ising_server* s, int32_t* queued, int32_t* resident, int32_t* finished, size_t* bytes_in_use) {
    if (!s) return fail(ISING_EINVAL, "ising_server_stats: null handle");
    if (queued) *queued = (int32_t)s->sched.queued();
    if (resident) *resident = s->sched.active();
    if (finished) *finished = (int32_t)s->done.size();
    if (bytes_in_use) *bytes_in_use = s->sched.bytes_in_use();
    return ISING_OK;
}

int ising_server_destroy(ising_server* s) {
    if (!s) return ISING_OK;
    hipError_t e = hipStreamSynchronize(s->stream);
    release(s);
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    return ISING_OK;
}

}  // extern "C"
