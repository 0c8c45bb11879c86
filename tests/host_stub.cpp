// The library's host code (ising_server.cpp, ising_lattice.cpp, ising_batch.cpp) without a GPU, for
// the paths that only a failure reaches: a stand-in HIP runtime that runs enqueued
// work late, in the order of the calls and only when the host waits for it, whose
// allocations can be made to fail, and stand-ins of the kernels' launchers that
// can be made to fail and that keep, in a lattice's first word, a number which
// depends on its seed and on every sweep applied to it, in order.
//   host_stub <scenario> [number ...]   prints one line per finding; see main()
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "../include/ising.h"
#include "../paper_1811_04384_amd/csrc/ising_launch.hpp"
#include "../paper_1811_04384_amd/csrc/ising_replicas.hpp"

using namespace ising;

// ---- runtime ----------------------------------------------------------------

namespace {

std::deque<std::function<void()>> work;
uint64_t enqueued = 0, executed = 0;
size_t fail_above = ~size_t(0);  // allocations of more bytes fail
int allocations = 0;
int fail_launch = 0;   // the n-th launch from now fails (0: none)
bool rewritten = false;  // a host buffer changed between a copy's enqueueing and its execution
bool wrong = false;      // a launcher was given something that does not fit
int captures = 0;        // handles whose resident launches a caller has captured
bool capturing = false;  // the stream is in a caller's capture
int n_persist = 0, n_swept = 0, n_strip_phase = 0, n_strip_lists = 0, n_strip_draws = 0;

void enqueue(std::function<void()> f) {
    work.push_back(std::move(f));
    ++enqueued;
}
void run_until(uint64_t seq) {
    while (executed < seq && !work.empty()) {
        work.front()();
        work.pop_front();
        ++executed;
    }
}
void run_all() { run_until(enqueued); }

// Where asked for, the order that streams and events give the launches of resident
// tiles and of half-sweeps: the launches that each comes after.
bool watch_order = false;
int n_watched = 0;
std::map<hipStream_t, std::set<int>> behind;
std::vector<std::pair<int, std::set<int>>> tile_launches, sweep_launches;

void watch(std::vector<std::pair<int, std::set<int>>>& launches, hipStream_t s) {
    if (!watch_order) return;
    launches.push_back({n_watched, behind[s]});
    behind[s].insert(n_watched++);
}
// Whether tiles may run beside half-sweeps.
bool beside() {
    for (const auto& t : tile_launches)
        for (const auto& h : sweep_launches)
            if (!t.second.count(h.first) && !h.second.count(t.first)) return true;
    return false;
}

struct Event {
    uint64_t seq = 0;
    std::set<int> behind;
};

hipError_t launch(std::function<void()> f) {
    if (fail_launch > 0 && --fail_launch == 0) return hipErrorLaunchFailure;
    enqueue(std::move(f));
    return hipSuccess;
}

}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    if (n > fail_above) return hipErrorOutOfMemory;
    ++allocations;
    *p = std::malloc(n ? n : 1);
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    run_all();
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::malloc(n ? n : 1);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    run_all();
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = reinterpret_cast<hipStream_t>(std::malloc(1));
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    std::free(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    run_all();
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    const std::set<int>& b = reinterpret_cast<Event*>(e)->behind;
    behind[s].insert(b.begin(), b.end());
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = reinterpret_cast<hipEvent_t>(new Event);
    return hipSuccess;
}
// A captured graph's work is enqueued once, when it is captured.
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    *g = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* g, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    *g = nullptr;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = reinterpret_cast<hipEvent_t>(new Event);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    delete reinterpret_cast<Event*>(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    reinterpret_cast<Event*>(e)->seq = enqueued;
    reinterpret_cast<Event*>(e)->behind = behind[s];
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    run_until(reinterpret_cast<Event*>(e)->seq);
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    return executed >= reinterpret_cast<Event*>(e)->seq ? hipSuccess : hipErrorNotReady;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t) {
    if (kind == hipMemcpyHostToDevice) {
        std::vector<char> was((const char*)src, (const char*)src + n);
        enqueue([=] {
            if (std::memcmp(was.data(), src, n) != 0) rewritten = true;
            std::memcpy(dst, src, n);
        });
    } else {
        enqueue([=] { std::memcpy(dst, src, n); });
    }
    return hipSuccess;
}
hipError_t hipMemcpy(void* dst, const void* src, size_t n, hipMemcpyKind) {
    run_all();
    std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) {
    enqueue([=] { std::memset(p, v, n); });
    return hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n) {
    run_all();
    std::memset(p, v, n);
    return hipSuccess;
}
}  // extern "C"

// ---- launchers ----------------------------------------------------------------

namespace ising {

// The number in a lattice's first word: its start, and a sweep t.
static uint64_t start_of(uint64_t seed, int hot) { return 2 * seed + (uint64_t)hot + 1; }
static uint64_t swept(uint64_t v, uint64_t t) { return v * 6364136223846793005ull + t + 1442695040888963407ull; }

hipError_t launch_init(uint64_t* W, const Geometry&, uint64_t seed, int hot, hipStream_t) {
    return launch([=] { *W = start_of(seed, hot); });
}
hipError_t launch_zero_words(uint64_t* p, uint64_t n, hipStream_t) {
    return launch([=] { std::memset(p, 0, 8 * n); });
}
hipError_t launch_halfsweep_multi(int, int, const LatticeDesc* descs, LatticeState* states, const WaveItem* waves,
                                  int64_t n_waves, bool, bool, int colour, uint32_t sweep_off, Partial*, const Partial*,
                                  uint32_t, hipStream_t s) {
    ++n_swept;
    watch(sweep_launches, s);
    return launch([=] {
        if (colour == 1)
            for (int64_t w = 0; w < n_waves; ++w) {
                const int32_t i = waves[w].lattice;
                if (waves[w].row == 0 && waves[w].w0 == 0 && (int32_t)sweep_off < descs[i].sweep_limit)
                    *descs[i].W = swept(*descs[i].W, states[i].t + sweep_off);
            }
    });
}
hipError_t launch_chunk_end(const LatticeDesc* descs, LatticeState* states, int32_t n, const Partial*, uint32_t, uint32_t k,
                            hipStream_t) {
    return launch([=] {
        for (int32_t i = 0; i < n; ++i) states[i].t += std::min(k, (uint32_t)descs[i].sweep_limit);
    });
}
hipError_t launch_observe_multi(const LatticeDesc* descs, LatticeState* states, const int32_t* ids, int32_t n, int64_t,
                                int64_t* out, hipStream_t) {
    return launch([=] {
        for (int32_t k = 0; k < n; ++k) {
            out[kObservedWords * k] = (int64_t)*descs[ids[k]].W;
            out[kObservedWords * k + 1] = (int64_t)states[ids[k]].t;
            out[kObservedWords * k + 2] = states[ids[k]].abandoned;
        }
    });
}
// Drawn codes: the first and last word of a sweep's codes hold its index.
hipError_t launch_draw_codes(const LatticeDesc* descs, const LatticeState* states, const DrawLat* lats, int32_t n, int32_t,
                             uint64_t* codes, int32_t off, int32_t S, hipStream_t) {
    return launch([=] {
        for (int32_t e = 0; e < n; ++e) {
            const LatticeDesc& d = descs[lats[e].lat];
            const int64_t NL = (int64_t)d.N * d.L;
            for (int32_t j = 0; j < S && off + j < d.sweep_limit; ++j) {
                uint64_t* c = codes + lats[e].base + j * NL;
                c[0] = c[NL - 1] = states[lats[e].lat].t + off + j;
            }
        }
    });
}
hipError_t launch_wave_apply(int wmax, int block, const LatticeDesc* descs, LatticeState* states, const DrawLat* lats,
                             int32_t n, const uint64_t* codes, int32_t off, int32_t S, int32_t, size_t, hipStream_t) {
    return launch([=] {
        for (int32_t e = 0; e < n; ++e) {
            const LatticeDesc& d = descs[lats[e].lat];
            const int64_t NL = (int64_t)d.N * d.L;
            if (NL / 2 > (int64_t)wmax * block || block > 1024) wrong = true;
            for (int32_t j = 0; j < S && off + j < d.sweep_limit; ++j) {
                const uint64_t* c = codes + lats[e].base + j * NL;
                const uint64_t t = states[lats[e].lat].t + off + j;
                if (c[0] != t || c[NL - 1] != t) wrong = true;
                *d.W = swept(*d.W, t);
            }
        }
    });
}
int32_t wave_apply_block(int32_t words, int32_t wmax) { return ((words + wmax - 1) / wmax + 63) / 64 * 64; }
int32_t wave_apply_words_per_thread(int32_t L, int32_t N, int32_t block) { return (N * (L / 2) + block - 1) / block; }
size_t wave_apply_lds_bytes(int32_t NL, int32_t) { return (size_t)NL * 8; }
size_t resident_lds_limit(int) { return 160 * 1024; }

// A wait bound of one tick expires at once: the launch leaves a state that is not the lattice's.
hipError_t launch_persist(const PersistLaunch& a, int, int32_t, int, size_t, hipStream_t s) {
    ++n_persist;
    watch(tile_launches, s);
    return launch([=] {
        if (!a.states) return;  // of a single lattice
        const int32_t i = a.tiles[0].lattice;
        uint64_t& w = *a.descs[i].W;
        if (a.wait_ticks == 1) *a.error = 1;
        if (*a.error) w ^= 0xDEADull;
        else
            for (int32_t j = 0; j < a.K; ++j) w = swept(w, a.states[i].t + a.sweep_off + j);
    });
}
int persist_form(int32_t, int32_t, int32_t, int) { return 0; }
size_t persist_lds_bytes(int32_t, int32_t, int32_t, int32_t) { return 1000; }
size_t persist_lds_limit(int) { return 160 * 1024; }
hipError_t allow_persist_lds(int, int, size_t) { return hipSuccess; }
static int tiles_per_cu = 1;
hipError_t persist_capacity(int, size_t, int, int64_t* tiles, int64_t* beside) {
    *tiles = 256 * tiles_per_cu;
    if (beside) *beside = 256 * ((tiles_per_cu + 1) / 2);
    return hipSuccess;
}
int persist_form_any() { return 0; }
hipError_t launch_begin_call(LatticeState*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_reset_sums(LatticeState*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_finalize_resident(const LatticeDesc*, LatticeState*, const int32_t*, int32_t, const Partial*, int32_t, int32_t,
                                    hipStream_t) {
    return hipSuccess;
}
size_t tile_lds_limit(int) { return 160 * 1024; }
hipError_t resident_gate(int, hipStream_t, const std::function<hipError_t()>& f, bool* captured) {
    if (capturing && captured) *captured = true;
    return f();
}
int resident_captures(int, int n) { return captures += n; }
hipError_t launch_samples(const Partial*, int32_t, int32_t, int32_t, int64_t*, int64_t*, Moments*, hipStream_t) {
    return hipSuccess;
}
// The codes' first and last word hold the sweep index; a lattice's first word counts its sweeps, which have to come in order.
hipError_t launch_drawn(const DrawnLaunch& a, hipStream_t) {
    return launch([=] {
        const int64_t NL = (int64_t)a.N * a.L;
        for (int32_t j = 0; j < a.n_apply; ++j) {
            if (a.codes[j * NL] != *a.W || a.codes[(j + 1) * NL - 1] != *a.W) wrong = true;
            *a.W += 1;
        }
        for (int32_t j = 0; j < a.n_draw; ++j) a.drawn[j * NL] = a.drawn[(j + 1) * NL - 1] = a.t_draw + j;
    });
}
// The strip dynamics: only that a phase's picks are all drawn, in order, and what is drawn lies within the buffers.
static uint64_t strip_picks_done = 0;
hipError_t launch_strip_phase(uint64_t*, const StripArgs& a, hipStream_t) {
    ++n_strip_phase;
    strip_picks_done += a.picks;
    return hipSuccess;
}
size_t strip_chain_lds_bytes(const StripArgs& a) { return (size_t)(a.width + 2) * (size_t)a.N * 8; }
size_t strip_apply_lds_bytes(const StripArgs&, int) { return 1024; }
hipError_t launch_strip_draws(const StripArgs& a, uint32_t, uint32_t n_k, uint32_t* pos, uint64_t* codes, hipStream_t) {
    ++n_strip_draws;
    const size_t n = (size_t)n_k * (size_t)a.strips;
    return launch([=] { pos[0] = pos[n - 1] = 7, codes[0] = codes[n - 1] = 7; });
}
hipError_t launch_strip_apply(uint64_t*, const StripArgs& a, uint32_t n_k, const uint32_t* pos, const uint64_t* codes, hipStream_t) {
    strip_picks_done += n_k;
    const size_t n = (size_t)n_k * (size_t)a.strips;
    return launch([=] {
        if (pos[0] != 7 || pos[n - 1] != 7 || codes[0] != 7 || codes[n - 1] != 7) wrong = true;
    });
}
uint32_t strip_list_picks(const StripArgs& a, int64_t max_entries) {
    return (int64_t)a.N * a.width > 512 ? 0u : (uint32_t)std::min<int64_t>(max_entries / a.strips, a.picks) & ~1u;
}
hipError_t allow_strip_list_lds() { return hipSuccess; }
hipError_t launch_strip_lists(uint64_t*, const StripArgs& a, const StripLists& l, const StripArgs& n, const StripLists& ln, hipStream_t) {
    ++n_strip_lists;
    strip_picks_done += l.n_k;
    return launch([=] {
        auto mark = [](const StripArgs& p, const StripLists& x, bool set) {
            const size_t e = (size_t)p.strips * x.n_k, f = (size_t)p.strips * (size_t)(p.N * p.width + 1);
            if (set) x.codes[0] = x.codes[e - 1] = x.k0 + 1, x.k[0] = x.k[e - 1] = 3, x.first[0] = x.first[f - 1] = 5;
            else if (x.codes[0] != x.k0 + 1 || x.codes[e - 1] != x.k0 + 1 || x.k[0] != 3 || x.k[e - 1] != 3 || x.first[0] != 5 ||
                     x.first[f - 1] != 5)
                wrong = true;
        };
        if (ln.n_k) mark(n, ln, true);
        if (l.n_k) mark(a, l, false);
    });
}
size_t finalize_scratch_bytes() { return 4096; }
int64_t observe_single_waves(const Geometry&) { return 16; }
int64_t halfsweep_single_waves(const Geometry&, int, int) { return 16; }
int32_t drawn_max_words() { return 2048; }
size_t drawn_lds_bytes(int32_t L, int32_t N) { return (size_t)L * N * 8; }
}  // namespace ising

// ---- scenarios ----------------------------------------------------------------

namespace {

struct Req {
    uint64_t id;
    int32_t L;
    int64_t sweeps;
};

uint64_t expected(const Req& r) {
    uint64_t v = ising::start_of(r.id, 1);
    for (int64_t t = 0; t < r.sweeps; ++t) v = ising::swept(v, (uint64_t)t);
    return v;
}

// Serve the requests as a program does that stops when nothing is resident or queued;
// prints each result and the launches of either kind.
void serve(ising_server* s, const std::vector<Req>& reqs, bool tolerate = false) {
    for (const Req& r : reqs)
        if (ising_server_submit(s, r.id, r.L, 2.0, r.sweeps, r.id, ISING_HOT) != ISING_OK) std::printf("refused %d\n", (int)r.id);
    int32_t active = 0, queued = 0;
    for (int step = 0; step < 1000; ++step) {
        const int rc = ising_server_step(s, &active);
        if (rc != ISING_OK) {
            std::printf("step error %d: %s\n", rc, ising_last_error());
            if (!tolerate) break;
        }
        (void)ising_server_stats(s, &queued, nullptr, nullptr, nullptr);
        if (active == 0 && queued == 0) break;
    }
    std::map<uint64_t, ising_result> got;
    std::vector<ising_result> out(reqs.size() + 1);
    int32_t n = 0;
    (void)ising_server_poll(s, out.data(), (int32_t)out.size(), &n);
    for (int32_t k = 0; k < n; ++k) got[out[k].req_id] = out[k];
    if (n != (int32_t)got.size()) std::printf("a result twice\n");
    double done_first = 1e300, admit_last = 0;
    for (const Req& r : reqs) {
        if (!got.count(r.id)) {
            std::printf("missing %d\n", (int)r.id);
            continue;
        }
        const ising_result& g = got[r.id];
        const bool right = g.status == ISING_OK && (uint64_t)g.E == expected(r) && g.M == r.sweeps;
        std::printf("%s %d\n", right ? "right" : g.status != ISING_OK ? "failed" : "WRONG", (int)r.id);
        done_first = std::min(done_first, g.t_done_s);
        admit_last = std::max(admit_last, g.t_admit_s);
    }
    std::printf("again %d persist %d halfsweeps %d\n", admit_last > done_first, n_persist, n_swept);
}

ising_server* server(size_t budget, int32_t slots, int32_t quantum) {
    ising_server* s = nullptr;
    if (ising_server_create(budget, slots, quantum, nullptr, &s) != ISING_OK) {
        std::printf("create: %s\n", ising_last_error());
        std::exit(1);
    }
    return s;
}

}  // namespace

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    std::vector<int64_t> num;
    for (int i = 2; i < argc; ++i) num.push_back(std::atoll(argv[i]));
    if (what == "abandon") {
        // sweeps of the large requests and of the small one, and whether waits expire
        ising_server* s = server(64 << 20, 16, 100);
        if (num[3]) (void)ising_server_set_resident_wait(s, 1);
        serve(s, {{1, 1024, num[0]}, {2, 64, num[1]}, {3, 512, num[2]}});
        ising_server_destroy(s);
    } else if (what == "tight") {
        // once the server is made, allocations of more than num[0] bytes fail
        ising_server* s = server(64 << 20, 400, 90);
        fail_above = (size_t)num[0];
        std::vector<Req> reqs;
        for (int k = 0; k < 60; ++k) reqs.push_back({(uint64_t)k, (int32_t)(4 + (k * 38) % 254 / 2 * 2), 20 + 37 * k % 230});
        reqs.push_back({60, 256, 130});
        serve(s, reqs);
        ising_server_destroy(s);
    } else if (what == "halfway") {
        // the num[0]-th launch from the first step on fails, in quanta of num[1] sweeps; the caller steps on
        ising_server* s = server(64 << 20, 16, (int32_t)num[1]);
        fail_launch = (int)num[0];
        serve(s, {{1, 64, 350}, {2, 2048, 320}, {3, 100, 80}, {4, 300, 700}}, true);
        std::printf("failed %d\n", fail_launch == 0);
        ising_server_destroy(s);
    } else if (what == "captured") {
        // a quantum of one large lattice while a handle's captured tiles may be replayed, and after it is gone
        ising_server* s = server(64 << 20, 16, 100);
        ising_lattice* h = nullptr;
        if (ising_create(1024, 1, ISING_HOT, nullptr, &h) != ISING_OK) return 1;
        const int tile_sets = (int)num[0];  // 1: the tiles are set anew before the server runs
        n_persist = 0;
        capturing = true;
        (void)ising_sweep(h, 2.0, 2500);
        capturing = false;
        std::printf("captures %d\n", captures);
        if (tile_sets) (void)ising_set_resident_tiles(h, 8, 512, 100);
        n_persist = 0;
        serve(s, {{1, 1024, 100}});
        ising_destroy(h);
        std::printf("captures %d\n", captures);
        serve(s, {{2, 1024, 100}});
        ising_server_destroy(s);
    } else if (what == "drawn") {
        // num[0] 0: a scan, 1: a plain run, whose num[1]-th launch fails; then the rest, and a scan once more
        ising_lattice* h = nullptr;
        if (ising_create(64, 1, ISING_HOT, nullptr, &h) != ISING_OK) return 1;
        void* W = nullptr;
        size_t bytes = 0;
        (void)ising_words(h, &W, &bytes);
        run_all();
        uint64_t& applied = *static_cast<uint64_t*>(W);
        applied = 0;
        const double T[3] = {1.5, 2.0, 2.5};
        ising_moments m[3];
        uint64_t t = 0;
        for (int call = 0; call < 3; ++call) {
            fail_launch = call == 1 ? (int)num[1] : 0;
            const int rc = num[0] == 0 || call == 2 ? ising_scan(h, 3, T, 300, 20, 1, m) : ising_sweep(h, 2.0, 900);
            run_all();
            (void)ising_get_sweep_count(h, &t);
            std::printf("%s t %s\n", rc == ISING_OK ? "ok" : "failed", t == applied ? "right" : "WRONG");
        }
        ising_destroy(h);
    } else if (what == "strips") {
        // strips of num[1], then of num[2] columns of L = num[0]; allocations of more than num[3] bytes fail
        ising_lattice* h = nullptr;
        if (ising_create((int32_t)num[0], 1, ISING_HOT, nullptr, &h) != ISING_OK) return 1;
        fail_above = (size_t)num[3];
        const int before = allocations;
        const uint64_t N = (uint64_t)ising_word_rows((int32_t)num[0]);
        for (int call = 0; call < 4; ++call) {
            const uint64_t cols = (uint64_t)num[1 + call % 2], want = ising::strip_picks_done + 3 * 10 * N * cols;
            const int rc = ising_random_iterations(h, 2.0, (int32_t)cols, 3, 0, nullptr, nullptr, nullptr);
            run_all();
            if (rc != ISING_OK || ising::strip_picks_done != want) std::printf("error %d: %s\n", rc, ising_last_error());
        }
        std::printf("allocations %d phase %d draws %d lists %d\n", allocations - before, n_strip_phase > 0,
                    n_strip_draws > 0, n_strip_lists > 0);
        ising_destroy(h);
    } else if (what == "samples") {
        // the sweeps of a launch that are sampled, from what the kernel is given and from the run
        int bad = 0;
        for (int64_t every : {1, 2, 3, 7, 255, 256, 257, 511, 512, 513, 1000, 2147483391, 2147483646, 2147483647})
            for (int64_t back = 0; back < 600; ++back)
                for (int32_t n : {1, 2, 7, 255, 256}) {
                    const int64_t done = 5 * every + (every - 1 - back % every);
                    DrawnLaunch a = {};
                    sampled_as(a, done, n, (int32_t)every);
                    int32_t count = 0;
                    for (int32_t j = 0; j < n; ++j) {
                        const bool sampled = a.every > 0 && (a.sweep_off + j + 1) % a.every == 0;
                        bad += sampled != ((done + j + 1) % every == 0);
                        count += sampled;
                    }
                    bad += count != (a.every > 0 ? (a.sweep_off + n) / a.every - a.sweep_off / a.every : 0);
                }
        DrawnLaunch none = {};
        sampled_as(none, 100, 5, 0);
        std::printf("bad %d none %d %d\n", bad, none.every, none.sweep_off);
    } else if (what == "beside") {
        // num[1] lattices of L = 512, num[2] of which are in 32 resident tiles each, num[0] of which a compute unit holds
        tiles_per_cu = (int)num[0];
        watch_order = true;
        std::vector<int32_t> L(num[1], 512), init(num[1], ISING_HOT);
        for (int64_t i = num[2]; i < num[1]; ++i) L[i] = 1024;
        std::vector<uint64_t> seed(num[1], 1);
        std::vector<double> T(num[1], 2.0);
        ising_batch* b = nullptr;
        if (ising_batch_create((int32_t)num[1], L.data(), seed.data(), init.data(), nullptr, &b) != ISING_OK) return 1;
        ising_batch_plan p = {};
        if (ising_batch_get_plan(b, &p) != ISING_OK) return 1;
        p.resident_max_L = 0;
        p.draw_sweeps = 0;
        p.tile_max_L = 512;
        p.tile_sweeps = 1;
        p.tile_cols = 16;
        p.tile_block = 512;
        p.tile_exchange = 1;
        if (ising_batch_set_plan(b, &p) != ISING_OK || ising_batch_sweep(b, T.data(), 10, 5, nullptr, nullptr) != ISING_OK)
            std::printf("error: %s\n", ising_last_error());
        run_all();
        std::printf("tiles %d halfsweeps %d beside %d\n", (int)tile_launches.size(), (int)sweep_launches.size(), beside());
        ising_batch_destroy(b);
    }
    std::printf("rewritten %d wrong %d\n", rewritten, wrong);
    return 0;
}
