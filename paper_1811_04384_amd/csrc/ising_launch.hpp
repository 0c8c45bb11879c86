// Host-side launchers of the gfx950 kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <functional>

#include "ising_common.hpp"

namespace ising {

// Tiled work of one colour of a lattice: segments of 2*wpt columns per row.
inline int32_t segments_per_row(int32_t L, int32_t wpt) { return (L + 2 * wpt - 1) / (2 * wpt); }
// Launch shape of one lattice's half-sweeps by its words of a colour (us per
// half-sweep on gfx950).  From 3 Mi words (L from about 11,500) four words per
// thread, whose position-20 blocks are shared best: L = 12288 30.7 against
// 32.4 with one, 16384 49.4 / 52.0, 32768 190 / 201.  From 1 Mi words one
// word per thread in 256-thread workgroups (L = 8000 17.1, 9998 23.8; the
// shapes are within 3 per cent there); below it 64-thread workgroups, which
// start faster (L = 2048 3.9 against 4.2), and below 64 Ki words, a handful of
// workgroups, 256 threads again.
inline void default_halfsweep_plan(const Geometry& g, int* wpt, int* block) {
    const int64_t words = (int64_t)g.N * (g.L / 2);
    *wpt = words < ((int64_t)3 << 20) ? 1 : 4;
    *block = (words >= ((int64_t)1 << 16) && words < ((int64_t)1 << 20)) ? 64 : 256;
}
// Wavefronts of a tiled half-sweep of one lattice: every word row starts a
// new wavefront.
inline int64_t waves_per_colour(const Geometry& g, int32_t wpt) {
    return (int64_t)g.N * ((segments_per_row(g.L, wpt) + 63) / 64);
}

// Whether the rows of a lattice in a table of wavefronts are a multiple of 8
// workgroups each, so that workgroups dealt to the 8 XCDs in turn put a column
// of words of all its rows on one XCD.
inline bool rows_fill_xcds(const Geometry& g, int32_t wpt, int block) {
    return (waves_per_colour(g, wpt) / g.N) % (8 * (block / 64)) == 0;
}

// Whether no word of a lattice has more than 16 live positions, so that five Philox
// blocks are more than it needs (up to L = 128; L = 42 and 84 have 21).
inline bool few_live(const Geometry& g) { return (g.L - 1) / g.N < 16; }

// Zero n 64-bit words with a kernel (usable inside a captured graph).
hipError_t launch_zero_words(uint64_t* p, uint64_t n, hipStream_t s);

// Spins of a fresh lattice: cold (all up) or hot (Philox stream 0 draw < 2^31).
hipError_t launch_init(uint64_t* W, const Geometry& g, uint64_t seed, int hot, hipStream_t s);

// One half-sweep of one lattice (colour 0 or 1).  With `partials` non-null
// (colour 1 only) every wavefront stores its bond/spin counts in
// partials[wave]; the number of launched wavefronts (the slots written) is
// returned in *n_waves.
hipError_t launch_halfsweep_single(int wpt, int block, uint64_t* W, const SweepArgs& a, int colour,
                                   Partial* partials, int64_t* n_waves, hipStream_t s);
int64_t halfsweep_single_waves(const Geometry& g, int wpt, int block);

// Sum the partials of one lattice into E, M and store them: sample index
// `idx` of series (if non-null), out_EM[0..1] (if non-null), and add them to
// the moment sums `mom` (if non-null, device memory).  `scratch`
// is finalize_scratch_bytes() of device memory, zeroed once before first use
// (the kernel leaves it ready for the next call); calls sharing a scratch
// buffer must be ordered on one stream.
size_t finalize_scratch_bytes();
hipError_t launch_finalize_single(const Partial* partials, int64_t n_partials, int32_t L, int64_t* series_E,
                                  int64_t* series_M, int64_t idx, int64_t* out_EM, Moments* mom, void* scratch,
                                  hipStream_t s);

// One phase of the strip dynamics over all strips of one lattice, in one
// kernel (each lane draws and applies its strip's picks).
hipError_t launch_strip_phase(uint64_t* W, const StripArgs& a, hipStream_t s);

// The same phase split in chunks of picks: launch_strip_draws computes the
// words and acceptance codes of picks [k0, k0 + n_k) of every strip into
// pos / codes (n_k * strips entries, pick-major), launch_strip_apply applies
// them in order (a window of picks per step, committing the prefix without
// conflicts), the strips' columns held in LDS.  Usable when one strip fits:
// strip_apply_lds_bytes(a, 1) <= kStripLdsBytes.
constexpr size_t kStripLdsBytes = 64 * 1024;
size_t strip_chain_lds_bytes(const StripArgs& a);
size_t strip_apply_lds_bytes(const StripArgs& a, int chains);
hipError_t launch_strip_draws(const StripArgs& a, uint32_t k0, uint32_t n_k, uint32_t* pos, uint64_t* codes,
                              hipStream_t s);
hipError_t launch_strip_apply(uint64_t* W, const StripArgs& a, uint32_t n_k, const uint32_t* pos,
                              const uint64_t* codes, hipStream_t s);

// The same phase by lists of picks per word, for strips of at most 512 words of a
// phase: a launch applies the lists `l` of phase a (l.n_k = 0: none) and draws
// those of phase n (ln, in other buffers) for the next one.  strip_list_picks:
// how many picks of a phase a list may hold (even; 0: not usable) when a buffer
// holds max_entries of them; allow_strip_list_lds once before the first launch.
constexpr size_t kStripListLds = 80 * 1024;
uint32_t strip_list_picks(const StripArgs& a, int64_t max_entries);
hipError_t allow_strip_list_lds();
hipError_t launch_strip_lists(uint64_t* W, const StripArgs& a, const StripLists& l, const StripArgs& n,
                              const StripLists& ln, hipStream_t s);

// Observables of one lattice: per-wavefront partials of right+down
// antiparallel bonds and up spins over all words.
hipError_t launch_observe_single(const uint64_t* W, const Geometry& g, Partial* partials, int64_t* n_waves,
                                 hipStream_t s);
int64_t observe_single_waves(const Geometry& g);

// Unpack an nrows x ncols window (indices mod L) to bytes; write the bytes
// of lattice rows r0 .. r0 + nrows - 1 (1 <= nrows <= N) into their words.
hipError_t launch_unpack(const uint64_t* W, const Geometry& g, int32_t r0, int32_t c0, int32_t nrows,
                         int32_t ncols, uint8_t* out, hipStream_t s);
hipError_t launch_pack_rows(const uint8_t* in, const Geometry& g, int32_t r0, int32_t nrows, uint64_t* W,
                            hipStream_t s);
// Every word from the bytes of the whole lattice (row major, nonzero = up).
hipError_t launch_pack_words(const uint8_t* in, const Geometry& g, uint64_t* W, hipStream_t s);

// ---- batches --------------------------------------------------------------

// Tiled half-sweep over a wave table covering many lattices.  partials
// (colour 1 of a measured sweep): each wavefront stores its sums there.
// fin_partials: before its own work, the launch finalizes every tiled
// lattice's measured sweep fin_off from those partials (written by an
// earlier launch on the same stream).  Lattices whose sweep_limit is <= an
// offset took no part in that sweep and are skipped.  runs: the table is dealt
// to the XCDs in runs of wavefronts, not workgroup by workgroup.  few: most of its
// wavefronts are of lattices with few live positions (few_live).
hipError_t launch_halfsweep_multi(int wpt, int block, const LatticeDesc* descs, LatticeState* states,
                                  const WaveItem* waves, int64_t n_waves, bool runs, bool few, int colour,
                                  uint32_t sweep_off, Partial* partials, const Partial* fin_partials,
                                  uint32_t fin_off, hipStream_t s);
// End of a chunk of k sweeps: finalize the tiled lattices' measured sweep
// fin_off (fin_partials non-null) and advance every lattice's sweep counter
// by min(k, sweep_limit).
hipError_t launch_chunk_end(const LatticeDesc* descs, LatticeState* states, int32_t n_lat,
                            const Partial* fin_partials, uint32_t fin_off, uint32_t k, hipStream_t s);
// One workgroup per listed lattice, K sweeps per launch; samples after local
// sweeps s with (s + 1) % every == 0 (every > 0).  lds_bytes > 0 keeps the
// lattice in LDS (it must fit; call set_resident_lds first, outside any
// graph capture).
hipError_t set_resident_lds(int wpt, size_t lds_bytes);
hipError_t launch_resident(int wpt, int block, const LatticeDesc* descs, LatticeState* states, const int32_t* ids,
                           int32_t n_ids, int32_t K, int32_t every, size_t lds_bytes, hipStream_t s);
// Current E and M into states[i].last_E / last_M for the lattices ids[0..n)
// (ids null: lattices 0..n), and E, M and the state's `abandoned` into the
// kObservedWords words out[kObservedWords k ...] for the k-th listed lattice when out
// is non-null; max_words: the words of the largest.
constexpr int kObservedWords = 3;
hipError_t launch_observe_multi(const LatticeDesc* descs, LatticeState* states, const int32_t* ids, int32_t n_lat,
                                int64_t max_words, int64_t* out, hipStream_t s);
// Zero the sample accumulators of every lattice; start a call (series_idx = 0).
hipError_t launch_reset_sums(LatticeState* states, int32_t n_lat, hipStream_t s);
hipError_t launch_begin_call(LatticeState* states, int32_t n_lat, hipStream_t s);

// ---- multi-sweep LDS tiles --------------------------------------------------

// Dynamic LDS of one tile of interior width w (w >= L: the whole lattice)
// for a launch of K sweeps.  A tile fits if its bytes are at most
// tile_lds_limit(device); allow_tile_lds(device) must have run once before
// the first launch_tiles (outside any graph capture).
size_t tile_lds_bytes(int32_t L, int32_t N, int32_t w, int32_t K);
size_t tile_lds_limit(int device);
hipError_t allow_tile_lds(int device);
// Words per tile of the halo copy for tiles of N word rows and launches of
// up to K sweeps.
int64_t tile_halo_stride(int32_t N, int32_t K);
// A launch of the tiles a.tiles[0 .. n_tiles_launched): the halo columns of
// the tiles narrower than their lattice are first copied into `halo`
// (n_tiles_launched x halo_stride words, halo_stride at least
// tile_halo_stride(N, a.K) for every such tile; 0 and null when every tile
// holds a whole lattice), then the tiles run.
hipError_t launch_tiles(const TileLaunch& a, int32_t n_tiles_launched, int block, size_t lds_bytes, uint64_t* halo,
                        int64_t halo_stride, hipStream_t s);
// The n_samples samples of one resident-tile launch of a batch (partials
// [sample][tile], a lattice's tiles at part_begin .. + part_count) for the
// listed lattices: series entries, moment sums, last E and M, in order.
hipError_t launch_finalize_resident(const LatticeDesc* descs, LatticeState* states, const int32_t* ids,
                                    int32_t n_lat, const Partial* partials, int32_t n_tiles, int32_t n_samples,
                                    hipStream_t s);
// E, M of n_samples samples of one lattice from its tiles' partials, in
// order: series entries idx0 .. idx0 + n_samples - 1, moment sums, and the
// last sample into out_EM[0..1] (each optional).
hipError_t launch_finalize_samples(const Partial* partials, int32_t n_tiles, int32_t n_samples, int32_t L,
                                   int64_t* series_E, int64_t* series_M, int64_t idx0, Moments* mom, int64_t* out_EM,
                                   hipStream_t s);

// The samples of one tile launch (sample_mask, first sweep sweep_off of the
// chunk) for the listed lattices of a batch: series entries, moment sums,
// last E and M, in order.
hipError_t launch_finalize_tiles(const LatticeDesc* descs, LatticeState* states, const int32_t* ids, int32_t n_lat,
                                 const Partial* partials, int32_t n_tiles, uint32_t sample_mask, uint32_t sweep_off,
                                 hipStream_t s);

// ---- resident LDS tiles with boundary exchange -------------------------------

// Dynamic LDS of the resident tiles of a lattice cut into bands of w word
// columns (w >= L: the whole lattice) for workgroups of `block` threads;
// the limit and the one-time attribute as for the tiles above.
size_t persist_lds_bytes(int32_t L, int32_t N, int32_t w, int32_t block);
size_t persist_lds_limit(int device);
// (of a form, below, and of the kernel that holds all of them)
hipError_t allow_persist_lds(int device, int form, size_t lds_bytes);
// How many resident tiles of `block` threads and lds_bytes of LDS the device
// holds at once (a launch must not exceed it).
// beside: how many are sure to find room where other kernels run beside the launch.
hipError_t persist_capacity(int block, size_t lds_bytes, int device, int64_t* tiles, int64_t* beside = nullptr);
// form: persist_form of the tiles of the launch (of the widest one of a lattice), or
// persist_form_any where its lattices' differ.
int persist_form(int32_t L, int32_t N, int32_t w, int block);
int persist_form_any();
hipError_t launch_persist(const PersistLaunch& a, int form, int32_t n_tiles, int block, size_t lds_bytes,
                          hipStream_t s);
// Runs launch(), which enqueues work holding resident tiles on stream s of
// `device`, ordered after the previous such work of this process on that
// device (a stream wait on its completion event), and makes it the previous
// one.  Inside a graph capture of s (then *captured, if given, becomes true), or
// with another device current, launch() runs unordered.
hipError_t resident_gate(int device, hipStream_t s, const std::function<hipError_t()>& launch,
                         bool* captured = nullptr);
// How many handles of the device hold resident launches that a caller has captured
// and may replay at any time beside others, after adding n.
int resident_captures(int device, int n = 0);
// The n_samples samples of one resident-tile launch of a batch (partials
// [sample][tile], a lattice's tiles at part_begin .. + part_count) for the
// listed lattices: series entries, moment sums, last E and M, in order.
hipError_t launch_finalize_resident(const LatticeDesc* descs, LatticeState* states, const int32_t* ids,
                                    int32_t n_lat, const Partial* partials, int32_t n_tiles, int32_t n_samples,
                                    hipStream_t s);
// E, M of n_samples samples of one lattice from its tiles' partials
// (sample k in partials[k n_tiles ...]) into out_E[k], out_M[k], then, with
// mom, added to the moment sums in order.
hipError_t launch_samples(const Partial* partials, int32_t n_tiles, int32_t n_samples, int32_t L, int64_t* out_E,
                          int64_t* out_M, Moments* mom, hipStream_t s);

// ---- small lattices with their draws taken ahead ----------------------------

// One workgroup per listed lattice, the lattice and the acceptance codes of
// `batch` sweeps (2..64) in LDS (small_lds_bytes), K sweeps, samples as
// launch_resident.  launch_resident uses it for LDS-resident lattices whose
// codes of two or more sweeps fit beside them.
size_t small_lds_bytes(int32_t L, int32_t N, int32_t batch);
size_t small_lds_limit(int device);
hipError_t allow_small_lds(int device);
hipError_t launch_small(int block, const LatticeDesc* descs, LatticeState* states, const int32_t* ids, int32_t n_ids,
                        int32_t K, int32_t every, int32_t batch, size_t lds_bytes, hipStream_t s);

// ---- small lattices with their draws spread over the chip --------------------

// Draw pass: the acceptance codes of sweeps [sweep_off, sweep_off + S) of
// the current chunk of each listed lattice into codes (DrawLat layout);
// max_n_draw = the largest n_draw of the list.
hipError_t launch_draw_codes(const LatticeDesc* descs, const LatticeState* states, const DrawLat* lats, int32_t n_lats,
                             int32_t max_n_draw, uint64_t* codes, int32_t sweep_off, int32_t S, hipStream_t s);
// Apply pass over the same sweeps: one workgroup of `block` threads (a
// multiple of 64; at most 256, or 1024 with one or two words per thread) per listed
// lattice, wmax (1 to 4: wave_apply_words_per_thread) words of a colour per thread, codes loaded
// from the buffer into registers ahead of use; lds_bytes =
// wave_apply_lds_bytes(largest N L, S).  Samples as launch_resident.
hipError_t launch_wave_apply(int wmax, int block, const LatticeDesc* descs, LatticeState* states, const DrawLat* lats,
                             int32_t n_lats, const uint64_t* codes, int32_t sweep_off, int32_t S, int32_t every,
                             size_t lds_bytes, hipStream_t s);
// (at most 48 KB: 2040 words and 4096 samples, so that no kernel needs leave for
// more than the 64 KB that every launch may use)
size_t wave_apply_lds_bytes(int32_t NL, int32_t max_samples);
// Threads of an apply workgroup of lattices of up to `words` words of a colour,
// wmax of them per thread: no wavefront without words, as an idle one still takes
// part in every barrier (8 lattices of L = 16: 0.40 us a sweep with four
// wavefronts, 0.30 with one, which needs no barrier).
int32_t wave_apply_block(int32_t words, int32_t wmax);
// Words of one colour per thread of a `block`-thread apply workgroup (0:
// more than 4).
int32_t wave_apply_words_per_thread(int32_t L, int32_t N, int32_t block);

// One lattice of a handle with its draws spread over the chip: a launch applies
// the n_apply sweeps whose codes the launch before drew, and draws the n_draw
// sweeps from t_draw on for the next one (either may be 0).
constexpr int32_t kDrawnMaxSweeps = 256;  // of one launch
struct DrawnLaunch {
    uint64_t* W;
    int32_t L, N, istar, sh_star;
    uint32_t k0, k1;
    uint64_t t_draw;
    uint64_t* drawn;        // n_draw x N L codes
    const uint64_t* codes;  // n_apply x N L codes
    uint32_t t4, t8;        // of the sweeps drawn
    int32_t n_draw, n_apply;
    // a sample after the applied sweep j when (sweep_off + j + 1) % every == 0
    // (every > 0; sampled_as); each output may be null
    int32_t sweep_off, every;
    int64_t* series_E;
    int64_t* series_M;
    Moments* mom;
};
// sweep_off and every of a launch of n sweeps, `done` sweeps after the start of a
// run sampled after every every-th: as they are, or, where the launch holds a
// sample at most, smaller ones that say the same, so that their sum with n, which
// the kernel divides, does not overflow at intervals near 2^31.
inline void sampled_as(DrawnLaunch& a, int64_t done, int32_t n, int32_t every) {
    a.every = every;
    a.sweep_off = every > 0 ? (int32_t)(done % every) : 0;
    if (every <= 2 * kDrawnMaxSweeps) return;
    const int32_t left = every - a.sweep_off;  // sweeps to the next sample
    a.every = left <= n ? 2 * kDrawnMaxSweeps : 0;
    a.sweep_off = left <= n ? a.every - left : 0;
}
int32_t drawn_max_words();  // most words of a colour of such a lattice
hipError_t launch_drawn(const DrawnLaunch& a, hipStream_t s);
// LDS of such a launch, to be compared with resident_lds_limit.
size_t drawn_lds_bytes(int32_t L, int32_t N);

// Largest dynamic LDS a resident workgroup may use on this device.
size_t resident_lds_limit(int device);

}  // namespace ising
