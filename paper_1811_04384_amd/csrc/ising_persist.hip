// Resident LDS tiles that exchange their boundary columns: many sweeps per
// launch with no redundant work.
//
// Every word row of a band of word columns [c0, c0 + w) of a lattice stays in
// one workgroup's LDS for all sweeps of a launch, beside two ghost columns
// (c0 - 1 and c0 + w, modulo L) holding copies of the neighbouring tiles'
// boundary words.  This is the paper's decomposition (Sections 4 and 5.2,
// Figs. 3 and 5: each process owns a vertical strip of the word lattice and
// trades its border columns with the processes beside it), with the
// workgroups of one GPU in the place of the MPI processes and the
// checkerboard in the place of the two-phase protocol.  Half-sweep s of
// colour c in a tile is one pass over its words of colour c:
//   - the boundary words (local columns 1 and w) come first; each reads its
//     ghost neighbour straight from the neighbouring tile's publication of
//     half-sweep s - 1 (from LDS in a launch's first half-sweep) and is
//     published at once to an exchange buffer in global memory;
//   - then the interior words (columns 2 .. w - 1), while the boundary words
//     travel, and the Philox blocks of the next half-sweep's position 20
//     (and, with at most two words of a colour per thread, the acceptance
//     codes of the next half-sweep's words, drawn into an LDS code table:
//     by the interior words' wavefronts while their own loads are in flight,
//     by the boundary words' wavefronts after they have published, so that
//     the neighbours never wait for draws).
// A published word carries its own tag in the two bits of every field that
// the spin coding leaves 0: the half-sweep in the middle bits and the launch
// in the upper ones.  A reader polls the word itself until the tag is the one
// it waits for, so that one store and one load are all that lies between the
// update of a boundary word and its use next door; no flag is raised behind
// the data and no store is waited for.  Small bands are bound by that path:
// 126 bands of 8 columns of L = 1008 take 1.25 us per half-sweep, against 2.69
// with a flag per tile, raised after every publisher's store had completed
// and polled before the barrier (three memory round trips after each other);
// bands of 16 columns (L = 4096: 3.79 against 3.97 us) are bound by the
// vector unit.
// Only colour-c words are exchanged, because the next half-sweep only reads
// those from a ghost column.  The exchange buffer alternates between two
// halves on the half-sweep's parity: a tile overwrites a half two
// half-sweeps later, after its neighbours have published the half-sweep that
// read it (each publisher reads its ghost word before it publishes, and this
// tile has read theirs).
//
// Every tile of a launch must be resident at once (the host launches at most
// as many tiles as the device holds).  Each wait is bounded in time: when
// it expires the launch sets an error word and every tile stops waiting, so
// a launch always ends; the host reports the error.
//
// A lattice with a single tile (w = L) keeps all its columns in LDS and
// wraps them there: no exchange at all.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <vector>

#include "ising_device.hpp"
#include "ising_launch.hpp"
#include "ising_lds_word.hpp"
#include "ising_moments.hpp"

namespace ising {

namespace {

constexpr int kPersistMaxBlock = 1024;
constexpr uint32_t kMaxPolls = 1u << 21;

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ uint64_t clock_ticks() { return __builtin_amdgcn_s_memrealtime(); }

// One word item of a half-sweep: the LDS addresses of the word and of its
// neighbourhood words, the byte offset of its position-20 uniform in the
// table of the half-sweep, its Philox counter word I L + J, its row and its
// side (-1 interior, 0 the left boundary column, 1 the right one).
struct WordItem {
    uint32_t w, lf, rt, up, dn, patch, u20, c1;
    int32_t I, side;
};

// What drawing a word's codes takes: its row and its Philox counter.
struct DrawItem {
    int32_t I;
    uint32_t c1;
};

// The tag bits of a published word: the middle bit of every field counts the
// launch's half-sweeps, the upper bit the launches of the tile's table.  A
// number is kept with its bits spread to those places; adding one carries
// through the bits between them when these are set first.
constexpr uint64_t kStepBits = kSpinBits << 1;
constexpr uint64_t kLaunchBits = kSpinBits << 2;
template <uint64_t BITS>
__device__ __forceinline__ uint64_t spread_next(uint64_t tag) {
    return ((tag | ~BITS) + 1) & BITS;
}

// How a tile's threads hold its word items: formed in every half-sweep, or
// once per launch with one or two items per thread and colour.
// kAny: a kernel whose tiles choose.
enum Items { kFormed, kOne, kTwo, kAny };

__host__ __device__ constexpr Items items_mode(int n_w, int block) {
    return n_w <= block ? kOne : n_w <= 2 * block ? kTwo : kFormed;
}

// Word items of a colour of a tile.
__host__ __device__ __forceinline__ int tile_items(int L, int N, int tile_w) {
    return tile_w >= L ? N * (L >> 1) : N + N * ((tile_w - 2) >> 1);
}

// One tile's launch.  WHOLE: the tile is the whole lattice.
template <int ITEMS, bool WHOLE>
__device__ __forceinline__ void persist_tile(const PersistLaunch& a, const PersistTile& tp, uint64_t* lds,
                                             uint32_t* red, int& stop) {
    const LatticeDesc& d = a.descs[tp.lattice];
    const int L = d.L, N = d.N, istar = d.istar, sh_star = d.sh_star;
    const int pstar = (L - 1) / N;
    uint64_t t0;
    uint32_t t4, t8, k0, k1;
    if (a.states) {
        t0 = a.states[tp.lattice].t + a.sweep_off;
        k0 = d.k0;
        k1 = d.k1;
        t4 = d.t4;
        t8 = d.t8;
    } else {
        t0 = a.t0;
        k0 = a.k0;
        k1 = a.k1;
        t4 = a.t4;
        t8 = a.t8;
    }
    const int K = a.K;
    constexpr bool whole = WHOLE;
    const int w = whole ? L : tp.w;
    const int width = whole ? L : w + 2;  // local column x <-> global c0 - 1 + x (halo form)
    const int gx0 = whole ? 0 : (tp.c0 == 0 ? L - 1 : tp.c0 - 1);
    auto col = [&](int x) {
        const int u = gx0 + x;
        return u < L ? u : u - L;
    };
    // position-20 blocks: one per (8-column group, row) of the interior
    // columns, for the current half-sweep
    const int xi0 = whole ? 0 : 1, xi1 = whole ? L : w + 1;  // interior local columns [xi0, xi1)
    const int g_lo = col(xi0) >> 3;
    const int g_hi_raw = col(xi1 - 1) >> 3;
    // the interior never wraps past the lattice end (tiles start at c0 >= 0
    // and end at c0 + w <= L), so its groups are g_lo .. g_hi_raw
    const int n_groups = g_hi_raw - g_lo + 1;
    uint64_t* __restrict__ T = lds;
    // two tables [n_groups][N]: this half-sweep's and the next one's
    uint4* __restrict__ u5tab = reinterpret_cast<uint4*>(lds + (size_t)N * width);
    const int tid = threadIdx.x, B = blockDim.x;
    const RoundKeys rk = round_keys(k0, k1);
    const bool all_blocks = pstar >= 16;
    auto sweep_of = [&](int hs) {  // half-sweep hs (0-based) of the launch
        const uint64_t t = t0 + (uint64_t)(hs >> 1);
        return LdsSweep{L, N, istar, sh_star, pstar, (uint32_t)t, (uint32_t)(t >> 32), k0, k1, t4, t8, all_blocks};
    };
    if (tid == 0) stop = 0;
    // the tag of this launch: every tile of a lattice counts the same launches
    const uint64_t launch_tag = a.flags[blockIdx.x];

    // load the band and its ghost columns, eight loads in flight per thread
    {
        constexpr int kInFlight = 8;
        const float rcp = 1.0f / (float)width;
        const int n = N * width;
        const uint64_t* __restrict__ G = d.W;
        for (int i0 = tid; i0 < n; i0 += kInFlight * B) {
            uint64_t v[kInFlight];
#pragma unroll
            for (int k = 0; k < kInFlight; ++k) {
                const int i = i0 + k * B;
                if (i < n) {
                    int I, x;
                    divmod_small(i, width, rcp, I, x);
                    v[k] = G[(size_t)((uint32_t)I * (uint32_t)L + (uint32_t)col(x))];
                }
            }
#pragma unroll
            for (int k = 0; k < kInFlight; ++k)
                if (i0 + k * B < n) T[i0 + k * B] = v[k];
        }
    }
    {  // position-20 blocks of the first half-sweep
        const LdsSweep sw0 = sweep_of(0);
        const float rcp = 1.0f / (float)n_groups;
        for (int f = tid; f < N * n_groups; f += B) {
            int I, k;
            divmod_small(f, n_groups, rcp, I, k);
            if (pstar + (I <= istar ? 1 : 0) == 21) u5tab[(size_t)k * N + I] = block5(sw0, rk, I, g_lo + k, 0);
        }
    }
    __syncthreads();

    const int n_hs = 2 * K;
    const int n_b = whole ? 0 : N;                  // boundary items (columns 1 and w)
    const int P = whole ? (L >> 1) : ((w - 2) >> 1);  // interior words of a colour per row
    const int n_i = N * P;
    const float rcp_P = P > 0 ? 1.0f / (float)P : 0.0f;
    const float rcp_g = 1.0f / (float)n_groups;
    const int64_t tw = a.exch_tile_words;
    const int n_w = n_b + n_i;  // word items of a half-sweep (tile_items)
    // wavefronts with a boundary word in their first / second item
    const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~63);
    const bool edge0 = wave0 < n_b, edge1 = wave0 + B < n_b;
    const lds_u64* T3 = (const lds_u64*)T;
    // word item f of a half-sweep of colour c: boundary items first (items
    // f < N/2 in column 1, the others in column w, on the rows with
    // (I + J) % 2 == c), then the interior words row by row
    auto make_item = [&](int f, int c) {
        int I, x, side = -1;
        if (f < n_b) {
            side = f >= (N >> 1) ? 1 : 0;
            x = side ? w : 1;
            I = 2 * (f - side * (N >> 1)) + ((col(x) + c) & 1);
        } else {
            int q;
            divmod_small(f - n_b, P, rcp_P, I, q);
            x = whole ? 2 * q + ((I + c) & 1) : 2 + 2 * q + ((2 + gx0 + I + c) & 1);
        }
        const int J = col(x);
        const int xl = whole && x == 0 ? L - 1 : x - 1;
        const int xr = whole && x == L - 1 ? 0 : x + 1;
        const int row = I * width;
        WordItem it;
        it.w = lds_addr(T3 + row + x);
        if (WHOLE) {  // otherwise the words beside it in the band
            it.lf = lds_addr(T3 + row + xl);
            it.rt = lds_addr(T3 + row + xr);
        }
        it.up = lds_addr(T3 + (I > 0 ? I - 1 : N - 1) * width + x);
        it.dn = lds_addr(T3 + (I < N - 1 ? I + 1 : 0) * width + x);
        // the patch word (row I* for I = 0, row 0 for I = I*); other rows
        // read row 0 and ignore it
        it.patch = lds_addr(T3 + (I == 0 ? istar : 0) * width + x);
        it.u20 = 16u * (uint32_t)(((J >> 3) - g_lo) * N + I) + 4u * (((uint32_t)J >> 1) & 3u);
        it.c1 = (uint32_t)I * (uint32_t)L + (uint32_t)J;
        it.I = I;
        it.side = side;
        return it;
    };
    // With at most two word items per thread and colour (kOne, kTwo: the usual
    // tile shapes), every thread's items are the same in every half-sweep of a
    // colour and are formed once, and the codes of positions 0..19 of every
    // word are drawn a half-sweep ahead into a code table (two, by the
    // half-sweep's parity, after the position-20 tables): in a half-sweep a
    // thread updates its words from the table and draws the codes of its
    // words of the other colour for the next one, while the loads of the
    // word's neighbourhood are in flight.  With at most one item per thread
    // (kOne: small bands, whose half-sweep is as long as the exchange of the
    // boundary words) the codes are drawn by the threads from the last
    // one down instead, so that the boundary words' wavefronts have nothing
    // else to do.  Otherwise every item is formed and drawn in its half-sweep.
    constexpr bool pre = ITEMS != kFormed;
    constexpr bool split = ITEMS == kOne;
    const uint32_t ctab = lds_addr((const lds_u64*)(u5tab + (size_t)2 * n_groups * N));
    WordItem cur0{}, cur1{}, oth0{}, oth1{};  // word items, this colour and the other
    DrawItem dcur0{}, dcur1{}, doth0{}, doth1{};  // the items whose codes this thread draws
    const int f0 = split ? B - 1 - tid : tid, f1 = tid + B;
    // Two words per thread of a band keep the vector unit busy: the form with
    // fewer instructions (heating of 16 lattices of L = 1008 2670 us with selects,
    // 2600 with it).  Whole lattices wait for their slowest wavefront at every
    // half-sweep: selects (us per sweep, without / with them: one of L = 64 in a
    // wavefront 4.48 / 4.27, 256 of L = 128 in four 4.90 / 4.64, 1024 of them
    // 8.66 / 8.71, 256 of L = 192 in eight 6.33 / 5.98).
    typedef std::conditional_t<ITEMS == kTwo && !WHOLE, AcceptWord, AcceptSelect> Accept;
    auto draw_codes = [&](const DrawItem& it, int f, const LdsSweep& swc, uint32_t table) {
        // the sweep index made opaque to the compiler (see the words below)
        LdsSweep swi = swc;
        asm volatile("" : "+s"(swi.t_lo), "+s"(swi.t_hi));
        lds_store64(table + 8u * (uint32_t)f, lds_word_codes<Accept>(swi, rk, it.I, it.c1));
    };
    if (pre) {
        // a thread without an item holds the last one's addresses: its loads
        // are in bounds and not used
        cur0 = make_item(min(tid, n_w - 1), 0);
        oth0 = make_item(min(tid, n_w - 1), 1);
        if (tid >= n_w) cur0.side = oth0.side = -1;
        if (!split) {
            cur1 = make_item(min(f1, n_w - 1), 0);
            oth1 = make_item(min(f1, n_w - 1), 1);
            dcur1 = {cur1.I, cur1.c1};
            doth1 = {oth1.I, oth1.c1};
            if (f1 >= n_w) cur1.side = oth1.side = -1;
        }
        if (f0 < n_w) {
            const WordItem d0 = make_item(f0, 0), d1 = make_item(f0, 1);
            dcur0 = {d0.I, d0.c1};
            doth0 = {d1.I, d1.c1};
        }
        // the codes of the first half-sweep
        const LdsSweep sw0 = sweep_of(0);
        if (f0 < n_w) draw_codes(dcur0, f0, sw0, ctab);
        if (!split && f1 < n_w) draw_codes(dcur1, f1, sw0, ctab);
        __syncthreads();
    }
    // the next half-sweep's position-20 blocks (of the rows with 21 live
    // positions) are dealt to the threads in rank order, items rank5,
    // rank5 + E5, ...  When the last round of words is partial, none go to
    // the wavefronts 0, 4, 8, ... (a workgroup's wavefronts go to the four
    // SIMDs in turn, so those share the SIMD that carries the most rounds
    // of words) and threads with fewer word items come first; otherwise the
    // threads in order (the oldest wavefronts, which the instruction arbiter
    // favours, first).  Both orders were the faster one in their case.
    const int rows21 = pstar == 20 ? istar + 1 : 0;
    const int r0 = n_w % B;  // threads below r0 have one word item more
    const bool skip0 = B >= 256 && (r0 & 255) != 0;
    auto elig_before = [&](int x) {  // eligible threads below x
        return skip0 ? x - ((x >> 8) * 64 + min(x & 255, 64)) : x;
    };
    const int E5 = elig_before(B);
    const int rank5 = !skip0                       ? tid
                      : ((tid >> 6) & 3) == 0       ? -1
                      : tid >= r0                   ? elig_before(tid) - elig_before(r0)
                                                    : E5 - elig_before(r0) + elig_before(tid);
    // the launch's next sampled sweep (a sample after sweep j iff
    // (sample_base + j + 1) % every == 0; -1 for none) and the samples taken
    // so far: counted, not divided out per half-sweep (a 64-bit division is
    // a long scalar routine)
    int64_t next_sample = a.every > 0 ? (int64_t)a.every - 1 - a.sample_base % a.every : -1;
    int n_taken = 0;
    auto fetch = [&](const uint64_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    // one ghost word, first read as v: polled until it carries the tag
    // `want`.  Bounded twice, by the clock (a failed poll counts for at least
    // 100 ns) and by the number of polls; when a bound is reached, or another
    // tile has set the error word, the launch is abandoned after this
    // sweep, whose number from 1 on `stop` holds: a wavefront that is already in the
    // next one when another reads it puts that one's number there, and all of them
    // leave after the same sweep (read after every half-sweep, L = 1008 2.45 us per
    // sweep, 2.36 so; 4096 7.61 / 7.48).  In small bands (kOne), whose half-sweep waits for these words
    // alone, two more reads follow the first at 0.1 us distance, so that a word
    // that just missed one is not seen a whole round trip later (us per
    // half-sweep with one read at a time / three: L = 300 1.31 / 1.16, 1008 1.34 /
    // 1.29; wider bands gain nothing, L = 4096 3.74 / 3.80).
    auto ghost = [&](const uint64_t* p, uint64_t v, uint64_t want, int hs) -> uint64_t {
        if constexpr (split) {
            __builtin_amdgcn_s_sleep(4);  // 256 cycles
            uint64_t v1 = fetch(p);
            __builtin_amdgcn_s_sleep(4);
            uint64_t v2 = fetch(p);
            if ((v & ~kSpinBits) != want) {
                const uint64_t start = clock_ticks() - 10;
                uint32_t err = 0;  // read behind the words, checked a round later
                for (uint32_t polls = 0;; ++polls) {
                    v = v1;
                    if ((v & ~kSpinBits) == want) break;
                    v1 = fetch(p);
                    v = v2;
                    if ((v & ~kSpinBits) == want) break;
                    v2 = fetch(p);
                    if (err != 0u || clock_ticks() - start > a.wait_ticks || polls > kMaxPolls) {
                        __hip_atomic_store(a.error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        stop = (hs >> 1) + 1;
                        break;
                    }
                    err = __hip_atomic_load(a.error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        } else if ((v & ~kSpinBits) != want) {
            const uint64_t start = clock_ticks() - 10;
            for (uint32_t polls = 0;; ++polls) {
                if (__hip_atomic_load(a.error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u ||
                    clock_ticks() - start > a.wait_ticks || polls > kMaxPolls) {
                    __hip_atomic_store(a.error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    stop = (hs >> 1) + 1;
                    break;
                }
                v = fetch(p);
                if ((v & ~kSpinBits) == want) break;
            }
        }
        return v & kSpinBits;
    };
    uint64_t step_tag = 0;  // tag of the half-sweep before (0: none in this launch)
    uint64_t ghost0 = 0;    // the ghost word of this half-sweep's first item (code-table mode)
    // one half-sweep: the word items of its colour (cur0, cur1), the first
    // item of the next one (oth0) and the items whose codes it draws for the
    // next one (d0, d1)
    auto half_sweep = [&](const int hs, const WordItem& cur0, const WordItem& cur1, const WordItem& oth0,
                          const DrawItem& d0, const DrawItem& d1) __attribute__((always_inline)) {
        const int c = hs & 1;
        const int j = hs >> 1;
        const LdsSweep sw = sweep_of(hs);
        const bool meas = c == 1 && j == next_sample;
        const uint32_t u5cur_addr = lds_addr((const lds_u64*)(u5tab + (size_t)(hs & 1) * n_groups * N));
        uint4* __restrict__ u5next = u5tab + (size_t)((hs + 1) & 1) * n_groups * N;
        const int n_u = hs + 1 < n_hs ? rows21 * n_groups : 0;
        const LdsSweep sw_next = sweep_of(hs + 1);
        // where the neighbours publish the ghost words of a boundary item
        // that follows a half-sweep of colour cc: the left one's right side,
        // the right one's left side
        auto ghost_at = [&](const WordItem& it, int cc) -> const uint64_t* {
            return it.side == 0 ? a.exch + (size_t)tp.left * tw + (size_t)cc * 2 * N + N + it.I
                                : a.exch + (size_t)tp.right * tw + (size_t)cc * 2 * N + it.I;
        };
        uint64_t* __restrict__ ex = a.exch + (size_t)blockIdx.x * tw + (size_t)c * 2 * N;
        const uint64_t want = step_tag | launch_tag;
        step_tag = spread_next<kStepBits>(step_tag);
        const uint64_t tag = step_tag | launch_tag;
        uint32_t anti = 0, ups = 0;
        bool fetch0 = false;
        // one word item: its neighbourhood from LDS (the ghost word of a
        // boundary item straight from the neighbour's publication after the
        // launch's first half-sweep) and the word `early` gives, then
        // `between` (while the loads are in flight; after the update in a
        // wavefront with boundary words, whose readers wait for it), the
        // update (by `update`, from the neighbourhood, the position-20
        // uniform and that word), and the publication of a boundary word.
        // valid: whether the thread has this item.
        auto poll = [&](const WordItem& it) {
            const uint64_t* p = ghost_at(it, 1 - c);
            return ghost(p, fetch(p), want, hs);
        };
        auto word = [&](const WordItem& it, bool valid, bool edge, auto ghost_of, auto early, auto between, auto update) {
            Nbhd nb;
            nb.w = lds_load64(it.w);
            nb.lf = lds_load64(WHOLE ? it.lf : it.w - 8u);
            nb.rt = lds_load64(WHOLE ? it.rt : it.w + 8u);
            nb.up = lds_load64(it.up);
            nb.dn = lds_load64(it.dn);
            nb.patch = lds_load64(it.patch);
            const uint32_t u20 = lds_load32(u5cur_addr + it.u20);
            const uint64_t e = early(it);
            if (edge && valid) {
                if (it.side >= 0 && hs > 0) {
                    const uint64_t g = ghost_of(it);
                    nb.lf = it.side == 0 ? g : nb.lf;
                    nb.rt = it.side == 0 ? nb.rt : g;
                }
                const uint64_t nw = update(it, nb, u20, e);
                if (it.side >= 0)
                    __hip_atomic_store(&ex[it.side * N + it.I], nw | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                lds_store64(it.w, nw);
            }
            between();
            if (!edge && valid) lds_store64(it.w, update(it, nb, u20, e));
        };
        if (pre) {
            // the words from the code table of this half-sweep; meanwhile the
            // codes of the same threads' words of the other colour for the
            // next half-sweep into the other table
            const uint32_t ccur = ctab + (uint32_t)(hs & 1) * 8u * (uint32_t)n_w;
            const uint32_t cnext = ctab + (uint32_t)((hs + 1) & 1) * 8u * (uint32_t)n_w;
            const bool draw = hs + 1 < n_hs;
            auto codes = [&](int f) { return [=](const WordItem&) { return lds_load64(ccur + 8u * (uint32_t)f); }; };
            auto from_table = [&](const WordItem& it, const Nbhd& nb, uint32_t u20, uint64_t cd) {
                return lds_word_apply(sw, nb, it.I, cd, u20, meas, true, anti, ups);
            };
            word(cur0, tid < n_w, edge0, [&](const WordItem&) { return ghost0; }, codes(min(tid, n_w - 1)),
                 [&] { if (draw && f0 < n_w) draw_codes(d0, f0, sw_next, cnext); }, from_table);
            // the ghost word of the next half-sweep's first item, on its way
            // while the second item and the position-20 blocks are worked on
            fetch0 = draw && edge0 && oth0.side >= 0;
            if (fetch0) ghost0 = fetch(ghost_at(oth0, c));
            if (!split)
                word(cur1, f1 < n_w, edge1, poll, codes(min(f1, n_w - 1)),
                     [&] { if (draw && f1 < n_w) draw_codes(d1, f1, sw_next, cnext); }, from_table);
        } else {
            // the words f = tid, tid + B, ..., each drawing its own codes:
            // the sweep index made opaque to the compiler, so that the
            // wave-uniform parts of the Philox rounds are formed per item on
            // the scalar unit instead of being hoisted out of the loop for
            // all five blocks (which overflows the scalar registers into
            // vector-lane spills)
            auto drawing = [&](const WordItem& it, const Nbhd& nb, uint32_t u20, uint64_t) {
                LdsSweep swi = sw;
                asm volatile("" : "+s"(swi.t_lo), "+s"(swi.t_hi));
                return lds_word_update_c1(swi, rk, nb, it.I, it.c1, u20, meas, true, anti, ups);
            };
            auto none = [](const WordItem&) { return 0ull; };
            for (int fw = tid; fw < n_w; fw += B) word(make_item(fw, c), true, true, poll, none, [] {}, drawing);
        }
        // then the next half-sweep's position-20 blocks, in a loop of their
        // own so that it keeps only its own wave-uniform values live
        if (rank5 >= 0) {
            for (int b = rank5; b < n_u; b += E5) {
                int I, k;
                divmod_small(b, n_groups, rcp_g, I, k);
                u5next[(size_t)k * N + I] = block5(sw_next, rk, I, g_lo + k, c ^ 1);
            }
        }
        if (fetch0) ghost0 = ghost(ghost_at(oth0, c), ghost0, tag, hs);
        if (meas) {
            if (pre) {
                // at most two words per thread: a wavefront's antiparallel
                // bonds (at most 168 per thread) and up spins (84) each fit
                // in 16 bits, so one sum covers both
                const uint32_t both = wave_sum_u32((anti << 16) | ups);
                anti = both >> 16;
                ups = both & 0xFFFFu;
            } else {
                anti = wave_sum_u32(anti);
                ups = wave_sum_u32(ups);
            }
            if (lane_id() == 0) {
                red[2 * (tid >> 6)] = anti;
                red[2 * (tid >> 6) + 1] = ups;
            }
        }
        __syncthreads();
        if (meas && tid >= B - 64) {
            // the tile's sums, by the last wavefront: lane l reads
            // wavefront l's pair, one sum over the lanes for each count
            const int l = tid - (B - 64);
            const bool in = l < (B >> 6);
            const uint32_t sa = wave_sum_u32(in ? red[2 * l] : 0u), su = wave_sum_u32(in ? red[2 * l + 1] : 0u);
            if (l == 0) a.partials[(size_t)n_taken * a.n_tiles + tp.part] = {sa, su};
        }
        if (meas) {
            next_sample += a.every;
            ++n_taken;
        }
    };
    if (pre) {
        // two half-sweeps per trip, so that the items of each colour stay in
        // the same registers (no exchange of the two sets between half-sweeps)
        for (int hs = 0; hs < n_hs; hs += 2) {
            half_sweep(hs, cur0, cur1, oth0, doth0, doth1);
            half_sweep(hs + 1, oth0, oth1, cur0, dcur0, dcur1);
            if (stop == (hs >> 1) + 1) break;
        }
    } else {
        for (int hs = 0; hs < n_hs; ++hs) {
            half_sweep(hs, cur0, cur1, oth0, doth0, doth1);
            if ((hs & 1) && stop == (hs >> 1) + 1) break;
        }
    }
    // the ghost columns in LDS are stale past the first half-sweep, but the
    // band's own words are exact
    if (tid == 0) a.flags[blockIdx.x] = spread_next<kLaunchBits>(launch_tag);  // also when abandoned

    // store the band (the ghost columns belong to the neighbours)
    {
        const float rcp = 1.0f / (float)w;
        uint64_t* __restrict__ G = d.W;
        for (int i = tid; i < N * w; i += B) {
            int I, xi;
            divmod_small(i, w, rcp, I, xi);
            const int x = xi0 + xi;
            G[(size_t)((uint32_t)I * (uint32_t)L + (uint32_t)col(x))] = T[I * width + x];
        }
    }
}

}  // namespace

// ITEMS: how the tiles of the launch hold their items, WHOLE: whether they are whole
// lattices (kAny: the lattices of the launch differ, and each tile chooses).  A kernel
// of each form by itself has the registers it needs and no others' (us per sweep,
// all of them in one kernel / each alone: L = 300 2.33 / 2.25, 512 2.41 / 2.32, 1024
// 2.64 / 2.53, 2048 3.48 / 3.38, 3072 5.60 / 5.42, 4096 7.66 / 7.58; 16 lattices of L =
// 512 in bands of 64 columns, 300 sampled sweeps 1830 / 1800; 256 whole lattices of L
// = 256 by 1024 threads 7.76 / 7.58).  Bands whose items are formed in every half-sweep
// have none of their own: with it they are the slower ones (L = 4610 13.3 / 13.8, 5120
// 14.4 / 14.9, 6144 19.5 / 20.2, 7680 31.3 / 31.9; 16 of L = 1008 in bands of 64 columns
// by 512 threads 10.6 / 10.9).
template <int ITEMS, bool WHOLE>
__global__ void __launch_bounds__(kPersistMaxBlock) k_persist(PersistLaunch a) {
    extern __shared__ uint64_t lds[];
    __shared__ uint32_t red[2 * (kPersistMaxBlock / 64)];
    __shared__ int stop;
    const PersistTile tp = a.tiles[blockIdx.x];
    if constexpr (ITEMS != kAny) {
        persist_tile<ITEMS, WHOLE>(a, tp, lds, red, stop);
    } else {
        const LatticeDesc& d = a.descs[tp.lattice];
        const bool whole = tp.w >= d.L;
        switch (items_mode(tile_items(d.L, d.N, tp.w), blockDim.x)) {
            case kOne:
                if (whole) persist_tile<kOne, true>(a, tp, lds, red, stop);
                else persist_tile<kOne, false>(a, tp, lds, red, stop);
                break;
            case kTwo:
                if (whole) persist_tile<kTwo, true>(a, tp, lds, red, stop);
                else persist_tile<kTwo, false>(a, tp, lds, red, stop);
                break;
            default:
                if (whole) persist_tile<kFormed, true>(a, tp, lds, red, stop);
                else persist_tile<kFormed, false>(a, tp, lds, red, stop);
        }
    }
}

namespace {

constexpr int kWhole = 4;  // added to the items of a form

typedef void (*PersistKernel)(PersistLaunch);
PersistKernel persist_kernel(int form) {
    switch (form) {
        case kOne: return &k_persist<kOne, false>;
        case kTwo: return &k_persist<kTwo, false>;
        case kOne + kWhole: return &k_persist<kOne, true>;
        case kTwo + kWhole: return &k_persist<kTwo, true>;
        case kFormed + kWhole: return &k_persist<kFormed, true>;
        default: return &k_persist<kAny, false>;
    }
}

}  // namespace

int persist_form(int32_t L, int32_t N, int32_t w, int block) {
    return items_mode(tile_items(L, N, w), block) + (w >= L ? kWhole : 0);
}
int persist_form_any() { return kAny; }

size_t persist_lds_bytes(int32_t L, int32_t N, int32_t w, int32_t block) {
    // a tile of width wi: its band with the ghost columns, two position-20
    // tables (a bound on their groups) and, with at most two word items per
    // thread and colour, two code tables; the widest need of the lattice's
    // tiles (all of width w but the last)
    auto need = [&](int64_t wi) {
        const bool whole = wi >= L;
        const int64_t width = whole ? L : wi + 2;
        const int64_t groups = whole ? (L + 7) / 8 : wi / 8 + 2;
        const int64_t items = (int64_t)N * (whole ? L : wi) / 2;
        const int64_t codes = items <= 2 * (int64_t)block ? 16 * items : 0;
        return (size_t)(8 * (int64_t)N * width + 2 * 16 * groups * (int64_t)N + codes);
    };
    const int64_t wf = w >= L ? L : w;
    const int64_t last = L - ((L + wf - 1) / wf - 1) * wf;
    return std::max(need(wf), need(last));
}

size_t persist_lds_limit(int device) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, device) != hipSuccess) return 0;
    const size_t static_bytes = sizeof(uint32_t) * 2 * (kPersistMaxBlock / 64) + 256;
    return v > (int)static_bytes ? (size_t)v - static_bytes : 0;
}

hipError_t allow_persist_lds(int device, int form, size_t lds_bytes) {
    // up to 64 KB, static part included, need no leave (setting it takes 10 us)
    if (lds_bytes <= 60 * 1024) return hipSuccess;
    const int limit = (int)persist_lds_limit(device);
    hipError_t e = hipSuccess;
    for (int f : {form, (int)kAny})
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(persist_kernel(f)),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, limit);
    return e;
}

// Beside other kernels a tile's registers and LDS are placed wherever theirs leave
// room, and once those have ended the holes between the tiles may all be too small for
// one more: then tiles wait for neighbours that are never placed (two tiles of 512
// threads per compute unit, launched behind the first of a row of half-sweeps: 30 to
// 40 of the 512 had found no place when the first ones gave up).  With c tiles in a
// compute unit that nothing else uses, k of them leave no hole for another only if
// 2 k + 1 > c, as every hole is smaller than a tile; so half of c, rounded up, is safe.
hipError_t persist_capacity(int block, size_t lds_bytes, int device, int64_t* tiles, int64_t* beside) {
    // of the kernel that holds every form: the others need no more
    int per_cu = 0, cus = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, reinterpret_cast<const void*>(persist_kernel(kAny)), block, lds_bytes);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return e;
    *tiles = (int64_t)per_cu * cus;
    if (beside) *beside = (int64_t)(per_cu + 1) / 2 * cus;
    return hipSuccess;
}

hipError_t launch_persist(const PersistLaunch& a, int form, int32_t n_tiles, int block, size_t lds_bytes,
                          hipStream_t s) {
    if (n_tiles <= 0 || a.K <= 0) return hipSuccess;
    if (block < 64 || block > kPersistMaxBlock || block % 64) return hipErrorInvalidValue;
    hipLaunchKernelGGL(persist_kernel(form), dim3(n_tiles), dim3(block), lds_bytes, s, a);
    return hipGetLastError();
}

// The completion of the last launch that holds resident tiles, per device
// (null until the first one).  Two such launches on different streams could
// each hold compute units that the other's remaining workgroups need, and
// both would then wait out their bound and fail; ordering every one after
// the device's previous one rules that out.
namespace {
std::mutex g_gate_mutex;
std::vector<hipEvent_t> g_gate;
std::vector<int> g_captures;
}  // namespace

int resident_captures(int device, int n) {
    std::lock_guard<std::mutex> lock(g_gate_mutex);
    if (device < 0) return 0;
    if ((size_t)device >= g_captures.size()) g_captures.resize((size_t)device + 1, 0);
    return g_captures[device] += n;
}

hipError_t resident_gate(int device, hipStream_t s, const std::function<hipError_t()>& launch, bool* captured) {
    std::lock_guard<std::mutex> lock(g_gate_mutex);
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    hipError_t e = hipStreamIsCapturing(s, &cs);
    if (e != hipSuccess) return e;
    int current = -1;
    e = hipGetDevice(&current);
    if (e != hipSuccess) return e;
    // inside a capture a dependency on work outside it is not allowed, and
    // the event belongs to the device current when it was made
    if (cs != hipStreamCaptureStatusNone && captured) *captured = true;
    if (cs != hipStreamCaptureStatusNone || device < 0 || current != device) return launch();
    if ((size_t)device >= g_gate.size()) g_gate.resize((size_t)device + 1, nullptr);
    if (g_gate[device]) {
        e = hipStreamWaitEvent(s, g_gate[device], 0);
    } else {
        e = hipEventCreateWithFlags(&g_gate[device], hipEventDisableTiming);
    }
    if (e != hipSuccess) return e;
    e = launch();
    if (e != hipSuccess) return e;
    return hipEventRecord(g_gate[device], s);
}

}  // namespace ising

namespace ising {

namespace {

// E and M of sample k from the tiles' partial sums (one workgroup per
// sample): out_E[k], out_M[k].
__global__ void __launch_bounds__(256) k_samples_em(const Partial* __restrict__ partials, int32_t n_tiles, int32_t L,
                                                    int64_t* __restrict__ out_E, int64_t* __restrict__ out_M) {
    __shared__ unsigned long long red[2 * 4];
    const int k = blockIdx.x;
    unsigned long long anti = 0, ups = 0;
    for (int i = threadIdx.x; i < n_tiles; i += blockDim.x) {
        const Partial p = partials[(size_t)k * n_tiles + i];
        anti += p.anti;
        ups += p.ups;
    }
    anti = wave_sum_u64(anti);
    ups = wave_sum_u64(ups);
    if (lane_id() == 0) {
        red[2 * (threadIdx.x >> 6)] = anti;
        red[2 * (threadIdx.x >> 6) + 1] = ups;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long A = 0, U = 0;
        for (int wv = 0; wv < (int)(blockDim.x + 63) / 64; ++wv) {
            A += red[2 * wv];
            U += red[2 * wv + 1];
        }
        const int64_t n = (int64_t)L * (int64_t)L;
        out_E[k] = 2 * (int64_t)A - 2 * n;
        out_M[k] = 2 * (int64_t)U - n;
    }
}

// Moment sums of n samples added to *mom, by one wavefront: per-lane sums
// of samples l, l + 64, ..., merged exactly.
__global__ void __launch_bounds__(64) k_samples_moments(const int64_t* __restrict__ E, const int64_t* __restrict__ M,
                                                        int32_t n, Moments* mom) {
    Moments part = {};
    for (int k = lane_id(); k < n; k += 64) add_sample(part, E[k], M[k]);
    wave_merge_moments(part);
    if (lane_id() == 0) {
        Moments m = *mom;
        merge_moments(m, part);
        *mom = m;
    }
}

}  // namespace

namespace {

// The samples of one launch of resident tiles for every tiled lattice of a
// batch, one wavefront per listed lattice: lane l takes samples l, l + 64,
// ... (the sum of the lattice's tile partials), writes their E, M to the
// series and adds them to its own moment sums; the lanes' sums are then
// merged exactly, and lane 0 adds them to the lattice's with the last E, M.
__global__ void __launch_bounds__(64) k_finalize_resident(const LatticeDesc* __restrict__ descs,
                                                          LatticeState* __restrict__ states,
                                                          const int32_t* __restrict__ ids,
                                                          const Partial* __restrict__ partials, int32_t n_tiles,
                                                          int32_t n_samples) {
    const int32_t lat = ids[blockIdx.x];
    const LatticeDesc& d = descs[lat];
    LatticeState& st = states[lat];
    const int n = min(n_samples, d.sweep_limit);  // a lattice past its limit took fewer samples
    if (n <= 0) return;
    const int64_t spins = (int64_t)d.L * (int64_t)d.L;
    const int64_t idx = st.series_idx;
    Moments part = {};
    int64_t E = 0, M = 0;
    for (int o = lane_id(); o < n; o += 64) {
        unsigned long long anti = 0, ups = 0;
        const Partial* __restrict__ p = partials + (size_t)o * n_tiles + d.part_begin;
        for (int i = 0; i < d.part_count; ++i) {
            anti += p[i].anti;
            ups += p[i].ups;
        }
        E = 2 * (int64_t)anti - 2 * spins;
        M = 2 * (int64_t)ups - spins;
        if (d.series_E) d.series_E[idx + o] = E;
        if (d.series_M) d.series_M[idx + o] = M;
        add_sample(part, E, M);
    }
    wave_merge_moments(part);
    // the lane that took the last sample holds its E, M
    const int last = (n - 1) & 63;
    const int64_t lE = __shfl(E, last, 64), lM = __shfl(M, last, 64);
    if (lane_id() == 0) {
        Moments m = st.mom;
        merge_moments(m, part);
        st.mom = m;
        st.last_E = lE;
        st.last_M = lM;
        st.series_idx = idx + n;
    }
}

}  // namespace

hipError_t launch_finalize_resident(const LatticeDesc* descs, LatticeState* states, const int32_t* ids,
                                    int32_t n_lat, const Partial* partials, int32_t n_tiles, int32_t n_samples,
                                    hipStream_t s) {
    if (n_lat <= 0 || n_samples <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_finalize_resident, dim3(n_lat), dim3(64), 0, s, descs, states, ids, partials, n_tiles,
                       n_samples);
    return hipGetLastError();
}

hipError_t launch_samples(const Partial* partials, int32_t n_tiles, int32_t n_samples, int32_t L, int64_t* out_E,
                          int64_t* out_M, Moments* mom, hipStream_t s) {
    if (n_samples <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_samples_em, dim3(n_samples), dim3(256), 0, s, partials, n_tiles, L, out_E, out_M);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !mom) return e;
    hipLaunchKernelGGL(k_samples_moments, dim3(1), dim3(64), 0, s, out_E, out_M, n_samples, mom);
    return hipGetLastError();
}

}  // namespace ising
