// gfx950 kernels of the multi-spin-coded checkerboard Metropolis sweep and
// their launchers.  See ising_device.hpp for the word layout and the
// per-word update.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ising_device.hpp"
#include "ising_launch.hpp"
#include "ising_moments.hpp"
#include "ising_row_words.hpp"

namespace ising {

namespace {

constexpr int kTiledMaxBlock = 256;
constexpr int kResidentMaxBlock = 1024;

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// ---------------------------------------------------------------------------
// Initial state.  Hot start: a site is up iff its stream-0 draw at t = 0 is below
// 2^31 (the random initialisation of Section 5.1 with a reproducible
// generator).  A wavefront takes 64 `runs` words of a word row, one to four per lane:
// with four the block of position 20, which eight columns share in two, is drawn
// once for four words; what is left is five Philox blocks and two instructions per
// position (the draw's upper bit shifted to its field, collected inverted).  L =
// 32768: 296 us, 419 with a word per thread that draws all six blocks.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_init(uint64_t* __restrict__ W, Geometry g, uint32_t k0, uint32_t k1, int hot,
                                              int runs) {
    __shared__ uint4 last[4][64];
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = lane_id();
    const int I = (int)blockIdx.y;
    const int w0 = ((int)blockIdx.x * 4 + wv) * 64 * runs;
    if (w0 >= g.L) return;
    const uint64_t live = live_mask(I, g.L, g.N);
    uint64_t* __restrict__ row = W + (size_t)I * (size_t)g.L;
    if (!hot) {
        for (int J = w0 + lane; J < min(g.L, w0 + 64 * runs); J += 64) row[J] = live;
        return;
    }
    const uint32_t row_base = (uint32_t)I * (uint32_t)g.L;
    const RoundKeys rk = round_keys(k0, k1);
    auto block = [&](uint32_t col, uint32_t b) { return philox_lane_c1(0u, row_base + col, 0u, b, k0, k1, rk); };
    if (live & 1ull) {
        const U4 r = block((uint32_t)(w0 + 8 * (lane >> 1) + (lane & 1)), 5u);
        last[wv][lane] = make_uint4(r.x, r.y, r.z, r.w);
        wave_lds_order();
    }
#pragma unroll 1
    for (int k = 0; k < runs; ++k) {
        const int x = 64 * k + lane, J = w0 + x;
        if (J >= g.L) break;
        uint32_t lo = 0, hi = 0;  // bits set where the draw is 2^31 or above
        auto put = [&](int p, uint32_t u) {
            const int bit = 3 * (20 - p);
            if (bit < 32) lo |= (u >> (31 - bit)) & (1u << bit);
            else hi |= (u >> (63 - bit)) & (1u << (bit - 32));
        };
#pragma unroll
        for (int b = 0; b < 5; ++b) {
            const U4 r = block((uint32_t)J, (uint32_t)b);
            put(4 * b, r.x);
            put(4 * b + 1, r.y);
            put(4 * b + 2, r.z);
            put(4 * b + 3, r.w);
        }
        if (live & 1ull)
            put(20, reinterpret_cast<const uint32_t*>(last[wv])[4 * (2 * (x >> 3) + (x & 1)) + ((x >> 1) & 3)]);
        row[J] = ~(((uint64_t)hi << 32) | lo) & live;
    }
}

// ---------------------------------------------------------------------------
// Half-sweep of one lattice held in global memory: every wavefront updates
// 64 WPT words of the colour of one word row.
// ---------------------------------------------------------------------------
// What a half-sweep of one lattice adds to a run of words of word row I (n_live
// live positions).  FEW: blocks past the last live position are not drawn.
template <bool MEASURE, bool FEW>
struct LatticeRule {
    typedef std::conditional_t<FEW, AcceptSelect, AcceptPair> Accept;
    const SweepArgs& a;
    int I, n_live;
    uint64_t live;
    uint32_t anti = 0, ups = 0;
    template <class Block>
    __device__ __forceinline__ void accept(Accept& acc, const Block& block) const {
        accept_word(acc, block, FEW ? n_live : 21, a.t4, a.t8);  // the bits of dead slots are masked by `live`
    }
    __device__ __forceinline__ void accept20(Accept& acc, uint32_t u) const {
        acc.template add<20>(u, a.t4, a.t8);  // a dead slot when n_live < 21
    }
    __device__ __forceinline__ void vertical(uint64_t& up, uint64_t& dn, uint64_t patch) const {
        const Nbhd nb = {0, 0, 0, up, dn, patch};
        up = fix_up(nb, I, a.sh_star);
        dn = fix_down(nb, I, a.N, a.istar, a.sh_star);
    }
    __device__ __forceinline__ void after(uint64_t nw, uint64_t up, uint64_t dn, uint64_t lf, uint64_t rt) {
        if (MEASURE) measure_word_packed(nw, up, dn, lf, rt, live, anti, ups);
    }
};

// The words w0 + 64 k + lane (k < WPT) of colour `colour` of word row I of
// one lattice, by one wavefront; with MEASURE its sums go to *partial.
template <int WPT, bool MEASURE, bool FEW = false>
__device__ __forceinline__ void update_lattice_row(uint64_t* __restrict__ W, const SweepArgs& a, int I, int w0, int colour,
                                                   uint32_t* __restrict__ table, Partial* __restrict__ partial) {
    const size_t L = (size_t)a.L;
    const int n_live = a.pstar + (I <= a.istar ? 1 : 0);
    const RowRun r = {W + (size_t)I * L,
                      W + (size_t)(I > 0 ? I - 1 : a.N - 1) * L,
                      W + (size_t)(I < a.N - 1 ? I + 1 : 0) * L,
                      W + (size_t)(I == 0 ? a.istar : 0) * L,
                      I == 0 || I == a.N - 1 || I == a.istar,
                      a.L,
                      (I + colour) & 1,
                      (uint32_t)I * (uint32_t)a.L,
                      a.t_lo,
                      a.t_hi,
                      1u << 3,
                      a.k0,
                      a.k1,
                      n_live == 21};
    LatticeRule<MEASURE, FEW> rule{a, I, n_live, kSpinBits & (~0ull << (3 * (21 - n_live)))};
    update_row_words<WPT>(r, w0, table, rule);
    if (MEASURE) {
        const uint32_t anti = wave_sum_u32(rule.anti), ups = wave_sum_u32(rule.ups);
        if (lane_id() == 0) *partial = {anti, ups};
    }
}

template <int WPT, bool MEASURE>
__global__ void __launch_bounds__(kTiledMaxBlock)
    k_halfsweep_single(uint64_t* __restrict__ W, SweepArgs a, int colour, int band, Partial* __restrict__ partials) {
    __shared__ __align__(16) uint32_t table[(kTiledMaxBlock / 64) * row_table_words<WPT>()];
    // one word row per workgroup: the row, its wrap cases, live slots and
    // counter base are wave-uniform (scalar unit)
    const RowBlock b = row_block(band);
    if (b.row >= a.N) return;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int waves = (int)(blockDim.x >> 6);
    const int x = b.x * waves + wv;  // wavefront of the row
    const int per_row = (int)(band > 0 ? gridDim.y : gridDim.x) * waves;
    update_lattice_row<WPT, MEASURE>(W, a, b.row, 64 * WPT * x, colour, table + wv * row_table_words<WPT>(),
                                     MEASURE ? partials + (size_t)b.row * per_row + x : nullptr);
}

// E = 2 A - 2 L^2 (A antiparallel bonds out of 2 L^2), M = 2 U - L^2.
__device__ __forceinline__ void energy_magnetisation(uint64_t anti, uint64_t ups, int32_t L, int64_t& E, int64_t& M) {
    const int64_t n = (int64_t)L * (int64_t)L;
    E = 2 * (int64_t)anti - 2 * n;
    M = 2 * (int64_t)ups - n;
}

// One wavefront turns a tiled lattice's wavefront partials of a measured
// sweep into its sample: series entry, moment sums, last E and M.
__device__ __forceinline__ void finalize_lattice(const LatticeDesc& d, LatticeState& st,
                                                 const Partial* __restrict__ partials) {
    // Every lane sums every 64th partial, eight loads in flight at a time: a
    // lattice has one partial per wavefront (6272 at L = 4096), and one load
    // waited for at a time made this wavefront, and with it the launch it
    // rides in, wait out ~100 memory latencies.  Indexes past the end are
    // clamped to the last partial (so every load is unconditional and in
    // bounds) and their values dropped.
    constexpr int kInFlight = 8;
    const Partial* __restrict__ part = partials + d.part_begin;
    const int n = d.part_count;
    unsigned long long anti = 0, ups = 0;
    for (int i0 = (int)lane_id(); i0 < n; i0 += 64 * kInFlight) {
        Partial v[kInFlight];
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) v[k] = part[min(i0 + 64 * k, n - 1)];
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) {
            const bool in = i0 + 64 * k < n;
            anti += in ? v[k].anti : 0u;
            ups += in ? v[k].ups : 0u;
        }
    }
    anti = wave_sum_u64(anti);
    ups = wave_sum_u64(ups);
    if (lane_id() == 0) {
        int64_t E, M;
        energy_magnetisation(anti, ups, d.L, E, M);
        const int64_t idx = st.series_idx;
        st.last_E = E;
        st.last_M = M;
        add_sample(st.mom, E, M);
        if (d.series_E) d.series_E[idx] = E;
        if (d.series_M) d.series_M[idx] = M;
        st.series_idx = idx + 1;
    }
}

// ---------------------------------------------------------------------------
// Half-sweep over a table of wavefronts covering many lattices.  Every
// wavefront belongs to one lattice, so the lattice's parameters (key, sweep
// index, thresholds) are wave-uniform and live in scalar registers.  With
// fin_partials set, the first wavefront of every lattice first finalizes the
// lattice's measured sweep fin_off from the partials that an earlier launch
// left (the launch boundary orders them), which saves a launch per sample.  FEW: a
// kernel for tables that are mostly of lattices with at most 16 live positions a
// word (few_live), which are over before the chip is full: their rows draw only the
// blocks that they need, and acceptance is by selects, which wait less (us per
// half-sweep of 8 lattices, without / with: a word per thread and 64 threads L = 4
// 3.33 / 2.66, 16 3.31 / 2.75, 64 3.39 / 3.12, 256 threads 4.05 / 2.78, 4.07 / 3.18, 3.21 /
// 2.99; for all lattices it would take L = 9998 from 23.7 to 24.2).
// ---------------------------------------------------------------------------
template <int WPT, bool MEASURE, bool FEW>
__global__ void __launch_bounds__(kTiledMaxBlock)
    k_halfsweep_multi(const LatticeDesc* __restrict__ descs, LatticeState* __restrict__ states,
                      const WaveItem* __restrict__ waves, uint32_t n_waves, uint32_t group, int colour,
                      uint32_t sweep_off, Partial* __restrict__ partials, const Partial* __restrict__ fin_partials,
                      uint32_t fin_off) {
    __shared__ __align__(16) uint32_t table[(kTiledMaxBlock / 64) * row_table_words<WPT>()];
    // groups of consecutive workgroups of the table to one XCD (see launch)
    uint32_t b = blockIdx.x;
    if (b < gridDim.x / (8 * group) * (8 * group)) {
        const uint32_t seq = b >> 3, g = seq / group;
        b = (8 * g + (b & 7u)) * group + (seq - g * group);
    }
    const uint32_t wave = __builtin_amdgcn_readfirstlane((b * blockDim.x + threadIdx.x) >> 6);
    if (wave >= n_waves) return;
    const WaveItem item = waves[wave];
    const LatticeDesc& d = descs[item.lattice];
    const uint64_t t = states[item.lattice].t + sweep_off;  // read before the finalize's stores: a scalar load
    if (fin_partials && wave == (uint32_t)d.part_begin && fin_off < (uint32_t)d.sweep_limit)
        finalize_lattice(d, states[item.lattice], fin_partials);
    if (sweep_off >= (uint32_t)d.sweep_limit) {  // this lattice has finished its sweeps of the chunk
        if (MEASURE && lane_id() == 0) partials[wave] = {0u, 0u};
        return;
    }
    const SweepArgs a = {d.L, d.N, d.istar, d.sh_star, d.pstar, (uint32_t)t, (uint32_t)(t >> 32), d.k0, d.k1, d.t4, d.t8};
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    update_lattice_row<WPT, MEASURE, FEW>(d.W, a, item.row, item.w0, colour, table + wv * row_table_words<WPT>(),
                                     MEASURE ? partials + wave : nullptr);
}

__device__ __forceinline__ void block_sum2(uint64_t& x, uint64_t& y, uint64_t* red /* 2 * 16 */) {
    x = wave_sum_u64(x);
    y = wave_sum_u64(y);
    const int wv = threadIdx.x >> 6;
    if (lane_id() == 0) {
        red[wv] = x;
        red[16 + wv] = y;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int nw = (blockDim.x + 63) >> 6;
        uint64_t sx = 0, sy = 0;
        for (int i = 0; i < nw; ++i) {
            sx += red[i];
            sy += red[16 + i];
        }
        x = sx;
        y = sy;
    }
    __syncthreads();
}

// Grid reduction of one lattice's wavefront partials: every workgroup sums a
// slice into block_sums[blockIdx.x]; the last workgroup to finish (ticket
// counter at device scope) adds the slices, turns them into E, M and resets
// the counter for the next call.
constexpr int kFinalizeBlocks = 256;

__global__ void __launch_bounds__(256) k_finalize_single(const Partial* __restrict__ partials, int64_t n_partials,
                                                         int32_t L, int64_t* series_E, int64_t* series_M,
                                                         int64_t idx, int64_t* out_EM, Moments* mom,
                                                         unsigned long long* __restrict__ block_sums,
                                                         unsigned int* __restrict__ ticket) {
    __shared__ uint64_t red[32];
    __shared__ bool last;
    uint64_t anti = 0, ups = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_partials;
         i += (int64_t)gridDim.x * blockDim.x) {
        anti += partials[i].anti;
        ups += partials[i].ups;
    }
    block_sum2(anti, ups, red);
    if (threadIdx.x == 0) {
        block_sums[2 * blockIdx.x] = anti;
        block_sums[2 * blockIdx.x + 1] = ups;
        __threadfence();
        last = atomicAdd(ticket, 1u) == gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    anti = 0;
    ups = 0;
    for (int i = threadIdx.x; i < (int)gridDim.x; i += blockDim.x) {
        anti += __atomic_load_n(&block_sums[2 * i], __ATOMIC_RELAXED);
        ups += __atomic_load_n(&block_sums[2 * i + 1], __ATOMIC_RELAXED);
    }
    block_sum2(anti, ups, red);
    if (threadIdx.x == 0) {
        int64_t E, M;
        energy_magnetisation(anti, ups, L, E, M);
        if (series_E) series_E[idx] = E;
        if (series_M) series_M[idx] = M;
        if (out_EM) {
            out_EM[0] = E;
            out_EM[1] = M;
        }
        if (mom) add_sample(*mom, E, M);
        *ticket = 0u;
    }
}

// End of a chunk of sweeps, one wavefront per lattice: finalize the tiled
// lattices' measured sweep fin_off (with fin_partials set) and advance every
// lattice's sweep counter by the sweeps it ran.
__global__ void __launch_bounds__(64) k_chunk_end(const LatticeDesc* __restrict__ descs,
                                                  LatticeState* __restrict__ states,
                                                  const Partial* __restrict__ fin_partials, uint32_t fin_off,
                                                  uint32_t k) {
    const LatticeDesc& d = descs[blockIdx.x];
    LatticeState& st = states[blockIdx.x];
    if (fin_partials && !d.resident && fin_off < (uint32_t)d.sweep_limit) finalize_lattice(d, st, fin_partials);
    if (threadIdx.x == 0) st.t += min(k, (uint32_t)d.sweep_limit);
}

__global__ void k_reset_sums(LatticeState* __restrict__ states, int32_t n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) states[i].mom = Moments{};
}

__global__ void k_begin_call(LatticeState* __restrict__ states, int32_t n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) states[i].series_idx = 0;
}

// ---------------------------------------------------------------------------
// Resident lattices: one workgroup owns a lattice for K sweeps; colours are
// separated by workgroup barriers.  With IN_LDS the words live in LDS for
// the whole launch (read once, written once).
// ---------------------------------------------------------------------------
template <int WPT, bool IN_LDS>
__global__ void __launch_bounds__(kResidentMaxBlock)
    k_resident(const LatticeDesc* __restrict__ descs, LatticeState* __restrict__ states,
               const int32_t* __restrict__ ids, int32_t K, int32_t every) {
    extern __shared__ uint64_t lds_words[];
    __shared__ uint64_t red[32];
    const int32_t lat = ids[blockIdx.x];
    const LatticeDesc& d = descs[lat];
    LatticeState& state = states[lat];
    const int L = d.L, N = d.N;
    uint64_t* __restrict__ G = d.W;
    const uint32_t n_words = (uint32_t)N * (uint32_t)L;
    if (IN_LDS) {
        for (uint32_t i = threadIdx.x; i < n_words; i += blockDim.x) lds_words[i] = G[i];
        __syncthreads();
    }
    uint64_t* __restrict__ W = IN_LDS ? lds_words : G;
    // word offsets: 32-bit inside LDS, 64-bit in global memory (N L may
    // exceed 2^31 words there)
    auto off = [&](int i, int j) {
        if constexpr (IN_LDS) return (uint32_t)i * (uint32_t)L + (uint32_t)j;
        else return (size_t)i * (size_t)L + (size_t)j;
    };
    auto ld = [&](int i, int j) { return W[off(i, j)]; };
    auto st = [&](int i, int j, uint64_t v) { W[off(i, j)] = v; };
    const int segs = (L + 2 * WPT - 1) / (2 * WPT);
    const uint32_t units = (uint32_t)N * (uint32_t)segs;
    const uint64_t t0 = state.t;
    const int32_t n_sweeps = min(K, d.sweep_limit);
    // sample accumulators stay in thread 0's registers for the whole launch
    int64_t series_idx = 0, last_E = 0, last_M = 0;
    Moments mom = {};
    int64_t* const series_E = d.series_E;
    int64_t* const series_M = d.series_M;
    if (threadIdx.x == 0) {
        series_idx = state.series_idx;
        mom = state.mom;
        last_E = state.last_E;
        last_M = state.last_M;
    }
    for (int s = 0; s < n_sweeps; ++s) {
        const uint64_t t = t0 + (uint64_t)s;
        const SweepArgs a = {L, N, d.istar, d.sh_star, d.pstar, (uint32_t)t, (uint32_t)(t >> 32), d.k0, d.k1, d.t4, d.t8};
        const bool meas = every > 0 && ((s + 1) % every) == 0;
        for (int colour = 0; colour < 2; ++colour) {
            uint32_t anti = 0, ups = 0;
            for (uint32_t u = threadIdx.x; u < units; u += blockDim.x) {
                const int I = (int)(u / (uint32_t)segs);
                const int seg = (int)(u - (uint32_t)I * (uint32_t)segs);
                const int J0 = seg * 2 * WPT + ((I + colour) & 1);
                if (meas && colour == 1) update_segment<WPT, true>(ld, st, I, J0, a, anti, ups);
                else update_segment<WPT, false>(ld, st, I, J0, a, anti, ups);
            }
            __syncthreads();
            if (meas && colour == 1) {
                uint64_t A = anti, U = ups;
                block_sum2(A, U, red);
                if (threadIdx.x == 0) {
                    int64_t E, M;
                    energy_magnetisation(A, U, L, E, M);
                    last_E = E;
                    last_M = M;
                    add_sample(mom, E, M);
                    if (series_E) series_E[series_idx] = E;
                    if (series_M) series_M[series_idx] = M;
                    series_idx += 1;
                }
            }
        }
    }
    if (threadIdx.x == 0) {
        state.series_idx = series_idx;
        state.mom = mom;
        state.last_E = last_E;
        state.last_M = last_M;
    }
    if (IN_LDS) {
        for (uint32_t i = threadIdx.x; i < n_words; i += blockDim.x) G[i] = lds_words[i];
    }
}

// Antiparallel right and down bonds (Section 5.3) and up spins of the words
// idx, idx + 256, ... below end of one lattice, a thread's share of a
// workgroup's consecutive words.
__device__ __forceinline__ void observe_words(const uint64_t* __restrict__ W, int L, int N, int istar, int sh_star,
                                              uint32_t idx, uint32_t end, uint32_t& anti, uint32_t& ups) {
    auto ld = [&](int i, int j) { return W[(size_t)i * L + j]; };
    int I = (int)(idx / (uint32_t)L);
    int J = (int)(idx - (uint32_t)I * (uint32_t)L);
    for (; idx < end; idx += 256) {
        const uint64_t live = live_mask(I, L, N);
        const uint64_t w = ld(I, J);
        const uint64_t rt = ld(I, J == L - 1 ? 0 : J + 1);
        const uint64_t dn = down_word(ld, I, J, N, istar, sh_star);
        anti += __popcll((w ^ rt) & live) + __popcll((w ^ dn) & live);
        ups += __popcll(w & live);
        J += 256;
        while (J >= L) {
            J -= L;
            I += 1;
        }
    }
}

// E and M of a lattice from its sums, into its state and out (may be null).
__device__ __forceinline__ void observed(uint64_t anti, uint64_t ups, int32_t L, LatticeState& st,
                                         int64_t* __restrict__ out) {
    int64_t E, M;
    energy_magnetisation(anti, ups, L, E, M);
    st.last_E = E;
    st.last_M = M;
    if (out) {
        out[0] = E;
        out[1] = M;
        out[2] = st.abandoned;
    }
}

// Words of a lattice per workgroup of k_observe_multi; and those of lattices that one
// workgroup takes whole and finishes, without the second launch (us per read of E
// and M with it / without: 8 lattices of L = 64 31.8 / 30.3, 500 of L = 256 42.5 / 39.5,
// 8 of L = 340, 6120 words, 33.4 / 36).
constexpr uint32_t kObserveWords = 2048;
constexpr int64_t kObserveWhole = 4096;

// Observables of every lattice of a table: workgroup part of `parts` of a
// lattice takes every parts-th run of kObserveWords words and adds its sums to the
// lattice's in device memory (a workgroup without words, of a smaller lattice of
// the table, does not take part); k_observed, launched behind it, forms E and M, or
// this kernel where a workgroup takes a whole lattice (parts = 1).
// Bound by the words' bytes: 256 lattices of L = 256 ... 2048 (137 MB) 74 us,
// against 379 with one workgroup per lattice; one of L = 4096 12 us against 790.
// A count of arrived workgroups in this kernel instead of the second launch took
// 287 us, for its acquire and release by each of them.
__global__ void __launch_bounds__(256) k_observe_multi(const LatticeDesc* __restrict__ descs,
                                                       LatticeState* __restrict__ states,
                                                       const int32_t* __restrict__ ids, int32_t parts,
                                                       int64_t* __restrict__ out) {
    __shared__ uint64_t red[32];
    const uint32_t k = blockIdx.x / (uint32_t)parts, part = blockIdx.x - k * (uint32_t)parts;
    const int32_t lat = ids ? ids[k] : (int32_t)k;
    const LatticeDesc& d = descs[lat];
    const int L = d.L, N = d.N;
    const uint32_t n_words = (uint32_t)N * (uint32_t)L;
    if ((uint64_t)part * kObserveWords >= n_words) return;
    uint64_t anti = 0, ups = 0;
    for (uint64_t w0 = (uint64_t)part * kObserveWords; w0 < n_words; w0 += (uint64_t)parts * kObserveWords) {
        uint32_t a = 0, u = 0;
        observe_words(d.W, L, N, d.istar, d.sh_star, (uint32_t)w0 + threadIdx.x,
                      (uint32_t)min((uint64_t)n_words, w0 + kObserveWords), a, u);
        anti += a;
        ups += u;
    }
    block_sum2(anti, ups, red);
    if (threadIdx.x == 0) {
        if (parts == 1) {
            observed(anti, ups, L, states[lat], out ? out + kObservedWords * k : nullptr);
        } else {
            atomicAdd(&states[lat].obs_anti, (unsigned long long)anti);
            atomicAdd(&states[lat].obs_ups, (unsigned long long)ups);
        }
    }
}

// E and M of the k-th listed lattice from its sums, which are left zero.
__global__ void __launch_bounds__(256) k_observed(const LatticeDesc* __restrict__ descs,
                                                  LatticeState* __restrict__ states, const int32_t* __restrict__ ids,
                                                  int32_t n_lat, int64_t* __restrict__ out) {
    const int32_t k = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (k >= n_lat) return;
    const int32_t lat = ids ? ids[k] : k;
    LatticeState& st = states[lat];
    observed(st.obs_anti, st.obs_ups, descs[lat].L, st, out ? out + kObservedWords * k : nullptr);
    st.obs_anti = 0;
    st.obs_ups = 0;
}

// The same of one lattice, `run` words (a multiple of 256) per workgroup, as
// wavefront partial sums.
__global__ void __launch_bounds__(256) k_observe_single(const uint64_t* __restrict__ W, Geometry g, uint32_t run,
                                                        Partial* __restrict__ partials) {
    const uint32_t n_words = (uint32_t)g.N * (uint32_t)g.L;
    const uint32_t w0 = blockIdx.x * run;
    uint32_t anti = 0, ups = 0;
    observe_words(W, g.L, g.N, g.istar, g.sh_star, w0 + threadIdx.x, min(n_words, w0 + run), anti, ups);
    anti = wave_sum_u32(anti);
    ups = wave_sum_u32(ups);
    if (lane_id() == 0) partials[blockIdx.x * 4 + (threadIdx.x >> 6)] = {anti, ups};
}

__global__ void __launch_bounds__(256) k_unpack(const uint64_t* __restrict__ W, Geometry g, int32_t r0, int32_t c0,
                                                int32_t nrows, int32_t ncols, uint8_t* __restrict__ out) {
    const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (uint64_t)nrows * (uint64_t)ncols) return;
    const int i = (int)(idx / (uint64_t)ncols);
    const int j = (int)(idx - (uint64_t)i * (uint64_t)ncols);
    const int r = (int)(((int64_t)r0 + i) % g.L);
    const int c = (int)(((int64_t)c0 + j) % g.L);
    const int I = r % g.N, p = r / g.N;
    out[idx] = (uint8_t)((W[(size_t)I * g.L + c] >> (3 * (20 - p))) & 1ull);
}

// Write nrows lattice rows r0 .. r0 + nrows - 1 (row-major bytes, nonzero =
// up) into their words: row r is position r div N of word row r mod N.  With
// nrows <= N every word is touched by one row at most, so the bit updates of
// one launch never share a word.
__global__ void __launch_bounds__(256) k_pack_rows(const uint8_t* __restrict__ in, Geometry g, int32_t r0,
                                                   int32_t nrows, uint64_t* __restrict__ W) {
    const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (uint64_t)nrows * (uint64_t)g.L) return;
    const int i = (int)(idx / (uint64_t)g.L);
    const int c = (int)(idx - (uint64_t)i * (uint64_t)g.L);
    const int r = r0 + i;
    const int I = r % g.N, p = r / g.N;
    const uint64_t bit = 1ull << (3 * (20 - p));
    uint64_t* w = W + ((size_t)I * g.L + c);
    *w = in[idx] ? (*w | bit) : (*w & ~bit);
}

// The words of a whole lattice from its L x L bytes, a thread per word: word
// (I, J) holds the rows I + p N of column J.
__global__ void __launch_bounds__(256) k_pack_words(const uint8_t* __restrict__ in, Geometry g,
                                                    uint64_t* __restrict__ W) {
    const uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (uint32_t)g.N * (uint32_t)g.L) return;
    const int I = (int)(idx / (uint32_t)g.L);
    const int n_live = (g.L - 1 - I) / g.N + 1;
    const size_t step = (size_t)g.N * (size_t)g.L;  // bytes from one position's row to the next one's
    uint64_t w = 0;
#pragma unroll
    for (int p = 0; p < 21; ++p)
        if (p < n_live) w |= (in[idx + p * step] ? 1ull : 0ull) << (3 * (20 - p));
    W[idx] = w;
}

__global__ void __launch_bounds__(256) k_zero_words(uint64_t* __restrict__ p, uint64_t n) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

inline unsigned grid_for(uint64_t n, int block) { return (unsigned)((n + block - 1) / block); }

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

hipError_t launch_zero_words(uint64_t* p, uint64_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_words, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_init(uint64_t* W, const Geometry& g, uint64_t seed, int hot, hipStream_t s) {
    // four words per lane only where there are wavefronts enough without (us per
    // launch with one / four: L = 2500 4.7 / 5.7, 4096 8.7 / 8.8, 5120 12.2 / 11.1,
    // 9998 42 / 36, 32768 362 / 296)
    const int runs = (int64_t)g.N * g.L >= (1 << 20) ? 4 : 1;
    hipLaunchKernelGGL(k_init, dim3(grid_for((uint64_t)g.L, 4 * 64 * runs), g.N), dim3(256), 0, s, W, g,
                       (uint32_t)seed, (uint32_t)(seed >> 32), hot, runs);
    return hipGetLastError();
}

int64_t halfsweep_single_waves(const Geometry& g, int wpt, int block) {
    return (int64_t)grid_for((uint64_t)segments_per_row(g.L, wpt), block) * g.N * (block / 64);
}

hipError_t launch_halfsweep_single(int wpt, int block, uint64_t* W, const SweepArgs& a, int colour,
                                   Partial* partials, int64_t* n_waves, hipStream_t s) {
    const Geometry g = {a.L, a.N, a.istar, a.sh_star};
    int band = 0;
    const dim3 grid = row_grid(a.N, grid_for((uint64_t)segments_per_row(a.L, wpt), block), (size_t)a.L * 8, &band);
    const dim3 blk(block);
    if (n_waves) *n_waves = halfsweep_single_waves(g, wpt, block);
    const bool m = partials != nullptr;
#define ISING_LAUNCH_HS(WPT_)                                                                                    \
    if (m) hipLaunchKernelGGL((k_halfsweep_single<WPT_, true>), grid, blk, 0, s, W, a, colour, band, partials);        \
    else hipLaunchKernelGGL((k_halfsweep_single<WPT_, false>), grid, blk, 0, s, W, a, colour, band, partials);
    switch (wpt) {
        case 1: ISING_LAUNCH_HS(1) break;
        case 2: ISING_LAUNCH_HS(2) break;
        case 4: ISING_LAUNCH_HS(4) break;
        default: return hipErrorInvalidValue;
    }
#undef ISING_LAUNCH_HS
    return hipGetLastError();
}

size_t finalize_scratch_bytes() { return 2 * kFinalizeBlocks * sizeof(unsigned long long) + 256; }

hipError_t launch_finalize_single(const Partial* partials, int64_t n_partials, int32_t L, int64_t* series_E,
                                  int64_t* series_M, int64_t idx, int64_t* out_EM, Moments* mom, void* scratch,
                                  hipStream_t s) {
    const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>(kFinalizeBlocks, (n_partials + 2047) / 2048));
    unsigned long long* sums = reinterpret_cast<unsigned long long*>(scratch);
    unsigned int* ticket = reinterpret_cast<unsigned int*>(reinterpret_cast<char*>(scratch) +
                                                           2 * kFinalizeBlocks * sizeof(unsigned long long));
    hipLaunchKernelGGL(k_finalize_single, dim3(blocks), dim3(256), 0, s, partials, n_partials, L, series_E, series_M,
                       idx, out_EM, mom, sums, ticket);
    return hipGetLastError();
}

namespace {

// Words per workgroup of k_observe_single: with 2048 L = 32768 takes 119 us (156
// with 256, and eight times the partial sums to add up), below 2^20 words that
// would leave compute units without a workgroup (L = 2016: 95).
uint32_t observe_run(const Geometry& g) { return (uint64_t)g.N * g.L >= (1u << 20) ? 2048 : 256; }

}  // namespace

int64_t observe_single_waves(const Geometry& g) { return (int64_t)grid_for((uint64_t)g.N * g.L, observe_run(g)) * 4; }

hipError_t launch_observe_single(const uint64_t* W, const Geometry& g, Partial* partials, int64_t* n_waves,
                                 hipStream_t s) {
    const uint64_t n = (uint64_t)g.N * g.L;
    const uint32_t run = observe_run(g);
    if (n_waves) *n_waves = observe_single_waves(g);
    hipLaunchKernelGGL(k_observe_single, dim3(grid_for(n, run)), dim3(256), 0, s, W, g, run, partials);
    return hipGetLastError();
}

hipError_t launch_unpack(const uint64_t* W, const Geometry& g, int32_t r0, int32_t c0, int32_t nrows,
                         int32_t ncols, uint8_t* out, hipStream_t s) {
    const uint64_t n = (uint64_t)nrows * (uint64_t)ncols;
    hipLaunchKernelGGL(k_unpack, dim3(grid_for(n, 256)), dim3(256), 0, s, W, g, r0, c0, nrows, ncols, out);
    return hipGetLastError();
}

hipError_t launch_pack_rows(const uint8_t* in, const Geometry& g, int32_t r0, int32_t nrows, uint64_t* W,
                            hipStream_t s) {
    if (nrows < 1 || nrows > g.N || r0 < 0 || r0 + nrows > g.L) return hipErrorInvalidValue;
    const uint64_t n = (uint64_t)nrows * (uint64_t)g.L;
    hipLaunchKernelGGL(k_pack_rows, dim3(grid_for(n, 256)), dim3(256), 0, s, in, g, r0, nrows, W);
    return hipGetLastError();
}

hipError_t launch_pack_words(const uint8_t* in, const Geometry& g, uint64_t* W, hipStream_t s) {
    hipLaunchKernelGGL(k_pack_words, dim3(grid_for((uint64_t)g.N * g.L, 256)), dim3(256), 0, s, in, g, W);
    return hipGetLastError();
}

hipError_t launch_halfsweep_multi(int wpt, int block, const LatticeDesc* descs, LatticeState* states,
                                  const WaveItem* waves, int64_t n_waves, bool runs, bool few, int colour,
                                  uint32_t sweep_off, Partial* partials, const Partial* fin_partials,
                                  uint32_t fin_off, hipStream_t s) {
    if (n_waves <= 0) return hipSuccess;
    const dim3 grid(grid_for((uint64_t)n_waves * 64, block)), blk(block);
    const bool m = partials != nullptr;
    const uint32_t nw = (uint32_t)n_waves;
    // Consecutive workgroups are dealt to the 8 XCDs in turn; runs of 256
    // wavefronts of the table (a few rows at least) go to one XCD, so that the rows
    // above and below are mostly in its L2, and the runs to the XCDs in turn, at
    // least eight each, so that lattices that have finished their sweeps leave
    // none of them idle.  us per half-sweep without and with, 256 lattices of L = 256
    // ... 2048: 101 / 68 with two words per thread and 256 threads, 92 / 67 with four
    // words; 64 of 64 ... 512: 5.8 / 4.9 with a word and 64 threads.  Not where most
    // rows are a multiple of 8 workgroups (runs = false), which keeps the rows above
    // and below on the XCD anyway: one L = 4096 with a word and 64 threads 8.1, in
    // runs 9.1.
    const uint32_t group = runs ? std::max(1u, std::min(grid.x / 64, 16384u / (unsigned)block)) : grid.x;
#define ISING_LAUNCH_HM_(WPT_, M_, F_)                                                                                 \
    hipLaunchKernelGGL((k_halfsweep_multi<WPT_, M_, F_>), grid, blk, 0, s, descs, states, waves, nw, group, colour, \
                       sweep_off, partials, fin_partials, fin_off)
#define ISING_LAUNCH_HM(WPT_)                       \
    if (m && few) ISING_LAUNCH_HM_(WPT_, true, true); \
    else if (m) ISING_LAUNCH_HM_(WPT_, true, false);  \
    else if (few) ISING_LAUNCH_HM_(WPT_, false, true); \
    else ISING_LAUNCH_HM_(WPT_, false, false);
    switch (wpt) {
        case 1: ISING_LAUNCH_HM(1) break;
        case 2: ISING_LAUNCH_HM(2) break;
        case 4: ISING_LAUNCH_HM(4) break;
        default: return hipErrorInvalidValue;
    }
#undef ISING_LAUNCH_HM
#undef ISING_LAUNCH_HM_
    return hipGetLastError();
}

hipError_t launch_chunk_end(const LatticeDesc* descs, LatticeState* states, int32_t n_lat,
                            const Partial* fin_partials, uint32_t fin_off, uint32_t k, hipStream_t s) {
    if (n_lat <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_chunk_end, dim3(n_lat), dim3(64), 0, s, descs, states, fin_partials, fin_off, k);
    return hipGetLastError();
}

hipError_t launch_reset_sums(LatticeState* states, int32_t n_lat, hipStream_t s) {
    if (n_lat <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_reset_sums, dim3(grid_for(n_lat, 256)), dim3(256), 0, s, states, n_lat);
    return hipGetLastError();
}

hipError_t launch_begin_call(LatticeState* states, int32_t n_lat, hipStream_t s) {
    if (n_lat <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_begin_call, dim3(grid_for(n_lat, 256)), dim3(256), 0, s, states, n_lat);
    return hipGetLastError();
}

hipError_t launch_observe_multi(const LatticeDesc* descs, LatticeState* states, const int32_t* ids, int32_t n_lat,
                                int64_t max_words, int64_t* out, hipStream_t s) {
    if (n_lat <= 0) return hipSuccess;
    // workgroups for every run of the largest lattice, up to 1024 per lattice and
    // 16384 in all (beyond, a workgroup takes several runs)
    const int64_t runs = max_words <= kObserveWhole ? 1 : (max_words + kObserveWords - 1) / kObserveWords;
    const int64_t parts = std::max<int64_t>(1, std::min({runs, (int64_t)1024, (int64_t)16384 / n_lat}));
    hipLaunchKernelGGL(k_observe_multi, dim3((unsigned)(parts * n_lat)), dim3(256), 0, s, descs, states, ids,
                       (int32_t)parts, out);
    if (parts > 1)
        hipLaunchKernelGGL(k_observed, dim3(grid_for(n_lat, 256)), dim3(256), 0, s, descs, states, ids, n_lat, out);
    return hipGetLastError();
}

size_t resident_lds_limit(int device) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, device) != hipSuccess) return 0;
    const size_t static_bytes = 32 * sizeof(uint64_t) + 64;
    return v > (int)static_bytes ? (size_t)v - static_bytes : 0;
}

hipError_t set_resident_lds(int wpt, size_t lds_bytes) {
    const void* f = wpt == 1 ? reinterpret_cast<const void*>(&k_resident<1, true>)
                  : wpt == 2 ? reinterpret_cast<const void*>(&k_resident<2, true>)
                             : reinterpret_cast<const void*>(&k_resident<4, true>);
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    int device = 0;
    if (e == hipSuccess) e = hipGetDevice(&device);
    if (e == hipSuccess) e = allow_small_lds(device);
    return e;
}

hipError_t launch_resident(int wpt, int block, const LatticeDesc* descs, LatticeState* states, const int32_t* ids,
                           int32_t n_ids, int32_t K, int32_t every, size_t lds_bytes, hipStream_t s) {
    if (n_ids <= 0 || K <= 0) return hipSuccess;
    if (block < 64 || block > kResidentMaxBlock || block % 64) return hipErrorInvalidValue;
    if (lds_bytes > 0) {
        // lattices small enough to keep the codes of two or more sweeps
        // beside them in LDS draw those ahead (k_small)
        int device = 0;
        hipError_t e = hipGetDevice(&device);
        if (e != hipSuccess) return e;
        const size_t limit = small_lds_limit(device);
        const int32_t batch = lds_bytes < limit ? (int32_t)std::min<size_t>(64, (limit - lds_bytes) / lds_bytes) : 0;
        if (batch >= 2)
            return launch_small(block, descs, states, ids, n_ids, K, every, batch, lds_bytes * (1 + batch), s);
    }
    const dim3 grid(n_ids), blk(block);
#define ISING_LAUNCH_RES(WPT_)                                                                                  \
    if (lds_bytes > 0) {                                                                                        \
        hipLaunchKernelGGL((k_resident<WPT_, true>), grid, blk, lds_bytes, s, descs, states, ids, K, every);    \
    } else {                                                                                                    \
        hipLaunchKernelGGL((k_resident<WPT_, false>), grid, blk, 0, s, descs, states, ids, K, every);           \
    }
    switch (wpt) {
        case 1: ISING_LAUNCH_RES(1) break;
        case 2: ISING_LAUNCH_RES(2) break;
        case 4: ISING_LAUNCH_RES(4) break;
        default: return hipErrorInvalidValue;
    }
#undef ISING_LAUNCH_RES
    return hipGetLastError();
}

}  // namespace ising
