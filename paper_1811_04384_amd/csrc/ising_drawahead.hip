// Small lattices whose acceptance codes are drawn by the whole chip and
// applied by one small workgroup per lattice.
//
// The acceptance codes of a site (Table 1's classes with the Metropolis rule
// of Section 2 applied to its uniform) do not depend on the spins, only on
// (seed, sweep, site) and the temperature.  A handful of small lattices (a
// temperature scan of a few L = 64 lattices, the paper's N = 4 lattice)
// leaves all but a few compute units idle when each lattice's workgroup
// draws its own codes; here a draw pass spreads the codes of many sweeps of
// every such lattice over the whole chip into a global buffer, and an apply
// pass then runs the sweeps: one workgroup of one to sixteen wavefronts per
// lattice, the lattice in LDS, each thread's codes loaded into registers
// several sweeps ahead of their use.  A batch runs the two passes as two
// launches; a single lattice's launches draw the next chunk of sweeps beside
// the workgroup that applies the last one.  What is left per half-sweep is one
// word update per thread and word -- a chain of a few hundred cycles -- and
// a workgroup barrier; with one wavefront not even that, as a wavefront's
// LDS operations complete in issue order, so one half-sweep's stores are
// seen by the next half-sweep's loads.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ising_device.hpp"
#include "ising_launch.hpp"
#include "ising_lds_word.hpp"
#include "ising_moments.hpp"

namespace ising {

namespace {

constexpr int kDrawBlock = 256;
constexpr int kApplyMaxBlock = 1024;

}  // namespace

// Draw pass: item f of lattice entry e (blockIdx.x div blocks_per_lat) is
// sweep j = f div n_draw of the pass (absolute sweep t = state.t +
// sweep_off + j) and (colour c, word row I, 8-column group); it writes the
// codes of the group's four words of that colour, drawn exactly as every
// other path draws them (Philox blocks 0..4 of counter (t, I L + J), the
// position-20 block 5 shared by the group).  Codes of sweep j, colour c are
// stored by word slot f = I (L/2) + h for column J = 2h + ((I + c) & 1), so
// the four words of an item are adjacent.  Sweeps past the lattice's sweep
// limit are not drawn.
__global__ void __launch_bounds__(kDrawBlock) k_draw_codes(const LatticeDesc* __restrict__ descs,
                                                           const LatticeState* __restrict__ states,
                                                           const DrawLat* __restrict__ lats, uint64_t* __restrict__ codes,
                                                           int32_t blocks_per_lat, int32_t sweep_off, int32_t S) {
    const int e = (int)(blockIdx.x / (unsigned)blocks_per_lat);
    const DrawLat dl = lats[e];
    const int f = (int)(blockIdx.x - (unsigned)e * (unsigned)blocks_per_lat) * kDrawBlock + (int)threadIdx.x;
    if (f >= S * dl.n_draw) return;
    const LatticeDesc& d = descs[dl.lat];
    const int L = d.L, N = d.N, istar = d.istar;
    const int j = f / dl.n_draw, r = f - j * dl.n_draw;
    if (sweep_off + j >= d.sweep_limit) return;
    const int groups = (L + 7) >> 3;
    const int c = r >= N * groups ? 1 : 0;
    const int rr = r - c * N * groups;
    const int I = rr / groups, grp = rr - I * groups;
    const int n_live = (L - 1) / N + (I <= istar ? 1 : 0);
    const uint64_t t = states[dl.lat].t + (uint64_t)(sweep_off + j);
    const uint32_t t_lo = (uint32_t)t, t_hi = (uint32_t)(t >> 32);
    const RoundKeys rk = round_keys(d.k0, d.k1);
    const int par = (I + c) & 1;
    const int half = L >> 1;
    uint4 u5 = make_uint4(0u, 0u, 0u, 0u);
    if (n_live == 21) {
        const U4 r5 = philox_lane_c1(t_lo, (uint32_t)I * (uint32_t)L + (uint32_t)(8 * grp + par), t_hi, 5u | (1u << 3),
                                     d.k0, d.k1, rk);
        u5 = make_uint4(r5.x, r5.y, r5.z, r5.w);
    }
    uint64_t* __restrict__ out = codes + dl.base + (size_t)j * (size_t)(N * L) + (size_t)(c * N * half + I * half + 4 * grp);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int J = 8 * grp + par + 2 * m;
        if (J >= L) break;
        AcceptWord acc;
        accept_word(
            acc,
            [&](int g) {
                return philox_lane_c1(t_lo, (uint32_t)I * (uint32_t)L + (uint32_t)J, t_hi, (uint32_t)g | (1u << 3), d.k0,
                                      d.k1, rk);
            },
            n_live, d.t4, d.t8);
        acc.add<20>(pick4(u5, (uint32_t)m), d.t4, d.t8);  // a dead slot when n_live < 21
        out[m] = acc.word();
    }
}

namespace {

// Issue the loads of sweep j's codes of this thread's words (slots past the
// last word load the last word's code, which is not used), without branches
// so that the compiler can count them and wait only for the oldest.
template <int WMAX>
__device__ __forceinline__ void load_codes(uint64_t (&cr)[2][WMAX], const uint64_t* __restrict__ cg, size_t NL,
                                           int words, int tid, int stride, int j) {
    const uint64_t* __restrict__ p = cg + (size_t)j * NL;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int k = 0; k < WMAX; ++k) cr[c][k] = __builtin_nontemporal_load(p + c * words + min(tid + stride * k, words - 1));
}

// A word slot of a thread, the same columns 2h and 2h + 1 of word row I in
// both colours: own[c] is the LDS address of the word of colour c (and the
// near neighbour of colour 1 - c), far[c] that of its other neighbour in the
// row, up / dn / pt those of the rows above and below and of the patch word.
// The wrap of rows 0, N - 1 and I* is formed by every lane with its own
// constants, without selects: the word above is shifted down one field in row
// 0 (su = 3), the one below up one field in row N - 1 (sd = 3; its bit 63 is
// masked by live), bit 60 of the word above row 0 comes from the patch word
// (mu), and bit sh_star of the word below row I* too (md).
struct Slot {
    uint32_t own[2], far[2], up[2], dn[2], pt[2];
    uint32_t su, sd, mu;
    uint64_t md, live;
};

__device__ __forceinline__ Slot make_slot(const lds_u64* T, int I, int h, int L, int N, int istar, int sh_star,
                                          int pstar) {
    Slot s;
    const lds_u64* row = T + I * L;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int par = (I + c) & 1;
        const int J = 2 * h + par;
        const int f = par ? (J == L - 1 ? 0 : J + 1) : (J == 0 ? L - 1 : J - 1);
        s.own[c] = lds_addr(row + J);
        s.far[c] = lds_addr(row + f);
        s.up[c] = lds_addr(T + (I > 0 ? I - 1 : N - 1) * L + J);
        s.dn[c] = lds_addr(T + (I < N - 1 ? I + 1 : 0) * L + J);
        // row I* for row 0; rows without a patch read row 0 and ignore it
        s.pt[c] = lds_addr(T + (I == 0 ? istar : 0) * L + J);
    }
    s.su = I == 0 ? 3u : 0u;
    s.sd = I == N - 1 ? 3u : 0u;
    s.mu = I == 0 ? 1u << 28 : 0u;
    s.md = I == istar ? 1ull << sh_star : 0ull;
    const int n_live = pstar + (I <= istar ? 1 : 0);
    s.live = kSpinBits & (~0ull << (3 * (21 - n_live)));
    return s;
}

// What an apply pass of one lattice needs (wave-uniform): n sweeps with the
// codes at `codes`, a sample after the local sweep j (from 0) when
// (sweep_off + j + 1) % every == 0, every > 0.
struct ApplyTask {
    uint64_t* W;
    int L, N, istar, sh_star;
    const uint64_t* codes;
    int n, sweep_off, every;
};

// The sweeps of an apply pass, the lattice in LDS (T, [N][L]) and the samples'
// (antiparallel bonds, up spins) added to stage[2 k]; returns the number of
// samples.  Thread tid holds the word slots tid + B k (k < WMAX) of each
// colour (past the last slot, one more copy of it: the same loads and the same
// store), and the codes of its words are loaded from the global buffer
// straight into registers, P sweeps ahead of their use.  In a half-sweep no
// word read is written (all neighbours, the wrap words and the patch word
// have the other colour), so every thread loads all of its neighbourhoods
// first and then flips and stores; half-sweeps are separated by a workgroup
// barrier, or, with one wavefront, by the in-order completion of its LDS
// operations.  A half-sweep is a chain -- LDS loads, about 30 vector
// instructions per word, the store, the barrier -- with few wavefronts to fill
// it, so everything that can be is taken off it: addresses and wrap constants
// are formed once; with several wavefronts, whose loads queue for the LDS, a
// slot's own two words stay in registers and only the four words of other
// slots are loaded (with one wavefront the two extra loads cost nothing); a
// sample's sum over the wavefront is formed while the loads of the next
// half-sweep are in flight; and no wavefront without words takes part.
// us per sweep, eight lattices, without samples / a sample each sweep, before
// (selects per half-sweep, six loads, four wavefronts always) and now: L = 16
// 0.41/0.57 and 0.30/0.43, 64 0.48/0.64 and 0.41/0.54, 128 0.94/1.18 and
// 0.73/0.89, 168 1.36/1.63 and 1.04/1.21, 204 1.68/2.00 and 1.30/1.59; 512
// lattices of L = 64 1.52/1.68 and 1.34/1.46, 2048 4.71/5.13 and 4.11/4.30
// (the draws included, which the larger counts are bound by).
template <int WMAX, int P, bool ONE_WAVE>
__device__ __forceinline__ int apply_sweeps(const ApplyTask& a, uint64_t* __restrict__ T, uint32_t* __restrict__ stage) {
    const int L = a.L, N = a.N;
    const int NL = N * L, half = L >> 1, words = N * half;  // words of one colour
    const int tid = threadIdx.x, B = blockDim.x;
    const int n = a.n, every = a.every, pstar = (L - 1) / N;
    const int n_samples = every > 0 ? (a.sweep_off + n) / every - a.sweep_off / every : 0;
    for (int i = tid; i < NL; i += B) T[i] = a.W[i];
    for (int i = tid; i < 2 * n_samples; i += B) stage[i] = 0u;
    Slot slot[WMAX];
#pragma unroll
    for (int k = 0; k < WMAX; ++k) {
        const int f = min(tid + B * k, words - 1);
        const int I = f / half;
        slot[k] = make_slot((const lds_u64*)T, I, f - I * half, L, N, a.istar, a.sh_star, pstar);
    }
    const int sh_up = 60 - a.sh_star;  // between the patch bits of rows L - 1 and 0
    uint64_t ring[P][2][WMAX];
#pragma unroll
    for (int r = 0; r < P; ++r) load_codes<WMAX>(ring[r], a.codes, (size_t)NL, words, tid, B, min(r, n - 1));
    __syncthreads();
    // both words of every slot stay in registers; LDS holds them for the others
    uint64_t held[WMAX][2];
#pragma unroll
    for (int k = 0; k < WMAX; ++k)
#pragma unroll
        for (int c = 0; c < 2; ++c) held[k][c] = lds_load64(slot[k].own[c]);
    __syncthreads();
    // sweeps left before the next sample, the LDS address of that sample, and
    // the thread's counts of the last one while they are not yet summed
    int until = every > 0 ? every - 1 - a.sweep_off % every : 0x7FFFFFFF;
    uint32_t at = lds_addr((const lds_u64*)reinterpret_cast<uint64_t*>(stage));
    bool open = false;
    uint32_t counts = 0;
    auto close_sample = [&] {
        // one wavefront sum of both counts: a wavefront's words (at most 256)
        // have fewer than 2^16 antiparallel bonds (84 per word) and up spins
        // (42 per word, with the near neighbour's)
        const uint32_t both = wave_sum_u32(counts);
        if ((tid & 63) == 0) {
            // one 64-bit LDS add (ups in the high half); the address is kept
            // opaque so that the compiler emits the add alone, not a loop over
            // the lanes in front of it
            asm("" : "+v"(at));
            __hip_atomic_fetch_add((lds_u64*)(size_t)at, ((uint64_t)(both & 0xFFFFu) << 32) | (both >> 16),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        at += 8;
        open = false;
    };
    // the next sweep, with its codes cc
    auto sweep = [&](const uint64_t (&cc)[2][WMAX]) {
        const bool meas = until == 0;
        until = meas ? every - 1 : until - 1;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            uint64_t w[WMAX], near[WMAX], far[WMAX], up[WMAX], dn[WMAX], pt[WMAX];
#pragma unroll
            for (int k = 0; k < WMAX; ++k) {
                const Slot& s = slot[k];
                w[k] = ONE_WAVE ? lds_load64(s.own[c]) : held[k][c];
                near[k] = ONE_WAVE ? lds_load64(s.own[1 - c]) : held[k][1 - c];
                far[k] = lds_load64(s.far[c]);
                up[k] = lds_load64(s.up[c]);
                dn[k] = lds_load64(s.dn[c]);
                pt[k] = lds_load64(s.pt[c]);
            }
            if (c == 0 && open) close_sample();
            uint32_t anti = 0, ups = 0;
#pragma unroll
            for (int k = 0; k < WMAX; ++k) {
                const Slot& s = slot[k];
                const uint32_t pu = (uint32_t)((pt[k] << sh_up) >> 32);  // bit sh_star -> 60
                const uint64_t pd = pt[k] >> sh_up;                     // bit 60 -> sh_star
                uint64_t u = up[k] >> s.su, d = dn[k] << s.sd;
                u |= (uint64_t)(pu & s.mu) << 32;
                d = (d & ~s.md) | (pd & s.md);
                const uint64_t nw = w[k] ^ flip_mask(w[k], u, d, near[k], far[k], cc[c][k], s.live);
                if (!ONE_WAVE) held[k][c] = nw;
                lds_store64(s.own[c], nw);  // a slot past the last word holds and stores that word
                // (near in the place of the left neighbour: the pair of
                // columns holds one word of each colour)
                if (c == 1 && meas && tid + B * k < words)
                    measure_word_packed(nw, u, d, near[k], far[k], s.live, anti, ups);
            }
            if (c == 1 && meas) {
                counts = (anti << 16) | ups;
                open = true;
            }
            if (ONE_WAVE)
                wave_lds_order();
            else
                __syncthreads();
        }
    };
    // whole groups of P sweeps: slot r's codes are used, then reloaded with
    // those P sweeps later
    int j0 = 0;
    for (; j0 + P <= n; j0 += P) {
#pragma unroll
        for (int r = 0; r < P; ++r) {
            sweep(ring[r]);
            load_codes<WMAX>(ring[r], a.codes, (size_t)NL, words, tid, B, min(j0 + r + P, n - 1));
        }
    }
#pragma unroll
    for (int r = 0; r < P; ++r)
        if (j0 + r < n) sweep(ring[r]);
    if (open) close_sample();
    __syncthreads();
    for (int i = tid; i < NL; i += B) a.W[i] = T[i];
    return n_samples;
}

// The samples of an apply pass, in the first wavefront: lane l takes samples
// l, l + 64, ...; E, M to the series (each optional), the moment sums merged
// exactly over the lanes into lane 0's result (when wanted: moments).
__device__ __forceinline__ Moments finish_samples(const uint32_t* __restrict__ stage, int n_samples, int L,
                                                  int64_t* series_E, int64_t* series_M, bool moments) {
    const int64_t nn = (int64_t)L * (int64_t)L;
    Moments part = {};
    for (int k = (int)threadIdx.x; k < n_samples; k += 64) {
        const int64_t E = 2 * (int64_t)stage[2 * k] - 2 * nn, M = 2 * (int64_t)stage[2 * k + 1] - nn;
        if (series_E) series_E[k] = E;
        if (series_M) series_M[k] = M;
        if (moments) add_sample(part, E, M);
    }
    if (moments) wave_merge_moments(part);
    return part;
}

}  // namespace

// Apply pass: one workgroup of at most BLOCK threads (64: one wavefront) per
// lattice entry, S sweeps of the pass (local sweep index s =
// sweep_off + j of the chunk; a sample after it when (s + 1) % every == 0,
// every > 0).  LDS: the lattice [N][L], then one (antiparallel bonds, up
// spins) pair per sample of the pass.
template <int WMAX, int P, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_wave_apply(const LatticeDesc* __restrict__ descs,
                                                               LatticeState* __restrict__ states,
                                                               const DrawLat* __restrict__ lats,
                                                               const uint64_t* __restrict__ codes, int32_t sweep_off,
                                                               int32_t S, int32_t every) {
    extern __shared__ uint64_t lds[];
    const DrawLat dl = lats[blockIdx.x];
    const LatticeDesc& d = descs[dl.lat];
    LatticeState& state = states[dl.lat];
    const int n = min(S, d.sweep_limit - sweep_off);
    if (n <= 0) return;  // uniform over the workgroup
    const int L = d.L;
    uint32_t* __restrict__ stage = reinterpret_cast<uint32_t*>(lds + d.N * L);  // [samples][2]
    const ApplyTask task = {d.W, L, d.N, d.istar, d.sh_star, codes + dl.base, n, sweep_off, every};
    const int n_samples = apply_sweeps<WMAX, P, BLOCK == 64>(task, lds, stage);
    if (threadIdx.x < 64 && n_samples > 0) {
        const int64_t idx = state.series_idx;
        const Moments part = finish_samples(stage, n_samples, L, d.series_E ? d.series_E + idx : nullptr,
                                            d.series_M ? d.series_M + idx : nullptr, true);
        if (threadIdx.x == 0) {
            Moments m = state.mom;
            merge_moments(m, part);
            state.mom = m;
            const int64_t nn = (int64_t)L * (int64_t)L;
            const int k = n_samples - 1;
            state.last_E = 2 * (int64_t)stage[2 * k] - 2 * nn;
            state.last_M = 2 * (int64_t)stage[2 * k + 1] - nn;
            state.series_idx = idx + n_samples;
        }
    }
}

// One lattice of a handle: workgroup 0 applies the sweeps drawn by the launch
// before, the others draw those of the next one, a word of one sweep per
// thread (the chip is otherwise idle, so the draws' latency is what counts:
// a thread's four words one after another would take four times as long).
// us per call with a sample each sweep, before (one resident workgroup that
// draws its own codes; from L = 194 bands of eight columns that exchange their
// boundary words) and now, 20 and 1000 sweeps: L = 16 70/2160 and 27/380, 64
// 82/2754 and 30/476, 128 97/3442 and 33/629, 192 137/5346 and 44/1029, 204
// 83/2745 and 43/1019, 256 82/2616 and 58/1766, 292 84/2770 and 59/1779.
template <int WMAX, int P, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_drawn(DrawnLaunch a) {
    extern __shared__ uint64_t lds[];
    const int L = a.L, N = a.N, NL = N * L;
    if (blockIdx.x > 0) {
        const int f = (int)(blockIdx.x - 1) * (int)blockDim.x + (int)threadIdx.x;
        const int j = f / NL, r = f - j * NL;
        if (j >= a.n_draw) return;
        const int half = L >> 1;
        const int c = r >= N * half ? 1 : 0;
        const int I = (r - c * N * half) / half, h = r - (c * N + I) * half;
        const int par = (I + c) & 1;
        const int J = 2 * h + par;
        const int n_live = (L - 1) / N + (I <= a.istar ? 1 : 0);
        const uint64_t t = a.t_draw + (uint64_t)j;
        const uint32_t t_lo = (uint32_t)t, t_hi = (uint32_t)(t >> 32);
        const RoundKeys rk = round_keys(a.k0, a.k1);
        auto block = [&](uint32_t c1, int g) {
            return philox_lane_c1(t_lo, c1, t_hi, (uint32_t)g | (1u << 3), a.k0, a.k1, rk);
        };
        AcceptWord acc;
        accept_word(acc, [&](int g) { return block((uint32_t)I * (uint32_t)L + (uint32_t)J, g); }, n_live, a.t4, a.t8);
        uint32_t u20 = 0;  // a dead slot when n_live < 21
        if (n_live == 21) {
            const U4 r5 = block((uint32_t)I * (uint32_t)L + (uint32_t)((J & ~7) | par), 5);
            u20 = pick4(make_uint4(r5.x, r5.y, r5.z, r5.w), (uint32_t)h & 3u);
        }
        acc.add<20>(u20, a.t4, a.t8);
        a.drawn[(size_t)j * (size_t)NL + r] = acc.word();
        return;
    }
    if (a.n_apply <= 0) return;
    uint32_t* __restrict__ stage = reinterpret_cast<uint32_t*>(lds + NL);  // [samples][2]
    const ApplyTask task = {a.W, L, N, a.istar, a.sh_star, a.codes, a.n_apply, a.sweep_off, a.every};
    const int n_samples = apply_sweeps<WMAX, P, BLOCK == 64>(task, lds, stage);
    if (threadIdx.x < 64 && n_samples > 0) {
        const Moments part = finish_samples(stage, n_samples, L, a.series_E, a.series_M, a.mom != nullptr);
        if (threadIdx.x == 0 && a.mom) {
            Moments m = *a.mom;
            merge_moments(m, part);
            *a.mom = m;
        }
    }
}

int32_t wave_apply_words_per_thread(int32_t L, int32_t N, int32_t block) {
    const int32_t w = (N * (L / 2) + block - 1) / block;
    return w <= 1 ? 1 : w <= 4 ? w : 0;
}

int32_t wave_apply_block(int32_t words, int32_t wmax) { return ((words + wmax - 1) / wmax + 63) / 64 * 64; }

size_t wave_apply_lds_bytes(int32_t NL, int32_t max_samples) { return (size_t)NL * 8 + (size_t)max_samples * 8; }

hipError_t launch_draw_codes(const LatticeDesc* descs, const LatticeState* states, const DrawLat* lats, int32_t n_lats,
                             int32_t max_n_draw, uint64_t* codes, int32_t sweep_off, int32_t S, hipStream_t s) {
    if (n_lats <= 0 || S <= 0) return hipSuccess;
    const int64_t bpl = ((int64_t)S * max_n_draw + kDrawBlock - 1) / kDrawBlock;
    if (bpl * n_lats > 0x7FFFFFFF || (int64_t)S * max_n_draw > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_draw_codes, dim3((unsigned)(bpl * n_lats)), dim3(kDrawBlock), 0, s, descs, states, lats, codes,
                       (int32_t)bpl, sweep_off, S);
    return hipGetLastError();
}

hipError_t launch_wave_apply(int wmax, int block, const LatticeDesc* descs, LatticeState* states, const DrawLat* lats,
                             int32_t n_lats, const uint64_t* codes, int32_t sweep_off, int32_t S, int32_t every,
                             size_t lds_bytes, hipStream_t s) {
    if (n_lats <= 0 || S <= 0) return hipSuccess;
    if (block < 64 || block > kApplyMaxBlock || block % 64) return hipErrorInvalidValue;
    const dim3 grid(n_lats), blk(block);
#define ISING_WAVE_APPLY(W_, P_, B_)                                                                              \
    hipLaunchKernelGGL((k_wave_apply<W_, P_, B_>), grid, blk, lds_bytes, s, descs, states, lats, codes, sweep_off, \
                       S, every)
    if (block == 64) {
        switch (wmax) {
            case 1: ISING_WAVE_APPLY(1, 8, 64); break;
            case 2: ISING_WAVE_APPLY(2, 8, 64); break;
            case 3: ISING_WAVE_APPLY(3, 4, 64); break;
            case 4: ISING_WAVE_APPLY(4, 4, 64); break;
            default: return hipErrorInvalidValue;
        }
    } else if (block <= 256) {
        switch (wmax) {
            case 1: ISING_WAVE_APPLY(1, 8, 256); break;
            case 2: ISING_WAVE_APPLY(2, 8, 256); break;
            case 3: ISING_WAVE_APPLY(3, 4, 256); break;
            case 4: ISING_WAVE_APPLY(4, 4, 256); break;
            default: return hipErrorInvalidValue;
        }
    } else if (wmax == 1) {
        ISING_WAVE_APPLY(1, 4, 1024);
    } else if (wmax == 2) {
        ISING_WAVE_APPLY(2, 2, 1024);
    } else {
        return hipErrorInvalidValue;
    }
#undef ISING_WAVE_APPLY
    return hipGetLastError();
}

// Two words per thread at the most: a third leaves the 1024 threads without
// registers for codes loaded ahead (L = 320, 1000 sweeps with a sample each: 2699 us
// against 2662 by bands of columns; L = 292 with two words 1779 against 2770).
int32_t drawn_max_words() { return 2 * kApplyMaxBlock; }

size_t drawn_lds_bytes(int32_t L, int32_t N) { return wave_apply_lds_bytes(N * L, kDrawnMaxSweeps); }

hipError_t launch_drawn(const DrawnLaunch& a, hipStream_t s) {
    const int64_t NL = (int64_t)a.N * a.L;
    const int32_t words = a.N * (a.L / 2);
    if (words > drawn_max_words() || a.n_apply > kDrawnMaxSweeps || a.n_draw > kDrawnMaxSweeps)
        return hipErrorInvalidValue;
    const int32_t wmax = wave_apply_words_per_thread(a.L, a.N, kApplyMaxBlock);
    const int block = wave_apply_block(words, wmax);
    const dim3 grid((unsigned)(1 + (a.n_draw * NL + block - 1) / block)), blk(block);
    const size_t lds_bytes = drawn_lds_bytes(a.L, a.N);
#define ISING_DRAWN(W_, P_, B_) hipLaunchKernelGGL((k_drawn<W_, P_, B_>), grid, blk, lds_bytes, s, a)
    if (wmax == 2) ISING_DRAWN(2, 2, 1024);
    else if (block > 256) ISING_DRAWN(1, 4, 1024);
    else if (block > 64) ISING_DRAWN(1, 8, 256);
    else ISING_DRAWN(1, 8, 64);
#undef ISING_DRAWN
    return hipGetLastError();
}

}  // namespace ising
