// gfx950 kernels of the paper's own dynamics: random word picks inside
// vertical strips of the word lattice, left half then right half of every
// strip per iteration (Sections 4 and 5.2, Table 2), and their launchers.
// The per-word update (neighbour words, acceptance codes, flip mask) is the
// one of ising_device.hpp.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ising_device.hpp"
#include "ising_launch.hpp"

namespace ising {

namespace {

// ---------------------------------------------------------------------------
// Strip dynamics (random word picks, two phases per iteration): one thread
// per strip applies that strip's picks of one phase in order.  Strips never
// touch each other's words inside a phase, so threads need no
// synchronisation; a thread sees its own earlier stores.  Pick k draws its
// word from Philox counter (t lo, strip, k div 2, 8 (2 + phase) + 256 t hi)
// -- outputs (x, y) for even k, (z, w) for odd k; row floor(x N / 2^32),
// column off + floor(y width / 2^32) -- and its 21 uniforms from counters
// (t lo, strip, k, g + 8 (4 + phase) + 256 t hi), g = 0..5.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(64) k_strip_phase(uint64_t* __restrict__ W, StripArgs a) {
    const int p = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (p >= a.strips) return;
    const int L = a.L, N = a.N;
    auto ld = [&](int i, int j) { return W[(size_t)i * (size_t)L + (size_t)j]; };
    const uint32_t c3_pick = 8u * (2u + a.phase) + (a.t_hi << 8);
    const uint32_t c3_word = 8u * (4u + a.phase) + (a.t_hi << 8);
    const int col0 = p * a.S + a.off;
    const RoundKeys rk = round_keys(a.k0, a.k1);
    U4 pick = {0u, 0u, 0u, 0u};
    for (uint32_t k = 0; k < a.picks; ++k) {
        if ((k & 1u) == 0u) pick = philox_lane_c1(a.t_lo, (uint32_t)p, k >> 1, c3_pick, a.k0, a.k1);
        const uint32_t x = (k & 1u) ? pick.z : pick.x;
        const uint32_t y = (k & 1u) ? pick.w : pick.y;
        const int I = (int)(((uint64_t)x * (uint64_t)(uint32_t)N) >> 32);
        const int J = col0 + (int)(((uint64_t)y * (uint64_t)(uint32_t)a.width) >> 32);
        const uint64_t w = ld(I, J);
        const uint64_t lf = ld(I, J == 0 ? L - 1 : J - 1);
        const uint64_t rt = ld(I, J == L - 1 ? 0 : J + 1);
        const uint64_t up = up_word(ld, I, J, N, a.istar, a.sh_star);
        const uint64_t dn = down_word(ld, I, J, N, a.istar, a.sh_star);
        // every position draws (dead slots are masked by `live`), so lanes
        // with different rows run the same instructions
        AcceptChain acc;
        accept_word(
            acc, [&](int g) { return philox_lane_c1(a.t_lo, (uint32_t)p, k, (uint32_t)g + c3_word, a.k0, a.k1, rk); }, 21,
            a.t4, a.t8);
        const U4 r5 = philox_lane_c1(a.t_lo, (uint32_t)p, k, 5u + c3_word, a.k0, a.k1, rk);
        acc.add<20>(r5.x, a.t4, a.t8);
        const uint64_t f = flip_mask(w, up, dn, lf, rt, acc.word(), live_mask(I, L, N));
        W[(size_t)I * (size_t)L + (size_t)J] = w ^ f;
    }
}

// The same phase in two steps.  The draws do not depend on the state, so a
// parallel kernel computes, for picks [k0, k0 + n_k) of every strip, the
// word (packed as I << 17 | column within the phase) and the 21 acceptance
// codes; then one lane per strip applies them in order with the strip's
// phase columns and its two frozen neighbour columns held in LDS.
constexpr int kStripColBits = 17;

__global__ void __launch_bounds__(256) k_strip_draws(StripArgs a, uint32_t k0, uint32_t n_k,
                                                    uint32_t* __restrict__ pos, uint64_t* __restrict__ codes_out) {
    const uint64_t total = (uint64_t)n_k * (uint64_t)a.strips;
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const uint32_t kk = (uint32_t)(i / (uint64_t)a.strips);
    const uint32_t p = (uint32_t)(i - (uint64_t)kk * (uint64_t)a.strips);
    const uint32_t k = k0 + kk;
    const uint32_t c3_pick = 8u * (2u + a.phase) + (a.t_hi << 8);
    const uint32_t c3_word = 8u * (4u + a.phase) + (a.t_hi << 8);
    const U4 pick = philox_lane_c1(a.t_lo, p, k >> 1, c3_pick, a.k0, a.k1);
    const uint32_t x = (k & 1u) ? pick.z : pick.x;
    const uint32_t y = (k & 1u) ? pick.w : pick.y;
    const uint32_t I = (uint32_t)(((uint64_t)x * (uint64_t)(uint32_t)a.N) >> 32);
    const uint32_t jl = (uint32_t)(((uint64_t)y * (uint64_t)(uint32_t)a.width) >> 32);
    const RoundKeys rk = round_keys(a.k0, a.k1);
    AcceptWord acc;
    accept_word(
        acc, [&](int g) { return philox_lane_c1(a.t_lo, p, k, (uint32_t)g + c3_word, a.k0, a.k1, rk); }, 21, a.t4, a.t8);
    const U4 r5 = philox_lane_c1(a.t_lo, p, k, 5u + c3_word, a.k0, a.k1, rk);
    acc.add<20>(r5.x, a.t4, a.t8);
    pos[i] = (I << kStripColBits) | jl;
    codes_out[i] = acc.word();
}

// Apply the drawn picks of a phase.  A workgroup (one wavefront) holds
// `chains` strips (1, 2 or 4) in LDS and gives each G = 64 / chains lanes.
// A strip's picks are applied in windows of G picks in pick order: first the
// picks deferred by the previous step, then the next fresh ones.  A pick of
// the window conflicts with an earlier pick of the window iff the earlier
// pick's word is its own word or one it reads (left, right, up, down, the
// wrap-row patch word); this relation is symmetric (each of these neighbour
// relations has its mirror).  Every pick without such a conflict is applied
// now, the others are deferred, in order: a pick applied now commutes with
// every earlier deferred one (neither reads the other's word), and the
// picks applied together read no word another of them writes, while every
// lane of a step loads before any lane stores, so the state is exactly that
// of applying the picks one by one.  The first pick of a window never
// conflicts, so every step applies at least one.  Conflicts are found
// through a claim per word: each lane takes the minimum of its index and the
// claim of its word, then a lane conflicts iff a word it reads carries a
// smaller index.
//
// LDS per strip q: words [q][cc][I] (cc = 0: the frozen column left of the
// phase columns, 1..width: the phase columns, width + 1: the frozen column
// right of them), claims of the same words, the pick data of the current
// block of kStripBlock picks and the deferred picks; then the live-slot mask
// of every word row.
constexpr int kStripBlock = 256;

__global__ void __launch_bounds__(64) k_strip_apply(uint64_t* __restrict__ W, StripArgs a, int chains,
                                                    uint32_t n_k, const uint32_t* __restrict__ pos,
                                                    const uint64_t* __restrict__ codes) {
    extern __shared__ uint64_t strip_lds[];
    const int lane = (int)threadIdx.x;
    const int p0 = (int)blockIdx.x * chains;
    const int n_chains = min(chains, a.strips - p0);
    const int L = a.L, N = a.N, width = a.width, cols = width + 2;
    const int chain_words = cols * N;
    uint64_t* __restrict__ words = strip_lds;
    uint64_t* __restrict__ live_row = words + (size_t)chains * chain_words;
    uint64_t* __restrict__ blk_codes = live_row + N;
    uint32_t* __restrict__ claims = reinterpret_cast<uint32_t*>(blk_codes + (size_t)chains * kStripBlock);
    uint32_t* __restrict__ blk_pos = claims + (size_t)chains * chain_words;
    uint32_t* __restrict__ deferred = blk_pos + (size_t)chains * kStripBlock;  // 64 entries, G per strip

    // cooperative fill: entry e = (row I, chain q, LDS column cc) with
    // (q, cc) fastest, so neighbouring threads read neighbouring columns
    const int per_row = n_chains * cols;
    const int n_fill = per_row * N;
    auto fill_col = [&](int e, int& q, int& cc, int& I) {
        I = e / per_row;
        const int rem = e - I * per_row;
        q = rem / cols;
        cc = rem - q * cols;
    };
    for (int e0 = lane; e0 < n_fill; e0 += 64 * 8) {
        uint64_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = e0 + 64 * u;
            if (e < n_fill) {
                int q, cc, I;
                fill_col(e, q, cc, I);
                const int J = ((p0 + q) * a.S + a.off + cc - 1 + L) % L;
                v[u] = W[(size_t)I * (size_t)L + (size_t)J];
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = e0 + 64 * u;
            if (e < n_fill) {
                int q, cc, I;
                fill_col(e, q, cc, I);
                words[(size_t)q * chain_words + (size_t)cc * N + I] = v[u];
            }
        }
    }
    for (int I = lane; I < N; I += 64) live_row[I] = live_mask(I, L, N);
    for (int e = lane; e < chains * chain_words; e += 64) claims[e] = 0xFFFFFFFFu;

    // lanes of a strip: group q = lane / G, index i = lane % G
    const int G = 64 / chains;
    const int q = lane / G;
    const int i = lane - q * G;
    const bool has_chain = q < n_chains;
    uint64_t* __restrict__ my = words + (size_t)q * chain_words;
    uint32_t* __restrict__ my_claim = claims + (size_t)q * chain_words;
    const int istar = a.istar, sh_star = a.sh_star;
    const size_t stride = (size_t)a.strips;

    // pick data of a block: entry e = (chain qq, pick j) with j fastest;
    // held in registers while the previous block is applied
    constexpr int kPer = kStripBlock * 4 / 64;  // entries per lane for up to 4 chains
    const int n_entries = chains * kStripBlock;
    uint32_t rq[kPer];
    uint64_t rd[kPer];
    auto fetch = [&](uint32_t b0) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int e = lane + 64 * u;
            const int qq = e / kStripBlock, j = e - (e / kStripBlock) * kStripBlock;
            const uint32_t k = min(b0 + (uint32_t)j, n_k - 1);
            const bool ok = e < n_entries && qq < n_chains;
            const size_t idx = (size_t)k * stride + (size_t)(p0 + (ok ? qq : 0));
            rq[u] = ok ? pos[idx] : 0u;
            rd[u] = ok ? codes[idx] : 0ull;
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int e = lane + 64 * u;
            if (e < n_entries) {
                blk_pos[e] = rq[u];
                blk_codes[e] = rd[u];
            }
        }
    };
    fetch(0u);
    __syncthreads();

    for (uint32_t b0 = 0; b0 < n_k; b0 += kStripBlock) {
        stash();
        fetch(b0 + kStripBlock);  // in flight while this block is applied
        __syncthreads();
        const uint32_t bend = min(b0 + (uint32_t)kStripBlock, n_k);
        uint32_t kk = b0;     // next fresh pick of this strip (same in all its lanes)
        uint32_t n_def = 0;   // picks of this strip deferred by the previous step
        const uint64_t gbits = (G == 64) ? ~0ull : (((1ull << G) - 1ull) << (q * G));
        const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));  // lanes before this one
        while (true) {
            const bool pending = has_chain && (n_def > 0u || kk < bend);
            if (__ballot(pending) == 0ull) break;  // every strip of the workgroup is through the block
            uint32_t k;
            bool act;
            if ((uint32_t)i < n_def) {
                k = deferred[q * G + i];
                act = true;
            } else {
                k = kk + ((uint32_t)i - n_def);
                act = has_chain && k < bend;
            }
            int w = 0, lf = 0, rt = 0, up = 0, dn = 0, patch = 0, I = 0;
            uint64_t cd = 0;
            if (act) {
                const uint32_t pk = blk_pos[q * kStripBlock + (int)(k - b0)];
                cd = blk_codes[q * kStripBlock + (int)(k - b0)];
                I = (int)(pk >> kStripColBits);
                const int base = ((int)(pk & ((1u << kStripColBits) - 1u)) + 1) * N;
                w = base + I;
                lf = w - N;
                rt = w + N;
                up = base + (I > 0 ? I - 1 : N - 1);
                dn = base + (I < N - 1 ? I + 1 : 0);
                // the patch word of the wrap rows (row I* for I = 0, row 0
                // for I = I*); other rows read their own word again
                patch = I == 0 ? base + istar : (I == istar ? base : w);
                atomicMin(&my_claim[w], (uint32_t)i);
            }
            bool conflict = false;
            uint64_t vw = 0, vlf = 0, vrt = 0, vup = 0, vdn = 0, vpatch = 0, vlive = 0;
            if (act) {
                // all twelve loads in flight together: the claims combined
                // without short-circuit, which would make six dependent round
                // trips of them
                const uint32_t ui = (uint32_t)i;
                const uint32_t c_w = my_claim[w], c_lf = my_claim[lf], c_rt = my_claim[rt], c_up = my_claim[up],
                               c_dn = my_claim[dn], c_pa = my_claim[patch];
                conflict = (c_w < ui) | (c_lf < ui) | (c_rt < ui) | (c_up < ui) | (c_dn < ui) | (c_pa < ui);
                vw = my[w];
                vlf = my[lf];
                vrt = my[rt];
                vup = my[up];
                vdn = my[dn];
                vpatch = my[patch];
                vlive = live_row[I];
            }
            if (act && !conflict) {
                uint64_t vu = vup, vd = vdn;
                if (I == 0) vu = (vu >> 3) | (((vpatch >> sh_star) & 1ull) << 60);
                if (I == N - 1) vd = (vd << 3) & kLow63;
                if (I == istar) vd = (vd & ~(1ull << sh_star)) | (((vpatch >> 60) & 1ull) << sh_star);
                my[w] = vw ^ flip_mask(vw, vu, vd, vlf, vrt, cd, vlive);
            }
            if (act) my_claim[w] = 0xFFFFFFFFu;
            // the conflicting picks, in order, head the next window
            const uint64_t cmask = __ballot(act && conflict) & gbits;
            const uint64_t amask = __ballot(act) & gbits;
            if (act && conflict) deferred[q * G + __builtin_popcountll(cmask & below)] = k;
            kk += (uint32_t)__builtin_popcountll(amask) - n_def;  // fresh picks taken into this window
            n_def = (uint32_t)__builtin_popcountll(cmask);
        }
        __syncthreads();
    }

    __syncthreads();
    // cooperative write-back of the phase columns (LDS columns 1..width)
    const int per_row_w = n_chains * width;
    const int n_back = per_row_w * N;
    for (int e = lane; e < n_back; e += 64) {
        const int I = e / per_row_w;
        const int rem = e - I * per_row_w;
        const int qq = rem / width;
        const int cc = rem - qq * width + 1;
        const int J = (p0 + qq) * a.S + a.off + cc - 1;
        W[(size_t)I * (size_t)L + (size_t)J] = words[(size_t)qq * chain_words + (size_t)cc * N + I];
    }
}

// ---------------------------------------------------------------------------
// The same phase from lists per word.  A word's picks are applied in order,
// and a pick commutes with every other one whose word it neither is nor reads;
// so the state is that of applying the picks one by one if a word's next pick is
// applied only when it is earlier than the next picks of the words it reads
// (its phase neighbours: left, right, up, down, the wrap rows' patch word; the
// relation is symmetric).  One to four wavefronts take a strip, a word of the
// phase (at most two) per lane: in every step the lanes whose next pick is the
// earliest of its neighbourhood apply it, all loads of a step before its stores,
// and put their word's next pick in its place.  That takes as many steps as the
// longest chain of dependent picks is long (46 on average and about 60 in the
// worst of 1008 strips, for the ten picks per word of a phase), with nothing
// claimed, deferred or looked up in between; what is left is the chain of a
// step, 0.4 us.  The lists are made by the launch before (in its other
// workgroups, a strip each, beside the strips that this one applies): the draws
// do not depend on the state.  us per phase with E and M after every second
// one, windows of picks with claims above / lists: L = 84 in strips of 2 columns
// 29 / 16, 1008 of 2 47 / 24, of 6 71 / 34, 2016 of 2 73 / 36 (28 of the 30 us of
// a launch are the application, 20 the draws beside it), of 4 90 / 37, of 6 110 / 59,
// 4200 of 2 182 / 138.  The windows stay with more
// than 512 words per phase, and with more than 1.5 Mi words in all strips.
// ---------------------------------------------------------------------------
constexpr int kListBlock = 256;
constexpr uint32_t kNoPick = 0xFFFFFFFFu;

// LDS of one applied strip: the words and the numbers of the next picks of its phase
// columns and of the two frozen columns beside them ([width + 2][N]), the codes
// and the pick numbers of its list (with an entry more of each, read and not
// used).
__host__ __device__ inline size_t list_strip_bytes(int cells, uint32_t n_k) {
    return ((size_t)cells * 12 + (size_t)(n_k + 1) * 10 + 15) / 16 * 16;
}

// LDS of drawing one strip's list: first entry and fill count per word, then word
// and bucket entry per pick.
__host__ __device__ inline size_t list_draw_bytes(int sites, uint32_t n_k) {
    return (size_t)(2 * sites + 2) * 4 + (size_t)n_k * 4;
}

// The list of strip p: its picks [k0, k0 + n_k) by word (column of the phase,
// row), in pick order for each word.
__device__ void draw_strip_list(const StripArgs& a, const StripLists& l, uint32_t p, uint64_t* lds) {
    const int N = a.N, sites = N * a.width, tid = threadIdx.x;
    const uint32_t n_k = l.n_k;
    uint32_t* __restrict__ first = reinterpret_cast<uint32_t*>(lds);  // [sites + 1]: counts, then their sums
    uint32_t* __restrict__ fill = first + sites + 1;                  // [sites + 1]
    uint16_t* __restrict__ site = reinterpret_cast<uint16_t*>(fill + sites + 1);
    uint16_t* __restrict__ bucket = site + n_k;
    const uint32_t c3_pick = 8u * (2u + a.phase) + (a.t_hi << 8);
    const uint32_t c3_word = 8u * (4u + a.phase) + (a.t_hi << 8);
    const RoundKeys rk = round_keys(a.k0, a.k1);
    for (int s = tid; s <= sites; s += kListBlock) first[s] = fill[s] = 0u;
    __syncthreads();
    // a Philox block holds two picks; k0 and n_k are even
    for (uint32_t h = tid; h < n_k / 2; h += kListBlock) {
        const U4 r = philox_lane_c1(a.t_lo, p, l.k0 / 2 + h, c3_pick, a.k0, a.k1, rk);
        const uint32_t x[2] = {r.x, r.z}, y[2] = {r.y, r.w};
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t I = (uint32_t)(((uint64_t)x[e] * (uint64_t)(uint32_t)N) >> 32);
            const uint32_t jl = (uint32_t)(((uint64_t)y[e] * (uint64_t)(uint32_t)a.width) >> 32);
            const uint32_t s = jl * (uint32_t)N + I;
            site[2 * h + e] = (uint16_t)s;
            atomicAdd(&first[s], 1u);
        }
    }
    __syncthreads();
    // sums over the words before each (at most 512 words: eight per lane)
    if (tid < 64) {
        uint32_t c[8], sum = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int s = 8 * tid + e;
            c[e] = sum;
            sum += s < sites ? first[s] : 0u;
        }
        uint32_t before = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_up(before, off, 64);
            before += tid >= off ? o : 0u;
        }
        before -= sum;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int s = 8 * tid + e;
            if (s < sites) first[s] = before + c[e];
        }
        if (tid == 0) first[sites] = n_k;
    }
    __syncthreads();
    uint16_t* __restrict__ out_first = l.first + (size_t)p * (size_t)(sites + 1);
    for (int s = tid; s <= sites; s += kListBlock) out_first[s] = (uint16_t)first[s];
    for (uint32_t k = tid; k < n_k; k += kListBlock) {
        const uint32_t s = site[k];
        bucket[first[s] + atomicAdd(&fill[s], 1u)] = (uint16_t)k;
    }
    __syncthreads();
    uint16_t* __restrict__ out_k = l.k + (size_t)p * n_k;
    uint64_t* __restrict__ out_codes = l.codes + (size_t)p * n_k;
    for (uint32_t i = tid; i < n_k; i += kListBlock) {
        const uint32_t k = bucket[i], s = site[k];
        uint32_t at = first[s], before = 0;
        const uint32_t end = first[s + 1];
        for (uint32_t j = at; j < end; j += 4) {
            // four reads in flight; those past the word's own entries count for nothing
            const uint32_t b0 = bucket[j], b1 = bucket[min(j + 1, n_k - 1)], b2 = bucket[min(j + 2, n_k - 1)],
                           b3 = bucket[min(j + 3, n_k - 1)];
            before += (b0 < k ? 1u : 0u) + (j + 1 < end && b1 < k ? 1u : 0u) + (j + 2 < end && b2 < k ? 1u : 0u) +
                      (j + 3 < end && b3 < k ? 1u : 0u);
        }
        at += before;
        AcceptWord acc;
        accept_word(
            acc,
            [&](int g) { return philox_lane_c1(a.t_lo, p, l.k0 + k, (uint32_t)g + c3_word, a.k0, a.k1, rk); }, 21, a.t4,
            a.t8);
        const U4 r5 = philox_lane_c1(a.t_lo, p, l.k0 + k, 5u + c3_word, a.k0, a.k1, rk);
        acc.add<20>(r5.x, a.t4, a.t8);
        out_k[at] = (uint16_t)k;
        out_codes[at] = acc.word();
    }
}

// The picks of strip p's list applied by V wavefronts, R words per lane.  With one
// wavefront its LDS operations keep the steps in order; with more a barrier of
// the workgroup follows the loads of a step and another its stores, and the
// workgroup's strips (p past the last one: none) step together; busy: two words
// of LDS, for the last step in which a wavefront of it had picks left.
template <int R, int V, bool ONE_COLUMN>
__device__ __forceinline__ void apply_strip_list(uint64_t* __restrict__ W, const StripArgs& a, const StripLists& l,
                                                 int p, uint64_t* lds, uint32_t* busy) {
    const bool strip = p < a.strips;
    p = min(p, a.strips - 1);
    const int L = a.L, N = a.N, width = ONE_COLUMN ? 1 : a.width, cells = (width + 2) * N, sites = N * width;
    constexpr int T = 64 * V;
    const int tid = (int)threadIdx.x & (T - 1);
    const uint32_t n_k = l.n_k;
    uint64_t* __restrict__ word = lds;
    uint64_t* __restrict__ codes = word + cells;
    uint32_t* __restrict__ next = reinterpret_cast<uint32_t*>(codes + n_k + 1);
    uint16_t* __restrict__ ks = reinterpret_cast<uint16_t*>(next + cells);
    const uint64_t* __restrict__ in_codes = l.codes + (size_t)p * n_k;
    const uint32_t* __restrict__ in_k = reinterpret_cast<const uint32_t*>(l.k + (size_t)p * n_k);  // n_k is even
    const uint16_t* __restrict__ in_first = l.first + (size_t)p * (size_t)(sites + 1);
    const int col0 = p * a.S + a.off - 1;  // column of cell 0
    auto order = [&] {
        if (V == 1) wave_lds_order();
        else __syncthreads();
    };
#pragma unroll 4
    for (uint32_t e = tid; e < n_k; e += T) codes[e] = in_codes[e];
#pragma unroll 4
    for (uint32_t e = tid; e < n_k / 2; e += T) reinterpret_cast<uint32_t*>(ks)[e] = in_k[e];
#pragma unroll 4
    for (int e = tid; e < cells; e += T) {
        // neighbouring lanes take neighbouring columns
        const int I = e / (width + 2), cc = e - I * (width + 2);
        int J = col0 + cc;
        J = J < 0 ? J + L : J >= L ? J - L : J;
        word[cc * N + I] = W[(size_t)I * (size_t)L + (size_t)J];
        next[cc * N + I] = kNoPick;
    }
    order();
    // LDS indexes of the words and their patch words, and the step to the column
    // to the right; the frozen words beside a single column stay in registers
    int at[R], up[R], dn[R], pt[R];
    uint32_t own[R], ptr[R], end[R], su[R], sd[R], mu[R];
    uint64_t code[R], w[R], live[R], md[R], fl[R], fr[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int s = tid + T * r, sc = min(s, sites - 1);
        const int cc = sc / N + 1, I = sc - (cc - 1) * N;
        at[r] = cc * N + I;
        up[r] = cc * N + (I > 0 ? I - 1 : N - 1);
        dn[r] = cc * N + (I < N - 1 ? I + 1 : 0);
        pt[r] = I == 0 ? cc * N + a.istar : I == a.istar ? cc * N : -1;
        su[r] = I == 0 ? 3u : 0u;
        sd[r] = I == N - 1 ? 3u : 0u;
        mu[r] = I == 0 ? 1u << 28 : 0u;
        md[r] = I == a.istar ? 1ull << a.sh_star : 0ull;
        live[r] = live_mask(I, L, N);
        w[r] = word[at[r]];
        fl[r] = word[at[r] - N];
        fr[r] = word[at[r] + N];
        const uint32_t first = in_first[sc];
        end[r] = in_first[sc + 1];
        own[r] = strip && s < sites && first < end[r] ? (uint32_t)ks[first] : kNoPick;
        code[r] = codes[first];
        ptr[r] = min(first + 1, n_k);
    }
    order();
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (tid + T * r < sites) next[at[r]] = own[r];
    order();
    const int sh_up = 60 - a.sh_star;  // between the patch bits of rows L - 1 and 0
    // Every step applies at least the strip's earliest pick left.  A step's loads
    // are all in flight together (the word's next entry of the list too), and
    // no more of them than a step needs: with eight wavefronts in a compute unit
    // the LDS is soon what bounds it (with all six words and numbers of every lane
    // by 128-bit loads a launch took 37 us instead of 30).
    for (uint32_t step = 1;; ++step) {
        bool left = false;
#pragma unroll
        for (int r = 0; r < R; ++r) left |= own[r] != kNoPick;
        const bool wave_left = __ballot(left) != 0ull;
        if (V == 1 && !wave_left) break;
        if (V > 1 && wave_left) busy[step & 1u] = step;
        uint64_t wu[R], wd[R], wl[R], wr[R], wp[R], ncode[R];
        uint32_t m[R], nk[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint32_t n_up = next[up[r]], n_dn = next[dn[r]], n_lf = kNoPick, n_rt = kNoPick, n_pt = kNoPick;
            wu[r] = word[up[r]];
            wd[r] = word[dn[r]];
            wl[r] = fl[r];
            wr[r] = fr[r];
            wp[r] = 0;
            if (!ONE_COLUMN) {
                n_lf = next[at[r] - N];
                n_rt = next[at[r] + N];
                wl[r] = word[at[r] - N];
                wr[r] = word[at[r] + N];
            }
            if (pt[r] >= 0) {
                n_pt = next[pt[r]];
                wp[r] = word[pt[r]];
            }
            nk[r] = ks[ptr[r]];
            ncode[r] = codes[ptr[r]];
            m[r] = min(min(n_up, n_dn), min(min(n_lf, n_rt), n_pt));
        }
        uint64_t nw[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t pu = (uint32_t)((wp[r] << sh_up) >> 32);  // bit sh_star -> 60
            const uint64_t pd = wp[r] >> sh_up;                     // bit 60 -> sh_star
            uint64_t u = wu[r] >> su[r], d = wd[r] << sd[r];
            u |= (uint64_t)(pu & mu[r]) << 32;
            d = (d & ~md[r]) | (pd & md[r]);
            nw[r] = w[r] ^ flip_mask(w[r], u, d, wl[r], wr[r], code[r], live[r]);
            nk[r] = ptr[r] < end[r] ? nk[r] : kNoPick;
        }
        if (V > 1) __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (own[r] < m[r]) {
                word[at[r]] = nw[r];
                next[at[r]] = nk[r];
                w[r] = nw[r];
                own[r] = nk[r];
                code[r] = ncode[r];
                ptr[r] = min(ptr[r] + 1, n_k);
            }
        }
        if (V > 1 && busy[step & 1u] != step) break;  // the same in every wavefront
        order();
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int s = tid + T * r;
        if (strip && s < sites) {
            const int c = s / N, I = s - c * N;
            W[(size_t)I * (size_t)L + (size_t)(col0 + 1 + c)] = w[r];
        }
    }
}

// Workgroups [0, apply_blocks) apply the lists `l` of phase a, 4 / V strips each; the
// others draw the lists `ln` of phase n, a strip each.
template <int R, int V, bool ONE_COLUMN>
__global__ void __launch_bounds__(kListBlock) k_strip_lists(uint64_t* __restrict__ W, StripArgs a, StripLists l,
                                                            int apply_blocks, StripArgs n, StripLists ln) {
    extern __shared__ uint64_t list_lds[];
    __shared__ uint32_t busy[2];
    if ((int)blockIdx.x >= apply_blocks) {
        draw_strip_list(n, ln, blockIdx.x - (uint32_t)apply_blocks, list_lds);
        return;
    }
    if (threadIdx.x < 2) busy[threadIdx.x] = 0u;  // (steps count from 1; barriers follow)
    const int group = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / (64 * V)));
    const int p = (int)blockIdx.x * (4 / V) + group;
    if (V == 1 && p >= a.strips) return;
    apply_strip_list<R, V, ONE_COLUMN>(
        W, a, l, p, list_lds + (size_t)group * (list_strip_bytes((a.width + 2) * a.N, l.n_k) / sizeof(uint64_t)), busy);
}

// Wavefronts of a strip of `sites` words per phase: a word per lane as far as four
// go (L = 2016 in strips of two columns, 96 words: two wavefronts 30 us per launch,
// one with two words per lane 33).
inline int list_waves(int sites) { return sites <= 64 ? 1 : sites <= 128 ? 2 : 4; }
inline int list_strips(const StripArgs& a) { return 4 / list_waves(a.N * a.width); }

inline unsigned strip_grid(uint64_t n, int block) { return (unsigned)((n + block - 1) / block); }

}  // namespace

size_t strip_apply_lds_bytes(const StripArgs& a, int chains) {
    const size_t words = (size_t)chains * (size_t)(a.width + 2) * (size_t)a.N;
    return words * (sizeof(uint64_t) + sizeof(uint32_t)) + (size_t)a.N * sizeof(uint64_t) +
           (size_t)chains * kStripBlock * (sizeof(uint64_t) + sizeof(uint32_t)) + 64 * sizeof(uint32_t);
}

hipError_t launch_strip_phase(uint64_t* W, const StripArgs& a, hipStream_t s) {
    if (a.strips <= 0 || a.picks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_strip_phase, dim3(strip_grid((uint64_t)a.strips, 64)), dim3(64), 0, s, W, a);
    return hipGetLastError();
}

size_t strip_chain_lds_bytes(const StripArgs& a) { return (size_t)(a.width + 2) * (size_t)a.N * sizeof(uint64_t); }

hipError_t launch_strip_draws(const StripArgs& a, uint32_t k0, uint32_t n_k, uint32_t* pos, uint64_t* codes,
                              hipStream_t s) {
    const uint64_t total = (uint64_t)n_k * (uint64_t)a.strips;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_strip_draws, dim3(strip_grid(total, 256)), dim3(256), 0, s, a, k0, n_k, pos, codes);
    return hipGetLastError();
}

hipError_t launch_strip_apply(uint64_t* W, const StripArgs& a, uint32_t n_k, const uint32_t* pos,
                              const uint64_t* codes, hipStream_t s) {
    if (a.strips <= 0 || n_k == 0) return hipSuccess;
    int chains = 2;  // two strips of 32 lanes per wavefront (measured best of 1, 2, 4)
    while (chains > 1 && strip_apply_lds_bytes(a, chains) > kStripLdsBytes) chains /= 2;
    const size_t lds = strip_apply_lds_bytes(a, chains);
    if (lds > kStripLdsBytes) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_strip_apply, dim3(strip_grid((uint64_t)a.strips, chains)), dim3(64), lds, s, W, a, chains,
                       n_k, pos, codes);
    return hipGetLastError();
}

uint32_t strip_list_picks(const StripArgs& a, int64_t max_entries) {
    const int64_t sites = (int64_t)a.N * a.width;
    if (sites > 512) return 0;
    const int64_t room = (int64_t)(kStripListLds / list_strips(a)) - (int64_t)list_strip_bytes((a.width + 2) * a.N, 1);
    int64_t n = std::min<int64_t>({room / 10, max_entries / a.strips, 65534, (int64_t)a.picks});
    n &= ~int64_t(1);
    return n < 2 || list_draw_bytes((int)sites, (uint32_t)n) > kStripListLds ? 0u : (uint32_t)n;
}

hipError_t allow_strip_list_lds() {
    const void* fs[] = {reinterpret_cast<const void*>(&k_strip_lists<1, 1, true>),
                        reinterpret_cast<const void*>(&k_strip_lists<1, 1, false>),
                        reinterpret_cast<const void*>(&k_strip_lists<1, 2, true>),
                        reinterpret_cast<const void*>(&k_strip_lists<1, 2, false>),
                        reinterpret_cast<const void*>(&k_strip_lists<1, 4, true>),
                        reinterpret_cast<const void*>(&k_strip_lists<1, 4, false>),
                        reinterpret_cast<const void*>(&k_strip_lists<2, 4, true>),
                        reinterpret_cast<const void*>(&k_strip_lists<2, 4, false>)};
    for (const void* f : fs) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStripListLds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_strip_lists(uint64_t* W, const StripArgs& a, const StripLists& l, const StripArgs& n,
                              const StripLists& ln, hipStream_t s) {
    const int per = l.n_k ? list_strips(a) : 1;
    const int apply_blocks = l.n_k ? (a.strips + per - 1) / per : 0;
    const int draw_blocks = ln.n_k ? n.strips : 0;
    if (apply_blocks + draw_blocks == 0) return hipSuccess;
    const int sites = l.n_k ? a.N * a.width : 1;
    size_t lds = l.n_k ? per * list_strip_bytes((a.width + 2) * a.N, l.n_k) : 0;
    if (ln.n_k) lds = std::max(lds, list_draw_bytes(n.N * n.width, ln.n_k));
    if (sites > 512 || (ln.n_k && n.N * n.width > 512) || lds > kStripListLds || l.n_k % 2 || ln.n_k % 2 || ln.k0 % 2)
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)(apply_blocks + draw_blocks)), blk(kListBlock);
#define ISING_STRIP_LISTS(R_, V_)                                                                        \
    if (a.width == 1)                                                                                    \
        hipLaunchKernelGGL((k_strip_lists<R_, V_, true>), grid, blk, lds, s, W, a, l, apply_blocks, n, ln); \
    else                                                                                                 \
        hipLaunchKernelGGL((k_strip_lists<R_, V_, false>), grid, blk, lds, s, W, a, l, apply_blocks, n, ln)
    if (sites <= 64) {
        ISING_STRIP_LISTS(1, 1);
    } else if (sites <= 128) {
        ISING_STRIP_LISTS(1, 2);
    } else if (sites <= 256) {
        ISING_STRIP_LISTS(1, 4);
    } else {
        ISING_STRIP_LISTS(2, 4);
    }
#undef ISING_STRIP_LISTS
    return hipGetLastError();
}

}  // namespace ising
