// gfx950 kernels of replica multi-spin coding: 21 independent L x L lattices
// (replicas) packed field by field into one word lattice, W[r][c] holding
// site (r, c) of replica k in field 20 - k (the coding family of Section 3
// applied across systems instead of down a column).  Replicas never
// interact; each runs the checkerboard Metropolis chain at its own
// temperature.  Neighbour words are the plain neighbours on the torus, every
// field is live, so the word update of ising_device.hpp applies with a
// threshold pair per field.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ising_device.hpp"
#include "ising_moments.hpp"
#include "ising_replicas.hpp"
#include "ising_row_words.hpp"

namespace ising {

namespace {

constexpr uint32_t kStreamSweep = 6;  // Philox counter word 3 = g + 8 stream
constexpr uint32_t kStreamInit = 7;
constexpr int kHalfSweepBlock = 64;

// Draw of replica k at site (r, c): block g = k div 4 (k < 20) keyed by the
// site, output k mod 4; replica 20 shares block 5 among the four same-colour
// sites 8 (c div 8) + (c mod 2) + 2m of the row, output (c div 2) mod 4.
__device__ __forceinline__ uint32_t replica_draw(uint32_t t_lo, uint32_t t_hi, uint32_t stream, int L, int k, int r,
                                                 int c, uint32_t k0, uint32_t k1) {
    const uint32_t col = k < 20 ? (uint32_t)c : (((uint32_t)c & ~7u) | ((uint32_t)c & 1u));
    const uint32_t g = k < 20 ? (uint32_t)(k >> 2) : 5u;
    const U4 o = philox_lane_c1(t_lo, (uint32_t)r * (uint32_t)L + col, t_hi, g + 8u * stream, k0, k1);
    const uint32_t q = k < 20 ? (uint32_t)(k & 3) : (((uint32_t)c >> 1) & 3u);
    return q == 0 ? o.x : q == 1 ? o.y : q == 2 ? o.z : o.w;
}

__global__ void __launch_bounds__(256) k_replica_init(uint64_t* __restrict__ W, int L, uint32_t k0, uint32_t k1,
                                                     int hot) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (uint64_t)L * (uint64_t)L) return;
    const int r = (int)(i / (uint64_t)L), c = (int)(i - (uint64_t)r * (uint64_t)L);
    uint64_t w = 0;
    for (int k = 0; k < kReplicas; ++k) {
        const bool up = !hot || replica_draw(0u, 0u, kStreamInit, L, k, r, c, k0, k1) < 0x80000000u;
        w |= (uint64_t)up << (3 * (20 - k));
    }
    W[i] = w;
}

// The four replicas of Philox block G, each with its own thresholds.
template <int G>
__device__ __forceinline__ void replica_accept(AcceptPair& acc, const U4& o, const ReplicaArgs& a) {
    acc.add<4 * G + 0>(o.x, a.t4[4 * G + 0], a.t8[4 * G + 0]);
    acc.add<4 * G + 1>(o.y, a.t4[4 * G + 1], a.t8[4 * G + 1]);
    acc.add<4 * G + 2>(o.z, a.t4[4 * G + 2], a.t8[4 * G + 2]);
    acc.add<4 * G + 3>(o.w, a.t4[4 * G + 3], a.t8[4 * G + 3]);
}

// What a half-sweep of the replicas does with a run of words: a threshold
// pair per field, all fields live, plain neighbours on the torus.
struct ReplicaRule {
    typedef AcceptPair Accept;
    const ReplicaArgs& a;
    uint64_t live = kSpinBits;
    template <class Block>
    __device__ __forceinline__ void accept(AcceptPair& acc, const Block& block) const {
        replica_accept<0>(acc, block(0), a);
        replica_accept<1>(acc, block(1), a);
        replica_accept<2>(acc, block(2), a);
        replica_accept<3>(acc, block(3), a);
        replica_accept<4>(acc, block(4), a);
    }
    __device__ __forceinline__ void accept20(AcceptPair& acc, uint32_t u) const { acc.add<20>(u, a.t4[20], a.t8[20]); }
    __device__ __forceinline__ void vertical(uint64_t&, uint64_t&, uint64_t) const {}
    __device__ __forceinline__ void after(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t) const {}
};

// One colour of every replica: every wavefront updates 64 WPT words of the
// colour of one row (row_block).
template <int WPT>
__global__ void __launch_bounds__(kHalfSweepBlock) k_replica_halfsweep(uint64_t* __restrict__ W, ReplicaArgs a, int colour,
                                                                      int band) {
    __shared__ __align__(16) uint32_t table[(kHalfSweepBlock / 64) * row_table_words<WPT>()];
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const RowBlock b = row_block(band);
    const int row = b.row;
    if (row >= a.L) return;
    const int x = b.x * (int)(blockDim.x >> 6) + wv;  // wavefront of the row
    const size_t L = (size_t)a.L;
    uint64_t* const W_row = W + (size_t)row * L;
    const RowRun r = {W_row,
                      W + (size_t)(row == 0 ? a.L - 1 : row - 1) * L,
                      W + (size_t)(row == a.L - 1 ? 0 : row + 1) * L,
                      W_row,
                      false,
                      a.L,
                      (row + colour) & 1,
                      (uint32_t)row * (uint32_t)a.L,
                      a.t_lo,
                      a.t_hi,
                      8u * kStreamSweep,
                      a.k0,
                      a.k1,
                      true};
    update_row_words<WPT>(r, 64 * WPT * x, table + wv * row_table_words<WPT>(), ReplicaRule{a});
}

// Per-replica antiparallel right+down bonds and up spins of all words.
// Each thread adds fields 0..19 in 6-bit lanes (even fields from bit 0, odd
// fields shifted down by 3), at most 2 per word, flushing to per-replica
// counters every 31 words; field 20 (bit 60, whose lane would have only 4
// bits) is counted directly.  The workgroup then sums the counters in LDS
// and adds them to one of kTotalCopies copies of the totals, [0..20] (bonds) and
// [21..41] (up spins).  A thread loads four words at a time: one by one, each
// waits for its loads in turn.  us per sample, before (one by one, 32 words per
// thread, one copy of the totals) and now: L = 256 22/9, 1024 29/13, 2048
// 32/17, 4096 68/42; with one copy of the totals 10, 17, 26, 48.
constexpr uint64_t kLaneFields = 0x0041041041041041ull;  // bits 0, 6, ..., 54

__device__ __forceinline__ void flush_lanes(uint64_t& even, uint64_t& odd, uint32_t* cnt) {
#pragma unroll
    for (int f = 0; f < 20; ++f) {
        const uint64_t v = (f & 1) ? (odd >> (6 * (f >> 1))) : (even >> (6 * (f >> 1)));
        cnt[20 - f] += (uint32_t)(v & 63u);  // field f holds replica 20 - f
    }
    even = 0;
    odd = 0;
}

__global__ void __launch_bounds__(256) k_replica_observe(const uint64_t* __restrict__ W, int L, uint32_t run,
                                                        unsigned long long* __restrict__ totals) {
    __shared__ uint32_t sums[2 * kReplicas];
    for (int i = threadIdx.x; i < 2 * kReplicas; i += blockDim.x) sums[i] = 0;
    __syncthreads();
    uint32_t anti[kReplicas], ups[kReplicas];
#pragma unroll
    for (int k = 0; k < kReplicas; ++k) anti[k] = ups[k] = 0;
    uint64_t ae = 0, ao = 0, ue = 0, uo = 0;
    int pending = 0;
    // a run of consecutive words per workgroup, four of them in flight per thread
    const uint64_t n = (uint64_t)L * (uint64_t)L;
    const uint64_t end = min(n, (uint64_t)(blockIdx.x + 1) * run);
    uint64_t i = (uint64_t)blockIdx.x * run + threadIdx.x;
    int r = (int)(i / (uint64_t)L), c = (int)(i - (uint64_t)r * (uint64_t)L);
    const int rows = 256 / L, cols = 256 - rows * L;  // from one word of a thread to its next
    while (i < end) {
        uint64_t w[4], rt[4], dn[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool in = i < end;
            const uint64_t* row = W + (in ? (size_t)r * L : 0);
            const uint64_t* below = W + (in && r < L - 1 ? (size_t)(r + 1) * L : 0);
            const int cc = in ? c : 0;
            w[k] = row[cc];
            rt[k] = row[cc == L - 1 ? 0 : cc + 1];
            dn[k] = below[cc];
            if (!in) w[k] = rt[k] = dn[k] = 0;
            i += 256;
            r += rows;
            c += cols;
            if (c >= L) {
                c -= L;
                r += 1;
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint64_t xr = w[k] ^ rt[k], xd = w[k] ^ dn[k];
            ae += (xr & kLaneFields) + (xd & kLaneFields);
            ao += ((xr >> 3) & kLaneFields) + ((xd >> 3) & kLaneFields);
            ue += w[k] & kLaneFields;
            uo += (w[k] >> 3) & kLaneFields;
            anti[0] += (uint32_t)(xr >> 60) + (uint32_t)(xd >> 60);  // field 20 = replica 0
            ups[0] += (uint32_t)(w[k] >> 60);
        }
        pending += 4;
        if (pending > 27) {
            flush_lanes(ae, ao, anti);
            flush_lanes(ue, uo, ups);
            pending = 0;
        }
    }
    flush_lanes(ae, ao, anti);
    flush_lanes(ue, uo, ups);
#pragma unroll
    for (int k = 0; k < kReplicas; ++k) {
        const uint32_t a = wave_sum_u32(anti[k]), u = wave_sum_u32(ups[k]);
        if ((threadIdx.x & 63) == 0) {
            atomicAdd(&sums[k], a);
            atomicAdd(&sums[kReplicas + k], u);
        }
    }
    __syncthreads();
    totals += (blockIdx.x % kTotalCopies) * kTotalStride;
    for (int i = threadIdx.x; i < 2 * kReplicas; i += blockDim.x) atomicAdd(&totals[i], (unsigned long long)sums[i]);
}

// totals -> E_k = 2 A_k - 2 L^2, M_k = 2 U_k - L^2; series slot `idx`
// (21 entries), moments, out_EM; totals cleared for the next observation.
__global__ void k_replica_finalize(unsigned long long* __restrict__ totals, int L, int64_t* series_E,
                                   int64_t* series_M, int64_t idx, Moments* mom, int64_t* out_EM) {
    const int k = threadIdx.x;
    if (k >= kReplicas) return;
    const int64_t n = (int64_t)L * (int64_t)L;
    int64_t bonds = 0, up = 0;
#pragma unroll
    for (int x = 0; x < kTotalCopies; ++x) {
        bonds += (int64_t)totals[x * kTotalStride + k];
        up += (int64_t)totals[x * kTotalStride + kReplicas + k];
    }
    const int64_t E = 2 * bonds - 2 * n;
    const int64_t M = 2 * up - n;
    if (series_E) series_E[idx * kReplicas + k] = E;
    if (series_M) series_M[idx * kReplicas + k] = M;
    if (mom) add_sample(mom[k], E, M);
    if (out_EM) {
        out_EM[k] = E;
        out_EM[kReplicas + k] = M;
    }
#pragma unroll
    for (int x = 0; x < kTotalCopies; ++x) {
        totals[x * kTotalStride + k] = 0;
        totals[x * kTotalStride + kReplicas + k] = 0;
    }
}

// Spins of replica k in rows r0 .. r0 + nrows - 1, row major.
__global__ void __launch_bounds__(256) k_replica_unpack(const uint64_t* __restrict__ W, int L, int k, int r0,
                                                       int nrows, uint8_t* __restrict__ out) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (uint64_t)nrows * (uint64_t)L) return;
    out[i] = (uint8_t)((W[(uint64_t)r0 * (uint64_t)L + i] >> (3 * (20 - k))) & 1u);
}

inline unsigned rgrid(uint64_t n, int block) { return (unsigned)((n + block - 1) / block); }

}  // namespace

hipError_t launch_replica_init(uint64_t* W, int L, uint64_t seed, int hot, hipStream_t s) {
    hipLaunchKernelGGL(k_replica_init, dim3(rgrid((uint64_t)L * L, 256)), dim3(256), 0, s, W, L, (uint32_t)seed,
                       (uint32_t)(seed >> 32), hot);
    return hipGetLastError();
}

hipError_t launch_replica_halfsweep(int wpt, uint64_t* W, const ReplicaArgs& a, int colour, hipStream_t s) {
    int band = 0;
    const dim3 grid = row_grid(a.L, rgrid((uint64_t)a.L / 2, kHalfSweepBlock * wpt), (size_t)a.L * 8, &band);
    const dim3 blk(kHalfSweepBlock);
    switch (wpt) {
        case 1: hipLaunchKernelGGL(k_replica_halfsweep<1>, grid, blk, 0, s, W, a, colour, band); break;
        case 2: hipLaunchKernelGGL(k_replica_halfsweep<2>, grid, blk, 0, s, W, a, colour, band); break;
        case 4: hipLaunchKernelGGL(k_replica_halfsweep<4>, grid, blk, 0, s, W, a, colour, band); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_replica_observe(const uint64_t* W, int L, unsigned long long* totals, int64_t* series_E,
                                  int64_t* series_M, int64_t idx, Moments* mom, int64_t* out_EM, hipStream_t s) {
    const uint64_t n = (uint64_t)L * (uint64_t)L;
    // about 512 workgroups (more add more counts than they save in loads: L = 4096
    // 42 us with 512, 43 with 1024), of at least eight words per thread
    const uint32_t run = (uint32_t)std::max<uint64_t>(256 * 8, (n + 512 * 256 - 1) / (512 * 256) * 256);
    const unsigned blocks = rgrid(n, run);
    hipLaunchKernelGGL(k_replica_observe, dim3(blocks), dim3(256), 0, s, W, L, run, totals);
    hipLaunchKernelGGL(k_replica_finalize, dim3(1), dim3(64), 0, s, totals, L, series_E, series_M, idx, mom, out_EM);
    return hipGetLastError();
}

hipError_t launch_replica_unpack(const uint64_t* W, int L, int k, int r0, int nrows, uint8_t* out, hipStream_t s) {
    if (r0 < 0 || nrows < 1 || r0 + nrows > L) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_replica_unpack, dim3(rgrid((uint64_t)nrows * L, 256)), dim3(256), 0, s, W, L, k, r0, nrows,
                       out);
    return hipGetLastError();
}

}  // namespace ising
