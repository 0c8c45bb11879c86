// Host-side helpers shared by the C-ABI translation units: thread-local
// error messages, HIP error mapping, argument checks, pinned staging.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdarg>
#include <cstdio>
#include <string>
#include <vector>

#include "../../include/ising.h"
#include "ising_common.hpp"

namespace ising {

// The device-side moment sums are handed out as ising_moments unchanged.
static_assert(sizeof(Moments) == sizeof(ising_moments), "Moments layout");
static_assert(offsetof(Moments, sum_E2) == offsetof(ising_moments, sum_E2), "Moments layout");
static_assert(offsetof(Moments, sum_absM) == offsetof(ising_moments, sum_absM), "Moments layout");
static_assert(offsetof(Moments, sum_M4) == offsetof(ising_moments, sum_M4), "Moments layout");

std::string& last_error_ref();

inline int fail(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    last_error_ref() = buf;
    return code;
}

inline int hip_fail(hipError_t e, const char* what) {
    return fail(ISING_EHIP, "%s failed: %s", what, hipGetErrorString(e));
}

#define ISING_HIP(call)                                      \
    do {                                                     \
        hipError_t ising_e_ = (call);                        \
        if (ising_e_ != hipSuccess) return ::ising::hip_fail(ising_e_, #call); \
    } while (0)

inline bool valid_L(int32_t L) { return L >= 4 && L <= kMaxL && (L % 2) == 0; }
inline bool valid_T(double T) { return std::isfinite(T) && T > 0.0; }

// floor(exp(x) 2^32) clamped to [0, 2^32 - 1], in IEEE double with the C
// library exp (the acceptance probability exp(-dE/kT) of Section 2, step 3,
// as an integer threshold for 32-bit uniforms).
inline uint32_t threshold_from_exponent(double x) {
    const double v = std::floor(std::exp(x) * 4294967296.0);
    if (v >= 4294967295.0) return 4294967295u;
    if (v <= 0.0) return 0u;
    return (uint32_t)v;
}

inline void thresholds_of(double T, uint32_t* t4, uint32_t* t8) {
    *t4 = threshold_from_exponent(-4.0 / T);
    *t8 = threshold_from_exponent(-8.0 / T);
}

inline bool valid_block(int b, int max_block) { return b >= 64 && b <= max_block && b % 64 == 0; }

// Spin input/output goes through a byte staging buffer in device memory that
// a handle allocates once, at creation: the whole L x L lattice when it is
// small, else 16 MiB, moved in pieces of whole rows.  No call that reads or
// writes spins allocates or frees device memory.
constexpr size_t kSpinStageMax = size_t(16) << 20;
inline size_t spin_stage_bytes(int32_t L) { return std::min((size_t)L * (size_t)L, kSpinStageMax); }

// The nrows x ncols window with top-left site (r0, c0), indices mod L, into
// host bytes (row major, 1 = up), staged through `stage` (cap bytes >= ncols);
// synchronises the stream.
int read_spin_window(const uint64_t* W, const Geometry& g, int32_t r0, int32_t c0, int32_t nrows, int32_t ncols,
                     uint8_t* host, uint8_t* stage, size_t cap, hipStream_t s);
// Replace every spin by the host bytes (L x L, nonzero = up), staged through
// `stage` (cap bytes >= L); synchronises the stream.
int write_spins(uint64_t* W, const Geometry& g, const uint8_t* host, uint8_t* stage, size_t cap, hipStream_t s);

// Resident tiles of a lattice of up to 7680 columns: up to L = 192 the whole
// lattice in one workgroup, a thread per word of a colour (a power of two, 64 to
// 1024); below L = 1024 bands of 8 columns, 512 threads; from there bands of
// 2 ceil(L / 512) columns (at most 256, one per compute unit), 1024 threads.
inline void default_resident_shape(const Geometry& g, int32_t* w, int32_t* block) {
    *w = 2 * ((g.L + 511) / 512);
    *block = 1024;
    if (g.L <= 192) {
        const int64_t items = (int64_t)g.N * g.L / 2;
        *w = g.L;
        *block = 64;
        while (*block < 1024 && *block < items) *block *= 2;
    } else if (g.L < 1024) {
        *w = 8;
        *block = 512;
    }
}

// The resident tiles of one lattice (interior width w, the last one
// narrower), indexed by workgroup: consecutive workgroups are dealt to the
// 8 XCDs in turn, so when the tile count is a multiple of 8 tile t goes to
// workgroup 8 (t mod m) + t div m (m = count / 8) and every XCD holds a run
// of neighbouring tiles, which then trade their boundary words inside one
// XCD except at the ends of the runs.  part_base offsets the partial slots.
inline std::vector<PersistTile> resident_tile_table(int32_t lattice, int32_t L, int32_t w, int32_t part_base) {
    int32_t n = 0;
    for (int32_t c0 = 0; c0 < L; c0 += w) ++n;
    const bool spread = n % 8 == 0;
    const int32_t m = n / 8;
    auto block_of = [&](int32_t t) { return spread ? 8 * (t % m) + t / m : t; };
    std::vector<PersistTile> tiles(n);
    for (int32_t t = 0; t < n; ++t) {
        const int32_t c0 = t * w;
        tiles[block_of(t)] = {lattice, c0, std::min(w, L - c0), block_of((t + n - 1) % n), block_of((t + 1) % n),
                              part_base + t};
    }
    return tiles;
}

}  // namespace ising
