// The update of a run of same-colour words of one row of a word lattice in
// global memory by one wavefront: the body of the half-sweep kernels (one
// lattice, many lattices, 21 replicas).
//
// Lane l of the wavefront updates the words w0 + 64 k + l, k < WPT, of the
// row's words of the colour (word w lies in column 2 w + par).  Neighbouring
// lanes hold neighbouring words, so every load of a run covers one
// contiguous stretch of memory (a wavefront whose lanes each hold WPT
// neighbouring words instead spreads every load over WPT times as many cache
// lines, and with four words per thread waits for the cache: L = 32768 290 us
// per half-sweep).  The rows are wave-uniform base addresses
// and the lane adds one 32-bit offset, so that the neighbourhoods need no
// address arithmetic.  The Philox blocks that serve position 20 (one per
// eight-column group, four words of the colour) are drawn for all the runs
// at once, one per lane, and passed through LDS: output m of group g is word
// 4 g + m, so the table is indexed by the word and each block is drawn once.
//
// Bound by the vector unit: 13.7 vector instructions per site (a quarter of
// them Philox's products), issued on practically every fourth cycle, which is
// what one costs in this mix.  L = 32768: 190 us per half-sweep, 2820
// spin-flip attempts/ns; 229 us with 16.6 instructions per site, when lanes
// held neighbouring words, formed 64-bit addresses and chose the fix-ups of
// the wrap rows by selects.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "ising_device.hpp"

namespace ising {

// Which row and which part of it a workgroup takes.  Consecutive workgroups go
// to the 8 XCDs in turn, each with an L2 of its own, and a word is read three
// times in a half-sweep (as a word of its row, from the row above and from
// the row below).  With `band` > 0 the grid is (8, workgroups per row, band):
// XCD x gets the rows [x band, (x + 1) band) in order, so that two of the
// three reads find the word in its L2, whatever the row length; otherwise
// the grid is (workgroups per row, rows), where that holds only if the number
// of workgroups per row is a multiple of 8.
struct RowBlock {
    int row, x;
};
__device__ __forceinline__ RowBlock row_block(int band) {
    if (band > 0) return {(int)blockIdx.x * band + (int)blockIdx.z, (int)blockIdx.y};
    return {(int)blockIdx.y, (int)blockIdx.x};
}

// Words of the position-20 table of one wavefront (the kernel's tables start at a
// multiple of 16 bytes: a block is stored whole).
template <int WPT>
constexpr int row_table_words() {
    return 64 * WPT;
}

// The wave-uniform part of a run: the row's words, the rows above and below,
// the row of the patch word (read only where `wraps`), the row length in
// columns and words of a colour, the parity of the colour's columns, the
// Philox counter words of column 0 and the key.
struct RowRun {
    uint64_t* row;
    const uint64_t* up;
    const uint64_t* dn;
    const uint64_t* patch;
    bool wraps;
    int L, par;
    uint32_t row_base, t_lo, t_hi, c3, k0, k1;
    bool last_block;  // position 20 is drawn
};

using GlobalByte = __attribute__((address_space(1))) char;

// Rule(run of one word) supplies the rest: rule.accept(acc, block) adds (to a
// Rule::Accept) the
// acceptance bits of positions 0..19 (block(g) draws block g),
// rule.accept20(acc, u) those of position 20, rule.vertical(up, dn, patch)
// finishes the vertical neighbours of a row that wraps, rule.live is the
// live-slot mask, and rule.after(new word, up, dn, left, right) sees every
// updated word.
template <int WPT, class Rule>
__device__ __forceinline__ void update_row_words(const RowRun& r, int w0, uint32_t* __restrict__ table, Rule&& rule) {
    using Byte = GlobalByte;
    using Word = __attribute__((address_space(1))) uint64_t;
    const int lane = (int)(threadIdx.x & 63u);
    const int half = r.L >> 1;
    const RoundKeys rk = round_keys(r.k0, r.k1);
    Byte* const row = (Byte*)r.row;

    if (r.last_block) {
        if (WPT == 4 || lane < 16 * WPT) {
            const U4 b = philox_lane_c1(r.t_lo, r.row_base + (uint32_t)(2 * w0 + r.par) + 8u * (uint32_t)lane, r.t_hi,
                                        5u | r.c3, r.k0, r.k1, rk);
            *reinterpret_cast<uint4*>(table + 4 * lane) = make_uint4(b.x, b.y, b.z, b.w);
        }
        wave_lds_order();
    }

#pragma unroll 1
    for (int k = 0; k < WPT; ++k) {
        const int wk = w0 + 64 * k;  // the run's first word
        if (wk + lane < half) {
            // the lane's byte offset in a row, kept opaque so that every
            // access takes it as it is beside the row's scalar base (grouped
            // otherwise, each becomes a 64-bit vector addition)
            const int J = 2 * (wk + lane) + r.par;
            uint32_t o = (uint32_t)J << 3;
            asm("" : "+v"(o));
            uint32_t o_lf = o - 8u, o_rt = o + 8u;
            if (r.par == 0 ? wk == 0 : wk + 64 >= half) {  // the run holds the row's first / last column
                o_lf = J == 0 ? (uint32_t)(r.L - 1) << 3 : o_lf;
                o_rt = J == r.L - 1 ? 0u : o_rt;
            }
            const uint64_t w = *(const Word*)(row + o), lf = *(const Word*)(row + o_lf), rt = *(const Word*)(row + o_rt);
            uint64_t up = *(const Word*)((const Byte*)r.up + o), dn = *(const Word*)((const Byte*)r.dn + o), patch = 0;
            if (r.wraps) patch = *(const Word*)((const Byte*)r.patch + o);
            const uint32_t u20 = r.last_block ? table[64 * k + lane] : 0u;

            const uint32_t c1 = r.row_base + (uint32_t)J;
            typename std::remove_reference_t<Rule>::Accept acc;
            rule.accept(acc, [&](int g) {
                return philox_lane_c1(r.t_lo, c1, r.t_hi, (uint32_t)g | r.c3, r.k0, r.k1, rk);
            });
            rule.accept20(acc, u20);
            if (r.wraps) rule.vertical(up, dn, patch);
            const uint64_t nw = w ^ flip_mask(w, up, dn, lf, rt, acc.a(), acc.b(), rule.live);
            *(Word*)(row + o) = nw;
            rule.after(nw, up, dn, lf, rt);
        }
    }
}

// The grid for `rows` rows of per_row workgroups, and its band: bands of
// rows per XCD where that leaves the XCDs evenly filled (at least 32 rows
// each) and three rows fit in an L2 of 4 MB beside the rest (rows of up to
// 512 KB).  With rows dealt to the XCDs in turn
// instead, a half-sweep of L = 9998 took 34 us (26 to 36 by launch shape; 24
// in bands), 13000 52 (34), 26000 170 (113).
inline dim3 row_grid(int rows, unsigned per_row, size_t row_bytes, int* band) {
    *band = rows >= 256 && row_bytes <= (size_t(512) << 10) ? (rows + 7) / 8 : 0;
    return *band ? dim3(8, per_row, (unsigned)*band) : dim3(per_row, (unsigned)rows);
}

}  // namespace ising
