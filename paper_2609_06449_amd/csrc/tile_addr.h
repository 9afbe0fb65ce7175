// Geometry and address maps of the tiles that the direct form and the batched
// kernel run (tile.h): the stage plan, the splits of N, tile widths, the places in
// the LDS exchange buffer, and which item of which buffer a pass loads or stores.
// The kernels compute with these functions, and a host audit
// (tests/audit/tile_audit.cpp) enumerates the same functions over every launch,
// workgroup, thread and item.  Plain C++ (no HIP header), as addr.h.
#pragma once

#include "addr.h"

namespace paco {

// ---------------------------------------------------------------------------
// Stage plan of an on-chip transform of length n = 2^l: radix-16 Stockham
// stages, then one radix-2^(l mod 4) stage when l is not a multiple of 4.
// ---------------------------------------------------------------------------
PACO_HD constexpr int stage_count(int l) { return l / 4 + (l % 4 ? 1 : 0); }
PACO_HD constexpr int stage_log2radix(int l, int s) { return s < l / 4 ? 4 : l % 4; }
PACO_HD constexpr int stage_log2ns(int l, int s)
{
    int a = 0;
    for (int i = 0; i < s; ++i) a += stage_log2radix(l, i);
    return a;
}

// Stage twiddles w_M^{-k r} (M = Ns*R, k < Ns, 1 <= r < R) are stored as two
// factor tables per stage S >= 1, indexed (r-1, .):
//   lo[r-1][kl] = w_M^{-kl*r},       kl < min(Ns, 16)
//   hi[r-1][kh] = w_M^{-16*kh*r},    kh < Ns/16        (only when Ns > 16)
// with k = 16*kh + kl, so w_M^{-k r} = hi * lo.  Lanes of a wave hold
// consecutive k, so every table read is a broadcast or a contiguous run.
PACO_HD constexpr int stage_lo_width(int l, int s)
{
    return (1 << stage_log2ns(l, s)) < 16 ? (1 << stage_log2ns(l, s)) : 16;
}
PACO_HD constexpr int stage_hi_width(int l, int s)
{
    return (1 << stage_log2ns(l, s)) > 16 ? (1 << stage_log2ns(l, s)) / 16 : 0;
}
PACO_HD constexpr int stage_tw_size(int l, int s)
{
    return s == 0 ? 0 : ((1 << stage_log2radix(l, s)) - 1) * (stage_lo_width(l, s) + stage_hi_width(l, s));
}
PACO_HD constexpr int stage_tw_offset(int l, int s)
{
    int a = 0;
    for (int i = 1; i < s; ++i) a += stage_tw_size(l, i);
    return a;
}
PACO_HD constexpr int stage_tw_total(int l) { return stage_tw_offset(l, stage_count(l)); }

// Row of the first output of butterfly j of the stage after 2^lns points, radix
// 2^lr (output r lies r 2^lns rows on).
template <int LNS, int LR>
PACO_HD int stage_dest(int j)
{
    return ((j >> LNS) << (LNS + LR)) + (j & ((1 << LNS) - 1));
}

// LDS index with 4 pad items per 64: the radix-16 first-stage writes (row
// stride 16*T items) land on distinct banks.
PACO_HD constexpr int lpad(int e) { return e + ((e >> 6) << 2); }

// ---- splits of N ----------------------------------------------------------------

constexpr int kDirectChipLog2 = 14;  // the largest transform of one workgroup
constexpr int kDirectMaxLog2 = 23;
constexpr int kBatchPassMax = 10;    // pass lengths of the batched kernel: up to 2^10
// The splits of N = 2^15 .. 2^20 that the batched form's tuner chooses from.
// Passes of 2^8 .. 2^10 points, 2^7 only at 2^15, where every split has one: a
// single plan's 4-column tile of 128 points is half a wave.  us per call as
// balanced / as N1 x N2: 256 x 1024 10.6 / 10.5, 1024 x 256 10.6 / 10.7, 512 x 1024 12.6 /
// 12.0, 128 x 256 8.8 / 8.9, all within a run's noise; but 512 x 128 8.8 / 9.0 and
// 1024 x 128 9.0 / 9.9, for which a large batch gave nothing back (512 of 2^17
// 384 / 386 us, 1024 of 2^16 374 / 369).
PACO_HD constexpr bool batch_split(int l1, int l2)
{
    return l1 + l2 > kDirectChipLog2 && l1 <= kBatchPassMax && l2 <= kBatchPassMax &&
           ((l1 >= 8 && l2 >= 8) || (l1 + l2 == 15 && l1 >= 7 && l2 >= 7));
}
// log2 of pass A's points in a plan of N1 x N2 = 2^l1 x 2^l2 (N > 2^kDirectChipLog2)
PACO_HD constexpr int direct_l1(int l1, int l2) { return batch_split(l1, l2) ? l1 : (l1 + l2 + 1) / 2; }

// ---- tiles -------------------------------------------------------------------

PACO_HD constexpr int tile_items(int l) { return l < 4 ? 1 << l : 16; }
// threads of a tile of 2^lt columns in h groups
PACO_HD constexpr int tile_threads(int l, int lt, int h) { return (1 << (l + lt)) / (h * tile_items(l)); }
PACO_HD constexpr int tile_tw(int l) { return (stage_tw_total(l) + 31) & ~31; }
// items of LDS: the stage twiddles and one group's exchange buffer with its
// padding (one item per 16 in both orders; transforms of at most 16 points
// exchange nothing)
PACO_HD constexpr int tile_lds(int l, int lt, int h)
{
    const int g = (1 << (l + lt)) / h;
    return tile_tw(l) + (l > 4 || lt > 0 ? g + (g >> 4) + 4 : 4);
}

// Place of (row, column t) in the exchange buffer.  Column fastest: lpad.
// Index fastest: one pad item per 16, which puts the stride-16 stores of a
// radix-16 stage on distinct banks.
template <int L, int LTG, bool JF>
PACO_HD int tile_slot(int row, int t)
{
    if constexpr (JF) {
        const int i = (t << L) + row;
        return i + (i >> 4);
    } else {
        return lpad((row << LTG) + t);
    }
}
template <int LTG, int LJ, bool JF>
PACO_HD int tile_col(int g)
{
    return JF ? g >> LJ : g & ((1 << LTG) - 1);
}
template <int LTG, int LJ, bool JF>
PACO_HD int tile_idx(int g)
{
    return JF ? g & ((1 << LJ) - 1) : g >> LTG;
}

// ---- tile widths -----------------------------------------------------------------

// The direct form's passes (direct_kernels.h).
// Tiles of 4 columns: 32-byte runs of x and of y, which the tiles beside it on
// the same XCD (tile_order) complete to lines in its L2.  What bounds a pass
// here is its launch and one chain of load, arithmetic, store per workgroup,
// so the most workgroups win: 4 columns against 8 in both passes took 11.2
// against 12.1 us at 2^16, 15.6 against 17.0 at 2^20, 34.0 against 39.4 at
// 2^22 (whole calls, back to back, of that trial; 14.7 and 32 us now).  The two
// kernels of 2^20 take 7.6 and 8.2 us in a trace, of 2^22 15.7 and 17.2.
// 4096-point columns (pass A of 2^23 only): 8 columns in two LDS groups, 1024
// threads and 136 KiB, whose 64-byte runs are read last-use (pass_a_tile).
// 2^23: 72 us, with 4 columns and two workgroups per CU 79; the three-pass forms
// it replaces took 95 to 130 by shape.  2^24 in two passes of 4 columns took 191
// us against 162 (now 132) for the symmetric form's three, which ends the range.
PACO_HD constexpr int tile_groups(int l) { return l == 12 ? 2 : 1; }
// (the split MFMA forms' butterflies need full waves: 8 columns of 128 points)
PACO_HD constexpr int tile_cols(int l, bool mfma) { return l == 12 || (mfma && l == 7) ? 3 : 2; }

// The batched kernel (batch.hip).

// Columns (log2) of a pass tile of 2^l points.  The shared queue serves few
// large transforms, which a full tile leaves on too few workgroups: half a
// tile there, 16 items per thread in one group (one transform of 2^16 32 -> 22
// us, of 2^20 35 -> 30, nine of 2^20 117 -> 95).
constexpr int kTileLog2 = 14;  // items of a pass tile: 32 per thread, in two groups
PACO_HD constexpr int pass_lt(int l, bool coh) { return (coh ? kTileLog2 - 1 : kTileLog2) - l; }
// transforms of 2^l points a small task of 2^lw threads holds: 16 items per
// thread (shorter ones: one transform per thread)
PACO_HD constexpr int small_lt(int l, int lw) { return l < 4 ? lw : lw + 4 - l; }

// ---- the two column passes: items of x, ws and y -------------------------------
// pass A: 2^l2 columns; stored blocked by 2^lb columns of pass B.  Loads and
// pass B's accesses are from the tile's first column (pass B's loads: the
// contiguous piece of ws from item col0 2^L on).
namespace addr {

PACO_HD uint32_t pass_a_load(uint32_t row, uint32_t col, int l2) { return (row << l2) + col; }
PACO_HD uint32_t pass_a_store(uint32_t k, uint32_t col, int l2, int lb)
{
    return ((k >> lb) << (l2 + lb)) + (col << lb) + (k & ((1u << lb) - 1u));
}
PACO_HD uint32_t pass_b_load(uint32_t row, uint32_t col, int lt) { return (row << lt) + col; }
PACO_HD uint32_t pass_b_store(uint32_t row, uint32_t col, int l1) { return (row << l1) + col; }
// entry of the table w_{16 M1}^{-k}, k < 16 M1 = 2^(l1 + 4)
PACO_HD uint32_t pass_b_cw(uint32_t col, uint32_t r, int l1) { return (col * r) & ((16u << l1) - 1u); }
// exponent e of w_N^{-e}, N = 2^log2N
PACO_HD uint32_t pass_b_top(uint32_t col, uint32_t row, int log2N)
{
    return (col * row) & uint32_t((uint64_t(1) << log2N) - 1);
}

}  // namespace addr
}  // namespace paco
