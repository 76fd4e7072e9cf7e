// How a backward launch is laid out, from sizes alone: the bf16 rules.  Plain C++ without a HIP header, so that a host program can go over
// the choices (tests/host/plan_check.cpp).
#pragma once
#include "lss_shape.h"

#include <math.h>

namespace lss {

constexpr int kSkinnyRows = 64;     // a segment of so many rows is one tile
constexpr int kOwnRows = 512;       // rows whose start values fit the LDS of a workgroup that computes them itself

// (a^6 + b^6)^(1/6): the larger of two times, and a little more where they are close.  Without pow, of which each of a
// call's up to 32 estimates took three (with that, and what they share computed per estimate, 2.6 us of host time; now 1.6).
inline double larger_or_both(double a, double b)
{
    const double hi = a > b ? a : b, r = (a > b ? b : a) / hi, r3 = r * r * r;
    return hi * cbrt(sqrt(1.0 + r3 * r3));
}

// Whether the workgroups compute D and the start values themselves (never where a gradient overlaps `out`, see
// launch_bwd_d): a launch less (2.3 us), for each dK/dV workgroup
// 0.75 us per 128 rows of 64 elements or 1.5 us per 64 of 128 ahead of its loop.  That is spread over the rounds of
// workgroups the chip takes (512 or 256 at once); a launch of one round or less pays it in full only if a dK/dV
// workgroup's walk over the queries, and not a dQ workgroup's over its keys, is what the launch waits for.
// 4 heads of 256 queries against 512 keys: backward 14.4 us with the preprocess kernel, 12.3 without; 10 x 4 heads of 67
// against 47,600: 450 and 469.  680 launches of 66 .. 4096 rows at d = 64, every split count and form: 0.4 % over the better one.
inline bool bwd_own_values(const SegShape &s, int n_splits, int groups)
{
    if (s.l_s <= kSkinnyRows) return true;      // one tile: loaded once per workgroup in any case
    if (s.l_s > kOwnRows) return false;
    const double chunk_us = s.d == 64 ? 0.75 : 1.5, row_tile_us = s.d == 64 ? 1.35 : 1.9, key_tile_us = s.d == 64 ? 1.0 : 1.4;
    const int chunk_rows = s.d == 64 ? 128 : 64, at_once = s.d == 64 ? 512 : 256;
    const int64_t seen = s.causal ? (s.s0 + s.l_s < s.l_x ? s.s0 + s.l_s : (int64_t)s.l_x) : (int64_t)s.l_x;
    const double own_us = chunk_us * ((s.l_s + chunk_rows - 1) / chunk_rows);
    const double walk_us = row_tile_us * ((s.l_s + 63) / 64) / groups, dq_us = key_tile_us * (double)((seen + 63) / 64) / (n_splits * groups);
    double rounds = (double)((seen + 127) / 128 * s.B * s.H) / at_once;
    if (rounds < 1.0 && dq_us < walk_us + own_us) rounds = 1.0;
    return own_us * rounds <= 2.0;
}

// bf16, d = 64, more than 64 rows: key splits of the dQ workgroups, and whether a workgroup is one or two groups of wavefronts
// (bwd_main_bf16_kernel).  A launch takes about, in us,
//     start + (longest^6 + balance^6)^(1/6) + zeros / 9 MB + merge
// longest: the longer of a dQ workgroup's walk over its 64-key tiles and a dK/dV workgroup's over the 64-row query tiles, each a few
// tiles more, the latter slower as two workgroups come to share a compute unit; balance: all walks over 256 compute units, and a part of a last
// dK/dV walk where the launch takes more than one round; zeros: the rows no query sees; merge: 1.8 us and the partial dQ's
// bytes at 11 MB per us where there is more than one split.  Fitted to 100 launches (65 .. 4096 rows, 512 .. 50,112 keys, 2 .. 64 heads, both forms
// with 1 .. 16 splits, after a forward call each): launches take 4.9 % less time
// than with one group and splits that only keep a dQ workgroup from outlasting the launch (8 heads of 1044 rows against 26,100 keys: 214 us, four splits
// 192; 4 heads of 3510 rows behind 1226: 83 us, in two groups 55; 2 heads of 1362 rows: 32 and 27).  The starts and what is saved where no
// preprocess launch is made are fitted to 680 more, each form with and without that launch: the choice costs
// 2.2 % over the best of them on average (2.3 % with the saving taken for one group and all segments of up to 512 rows, whether
// bwd_own_values says so or not; eleven launches 3 to 8 % slower then, two faster: 15 heads of 365 rows against 1873 keys 25.5 us and now 23.8).
// Two groups gain nothing over their preprocess launch (a start of 4.0 with 0.4 saved fitted those launches as well, but gave 13 heads of
// 1291 rows and 20 of 1363 to one group: 33 -> 37 and 42 -> 46 us).
// With dropout a tile takes longer, most in two groups, and splits pay sooner: starts and tile times fitted to 193 launches of their own, in
// every form; the choice costs 1.9 % over the best of them on average, with half of them fitted 2.3 % over the other half, and 3.6 % by the figures
// without dropout (6 heads of 1034 rows against 2121 keys: 53.4 us, in two ranges 40.6; 14 of 152 behind 401: 23.4 and 19.4).
struct BwdPlan { int splits, groups; };

// What all estimates of a launch share
struct BwdWork {
    int64_t tiles, q_tiles;                                       // 64-key tiles that some row sees, 64-row query tiles
    double n_dq, n_dkv, dq_walks, dkv_walks, zeros_us, dq_mb;      // workgroups (dQ: per split) and the tiles they walk
};
inline BwdWork bwd_work(const SegShape &s)
{
    const double bhs = (double)s.B * s.H;
    const int64_t seen = s.causal && s.s0 + s.l_s < s.l_x ? s.s0 + s.l_s : (int64_t)s.l_x, first = s.causal ? s.s0 + (s.l_s < 128 ? s.l_s : 128) : (int64_t)s.l_x;
    const int64_t tiles = (seen + 63) / 64, q_tiles = (s.l_s + 63) / 64, dq_tiles = (s.l_s + 127) / 128, key_tiles = (seen + 127) / 128;
    const int64_t full = s.causal && s.s0 / 128 < key_tiles ? s.s0 / 128 : key_tiles;      // key tiles that all rows see; the others half of them
    const double mean_tiles = 0.5 * (double)((first + 63) / 64 + tiles);
    return {tiles, q_tiles, (double)dq_tiles * bhs, (double)key_tiles * bhs, (double)dq_tiles * bhs * mean_tiles,
            bhs * ((double)full + 0.5 * (double)(key_tiles - full)) * (double)q_tiles, (double)(s.l_x - seen) * bhs * s.d * 8e-6 / 9.0,
            bhs * s.l_s * s.d * 1e-6};
}

// The estimate for one form and split count; `own`: no preprocess launch (bwd_own_values), which the start counts
inline double bwd_estimate(const BwdWork &w, int splits, int groups, bool own, bool with_drop)
{
    struct Cost { double start, own, dq_us, dq_more, dkv_us, dkv_more, dkv_slow, rate, last; };
    static const Cost forms[2][2] = {{{5.8, 1.6, 0.70, 1.7, 1.02, 3.7, 0.35, 0.85, 0.31}, {3.4, 0.0, 1.11, 2.6, 1.52, 4.6, 0.0, 1.06, 0.51}},
                                     {{17.7, 2.1, 0.919, 1.7, 1.229, 3.7, 0.35, 0.85, 0.31}, {9.4, 0.43, 1.693, 2.6, 1.879, 4.6, 0.0, 1.06, 0.51}}};
    const Cost &c = forms[with_drop][groups - 1];
    const double n_dq = w.n_dq * splits, N = n_dq + w.n_dkv, per_group = groups == 1 ? 1.0 : 0.5;
    const double shared = N < 256.0 ? 0.0 : N > 512.0 ? 1.0 : N / 256.0 - 1.0;
    const double dq = ((double)((((int)w.tiles + splits - 1) / splits + groups - 1) / groups) + c.dq_more + 1.0) * c.dq_us;
    const double dkv = ((double)((w.q_tiles + groups - 1) / groups) + c.dkv_more) * c.dkv_us * (1.0 + c.dkv_slow * shared);
    double balance = c.rate / 256.0 * ((w.dq_walks * per_group + n_dq * c.dq_more) * c.dq_us +
                                       (w.dkv_walks * per_group + w.n_dkv * c.dkv_more) * c.dkv_us);
    if (N > 512.0 * per_group) balance += c.last * dkv;
    const double t = c.start - (own ? c.own : 0.0) + larger_or_both(dq > dkv ? dq : dkv, balance) + w.zeros_us;
    return splits > 1 ? t + 1.8 + w.dq_mb * (4 * splits + 2) / 11.0 : t;
}

// `may_own`: bwd_own_values decides (no gradient overlaps `out`)
inline BwdPlan pick_bwd_plan(const SegShape &s, bool with_drop, int most, bool may_own)
{
    const BwdWork w = bwd_work(s);
    BwdPlan best{1, 1};
    double best_t = 0.0;
    for (int groups = 1; groups <= (s.l_s > 128 ? 2 : 1); ++groups)      // (two tiles of rows: nothing to share)
        for (int splits = 1; splits <= most; ++splits) {
            if (splits > 1 && w.tiles < 4 * splits) break;
            const double t = bwd_estimate(w, splits, groups, may_own && bwd_own_values(s, splits, groups), with_drop);
            if (best_t == 0.0 || t < best_t) { best_t = t; best = {splits, groups}; }
        }
    return best;
}

// Whether a launch takes eight wavefronts of 16 rows per workgroup (NJ = 1).  At d = 128 where no compute unit gets more than 32 walks of 64 query
// rows past 128 keys.  Longer ones are held by the chip's power, of which twice the LDS reads take more: with NJ = 1 a 32k segment's
// compute units are busy 12 % fewer cycles, but at a lower clock, 2.40 ms instead of 2.36.  50 launches, forward and backward:
// those of 24 walks and less 0 to 12 % faster, 4.3 % on average (8 heads of 770 rows behind 1654: 82 -> 72 us, 4 of 813: 52 -> 49); above, 2 %
// slower on average.
// At d = 64 where every compute unit gets at most one workgroup of one group, rows that no query sees aside: wavefronts that are
// alone on their SIMD wait for their own chains, which are half as long with 16 rows, and the LDS has time for twice the reads (4 heads of 256
// rows behind 768: 15.6 us, 14.2).  But not with
//   * more than 32 workgroups of either kind on an XCD, which waits for the one that comes last: with 252 to 256 of them and 33 on some
//     XCD 7 % more time on average, at worst 20 % (15 heads of 374 rows against 1351: 26.4 us, 30.4), with 32 on each 3.6 % less;
//   * many tiles to clear: a compute unit holds one workgroup of this form and two of the other, beside which they are cleared from the start; here the
//     idle ones have to clear them in the others' time, some 1.8 us a tile -- and the others a few of them at the end, which 32 idle ones stand for
//     (6 heads of 339 rows behind 3069 of 34,850, 1470 tiles on four idle units: 24.6 us, 31.7; 24 of 123 behind 103 of 3718, 648 on 184: 17.1, 15.3).
// 11,200 launches of 65 .. 4096 rows that pass the first line, in either form: 5 % less time than the wider one, 0.1 % over the better one (0.6 % without
// the second line; a walk with dropout taken for as long as one without, 0.24 % over the better one in those).
inline bool bwd_narrow(const SegShape &s, int n_splits, int groups, bool with_drop)
{
    const int64_t seen = s.causal && s.s0 + s.l_s < s.l_x ? s.s0 + s.l_s : (int64_t)s.l_x, bhs = (int64_t)s.B * s.H;
    const int64_t dkv = (seen + 127) / 128 * bhs, dq = (int64_t)((s.l_s + 127) / 128) * bhs * n_splits;
    if (s.d != 64) return dkv * ((s.l_s + 63) / 64) <= 32 * 256;
    if (s.l_s <= kSkinnyRows || groups != 1 || (dq + 7) / 8 + (dkv + 7) / 8 > 32) return false;
    const int64_t zeros = s.skip_tail ? 0 : (s.l_x - seen) / 128 * bhs;
    const double row_us = 1.35 * (double)((s.l_s + 63) / 64), key_us = (double)(((seen + 63) / 64 + n_splits - 1) / n_splits);
    const double walk_us = (row_us > key_us ? row_us : key_us) * (with_drop ? 2.0 : 1.0) + 4.0;
    return (double)zeros * 1.8 <= walk_us * (double)(dq + dkv < 224 ? 256 - dq - dkv : 32);
}

// A whole backward launch.  one_pass: the kernel that makes all three gradients of a short segment (bf16, d = 64); own: no
// preprocess launch; skinny: dK/dV workgroups for at most 64 rows; narrow: wavefronts of 16 rows (all three: bf16, else false)
struct BwdLaunch { int splits, groups; bool one_pass, own, skinny, narrow; };

} // namespace lss
