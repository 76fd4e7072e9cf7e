// Form and key splits of a bf16 forward launch, from sizes alone.  Plain C++ without a HIP header, so that a host program can go
// over the choices (tests/host/fwd_plan_check.cpp).
#pragma once
#include "lss_shape.h"

#include <math.h>

namespace lss {

// The workgroup's form -- blocks of 32 query rows x groups of wavefronts that have a part of the keys each -- and the key splits
enum FwdForm { FWD_4x1, FWD_2x2, FWD_4x2, FWD_8x1, FWD_2x4, FWD_1x4 };
struct FwdPlan { FwdForm form; int splits; };

// A launch takes about, in us,
//     start + tile_us max(walk, share) + merge
//     walk  = (longest + few) first + shared (n - 1) (average + few) all         share = (1 + shared (n - 1)) (average + few) all W / (256 n) + rest
// with W workgroups, n of them (rounded up, at most per_cu) on a compute unit at a time, `longest` and `average` the 64-key
// tiles that a workgroup's group of wavefronts walks, and the merge launch where the keys are split: 2.4 to 2.9 us and the partial results' bytes
// at 3.9 to 4.3 MB per us.
//   * walk: the longest workgroup's, which its neighbours on the compute unit slow down for as long as they are there, themselves
//     of average length (under the causal mask, in the first segments, half the longest: 40 heads of 1459 rows take 25.6 us in 128-row
//     workgroups, three to a compute unit, and were given 64-row ones, 33.3 us, with all of the longest one's time slowed down).
//   * share: a compute unit's part of all walks, and where W > 256 per_cu the rest that part-filled last rounds leave: `tail` of a workgroup's
//     time, or whole rounds where a compute unit holds one workgroup and all are about as long (`even`, d = 128).  A longer walk hides it:
//     48 heads of 1537 rows, d = 128, 54.5 us in 8x1, were given 4x2, 65 us, with the rest added to either.
//   * A wavefront none of whose rows exist only moves tiles and meets the barriers: a last query tile of which a share `a` of the
//     wavefronts has rows takes idle + (1 - idle) a per key tile; `first` is that of the launch's longest workgroup, `all` the mean.
//   * Four groups (FWD_1x4: 32 query rows, FWD_2x4: 64): a launch whose query tiles alone leave most compute units idle shortens its walks without
//     partial results and their merge.  28 heads of 226 rows behind 834 others take 12.8 us in 1x4, 14.5 in 2x2; 16 heads of 1024 rows behind
//     3072 28.6 us in 2x4, 31.3 in 4x2 and two ranges, behind 7168 49.2 in 4x2, 53.0 in 2x4, whose
//     workgroups read every K and V tile for half as many rows.  Only where all workgroups run at once, one per compute unit: 312 of 2x4 (12 heads of
//     1622 rows behind 1531) take 34.3 us, as many of 2x2 29.4.  359 launches as below: 2.4 % less time on average than without these two, the
//     choice costs 1.1 % over the best (3.6 % without them); 200 with dropout 2.7 %, 0.9 and 4.3.  3634 more that are given four groups, in every form:
//     7.2 % less time than without, 0.5 % over the best, 96 more than 3 % slower than without (at worst 47.7 us for 36.4: 2 x 16 heads of 357
//     rows, 2 KB from one row of a head to the next).
//   * Their K and V bytes count for more (`kv` below), by the fourth root of 256 / workgroups and by how unevenly the groups share the keys: what fits
//     the launch of 32 heads that is named there.  On those 3634 the exact factor hardly matters: once to twice as much of it, or all
//     tiles' bytes at 12 to 25 MB per us in its place, and the choice costs 0.48 to 0.55 % over the best.
//   * With dropout (tables of their own) a tile takes 1.5 to 2 times as long: the generator's work is in vector slots of which the
//     forward has none to spare.  FWD_4x2 at d = 64 is not built with dropout: by its figures there (5.42, 0.87, 2.18 per
//     tile) it is never the shortest, over 15 million sizes.
// Fitted to 374 launches at d = 64 and 322 with dropout, 251 and 97 at d = 128 (58 .. 4096 rows, 512 .. 50,112 keys, 2 .. 64 heads, each in every
// form with 1 .. 16 splits, a backward pass before each call: alone, a loop of forward calls runs at a higher clock and flatters forms that load
// more), so that estimates off by 1.2 % either way still choose well: the choice costs 0.5, 1.0, 0.6 and 1.1 % over the best of them on average,
// over 140 launches that were not fitted 1.5, 2.0, 1.1 and 1.1 %.
// (Fitted to others, with the neighbours' slowing over the whole longest walk and the rest added to it, 1.6, 1.2, 1.5 and 1.7 % over a part of those fitted.)
inline FwdPlan pick_fwd_plan(const SegShape &s, bool with_drop, int max_splits)
{
    // (not below K's and V's bytes at 4.4 TB/s, the fourth powers added: 32 heads of 58 rows against 25,058 keys read 205 MB,
    // 47 us from HBM, and gain nothing from more than 8 splits: 41.6 us in 2x2, whose groups walk 25 and 24 tiles, 43.1 in 2x4, 13, 13, 13 and 10,
    // or with 7 splits, 224 workgroups)
    struct Cost { FwdForm form; int rows, groups, per_cu; double start, few, tile_us, shared, tail, idle; };
    struct Table { int forms; Cost form[5]; double merge, mb_per_us; bool rounds; };
    static const Table tables[2][2] = {
        {{5, {{FWD_4x1, 128, 1, 3, 9.05, -2.38, 0.719, 0.542, 0.542, 0.399}, {FWD_2x2, 64, 2, 2, 5.02, 2.09, 0.821, 0.401, 1.135, 0.688},
              {FWD_4x2, 128, 2, 1, 5.39, 2.14, 1.078, 0.0, 0.789, 0.630}, {FWD_2x4, 64, 4, 1, 5.93, 1.89, 1.300, 0.0, 0.0, 0.807},
              {FWD_1x4, 32, 4, 1, 4.61, 1.38, 1.164, 0.0, 0.0, 1.000}},
          2.74, 3.85, false},
         {4, {{FWD_4x1, 128, 1, 3, 10.97, -0.43, 1.319, 0.683, 0.552, 0.443}, {FWD_2x2, 64, 2, 2, 4.90, 1.50, 1.512, 0.550, 0.552, 0.000},
              {FWD_2x4, 64, 4, 1, 5.33, 1.52, 2.440, 0.0, 0.0, 0.300}, {FWD_1x4, 32, 4, 1, 4.80, 1.11, 1.944, 0.0, 0.0, 1.000}},
          2.42, 4.32, false}},
        {{2, {{FWD_8x1, 256, 1, 1, 2.55, 4.36, 1.512, 0.0, 0.556, 0.563}, {FWD_4x2, 128, 2, 1, 5.97, 2.31, 1.821, 0.0, 0.489, 1.000}}, 2.85, 4.19, true},
         {2, {{FWD_8x1, 256, 1, 1, 2.55, 4.36, 2.525, 0.0, 0.556, 0.563}, {FWD_4x2, 128, 2, 1, 5.97, 2.31, 2.859, 0.0, 0.489, 1.000}}, 2.85, 4.19, true}}};
    const Table &table = tables[s.d == 128][with_drop];
    const double out_mb = (double)s.B * s.H * s.l_s * s.d * 1e-6;     // elements
    const int64_t most = s.causal && s.s0 + s.l_s < s.l_x ? s.s0 + s.l_s : (int64_t)s.l_x;
    const int tiles = (int)((most + 63) / 64);
    const double kv_us = (double)s.B * s.H * most * s.d * 4.0 / 4.4e6;
    const bool few_rows = (int64_t)((s.l_s + 63) / 64) * s.B * s.H <= 16;       // at most 16 workgroups of 64 rows
    FwdPlan best{table.form[0].form, 1};
    double best_t = 0.0;
    for (const Cost *c = table.form, *end = c + table.forms; c != end; ++c) {
        const int64_t q_tiles = (s.l_s + c->rows - 1) / c->rows, first = s.causal ? s.s0 + (s.l_s < c->rows ? s.l_s : c->rows) : (int64_t)s.l_x;
        const double mean_tiles = 0.5 * (double)((first + 63) / 64 + tiles);
        const int rest = s.l_s - (int)(q_tiles - 1) * c->rows;
        const double last = c->idle + (1.0 - c->idle) * (double)((rest + 31) / 32) * 32.0 / c->rows, all = ((double)(q_tiles - 1) + last) / (double)q_tiles;
        for (int sp = 1; sp <= max_splits; ++sp) {
            const double W = (double)(q_tiles * s.B * s.H * sp);
            if (c->groups == 4 && W > 256.0) break;                 // (see above)
            if (sp > 1 && tiles / (sp * c->groups) < 2) break;      // shorter ones cost more than they gain
            // At most 16 workgroups for eight tiles and more: split in any case, as these launches always were and as the
            // tests of the merge's rounding expect of them.  It costs them 0 to 1.5 us (4 heads of 256 rows behind 256: 9.7
            // instead of 8.3) and 0.1 % over all those launches.
            if (sp == 1 && max_splits > 1 && W <= 16.0 && tiles >= 8) continue;
            if (c->groups == 4 && (W <= 16.0 || (few_rows && tiles >= 8))) continue;      // (nor do those few change their form)
            const double longest = (double)(((tiles + sp - 1) / sp + c->groups - 1) / c->groups);
            const double average = mean_tiles / (sp * c->groups) + (sp * c->groups > 1 ? 0.5 : 0.0);
            const double rounds = ceil(W / 256.0), n = rounds < c->per_cu ? rounds : (double)c->per_cu;
            const double shared = c->shared * (n - 1.0), mean = (average + c->few) * all, longest_walk = (longest + c->few) * (q_tiles == 1 ? last : 1.0);
            double share = (1.0 + shared) * mean * W / (256.0 * n);
            if (W > 256.0 * c->per_cu) {
                const double even = !table.rounds || c->per_cu > 1 || first < 0.6 * most ? 0.0 : ((double)first / (double)most - 0.6) / 0.4;
                share += ((1.0 - even) * c->tail + even * (rounds - W / 256.0)) * mean;
            }
            const double walk = longest_walk + shared * (mean < longest_walk ? mean : longest_walk);
            double t = c->start + c->tile_us * (walk > share ? walk : share);
            // (four groups that do not all have a tile at the end, or not on every compute unit, read less at once)
            const double kv = kv_us * (c->groups == 4 ? sqrt(sqrt(256.0 / W)) * (longest * 4.0 * sp / (double)tiles) : 1.0);
            const double merge = sp > 1 ? table.merge + out_mb * (8 * sp + 2) / table.mb_per_us : 0.0;
            if (best_t > 0.0 && (t > kv ? t : kv) + merge >= best_t) continue;      // (spares most estimates the two roots)
            t = sqrt(sqrt(t * t * t * t + kv * kv * kv * kv)) + merge;
            if (best_t == 0.0 || t < best_t) { best_t = t; best = {c->form, sp}; }
        }
    }
    return best;
}

} // namespace lss
