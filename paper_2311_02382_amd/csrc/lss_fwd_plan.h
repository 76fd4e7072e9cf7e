// Form and key splits of a bf16 forward launch, from sizes alone.  Plain C++ without a HIP header, so that a host program can go
// over the choices (tests/host/fwd_plan_check.cpp).
#pragma once
#include "lss_shape.h"

#include <math.h>

namespace lss {

// The workgroup's form -- blocks of 32 query rows x groups of wavefronts that have a part of the keys each -- and the key splits
enum FwdForm { FWD_4x1, FWD_2x2, FWD_4x2, FWD_8x1 };
struct FwdPlan { FwdForm form; int splits; };

// A launch takes about, in us,
//     start + tile_us (1 + shared (n - 1)) max((longest + few) first, (average + few) all W / (256 n)) + rest (average + few) tile_us all + merge
// with W workgroups, n of them (rounded up, at most per_cu) on a compute unit at a time, `longest` and `average` the 64-key
// tiles that a workgroup's group of wavefronts walks, the rest where W > 256 per_cu and the merge launch where the keys are
// split: about 2.5 us and the partial results' bytes at 3.4 to 5.2 MB per us.
//   * A wavefront none of whose rows exist only moves tiles and meets the barriers: a last query tile of which a share `a` of the
//     wavefronts has rows takes idle + (1 - idle) a per key tile; `first` is that of the launch's longest workgroup, `all` the mean.
//   * The rest is `tail` of a workgroup's time; where a compute unit holds one workgroup and all are about as long (`even`), the
//     launch takes whole rounds of them.
//   * With dropout (tables of their own) a tile takes 1.5 to 2 times as long: the generator's work is in vector slots of which the
//     forward has none to spare.  FWD_4x2 at d = 64 is not built with dropout: by its figures there (5.42, 0.87, 2.18 per
//     tile) it is never the shortest, over 15 million sizes.
// Fitted to 454 launches at d = 64 and 436 at 128 (58 .. 4096 rows, 512 .. 50,112 keys, 2 .. 64 heads, 45 % with dropout, each in every form with 1 .. 16
// splits, a backward pass before each call: alone, a loop of forward calls runs at a higher clock and flatters forms that load more): the
// choice costs 1.4 % over the best of them on average with dropout at d = 64, 1.1 % at d = 128 (4.7 % and 3.7 % by the figures for d = 64
// without dropout and by such ones for d = 128, with none of the three terms: 24 heads of 92 rows against 525 keys, d = 128, 11.1 us
// in 4x2, 9.1 in 8x1; 26 of 888 rows with dropout 23.2, now 16.4).  d = 64 without dropout: fitted to 145 launches of its own, without these terms
// (2.9 %; with the three terms 1.9, but a sweep of eight segments of 1024 rows, 16 heads, took 965 us instead of 949).
inline FwdPlan pick_fwd_plan(const SegShape &s, bool with_drop, int max_splits)
{
    // (not below K's and V's bytes at 4.4 TB/s, the fourth powers added: 32 heads of 58 rows against 25,058 keys read 205 MB,
    // 47 us from HBM, and gain nothing from more than 8 splits)
    struct Cost { FwdForm form; int rows, groups, per_cu; double start, few, tile_us, shared, tail, idle; };
    struct Table { int forms; Cost form[3]; double merge, mb_per_us; bool rounds; };
    static const Table tables[2][2] = {
        {{3, {{FWD_4x1, 128, 1, 3, 8.2, -3.3, 0.733, 0.51, 0.81, 1.0}, {FWD_2x2, 64, 2, 2, 4.7, 1.2, 0.799, 0.51, 0.55, 1.0}, {FWD_4x2, 128, 2, 1, 4.8, 1.7, 1.068, 0.0, 0.64, 1.0}},
          2.8, 4.5, false},
         {2, {{FWD_4x1, 128, 1, 3, 8.07, -1.43, 1.32, 0.467, 0.412, 0.623}, {FWD_2x2, 64, 2, 2, 2.11, 2.53, 1.38, 0.417, 0.447, 0.0}},
          2.03, 3.41, true}},
        {{2, {{FWD_8x1, 256, 1, 1, 3.38, 3.02, 1.50, 0.0, 0.645, 0.468}, {FWD_4x2, 128, 2, 1, 3.92, 2.36, 1.787, 0.0, 0.63, 1.0}}, 2.5, 5.2, true},
         {2, {{FWD_8x1, 256, 1, 1, 3.38, 3.02, 2.385, 0.0, 0.645, 0.468}, {FWD_4x2, 128, 2, 1, 3.92, 2.36, 2.704, 0.0, 0.63, 1.0}}, 2.5, 5.2, true}}};
    const Table &table = tables[s.d == 128][with_drop];
    const double out_mb = (double)s.B * s.H * s.l_s * s.d * 1e-6;     // elements
    const int64_t most = s.causal && s.s0 + s.l_s < s.l_x ? s.s0 + s.l_s : (int64_t)s.l_x, tiles = (most + 63) / 64;
    const double kv_us = (double)s.B * s.H * most * s.d * 4.0 / 4.4e6;
    FwdPlan best{table.form[0].form, 1};
    double best_t = 0.0;
    for (const Cost *c = table.form, *end = c + table.forms; c != end; ++c) {
        const int64_t q_tiles = (s.l_s + c->rows - 1) / c->rows, first = s.causal ? s.s0 + (s.l_s < c->rows ? s.l_s : c->rows) : (int64_t)s.l_x;
        const double mean_tiles = 0.5 * (double)((first + 63) / 64 + tiles);
        const int rest = s.l_s - (int)(q_tiles - 1) * c->rows;
        const double last = c->idle + (1.0 - c->idle) * (double)((rest + 31) / 32) * 32.0 / c->rows, all = ((double)(q_tiles - 1) + last) / (double)q_tiles;
        for (int sp = 1; sp <= max_splits; ++sp) {
            if (sp > 1 && tiles / (sp * c->groups) < 2) break;      // shorter ones cost more than they gain
            const double W = (double)(q_tiles * s.B * s.H * sp);
            // At most 16 workgroups for eight tiles and more: split in any case, as these launches always were and as the
            // tests of the merge's rounding expect of them.  It costs them 0 to 1.5 us (4 heads of 256 rows behind 256: 9.7
            // instead of 8.3) and 0.1 % over all those launches.
            if (sp == 1 && max_splits > 1 && W <= 16.0 && tiles >= 8) continue;
            const double longest = (double)(((tiles + sp - 1) / sp + c->groups - 1) / c->groups);
            const double average = mean_tiles / (sp * c->groups) + (sp * c->groups > 1 ? 0.5 : 0.0);
            const double rounds = ceil(W / 256.0), n = rounds < c->per_cu ? rounds : (double)c->per_cu;
            const double walk = (longest + c->few) * (q_tiles == 1 ? last : 1.0), share = (average + c->few) * all * W / (256.0 * n);
            double t = c->start + c->tile_us * (1.0 + c->shared * (n - 1.0)) * (walk > share ? walk : share);
            if (W > 256.0 * c->per_cu) {
                const double even = !table.rounds || c->per_cu > 1 || first < 0.6 * most ? 0.0 : ((double)first / (double)most - 0.6) / 0.4;
                t += ((1.0 - even) * c->tail + even * (rounds - W / 256.0)) * (average + c->few) * c->tile_us * all;
            }
            t = sqrt(sqrt(t * t * t * t + kv_us * kv_us * kv_us * kv_us));
            if (sp > 1) t += table.merge + out_mb * (8 * sp + 2) / table.mb_per_us;
            if (best_t == 0.0 || t < best_t) { best_t = t; best = {c->form, sp}; }
        }
    }
    return best;
}

} // namespace lss
