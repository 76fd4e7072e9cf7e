// Which tile a matrix product of lss_proj.hip takes, and how a weight gradient's rows are shared out, from sizes alone.  Plain C++ without a
// HIP header, so that a host program can go over the choices (tests/host/gemm_plan_check.cpp).
#pragma once
#include <stdint.h>

namespace lss {

constexpr int kGemmK = 64;          // contraction tile

// A workgroup's tile of C (tm x tn), the groups of wavefronts that share its contraction, the workgroups a compute unit holds (lss_proj.hip says
// why; it checks these against its shapes), and what a round of workgroups costs:
//     fixed + contraction tiles x per_tile   microseconds;
// where compute units hold one workgroup each (per_cu = 1: where half of them have one) a contraction tile takes
// per_tile[0], where they are full per_tile[1].
enum GemmTile { TILE_L, TILE_M, TILE_M2, TILE_M8, TILE_S, TILE_S4, TILE_T4, TILE_T8, TILE_COUNT };
struct GemmTileCost { int tm, tn, groups, per_cu; double fixed, per_tile[2]; };
// The figures are fitted to linear_fwd and linear_bwd_input at 230 .. 98304 rows and
// 512 .. 8192 columns either way (20 launches in a graph each), with the loop of 32 x 32 x 16 instructions that there was; those of M8, T4 and T8 came
// later, fitted to linear_fwd, bwd_input and bwd_weight at 58 .. 2048 rows and 256 .. 7680 columns.  L has been 10 % faster since, S4, T4 and T8 with other groups and slots
// 10 to 20 %, and times beside the rules below that name these tiles are of the kernels before that; GeLU behind a product is in no figure.  What that costs,
// 300 drawn feed-forward units and 240 projections, each product in every tile in a graph, behind a kernel that writes its operand, over the best tile: linear_fwd 1.7 % on average
// (at worst 28, long contractions of 4000 to 8000 rows in 128 x 128 tiles: 7697 x 5120 -> 1280 118.7 us, in 256 x 256 ones 92.4), bwd_input 2.4 (36, likewise), with GeLU 0.9
// and 1.0, project_qkv 0.8, bwd_weight 0.7, project_bwd 1.5, its float weight gradient 2.5.  Large tiles move the fewest bytes per flop
// but a launch of few of them leaves compute units idle (2048 x 2048 -> 512: 16 workgroups of 256 x 256, 44 us;
// 256 of 64 x 64, 14), and where even 64 x 64 tiles leave one wavefront per SIMD the chain of contraction
// tiles is what takes the time, which groups of wavefronts share.
constexpr GemmTileCost kGemmTiles[TILE_COUNT] = {
    {256, 256, 1, 1, 6.5, {1.40, 1.70}}, {128, 128, 1, 2, 2.8, {0.62, 1.00}}, {128, 128, 2, 1, 3.0, {0.50, 0.58}}, {128, 128, 1, 1, 2.5, {0.51, 0.585}},
    {64, 64, 1, 2, 2.5, {0.30, 0.40}}, {64, 64, 2, 1, 3.3, {0.165, 0.22}}, {32, 64, 4, 1, 3.0, {0.117, 0.165}}, {32, 32, 4, 1, 3.2, {0.069, 0.107}}};

// What a kernel's contraction goes through: groups of wavefronts, and slots of the LDS ring of each (of the activations, where a 256 x 256 tile has fewer for
// the weights).  `length`: of a map's contraction, or the rows of a chunk of a weight gradient.
struct GemmForm { int groups, slots; };
constexpr int kLongFloat = 832;
// Float operands travel through registers a tile per group at a time: more slots gain them nothing, and their long contractions are better off with more groups.
// project_bwd_weight with dW_kv in 64 x 64 tiles of two and of four groups, us: chunks of 367 rows 8.8 and 9.2, 584 12.2 and 12.8, 746 11.7 and 12.0, 905 13.0 and
// 12.7, 1106 14.9 and 14.6, 1352 15.8 and 15.2, 1855 20.0 and 19.3, 2983 27.0 and 24.7; in 32 x 32 ones of four and of eight 346 6.9 and 7.1, 569 7.3 and 7.5, 850 8.6 and
// 8.5, 947 7.9 and 7.8, 1352 11.4 and 10.6, 1939 12.8 and 12.1.  project_bwd in 32 x 32 ones: contractions of 1024 6.0 and 6.0, 1280 5.4 and 5.1, 2048 7.0 and 6.2, 4096
// 15.1 and 12.2; in 64 x 64 ones 512 5.9 and 6.6, 1024 8.3 and 8.5, 1536 10.1 and 9.6, 2816 20.0 and 18.6 (four groups for all).
constexpr GemmForm gemm_form(GemmTile t, bool weight_gradient, bool floats, int length)
{
    if (floats && t == TILE_S4 && (!weight_gradient || length > kLongFloat)) return {4, 2};
    if (floats && t == TILE_T4) return {4, 2};
    if (floats && t == TILE_T8 && length > kLongFloat) return {8, 2};
    constexpr int slots[TILE_COUNT] = {3, 2, 2, 4, 4, 4, 3, 4};
    return {kGemmTiles[t].groups, slots[t]};
}

// `tiles`: contraction tiles of a workgroup on average, `rest_tiles`: of those in the last, part-filled round
inline double gemm_estimate(const GemmTileCost &c, double wgs, double tiles, double rest_tiles)
{
    const double room = 256.0 * c.per_cu, full = (double)(int64_t)(wgs / room), rest = wgs - full * room;
    return full * (c.fixed + tiles * c.per_tile[1]) + (rest > 0 ? c.fixed + rest_tiles * c.per_tile[rest > (c.per_cu == 1 ? 128 : 256)] : 0.0);
}

// One product of a launch, C [batches][rows][N] = A [batches][rows][K] W; rows_ok: leading rows of A that hold data
struct GemmWork { int batches, rows, rows_ok, N, K, a_f32; };
inline int64_t gemm_rows_ok(const GemmWork &w) { return w.rows < w.rows_ok ? w.rows : w.rows_ok; }

// Whether C is written with non-temporal stores: where A and C together are more than half the last-level cache
// (256 MB), results kept there and in the L2s only push out the operand tiles that other workgroups are about
// to read again.  The product and a pass over its results right after it: 32768 x 512 -> 2048 with GeLU in the product 205 -> 175 us, GeLU
// behind it 141 -> 132; 98304 x 1024 -> 2048 and -> 1024 more (projections of 4 x 24576 rows) 446 -> 434 alone; the gradient of 4 x 12000 rows of 512
// columns 92 -> 87; 31 such pairs of 138 MB and more 3.6 % less time on average, the worst 1.6 % more.  Below that the product gains
// as much, but who reads its results pays more (8192 x 1024 -> 4096 with GeLU and the next product 155 -> 159, 4096 rows 84 -> 94).
inline bool gemm_streams(const GemmWork *work, int n, bool out_f32)
{
    double bytes = 0.0;
    for (const GemmWork *w = work; w != work + n; ++w)
        bytes += (double)w->batches * ((double)gemm_rows_ok(*w) * w->K * (w->a_f32 ? 4 : 2) + (double)w->rows * w->N * (out_f32 ? 4 : 2));
    return bytes > 128e6;
}

// Workgroups of one product in tiles `c`; on_xcds: eight times those of the XCD that has the most (xcd_tile in lss_grid.h deals a product's tiles out evenly)
inline double gemm_workgroups(const GemmTileCost &c, const GemmWork &w, bool on_xcds)
{
    const int64_t tiles = (int64_t)w.batches * ((gemm_rows_ok(w) + c.tm - 1) / c.tm) * ((w.N + c.tn - 1) / c.tn);
    return (double)(on_xcds ? (tiles + 7) / 8 * 8 : tiles);
}

// What a launch of the products `work` takes in tiles `t`
inline double gemm_launch_estimate(GemmTile t, const GemmWork *work, int n, bool skip_tail)
{
    const GemmTileCost &c = kGemmTiles[t];
    // A launch waits for the XCD that has the most workgroups: projections of 3 x 5193 rows of 128 columns and 500 of each have 33 of 128 x 128 for the
    // 32 compute units of some, 12.6 us, and where each holds two of them 10.2.  2159 drawn projections in every tile: 0.13 % over the best one on
    // average and at worst 8 %, 0.32 and 47 % with both products' workgroups just added up.  (Not with a float A, whose figures fit the plain sum:
    // 4737 drawn calls, 1.90 % over the best tile and 19 more than 3 % slower than without 32-wide tiles, 1.89 and 3 so.)
    const bool on_xcds = !work->a_f32;
    double wgs = 0, tiles_all = 0, sum = 0, last_n = 0, last_tiles = 0;
    for (const GemmWork *w = work; w != work + n; ++w) {
        const double count = gemm_workgroups(c, *w, false);
        // A float A costs more the smaller the tile, whose workgroups re-read it more often, and the less of it
        // fits the last-level cache (project_bwd, 1024 columns: 256 x 256 against 128 x 128 tiles take 64 and
        // 57 us at 8192 rows, 102 and 97 at 16384, 156 and 165 at 24000)
        double slow = 1.0, more = 0.0;
        if (w->a_f32) {
            const int64_t zero_rows = skip_tail ? 0 : w->rows - gemm_rows_ok(*w);       // their stores pass through it too
            const double bytes = (double)w->batches * ((double)w->rows_ok * w->K + (double)zero_rows * w->N) * 4.0;
            const double far = bytes < 256e6 ? bytes / 256e6 : 1.0;
            slow = c.tm == 256 ? 1.05 + 0.35 * far : c.tm == 128 ? 1.15 + 0.35 * far : 1.6 + 0.5 * far;
            more = c.tm == 256 ? 1.5 : c.tm == 128 ? 6.0 + 2.0 * far : 0.0;
        }
        wgs += gemm_workgroups(c, *w, on_xcds);
        tiles_all += count;
        last_n = count;
        last_tiles = w->K / kGemmK * slow + more;
        sum += count * last_tiles;
    }
    if (wgs <= 0) return 0.0;
    const double room = 256.0 * c.per_cu, rest = wgs - room * (double)(int64_t)(wgs / room), tiles = sum / tiles_all;
    return gemm_estimate(c, wgs, tiles, rest <= last_n ? last_tiles : tiles);     // (the last job's workgroups start last)
}

// Rows of C without data are cleared by workgroups of their own, 64 KB each or a tile where that is more.  By tiles, those of the 32- and
// 64-wide ones -- 512 or 1024 threads that store 4 to 16 KB, one of which fills a compute unit's LDS -- took longer than their bytes: project_bwd of
// 43,186 rows of 128 columns of which 2081 have data, 10.6 us in 64 x 64 tiles and 20.0 in 32 x 32 ones, which the estimates then chose: they leave these
// rows out, whose time hardly depends on the tile now.  A 256 x 256 one is 256 KB: by 64 KB, 4 x 16,919 rows of 768 columns of which 3949 each have data
// took 100 us, 91 by tiles (2431 workgroups and 608, each with a compute unit's whole LDS).
// gemm_zero_end: the end of the rows to clear (skip_tail leaves those from the next multiple of 256 on unwritten); gemm_zero_tiles: workgroups per
// batch entry and tile of columns, gemm_zero_rows() rows each.  The last tile of rows with data clears its own rest.
constexpr int gemm_zero_rows(int tm, int tn) { return tm * tn > 16384 ? tm : 16384 / tn; }
inline int gemm_zero_end(int rows, int rows_ok, bool skip_tail)
{
    const int64_t next = ((int64_t)rows_ok + 255) / 256 * 256;
    return skip_tail && next < rows ? (int)next : rows;
}
inline int gemm_zero_tiles(int rows, int rows_ok, bool skip_tail, int tm, int tn)
{
    const int64_t done = ((int64_t)(rows < rows_ok ? rows : rows_ok) + tm - 1) / tm * tm, left = gemm_zero_end(rows, rows_ok, skip_tail) - done;
    return left > 0 ? (int)((left + gemm_zero_rows(tm, tn) - 1) / gemm_zero_rows(tm, tn)) : 0;
}

// Whether a launch may take tiles `t`.  32-wide ones only where one round of workgroups takes them all (with the kernels of two slots none of 4000 drawn linear maps that
// need more was faster in them: the weights come once more from the last-level cache, which the estimate does not know; with the present ones
// 644 x 6144 -> 1536, 504 workgroups, takes 40.4 us, 40.1 in 64 x 64 tiles, 581 x 6656 -> 1664 36.6 and 42.5; counted as the launch's estimate counts them, per XCD unless A is float:
// project_bwd's 252 for 282 x 2304 floats -> 1152 and 152 x 1152 -> 1152 13.8 us, in 64 x 64 tiles 16.3), and never with results past the caches,
// without which their kernel is built
inline bool gemm_takes(GemmTile t, const GemmWork *work, int n, bool a_any, bool streams)
{
    const GemmTileCost &c = kGemmTiles[t];
    if (t == (a_any ? TILE_M8 : TILE_M2)) return false;
    if (c.tm != 32) return true;
    double wgs = 0.0;
    for (const GemmWork *w = work; w != work + n; ++w) wgs += gemm_workgroups(c, *w, !work->a_f32);
    return !streams && wgs <= 256.0;
}

// The tile of a launch: the one with the smallest estimate.
// 128 x 128 tiles of which a compute unit holds one: a short contraction is all on its way at once in four slots, and nothing is left to add up
// (linear_fwd and bwd_input of 2048 x 512 -> 2048 9.9 -> 9.2 us, 9.7 -> 9.1; linear_fwd of long contractions whose A has just been written takes 1 to 4 %
// longer so, 1047 x 8192 -> 2048 67 -> 70, but among the other launches of a layer, from colder operands, less: 1828 x 8192 -> 2048 92 -> 77).  Not with a float A, whose
// tiles travel through registers one at a time (project_bwd of 1500 x 2048 50.6 us in two groups, 54.2 so), nor for the weight
// gradients, both of whose operands are read transposed, more often in smaller parts (2048 x 2048 from 2048 rows 24.8 and 26.0).
// a_any: the kernels that take a float A, in any of the products
inline GemmTile pick_gemm_tile(const GemmWork *work, int n, bool a_any, bool skip_tail, bool streams)
{
    GemmTile best = TILE_L;
    double best_t = gemm_launch_estimate(TILE_L, work, n, skip_tail);
    for (int i = TILE_M; i < TILE_COUNT; ++i) {
        if (!gemm_takes((GemmTile)i, work, n, a_any, streams)) continue;
        const double t = gemm_launch_estimate((GemmTile)i, work, n, skip_tail);
        if (t < best_t) { best_t = t; best = (GemmTile)i; }
    }
    return best;
}

// The most chunks of rows a weight gradient is split into, per batch entry: what two 256 x 256 workgroups per
// compute unit would take (wgrad_max_chunks: for any number of rows), of at least eight 64-row tiles each.
// The scratch sizes the header promises follow from it.
inline int wgrad_max_chunks(int batches, int K, int N)
{
    const int tiles = ((K + 255) / 256) * ((N + 255) / 256);
    return ((512 + tiles - 1) / tiles + batches - 1) / batches;
}
inline int wgrad_most_chunks(int rows, int batches, int K, int N)
{
    const int R = (rows + kGemmK - 1) / kGemmK, want = wgrad_max_chunks(batches, K, N);
    int chunk_tiles = (R + want - 1) / want;
    if (chunk_tiles < 8) chunk_tiles = R < 8 ? R : 8;
    return chunk_tiles < 1 ? 1 : (R + chunk_tiles - 1) / chunk_tiles;
}

// Tile and split of the rows: the pair with the smallest estimated time, the sum of the chunks' partial results
// (3.5 us and their bytes at 4 TB/s) included; a chunk never crosses batch entries.  Shape-only,
// deterministic.
struct WgradPlan { GemmTile tile; int splits_per_batch, chunk_rows; };
inline WgradPlan pick_wgrad_plan(int rows, int batches, int K, int N, bool dc_f32)
{
    const int R = (rows + kGemmK - 1) / kGemmK, most = wgrad_most_chunks(rows, batches, K, N);
    WgradPlan best{TILE_L, 1, kGemmK};
    double best_t = 0.0;
    for (int want = 1; want <= most; want = want < 4 ? want + 1 : want + want / 3) {
        const int chunk_tiles = (R + want - 1) / want, splits = (R + chunk_tiles - 1) / chunk_tiles;      // splits <= want
        const double parts = (double)batches * splits;
        const double sum = parts > 1 ? 3.5 + (parts + 1) * K * N * 4e-6 / 4.0 : 0.0;
        for (int i = 0; i < TILE_COUNT; ++i) {
            if (i == TILE_M8) continue;
            const GemmTileCost &c = kGemmTiles[i];
            // (both operands through transposing reads: a fifth slower per tile, but for the largest)
            // (32-wide tiles: not for fewer contraction tiles than groups of wavefronts, which gain nothing -- dW of 256 x 1024 from 130 to 190 rows 6.5 us in
            // 64 x 64 ones, 7.0 -- and dearer the longer the chunk: they read every operand more often, from the last-level cache where it has just been
            // written -- behind two copies dW of 256 x 1024 from 2000 rows 17.9 -> 16.5 us, copies included, but from 4000, which larger tiles share out in
            // chunks, 24.2 -> 26.9.  A float dC travels through registers, a tile at a time: of 256 x 512 from 1512 rows 25.3 -> 20.7, from 4064 27.8 -> 33.2)
            if (c.tm == 32 && chunk_tiles < 4) continue;
            if (dc_f32 && i == TILE_T4) continue;       // (never the shortest of the others, and not built)
            const double dearer = c.tm != 32 ? 1.0 : dc_f32 ? 2.2 : 1.0 + 0.015 * (chunk_tiles > 24 ? chunk_tiles - 24 : 0);
            const double tiles = chunk_tiles * (c.tm == 256 ? 1.0 : 1.2) * dearer;
            const double t = sum + gemm_estimate(c, parts * ((K + c.tm - 1) / c.tm) * ((N + c.tn - 1) / c.tn), tiles, tiles);
            if (best_t == 0.0 || t < best_t) { best_t = t; best = {(GemmTile)i, splits, chunk_tiles * kGemmK}; }
        }
    }
    return best;
}

} // namespace lss
