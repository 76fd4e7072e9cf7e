// Goes over the choices of csrc/lss_gemm_plan.h on the host: a launch takes a tile that it has a kernel for, none of the others is estimated
// shorter, and launches that were measured in every tile stay in the tiles they were found in; a weight gradient's chunks cover its rows within the scratch
// that the header promises; the rows without data are cleared 16384 elements at a time, or a tile where that is more.
#include "lss_gemm_plan.h"

#include <cstdio>
#include <initializer_list>
#include <vector>

using namespace lss;

static int fail(const char *what, const GemmWork &w, int tile)
{
    std::printf("%s: %d x %d of %d rows, K %d, N %d, float %d: tile %d\n", what, w.batches, w.rows_ok, w.rows, w.K, w.N, w.a_f32, tile);
    return 1;
}

// Launches that were timed in every tile, behind a launch that writes their operands, and the tile they take, the shortest with the kernels that the rules were
// drawn from.  (Times of the present kernels, in graphs: 32-wide tiles have become shorter by more than the others.)
struct Measured {
    GemmWork work[2];
    int n;
    std::vector<GemmTile> good;
};
static const Measured measured[] = {
    {{{1, 644, 644, 1536, 6144, 0}}, 1, {TILE_S}},                                                  // 40.1 us, 40.4 in 32 x 64 tiles
    {{{1, 581, 581, 1664, 6656, 0}}, 1, {TILE_S}},                                                  // 42.5, 36.6
    {{{1, 120, 120, 1280, 1280, 0}}, 1, {TILE_T4, TILE_T8}},                                        // 6.2 and 5.5, 7.4 in 64 x 64 ones
    {{{1, 15579, 15579, 256, 128, 0}, {3, 500, 500, 128, 128, 0}}, 2, {TILE_M}},                    // projections: 7.1, 9.4 in 128 x 128 ones of eight wavefronts
    {{{1, 3699, 3699, 2816, 1408, 0}, {3, 1233, 1233, 1408, 1408, 0}}, 2, {TILE_M}},                // 48.6, 68.5 in 256 x 256 ones
    {{{1, 11969, 11969, 1280, 640, 0}, {1, 1426, 1426, 640, 640, 0}}, 2, {TILE_M}},                 // 29.0, 44.4
    {{{4, 2262, 1768, 1280, 2560, 1}, {4, 1463, 1463, 1280, 1280, 0}}, 2, {TILE_L}},                // project_bwd: 71.6, 95.3 in 128 x 128 ones
    {{{3, 653, 610, 640, 1280, 1}, {3, 403, 403, 640, 640, 0}}, 2, {TILE_S}},                       // 17.8, 21.6 in 128 x 128 ones of two groups
    {{{1, 870, 282, 1152, 2304, 1}, {1, 152, 152, 1152, 1152, 0}}, 2, {TILE_T4}},                   // 13.8 (252 workgroups), 16.3 in 64 x 64 ones of groups
    {{{1, 43186, 2081, 128, 256, 1}, {1, 689, 689, 128, 128, 0}}, 2, {TILE_S, TILE_S4, TILE_T4, TILE_T8}},  // 8.5, 8.1 in 64 x 64 ones; their rows without data cost the same in all
};

int main()
{
    for (const Measured &m : measured) {
        const GemmTile t = pick_gemm_tile(m.work, m.n, m.work[0].a_f32, false, false);
        bool good = false;
        for (const GemmTile g : m.good) good = good || g == t;
        if (!good) return fail("not among the shortest", m.work[0], t);
    }
    const struct { int rows, batches, K, N; bool dc_f32; std::vector<GemmTile> good; } gradients[] = {
        {142, 1, 256, 1024, false, {TILE_S}},                       // 3.6 us, 3.8 in 64 x 64 ones of groups
        {161, 1, 1024, 256, false, {TILE_S}},                       // 2.9, 3.1
        {250, 1, 384, 384, false, {TILE_S, TILE_T4, TILE_T8}},      // 3.9, 4.1, 3.6
        {815, 1, 1024, 256, false, {TILE_T4, TILE_T8}},             // 6.1 and 5.9, 6.6 in 64 x 64 ones of groups
        {2964, 1, 256, 256, false, {TILE_T4, TILE_T8, TILE_S, TILE_S4}},      // 8.5, 9.3, 8.9, 8.9
        {3040, 1, 1024, 256, false, {TILE_S4, TILE_S}},             // 10.5, 11.0, 10.8 in 32 x 32 ones
        {1512, 1, 256, 512, true, {TILE_T4, TILE_T8}},              // 9.1, 10.9 in 64 x 64 ones
    };
    for (const auto &g : gradients) {
        const WgradPlan p = pick_wgrad_plan(g.rows, g.batches, g.K, g.N, g.dc_f32);
        bool good = false;
        for (const GemmTile t : g.good) good = good || t == p.tile;
        if (!good || (kGemmTiles[p.tile].tm == 32 && p.chunk_rows < 4 * kGemmK))
            return fail("weight gradient not in one of the shortest", {g.batches, g.rows, g.rows, g.N, g.K, g.dc_f32}, p.tile);
    }
    for (int batches : {1, 4, 65535})
        for (int rows : {1, 31, 58, 256, 1000, 2048, 16384, 98304, 0x7fffffff})
            for (int ok : {1, 64, 0x7fffffff})
                for (int K : {128, 512, 2048, 65536})
                    for (int N : {128, 640, 4096, 65536})
                        for (int form = 0; form < 4; ++form) {
                            if (ok < rows && ok > 64) ok = rows;
                            const bool any = form & 1, skip = form & 2;
                            const GemmWork work[2] = {{batches, rows, ok, N, K, any}, {batches, rows, rows, N, K, 0}};
                            for (int n : {1, 2})
                                for (bool streams : {false, true}) {
                                    const GemmTile t = pick_gemm_tile(work, n, any, skip, streams);
                                    if (t < 0 || t >= TILE_COUNT || t == (any ? TILE_M8 : TILE_M2) || (streams && kGemmTiles[t].tm == 32))
                                        return fail("no such kernel", work[0], t);
                                    double wgs = 0.0;
                                    for (int i = 0; i < n; ++i) wgs += gemm_workgroups(kGemmTiles[t], work[i], !work->a_f32);
                                    if (kGemmTiles[t].tm == 32 && wgs > 256.0) return fail("small tiles, more than one round", work[0], t);
                                    const double us = gemm_launch_estimate(t, work, n, skip);
                                    if (!(us > 0.0)) return fail("no time", work[0], t);
                                    for (int o = 0; o < TILE_COUNT; ++o)
                                        if (gemm_takes((GemmTile)o, work, n, any, streams) && gemm_launch_estimate((GemmTile)o, work, n, skip) < us)
                                            return fail("a shorter one is there", work[0], t);
                                }
                            if (rows > 1 << 20) continue;
                            const WgradPlan p = pick_wgrad_plan(rows, batches, K, N, any);
                            if (p.tile < 0 || p.tile >= TILE_COUNT || p.tile == TILE_M8 || (any && p.tile == TILE_T4) ||
                                (kGemmTiles[p.tile].tm == 32 && p.chunk_rows < 4 * kGemmK))
                                return fail("no such weight gradient", work[0], p.tile);
                            if (p.splits_per_batch < 1 || p.splits_per_batch > wgrad_most_chunks(rows, batches, K, N) || p.splits_per_batch > wgrad_max_chunks(batches, K, N) ||
                                p.chunk_rows % kGemmK != 0 || (int64_t)p.splits_per_batch * p.chunk_rows < rows || (int64_t)(p.splits_per_batch - 1) * p.chunk_rows >= rows)
                                return fail("chunks", work[0], p.tile);
                        }
    for (int rows : {1, 31, 32, 33, 255, 256, 257, 511, 4096, 50112, 0x7fffffff})
        for (int ok : {0, 1, 31, 32, 64, 200, 256, 300, 4095, 4096, 50112, 0x7fffffff})
            for (bool skip : {false, true})
                for (const GemmTileCost &c : kGemmTiles) {
                    if (ok > rows) continue;
                    const int64_t done = ((int64_t)ok + c.tm - 1) / c.tm * c.tm, end = skip ? ((int64_t)ok + 255) / 256 * 256 : rows;
                    const int tiles = gemm_zero_tiles(rows, ok, skip, c.tm, c.tn), zero_end = gemm_zero_end(rows, ok, skip), each = gemm_zero_rows(c.tm, c.tn);
                    if (zero_end != (end < rows ? end : rows) || each * c.tn != (c.tm * c.tn > 16384 ? c.tm * c.tn : 16384) || tiles > ((int64_t)rows - ok + each - 1) / each ||
                        done + (int64_t)tiles * each < zero_end || (tiles > 0 && done + (int64_t)(tiles - 1) * each >= zero_end))
                        return fail("rows without data", {1, rows, ok, 128, 128, 1}, c.tm);
                }
    std::printf("clean\n");
    return 0;
}
