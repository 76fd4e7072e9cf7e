// Walks the workgroup grids of csrc/lss_grid.h on the host: every work item belongs to exactly one workgroup, workgroups
// past the last item get none, and no id makes the arithmetic undefined (built with -fsanitize=undefined).
#include "lss_grid.h"

#include <cstdio>
#include <vector>

static int fail(const char *what, int a, int b, int id)
{
    std::printf("%s: %d x %d, id %d\n", what, a, b, id);
    return 1;
}

int main()
{
    for (int m = 0; m <= 37; ++m)
        for (int n : {1, 2, 3, 5, 8, 16, 33}) {
            std::vector<int> seen(m * n + 1);
            for (int id = 0; id < lss::xcd_tile_grid(m, n); ++id) {
                const lss::TileId t = lss::xcd_tile(id, m, n);
                if (!t.ok) continue;
                if (t.m < 0 || t.m >= m || t.n < 0 || t.n >= n) return fail("tile outside the matrix", m, n, id);
                ++seen[t.m * n + t.n];
            }
            for (int i = 0; i < m * n; ++i)
                if (seen[i] != 1) return fail("tile not taken once", m, n, i);
        }
    for (int bhs : {1, 2, 3, 7, 8, 9, 13, 16, 27, 64, 171, 513})
        for (int n : {1, 2, 3, 9, 40, 64})
            for (bool uneven : {false, true}) {
                std::vector<int> seen(bhs * n);
                for (int id = 0; id < lss::xcd_grid(bhs, n); ++id) {
                    int bh = -1, inner = -1;
                    if (!lss::xcd_item(id, bhs, n, uneven, bh, inner)) continue;
                    if (bh < 0 || bh >= bhs || inner < 0 || inner >= n) return fail("item outside the grid", bhs, n, id);
                    ++seen[bh * n + inner];
                }
                for (int i = 0; i < bhs * n; ++i)
                    if (seen[i] != 1) return fail("item not taken once", bhs, n, i);
            }
    std::puts("clean");
    return 0;
}
