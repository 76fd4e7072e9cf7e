// Which workgroup takes which work item.  Plain integer arithmetic without a HIP header, so that a host program can walk
// whole grids.
#pragma once
#include <stdint.h>

#if defined(__HIP__)
#define LSS_HD __host__ __device__ __attribute__((always_inline))
#else
#define LSS_HD
#endif

namespace lss {

// Workgroup order for grids of (batch*head, inner) work items.  Consecutive workgroup ids go to
// consecutive XCDs (8 of them, each with its own L2 and an eighth of the compute units).
//   * Whole rounds of eight heads: item `id` is head id % 8 + 8 * (id / 8 / n_inner), inner index
//     (id / 8) % n_inner, so an XCD sees ONE head at a time (all inner items of head x, then of head
//     x + 8, ...) and what the workgroups of a head share (K and V, or Q and dO) stays in its L2.
//   * The r = bhs % 8 heads that are left are dealt out item by item, item i being head i % r, inner index
//     i / r: all XCDs get their share, an XCD sees r / gcd(r, 8) heads at once.  One head per XCD
//     here too would leave 8 - r of the eight with nothing to do: three heads of 1721 queries against
//     12,712 keys in float took 250 us on three XCDs, whatever the split of the keys, and take 105 on eight.
//   * All heads are dealt out when the work of the items differs (`uneven`: under the causal mask key tiles do, and
//     query tiles where the segment is a good part of the keys) and they all fit the chip at once (512): the longest items of every head then start before the shortest of any, and each
//     compute unit gets one of each (4 x 13 heads of 948 tokens: backward 50 us, dealt out 42).
// Grid size xcd_grid(bhs, n_inner), a multiple of 8; ids past the last item: xcd_item returns false.
constexpr int kXcds = 8;
inline int xcd_grid(int bhs, int n_inner) { return kXcds * (int)(((int64_t)bhs * n_inner + kXcds - 1) / kXcds); }
LSS_HD inline bool xcd_item(int id, int bhs, int n_inner, bool uneven, int &bh, int &inner)
{
    const int left = uneven && bhs * n_inner <= 512 ? bhs : bhs % kXcds, whole = bhs - left, i = id - whole * n_inner;
    if (i < 0) {
        const int rest = id / kXcds;
        inner = rest % n_inner;
        bh = id % kXcds + kXcds * (rest / n_inner);
        return true;
    }
    if (i >= left * n_inner) return false;
    inner = i / left;
    bh = whole + i % left;
    return true;
}

// Position of workgroup `id` of a grid of m_tiles x n_tiles tiles: consecutive ids go to consecutive XCDs
// (each with its own L2), and every XCD gets a contiguous run of tiles, so that few row tiles still fill all
// XCDs.  Tiles are numbered in blocks of four row tiles, column by column: the 32 workgroups an XCD runs at a
// time then read few different operand strips (4 + 8 instead of 2 + 16 where a row has 16 column tiles).
struct TileId { int m, n; bool ok; };
LSS_HD inline TileId xcd_tile(int id, int m_tiles, int n_tiles)
{
    const int tiles = m_tiles * n_tiles, per_xcd = (tiles + kXcds - 1) / kXcds;
    const int t = id % kXcds * per_xcd + id / kXcds;
    if (id / kXcds >= per_xcd || t >= tiles) return {0, 0, false};     // (first of all: past the last tile `rows` would be 0 or negative)
    const int block = t / (4 * n_tiles), in = t % (4 * n_tiles), rows = m_tiles - 4 * block < 4 ? m_tiles - 4 * block : 4;
    return {4 * block + in % rows, in / rows, true};
}
LSS_HD inline int xcd_tile_grid(int m_tiles, int n_tiles) { return kXcds * ((m_tiles * n_tiles + kXcds - 1) / kXcds); }

} // namespace lss
