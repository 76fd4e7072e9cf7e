// bf16-only building blocks of the tuned kernels (gfx950): direct global -> LDS tile loads into
// swizzled tiles, LDS transpose reads, packed conversions.
#pragma once
#include "lss_common.h"
#include "lss_grid.h"

namespace lss {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// Global -> LDS load without a register in between: lane i moves BYTES (4 or 16) bytes from
// g_uniform + voff to lds_uniform + i * BYTES.  Base pointers are wavefront-uniform, voff per lane.
// Completion is counted like any vector-memory load (wait_vmem_all(), then a barrier, before any
// wavefront reads the data).  Written as inline assembly on purpose: through the compiler builtin
// every later LDS read that the compiler cannot prove disjoint would wait for the load at once,
// which defeats loading a ring slot a whole loop iteration ahead.
// M0 is not saved (two scalar instructions more per load): nothing but these assembly blocks uses it, which tests/test_generated_code.py looks at.  The compiler
// warns of every copy that a reserved register stands among the clobbers.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int BYTES>
__device__ __forceinline__ void lds_dma(const void *g_uniform, uint32_t voff, const void *lds_uniform)
{
    static_assert(BYTES == 4 || BYTES == 16, "");
    const uint32_t lds_addr = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)lds_uniform;
    if (BYTES == 16) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_addr), "v"(voff), "s"(g_uniform) : "memory", "m0");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" : : "s"(lds_addr), "v"(voff), "s"(g_uniform) : "memory", "m0");
}

// A pointer that is wavefront-uniform by contract; said again so that it is kept in scalar registers.  Not a way to bring one there from vector registers
// right before lds_dma(): a vector-memory instruction may read a scalar register that a vector instruction wrote five wait states later at the earliest,
// and the compiler, which keeps to that elsewhere, does not look into assembly.  (tests/test_generated_code.py looks at every kernel of the build.)
__device__ __forceinline__ const void *uniform_ptr(const void *ptr)
{
    const uint64_t p = (uint64_t)ptr;
    return reinterpret_cast<const void *>((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p) |
                                          (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32)) << 32);
}

// N loads of 16 bytes per lane like lds_dma<16>, all from one wavefront-uniform base, load i to lds_uniform + i * STEP
// bytes: one assembly block, so that M0 is saved and restored once and merely stepped from load to load.
template <int N, int STEP>
__device__ __forceinline__ void lds_dma_n(const void *g_uniform, const uint32_t (&off)[N], const void *lds_uniform)
{
    static_assert(N == 1 || N == 2 || N == 4 || N == 8, "");
    g_uniform = uniform_ptr(g_uniform);
    const uint32_t lds_addr = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)lds_uniform;
    uint32_t saved;
#define LSS_FIRST "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, %2\n\t"
#define LSS_NEXT(v) "s_add_u32 m0, m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %" #v ", %2\n\t"
#define LSS_LAST "s_mov_b32 m0, %0"
    if constexpr (N == 1)
        asm volatile(LSS_FIRST LSS_LAST : "=&s"(saved) : "s"(lds_addr), "s"(g_uniform), "i"(STEP), "v"(off[0]) : "memory", "scc");
    else if constexpr (N == 2)
        asm volatile(LSS_FIRST LSS_NEXT(5) LSS_LAST
                     : "=&s"(saved) : "s"(lds_addr), "s"(g_uniform), "i"(STEP), "v"(off[0]), "v"(off[1]) : "memory", "scc");
    else if constexpr (N == 4)
        asm volatile(LSS_FIRST LSS_NEXT(5) LSS_NEXT(6) LSS_NEXT(7) LSS_LAST
                     : "=&s"(saved) : "s"(lds_addr), "s"(g_uniform), "i"(STEP), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3])
                     : "memory", "scc");
    else
        asm volatile(LSS_FIRST LSS_NEXT(5) LSS_NEXT(6) LSS_NEXT(7) LSS_NEXT(8) LSS_NEXT(9) LSS_NEXT(10) LSS_NEXT(11) LSS_LAST
                     : "=&s"(saved)
                     : "s"(lds_addr), "s"(g_uniform), "i"(STEP), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "v"(off[4]),
                       "v"(off[5]), "v"(off[6]), "v"(off[7])
                     : "memory", "scc");
#undef LSS_FIRST
#undef LSS_NEXT
#undef LSS_LAST
}

// Chunk permutation of a row-major LDS tile with D bf16 columns (D / 8 chunks of 16 bytes per row): chunk c
// of row r sits at chunk position c ^ tile_swizzle<D>(r).  The LDS has 64 banks of 4 bytes, i.e. 16 chunk-wide bank groups, and
// serves 16 lanes of a 16-byte read at once -- lanes 0-3, 12-15 and 20-27, then 4-11, 16-19 and 28-31, then the same of the upper
// half -- and 32 lanes of an 8-byte one.  The permutation is linear in bits 0 .. 3 of r, picked by going over all such maps so that no
// two chunks that are served at once share a bank group, for plain fragment reads of 32 rows (32 x 32 x 16
// instructions) and of 16 (16 x 16 x 32) as for transposing reads of 64 and of 32 bytes per row (load_frag_tr_sw,
// load_frag_tr16_sw).  With r & 7 for D = 64 half of the LDS' cycles of the lx50k forward were counted as conflicts; at D = 128, with the
// one that there was, a third of the backward's.  Those kernels do not wait for the LDS:
// 32k keys at d = 128 2350 -> 2339 us, lx24k sweep 21.80 -> 21.76 ms; what it buys is room for more reads.
template <int D>
__device__ __forceinline__ int tile_swizzle(int r)
{
    static_assert(D == 64 || D == 128, "");
    return (D == 64 ? (r & 2) << 1 : (r & 3) << 2) ^ ((r & 4) >> 1) ^ ((r & 8) >> 2) ^ ((r & 8) >> 3);
}

// [ROWS][D] bf16 tile loaded global -> LDS directly (no registers in between), by WAVES wavefronts.
// One such load instruction moves 16 bytes per lane and writes the wavefront's 64 chunks back to
// back (1 KB), so rows cannot be padded; instead the 16-byte chunk c of row r sits at chunk
// position c ^ tile_swizzle<D>(r) of its row, which spreads a column of chunks over the LDS banks as
// padding would.  The permutation is applied on the global side: the lane that fills position p of
// row r fetches chunk p ^ tile_swizzle<D>(r).
template <int D, int ROWS, int WAVES = 4>
struct DirectTile {
    static constexpr int CPR = D / 8;                 // 16-byte chunks per row
    static constexpr int RPI = 64 / CPR;              // rows per load instruction of one wavefront
    static constexpr int NI = ROWS / RPI / WAVES;     // load instructions per wavefront
    static constexpr int BYTES = ROWS * D * 2;
    static_assert(ROWS % (RPI * WAVES) == 0, "tile must divide among the wavefronts");

    // global byte offsets (from the tile's first row) of this lane's chunks; rows >= rows_ok
    // re-read row rows_ok - 1 and chunks >= chunks_ok re-read chunk chunks_ok - 1 (the kernels mask
    // or discard what such rows and columns produce).  Load instruction i of wavefront `wave` fills
    // the 1 KB at byte (i * WAVES + wave) * 1024 of the tile.  Needs ROWS * row_stride * 2 < 2^32.
    static __device__ __forceinline__ void offsets(uint32_t (&off)[NI], int64_t row_stride, int rows_ok, int wave, int lane,
                                                   int chunks_ok = CPR)
    {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int row = (i * WAVES + wave) * RPI + lane / CPR, pos = lane % CPR;
            const int chunk = min(pos ^ tile_swizzle<D>(row), chunks_ok - 1);
            off[i] = ((uint32_t)min(row, rows_ok - 1) * (uint32_t)row_stride + (uint32_t)chunk * 8u) * 2u;
        }
    }
    // Two tensors' tiles, the second following the first in LDS (lds_tile + BYTES), loaded by one assembly block (see lds_dma for
    // why assembly).  Here a wavefront's NI load instructions fill NI consecutive KB of either tile: what the instruction adds to
    // its LDS address it adds to the global one too, so that one LDS address (M0) serves a tile's loads -- each scalar
    // instruction beside the matrix instructions costs a lone wavefront about 8 cycles.  pair_offsets() makes up for that on
    // the global side: its offsets are counted from PAIR_BIAS bytes ahead of the tile's first element (pair_base()).
    static constexpr int PAIR_GROUP = NI < 4 ? NI : 4;        // (what an offset field reaches)
    static constexpr uint32_t PAIR_BIAS = (PAIR_GROUP - 1) * 1024;
    static __device__ __forceinline__ void pair_offsets(uint32_t (&off)[NI], int64_t row_stride, int rows_ok, int wave, int lane)
    {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int row = (wave * NI + i) * RPI + lane / CPR, chunk = (lane % CPR) ^ tile_swizzle<D>(row);
            off[i] = ((uint32_t)min(row, rows_ok - 1) * (uint32_t)row_stride + (uint32_t)chunk * 8u) * 2u + PAIR_BIAS - (uint32_t)(i % PAIR_GROUP) * 1024u;
        }
    }
    static __device__ __forceinline__ const char *pair_base(const bf16_t *first) { return reinterpret_cast<const char *>(first) - PAIR_BIAS; }
    // off0 and off1 may be the same; base pointers (of pair_base()), `lds_tile` and `wave` must be wavefront-uniform
    static __device__ __forceinline__ void issue_pair(const char *g0_uniform, const char *g1_uniform, const uint32_t (&off0)[NI],
                                                      const uint32_t (&off1)[NI], char *lds_tile, int wave)
    {
        static_assert(NI == 1 || NI == 2 || NI == 4 || NI == 8, "");
        const uint32_t lds0 = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)(lds_tile + wave * (NI * 1024));
        const uint32_t lds1 = lds0 + BYTES;
        if constexpr (NI == 1) {
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %4\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %5"
                         : : "s"(lds0), "s"(lds1), "v"(off0[0]), "v"(off1[0]), "s"(g0_uniform), "s"(g1_uniform) : "memory", "m0");
        } else if constexpr (NI == 2) {
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %6\n\tglobal_load_lds_dwordx4 %3, %6 offset:1024\n\t"
                         "s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, %7\n\tglobal_load_lds_dwordx4 %5, %7 offset:1024"
                         : : "s"(lds0), "s"(lds1), "v"(off0[0]), "v"(off0[1]), "v"(off1[0]), "v"(off1[1]), "s"(g0_uniform), "s"(g1_uniform) : "memory", "m0");
        } else {
#pragma unroll
            for (int i = 0; i < NI; i += 4)
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %10\n\tglobal_load_lds_dwordx4 %3, %10 offset:1024\n\t"
                             "global_load_lds_dwordx4 %4, %10 offset:2048\n\tglobal_load_lds_dwordx4 %5, %10 offset:3072\n\t"
                             "s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %6, %11\n\tglobal_load_lds_dwordx4 %7, %11 offset:1024\n\t"
                             "global_load_lds_dwordx4 %8, %11 offset:2048\n\tglobal_load_lds_dwordx4 %9, %11 offset:3072"
                             : : "s"(lds0 + i * 1024), "s"(lds1 + i * 1024), "v"(off0[i]), "v"(off0[i + 1]), "v"(off0[i + 2]), "v"(off0[i + 3]), "v"(off1[i]),
                                 "v"(off1[i + 1]), "v"(off1[i + 2]), "v"(off1[i + 3]), "s"(g0_uniform), "s"(g1_uniform)
                             : "memory", "m0");
        }
    }
    // byte offset inside the tile of the 16-byte chunk c of row r
    static __device__ __forceinline__ int chunk_offset(int r, int c) { return r * (D * 2) + ((c ^ tile_swizzle<D>(r)) * 16); }
};
#pragma clang diagnostic pop

// DS_READ_B64_TR_B16: within each group of 16 lanes, lane i receives element (i % 4) of the
// 8-byte rows addressed by lanes (i / 4) + 4 * t, t = 0..3.  With lane s of a group addressing
// row (s / 4), 4-element column chunk (s % 4) of a row-major tile, lane i ends up with column i
// of 4 consecutive rows: a 4 x 16 block read transposed.  (Lane mapping measured on the GPU.)
//
// A-operand fragment of the TRANSPOSE of a DirectTile: rows [row0, row0+16) become the contraction
// slots, the 32 columns of block `db` the 32 rows of the operand.  `lane_off` is this lane's byte
// offset for that column block (tr_lane_offset_sw), `row0` a multiple of 16.  Over the two reads
// the lane receives, for tile column (lane % 32), the 8 rows 8*a + 4*(lane/32) + t (a = 0, 1;
// t = 0..3) -- exactly the rows that slots 4*a + t of a C-tile half carry (see lss_common.h).
// The second read's rows lie 8 further down: chunk position ^ 3.
template <int D>
__device__ __forceinline__ Frag<bf16_t> load_frag_tr_sw(const char *tile, int row0, int lane_off, int lane_off_8)
{
    const char *p = tile + row0 * (D * 2) + lane_off;
    const char *p8 = tile + row0 * (D * 2) + lane_off_8 + 8 * (D * 2);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p8));
    const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    Frag<bf16_t> f;
    f.v = __builtin_bit_cast(bf16x8, both);
    return f;
}
template <int D>
__device__ __forceinline__ Frag<bf16_t> load_frag_tr_sw(const char *tile, int row0, int lane_off)
{
    return load_frag_tr_sw<D>(tile, row0, lane_off, lane_off ^ 48);
}
// Byte offset for load_frag_tr_sw, columns [32 db, 32 db + 32): within its group of 16 lanes, lane
// s addresses row 4*hh + s/4 (+ row0, a multiple of 16, which does not change the permutation; + 8 for the
// second read, see load_frag_tr_sw) and the 8-byte piece (s % 4) of the 32-byte column group nh (hh,
// nh: bits 1 and 0 of the group index), at the position the chunk permutation of DirectTile gives it.
template <int D>
__device__ __forceinline__ int tr_lane_offset_sw(int lane, int db)
{
    const int grp = lane >> 4, hh = grp >> 1, nh = grp & 1, s = lane & 15;
    const int row = 4 * hh + (s >> 2), chunk = 4 * db + 2 * nh + ((s & 3) >> 1);
    return DirectTile<D, 64>::chunk_offset(row, chunk) + (s & 1) * 8;
}

// The same for 16 x 16 x 32 instructions: rows [row0, row0 + 32) become the contraction slots, the 16 columns of block `db` the
// rows of the operand.  Lane s of group g of 16 addresses row 4 g + s / 4 (the second read: 16 further down, the same
// permutation) and the 8-byte piece s % 4 of the block's 32 bytes, so that slot 4 i + t of group g carries row
// 16 i + 4 g + t -- what the elements of two C blocks of 16 rows carry (mma16).
template <int D>
__device__ __forceinline__ int tr16_lane_offset_sw(int lane, int db)
{
    const int g = lane >> 4, s = lane & 15;
    return DirectTile<D, 64>::chunk_offset(4 * g + (s >> 2), 2 * db + ((s & 3) >> 1)) + (s & 1) * 8;
}
template <int D>
__device__ __forceinline__ Frag<bf16_t> load_frag_tr16_sw(const char *tile, int row0, int lane_off)
{
    const char *p = tile + row0 * (D * 2) + lane_off;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 16 * (D * 2)));
    const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    Frag<bf16_t> f;
    f.v = __builtin_bit_cast(bf16x8, both);
    return f;
}

// Address of tile `tile` of a tensor whose tiles lie `tile_bytes` apart (below 2^32: 64 rows of at most 2^23
// elements): one 32 x 32 -> 64-bit scalar multiply and a 64-bit add, wavefront-uniform.
template <typename T>
__device__ __forceinline__ const T *tile_ptr(const T *base, int tile, uint32_t tile_bytes)
{
    return reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + (uint64_t)(uint32_t)tile * tile_bytes);
}

// Wait until every outstanding vector-memory load of this wave has returned, the direct
// global -> LDS ones included (their data is then in LDS; a barrier publishes it to the other
// wavefronts).
// Wait until at most N of this wave's vector-memory operations are outstanding (they complete in order).
template <int N>
__device__ __forceinline__ void wait_vmem()
{
    static_assert(N >= 0 && N < 64, "");
    asm volatile("s_waitcnt vmcnt(%0)" :: "i"(N) : "memory");       // (also keeps the compiler from moving stores past it)
}
__device__ __forceinline__ void wait_vmem_all() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0), others untouched
// at most N of the LDS reads (and scalar loads) on their way
template <int N>
__device__ __forceinline__ void wait_lds() { static_assert(N >= 0 && N < 16, ""); __builtin_amdgcn_s_waitcnt(0xC07F | N << 8); }
__device__ __forceinline__ void wait_lds_reads() { __builtin_amdgcn_s_waitcnt(0xC07F); }  // lgkmcnt(0), others untouched

// 4 floats -> 4 bf16 (round to nearest even), as one 8-byte value
__device__ __forceinline__ bf16x4 pack4(float a, float b, float c, float d)
{
    bf16x4 v;
    v[0] = (bf16_t)a; v[1] = (bf16_t)b; v[2] = (bf16_t)c; v[3] = (bf16_t)d;
    return v;
}

} // namespace lss
