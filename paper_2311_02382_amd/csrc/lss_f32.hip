// Single-precision forward and backward of Eq. 2 (Section 3, Principle 3) for one segment.  The matrix products run
// on the bf16 matrix cores, every float split into three bf16 parts.
//
// A float x is the exact sum of three bf16 numbers: x0 = bf16(x), x1 = bf16(x - x0), x2 = x - x0 - x1 (rounded to
// nearest, each part takes 8 of the 24 significand bits; both differences are exact; the method of Henry, Tang
// and Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", ARITH 2019).
// That holds for 0 and for 2^-103 <= |x| < 3.39e38; what lies outside is found and done on the fp32 matrix cores
// (product_f32).  Weights and score gradients below 2^-103 are carried to 2^-134.  A product of two
// floats is then nine products of parts, |x_i y_j| <= 2^-8(i+j) |x y|, each exact in the matrix core's fp32
// accumulation.  The six with i + j <= 2 are added, smallest first; the three left out are together below 2^-23
// of |x y|, the size of the rounding an fp32 multiply-add makes at every step, while a matrix instruction here
// adds 32 products per rounding instead of two (with eight of the nine the errors below stay as they are).
// Relative errors against fp64 (512 rows, 2000 keys, N(0, 1) inputs; in brackets those of V_MFMA_F32_32X32X2_F32, which these kernels
// used at first): out 4.3e-7 (5.8e-7), dq 3.9e-7 (6.4e-7), dk 4.8e-7 (7.0e-7), dv 4.8e-7 (6.8e-7); at three times the standard
// deviation out 1.0e-6 (1.5e-6), dq 2.7e-6 (3.5e-6).
// What it buys: six V_MFMA_F32_16X16X32_BF16 (96 cycles) do what eight 16x16x4 fp32 ones (256 cycles) did: lx8k in single
// precision, eight segments: forward 1605 -> 910 us, backward 5460 -> 2750 us (with 32x32x16 instructions).
// 16x16x32 instructions take less power per product than 32x32x16 and add twice as many products per rounding: with them, operands read
// one step ahead of their use and a maximum that is raised only when it must be, forward 892 -> 816 us, backward 2738 -> 2553
// (the same eight segments, another card). What is left is the chain of a workgroup's tiles in launches that fill the chip
// once or twice, and in the forward the vector work (splitting costs 5.5 instructions for every float of a tile and every weight).
//
// Operand roles, layouts and the online softmax are those of the bf16 kernels: scores transposed with one query
// per lane in the forward and dQ workgroups, one key per lane in the dK/dV workgroups; K/V (or Q/dO) tiles go
// global -> registers -> three bf16 planes in LDS (row-major, swizzled), from where the products over tile rows
// read them transposed.  Two workgroups share a compute unit: one splits and stores a tile while the other
// multiplies.
#include "lss_bf16.h"
#include "lss_kernels.h"

#include <type_traits>

namespace lss {

namespace {

struct Frag3 { Frag<bf16_t> p[3]; };            // the three parts of one operand fragment

// Pairs at a time, through the bits: one packed conversion per pair and part, 5.5 vector instructions per element
// (converted one by one, the parts that are needed as floats again take a conversion each: 7.5).
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t round_pair(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ float low_of(uint32_t pair) { return __builtin_bit_cast(float, pair << 16); }
__device__ __forceinline__ float high_of(uint32_t pair) { return __builtin_bit_cast(float, pair & 0xffff0000u); }
__device__ __forceinline__ Frag3 split8(const float (&x)[8])
{
    u32x4 part[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t b0 = round_pair(x[2 * i], x[2 * i + 1]);
        const float r0 = x[2 * i] - low_of(b0), r1 = x[2 * i + 1] - high_of(b0);
        const uint32_t b1 = round_pair(r0, r1);
        part[0][i] = b0;
        part[1][i] = b1;
        part[2][i] = round_pair(r0 - low_of(b1), r1 - high_of(b1));
    }
    Frag3 f;
#pragma unroll
    for (int p = 0; p < 3; ++p) f.p[p].v = __builtin_bit_cast(bf16x8, part[p]);
    return f;
}
// Below 2^-103 the third part is subnormal and loses bits (bf16 has the exponents of float).  Inputs that small, other than
// 0, are looked for in two steps: the least magnitude costs half an instruction per float, and only where it is
// small (zeros make it so as well) is every value looked at.
constexpr float kTiny = 0x1p-103f;
template <int N>
__device__ __forceinline__ float least_magnitude(const f32x4 (&x)[N], float least)
{
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int e = 0; e < 4; e += 2) asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(least) : "v"(x[i][e]), "v"(x[i][e + 1]));
    return least;
}
// The bits of a float without the sign, doubled: ordered like |x|.  Less one, zeros come last.
__device__ __forceinline__ uint32_t twice_magnitude(float x) { return __builtin_bit_cast(uint32_t, x) << 1; }
template <int N>
__device__ __forceinline__ bool some_below(const f32x4 (&x)[N], float limit)
{
    uint32_t least_nonzero = ~0u;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) least_nonzero = min(least_nonzero, twice_magnitude(x[i][e]) - 1u);
    return least_nonzero < twice_magnitude(limit) - 1u;
}
// (NJ: blocks of 16 queries or keys that a wavefront holds: two in the forward, kBlocks in the backward)
// This lane's fragments of its NJ rows: D / 32 times 8 floats of each, 32 apart.  Returns whether some lane's rows hold tiny values.
template <int D, int NJ>
__device__ __forceinline__ bool split_rows(const float *p, const int64_t (&off)[NJ], Frag3 (&f)[D / 32][NJ])
{
    float least = INFINITY;
    f32x4 v[D / 32][NJ][2];
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int n = 0; n < 2; ++n) v[ks][j][n] = *reinterpret_cast<const f32x4 *>(p + off[j] + ks * 32 + 4 * n);
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const f32x4 *const w = v[ks][j];
            least = least_magnitude(v[ks][j], least);
            const float x[8] = {w[0][0], w[0][1], w[0][2], w[0][3], w[1][0], w[1][1], w[1][2], w[1][3]};
            f[ks][j] = split8(x);
        }
    bool tiny = false;
    if (__any(least < kTiny)) {
#pragma unroll 1
        for (int ks = 0; ks < D / 32; ++ks)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const f32x4 w[2] = {*reinterpret_cast<const f32x4 *>(p + off[j] + ks * 32), *reinterpret_cast<const f32x4 *>(p + off[j] + ks * 32 + 4)};
                tiny = tiny || some_below(w, kTiny);
            }
        tiny = __any(tiny);
    }
    return tiny;
}
// 32 tile rows against the wavefront's 16 NJ queries (or keys) as 16 x 16 blocks: element e of block (i, j) is, in lane
// l, tile row 16 i + 4 (l / 16) + e and query 16 j + l % 16.
template <int NJ> struct Block { f32x4 v[2][NJ]; };
template <int NJ>
__device__ __forceinline__ Frag3 split_acc(const Block<NJ> &c, int j)      // as the operand of a product over the tile rows
{
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = c.v[e >> 2][j][e & 3];
    return split8(x);
}
// The five products below x0 y0, of one operand with NJ others
template <int NJ>
__device__ __forceinline__ void mma_small(const Frag3 &a, const Frag3 (&b)[NJ], f32x4 (&c)[NJ])
{
    constexpr int pa[5] = {2, 0, 1, 1, 0}, pb[5] = {0, 2, 1, 0, 1};
#pragma unroll
    for (int t = 0; t < 5; ++t)
#pragma unroll
        for (int j = 0; j < NJ; ++j) c[j] = mma16(a.p[pa[t]], b[j].p[pb[t]], c[j]);
}
template <int NJ>
__device__ __forceinline__ void mma6(const Frag3 &a, const Frag3 (&b)[NJ], f32x4 (&c)[NJ])
{
    mma_small(a, b, c);
#pragma unroll
    for (int j = 0; j < NJ; ++j) c[j] = mma16(a.p[0], b[j].p[0], c[j]);
}

// A [ROWS][D] float tile as three bf16 planes in LDS, each laid out like a DirectTile<D, ROWS>.
template <int D, int THREADS = 256>
struct PlaneTile {
    static constexpr int ROWS = D == 64 ? 64 : 32;      // two tensors' planes: 48 KB
    static constexpr int CPR = D / 8, NT = THREADS, CHUNKS = ROWS * CPR / NT;       // 8-element chunks per row; per thread
    static constexpr int PLANE = ROWS * D * 2, BYTES = 3 * PLANE;
    static_assert(ROWS * CPR % NT == 0, "");
    static __device__ __forceinline__ int chunk_offset(int r, int c) { return r * (D * 2) + ((c ^ tile_swizzle<D>(r)) * 16); }
    struct Regs { f32x4 v[2 * CHUNKS]; };
    // `word` (in LDS) becomes 1 where a thread's part of two tiles holds tiny values; everybody may read it after the tiles' barrier
    static __device__ __forceinline__ void note_tiny(const Regs &a, const Regs &b, uint32_t *word)
    {
        if (__any(least_magnitude(b.v, least_magnitude(a.v, INFINITY)) < kTiny))
            if (some_below(a.v, kTiny) || some_below(b.v, kTiny)) *word = 1u;
    }
    // rows >= rows_ok re-read row rows_ok - 1 (the kernels mask or discard what they produce)
    static __device__ __forceinline__ void fetch(Regs &g, const float *base, int64_t ld, int rows_ok, int tid)
    {
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) {
            const int c = i * NT + tid;
            const f32x4 *p = reinterpret_cast<const f32x4 *>(base + (int64_t)min(c / CPR, rows_ok - 1) * ld + (c % CPR) * 8);
            g.v[2 * i] = p[0];
            g.v[2 * i + 1] = p[1];
        }
    }
    static __device__ __forceinline__ void store(char *tile, const Regs &g, int tid)
    {
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) {
            const int c = i * NT + tid;
            float x[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) { x[e] = g.v[2 * i][e]; x[4 + e] = g.v[2 * i + 1][e]; }
            const Frag3 f = split8(x);
#pragma unroll
            for (int p = 0; p < 3; ++p) *reinterpret_cast<bf16x8 *>(tile + p * PLANE + chunk_offset(c / CPR, c % CPR)) = f.p[p].v;
        }
    }
    // A-operand fragment of rows [row0, row0 + 16)
    static __device__ __forceinline__ Frag3 rows_frag(const char *tile, int row0, int off)
    {
        Frag3 f;
#pragma unroll
        for (int p = 0; p < 3; ++p) f.p[p] = load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(tile + p * PLANE + row0 * (D * 2) + off));
        return f;
    }
    // 32 tile rows against the operand `b` over the whole width: every step's small products first, the
    // large ones at the end, so that the sum is rounded at its full size D / 32 times and not six times as often
    // (scores and dP enter differences of large terms).
    // Operands are read one step ahead of their use: `ahead` holds those of the first step on entry, and what `next` reads on return.
    template <int NJ, typename Next>
    static __device__ __forceinline__ Block<NJ> product(const char *tile, int row0, const int (&off)[D / 32], const Frag3 (&b)[D / 32][NJ], Frag3 &ahead,
                                                        Next &&next)
    {
        constexpr int NS = D / 32;
        Block<NJ> c;
        Frag<bf16_t> high[NS];
#pragma unroll
        for (int u = 0; u < 2 * NS; ++u) {
            const int i = u / NS, ks = u % NS;
            const Frag3 a = ahead;
            ahead = u + 1 < 2 * NS ? rows_frag(tile, row0 + 16 * ((u + 1) / NS), off[(u + 1) % NS]) : next();
            __builtin_amdgcn_sched_barrier(0);
            if (ks == 0)
#pragma unroll
                for (int j = 0; j < NJ; ++j) c.v[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            high[ks] = a.p[0];
            mma_small(a, b[ks], c.v[i]);
            if (ks == NS - 1) {
#pragma unroll
                for (int k2 = 0; k2 < NS; ++k2)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) c.v[i][j] = mma16(high[k2], b[k2][j].p[0], c.v[i][j]);
            }
        }
        return c;
    }
    // ... of the transposed tile: rows [row0, row0 + 32) are the contraction slots (load_frag_tr16_sw)
    static __device__ __forceinline__ Frag3 cols_frag(const char *tile, int row0, int off)
    {
        Frag3 f;
#pragma unroll
        for (int p = 0; p < 3; ++p) f.p[p] = load_frag_tr16_sw<D>(tile + p * PLANE, row0, off);
        return f;
    }
    // put(db, 16 columns of the transposed tile), each read one ahead, likewise
    template <typename Put, typename Next>
    static __device__ __forceinline__ void columns(const char *tile, int row0, const int (&off)[D / 16], Frag3 &ahead, Put &&put, Next &&next)
    {
#pragma unroll
        for (int db = 0; db < D / 16; ++db) {
            const Frag3 a = ahead;
            ahead = db + 1 < D / 16 ? cols_frag(tile, row0, off[db + 1]) : next();
            put(db, a);
            if (db & 1) __builtin_amdgcn_sched_barrier(0);
        }
    }
};

constexpr int kRowsPerWg = 128;             // query rows of a workgroup: four wavefronts of 32
// Keys of a dK/dV workgroup: 128, a block of 32 per wavefront; or (HALVES = 2, d = 64) two blocks of 32, each held by
// two wavefronts that take one of the two 32-row halves of every Q/dO tile and add their results up at the end --
// twice as many workgroups, with chains half as long, for launches that do not fill the chip.
template <int HALVES> constexpr int kKeysPerWg = 128 / HALVES;

// Blocks of 16 keys or query rows that a wavefront of a backward workgroup holds.  At d = 128 one, eight wavefronts per workgroup:
// with two a wavefront needs 440 registers and is alone on its SIMD, vector work and matrix instructions take turns.  54 launches,
// forward and backward, 3.4 % faster on average, 14 % at best, never 1 % slower (1024 rows behind 7168, 8 heads, dropout: backward
// 618 -> 594 us).
template <int D> constexpr int kBlocks = D == 64 ? 2 : 1;

// lse * log2 e less its rounded value l2 (1.93e-8: what kLog2e was rounded off by); 0 for infinities and NaNs
__device__ __forceinline__ float rounded_off(float lse, float l2)
{
    const float r = fmaf(lse, kLog2e, -l2) + lse * 1.925963e-8f;
    return fabsf(r) < 1.f ? r : 0.f;
}

// A wavefront's sums, transposed: 16 columns x 16 rows (or keys) each
template <int D, int NJ> struct Sums {
    f32x4 v[D / 16][NJ];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int db = 0; db < D / 16; ++db)
#pragma unroll
            for (int j = 0; j < NJ; ++j) v[db][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
};

// ---- The products on the fp32 matrix cores, operands straight from memory, for what three bf16 parts miss: `tiny` inputs,
// and infinities, NaNs and values whose first part overflows (3.39e38), which all leave NaN in the results (an infinite x has
// x - x0 = NaN).  A wavefront with such results, or with results so small that parts of the weights
// were subnormal, does its rows or keys over again this way, without LDS or barriers (1024 rows against 8192 keys, 16 heads:
// forward 206 us, over again 622; backward 556 and 1866).  Finding out costs 1.5 % of lx8k and 3 us of a launch of few tiles.

// 32 rows of a matrix (this lane's two, at a + ao) against 16 NJ others (b + bo) over the whole width
template <int D, int NJ>
__device__ __forceinline__ Block<NJ> product_f32(const float *a, const int64_t (&ao)[2], const float *b, const int64_t (&bo)[NJ])
{
    Block<NJ> c;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) c.v[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int ks = 0; ks < D / 32; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    c.v[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ao[i] + ks * 32 + e], b[bo[j] + ks * 32 + e], c.v[i][j], 0, 0, 0);
    return c;
}
// acc += transpose of 32 rows (from `rows` on, rows_ok of which exist) x the weights w
template <int D, int NJ>
__device__ __forceinline__ void add_product_f32(const float *rows, int64_t ld, int rows_ok, const Block<NJ> &w, Sums<D, NJ> &acc, int lq, int g)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int row = 16 * (e >> 2) + 4 * g + (e & 3);
        const float *const p = rows + (int64_t)min(row, rows_ok - 1) * ld + lq;
#pragma unroll
        for (int db = 0; db < D / 16; ++db) {
            const uint32_t x = __builtin_bit_cast(uint32_t, p[db * 16]) & (row < rows_ok ? ~0u : 0u);       // 0 past the end
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                acc.v[db][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, x), w.v[e >> 2][j][e & 3], acc.v[db][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);      // (a row at a time: its registers must not add to the main loop's)
    }
}
// Whether some result is not finite, or below 2^-100 and not 0 (again looked at closely only where the least magnitude is small)
template <int D, int NJ>
__device__ __forceinline__ bool missed(const Sums<D, NJ> &acc)
{
    float least = INFINITY, zero = 0.f;
    bool small = false;
#pragma unroll
    for (int n = 0; n < D / 16 * NJ; ++n) {
        const f32x4 a = acc.v[n / NJ][n % NJ];
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
            asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(least) : "v"(a[e]), "v"(a[e + 1]));
            zero = __builtin_fmaf(a[e], 0.f, zero);                     // NaN from infinities and NaNs on
            zero = __builtin_fmaf(a[e + 1], 0.f, zero);
        }
    }
    if (__any(least < 0x1p-100f)) {
        uint32_t least_nonzero = ~0u;
#pragma unroll
        for (int n = 0; n < D / 16 * NJ; ++n)
#pragma unroll
            for (int e = 0; e < 4; ++e) least_nonzero = min(least_nonzero, twice_magnitude(acc.v[n / NJ][n % NJ][e]) - 1u);
        small = least_nonzero < twice_magnitude(0x1p-100f) - 1u;
    }
    return small || zero != zero;
}

// ------------------------------------------------------------------------------------------ forward
template <int D, bool DROP>
__global__ __launch_bounds__(256, D == 64 ? 3 : 2) void fwd_f32_kernel(SegShape s, DropArgs dr, const float *__restrict__ q,
                                                         const float *__restrict__ k, const float *__restrict__ v,
                                                         float *__restrict__ out, float *__restrict__ lse,
                                                         float *__restrict__ o_part, float *__restrict__ lse_part, int n_splits,
                                                         int n_q_tiles)
{
    using Tile = PlaneTile<D>;
    constexpr int NS = D / 32, BC = Tile::ROWS;
    __shared__ __attribute__((aligned(1024))) char smem[2 * Tile::BYTES + 16];
    char *const sk = smem, *const sv = smem + Tile::BYTES;
    uint32_t *const tiny_word = reinterpret_cast<uint32_t *>(smem + 2 * Tile::BYTES);

    const int tid = threadIdx.x, lane = tid & 63, lq = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bhs = s.B * s.H;
    int bh, inner;
    if (!xcd_item(blockIdx.x, bhs, n_q_tiles * n_splits, s.causal && s.s0 < s.l_s, bh, inner)) return;
    const int b = bh / s.H, h = bh % s.H, split = inner / n_q_tiles;
    const int r0 = (n_q_tiles - 1 - inner % n_q_tiles) * kRowsPerWg, rw0 = r0 + wave * 32;
    const int64_t ld = (int64_t)s.H * D;

    // the keys any row of this tile sees, and this split's share of their tiles
    const int r_last = min(r0 + kRowsPerWg, s.l_s) - 1;
    const int kv_end = s.causal ? (int)min<int64_t>(s.l_x, s.s0 + r_last + 1) : s.l_x;
    const int n_tiles = (kv_end + BC - 1) / BC, per = (n_tiles + n_splits - 1) / n_splits;
    const int t_begin = split * per, t_end = min(n_tiles, t_begin + per);

    // this lane's two query rows, r + 16 j; rows past the segment re-read its last row and are never stored
    const int r = rw0 + lq;
    Frag3 qf[NS][2];
    const float *const qp = q + (int64_t)b * s.l_s * ld + (int64_t)h * D + g * 8;
    const bool tiny = split_rows<D, 2>(qp, {min(r, s.l_s - 1) * ld, min(r + 16, s.l_s - 1) * ld}, qf);
    if (tid == 0) *tiny_word = 0u;
    Sums<D, 2> o;
    o.clear();
    float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f};     // running maximum (log2 domain); this lane's quarter of the row sum
    const float c = kLog2e / sqrtf((float)D);
    uint32_t drop_rk[2] = {0u, 0u}, drop_cs = 0u;
    if (DROP) {
        drop_cs = drop_col_seed(dr.seed_hi);
#pragma unroll
        for (int j = 0; j < 2; ++j) drop_rk[j] = drop_row_key(dr.seed_lo, (uint32_t)bh, (uint32_t)(s.s0 + r + 16 * j));
    }

    const float *kbase = k + (int64_t)b * s.l_x * ld + (int64_t)h * D, *vbase = v + (int64_t)b * s.l_x * ld + (int64_t)h * D;
    int a_off[NS], t_off[D / 16];
#pragma unroll
    for (int ks = 0; ks < NS; ++ks) a_off[ks] = Tile::chunk_offset(lq, 4 * ks + g);
#pragma unroll
    for (int db = 0; db < D / 16; ++db) t_off[db] = tr16_lane_offset_sw<D>(lane, db);

    // keys [jb, jb + 32): in half kb2 of the tile in LDS, or (EXACT) in memory
    auto block = [&](auto exact, int jb, int kb2) __attribute__((always_inline)) {
        constexpr bool EXACT = decltype(exact)::value;
        // a block no row of this wavefront sees
        if (jb >= s.l_x || (s.causal && jb > (int)s.s0 + rw0 + 31)) return;
        Block<2> sc;
        Frag3 ahead;
        if constexpr (EXACT) {
            sc = product_f32<D, 2>(kbase, {(int64_t)min(jb + lq, s.l_x - 1) * ld + g * 8, (int64_t)min(jb + 16 + lq, s.l_x - 1) * ld + g * 8}, qp,
                                   {min(r, s.l_s - 1) * ld, min(r + 16, s.l_s - 1) * ld});
        } else {
            ahead = Tile::rows_frag(sk, kb2 * 32, a_off[0]);
            sc = Tile::product(sk, kb2 * 32, a_off, qf, ahead, [&] { return Tile::cols_frag(sv, kb2 * 32, t_off[0]); });
        }
        // element (i, e) of this lane is key jb + 16 i + 4 g + e
        if ((s.causal && jb + 31 > (int)s.s0 + rw0) || jb + 32 > s.l_x) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int last = s.causal ? min((int)s.s0 + r + 16 * j, s.l_x - 1) : s.l_x - 1, rel = last - jb - 4 * g;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (16 * (e >> 2) + (e & 3) > rel) sc.v[e >> 2][j][e & 3] = -INFINITY;
            }
        }
        // The weights subtract the running maximum as it stands, until one would exceed 2^8 (or a row sees its first key): then it is
        // raised to the exact one and what was accumulated is rescaled.  (The division by the row sum, which uses the
        // same m, makes the result independent of when m was raised.  EXACT keeps all weights at 1 or below, so that sums of values
        // near the largest float stay finite.)
        float mx[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            mx[j] = sc.v[0][j][0];
#pragma unroll
            for (int e = 1; e < 8; ++e) mx[j] = fmaxf(mx[j], sc.v[e >> 2][j][e & 3]);
            mx[j] *= c;
        }
        constexpr float kOver = EXACT ? 0.f : 8.f;
        if (__any(mx[0] > m[0] + kOver || mx[1] > m[1] + kOver)) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                mx[j] = fmaxf(mx[j], __shfl_xor(mx[j], 16));
                const float m_new = fmaxf(m[j], fmaxf(mx[j], __shfl_xor(mx[j], 32)));
                const float alpha = m_new > m[j] ? fast_exp2(m[j] - m_new) : 1.f;
                l[j] *= alpha;
#pragma unroll
                for (int db = 0; db < D / 16; ++db)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o.v[db][j][e] *= alpha;
                m[j] = m_new;
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float m_use = m[j] == -INFINITY ? 0.f : m[j];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float p = fast_exp2(sc.v[e >> 2][j][e & 3] * c - m_use);
                l[j] += p;          // the row sum (hence lse and the normalisation) is that of the softmax
                if (DROP) {
                    const int key = jb + 16 * (e >> 2) + 4 * g + (e & 3);
                    p = drop_keep(drop_rk[j], drop_col_key(drop_cs, (uint32_t)key), dr.thr) ? p * dr.scale : 0.f;
                }
                sc.v[e >> 2][j][e & 3] = p;
            }
        }
        if constexpr (EXACT) {
            add_product_f32<D>(vbase + (int64_t)jb * ld, ld, s.l_x - jb, sc, o, lq, g);
        } else {
            const Frag3 pf[2] = {split_acc(sc, 0), split_acc(sc, 1)};
            Tile::columns(sv, kb2 * 32, t_off, ahead, [&](int db, const Frag3 &a) __attribute__((always_inline)) { mma6(a, pf, o.v[db]); },
                          [&] { return ahead; });
        }
    };
    for (int t = t_begin; t < t_end; ++t) {
        {
            typename Tile::Regs gk, gv;
            Tile::fetch(gk, kbase + (int64_t)t * BC * ld, ld, s.l_x - t * BC, tid);
            Tile::fetch(gv, vbase + (int64_t)t * BC * ld, ld, s.l_x - t * BC, tid);
            __syncthreads();                    // the tile before has been read
            Tile::store(sk, gk, tid);
            Tile::store(sv, gv, tid);
            Tile::note_tiny(gk, gv, tiny_word);
        }
        __syncthreads();
        if (rw0 >= s.l_s) continue;             // none of this wavefront's rows exists
#pragma unroll
        for (int kb2 = 0; kb2 < BC / 32; ++kb2) block(std::false_type{}, t * BC + kb2 * 32, kb2);
    }
    if (rw0 < s.l_s && t_begin < t_end && (tiny || __builtin_amdgcn_readfirstlane((int)*tiny_word) != 0 || __any(missed(o)))) {
        o.clear();
        m[0] = m[1] = -INFINITY;
        l[0] = l[1] = 0.f;
        for (int jb = t_begin * BC; jb < t_end * BC; jb += 32) block(std::true_type{}, jb, 0);
    }

#pragma unroll
    for (int j = 0; j < 2; ++j) {
        float l_tot = l[j] + __shfl_xor(l[j], 16);
        l_tot += __shfl_xor(l_tot, 32);
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        const float lse_nat = l_tot > 0.f ? (m[j] + log2f(l_tot)) * kLn2 : -INFINITY;
        const int rj = r + 16 * j;
        if (rj >= s.l_s) continue;
        const int64_t row = ((int64_t)split * bhs + bh) * s.l_s + rj;
        float *op = n_splits == 1 ? out + ((int64_t)b * s.l_s + rj) * ld + (int64_t)h * D : o_part + row * D;
#pragma unroll
        for (int db = 0; db < D / 16; ++db) {
            const f32x4 a = o.v[db][j];
            *reinterpret_cast<f32x4 *>(op + db * 16 + 4 * g) = f32x4{a[0] * inv, a[1] * inv, a[2] * inv, a[3] * inv};
        }
        if (g == 0) {
            if (n_splits == 1) lse[(int64_t)bh * s.l_s + rj] = lse_nat;
            else lse_part[row] = lse_nat;
        }
    }
}

// ------------------------------------------------------------------------------------------ dQ
// S^T = K Q^T, dP^T = V dO^T, dS = P (dP - D) (dropout: P (M dP - D)), dQ^T += K^T dS^T.
template <int D, bool DROP>
__device__ __forceinline__ void bwd_dq_f32_body(char *smem, const SegShape &s, const DropArgs &dr, const float *__restrict__ q,
                                                const float *__restrict__ k, const float *__restrict__ v,
                                                const float *__restrict__ dO, const float *__restrict__ lse,
                                                const float *__restrict__ Dv, float *__restrict__ dq, float *__restrict__ dq_part,
                                                int n_splits, int q_tile, int n_q_tiles, int bh, int split)
{
    constexpr int NJ = kBlocks<D>;
    using Tile = PlaneTile<D, 512 / NJ>;
    constexpr int NS = D / 32, BC = Tile::ROWS;
    char *const sk = smem, *const sv = smem + Tile::BYTES;
    uint32_t *const tiny_word = reinterpret_cast<uint32_t *>(smem + 2 * Tile::BYTES);
    const int tid = threadIdx.x, lane = tid & 63, lq = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = bh / s.H, h = bh % s.H;
    const int r0 = (n_q_tiles - 1 - q_tile) * kRowsPerWg, rw0 = r0 + wave * 16 * NJ;
    const int64_t ld = (int64_t)s.H * D;
    const int r_last = min(r0 + kRowsPerWg, s.l_s) - 1;
    const int kv_end = s.causal ? (int)min<int64_t>(s.l_x, s.s0 + r_last + 1) : s.l_x;
    const int n_tiles = (kv_end + BC - 1) / BC, per = (n_tiles + n_splits - 1) / n_splits;
    const int t_begin = split * per, t_end = min(n_tiles, t_begin + per);

    // this lane's rows, r + 16 j; rows past the segment re-read its last row, get lse = +inf (P = dS = 0) and are never stored
    const int r = rw0 + lq;
    Frag3 qf[NS][NJ], gf[NS][NJ];
    bool tiny;
    {
        const int64_t head = (int64_t)b * s.l_s * ld + (int64_t)h * D + g * 8;
        int64_t off[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) off[j] = head + min(r + 16 * j, s.l_s - 1) * ld;
        tiny = split_rows<D, NJ>(q, off, qf);
        tiny = split_rows<D, NJ>(dO, off, gf) || tiny;
    }
    float L2[NJ], Dr[NJ], scale[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int rc = min(r + 16 * j, s.l_s - 1);
        const float lv = lse[(int64_t)bh * s.l_s + rc], l2 = lv * kLog2e;
        L2[j] = r + 16 * j < s.l_s ? l2 : INFINITY;
        Dr[j] = Dv[(int64_t)bh * s.l_s + rc];
        // (what l2 was rounded off by is a factor of all the row's weights, hence of its result: dq's error 4.3e-7 -> 3.4e-7)
        scale[j] = (1.f - rounded_off(lv, l2) * kLn2) / sqrtf((float)D);
    }
    if (tid == 0) *tiny_word = 0u;
    const float c = kLog2e / sqrtf((float)D);
    uint32_t drop_rk[NJ], drop_cs = 0u;
    if (DROP) {
        drop_cs = drop_col_seed(dr.seed_hi);
#pragma unroll
        for (int j = 0; j < NJ; ++j) drop_rk[j] = drop_row_key(dr.seed_lo, (uint32_t)bh, (uint32_t)(s.s0 + r + 16 * j));
    }

    Sums<D, NJ> acc;
    acc.clear();
    const float *kbase = k + (int64_t)b * s.l_x * ld + (int64_t)h * D, *vbase = v + (int64_t)b * s.l_x * ld + (int64_t)h * D;
    int a_off[NS], t_off[D / 16];
#pragma unroll
    for (int ks = 0; ks < NS; ++ks) a_off[ks] = Tile::chunk_offset(lq, 4 * ks + g);
#pragma unroll
    for (int db = 0; db < D / 16; ++db) t_off[db] = tr16_lane_offset_sw<D>(lane, db);

    // keys [jb, jb + 32): in half kb2 of the tile in LDS, or (EXACT) in memory
    auto block = [&](auto exact, int jb, int kb2) __attribute__((always_inline)) {
        constexpr bool EXACT = decltype(exact)::value;
        if (jb >= s.l_x || (s.causal && jb > (int)s.s0 + rw0 + 16 * NJ - 1)) return;
        Block<NJ> sc, dp;
        Frag3 ahead;
        if constexpr (EXACT) {
            int row = r;
            asm volatile("" : "+v"(row));      // (so that its address is made here, not kept through the main loop)
            const int64_t key_at[2] = {(int64_t)min(jb + lq, s.l_x - 1) * ld + g * 8, (int64_t)min(jb + 16 + lq, s.l_x - 1) * ld + g * 8};
            const int64_t head = (int64_t)b * s.l_s * ld + (int64_t)h * D + g * 8;
            int64_t row_at[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) row_at[j] = head + min(row + 16 * j, s.l_s - 1) * ld;
            sc = product_f32<D, NJ>(kbase, key_at, q, row_at);
            dp = product_f32<D, NJ>(vbase, key_at, dO, row_at);
        } else {
            ahead = Tile::rows_frag(sk, kb2 * 32, a_off[0]);
            sc = Tile::product(sk, kb2 * 32, a_off, qf, ahead, [&] { return Tile::rows_frag(sv, kb2 * 32, a_off[0]); });
            dp = Tile::product(sv, kb2 * 32, a_off, gf, ahead, [&] { return ahead; });
        }
        if ((s.causal && jb + 31 > (int)s.s0 + rw0) || jb + 32 > s.l_x) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int last = s.causal ? min((int)s.s0 + r + 16 * j, s.l_x - 1) : s.l_x - 1, rel = last - jb - 4 * g;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (16 * (e >> 2) + (e & 3) > rel) sc.v[e >> 2][j][e & 3] = -INFINITY;
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t ck = DROP ? drop_col_key(drop_cs, (uint32_t)(jb + 16 * (e >> 2) + 4 * g + (e & 3))) : 0u;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const float p = fast_exp2(sc.v[e >> 2][j][e & 3] * c - L2[j]);
                float dpe = dp.v[e >> 2][j][e & 3];
                if (DROP) dpe = drop_keep(drop_rk[j], ck, dr.thr) ? dpe * dr.scale : 0.f;
                dp.v[e >> 2][j][e & 3] = p * (dpe - Dr[j]);
            }
            if (DROP && (e & 1)) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (EXACT) {
            add_product_f32<D>(kbase + (int64_t)jb * ld, ld, s.l_x - jb, dp, acc, lq, g);
        } else {
            // The block's 32 keys are added up before they meet the accumulator, which is rounded at its full size once
            // per block and not six times.
            Frag3 df[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) df[j] = split_acc(dp, j);
            ahead = Tile::cols_frag(sk, kb2 * 32, t_off[0]);
            f32x4 sum[2][NJ];
            auto add = [&](int db) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc.v[db][j][e] += sum[db & 1][j][e];
            };
            Tile::columns(sk, kb2 * 32, t_off, ahead, [&](int db, const Frag3 &a) __attribute__((always_inline)) {
                #pragma unroll
                for (int j = 0; j < NJ; ++j) sum[db & 1][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                mma6(a, df, sum[db & 1]);
                if (db > 0) add(db - 1);        // (not the one just issued: its result would be waited for)
            }, [&] { return ahead; });
            add(D / 16 - 1);
        }
    };
    for (int t = t_begin; t < t_end; ++t) {
        const int j0 = t * BC;
        typename Tile::Regs gk, gv;
        Tile::fetch(gk, kbase + (int64_t)j0 * ld, ld, s.l_x - j0, tid);
        Tile::fetch(gv, vbase + (int64_t)j0 * ld, ld, s.l_x - j0, tid);
        __syncthreads();
        Tile::store(sk, gk, tid);
        Tile::store(sv, gv, tid);
        Tile::note_tiny(gk, gv, tiny_word);
        __syncthreads();
        if (rw0 >= s.l_s) continue;
#pragma unroll
        for (int kb2 = 0; kb2 < BC / 32; ++kb2) block(std::false_type{}, j0 + kb2 * 32, kb2);
    }
    if (rw0 < s.l_s && t_begin < t_end && (tiny || __builtin_amdgcn_readfirstlane((int)*tiny_word) != 0 || __any(missed(acc)))) {
        acc.clear();
        for (int jb = t_begin * BC; jb < t_end * BC; jb += 32) block(std::true_type{}, jb, 0);
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int rj = r + 16 * j;
        if (rj >= s.l_s) continue;
        float *dst = (n_splits == 1 ? dq : dq_part + (int64_t)split * s.B * s.l_s * ld) + ((int64_t)b * s.l_s + rj) * ld + (int64_t)h * D;
#pragma unroll
        for (int db = 0; db < D / 16; ++db) {
            const f32x4 a = acc.v[db][j];
            *reinterpret_cast<f32x4 *>(dst + db * 16 + 4 * g) = f32x4{a[0] * scale[j], a[1] * scale[j], a[2] * scale[j], a[3] * scale[j]};
        }
    }
}

// ------------------------------------------------------------------------------------------ dK, dV
// Key-owned: S = Q K^T, dP = dO V^T over the query tiles that see the keys, then dV^T += dO^T P, dK^T += Q^T dS.
template <int D, bool DROP, int HALVES>
__device__ __forceinline__ void bwd_dkv_f32_body(char *smem, const SegShape &s, const DropArgs &dr, const float *__restrict__ q,
                                                 const float *__restrict__ k, const float *__restrict__ v,
                                                 const float *__restrict__ dO, const float *__restrict__ lse,
                                                 const float *__restrict__ Dv, float *__restrict__ dk_part,
                                                 float *__restrict__ dv_part, int bh, int key_tile)
{
    constexpr int NJ = kBlocks<D>;
    using Tile = PlaneTile<D, 512 / NJ>;
    constexpr int NS = D / 32, BQ = Tile::ROWS;
    char *const sq = smem, *const sg = smem + Tile::BYTES;
    float *const sl = reinterpret_cast<float *>(smem + 2 * Tile::BYTES), *const sd = sl + 64;
    uint32_t *const sr = reinterpret_cast<uint32_t *>(sd + 64), *const tiny_word = sr + 128;
    const int tid = threadIdx.x, lane = tid & 63, lq = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = bh / s.H, h = bh % s.H;
    constexpr int KEYS = kKeysPerWg<HALVES>;
    static_assert(HALVES == 1 || (BQ == 64 && NJ == 2), "");
    const int key_block = wave / HALVES, my_half = wave % HALVES;
    const int j0 = key_tile * KEYS, jw0 = j0 + key_block * 16 * NJ, key0 = jw0 + lq;
    const int64_t ld = (int64_t)s.H * D, kv_base = (int64_t)b * s.l_x * ld + (int64_t)h * D;

    if (s.causal && j0 >= s.s0 + s.l_s) {       // no query of the segment sees this tile: zeros, or (whole 128-key tiles) left unwritten
        if (s.skip_tail && j0 / 128 * 128 >= s.s0 + s.l_s) return;
        constexpr int F4 = D / 4;
        for (int i = tid; i < KEYS * F4; i += Tile::NT) {
            const int row = j0 + i / F4, c4 = (i % F4) * 4;
            if (row < s.l_x) {
                *reinterpret_cast<f32x4 *>(dk_part + kv_base + (int64_t)row * ld + c4) = f32x4{0.f, 0.f, 0.f, 0.f};
                *reinterpret_cast<f32x4 *>(dv_part + kv_base + (int64_t)row * ld + c4) = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
        return;
    }
    // first query row that sees any key of this tile
    int rq_begin = 0;
    if (s.causal) rq_begin = (int)min<int64_t>(max<int64_t>((int64_t)j0 - s.s0, 0), s.l_s) / BQ * BQ;

    // this lane's keys, key0 + 16 j; keys past the sequence re-read its last row and are never stored
    Frag3 kf[NS][NJ], vf[NS][NJ];
    bool tiny;
    {
        int64_t off[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) off[j] = kv_base + (int64_t)min(key0 + 16 * j, s.l_x - 1) * ld + g * 8;
        tiny = split_rows<D, NJ>(k, off, kf);
        tiny = split_rows<D, NJ>(v, off, vf) || tiny;
    }
    if (tid == 0) *tiny_word = 0u;
    Sums<D, NJ> dk, dv;
    dk.clear();
    dv.clear();
    const float c = kLog2e / sqrtf((float)D);
    const float *qbase = q + (int64_t)b * s.l_s * ld + (int64_t)h * D, *gbase = dO + (int64_t)b * s.l_s * ld + (int64_t)h * D;
    uint32_t drop_ck[NJ];
    if (DROP)
#pragma unroll
        for (int j = 0; j < NJ; ++j) drop_ck[j] = drop_col_key(drop_col_seed(dr.seed_hi), (uint32_t)(key0 + 16 * j));
    int a_off[NS], t_off[D / 16];
#pragma unroll
    for (int ks = 0; ks < NS; ++ks) a_off[ks] = Tile::chunk_offset(lq, 4 * ks + g);
#pragma unroll
    for (int db = 0; db < D / 16; ++db) t_off[db] = tr16_lane_offset_sw<D>(lane, db);

    // rows [rb, rb + 32) of the segment: block qb of the tile in LDS, or (EXACT) in memory
    auto block = [&](auto exact, int rb, int qb) __attribute__((always_inline)) {
        constexpr bool EXACT = decltype(exact)::value;
        // a block none of whose rows sees a key of this wavefront, or past the segment
        if (rb >= s.l_s || (s.causal && (int)s.s0 + rb + 31 < jw0)) return;
        Block<NJ> sc, dp;
        Frag3 ahead;
        if constexpr (EXACT) {
            int key = key0;
            asm volatile("" : "+v"(key));      // (so that its address is made here, not kept through the main loop)
            const int64_t row_at[2] = {(int64_t)min(rb + lq, s.l_s - 1) * ld + g * 8, (int64_t)min(rb + 16 + lq, s.l_s - 1) * ld + g * 8};
            int64_t key_at[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) key_at[j] = kv_base + (int64_t)min(key + 16 * j, s.l_x - 1) * ld + g * 8;
            sc = product_f32<D, NJ>(qbase, row_at, k, key_at);
            dp = product_f32<D, NJ>(gbase, row_at, v, key_at);
        } else {
            ahead = Tile::rows_frag(sq, qb * 32, a_off[0]);
            sc = Tile::product(sq, qb * 32, a_off, kf, ahead, [&] { return Tile::rows_frag(sg, qb * 32, a_off[0]); });
            dp = Tile::product(sg, qb * 32, a_off, vf, ahead, [&] { return ahead; });
        }
        const bool diag = s.causal && jw0 + 16 * NJ - 1 > (int)s.s0 + rb;
        // element (i, e) of this lane is row rb + 16 i + 4 g + e
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int rl = qb * 32 + 16 * i + 4 * g, r4 = rb + 16 * i + 4 * g;          // in the tile; in the segment
            f32x4 l4, d4, lo4;
            if constexpr (EXACT) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int64_t at = (int64_t)bh * s.l_s + min(r4 + e, s.l_s - 1);
                    const float lv = lse[at], l2 = lv * kLog2e;
                    l4[e] = r4 + e < s.l_s ? l2 : INFINITY;
                    lo4[e] = rounded_off(lv, l2);
                    d4[e] = Dv[at];
                }
            } else {
                l4 = *reinterpret_cast<const f32x4 *>(sl + rl);
                d4 = *reinterpret_cast<const f32x4 *>(sd + rl);
                lo4 = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(sr) + 64 + rl);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t rk = !DROP ? 0u : EXACT ? drop_row_key(dr.seed_lo, (uint32_t)bh, (uint32_t)(s.s0 + r4 + e)) : sr[rl + e];
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    float p = fast_exp2(fmaf(sc.v[i][j][e], c, -l4[e]) - lo4[e]);
                    if (diag && key0 + 16 * j > (int)s.s0 + r4 + e) p = 0.f;
                    float pv = p, dpe = dp.v[i][j][e];
                    if (DROP) {
                        const float mk = drop_keep(rk, drop_ck[j], dr.thr) ? dr.scale : 0.f;
                        pv = p * mk;
                        dpe *= mk;
                    }
                    sc.v[i][j][e] = pv;
                    dp.v[i][j][e] = p * (dpe - d4[e]);
                }
                if (DROP && (e & 1)) __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (EXACT || D == 64) __builtin_amdgcn_sched_barrier(0);     // (one row block at a time: 1 and 3 spills instead of 12 and 7)
        }
        if constexpr (EXACT) {
            add_product_f32<D>(gbase + (int64_t)rb * ld, ld, s.l_s - rb, sc, dv, lq, g);
            add_product_f32<D>(qbase + (int64_t)rb * ld, ld, s.l_s - rb, dp, dk, lq, g);
        } else {
            ahead = Tile::cols_frag(sg, qb * 32, t_off[0]);
            Frag3 wf[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) wf[j] = split_acc(sc, j);
            Tile::columns(sg, qb * 32, t_off, ahead, [&](int db, const Frag3 &a) __attribute__((always_inline)) { mma6(a, wf, dv.v[db]); },
                          [&] { return Tile::cols_frag(sq, qb * 32, t_off[0]); });
#pragma unroll
            for (int j = 0; j < NJ; ++j) wf[j] = split_acc(dp, j);
            Tile::columns(sq, qb * 32, t_off, ahead, [&](int db, const Frag3 &a) __attribute__((always_inline)) { mma6(a, wf, dk.v[db]); },
                          [&] { return ahead; });
        }
    };
    for (int rq0 = rq_begin; rq0 < s.l_s; rq0 += BQ) {
        typename Tile::Regs gq, gg;
        Tile::fetch(gq, qbase + (int64_t)rq0 * ld, ld, s.l_s - rq0, tid);
        Tile::fetch(gg, gbase + (int64_t)rq0 * ld, ld, s.l_s - rq0, tid);
        __syncthreads();
        Tile::store(sq, gq, tid);
        Tile::store(sg, gg, tid);
        Tile::note_tiny(gq, gg, tiny_word);
        if (tid < BQ) {     // rows past the segment: lse = +inf makes P (hence dS) exactly 0
            const int rr = rq0 + tid;
            const float lv = lse[(int64_t)bh * s.l_s + min(rr, s.l_s - 1)], l2 = lv * kLog2e, off_by = rounded_off(lv, l2);
            sl[tid] = rr < s.l_s ? l2 : INFINITY;
            reinterpret_cast<float *>(sr)[64 + tid] = off_by;   // subtracted too: dk's and dv's errors fall by 4 to 20 %, for 1 % of lx8k
            sd[tid] = rr < s.l_s ? Dv[(int64_t)bh * s.l_s + rr] : 0.f;
            if (DROP) sr[tid] = drop_row_key(dr.seed_lo, (uint32_t)bh, (uint32_t)(s.s0 + rr));
        }
        __syncthreads();
#pragma nounroll      // (unrolled, the kernel with dropout spills 40 registers, against 3)
        for (int qi = 0; qi < BQ / 32 / HALVES; ++qi) {
            const int qb = HALVES == 1 ? qi : my_half;
            block(std::false_type{}, rq0 + 32 * qb, qb);
        }
    }
    tiny = tiny || (rq_begin < s.l_s && __builtin_amdgcn_readfirstlane((int)*tiny_word) != 0);
    if constexpr (HALVES == 2) {        // second half's results -> first half's wavefront, through the planes' LDS
        static_assert(2 * 2 * (D / 8) * 1024 <= 2 * Tile::BYTES, "");
        __syncthreads();
        auto at = [&](int n) { return reinterpret_cast<f32x4 *>(smem + (key_block * 2 * (D / 8) + n) * 1024 + lane * 16); };
        if (my_half == 1)
#pragma unroll
            for (int n = 0; n < D / 8; ++n) {
                *at(2 * n) = dk.v[n >> 1][n & 1];
                *at(2 * n + 1) = dv.v[n >> 1][n & 1];
            }
        __syncthreads();
        if (my_half == 1) return;
#pragma unroll
        for (int n = 0; n < D / 8; ++n) {
            const f32x4 a = *at(2 * n), d = *at(2 * n + 1);
#pragma unroll
            for (int e = 0; e < 4; ++e) { dk.v[n >> 1][n & 1][e] += a[e]; dv.v[n >> 1][n & 1][e] += d[e]; }
        }
    }
    if (jw0 < s.l_x && (tiny || __any(missed(dk) || missed(dv)))) {
        dk.clear();
        dv.clear();
        for (int rb = rq_begin; rb < s.l_s; rb += 32) block(std::true_type{}, rb, 0);
    }
    const float scale = 1.f / sqrtf((float)D);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        if (key0 + 16 * j >= s.l_x) continue;
        const int64_t off = kv_base + (int64_t)(key0 + 16 * j) * ld + 4 * g;
#pragma unroll
        for (int db = 0; db < D / 16; ++db) {
            const f32x4 a = dk.v[db][j];
            *reinterpret_cast<f32x4 *>(dk_part + off + db * 16) = f32x4{a[0] * scale, a[1] * scale, a[2] * scale, a[3] * scale};
            *reinterpret_cast<f32x4 *>(dv_part + off + db * 16) = dv.v[db][j];
        }
    }
}

// Both kinds of workgroup in one launch, dQ first, in XCD order: see bwd_main_bf16_kernel.
template <int D, bool DROP, int HALVES>
__global__ __launch_bounds__(512 / kBlocks<D>, 2) void bwd_main_f32_kernel(
    SegShape s, DropArgs dr, const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v,
    const float *__restrict__ dO, const float *__restrict__ lse, const float *__restrict__ Dv, float *__restrict__ dq,
    float *__restrict__ dq_part, float *__restrict__ dk_part, float *__restrict__ dv_part, int n_splits, int n_dq, int n_q_tiles,
    int n_key_tiles)
{
    __shared__ __attribute__((aligned(1024))) char smem[2 * PlaneTile<D>::BYTES + 4 * 64 * 4 + 16];
    const int bhs = s.B * s.H, id = blockIdx.x;
    int bh, inner;
    if (id >= n_dq) {
        if (!xcd_item(id - n_dq, bhs, n_key_tiles, s.causal, bh, inner)) return;
        bwd_dkv_f32_body<D, DROP, HALVES>(smem, s, dr, q, k, v, dO, lse, Dv, dk_part, dv_part, bh, inner);
    } else {
        if (!xcd_item(id, bhs, n_q_tiles * n_splits, s.causal && s.s0 < s.l_s, bh, inner)) return;
        bwd_dq_f32_body<D, DROP>(smem, s, dr, q, k, v, dO, lse, Dv, dq, dq_part, n_splits, inner % n_q_tiles, n_q_tiles, bh,
                                 inner / n_q_tiles);
    }
}

template <int D>
hipError_t launch_fwd_d(const SegShape &s, const DropArgs &dr, const float *q, const float *k, const float *v, float *out,
                        float *lse, const Workspace &ws, int n_splits, hipStream_t st)
{
    const int n_q_tiles = (s.l_s + kRowsPerWg - 1) / kRowsPerWg;
    const auto kernel = dr.thr != 0 ? fwd_f32_kernel<D, true> : fwd_f32_kernel<D, false>;
    TimedLaunch tl(K_FWD_F32, st);
    hipLaunchKernelGGL(kernel, dim3((unsigned)xcd_grid(s.B * s.H, n_q_tiles * n_splits)), dim3(256), 0, st, s, dr, q, k, v, out, lse,
                       ws.o_part, ws.lse_part, n_splits, n_q_tiles);
    return hipGetLastError();
}
template <int D>
hipError_t launch_bwd_d(const SegShape &s, const DropArgs &dr, const float *q, const float *k, const float *v, const float *lse,
                        const float *dO, float *dq, float *dk_part, float *dv_part, const Workspace &ws, int n_splits, hipStream_t st)
{
    const bool halves = f32_bwd_halves(s, n_splits);
    const int keys = halves ? 64 : 128, n_q_tiles = (s.l_s + kRowsPerWg - 1) / kRowsPerWg, n_key_tiles = (s.l_x + keys - 1) / keys;
    const int n_dq = xcd_grid(s.B * s.H, n_q_tiles * n_splits), n_dkv = xcd_grid(s.B * s.H, n_key_tiles);
    constexpr int H2 = D == 64 ? 2 : 1;
    const auto kernel = dr.thr != 0 ? (halves ? bwd_main_f32_kernel<D, true, H2> : bwd_main_f32_kernel<D, true, 1>)
                                    : (halves ? bwd_main_f32_kernel<D, false, H2> : bwd_main_f32_kernel<D, false, 1>);
    TimedLaunch tl(K_BWD_MAIN_F32, st);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(n_dq + n_dkv)), dim3(512 / kBlocks<D>), 0, st, s, dr, q, k, v, dO, lse, ws.D, dq, ws.dq_part, dk_part,
                       dv_part, n_splits, n_dq, n_q_tiles, n_key_tiles);
    return hipGetLastError();
}

} // namespace

int f32_rows_per_workgroup() { return kRowsPerWg; }

// Two wavefronts per key block where a dK/dV workgroup's walk over the queries is what the launch waits for: the key
// tiles fit the chip about once (two workgroups per compute unit) and a dQ workgroup does not walk much longer.  2048 rows,
// 8 heads, 2048 keys: 214 -> 148 us; but 600 rows, 4 heads, 8192 keys 109 -> 119 (dQ walks 16 tiles, the queries are 10), 64
// rows against 1664 key tiles 103 -> 121.  On 156 launches (64..2048 rows, 2..96 heads, 100..1700 key tiles) the
// rule costs 0.9 % over the better choice on average; never 2.3 %, always 3.4 %.
bool f32_bwd_halves(const SegShape &s, int n_splits)
{
    const int64_t seen = s.causal && s.s0 + s.l_s < s.l_x ? s.s0 + s.l_s : (int64_t)s.l_x;
    const int64_t dq_tiles = ((seen + 63) / 64 + n_splits - 1) / n_splits;
    return s.d == 64 && (seen + 127) / 128 * s.B * s.H <= 640 && 4 * ((s.l_s + 63) / 64) >= 3 * dq_tiles;
}

hipError_t launch_fwd_f32_main(const SegShape &s, const DropArgs &drop, const float *q, const float *k, const float *v, float *out,
                               float *lse, const Workspace &ws, int n_splits, hipStream_t st)
{
    if (s.d == 64) return launch_fwd_d<64>(s, drop, q, k, v, out, lse, ws, n_splits, st);
    return launch_fwd_d<128>(s, drop, q, k, v, out, lse, ws, n_splits, st);
}

// dQ and the dK/dV partials in one launch; the caller has run the row-dot kernel and runs the dQ split merge
hipError_t launch_bwd_f32_main(const SegShape &s, const DropArgs &drop, const float *q, const float *k, const float *v,
                               const float *lse, const float *dO, float *dq, float *dk_part, float *dv_part, const Workspace &ws,
                               int n_splits, hipStream_t st)
{
    if (s.d == 64) return launch_bwd_d<64>(s, drop, q, k, v, lse, dO, dq, dk_part, dv_part, ws, n_splits, st);
    return launch_bwd_d<128>(s, drop, q, k, v, lse, dO, dq, dk_part, dv_part, ws, n_splits, st);
}

} // namespace lss
