// The linear maps either side of the segment attention, in the fused-communication form of
// Section 3, Principle 3 (Fig. 2(ii), (iii), (v)), as bf16 matrix-core GEMMs for gfx950:
//     forward   Q_i = x_i W_q (the segment's own rows),  [K | V] = x [W_k | W_v] (gathered sequence)
//     backward  dx_q = dQ_i W_q^T,  dx_partial = dK_part W_k^T + dV_part W_v^T
// dx_partial is what the segment sum (the reduce-scatter's arithmetic) then adds over segments.
//
// One kernel template computes C[m, n] = sum_k A[m, k] W'[k, n] for a short list of jobs.  A
// workgroup owns a TM x TN tile of C, held transposed in the accumulators (lane = row m of A, as the
// attention kernels hold one query per lane): C^T += W'^T A^T, so the weights are the A operand of the
// matrix instruction and the activations its B operand.  Each wavefront owns a WM x WN part.  The
// contraction runs in tiles of 64 through a ring of STAGES LDS slots that are filled global -> LDS
// directly, one barrier per tile.  The finished tile goes through LDS once more so that it is written to
// memory as whole rows.  The tile is chosen per launch (pick_gemm_tile): 2048 x 512 -> 2048 takes 17.8 us in
// 256 x 256 tiles and 9.8 as chosen, 2048 x 2048 -> 512 44.1 and 14.2 (in a graph, behind a kernel that writes their operand).
// Matrix instructions of 16 x 16 x 32, not 32 x 32 x 16: loops on Gaussian operands (lss_microbench, section 7) reach 1700 TFLOP/s
// with the former and 1630 with the latter in registers, 1500 and 1445 with an LDS read per 65,536 flop.  16384 x 4096 -> 1024:
// 128 -> 116 us, 16384 x 1024 -> 4096: 146 -> 136, the contraction of 98304 x 2048 floats 581 -> 532; weight gradients of
// 16384 rows 148 -> 138, all of these with 256 x 256 tiles as eight wavefronts held them (gemm_wide_loop has what they take now).  Launches of 10 to 25 us gain
// 1 % and weight gradients among them lose up to 4 %.
//   W_TR   weights stored [k][n] (forward: W as given).  Their fragments come from the LDS tile
//          by transposing reads; otherwise the weights are stored [n][k] (backward: W as given
//          IS W'^T) and are read plainly.
//   OUT_F32  C is written as float (the backward maps, whose results are summed over segments
//          afterwards), else rounded once to bf16.
//   A_ANY  a job's A may be float (the dK/dV partials; `a_f32` of the job): rounded to bf16 on the
//          way into LDS, through registers; the contraction index runs over dK's columns, then
//          dV's.  Jobs with bf16 A (dQ) share the launch.
#include "lss_bf16.h"
#include "lss_gemm_plan.h"
#include "lss_kernels.h"

#include <algorithm>
#include <type_traits>
#include <vector>

namespace lss {

namespace {

constexpr int PK = kGemmK;                      // contraction tile
constexpr int kLdsPerCu = 160 * 1024;

// A workgroup's tile of C, its wavefronts' parts and its ring.  KG > 1: KG groups of wavefronts, each with a
// ring of its own, take every KG-th contraction tile and add their results up (in group order) at the end.
template <int TM_, int TN_, int WM_, int WN_, int STAGES_, int KG_ = 1>
struct GemmShape {
    static constexpr bool WIDE = false;
    static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, STAGES = STAGES_, KG = KG_;
    static constexpr int MW = TM / WM, NW = TN / WN, GW = MW * NW;      // wavefronts of a group
    static constexpr int WAVES = KG * GW, NT = 64 * WAVES, GT = 64 * GW;
    static constexpr int MB = WM / 16, NB = WN / 16;            // accumulator blocks of a wavefront
    static constexpr int HB = MB < 4 ? MB : 4;                  // row blocks of a step: at most 4 x 4 fragments are held twice
    static constexpr int MH = MB / HB, STEPS = PK / 32 * MH;    // steps per contraction tile
    static constexpr int ABYTES = TM * PK * 2, WBYTES = TN * PK * 2, SLOT = ABYTES + WBYTES, RING = STAGES * SLOT;
    static constexpr int LDS = KG * RING;
    static constexpr int PER_CU = kLdsPerCu / LDS;              // workgroups a compute unit holds at once
    static constexpr int WAVES_PER_SIMD = PER_CU * WAVES / 4;   // what the register count has to allow
    static_assert(STAGES >= 2 && LDS <= kLdsPerCu && (KG - 1) * GW * MB * NB * 1024 <= LDS && STEPS % 2 == 0, "");
};

// The 256 x 256 tile: four wavefronts of 128 x 128, one per SIMD, which take all 512 registers of theirs (the accumulators are half of them).  A
// compute unit's LDS serves 128 bytes a cycle; eight wavefronts of 128 x 64 read 24 KB a piece per contraction tile, and with the 64 KB that the loads
// write that is 2048 cycles, as many as the matrix instructions take.  Four of 128 x 128 read 128 KB in all.  Three slots for the activations, which
// come from memory, two for the weights, which other workgroups have just read: all 160 KB.
struct GemmWide {
    static constexpr bool WIDE = true;
    static constexpr int TM = 256, TN = 256, WM = 128, WN = 128, KG = 1;
    static constexpr int MW = TM / WM, NW = TN / WN, GW = MW * NW;
    static constexpr int WAVES = GW, NT = 64 * WAVES, GT = NT;
    static constexpr int MB = WM / 16, NB = WN / 16;
    static constexpr int A_SLOTS = 3, W_SLOTS = 2;
    static constexpr int ABYTES = TM * PK * 2, WBYTES = TN * PK * 2, W_RING = A_SLOTS * ABYTES, LDS = W_RING + W_SLOTS * WBYTES;
    static constexpr int PER_CU = 1, WAVES_PER_SIMD = 1;
    static_assert(LDS <= kLdsPerCu && MB == 8 && NB == 8 && PK == 64, "");
};

struct ProjJob {
    const void *a0, *a1;        // A: [batches][rows][lda]; a1 serves contraction indices >= k_split (or is unused)
    const bf16_t *w;            // weights, row stride ldw
    void *c0, *c1;              // C: [batches][rows][ldc]; columns >= n_split go to c1 (column n - n_split)
    int64_t a_batch_stride, c_batch_stride;     // elements
    int rows, rows_ok;          // rows per batch; leading rows of A that hold data (the rest count as 0)
    int batches, N, K, k_split, n_split, ldw;
    int a_f32;                  // A is float (only in kernels compiled with A_ANY)
    int wg_begin, m_data, n_tiles;              // first workgroup id of the job; row tiles with data per batch; column tiles
};
// What happens to a finished bf16 tile on its way to memory (the feed-forward unit, whose GeLU
// would otherwise be a pass over memory of its own):
//   EPI_GELU       C is written to c0 and GeLU(C), of the rounded C, to c1 (same layout)
//   EPI_GELU_BWD   C, rounded, is multiplied by GeLU'(U) before it is written; U = a1, laid out like C
enum { EPI_NONE = 0, EPI_GELU = 1, EPI_GELU_BWD = 2 };

struct ProjArgs {
    ProjJob job[2];
    int n_jobs, lda, ldc, skip_tail;
    int stream;                 // C is written past the caches (gemm_streams)
    // rows of job 0 that have no data (the others have none): first workgroup id, workgroups per batch and column tile, end of the rows to clear
    int zero_begin, zero_tiles, zero_end;
};

// Operand tile [64 k][COLS], to be read transposed.  Loaded directly like a DirectTile.  Its rows start
// at the same LDS bank (COLS >= 128) or alternate between two or four (COLS = 64, 32), so the 16-byte chunk c of row
// r sits at chunk position c ^ swizzle(r): the rows of which one transposing read takes 32 bytes each (four
// consecutive ones per 16 lanes, eight further down the next four) then spread evenly over the 64 banks.
template <int COLS, int WAVES>
struct TrTile {
    static constexpr int CPR = COLS / 8;                        // 16-byte chunks per row
    static constexpr int NI = PK * CPR / 64 / WAVES;            // load instructions per wavefront
    static_assert(PK * CPR % (64 * WAVES) == 0 && NI >= 1, "");
    static __device__ __forceinline__ int swizzle(int r)
    {
        return (COLS >= 128 ? 4 * (r & 3) : COLS == 64 ? 4 * ((r >> 1) & 1) : 0) ^ (2 * ((r >> 3) & 1));
    }
    static __device__ __forceinline__ int row_of(int i, int wave, int lane) { return ((i * WAVES + wave) * 64 + lane) / CPR; }
    // chunks >= chunks_ok (columns past the matrix) re-read chunk chunks_ok - 1; rows >= rows_ok re-read row
    // rows_ok - 1
    static __device__ __forceinline__ void offsets(uint32_t (&off)[NI], int ldw, int wave, int lane, int chunks_ok,
                                                   int rows_ok = PK)
    {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int row = row_of(i, wave, lane), pos = lane % CPR;
            const int chunk = min(pos ^ swizzle(row), chunks_ok - 1);
            off[i] = ((uint32_t)min(row, rows_ok - 1) * (uint32_t)ldw + (uint32_t)chunk * 8u) * 2u;
        }
    }
    static __device__ __forceinline__ int chunk_offset(int r, int c) { return r * (COLS * 2) + ((c ^ swizzle(r)) * 16); }
    // Transposing reads (see load_frag_tr_sw for the instruction's lane mapping): lane s of group g of 16 lanes
    // addresses row 8 g + s / 4 and the 8-byte piece s % 4 of the 32 bytes of column block nb (16 columns).
    static __device__ __forceinline__ int lane_offset(int lane, int nb)
    {
        const int g = lane >> 4, s = lane & 15;
        return chunk_offset(8 * g + (s >> 2), 2 * nb + ((s & 3) >> 1)) + (s & 1) * 8;
    }
    // Operand fragment of the transposed tile for contraction step ks: operand row = column
    // (lane % 16) of block nb, slot e = contraction index 32 ks + 8 (lane / 16) + e -- the order in which a
    // plain 16-byte read delivers the other operand.  (Rows 32 and 4 further down keep the permutation.)
    static __device__ __forceinline__ Frag<bf16_t> load_frag(const char *tile, int ks, int lane_off)
    {
        const char *p = tile + ks * 32 * (COLS * 2) + lane_off;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * (COLS * 2)));
        const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        Frag<bf16_t> f;
        f.v = __builtin_bit_cast(bf16x8, both);
        return f;
    }
};

// Operand fragments, two sets: step j (contraction index 32 (j / MH), row blocks HB (j % MH) ..) uses fb[j % 2] and
// fw[(j / MH) % 2]
template <typename S>
struct GemmFrags { Frag<bf16_t> fb[2][S::HB], fw[2][S::NB]; };

// The contraction.  Tile i of this wavefront's group (contraction tile g + KG i) is multiplied from slot
// i % STAGES, in steps of 32 indices and at most four row blocks.  Operand fragments are read from LDS one step ahead of their
// matrix instructions, across tiles too: the barrier that publishes the next tile stands before the last step
// of the current one, so that the reads of the next tile's first fragments -- every wavefront's at once,
// right after the barrier -- run under that step's matrix instructions.  (With the barrier at the end of the
// tile the matrix cores idled through them: a quarter of a 256 x 256 workgroup's time.)  Behind that
// barrier no wavefront reads the current tile any more: its slot takes the tile STAGES further on.
//   issue(t, slot)       starts the direct loads of contraction tile t: LOADS instructions
//   load(slot, j, f)     reads the fragments that step j needs and step j - 1 did not
//   publish(t, slot)     what is left to do for tile t before the barrier that publishes it, its loads having landed
//   fetch(t)             REGS: starts the loads of the part of tile t that travels through registers, before those of issue(t)
//   stash(t, slot)       REGS: writes it to LDS, before issue(t)'s loads are waited for (with both the other way round
//                        a launch of 8192 x 2048 floats takes 63 us instead of 57)
//   WAIT                 the last step's fragments are waited for ahead of the branch around the barrier, as the barrier does anyway: the compiler's
//                        own wait, behind the branch, is one for the next tile's fragments too, and those reads would not run under the
//                        step.  80 drawn feed-forward units and projections: forward maps 0.5 to 1 % faster, bf16 input gradients 0.3 %; none
//                        for the weight gradients, which lose 0.3 %, and floats (no difference), whose LDS writes it would hold up
template <typename S, int LOADS, bool WAIT, typename Issue, typename Load, typename Publish, typename Fetch, typename Stash>
__device__ __forceinline__ void gemm_loop(f32x4 (&acc)[S::MB][S::NB], int T, int group, bool regs, Issue &&issue, Load &&load,
                                          Publish &&publish, Fetch &&fetch, Stash &&stash)
{
    const int iters = (T + S::KG - 1) / S::KG, mine = (T - group + S::KG - 1) / S::KG;      // tiles of the longest and of this group
    auto tile = [&](int i) { return group + S::KG * i; };
    // all but the loads of the `ahead` tiles issued last have landed (REGS: all)
    auto landed = [&](int ahead_have, auto ahead) {
        if (!regs && ahead_have >= decltype(ahead)::value) wait_vmem<decltype(ahead)::value * LOADS>();
        else wait_vmem_all();
    };
    using std::integral_constant;
#pragma unroll
    for (int i = 0; i < S::STAGES; ++i)
        if (i < mine) issue(tile(i), i);
    if (regs && mine > 0) { fetch(tile(0)); stash(tile(0), 0); }
    landed(mine - 1, integral_constant<int, S::STAGES - 1>{});
    if (mine > 0) publish(tile(0), 0);
    __syncthreads();
    if (regs && mine > 1) fetch(tile(1));
    GemmFrags<S> f;
    auto multiply = [&](int j) __attribute__((always_inline)) {
#pragma unroll
        for (int mb = 0; mb < S::HB; ++mb)
#pragma unroll
            for (int nb = 0; nb < S::NB; ++nb) {
                f32x4 &c = acc[j % S::MH * S::HB + mb][nb];
                c = mma16(f.fw[j / S::MH & 1][nb], f.fb[j & 1][mb], c);
            }
#pragma unroll
        for (int i = 0; i < S::HB * S::NB; ++i) {       // a matrix instruction, a read of the next step's, ...
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    if (S::KG == 1 || mine > 0) load(0, 0, f);
    int slot = 0;
    for (int i = 0; i < iters; ++i) {
        const int nxt = slot + 1 == S::STAGES ? 0 : slot + 1;
        const bool busy = S::KG == 1 || i < mine;
        if (busy) {
#pragma unroll
            for (int j = 0; j + 1 < S::STEPS; ++j) {
                load(slot, j + 1, f);
                multiply(j);
            }
        }
        if constexpr (WAIT) wait_lds_reads();
        if (i + 1 < iters) {
            const bool more = S::KG == 1 || i + 1 < mine;
            if (regs && more) stash(tile(i + 1), nxt);
            landed(mine - 2 - i, integral_constant<int, S::STAGES - 2>{});
            if (more) publish(tile(i + 1), nxt);
            if (regs && i + 2 < mine) fetch(tile(i + 2));
            __syncthreads();
            if (i + S::STAGES < mine) issue(tile(i + S::STAGES), slot);
            if (more) load(nxt, 0, f);
        }
        if (busy) multiply(S::STEPS - 1);
        slot = nxt;
    }
}
// The contraction of a GemmWide tile.  A contraction tile is two phases of 32 indices, 64 matrix instructions each, between which everything else is
// placed one by one: a wavefront alone on its SIMD hides what it issues between two of them and nothing else.  Phase 0 of tile t multiplies the fragments read ahead and
// reads those of phase 1; then comes the barrier that publishes tile t + 1, behind which no wavefront reads tile t any more, and phase 1 reads the first fragments
// of t + 1.  Tile t + 2 of A is requested in phase 0 (its slot was tile t - 1's), that of the weights in phase 1 (tile t's own slot).
//   issue_a(t, slot, i), issue_w(t, slot, i)    load instruction i of a wavefront's NI
//   load_a(slot, ks, mb), load_w(slot, ks, nb)  a fragment of phase ks
//   publish(t, aslot, wslot)                    what is left to do for tile t before the barrier that publishes it
//   REG: the operand that is float and travels through registers instead, in CHUNKS parts of two 16-byte loads per lane: in phase 0 of tile t part c of
//   tile t + 1 is converted and written to LDS (stash(t + 1, slot, c)) and that of t + 2 requested in its place (fetch(t + 2, c)), a whole tile ahead
// The matrix instructions are assembly, with accumulators in the accumulation half of the registers: left to itself the compiler rotates the accumulators through
// the register file, 132 copies per 128 matrix instructions.  An accumulator comes up again 64 instructions later; the wait states before other instructions may read
// one stand at the end.
// Behind a copy that writes the operand, against eight wavefronts of 128 x 64 whose loads started all at once behind one barrier per tile, two slots for either
// operand: 16384 x 4096 -> 1024 104 -> 95 us, 16384 x 1024 -> 4096 125 -> 111, their input gradients 104 -> 94 and 120 -> 106, 8192 x 8192 -> 8192 797 -> 720
// (1530 TFLOP/s), its gradients 790 -> 709 and 849 -> 773; projections of 4 x 24576 rows 435 -> 370.
enum WideReg { REG_NONE, REG_A, REG_W };
struct WideFrags { Frag<bf16_t> a[GemmWide::MB], w[GemmWide::NB]; };
template <WideReg REG, int A_NI, int W_NI, int CHUNKS, typename IssueA, typename IssueW, typename LoadA, typename LoadW, typename Publish, typename Fetch,
          typename Stash>
__device__ __forceinline__ void gemm_wide_loop(f32x4 (&acc)[GemmWide::MB][GemmWide::NB], int T, IssueA &&issue_a, IssueW &&issue_w, LoadA &&load_a,
                                               LoadW &&load_w, Publish &&publish, Fetch &&fetch, Stash &&stash)
{
    using S = GemmWide;
    constexpr int SLOTS = S::MB * S::NB, READS = S::MB + S::NB;
    constexpr bool DIRECT_A = REG != REG_A, DIRECT_W = REG != REG_W;
    constexpr int FETCHES = REG == REG_NONE ? 0 : 2 * CHUNKS;
    constexpr int A_LOADS = DIRECT_A ? A_NI : 0, W_LOADS = DIRECT_W ? W_NI : 0;
    auto issue_all = [&](int t) __attribute__((always_inline)) {
        if constexpr (DIRECT_A)
#pragma unroll
            for (int i = 0; i < A_NI; ++i) issue_a(t, t, i);
        if constexpr (DIRECT_W)
#pragma unroll
            for (int i = 0; i < W_NI; ++i) issue_w(t, t, i);
    };
    auto fetch_all = [&](int t) __attribute__((always_inline)) {
        if constexpr (REG != REG_NONE)
#pragma unroll
            for (int c = 0; c < CHUNKS; ++c) fetch(t, c);
    };
    fetch_all(0);
    issue_all(0);
    if (T > 1) issue_all(1);
    // Cleared while the loads are on their way, by the shortest matrix instruction that writes four registers (of zeros).  Left to the compiler that is 256
    // vector instructions behind the barrier, 0.8 us of a lone wavefront's time, and in the weight gradients as many copies of a cleared register again.
    float zero;
    asm volatile("v_mov_b32 %0, 0\n\ts_nop 1" : "=v"(zero));
#pragma unroll
    for (int mb = 0; mb < S::MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < S::NB; ++nb) asm volatile("v_mfma_f32_4x4x1_16b_f32 %0, %1, %1, 0" : "=a"(acc[mb][nb]) : "v"(zero));
    if constexpr (REG != REG_NONE)
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) stash(0, 0, c);
    if (T > 1) {
        fetch_all(1);
        wait_vmem<A_LOADS + W_LOADS + FETCHES>();
    } else wait_vmem_all();
    publish(0, 0, 0);
    __syncthreads();
    WideFrags f[2];
#pragma unroll
    for (int i = 0; i < S::NB; ++i) f[0].w[i] = load_w(0, 0, i);
#pragma unroll
    for (int i = 0; i < S::MB; ++i) f[0].a[i] = load_a(0, 0, i);
    int a_slot = 0, w_slot = 0;
    // AHEAD: there is a tile t + 2, NEXT: a tile t + 1
    auto tile = [&](int t, auto ahead, auto next) __attribute__((always_inline)) {
        constexpr bool AHEAD = decltype(ahead)::value, NEXT = decltype(next)::value;
        const int a_next = a_slot == 2 ? 0 : a_slot + 1, a_free = a_slot == 0 ? 2 : a_slot - 1, w_next = w_slot ^ 1;
#pragma unroll
        for (int ph = 0; ph < 2; ++ph) {
            if (ph == 1 && NEXT) {
                wait_lds_reads();
                if constexpr (AHEAD) wait_vmem<A_LOADS + FETCHES>();        // (all but what phase 0 has requested of tile t + 2)
                else wait_vmem_all();
                publish(t + 1, a_next, w_next);
                __syncthreads();
            }
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) {
                const int mb = s / S::NB, nb = s % S::NB;
                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[mb][nb]) : "v"(f[ph].w[nb].v), "v"(f[ph].a[mb].v));
                if ((ph == 0 || NEXT) && s % 2 == 0 && s / 2 < READS) {
                    const int r = s / 2;
                    if (r < S::NB) f[ph ^ 1].w[r] = load_w(ph == 0 ? w_slot : w_next, ph ^ 1, r);
                    else f[ph ^ 1].a[r - S::NB] = load_a(ph == 0 ? a_slot : a_next, ph ^ 1, r - S::NB);
                }
                if constexpr (REG != REG_NONE) {
                    constexpr int PER = SLOTS / CHUNKS;
                    if (ph == 0 && NEXT && s % PER == PER - 1) {
                        stash(t + 1, REG == REG_A ? a_next : w_next, s / PER);
                        if (AHEAD) fetch(t + 2, s / PER);
                    }
                }
                if (DIRECT_A && AHEAD && ph == 0 && s % (SLOTS / A_NI) == SLOTS / A_NI / 2 + 1) issue_a(t + 2, a_free, s / (SLOTS / A_NI));
                if (DIRECT_W && AHEAD && ph == 1 && s % (SLOTS / W_NI) == SLOTS / W_NI / 2 + 1) issue_w(t + 2, w_slot, s / (SLOTS / W_NI));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        a_slot = a_next;
        w_slot = w_next;
    };
    int t = 0;
    for (; t + 2 < T; ++t) tile(t, std::true_type{}, std::true_type{});
    if (t + 1 < T) tile(t++, std::false_type{}, std::true_type{});
    tile(t, std::false_type{}, std::false_type{});
#pragma unroll
    for (int mb = 0; mb < S::MB; ++mb)
        asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[mb][0]), "+a"(acc[mb][1]), "+a"(acc[mb][2]), "+a"(acc[mb][3]), "+a"(acc[mb][4]), "+a"(acc[mb][5]),
                     "+a"(acc[mb][6]), "+a"(acc[mb][7]));
}
// Adds the groups' accumulators up into group 0's, in group order, through the (now free) LDS.
template <typename S>
__device__ __forceinline__ void gemm_add_groups(char *smem, f32x4 (&acc)[S::MB][S::NB], int group, int gwave, int lane)
{
    if constexpr (S::KG > 1) {
        constexpr int BLOCKS = S::MB * S::NB;
        auto at = [&](int g, int blk) {
            return reinterpret_cast<f32x4 *>(smem + (((g - 1) * S::GW + gwave) * BLOCKS + blk) * 1024 + lane * 16);
        };
        __syncthreads();
#pragma unroll
        for (int blk = 0; blk < BLOCKS; ++blk)
            if (group > 0) *at(group, blk) = acc[blk / S::NB][blk % S::NB];
        __syncthreads();
        if (group == 0) {
#pragma unroll
            for (int g = 1; g < S::KG; ++g)
#pragma unroll
                for (int blk = 0; blk < BLOCKS; ++blk) {
                    const f32x4 v = *at(g, blk);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[blk / S::NB][blk % S::NB][e] += v[e];
                }
        }
    }
}
template <typename S>
__device__ __forceinline__ void gemm_clear(f32x4 (&acc)[S::MB][S::NB])
{
#pragma unroll
    for (int mb = 0; mb < S::MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < S::NB; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[mb][nb][e] = 0.f;
}

// The finished tile -> LDS, from where every wavefront reads whole row pieces: the 16-byte chunk c of row m sits at chunk position c ^ (m % chunks per row).
// Accumulator block (mb, nb), element v of a lane: row m = WM wm + 16 mb + lane % 16, column n = WN wn +
// 16 nb + 4 (lane / 16) + v.  ZEROS: rows >= rows_data are written as zeros.
template <typename S, bool OUT_F32, bool ZEROS>
struct GemmStore {
    static constexpr int EB = OUT_F32 ? 4 : 2, CW = 16 / EB, CPR = S::TN / CW;      // bytes per element, columns per chunk, chunks per row
    static_assert(S::TM * S::TN * EB <= S::LDS && S::NT % CPR == 0, "");
    static constexpr int ROWS_PER_IT = S::NT / CPR, ITS = (S::TM + ROWS_PER_IT - 1) / ROWS_PER_IT;
    static __device__ __forceinline__ int offset(int m, int c) { return m * (S::TN * EB) + ((c ^ (m & (CPR - 1))) * 16); }
    static __device__ __forceinline__ void to_lds(char *smem, const f32x4 (&acc)[S::MB][S::NB], int wm, int wn, int lane, int rows_data)
    {
        const int c_first = wn * S::WN / CW;
#pragma unroll
        for (int mb = 0; mb < S::MB; ++mb) {
            const int m = S::WM * wm + 16 * mb + (lane & 15), g = lane >> 4;
            const bool data = m < rows_data;
#pragma unroll
            for (int nb = 0; nb < S::NB; ++nb) {
                f32x4 val = acc[mb][nb];
                if (ZEROS && !data) val = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (OUT_F32)
                    *reinterpret_cast<f32x4 *>(smem + offset(m, c_first + 4 * nb + g)) = val;
                else
                    *reinterpret_cast<bf16x4 *>(smem + offset(m, c_first + 2 * nb + (g >> 1)) + (g & 1) * 8) = pack4(val[0], val[1], val[2], val[3]);
            }
        }
    }
};

// A finished GemmWide tile goes out in four quarters of 64 rows, 32 from either pair of wavefronts, through two regions of LDS by turns: a quarter's stores
// are on their way while the next one is converted, and one barrier per quarter will do.  (In one piece, or floats in halves by columns, which left two of the
// four wavefronts idle at a time, a tile took 2.1 us to get into LDS and 3.1 out of it, one after the other.)
//   put(m, raw)        16 bytes of row m; their column is CW (t % CPR)
template <bool OUT_F32, bool ZEROS>
struct WideStore {
    using S = GemmWide;
    static constexpr int EB = OUT_F32 ? 4 : 2, CW = 16 / EB, CPR = S::TN / CW;      // bytes per element, columns per chunk, chunks per row
    static constexpr int REGION = 64 * S::TN * EB, ITS = 64 * CPR / S::NT, RPI = S::NT / CPR;
    static_assert(2 * REGION <= S::LDS, "");
    static __device__ __forceinline__ int offset(int r, int c) { return r * (S::TN * EB) + ((c ^ (r & (CPR - 1))) * 16); }
    template <typename Put>
    static __device__ __forceinline__ void store(char *smem, const f32x4 (&acc)[S::MB][S::NB], int wm, int wn, int t, int rows_data, Put &&put)
    {
        const int lane = t & 63, g = lane >> 4;
        __syncthreads();        // every wavefront is done with what the LDS held
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            char *const region = smem + (q & 1) * REGION;
            auto row = [&](int k) { const int r = k * RPI + t / CPR; return S::WM * (r >> 5) + 32 * q + (r & 31); };
#pragma unroll
            for (int mb = 2 * q; mb < 2 * q + 2; ++mb) {
                const int r = 32 * wm + 16 * (mb & 1) + (lane & 15);
                const bool data = S::WM * wm + 16 * mb + (lane & 15) < rows_data;
#pragma unroll
                for (int nb = 0; nb < S::NB; ++nb) {
                    f32x4 val = acc[mb][nb];
                    if (ZEROS && !data) val = f32x4{0.f, 0.f, 0.f, 0.f};
                    const int c = (S::WN * wn + 16 * nb) / CW;
                    if constexpr (OUT_F32) *reinterpret_cast<f32x4 *>(region + offset(r, c + g)) = val;
                    else *reinterpret_cast<bf16x4 *>(region + offset(r, c + (g >> 1)) + (g & 1) * 8) = pack4(val[0], val[1], val[2], val[3]);
                }
            }
            __syncthreads();
            f32x4 raw[8];
#pragma unroll
            for (int k = 0; k < ITS; ++k) {
                if (k % 8 == 0) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) raw[i] = *reinterpret_cast<const f32x4 *>(region + offset((k + i) * RPI + t / CPR, t % CPR));
#pragma unroll
                    for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(raw[i]));        // (not read one by one, each ahead of its store)
                }
                put(row(k), raw[k % 8]);
            }
        }
    }
};

// STREAMS: whether args.stream may be set (not where launches are small)
template <typename S, bool A_ANY, bool W_TR, bool OUT_F32, int EPI, bool STREAMS>
__device__ __forceinline__ void proj_gemm_body(const ProjArgs &args)
{
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    using OutT = typename std::conditional<OUT_F32, float, bf16_t>::type;
    using ATile = DirectTile<PK, S::TM, S::GW>;         // activations [TM m][64 k]
    using WPlain = DirectTile<PK, S::TN, S::GW>;        // weights [TN n][64 k]
    using WTr = TrTile<S::TN, S::GW>;                   // weights [64 k][TN n]
    constexpr int W_NI = W_TR ? WTr::NI : WPlain::NI, LOADS = ATile::NI + W_NI;     // load instructions per wavefront and tile
    static_assert(EPI == EPI_NONE || !OUT_F32, "the GeLU epilogues work on bf16 results");

    const int tid = threadIdx.x, lane = tid & 63;
    const int all_waves = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = all_waves / S::GW, wave = all_waves % S::GW, gtid = tid % S::GT;     // wave, gtid: within the group
    const int wm = wave % S::MW, wn = wave / S::MW;

    int ji = 0;
    if (args.n_jobs > 1 && (int)blockIdx.x >= args.job[1].wg_begin && (int)blockIdx.x < args.zero_begin) ji = 1;
    const ProjJob &J = args.job[ji];
    // Row tiles with data first, of all batches and jobs, then those without, each kind spread over all XCDs: with 28 % of two
    // batches' rows valid (59,486 x 1024 floats) a plain numbering left all products to three or four of the
    // eight XCDs, 375 us.
    const bool data = !A_ANY || (int)blockIdx.x < args.zero_begin;      // (no other product has rows without data)
    const int per_batch = data ? J.m_data : args.zero_tiles;
    const TileId tile = xcd_tile(blockIdx.x - (data ? J.wg_begin : args.zero_begin), J.batches * per_batch, J.n_tiles);
    if (!tile.ok) return;
    const int batch = tile.m / per_batch, n0 = tile.n * S::TN;
    const int m0 = data ? tile.m % per_batch * S::TM : J.m_data * S::TM + tile.m % per_batch * gemm_zero_rows(S::TM, S::TN);

    const int rows_here = data ? min(J.rows - m0, S::TM) : min(args.zero_end - m0, gemm_zero_rows(S::TM, S::TN));      // rows of C this workgroup owns
    const int rows_data = min(min(J.rows, J.rows_ok) - m0, S::TM);      // of which this many have data in A
    const int cols_here = min(J.N - n0, S::TN);                         // a multiple of 32

    // (copies: the loads' assembly counts as a write to memory, after which what is read through `J` is fetched again, by scalar loads that a
    // finished tile would wait for before its first store: 1 % of all launches)
    const int ldc = args.ldc, n_split = J.n_split;
    int stream = STREAMS ? args.stream : 0;
    asm("" : "+s"(stream));
    const int64_t c_tile0 = (int64_t)batch * J.c_batch_stride + (int64_t)m0 * ldc;
    OutT *const c0 = static_cast<OutT *>(J.c0) + c_tile0, *const c1 = static_cast<OutT *>(J.c1) + c_tile0;
    const bf16_t *const gelu_u = static_cast<const bf16_t *>(J.a1) + c_tile0;         // (EPI_GELU_BWD)

    auto put16 = [&](void *to, f32x4 v) __attribute__((always_inline)) {
        if (STREAMS && stream) {
            asm volatile("");       // (two stores that differ in this respect only are merged into one plain store, ahead of the branch or behind it)
            __builtin_nontemporal_store(v, static_cast<f32x4 *>(to));
            asm volatile("");
        } else *static_cast<f32x4 *>(to) = v;
    };
    if (!data) {
        constexpr int CW = OUT_F32 ? 4 : 8, CPR = S::TN / CW, ROWS_PER_IT = S::NT / CPR;
        int t = tid;
        asm("" : "+v"(t));      // (or column and row are worked out ahead of the branch and kept in registers for the other side's stores)
        const int col = t % CPR * CW;
        if (col < cols_here)
            for (int m = t / CPR; m < rows_here; m += ROWS_PER_IT) put16(c0 + n0 + col + (int64_t)m * ldc, f32x4{0.f, 0.f, 0.f, 0.f});
        return;
    }
    // 16 bytes of results, the element `at` of the tile's rows of C, to `to`
    auto put_chunk = [&](OutT *to, int64_t at, f32x4 raw, const bf16x8 &uu) __attribute__((always_inline)) {
        if constexpr (EPI == EPI_GELU_BWD) {
            bf16x8 cv = __builtin_bit_cast(bf16x8, raw);
#pragma unroll
            for (int e = 0; e < 8; ++e) cv[e] = (bf16_t)((float)cv[e] * gelu_slope((float)uu[e]));
            raw = __builtin_bit_cast(f32x4, cv);
        }
        put16(to, raw);
        if constexpr (EPI == EPI_GELU) {
            bf16x8 cv = __builtin_bit_cast(bf16x8, raw);
#pragma unroll
            for (int e = 0; e < 8; ++e) cv[e] = (bf16_t)gelu_value((float)cv[e]);
            put16(c1 + at, __builtin_bit_cast(f32x4, cv));
        }
    };
    // U of a chunk, read ahead of the results' way through LDS.  (Behind it, chunk by chunk, a wavefront waited 1.3 us for each: input
    // gradient with GeLU' of 6400 x 896 -> 3584 in 128 x 128 tiles 62.4 -> 56.6 us, 12000 x 1280 -> 5120 in 256 x 256 ones 179 -> 173, 2048 x 512 -> 2048 13.6 -> 13.0.)
    auto fetch_u = [&](int m, int n) __attribute__((always_inline)) {
        return *reinterpret_cast<const bf16x8 *>(gelu_u + (int64_t)min(m, rows_here - 1) * ldc + min(n, n0 + cols_here - 8));
    };
    auto store_tiles = [&](const f32x4 (&acc)[S::MB][S::NB]) __attribute__((always_inline)) {
        int t = tid;
        if constexpr (S::WIDE) {
            using Store = WideStore<OUT_F32, A_ANY>;
            if constexpr (A_ANY) asm("" : "+v"(t));       // (what is worked out from it is not kept through the loop, which spills)
            const int n = n0 + t % Store::CPR * Store::CW;          // column of C; a chunk never straddles n_split
            OutT *const dst = n < n_split ? c0 + n : c1 + (n - n_split);
            const bool column = n < n0 + cols_here;
            static_assert(EPI == EPI_NONE, "");
            Store::store(smem, acc, wm, wn, t, rows_data, [&](int m, f32x4 raw) __attribute__((always_inline)) {
                if (column && m < rows_here) put16(dst + (int64_t)m * ldc, raw);
            });
        } else {
            using Store = GemmStore<S, OUT_F32, A_ANY>;
            const int c = t % Store::CPR, col = c * Store::CW;
            const int n = n0 + col;         // column of C; a chunk never straddles n_split
            OutT *const dst = n < n_split ? c0 + n : c1 + (n - n_split);
            constexpr int AHEAD = Store::ITS < 8 ? Store::ITS : 8;
            bf16x8 uu[AHEAD];
            auto begin = [&](int i0) __attribute__((always_inline)) {
                if constexpr (EPI == EPI_GELU_BWD)
#pragma unroll
                    for (int k = 0; k < AHEAD; ++k) uu[k] = fetch_u((i0 + k) * Store::ROWS_PER_IT + t / Store::CPR, n);
            };
            begin(0);
            __syncthreads();        // every wavefront is done with what the LDS held
            if (group == 0) Store::to_lds(smem, acc, wm, wn, t & 63, rows_data);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < Store::ITS; ++i) {
                const int m = i * Store::ROWS_PER_IT + t / Store::CPR;
                if (i > 0 && i % AHEAD == 0) begin(i);
                f32x4 raw = {0.f, 0.f, 0.f, 0.f};
                if (m < S::TM) raw = *reinterpret_cast<const f32x4 *>(smem + Store::offset(m, c));
                if (col < cols_here && m < rows_here) put_chunk(dst + (int64_t)m * ldc, (int64_t)m * ldc + n, raw, uu[i % AHEAD]);
            }
        }
    };

    f32x4 acc[S::MB][S::NB];
    if constexpr (!S::WIDE) gemm_clear<S>(acc);

    const int T = J.K / PK;
    const int t_split = J.k_split / PK;

    // ---- tile loads
    uint32_t offA[ATile::NI], offW[W_NI];
    const bool a_f32 = A_ANY && J.a_f32 != 0;   // workgroup-uniform
    ATile::offsets(offA, args.lda, rows_data, wave, lane);
    if constexpr (W_TR) WTr::offsets(offW, J.ldw, wave, lane, cols_here / 8);
    else WPlain::offsets(offW, J.ldw, cols_here, wave, lane);

    // (copies: the loads' assembly counts as a write to memory, after which what is read through `J` is fetched again, by a
    // scalar load in every contraction tile whose result waits for all LDS reads on their way)
    const char *a0 = static_cast<const char *>(J.a0), *a1 = static_cast<const char *>(J.a1);
    const bf16_t *const w0 = J.w + (W_TR ? (int64_t)n0 : (int64_t)n0 * J.ldw);
    const int lda = args.lda, ldw = J.ldw;
    const int AE = a_f32 ? 4 : 2;               // bytes per element of A
    const int64_t a_tile0 = ((int64_t)batch * J.a_batch_stride + (int64_t)m0 * args.lda) * AE;
    auto a_src = [&](int t) -> const char * {   // first element of contraction tile t of this row tile
        return (t < t_split ? a0 + (int64_t)t * PK * AE : a1 + (int64_t)(t - t_split) * PK * AE) + a_tile0;
    };
    auto w_src = [&](int t) -> const bf16_t * { return w0 + (W_TR ? (int64_t)t * PK * ldw : (int64_t)t * PK); };
    // float A: thread `gtid` converts the 8-element chunks gtid, gtid + GT, ... of the tile
    // (chunk c is columns 8 (c % 8) .. + 7 of row c / 8) and writes them where the direct load would
    constexpr int FCH = S::TM * 8 / S::GT;      // chunks per thread
    f32x4 stage[A_ANY ? 2 * FCH : 1];
    auto fetch_a = [&](int t, int i) __attribute__((always_inline)) {
        if constexpr (A_ANY) {
            const int c = i * S::GT + gtid, row = min(c >> 3, rows_data - 1);
            const f32x4 *p = reinterpret_cast<const f32x4 *>(a_src(t) + (uint32_t)(row * lda + (c & 7) * 8) * 4u);
            stage[2 * i] = p[0];       // (re-read from L2 by the workgroups of the other column tiles)
            stage[2 * i + 1] = p[1];
        }
    };
    auto stash_a = [&](char *tile_a, int i) __attribute__((always_inline)) {
        if constexpr (A_ANY) {
            const int c = i * S::GT + gtid;
            bf16x8 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[e] = (bf16_t)stage[2 * i][e]; v[4 + e] = (bf16_t)stage[2 * i + 1][e]; }
            *reinterpret_cast<bf16x8 *>(tile_a + ATile::chunk_offset(c >> 3, c & 7)) = v;
        }
    };

    // ---- per-lane LDS offsets of the operand fragments of contraction step ks (32 indices): slot e
    // of a fragment carries index 32 ks + 8 (lane / 16) + e.  (A row 16 further down keeps the permutation.)
    int b_off[PK / 32], w_off[PK / 32], wt_off[S::NB];
#pragma unroll
    for (int ks = 0; ks < PK / 32; ++ks) {
        b_off[ks] = ATile::chunk_offset(S::WM * wm + (lane & 15), 4 * ks + (lane >> 4));
        w_off[ks] = WPlain::chunk_offset(S::WN * wn + (lane & 15), 4 * ks + (lane >> 4));
    }
#pragma unroll
    for (int nb = 0; nb < S::NB; ++nb) wt_off[nb] = WTr::lane_offset(lane, S::NB * wn + nb);
    if constexpr (S::WIDE) {
        auto load_a = [&](int slot, int ks, int mb) __attribute__((always_inline)) {
            return load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(smem + slot * S::ABYTES + b_off[ks] + mb * 16 * PK * 2));
        };
        auto load_w = [&](int slot, int ks, int nb) __attribute__((always_inline)) {
            const char *wt = smem + S::W_RING + slot * S::WBYTES;
            if constexpr (W_TR) return WTr::load_frag(wt, ks, wt_off[nb]);
            else return load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(wt + w_off[ks] + nb * 16 * PK * 2));
        };
        auto issue_a = [&](int t, int slot, int i) __attribute__((always_inline)) {
            lds_dma<16>(uniform_ptr(a_src(t)), offA[i], smem + slot * S::ABYTES + (i * S::GW + wave) * 1024);
        };
        auto issue_w = [&](int t, int slot, int i) __attribute__((always_inline)) {
            lds_dma<16>(uniform_ptr(w_src(t)), offW[i], smem + S::W_RING + slot * S::WBYTES + (i * S::GW + wave) * 1024);
        };
        auto stash = [&](int, int slot, int i) __attribute__((always_inline)) { stash_a(smem + slot * S::ABYTES, i); };
        auto publish = [](int, int, int) {};
        if (a_f32) gemm_wide_loop<REG_A, ATile::NI, W_NI, FCH>(acc, T, issue_a, issue_w, load_a, load_w, publish, fetch_a, stash);
        else gemm_wide_loop<REG_NONE, ATile::NI, W_NI, FCH>(acc, T, issue_a, issue_w, load_a, load_w, publish, fetch_a, stash);
    } else {
        char *const ring = smem + group * S::RING;
        auto load = [&](int slot, int j, GemmFrags<S> &f) __attribute__((always_inline)) {
            const char *at = ring + slot * S::SLOT, *wt = at + S::ABYTES;
            const int ks = j / S::MH, first = j % S::MH * S::HB;
            if (first == 0) {
#pragma unroll
                for (int nb = 0; nb < S::NB; ++nb) {
                    if constexpr (W_TR) f.fw[ks & 1][nb] = WTr::load_frag(wt, ks, wt_off[nb]);
                    else f.fw[ks & 1][nb] = load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(wt + w_off[ks] + nb * 16 * PK * 2));
                }
            }
#pragma unroll
            for (int mb = 0; mb < S::HB; ++mb)
                f.fb[j & 1][mb] = load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(at + b_off[ks] + (first + mb) * 16 * PK * 2));
        };
        auto issue = [&](int t, int slot) {
            char *const dst = ring + slot * S::SLOT + wave * 1024;
            if (!a_f32) lds_dma_n<ATile::NI, S::GW * 1024>(a_src(t), offA, dst);        // bf16 A: direct
            lds_dma_n<W_NI, S::GW * 1024>(w_src(t), offW, dst + S::ABYTES);
        };
        auto fetch = [&](int t) {
#pragma unroll
            for (int i = 0; i < FCH; ++i) fetch_a(t, i);
        };
        auto stash = [&](int, int slot) {
#pragma unroll
            for (int i = 0; i < FCH; ++i) stash_a(ring + slot * S::SLOT, i);
        };
        gemm_loop<S, LOADS, !A_ANY>(acc, T, group, a_f32, issue, load, [](int, int) {}, fetch, stash);
        gemm_add_groups<S>(smem, acc, group, wave, lane);
    }
    store_tiles(acc);
}
template <typename S, bool A_ANY, bool W_TR, bool OUT_F32, int EPI>
__global__ __launch_bounds__(S::NT, S::WAVES_PER_SIMD) void proj_gemm_kernel(ProjArgs args)
{
    proj_gemm_body<S, A_ANY, W_TR, OUT_F32, EPI, true>(args);
}
template <typename S, bool A_ANY, bool W_TR, bool OUT_F32, int EPI>
__global__ __launch_bounds__(S::NT, S::WAVES_PER_SIMD) void proj_small_gemm_kernel(ProjArgs args)
{
    proj_gemm_body<S, A_ANY, W_TR, OUT_F32, EPI, false>(args);
}

// Weight gradient of a linear map: dW[k, n] = sum_r A[r, k] dC[r, n], the contraction running over
// the rows of both operands.  Both are therefore loaded as [64 rows][columns] tiles and read
// through transposing LDS reads (TrTile); a workgroup owns a TM (k) x TN (n) tile of dW for one
// chunk of rows of one batch entry and writes it in fp32, to dW itself when there is a single chunk,
// else to that chunk's partial result, which a fixed-order sum adds up afterwards.  Same wavefront
// layout, ring and LDS-staged stores as proj_gemm_kernel.
//   DC_F32  dC is float and may come from two tensors side by side (the dK and dV partials): it is
//           rounded to bf16 on its way into LDS, through registers, as proj_gemm_kernel does for a
//           float A.
struct WgradArgs {
    const bf16_t *a;            // batch b, row r: a + b * a_batch_stride + r * lda  (K columns)
    const void *dc0, *dc1;      // dC: columns < n_split from dc0, the others from dc1 (column n - n_split); row stride ldc
    int64_t a_batch_stride, dc_batch_stride;    // elements
    float *out;                 // [splits][K][N]
    int rows;                   // rows of every batch entry
    int batches, K, N, n_split, lda, ldc;
    int chunk_rows;             // rows per split, a multiple of 64
    int splits_per_batch, m_tiles, n_tiles;
};

template <typename S, bool DC_F32>
__global__ __launch_bounds__(S::NT, S::WAVES_PER_SIMD) void wgrad_gemm_kernel(WgradArgs g)
{
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    using ATile = TrTile<S::TM, S::GW>;
    using WTile = TrTile<S::TN, S::GW>;
    constexpr int LOADS = ATile::NI + (DC_F32 ? 0 : WTile::NI);
    const int tid = threadIdx.x, lane = tid & 63;
    const int all_waves = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = all_waves / S::GW, wave = all_waves % S::GW, gtid = tid % S::GT;     // wave, gtid: within the group
    const int wm = wave % S::MW, wn = wave / S::MW;

    // An XCD walks the output tiles of one chunk of rows after the other, so that the chunk's rows of A and dC are read from HBM
    // once per XCD, and those in blocks of four tiles down, tile by tile of a column: where an XCD has only some of a chunk's tiles,
    // its workgroups read few strips of either.  Row by row of tiles -> in these blocks: dW of 512 x 2048 from 2048 rows
    // 15.5 -> 11.8 us, 1024 x 4096 from 4096 47.6 -> 40.5, 640 x 2560 from 1000 12.8 -> 11.3, 2048 x 512 from 2048 11.1 -> 11.4.
    const int splits = g.batches * g.splits_per_batch;
    const int tiles = g.m_tiles * g.n_tiles, per_xcd = (splits * tiles + kXcds - 1) / kXcds;
    const int item = blockIdx.x % kXcds * per_xcd + blockIdx.x / kXcds;
    if ((int)blockIdx.x / kXcds >= per_xcd || item >= splits * tiles) return;
    // (The compiler leaves some of these divisions in vector registers.  Read out here, what follows from them, the bases of the loads among it, is scalar
    // arithmetic: see uniform_ptr.)
    auto scalar = [](int v) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(v); };
    const int split = scalar(item / tiles), tile = item - split * tiles;
    const int batch = scalar(split / g.splits_per_batch);
    const int block = scalar(tile / (4 * g.n_tiles)), in = tile - block * 4 * g.n_tiles, down = min(g.m_tiles - 4 * block, 4);
    const int col = scalar(down == 4 ? in >> 2 : in / down);       // (a division is some 40 instructions, 1 % of a launch of 64 x 64 tiles)
    const int m0 = (4 * block + in - col * down) * S::TM, n0 = col * S::TN;
    const int r0 = (split - batch * g.splits_per_batch) * g.chunk_rows, r1 = min(r0 + g.chunk_rows, g.rows);
    const int T = (r1 - r0 + PK - 1) / PK;          // >= 1: the host sizes the splits so
    const int tail = (r1 - r0) - (T - 1) * PK;      // rows of the last tile, 1 .. 64
    const int cols_m = min(g.K - m0, S::TM), cols_n = min(g.N - n0, S::TN);

    uint32_t offA[ATile::NI], offA_last[ATile::NI], offW[DC_F32 ? 1 : WTile::NI], offW_last[DC_F32 ? 1 : WTile::NI];
    ATile::offsets(offA, g.lda, wave, lane, cols_m / 8);
    ATile::offsets(offA_last, g.lda, wave, lane, cols_m / 8, tail);
    if constexpr (!DC_F32) {
        WTile::offsets(offW, g.ldc, wave, lane, cols_n / 8);
        WTile::offsets(offW_last, g.ldc, wave, lane, cols_n / 8, tail);
    }
    const bf16_t *a_base = g.a + (int64_t)batch * g.a_batch_stride + (int64_t)r0 * g.lda + m0;
    auto a_src = [&](int t) -> const bf16_t * { return a_base + (int64_t)t * PK * g.lda; };
    auto w_src = [&](int t) -> const bf16_t * {
        return static_cast<const bf16_t *>(g.dc0) + (int64_t)batch * g.dc_batch_stride + (int64_t)(r0 + t * PK) * g.ldc + n0;
    };
    // Rows past the end of the chunk re-read its last row; their copies in the tiles are replaced
    // by zeros, each lane clearing exactly the 16 bytes its own loads wrote (after waiting for them).
    auto clear_tail = [&](char *tile_a, char *tile_w) {
        if (tail == PK) return;
#pragma unroll
        for (int i = 0; i < ATile::NI; ++i)
            if (ATile::row_of(i, wave, lane) >= tail)
                *reinterpret_cast<f32x4 *>(tile_a + (i * S::GW + wave) * 1024 + lane * 16) = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (!DC_F32) {
#pragma unroll
            for (int i = 0; i < WTile::NI; ++i)
                if (WTile::row_of(i, wave, lane) >= tail)
                    *reinterpret_cast<f32x4 *>(tile_w + (i * S::GW + wave) * 1024 + lane * 16) = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    // float dC: thread `gtid` converts the 8-column chunks gtid, gtid + GT, ... of the [64][TN] tile and
    // writes them where the direct load would; rows past the end of the chunk are written as zeros
    constexpr int FCH = PK * (S::TN / 8) / S::GT;   // chunks per thread
    f32x4 stage[DC_F32 ? 2 * FCH : 1];
    auto fetch_w = [&](int t, int i) __attribute__((always_inline)) {
        if constexpr (DC_F32) {
            const int rows_here = t == T - 1 ? tail : PK;
            const int c = i * S::GT + gtid, row = min(c / WTile::CPR, rows_here - 1), col = min(c % WTile::CPR, cols_n / 8 - 1);
            const int n = n0 + col * 8;
            const float *src = n < g.n_split ? static_cast<const float *>(g.dc0) + n : static_cast<const float *>(g.dc1) + (n - g.n_split);
            const f32x4 *p = reinterpret_cast<const f32x4 *>(src + (int64_t)batch * g.dc_batch_stride + (int64_t)(r0 + t * PK + row) * g.ldc);
            stage[2 * i] = p[0];
            stage[2 * i + 1] = p[1];
        }
    };
    auto stash_w = [&](int t, char *tile_w, int i) __attribute__((always_inline)) {
        if constexpr (DC_F32) {
            const int rows_here = t == T - 1 ? tail : PK;
            const int c = i * S::GT + gtid, row = c / WTile::CPR, col = c % WTile::CPR;
            bf16x8 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = row < rows_here ? (bf16_t)stage[2 * i][e] : (bf16_t)0.f;
                v[4 + e] = row < rows_here ? (bf16_t)stage[2 * i + 1][e] : (bf16_t)0.f;
            }
            *reinterpret_cast<bf16x8 *>(tile_w + WTile::chunk_offset(row, col)) = v;
        }
    };

    // (column block mb of A: the first one's chunk position with bits flipped; eight offsets kept apart would not fit
    // the registers next to a float dC's)
    const int at_off = ATile::lane_offset(lane, S::MB * wm);
    int wt_off[S::NB];
#pragma unroll
    for (int nb = 0; nb < S::NB; ++nb) wt_off[nb] = WTile::lane_offset(lane, S::NB * wn + nb);
    f32x4 acc[S::MB][S::NB];
    if constexpr (!S::WIDE) gemm_clear<S>(acc);
    if constexpr (S::WIDE) {
        auto load_a = [&](int slot, int ks, int mb) __attribute__((always_inline)) { return ATile::load_frag(smem + slot * S::ABYTES, ks, at_off ^ (mb * 32)); };
        auto load_w = [&](int slot, int ks, int nb) __attribute__((always_inline)) {
            return WTile::load_frag(smem + S::W_RING + slot * S::WBYTES, ks, wt_off[nb]);
        };
        auto issue_a = [&](int t, int slot, int i) __attribute__((always_inline)) {
            lds_dma<16>(uniform_ptr(a_src(t)), t == T - 1 ? offA_last[i] : offA[i], smem + slot * S::ABYTES + (i * S::GW + wave) * 1024);
        };
        auto issue_w = [&](int t, int slot, int i) __attribute__((always_inline)) {
            if constexpr (!DC_F32) lds_dma<16>(uniform_ptr(w_src(t)), t == T - 1 ? offW_last[i] : offW[i], smem + S::W_RING + slot * S::WBYTES + (i * S::GW + wave) * 1024);
        };
        auto publish = [&](int t, int a_slot, int w_slot) __attribute__((always_inline)) {
            if (t == T - 1) clear_tail(smem + a_slot * S::ABYTES, smem + S::W_RING + w_slot * S::WBYTES);
        };
        auto stash = [&](int t, int slot, int i) __attribute__((always_inline)) { stash_w(t, smem + S::W_RING + slot * S::WBYTES, i); };
        gemm_wide_loop<DC_F32 ? REG_W : REG_NONE, ATile::NI, WTile::NI, FCH>(acc, T, issue_a, issue_w, load_a, load_w, publish, fetch_w, stash);
    } else {
        char *const ring = smem + group * S::RING;
        static_assert(S::MH == 1, "");
        auto load = [&](int slot, int ks, GemmFrags<S> &f) __attribute__((always_inline)) {
            const char *at = ring + slot * S::SLOT, *wt = at + S::ABYTES;
#pragma unroll
            for (int nb = 0; nb < S::NB; ++nb) f.fw[ks & 1][nb] = WTile::load_frag(wt, ks, wt_off[nb]);
#pragma unroll
            for (int mb = 0; mb < S::HB; ++mb) f.fb[ks & 1][mb] = ATile::load_frag(at, ks, at_off ^ (mb * 32));
        };
        auto issue = [&](int t, int slot) {
            char *const dst = ring + slot * S::SLOT + wave * 1024;
            if (t == T - 1) lds_dma_n<ATile::NI, S::GW * 1024>(a_src(t), offA_last, dst);
            else lds_dma_n<ATile::NI, S::GW * 1024>(a_src(t), offA, dst);
            if constexpr (!DC_F32) {
                if (t == T - 1) lds_dma_n<WTile::NI, S::GW * 1024>(w_src(t), offW_last, dst + S::ABYTES);
                else lds_dma_n<WTile::NI, S::GW * 1024>(w_src(t), offW, dst + S::ABYTES);
            }
        };
        auto publish = [&](int t, int slot) {
            if (t == T - 1) clear_tail(ring + slot * S::SLOT, ring + slot * S::SLOT + S::ABYTES);
        };
        auto fetch = [&](int t) {
#pragma unroll
            for (int i = 0; i < FCH; ++i) fetch_w(t, i);
        };
        auto stash = [&](int t, int slot) {
#pragma unroll
            for (int i = 0; i < FCH; ++i) stash_w(t, ring + slot * S::SLOT + S::ABYTES, i);
        };
        gemm_loop<S, LOADS, false>(acc, T, group, DC_F32, issue, load, publish, fetch, stash);
        gemm_add_groups<S>(smem, acc, group, wave, lane);
    }

    float *out = g.out + (int64_t)split * g.K * g.N + (int64_t)m0 * g.N + n0;
    if constexpr (S::WIDE) {
        using Store = WideStore<true, false>;
        int t = tid;
        if constexpr (DC_F32) asm("" : "+v"(t));       // (what is worked out from it is not kept through the loop, which spills)
        const int col = t % Store::CPR * Store::CW;
        Store::store(smem, acc, wm, wn, t, S::TM, [&](int m, f32x4 raw) __attribute__((always_inline)) {
            if (col < cols_n && m < cols_m) *reinterpret_cast<f32x4 *>(out + (int64_t)m * g.N + col) = raw;
        });
    } else {
        using Store = GemmStore<S, true, false>;
        __syncthreads();
        if (group == 0) Store::to_lds(smem, acc, wm, wn, lane, S::TM);
        __syncthreads();
        const int c = tid % Store::CPR, col = c * Store::CW;
        if (col < cols_n) {
#pragma unroll
            for (int i = 0; i < Store::ITS; ++i) {
                const int m = i * Store::ROWS_PER_IT + tid / Store::CPR;
                if (m < cols_m)
                    *reinterpret_cast<f32x4 *>(out + (int64_t)m * g.N + col) = *reinterpret_cast<const f32x4 *>(smem + Store::offset(m, c));
            }
        }
    }
}

// ---- the tiles a launch may take
using ShapeL = GemmWide;                                // four wavefronts, one workgroup per compute unit
// ... eight of 128 x 64 where a feed-forward unit's epilogue follows: GeLU is some twenty vector instructions per element, of which a wavefront alone on its
// SIMD issues one in 7.5 cycles and two together twice as many.  linear_gelu_fwd of 6000 x 640 -> 2560 by four and by eight 38.0 and 34.9 us in a layer's pass,
// 3244 x 1152 -> 4608 51.1 and 48.4, 16384 x 1024 -> 4096 188 and 177; linear_bwd_input_gelu of the first two 38.9 and 35.6, 51.2 and 49.2.
using ShapeL8 = GemmShape<256, 256, 128, 64, 2>;
using ShapeM = GemmShape<128, 128, 64, 64, 2>;          // four wavefronts, two workgroups per compute unit
using ShapeM2 = GemmShape<128, 128, 64, 64, 2, 2>;      // ... two such groups share the contraction
using ShapeM8 = GemmShape<128, 128, 64, 32, 4>;         // ... eight wavefronts of one group, four tiles on their way
using ShapeS = GemmShape<64, 64, 32, 32, 4>;
// The smaller tiles wait for their operands' bytes, of which two or four groups of wavefronts with three or four tiles each on their way ask for more at a time
// than twice the groups with two: the six products of a feed-forward unit in a row, 2048 x 512 67.2 -> 60.5 us in 64 x 64 tiles (one group with eight
// 70.5), 500 x 1024 75.4 -> 68.4 in 32 x 64 ones (two groups with five 69.8), 232 x 1024 58.3 -> 53.3 in 32 x 32 ones (two groups with eight 56.0).
using ShapeS4 = GemmShape<64, 64, 32, 32, 4, 2>;        // two groups of four wavefronts
// Where 64 x 64 tiles leave most compute units without one, what a launch waits for is a workgroup's own operand bytes, of which a compute unit
// gets 40 to 60 per cycle: smaller tiles spread them, although there are more of them.  58 x 4096 -> 1024: S4 16.0 us, T4 11.2, T8 9.4;
// 256 x 2048 -> 2048 10.8, 8.4, 12.8; dW of 512 x 512 from 1024 rows 6.1, 5.2, 4.9.
using ShapeT4 = GemmShape<32, 64, 32, 32, 3, 4>;        // two wavefronts, four such groups
using ShapeT8 = GemmShape<32, 32, 32, 32, 4, 4>;        // one wavefront, four such groups
// ... as gemm_form() says for float operands.  project_bwd in 32 x 64 tiles with two slots and with three: 145 rows and contractions of 3584 15.7 and 16.1 us,
// 96 and 4096 16.2 and 16.9, 337 and 1280 6.0 and 6.0.
using ShapeS4F = GemmShape<64, 64, 32, 32, 2, 4>;
using ShapeT4F = GemmShape<32, 64, 32, 32, 2, 4>;
using ShapeT8F = GemmShape<32, 32, 32, 32, 2, 8>;

template <typename S, bool A_ANY, bool W_TR, bool OUT_F32, int EPI>
hipError_t launch_proj_shape(ProjArgs &args, int kernel_id, hipStream_t st)
{
    int wgs = 0;
    for (int j = 0; j < args.n_jobs; ++j) {
        ProjJob &J = args.job[j];
        J.n_tiles = (J.N + S::TN - 1) / S::TN;
        J.m_data = (std::min(J.rows, J.rows_ok) + S::TM - 1) / S::TM;
        J.wg_begin = wgs;
        wgs += xcd_tile_grid(J.batches * J.m_data, J.n_tiles);
    }
    const ProjJob &first = args.job[0];
    args.zero_begin = wgs;
    args.zero_end = gemm_zero_end(first.rows, first.rows_ok, args.skip_tail);
    args.zero_tiles = gemm_zero_tiles(first.rows, first.rows_ok, args.skip_tail, S::TM, S::TN);
    wgs += xcd_tile_grid(first.batches * args.zero_tiles, first.n_tiles);
    if (wgs == 0) return hipSuccess;
    static DeviceOnce once;
    constexpr bool SMALL = S::TM == 32;
    void (*kernel)(ProjArgs);
    if constexpr (SMALL) kernel = proj_small_gemm_kernel<S, A_ANY, W_TR, OUT_F32, EPI>;
    else kernel = proj_gemm_kernel<S, A_ANY, W_TR, OUT_F32, EPI>;
    if (SMALL)
        kernel_id = kernel_id == K_PROJ_FWD ? K_PROJ_FWD_SMALL : kernel_id == K_PROJ_BWD ? K_PROJ_BWD_SMALL : kernel_id == K_LINEAR_FWD ? K_LINEAR_FWD_SMALL : K_LINEAR_BWD_SMALL;
    if (const hipError_t e = allow_lds(kernel, S::LDS, once); e != hipSuccess) return e;
    TimedLaunch tl(kernel_id, st);
    hipLaunchKernelGGL(kernel, dim3(wgs), dim3(S::NT), S::LDS, st, args);
    return hipGetLastError();
}

// The shapes of lss_gemm_plan.h's tiles
template <GemmTile T> struct TileShape;
template <> struct TileShape<TILE_L> { using type = ShapeL; };
template <> struct TileShape<TILE_M> { using type = ShapeM; };
template <> struct TileShape<TILE_M2> { using type = ShapeM2; };
template <> struct TileShape<TILE_M8> { using type = ShapeM8; };
template <> struct TileShape<TILE_S> { using type = ShapeS; };
template <> struct TileShape<TILE_S4> { using type = ShapeS4; };
template <> struct TileShape<TILE_T4> { using type = ShapeT4; };
template <> struct TileShape<TILE_T8> { using type = ShapeT8; };
template <typename S>
constexpr bool is_form(const GemmForm &f)
{
    if constexpr (S::WIDE) return f.groups == S::KG && f.slots == S::A_SLOTS;
    else return f.groups == S::KG && f.slots == S::STAGES;
}
template <GemmTile T>
constexpr bool tile_agrees()
{
    using S = typename TileShape<T>::type;
    return S::TM == kGemmTiles[T].tm && S::TN == kGemmTiles[T].tn && S::KG == kGemmTiles[T].groups && S::PER_CU == kGemmTiles[T].per_cu &&
           is_form<S>(gemm_form(T, false, false, kGemmK));
}
static_assert(tile_agrees<TILE_L>() && tile_agrees<TILE_M>() && tile_agrees<TILE_M2>() && tile_agrees<TILE_M8>() && tile_agrees<TILE_S>() &&
              tile_agrees<TILE_S4>() && tile_agrees<TILE_T4>() && tile_agrees<TILE_T8>(), "the plan's table is about other shapes");

static_assert(is_form<ShapeS4F>(gemm_form(TILE_S4, false, true, kGemmK)) && is_form<ShapeS4>(gemm_form(TILE_S4, true, true, kLongFloat)) &&
              is_form<ShapeS4F>(gemm_form(TILE_S4, true, true, kLongFloat + 1)) && is_form<ShapeT4F>(gemm_form(TILE_T4, false, true, kGemmK)) &&
              is_form<ShapeT8>(gemm_form(TILE_T8, false, true, kLongFloat)) && is_form<ShapeT8F>(gemm_form(TILE_T8, false, true, kLongFloat + 1)), "");

int proj_work(const ProjArgs &args, GemmWork (&work)[2])
{
    for (int j = 0; j < args.n_jobs; ++j) {
        const ProjJob &J = args.job[j];
        work[j] = {J.batches, J.rows, J.rows_ok, J.N, J.K, J.a_f32};
    }
    return args.n_jobs;
}
bool proj_streams(const ProjArgs &args, bool out_f32)
{
    GemmWork work[2];
    const int n = proj_work(args, work);
    return gemm_streams(work, n, out_f32);
}
GemmTile proj_tile(const ProjArgs &args, bool a_any, bool streams)
{
    GemmWork work[2];
    const int n = proj_work(args, work);
    return pick_gemm_tile(work, n, a_any, args.skip_tail, streams);
}

GemmForm proj_form(const ProjArgs &args, GemmTile tile, bool a_any) { return gemm_form(tile, false, a_any, args.job[0].K); }
template <bool A_ANY, bool W_TR, bool OUT_F32, int EPI = EPI_NONE>
hipError_t launch_proj(ProjArgs &args, int kernel_id, hipStream_t st)
{
    args.stream = proj_streams(args, OUT_F32);
    const GemmTile tile = proj_tile(args, A_ANY, args.stream);
    switch (tile) {
    case TILE_L: return launch_proj_shape<typename std::conditional<EPI == EPI_NONE, ShapeL, ShapeL8>::type, A_ANY, W_TR, OUT_F32, EPI>(args, kernel_id, st);
    case TILE_M: return launch_proj_shape<ShapeM, A_ANY, W_TR, OUT_F32, EPI>(args, kernel_id, st);
    case TILE_M2:
        if constexpr (A_ANY) return launch_proj_shape<ShapeM2, A_ANY, W_TR, OUT_F32, EPI>(args, kernel_id, st);
        break;
    case TILE_M8:
        if constexpr (!A_ANY) return launch_proj_shape<ShapeM8, A_ANY, W_TR, OUT_F32, EPI>(args, kernel_id, st);
        break;
    case TILE_S: return launch_proj_shape<ShapeS, A_ANY, W_TR, OUT_F32, EPI>(args, kernel_id, st);
    case TILE_S4:
        if constexpr (A_ANY) return launch_proj_shape<ShapeS4F, A_ANY, W_TR, OUT_F32, EPI>(args, kernel_id, st);
        else return launch_proj_shape<ShapeS4, A_ANY, W_TR, OUT_F32, EPI>(args, kernel_id, st);
    case TILE_T4:
        if constexpr (A_ANY) return launch_proj_shape<ShapeT4F, A_ANY, W_TR, OUT_F32, EPI>(args, kernel_id, st);
        else return launch_proj_shape<ShapeT4, A_ANY, W_TR, OUT_F32, EPI>(args, kernel_id, st);
    case TILE_T8:
        if constexpr (A_ANY)
            if (is_form<ShapeT8F>(proj_form(args, tile, A_ANY))) return launch_proj_shape<ShapeT8F, A_ANY, W_TR, OUT_F32, EPI>(args, kernel_id, st);
        return launch_proj_shape<ShapeT8, A_ANY, W_TR, OUT_F32, EPI>(args, kernel_id, st);
    default: break;
    }
    return hipErrorInvalidConfiguration;        // (pick_gemm_tile: none of the others)
}

ProjArgs qkv_args(const bf16_t *x, const bf16_t *w_q, const bf16_t *w_kv, int64_t s0, int l_s, int l_x, int B, int E, bf16_t *q_seg, bf16_t *k, bf16_t *v)
{
    ProjArgs args{};
    args.lda = args.ldc = E;
    args.skip_tail = 0;
    int n = 0;
    {   // [K | V] = x [W_k | W_v]: the batches of x are contiguous, one tall matrix
        ProjJob &J = args.job[n++];
        J.a0 = x; J.a1 = nullptr; J.w = w_kv; J.c0 = k; J.c1 = v;
        J.a_batch_stride = J.c_batch_stride = 0;
        J.rows = J.rows_ok = B * l_x; J.batches = 1;
        J.N = 2 * E; J.K = E; J.k_split = E; J.n_split = E; J.ldw = 2 * E;
    }
    if (l_s > 0) {  // Q_i = x_i W_q
        ProjJob &J = args.job[n++];
        J.a0 = x ? x + s0 * E : nullptr; J.a1 = nullptr; J.w = w_q; J.c0 = q_seg; J.c1 = nullptr;
        J.a_batch_stride = (int64_t)l_x * E; J.c_batch_stride = (int64_t)l_s * E;
        J.rows = J.rows_ok = l_s; J.batches = B;
        J.N = E; J.K = E; J.k_split = E; J.n_split = E; J.ldw = E;
    }
    args.n_jobs = n;
    return args;
}

ProjArgs bwd_args(const bf16_t *dq, const float *dk_part, const float *dv_part, const bf16_t *w_q, const bf16_t *w_kv, int l_s, int l_x, int rows_valid,
                  int B, int E, int skip_tail, float *dx_q, float *dx_part)
{
    ProjArgs args{};
    args.lda = args.ldc = E;
    args.skip_tail = skip_tail;
    int n = 0;
    {   // dx_partial = dK_part W_k^T + dV_part W_v^T: one contraction over the 2E columns of [dK | dV]
        ProjJob &J = args.job[n++];
        J.a0 = dk_part; J.a1 = dv_part; J.w = w_kv; J.c0 = dx_part; J.c1 = nullptr;
        J.a_batch_stride = J.c_batch_stride = (int64_t)l_x * E;
        J.rows = l_x; J.rows_ok = rows_valid; J.batches = B;
        J.N = E; J.K = 2 * E; J.k_split = E; J.n_split = E; J.ldw = 2 * E;
        J.a_f32 = 1;
    }
    if (l_s > 0) {  // dx_q = dQ_i W_q^T, in the same launch
        ProjJob &J = args.job[n++];
        J.a0 = dq; J.a1 = nullptr; J.w = w_q; J.c0 = dx_q; J.c1 = nullptr;
        J.a_batch_stride = J.c_batch_stride = (int64_t)l_s * E;
        J.rows = J.rows_ok = l_s; J.batches = B;
        J.N = E; J.K = E; J.k_split = E; J.n_split = E; J.ldw = E;
        J.a_f32 = 0;
    }
    args.n_jobs = n;
    return args;
}

// c = a w for any row count: one job, one tall matrix; with gelu_c also gelu_c = GeLU(c)
ProjArgs linear_fwd_args(const bf16_t *a, const bf16_t *w, int rows, int K, int N, bf16_t *c, bf16_t *gelu_c)
{
    ProjArgs args{};
    args.lda = K; args.ldc = N; args.skip_tail = 0; args.n_jobs = 1;
    ProjJob &J = args.job[0];
    J.a0 = a; J.a1 = nullptr; J.w = w; J.c0 = c; J.c1 = gelu_c;
    J.a_batch_stride = J.c_batch_stride = 0;
    J.rows = J.rows_ok = rows; J.batches = 1;
    J.N = N; J.K = K; J.k_split = K; J.n_split = N; J.ldw = N;
    return args;
}

// da = dc w^T: w as stored, [K][N], is the [output column][contraction index] layout read plainly;
// with gelu_u, da = (dc w^T) * GeLU'(gelu_u)
ProjArgs linear_bwd_input_args(const bf16_t *dc, const bf16_t *w, const bf16_t *gelu_u, int rows, int K, int N, bf16_t *da)
{
    ProjArgs args{};
    args.lda = N; args.ldc = K; args.skip_tail = 0; args.n_jobs = 1;
    ProjJob &J = args.job[0];
    J.a0 = dc; J.a1 = gelu_u; J.w = w; J.c0 = da; J.c1 = nullptr;
    J.a_batch_stride = J.c_batch_stride = 0;
    J.rows = J.rows_ok = rows; J.batches = 1;
    J.N = K; J.K = N; J.k_split = N; J.n_split = K; J.ldw = N;
    return args;
}

} // namespace

hipError_t launch_project_qkv(const bf16_t *x, const bf16_t *w_q, const bf16_t *w_kv, int64_t s0, int l_s, int l_x,
                              int B, int E, bf16_t *q_seg, bf16_t *k, bf16_t *v, hipStream_t st)
{
    ProjArgs args = qkv_args(x, w_q, w_kv, s0, l_s, l_x, B, E, q_seg, k, v);
    return launch_proj<false, true, false>(args, K_PROJ_FWD, st);
}

hipError_t launch_project_bwd(const bf16_t *dq, const float *dk_part, const float *dv_part, const bf16_t *w_q,
                              const bf16_t *w_kv, int l_s, int l_x, int rows_valid, int B, int E, int skip_tail,
                              float *dx_q, float *dx_part, hipStream_t st)
{
    ProjArgs args = bwd_args(dq, dk_part, dv_part, w_q, w_kv, l_s, l_x, rows_valid, B, E, skip_tail, dx_q, dx_part);
    return launch_proj<true, false, true>(args, K_PROJ_BWD, st);
}

hipError_t launch_linear_fwd(const bf16_t *a, const bf16_t *w, int rows, int K, int N, bf16_t *c, bf16_t *gelu_c,
                             hipStream_t st)
{
    ProjArgs args = linear_fwd_args(a, w, rows, K, N, c, gelu_c);
    if (gelu_c) return launch_proj<false, true, false, EPI_GELU>(args, K_LINEAR_FWD, st);
    return launch_proj<false, true, false>(args, K_LINEAR_FWD, st);
}

hipError_t launch_linear_bwd_input(const bf16_t *dc, const bf16_t *w, const bf16_t *gelu_u, int rows, int K, int N,
                                   bf16_t *da, hipStream_t st)
{
    ProjArgs args = linear_bwd_input_args(dc, w, gelu_u, rows, K, N, da);
    if (gelu_u) return launch_proj<false, false, false, EPI_GELU_BWD>(args, K_LINEAR_BWD, st);
    return launch_proj<false, false, false>(args, K_LINEAR_BWD, st);
}

// plan: what lss_plan.h says
void plan_linear(int op, int rows, int K, int N, int *plan)
{
    if (op == 2) {
        const WgradPlan p = pick_wgrad_plan(rows, 1, K, N, false);
        const GemmForm f = gemm_form(p.tile, true, false, p.chunk_rows);
        const int all[4] = {p.tile, p.splits_per_batch, f.groups, f.slots};
        std::copy(all, all + 4, plan);
        return;
    }
    const ProjArgs args = op == 0 ? linear_fwd_args(nullptr, nullptr, rows, K, N, nullptr, nullptr) : linear_bwd_input_args(nullptr, nullptr, nullptr, rows, K, N, nullptr);
    const GemmTile tile = proj_tile(args, false, proj_streams(args, false));
    const GemmForm f = proj_form(args, tile, false);
    const int all[4] = {tile, 1, f.groups, f.slots};
    std::copy(all, all + 4, plan);
}
void plan_project(int op, int l_s, int l_x, int rows_valid, int B, int E, int *plan)
{
    const ProjArgs args = op == 0 ? qkv_args(nullptr, nullptr, nullptr, 0, l_s, l_x, B, E, nullptr, nullptr, nullptr)
                                  : bwd_args(nullptr, nullptr, nullptr, nullptr, nullptr, l_s, l_x, rows_valid, B, E, 0, nullptr, nullptr);
    const GemmTile tile = proj_tile(args, op == 1, proj_streams(args, op == 1));
    const GemmForm f = proj_form(args, tile, op == 1);
    const int all[3] = {tile, f.groups, f.slots};
    std::copy(all, all + 3, plan);
}
void plan_project_bwd_weight(int l_s, int rows_valid, int B, int E, int *plan)
{
    const WgradPlan q = pick_wgrad_plan(l_s, B, E, E, false), kv = pick_wgrad_plan(rows_valid, B, E, 2 * E, true);
    const GemmForm fq = gemm_form(q.tile, true, false, q.chunk_rows), fkv = gemm_form(kv.tile, true, true, kv.chunk_rows);
    const int all[8] = {q.tile, q.splits_per_batch, kv.tile, kv.splits_per_batch, fq.groups, fq.slots, fkv.groups, fkv.slots};
    std::copy(all, all + 8, plan);
}

static size_t wgrad_scratch_bytes(int rows, int batches, int K, int N)
{
    const int spb = wgrad_most_chunks(rows, batches, K, N);
    return batches * spb > 1 ? (size_t)batches * spb * K * N * sizeof(float) : 0;
}

template <typename S, bool DC_F32>
static hipError_t launch_wgrad_shape(WgradArgs &g, hipStream_t st)
{
    g.m_tiles = (g.K + S::TM - 1) / S::TM;
    g.n_tiles = (g.N + S::TN - 1) / S::TN;
    static DeviceOnce once;
    const auto kernel = wgrad_gemm_kernel<S, DC_F32>;
    if (const hipError_t e = allow_lds(kernel, S::LDS, once); e != hipSuccess) return e;
    TimedLaunch tl(K_LINEAR_WGRAD, st);
    hipLaunchKernelGGL(kernel, dim3(xcd_tile_grid(g.batches * g.splits_per_batch, g.m_tiles * g.n_tiles)), dim3(S::NT), S::LDS, st, g);
    return hipGetLastError();
}

// g: operands, rows, batches, K, N, strides filled in; dw [K][N]; rows >= 1, batches >= 1
template <bool DC_F32>
static hipError_t launch_wgrad(WgradArgs &g, float *dw, float *scratch, hipStream_t st)
{
    const WgradPlan p = pick_wgrad_plan(g.rows, g.batches, g.K, g.N, DC_F32);
    g.splits_per_batch = p.splits_per_batch;
    g.chunk_rows = p.chunk_rows;
    const int splits = g.batches * g.splits_per_batch;
    g.out = splits > 1 ? scratch : dw;
    hipError_t e;
    switch (p.tile) {
    case TILE_L: e = launch_wgrad_shape<ShapeL, DC_F32>(g, st); break;
    case TILE_M: e = launch_wgrad_shape<ShapeM, DC_F32>(g, st); break;
    case TILE_M2: e = launch_wgrad_shape<ShapeM2, DC_F32>(g, st); break;
    case TILE_S: e = launch_wgrad_shape<ShapeS, DC_F32>(g, st); break;
    case TILE_S4:
        if constexpr (DC_F32)
            if (is_form<ShapeS4F>(gemm_form(p.tile, true, true, g.chunk_rows))) { e = launch_wgrad_shape<ShapeS4F, DC_F32>(g, st); break; }
        e = launch_wgrad_shape<ShapeS4, DC_F32>(g, st);
        break;
    case TILE_T4:
        if constexpr (!DC_F32) e = launch_wgrad_shape<ShapeT4, DC_F32>(g, st);
        else e = hipErrorInvalidConfiguration;              // (pick_wgrad_plan: not with a float dC)
        break;
    case TILE_T8:
        if constexpr (DC_F32)
            if (is_form<ShapeT8F>(gemm_form(p.tile, true, true, g.chunk_rows))) { e = launch_wgrad_shape<ShapeT8F, DC_F32>(g, st); break; }
        e = launch_wgrad_shape<ShapeT8, DC_F32>(g, st);
        break;
    default: e = hipErrorInvalidConfiguration; break;       // (pick_wgrad_plan: no other)
    }
    if (e != hipSuccess || splits == 1) return e;
    std::vector<const float *> parts(splits);
    for (int i = 0; i < splits; ++i) parts[i] = scratch + (size_t)i * g.K * g.N;
    return launch_reduce(parts.data(), splits, nullptr, g.K, 1, 1, g.N, dw, st);   // chunk 0 + chunk 1 + ..., in that order
}

size_t linear_bwd_weight_scratch_bytes(int rows, int K, int N) { return wgrad_scratch_bytes(rows, 1, K, N); }

// dw = a^T dc.  rows >= 1.
hipError_t launch_linear_bwd_weight(const bf16_t *a, const bf16_t *dc, int rows, int K, int N, float *dw, float *scratch,
                                    hipStream_t st)
{
    WgradArgs g{};
    g.a = a; g.dc0 = dc; g.dc1 = nullptr;
    g.rows = rows; g.batches = 1; g.K = K; g.N = N; g.n_split = N; g.lda = K; g.ldc = N;
    return launch_wgrad<false>(g, dw, scratch, st);
}

// enough for any rows_valid <= l_x: a plan never has more chunks per batch entry than wgrad_max_chunks()
size_t project_bwd_weight_scratch_bytes(int l_s, int l_x, int B, int E)
{
    (void)l_x;
    const size_t q = l_s > 0 ? wgrad_scratch_bytes(l_s, B, E, E) : 0;
    const size_t kv = (size_t)B * wgrad_max_chunks(B, E, 2 * E) * E * 2 * E * sizeof(float);
    return q > kv ? q : kv;
}
size_t project_bwd_weight_scratch_needed(int l_s, int rows_valid, int B, int E)
{
    const size_t q = l_s > 0 ? wgrad_scratch_bytes(l_s, B, E, E) : 0;
    const size_t kv = rows_valid > 0 ? wgrad_scratch_bytes(rows_valid, B, E, 2 * E) : 0;
    return q > kv ? q : kv;
}

// dw_q = sum_b x_i^T dQ_i (l_s >= 1) and dw_kv = sum_b x[:rows_valid]^T [dK_part | dV_part][:rows_valid] (rows_valid >= 1);
// either is skipped when its row count is 0 (the caller writes the zeros)
hipError_t launch_project_bwd_weight(const bf16_t *x, const bf16_t *dq, const float *dk_part, const float *dv_part, int64_t s0,
                                     int l_s, int l_x, int rows_valid, int B, int E, float *dw_q, float *dw_kv, float *scratch,
                                     hipStream_t st)
{
    if (l_s > 0) {
        WgradArgs g{};
        g.a = x + s0 * E; g.a_batch_stride = (int64_t)l_x * E; g.lda = E;
        g.dc0 = dq; g.dc1 = nullptr; g.dc_batch_stride = (int64_t)l_s * E; g.ldc = E;
        g.rows = l_s; g.batches = B; g.K = E; g.N = E; g.n_split = E;
        const hipError_t e = launch_wgrad<false>(g, dw_q, scratch, st);
        if (e != hipSuccess) return e;
    }
    if (rows_valid > 0) {
        WgradArgs g{};
        g.a = x; g.a_batch_stride = (int64_t)l_x * E; g.lda = E;
        g.dc0 = dk_part; g.dc1 = dv_part; g.dc_batch_stride = (int64_t)l_x * E; g.ldc = E;
        g.rows = rows_valid; g.batches = B; g.K = E; g.N = 2 * E; g.n_split = E;
        return launch_wgrad<true>(g, dw_kv, scratch, st);
    }
    return hipSuccess;
}

} // namespace lss
