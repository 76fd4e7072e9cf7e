// Tuned bf16 backward of Eq. 2 (Section 3, Principle 3) for gfx950 (mathematics: lss_bwd.hip): dQ and dK/dV as two kinds of
// workgroup that share one launch (bwd_main_bf16_kernel); short segments take one pass for all three gradients
// (bwd_skinny_bf16_kernel).  In the former:
//   * 32 x 32 blocks, in 16 x 16 x 32 instructions, three stages per block (score-side products, vector
//     work, output-side products), software-pipelined so that the vector work of one block sits between
//     the matrix instructions of its neighbours.  16 x 16 x 32 and not 32 x 32 x 16 for what it measures on the kernels: with it in
//     dK/dV 8,192 x 8,192 causal passes fell from 1,014 to 994 us, 32,768 keys at d = 128 from 2,535 to 2,505; in dQ then to 984 and
//     2,464.  Loops on Gaussian bf16 (lss_microbench, section 7) do not show why: 1,700 against 1,630 TFLOP/s in registers, but 1,390
//     either way with the backward's vector work in between, and 1,163 against 1,226 with an LDS read per 32,768 flop besides, as here;
//   * 64-row tiles loaded global -> LDS directly into a ring of three unpadded, swizzled tiles, a
//     full loop iteration ahead, one barrier per tile.  A ring of four, two iterations ahead, changed nothing;
//   * as few scalar instructions per step as can be: beside matrix and vector work each costs a lone wavefront about 8 cycles
//     (lss_microbench, section 3).  With tile addresses and ring slots that move on from iteration to iteration instead of being
//     computed in each, one address register for the loads of a tile (DirectTile::issue_pair) and one compare for the masks a dK/dV
//     iteration has 26 of them fewer, a dQ one 30, a forward one 27: forward and backward of 16 heads of 8,192 tokens in
//     eight segments 953 -> 937 us, 64 of 24,576 in six 21.63 -> 21.16 ms, 32,768 keys at d = 128 2,347 -> 2,300.  With LDS addresses that
//     move on likewise, one wait for a unit's LDS reads instead of three or four and the vector work spread evenly (b_elems) 931 -> 907 us,
//     21.38 -> 20.68 ms, 2,311 -> 2,240;
//   * row-major LDS tiles read transposed with DS_READ_B64_TR_B16 where the contraction runs over
//     tile rows (K^T for dQ, Q^T and dO^T for dK and dV) -- no transposing stores;
//   * lse, D = rowsum(dO * out) and the masks folded into accumulator start values where the
//     layout allows (-D and -lse * sqrt(d) per row come from a small kernel, or from the workgroup itself: bwd_own_values).
#include "lss_bf16.h"
#include <type_traits>
#include "lss_bwd_plan.h"
#include "lss_kernels.h"
#include <algorithm>
#include <cmath>

namespace lss {

// ------------------------------------------------------------------------------------------ dQ
template <int D, int NJ = 2>
struct DqBf16Cfg {
    static constexpr int WAVES = 8 / NJ, RW = 16 * NJ;  // query rows per wavefront: NJ blocks of 16
    static constexpr int BR = WAVES * RW, BC = 64, NT = 64 * WAVES;
    static constexpr int RING = 3;                      // K/V tiles resident in LDS
    static constexpr int NU = D / 16;                   // operand steps of the S/dP products; same for dQ
    using Tile = DirectTile<D, BC, WAVES>;
    static constexpr int OFF_V = Tile::BYTES, SLOT = 2 * Tile::BYTES;   // one ring slot: K tile, V tile
    // (dropout: behind the ring, the column keys of the last four tiles issued, 64 each)
    static constexpr int group_lds(bool drop) { return RING * SLOT + (drop ? 4 * BC * 4 : 0); }
};

// KG: groups of wavefronts in the workgroup, see bwd_main_bf16_kernel.
// Transposed formulation: S^T = K Q^T and dP^T = V dO^T put the wavefront's 16 NJ queries on the lanes
// (lse and D are per-lane scalars), and dS^T comes out of the accumulators in the layout the
// dQ^T += K^T dS^T product wants as its second operand.  The keys are walked in blocks of 32 (two
// per 64-key K/V tile).  Per block g three stages:
//     A(g): S^T and dP^T products (matrix),  B(g): dS^T (vector: exp, multiplies, bf16 packing),
//     C(g): dQ^T product (matrix).
// As in the dK/dV kernel below the stages are software-pipelined, step g issuing the matrix
// instructions of A(g+1) and C(g-1) with the vector work of B(g) spread between them, over a ring
// of three K/V tiles that are loaded global -> LDS directly, a full loop iteration ahead.
// -D = -rowsum(dO * out) of the wavefront's rows comes from the preprocess kernel (`Dn`), or is computed here (OWN).
// DROP: dropout on the weights (mask M = keep / (1 - p), decided by drop_keep() of (seed,
// batch*head, global row, key)): dS = P * (M dP - D).
template <int D, bool DROP, bool OWN, int KG, int NJ>
__device__ __forceinline__ void bwd_dq_body(char *smem, const SegShape &s, const DropArgs &dr, const bf16_t *__restrict__ q,
                                            const bf16_t *__restrict__ k, const bf16_t *__restrict__ v,
                                            const bf16_t *__restrict__ out, const bf16_t *__restrict__ dO, const float *__restrict__ lse,
                                            const float *__restrict__ Dn, bf16_t *__restrict__ dq,
                                            float *__restrict__ dq_part, int n_splits, int q_tile, int n_q_tiles, int bh,
                                            int split)
{
    using C = DqBf16Cfg<D, NJ>;
    using Tile = typename C::Tile;
    constexpr int NU = C::NU;

    const int tid = threadIdx.x, lane = tid & 63, lq = lane & 15, g = lane >> 4;
    const int all_waves = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = KG > 1 ? all_waves / C::WAVES : 0, wave = KG > 1 ? all_waves % C::WAVES : all_waves;     // wave: within the group
    char *const ring = smem + group * C::group_lds(DROP);
    const int b = bh / s.H, h = bh % s.H;
    // query tiles are dispatched last-first: under the causal mask the last tiles see the most
    // keys, and starting the longest workgroups first shortens the tail of the launch
    const int r0 = (n_q_tiles - 1 - q_tile) * C::BR;
    const int rw0 = r0 + wave * C::RW;
    const int64_t ld = (int64_t)s.H * D;

    const int r_last = min(r0 + C::BR, s.l_s) - 1;
    const int kv_end = s.causal ? (int)min<int64_t>(s.l_x, s.s0 + r_last + 1) : s.l_x;
    const int n_tiles = (kv_end + C::BC - 1) / C::BC;
    const int per = (n_tiles + n_splits - 1) / n_splits;
    const int s_begin = split * per, s_tiles = max(min(n_tiles, s_begin + per) - s_begin, 0);
    // this group's tiles; the first group has `iters` of them, the other one fewer or none
    const int iters = KG > 1 ? (s_tiles + KG - 1) / KG : s_tiles;
    const int t_begin = s_begin + group * iters, T = KG > 1 ? max(min(s_tiles - group * iters, iters), 0) : s_tiles;

    // this lane's query rows (columns of the S^T blocks), rw0 + 16 j + lq; rows past the segment re-read its last row
    // (unconditional loads), get lse = +inf, which makes their P and dS exactly 0, and are never stored
    Frag<bf16_t> qf[NU / 2][NJ], gf[NU / 2][NJ];        // operand step ks (32 columns), row block j
    float L2[NJ], Dr[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int r = rw0 + 16 * j + lq, rc = min(r, s.l_s - 1);
        const int64_t off = ((int64_t)b * s.l_s + rc) * ld + (int64_t)h * D + g * 8;
        Dr[j] = 0.f;
#pragma unroll
        for (int ks = 0; ks < NU / 2; ++ks) {
            qf[ks][j] = load_frag<bf16_t>(q + off + ks * 32);
            gf[ks][j] = load_frag<bf16_t>(dO + off + ks * 32);
            if constexpr (OWN) {    // the lane's quarter of the row
                const Frag<bf16_t> of = load_frag<bf16_t>(out + off + ks * 32);
#pragma unroll
                for (int e = 0; e < 8; ++e) Dr[j] += (float)gf[ks][j].v[e] * (float)of.v[e];
            }
        }
        if constexpr (OWN) {
            Dr[j] += __shfl_xor(Dr[j], 16);
            Dr[j] += __shfl_xor(Dr[j], 32);
        } else {
            Dr[j] = -Dn[(int64_t)bh * s.l_s + rc] * (DROP ? dr.scale : 1.f);
        }
        const float lv = lse[(int64_t)bh * s.l_s + rc];
        L2[j] = r < s.l_s ? lv * kLog2e : INFINITY;
    }
    const float c = kLog2e / sqrtf((float)D);
    // -D in all accumulator slots: third operand of each block's first dP^T instructions (not with dropout, whose mask comes between)
    const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
    f32x4 neg_d[NJ], acc[NU][NJ];                         // acc: 16 columns x 16 rows each, transposed
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        neg_d[j] = f32x4{-Dr[j], -Dr[j], -Dr[j], -Dr[j]};
#pragma unroll
        for (int db = 0; db < NU; ++db) acc[db][j] = zero4;
    }

    if (s_tiles > 0) {
        const bf16_t *kbase = k + (int64_t)b * s.l_x * ld + (int64_t)h * D;
        const bf16_t *vbase = v + (int64_t)b * s.l_x * ld + (int64_t)h * D;

        // dropout: this lane's row keys; the column seed; the column keys of tile t (global tile index)
        // are computed once, by one wavefront when the tile's loads are issued, into quarter t % 4 of
        // a small ring behind the tiles -- published by the same barrier as the tile
        uint32_t drop_rk[NJ], drop_cs = 0u;
        if (DROP) {
            drop_cs = drop_col_seed(dr.seed_hi);
#pragma unroll
            for (int j = 0; j < NJ; ++j) drop_rk[j] = drop_row_key(dr.seed_lo, (uint32_t)bh, (uint32_t)(s.s0 + rw0 + 16 * j + lq));
        }
        char *const ck_ring = ring + C::RING * C::SLOT;

        // ---- tile loads, by all wavefronts of the group.  No branch and few scalar instructions on purpose: a branch inside a
        // pipeline step splits it into basic blocks, and the vector work that was meant to sit between the step's matrix
        // instructions is then moved behind the branch in one lump; addresses move on between the iterations instead.
        uint32_t off[Tile::NI], offD[Tile::NI];         // this lane's global offsets within a full tile; and what must be
        Tile::pair_offsets(off, ld, C::BC, wave, lane); // added to them in the sequence's last, partial tile (rows past the end
        const int t_part = s.l_x % C::BC ? s.l_x / C::BC : -1;     // re-read the last row)
        {
            uint32_t offL[Tile::NI];
            Tile::pair_offsets(offL, ld, t_part >= 0 ? s.l_x % C::BC : C::BC, wave, lane);
#pragma unroll
            for (int i = 0; i < Tile::NI; ++i) offD[i] = offL[i] - off[i];
        }
        const uint32_t tile_bytes = (uint32_t)(C::BC * ld * 2);
        // the next tile to load; past the group's last one that one again, into a slot that nobody reads any more
        const int t_last = t_begin + max(T, 1) - 1;
        int t_next = t_begin;
        const char *k_next = tile_ptr(Tile::pair_base(kbase), t_begin, tile_bytes), *v_next = tile_ptr(Tile::pair_base(vbase), t_begin, tile_bytes);
        auto to_part = [&] {
            if (t_next == t_part)
#pragma unroll
                for (int i = 0; i < Tile::NI; ++i) off[i] += offD[i];
        };
        to_part();
        auto advance = [&] {
            if (t_next < t_last) {
                ++t_next;
                k_next += tile_bytes;
                v_next += tile_bytes;
                to_part();
            }
        };
        auto issue_next = [&](char *slot) __attribute__((always_inline)) {
            static_assert(C::OFF_V == Tile::BYTES, "V tile follows K tile");
            Tile::issue_pair(k_next, v_next, off, off, slot, wave);
            if (DROP && wave == 0)
                reinterpret_cast<uint32_t *>(ck_ring)[(t_next & 3) * C::BC + lane] = drop_col_key(drop_cs, (uint32_t)(t_next * C::BC + lane));
        };

        // ---- this lane's LDS addresses (bytes from smem) in the tile that A and in the one that C reads next; they move to the
        // next tile once per iteration (one vector addition each, not one per use)
        const int ring_at = group * C::group_lds(DROP);
        int a_at[NU / 2];                               // A-operand chunk of row lq for operand step ks
#pragma unroll
        for (int ks = 0; ks < NU / 2; ++ks) a_at[ks] = ring_at + Tile::chunk_offset(lq, 4 * ks + g);
        int t_at[NU];                                   // transposed reads, column block db
#pragma unroll
        for (int db = 0; db < NU; ++db) t_at[db] = ring_at + tr16_lane_offset_sw<D>(lane, db);

        // ---- stage pieces.  `kb2`: which half of the tile, a block of 32 keys.
        // Unit u: A operands of key block u % 2, operand step u / 2; C operand of column block u.
        auto load_a = [&](int kb2, int u, Frag<bf16_t> &fk, Frag<bf16_t> &fv) __attribute__((always_inline)) {
            const char *p = smem + a_at[u / 2] + (kb2 * 32 + u % 2 * 16) * (D * 2);
            fk = load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(p));
            fv = load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(p + C::OFF_V));
        };
        auto load_c = [&](int kb2, int u, Frag<bf16_t> &fk) __attribute__((always_inline)) {
            fk = load_frag_tr16_sw<D>(smem, kb2 * 32, t_at[u]);
        };
        // B for halves [h0, h1) of elements, element e = (i, j, v) = (e / (4 NJ), e / 4 % NJ, e % 4): P = 2^(c * S - lse * log2 e), dS = P * (dP - D);
        // finished pairs are rounded to bf16 into the operand fragments of C: slots 4 i + v of row block j
        // Nothing reads the result of the instruction before it, least of all a transcendental's: an exponent is made one element ahead of
        // its exponential, which the multiply that consumes it follows one element behind.  Half an element's work at a time -- even h:
        // exponential of element h / 2 and exponent of the next, odd h: the rest of the element before -- so that every
        // matrix instruction has some of it beside it and no two stand back to back, where the second's issue waits for the first.
        constexpr int NE = 8 * NJ;
        struct Block { f32x4 v[2][NJ]; };               // [key block i][row block j]: element v of this lane is key 16 i + 4 g + v
        // Dropout: a decision is a chain of eight instructions; its first round stands half an element ahead of the exponential, the second
        // beside it, the comparison and the choice beside the next one.  (All behind the exponential, and the factor 1 / (1 - p) in every dK/dV
        // element: 16 heads x 2 of 4096 rows behind 16384, 2765 us for the whole backward; 2690 so.)
        u32x4 ck4;      // the column keys of four consecutive keys
        uint32_t r1, r2;
        float mask;                 // M of the element that finish() is about to do
        auto load_keys = [&](int jb, int i) __attribute__((always_inline)) {
            if (DROP) ck4 = *reinterpret_cast<const u32x4 *>(ck_ring + (((jb >> 6) & 3) * C::BC + (jb & 63) + 16 * i + 4 * g) * 4);
        };
        auto round1 = [&](int e) __attribute__((always_inline)) { r1 = drop_round1(drop_rk[e / 4 % NJ], ck4[e & 3]); };
        auto choose = [&] __attribute__((always_inline)) { mask = drop_decide(r2, dr.thr) ? dr.scale : 0.f; };
        auto b_elems = [&](Block &sc, Block &dp, int jb, int h0, int h1, Frag<bf16_t> (&df)[NJ]) __attribute__((always_inline)) {
            auto finish = [&](int e) __attribute__((always_inline)) {       // sc holds P by now
                const int i = e / (4 * NJ), j = e / 4 % NJ, v = e & 3;
                f32x4 &d4 = dp.v[i][j];
                if (DROP) d4[v] = fmaf(d4[v], mask, -Dr[j]);            // (d4 holds dP, else dP - D)
                d4[v] = sc.v[i][j][v] * d4[v];
                if (v & 1) { df[j].v[4 * i + v - 1] = (bf16_t)d4[v - 1]; df[j].v[4 * i + v] = (bf16_t)d4[v]; }
            };
#pragma unroll
            for (int h = h0; h < h1; ++h) {
                const int e = h / 2, n = e + 1;
                if (h % 2 == 0) {
                    f32x4 &p4 = sc.v[e / (4 * NJ)][e / 4 % NJ], &n4 = sc.v[n / (4 * NJ) % 2][n / 4 % NJ];
                    if (e == 0) p4[0] = p4[0] * c - L2[0];
                    if (DROP && e == 0) round1(0);
                    const float next = n < NE ? n4[n & 3] * c - L2[n / 4 % NJ] : 0.f;
                    p4[e & 3] = fast_exp2(p4[e & 3]);
                    if (n < NE) n4[n & 3] = next;
                    if (DROP) {
                        if (e > 0) choose();
                        r2 = drop_round2(r1);
                    }
                } else {
                    if (e > 0) finish(e - 1);
                    if (DROP && n < NE) round1(n);
                    if (n == 4 * NJ - 1) load_keys(jb, 1);              // (the four before are done with)
                    if (n == NE) {
                        if (DROP) choose();
                        finish(e);
                    }
                }
            }
        };
        // Where the causal diagonal or the end of the sequence crosses a block (first key jb), the
        // masked elements of its finished S^T are set to -inf before B, which turns them
        // into P = dS = 0: keys after the lane's row, and keys past the sequence (whose loads
        // re-read its last row).
        // (positions are below 2^30, checked on the host: one 32-bit scalar compare, no vector work per step)
        const int last_whole = min(s.causal ? (int)s.s0 + rw0 - 31 : s.l_x, s.l_x - 32);       // blocks from here on need no mask
        auto mask_s = [&](int jb, Block &sc) __attribute__((always_inline)) {
            if (jb > last_whole) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const int last = s.causal ? min((int)s.s0 + rw0 + 16 * j + lq, s.l_x - 1) : s.l_x - 1;
                    const int rel = max(min(last - jb - 4 * g, 64), -1);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (16 * i + v > rel) sc.v[i][j][v] = -INFINITY;
                }
            }
        };

        // One pipeline step.  A: half kb2_a of its tile into (sc_a, dp_a).  B: (sc_b, dp_b), first key
        // jb_b, packing into df_b.  C: half kb2_c of its tile from df_c into acc.  Per unit NJ matrix
        // instructions of C and 2 NJ of A (A first in the last unit); after each one come the B elements that fall to its slot.
        // Operand fragments are read from LDS one unit ahead of their use; those of the first unit
        // by the step before (ak[0], av[0], ck[0] on entry), and this step leaves there those of
        // the next step: halves kb2_an and kb2_cn.  `mid` runs before those last reads: the even steps put the loop's barrier
        // there, because the next step's blocks may lie in the tile that the barrier publishes, and move the addresses on.
        Frag<bf16_t> ak[2], av[2], ck[2];
        auto step = [&](auto has_a, auto has_b, auto has_c, int kb2_a, Block &sc_a, Block &dp_a, Block &sc_b, Block &dp_b,
                        int jb_b, Frag<bf16_t> (&df_b)[NJ], int kb2_c, Frag<bf16_t> (&df_c)[NJ], int kb2_an, int kb2_cn, auto &&mid)
            __attribute__((always_inline)) {
            constexpr bool HA = decltype(has_a)::value, HB = decltype(has_b)::value, HC = decltype(has_c)::value;
            constexpr int PU = 3 * NJ, NS = PU * NU;    // slots per unit and in all; the elements of B spread over them
            static_assert(NU % 2 == 0, "fragment double buffers assume an even number of units");
            auto b_slot = [&](int slot) __attribute__((always_inline)) {
                if (HB) {
                    const int h0 = slot * 2 * NE / NS, h1 = (slot + 1) * 2 * NE / NS;
                    if (h0 == h1) return;
                    __builtin_amdgcn_sched_barrier(0);
                    b_elems(sc_b, dp_b, jb_b, h0, h1, df_b);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            if (HB) {
                load_keys(jb_b, 0);
                mask_s(jb_b, sc_b);
                // B's inputs pass through an empty asm here: its arithmetic depends on nothing else in
                // this step, and the compiler would otherwise move all of it out of the step, in one lump
#pragma unroll
                for (int n = 0; n < 2 * NJ; ++n) asm volatile("" : "+v"(sc_b.v[n / NJ][n % NJ]), "+v"(dp_b.v[n / NJ][n % NJ]));
            }
            auto do_a = [&](int u, int slot) __attribute__((always_inline)) {
                const int i = u % 2, ks = u / 2;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    if (HA) sc_a.v[i][j] = mma16(ak[u & 1], qf[ks][j], ks == 0 ? zero4 : sc_a.v[i][j]);
                    b_slot(slot + j);
                }
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    if (HA) dp_a.v[i][j] = mma16(av[u & 1], gf[ks][j], ks == 0 ? (DROP ? zero4 : neg_d[j]) : dp_a.v[i][j]);
                    b_slot(slot + NJ + j);
                }
            };
            auto do_c = [&](int u, int slot) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    if (HC) acc[u][j] = mma16(ck[u & 1], df_c[j], acc[u][j]);
                    b_slot(slot + j);
                }
            };
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                if (u + 1 < NU) {
                    if (HC) load_c(kb2_c, u + 1, ck[(u + 1) & 1]);
                    if (HA) load_a(kb2_a, u + 1, ak[(u + 1) & 1], av[(u + 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    wait_lds<(HC ? 2 : 0) + (HA ? 2 : 0)>();        // this unit's are there (one wait, not one per fragment)
                    __builtin_amdgcn_sched_barrier(0);
                    do_c(u, PU * u);
                    do_a(u, PU * u + NJ);
                } else {
                    // last unit: A first, so that its results are there when the next step's B wants them
                    do_a(u, PU * u);
                    mid();
                    load_c(kb2_cn, 0, ck[0]);
                    load_a(kb2_an, 0, ak[0], av[0]);
                    __builtin_amdgcn_sched_barrier(0);
                    do_c(u, PU * u + 2 * NJ);
                }
            }
            // ... and its results through another one, so that it is not sunk below the step either
            if (HB)
#pragma unroll
                for (int j = 0; j < NJ; ++j) asm volatile("" : "+v"(df_b[j].v));
        };
        using std::true_type;
        using std::false_type;

        // ---- pipeline.  Block g = keys (t_begin + g/2) * 64 + (g%2) * 32 ..; tile t = blocks 2t, 2t+1.
        if (T > 0) issue_next(ring);
        advance();
        if (T > 1) issue_next(ring + C::SLOT);
        advance();
        wait_vmem_all();
        __syncthreads();

        if (rw0 >= s.l_s) {
            // None of this wavefront's rows exists (a partly filled last query tile; half the workgroup for
            // a segment of at most 64 rows): it only keeps moving tiles and meeting the loop's barriers.
            char *cur = ring, *nxt = ring + C::SLOT, *prv = ring + 2 * C::SLOT;
            for (int t = 0; t < T; ++t) {
                wait_vmem_all();
                __syncthreads();
                issue_next(prv);
                advance();
                char *const free = cur;
                cur = nxt, nxt = prv, prv = free;
            }
        } else if (KG == 1 || T > 0) {
            Block sc0, dp0, sc1, dp1;                       // even / odd blocks
            Frag<bf16_t> df0[NJ], df1[NJ];
            // step -1: A(0) alone.  The first loop step has no C(-1): it multiplies zeros with tile 0 instead.
            load_a(0, 0, ak[0], av[0]);
            auto nothing = [] {};
            step(true_type{}, false_type{}, false_type{}, 0, sc0, dp0, sc1, dp1, 0, df0, 0, df1, 1, 1, nothing);
    #pragma unroll
            for (int j = 0; j < NJ; ++j)
    #pragma unroll
                for (int e = 0; e < 8; ++e) df1[j].v[e] = (bf16_t)0.f;

            // ring slots (bytes): of tile t, of the next, the one that takes the tile after that (tile t - 1's); C's way to tile t
            int cur = 0, nxt = C::SLOT, prv = 2 * C::SLOT, c_step = 0;
            int j0 = t_begin * C::BC;
            for (int t = 0; t < T; ++t) {
                // even step g = 2t: A(2t+1) [tile t, second half], B(2t), C(2t-1) [tile t-1, second half;
                // for t = 0 tile 0, times zero]
                // Before its last reads (which may touch tile t+1): tile t+1's loads, issued one iteration
                // ago, have landed for this wavefront; after the barrier for all, and every wavefront has
                // requested its last operands from tile t-1, whose slot takes tile t+2.
                step(true_type{}, true_type{}, true_type{}, 1, sc1, dp1, sc0, dp0, j0, df0, 1, df1, 0, 0, [&] {
                    wait_vmem_all();
                    __syncthreads();
                    issue_next(ring + prv);
#pragma unroll
                    for (int ks = 0; ks < NU / 2; ++ks) a_at[ks] += nxt - cur;
#pragma unroll
                    for (int db = 0; db < NU; ++db) t_at[db] += c_step;
                });
                // odd step g = 2t+1: A(2t+2) [tile t+1, first half; past the end of whatever its slot holds, result unused],
                // B(2t+1), C(2t) [tile t, first half]
                step(true_type{}, true_type{}, true_type{}, 0, sc0, dp0, sc1, dp1, j0 + 32, df1, 0, df0, 1, 1, nothing);
                advance();
                c_step = nxt - cur;
                const int used = cur;
                cur = nxt, nxt = prv, prv = used;
                j0 += C::BC;
            }
            // step 2T: C(2T-1) [tile T-1, second half] alone
            step(false_type{}, false_type{}, true_type{}, 0, sc0, dp0, sc0, dp0, 0, df0, 1, df1, 0, 1, nothing);
        }
        if (KG > 1)
            for (int t = T; t < iters; ++t) __syncthreads();           // the barriers of the group that has more tiles
        wait_vmem_all();                                // the last, redundant prefetches must land before the workgroup's LDS is given away
    }

    if constexpr (KG > 1) {
        // The groups' sums meet in LDS, where the tiles were: each adds up half the columns, in group order.
        static_assert(KG == 2 && D == 64 && NJ == 2, "");
        auto hand = [&](int of, int u) { return reinterpret_cast<f32x4 *>(smem + ((of * C::WAVES + wave) * NU + u) * 1024 + lane * 16); };
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NU; ++u) *hand(group, u) = group == 0 ? acc[NU / 2 + u / 2][u % 2] : acc[u / 2][u % 2];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NU; ++u)
            acc[u / 2][u % 2] = (group == 0 ? acc[u / 2][u % 2] : acc[NU / 2 + u / 2][u % 2]) + *hand(group ^ 1, u);
    }
    const float scale = 1.f / sqrtf((float)D);
    constexpr int DB = KG > 1 ? NU / 2 : NU;            // (two groups: half the column blocks, in the first half of acc)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int r = rw0 + 16 * j + lq;
        if (r >= s.l_s) continue;
        const int64_t at = ((int64_t)b * s.l_s + r) * ld + (int64_t)h * D + (KG > 1 ? 16 * DB * group : 0) + 4 * g;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const f32x4 a = acc[db][j];
            const f32x4 val = {a[0] * scale, a[1] * scale, a[2] * scale, a[3] * scale};
            if (n_splits == 1) *reinterpret_cast<bf16x4 *>(dq + at + 16 * db) = pack4(val[0], val[1], val[2], val[3]);
            else *reinterpret_cast<f32x4 *>(dq_part + (int64_t)split * s.B * s.l_s * ld + at + 16 * db) = val;
        }
    }
}

// ------------------------------------------------------------------------------------------ dK, dV
// A wavefront's finished [32 keys][D] tile (accumulator layout: lane = key lq, element e of block db =
// column 32 db + 8 (e / 4) + 4 hh + e % 4) goes to memory through a wavefront-private LDS buffer of
// 32 * D * 4 bytes, so that every store instruction writes whole rows (1 KB contiguous per four or
// two keys) instead of 32-byte pieces of 32 rows.  16-byte chunk c of key row r sits at chunk
// position c ^ (r % chunks per row).  `rows_ok` keys of the block exist.
template <int D>
__device__ __forceinline__ void store_key_rows(char *buf, const f32x16 (&acc)[D / 32], float scale, float *__restrict__ dst,
                                               int64_t ld, int rows_ok, int lane)
{
    constexpr int CH = D / 4;                           // 16-byte chunks per row
    const int lq = lane & 31, hh = lane >> 5;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            const int c = db * 8 + 2 * e4 + hh;
            *reinterpret_cast<f32x4 *>(buf + lq * (D * 4) + ((c ^ (lq & (CH - 1))) * 16)) =
                f32x4{acc[db][4 * e4] * scale, acc[db][4 * e4 + 1] * scale, acc[db][4 * e4 + 2] * scale, acc[db][4 * e4 + 3] * scale};
        }
    constexpr int RPI = 64 / CH;                        // rows per store instruction
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
        const int row = i * RPI + lane / CH, c = lane % CH;
        const f32x4 val = *reinterpret_cast<const f32x4 *>(buf + row * (D * 4) + ((c ^ (row & (CH - 1))) * 16));
        if (row < rows_ok) *reinterpret_cast<f32x4 *>(dst + (int64_t)row * ld + c * 4) = val;
    }
}

// The same for a tile held as 16 x 16 blocks: block (db, j), element v of a lane is key 16 j + lane % 16, column
// 16 db + 4 (lane / 16) + v.
template <int D, int NJ>
__device__ __forceinline__ void store_key_rows16(char *buf, const f32x4 (&acc)[D / 16][NJ], float scale, float *__restrict__ dst,
                                                 int64_t ld, int rows_ok, int lane)
{
    constexpr int CH = D / 4;                           // 16-byte chunks per row
#pragma unroll
    for (int db = 0; db < D / 16; ++db)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int key = 16 * j + (lane & 15), c = 4 * db + (lane >> 4);
            const f32x4 a = acc[db][j];
            *reinterpret_cast<f32x4 *>(buf + key * (D * 4) + ((c ^ (key & (CH - 1))) * 16)) = f32x4{a[0] * scale, a[1] * scale, a[2] * scale, a[3] * scale};
        }
    constexpr int RPI = 64 / CH;                        // rows per store instruction
#pragma unroll
    for (int i = 0; i < 16 * NJ / RPI; ++i) {
        const int row = i * RPI + lane / CH, c = lane % CH;
        const f32x4 val = *reinterpret_cast<const f32x4 *>(buf + row * (D * 4) + ((c ^ (row & (CH - 1))) * 16));
        if (row < rows_ok) *reinterpret_cast<f32x4 *>(dst + (int64_t)row * ld + c * 4) = val;
    }
}

template <int D, bool DROP = false, int NJ = 2>
struct DkvBf16Cfg {
    // One 32-row key block per wavefront.  Two blocks would halve the LDS traffic per flop but
    // their accumulators leave room for only one wavefront per SIMD, which measures slower.
    static constexpr int WAVES = 8 / NJ, KW = 16 * NJ;  // key rows per wavefront: NJ blocks of 16
    static constexpr int BKV = WAVES * KW, BQ = 64, NT = 64 * WAVES;
    static constexpr int RING = 3;                      // Q/dO tiles resident in LDS
    static constexpr int NU = D / 16;                   // operand steps of the S/dP products; same for dV/dK
    using Tile = DirectTile<D, BQ, WAVES>;
    // one ring slot: Q tile, dO tile, 64 S-accumulator start values, 64 dP-accumulator start values
    // (with dropout also the 64 rows' generator keys)
    static constexpr int OFF_G = Tile::BYTES, OFF_L = 2 * Tile::BYTES, OFF_D = OFF_L + BQ * 4, OFF_R = OFF_D + BQ * 4;
    static constexpr int SLOT = OFF_R + (DROP ? BQ * 4 : 0);
    // OWN workgroups: the start values (and keys) of all rows behind the rings, up to OWN_MAX rows and one more tile
    static constexpr int OWN_MAX = kOwnRows, OWN_ROWS = OWN_MAX + BQ, OWN_BYTES = OWN_ROWS * 4 * (DROP ? 3 : 2);
};

// -D = -rowsum(dO * out) of a row from its parts: D/8 consecutive lanes hold one 16-byte chunk each.
template <int D>
__device__ __forceinline__ float neg_row_dot(const Frag<bf16_t> &g, const Frag<bf16_t> &o)
{
    float dsum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) dsum += (float)g.v[e] * (float)o.v[e];
#pragma unroll
    for (int sh = 1; sh < D / 8; sh <<= 1) dsum += __shfl_xor(dsum, sh);
    return -dsum;
}
// The same for `n` rows that lie `ld` elements apart, by a workgroup of NT: put(row, -D, lse) on one lane per row.  The
// loads of 128 (d = 64) or 64 rows are in flight at once.
template <int D, int NT = 256, typename Put>
__device__ __forceinline__ void neg_row_dots(const bf16_t *__restrict__ out, const bf16_t *__restrict__ dO,
                                             const float *__restrict__ lse, int64_t ld, int n, int tid, Put &&put)
{
    constexpr int CPR = D / 8, STEP = NT / CPR, U = 4;
    const int cpos = tid % CPR;
    for (int i0 = tid / CPR; i0 - tid / CPR < n; i0 += U * STEP) {
        Frag<bf16_t> g[U], o[U];
        float l[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = min(i0 + u * STEP, n - 1);
            const int64_t off = i * ld + cpos * 8;
            l[u] = lse[i];
            g[u] = load_frag<bf16_t>(dO + off);
            o[u] = load_frag<bf16_t>(out + off);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float nd = neg_row_dot<D>(g[u], o[u]);
            if (cpos == 0 && i0 + u * STEP < n) put(i0 + u * STEP, nd, l[u]);
        }
    }
}

// The query rows are walked in blocks of 32 (two per 64-row Q/dO tile).  Per block g three stages:
//     A(g): S and dP products (matrix),  B(g): weights P, dS (vector: exp, multiplies, bf16 packing),
//     C(g): dV^T and dK^T products (matrix).
// A wavefront issues in order, and vector work costs it several times the issue time of a matrix
// instruction, so the stages are software-pipelined: step g issues the matrix instructions of
// A(g+1) and C(g-1) with the vector work of B(g) spread between them, one element per matrix
// instruction.  Block g+1 may belong to the next tile and block g-1 to the previous one, hence a
// ring of three tiles in LDS; tiles travel global -> LDS directly, a full loop iteration ahead.
//
// With dropout (DROP) the weight that enters dV is A = P * M (M = 1 / (1 - p) where the weight is
// kept, else 0) and dS = P * (M * dP - D); the dP accumulator starts at 0.  Both are made without the factor 1 / (1 - p), which the
// finished sums get: K (kept) = P or 0, dS = K * dP - P * D (1 - p).  The keep decision of an element needs its row's key
// (precomputed per query row, travelling with the tile like the start values) and this lane's column key; -D (1 - p) of the element's row is read from the tile's start values.
//
// OWN: the workgroup computes the start values (and keys) of its rows itself, into LDS, while its first
// tiles are on their way, instead of finding them in memory (bwd_own_values).
template <int D, bool DROP, bool OWN, int KG, int NJ>
__device__ __forceinline__ void bwd_dkv_body(char *smem, const SegShape &s, const DropArgs &dr, const bf16_t *__restrict__ q,
                                             const bf16_t *__restrict__ k, const bf16_t *__restrict__ v,
                                             const bf16_t *__restrict__ out, const bf16_t *__restrict__ dO,
                                             const float *__restrict__ lse, const float *__restrict__ Ls,
                                             const float *__restrict__ Dn, const uint32_t *__restrict__ row_key,
                                             float *__restrict__ dk_part, float *__restrict__ dv_part, int bh, int key_tile)
{
    using C = DkvBf16Cfg<D, DROP, NJ>;
    using Tile = typename C::Tile;
    constexpr int NU = C::NU;

    const int tid = threadIdx.x, lane = tid & 63, lk = lane & 15, g = lane >> 4;
    const int all_waves = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = KG > 1 ? all_waves / C::WAVES : 0, wave = KG > 1 ? all_waves % C::WAVES : all_waves;     // wave: within the group
    char *const ring = smem + group * (C::RING * C::SLOT), *const own_values = smem + KG * (C::RING * C::SLOT);
    const int b = bh / s.H, h = bh % s.H;
    const int j0 = key_tile * C::BKV;
    const int jw0 = j0 + wave * C::KW;                  // first key of this wavefront
    const int64_t ld = (int64_t)s.H * D;
    const int64_t kv_base = (int64_t)b * s.l_x * ld + (int64_t)h * D;

    // first query row that sees any key of this workgroup's tile
    int rq_begin = 0;
    if (s.causal) {
        const int64_t first = (int64_t)j0 - s.s0;
        rq_begin = first > 0 ? (int)min<int64_t>(first, s.l_s) : 0;
        rq_begin = rq_begin / C::BQ * C::BQ;
    }

    if (s.causal && j0 >= s.s0 + s.l_s) {
        // no query of the segment sees this tile: its partial rows are zero (coalesced fill), or stay
        // unwritten if the caller asked for that
        if (s.skip_tail) return;
        constexpr int F4 = D / 4;                       // float4 per (row, head)
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        for (int i = tid; i < C::BKV * F4; i += KG * C::NT) {
            const int row = j0 + i / F4, c4 = (i % F4) * 4;
            if (row < s.l_x) {
                *reinterpret_cast<f32x4 *>(dk_part + kv_base + (int64_t)row * ld + c4) = z;
                *reinterpret_cast<f32x4 *>(dv_part + kv_base + (int64_t)row * ld + c4) = z;
            }
        }
        return;
    }

    // this lane's keys (columns of the S blocks), jw0 + 16 j + lk; keys past the sequence re-read its last row
    // (unconditional loads), take part in all the arithmetic and are never stored
    Frag<bf16_t> kf[NU / 2][NJ], vf[NU / 2][NJ];        // operand step ks (32 columns), key block j
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int64_t off = kv_base + (int64_t)min(jw0 + 16 * j + lk, s.l_x - 1) * ld + g * 8;
#pragma unroll
        for (int ks = 0; ks < NU / 2; ++ks) {
            kf[ks][j] = load_frag<bf16_t>(k + off + ks * 32);
            vf[ks][j] = load_frag<bf16_t>(v + off + ks * 32);
        }
    }
    if constexpr (D == 128 && NJ == 2) {
        // At d = 128 the kernel needs more than 256 registers and the allocator parks these 64 in the
        // accumulation half of the register file -- then copies each into a vector register before
        // every use (54 to 68 copies per 32 matrix instructions).  A matrix instruction can read its
        // B operand from that half directly: naming the class here makes it do so.
#pragma unroll
        for (int n = 0; n < NU; ++n) {
            asm volatile("" : "+a"(kf[n / 2][n % 2].v));
            asm volatile("" : "+a"(vf[n / 2][n % 2].v));
        }
    }

    const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
    f32x4 dk[NU][NJ], dv[NU][NJ];                       // 16 columns x 16 keys each, transposed
#pragma unroll
    for (int db = 0; db < NU; ++db)
#pragma unroll
        for (int j = 0; j < NJ; ++j) dk[db][j] = dv[db][j] = zero4;

    const float sqrt_d = sqrtf((float)D);
    const float c = kLog2e / sqrt_d;
    const bf16_t *qbase = q + (int64_t)b * s.l_s * ld + (int64_t)h * D;
    const bf16_t *gbase = dO + (int64_t)b * s.l_s * ld + (int64_t)h * D;
    const float *lbase = Ls + (int64_t)bh * s.l_s, *dbase = Dn + (int64_t)bh * s.l_s;
    const uint32_t *rbase = DROP ? row_key + (int64_t)bh * s.l_s : nullptr;
    uint32_t drop_ck[NJ];                                // this lane's keys
    if (DROP)
#pragma unroll
        for (int j = 0; j < NJ; ++j) drop_ck[j] = drop_col_key(drop_col_seed(dr.seed_hi), (uint32_t)(jw0 + 16 * j + lk));

    // ---- tile loads: all wavefronts of the group move Q and dO, and the 64 start values of either kind (even
    // wavefronts -lse*sqrt(d), odd ones -D; each several times, which is cheaper than a branch inside a pipeline
    // step).  As in the dQ workgroups addresses move on between the iterations.
    // (two groups: the first has `iters` tiles, the other one fewer or none; row_base: of the group's first row, from rq_begin)
    const int all_tiles = (s.l_s - rq_begin + C::BQ - 1) / C::BQ, iters = (all_tiles + KG - 1) / KG;
    const int T = KG > 1 ? min(all_tiles - group * iters, iters) : all_tiles, row_base = group * iters * C::BQ;
    const int tq_begin = (rq_begin + row_base) / C::BQ;
    uint32_t off[Tile::NI], offD[Tile::NI];             // this lane's global offsets within a full tile; and what must be
    Tile::pair_offsets(off, ld, C::BQ, wave, lane);     // added to them in the segment's last, partial tile (rows past the end
    const int tq_part = s.l_s % C::BQ ? s.l_s / C::BQ : -1;        // re-read the last row)
    {
        uint32_t offL[Tile::NI];
        Tile::pair_offsets(offL, ld, tq_part >= 0 ? s.l_s % C::BQ : C::BQ, wave, lane);
#pragma unroll
        for (int i = 0; i < Tile::NI; ++i) offD[i] = offL[i] - off[i];
    }
    const uint32_t tile_bytes = (uint32_t)(C::BQ * ld * 2);
    const float *const sv_base = (wave & 1) ? dbase : lbase;
    const int sv_slot = (wave & 1) ? C::OFF_D : C::OFF_L;
    // the next tile to load (tile tq: query rows [64 tq, 64 tq + 64) of the segment); past the group's last one that one again, into a
    // slot that nobody reads any more.  (A second group without tiles loads nothing.)
    const int tq_last = tq_begin + max(T, 1) - 1;
    int tq_next = tq_begin;
    const char *q_next = tile_ptr(Tile::pair_base(qbase), tq_begin, tile_bytes), *g_next = tile_ptr(Tile::pair_base(gbase), tq_begin, tile_bytes);
    uint32_t sv_off = (uint32_t)(tq_begin * C::BQ + lane) * 4u;
    const uint32_t sv_end = (uint32_t)(s.l_s - 1) * 4u;
    auto to_part = [&] {
        if (tq_next == tq_part)
#pragma unroll
            for (int i = 0; i < Tile::NI; ++i) off[i] += offD[i];
    };
    to_part();
    auto advance = [&] {
        if (tq_next < tq_last) {
            ++tq_next;
            q_next += tile_bytes;
            g_next += tile_bytes;
            sv_off += C::BQ * 4u;
            to_part();
        }
    };
    auto issue_next = [&](char *slot) __attribute__((always_inline)) {
        static_assert(C::OFF_G == Tile::BYTES, "dO tile follows Q tile");
        Tile::issue_pair(q_next, g_next, off, off, slot, wave);
        if constexpr (!OWN) {
            const uint32_t so = min(sv_off, sv_end);
            lds_dma<4>(sv_base, so, slot + sv_slot);
            if (DROP && wave == 2) lds_dma<4>(rbase, so, slot + C::OFF_R);
        }
    };

    // ---- this lane's LDS addresses (bytes from smem) in the tile that A and in the one that C reads next; they move to the
    // next tile once per iteration (one vector addition each, not one per use)
    const int ring_at = group * (C::RING * C::SLOT);
    int a_at[NU / 2];                                   // A-operand chunk of row lk for operand step ks
#pragma unroll
    for (int ks = 0; ks < NU / 2; ++ks) a_at[ks] = ring_at + Tile::chunk_offset(lk, 4 * ks + g);
    int t_at[NU];                                       // transposed reads, column block db
#pragma unroll
    for (int db = 0; db < NU; ++db) t_at[db] = ring_at + tr16_lane_offset_sw<D>(lane, db);
    // Accumulators of A start at -lse*sqrt(d) and -D of their rows: element v of this lane's block (i, j) is
    // query row 16 i + 4 g + v.  sv_at: those of A's tile, in its slot, or with OWN behind the rings in the order of the rows, counted
    // from rq_begin; the -D and the row keys follow SV_D and SV_R bytes on.
    constexpr int SV_D = OWN ? C::OWN_ROWS * 4 : C::OFF_D - C::OFF_L, SV_R = 2 * SV_D;
    static_assert(OWN || SV_R == C::OFF_R - C::OFF_L, "start values lie in one row of arrays");
    int sv_at = (OWN ? KG * (C::RING * C::SLOT) + row_base * 4 : ring_at + C::OFF_L) + 4 * g * 4;

    // ---- stage pieces.  `qb`: which half of the tile, a block of 32 rows.
    // Unit u: A operands of row block u % 2, operand step u / 2; C operands of column block u.
    auto load_a = [&](int qb, int u, Frag<bf16_t> &fq, Frag<bf16_t> &fg) __attribute__((always_inline)) {
        const char *p = smem + a_at[u / 2] + (qb * 32 + u % 2 * 16) * (D * 2);
        fq = load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(p));
        fg = load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(p + C::OFF_G));
    };
    auto load_c = [&](int qb, int u, Frag<bf16_t> &fq, Frag<bf16_t> &fg) __attribute__((always_inline)) {
        fq = load_frag_tr16_sw<D>(smem, qb * 32, t_at[u]);
        fg = load_frag_tr16_sw<D>(smem + C::OFF_G, qb * 32, t_at[u]);
    };
    f32x4 sv_l[2], sv_d[2];
    auto init_load = [&](int qb) __attribute__((always_inline)) {
        const char *sv = smem + sv_at + qb * 32 * 4;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            sv_l[i] = *reinterpret_cast<const f32x4 *>(sv + i * 64);
            if constexpr (!DROP) sv_d[i] = *reinterpret_cast<const f32x4 *>(sv + SV_D + i * 64);
        }
    };
    // Where the causal diagonal or the end of the segment crosses the block (first row: local row
    // r0), the masked elements of its finished S are set to -inf, which B turns into P = dS = 0: rows before
    // the lane's key, and rows past the segment (whose loads re-read its last row).
    constexpr int NE = 8 * NJ;
    struct Block { f32x4 v[2][NJ]; };                   // [row block i][key block j]
    // Blocks whose first row lies in [whole_from, whole_from + whole_span] need no mask (positions are below 2^30: one 32-bit scalar
    // compare per step); where there is none, whole_from is out of every block's reach.
    const int from = s.causal ? max(jw0 + C::KW - 1 - (int)s.s0, 0) : 0;
    const int whole_from = from > s.l_s - 32 ? 0x7fffffff : from;
    const uint32_t whole_span = from > s.l_s - 32 ? 0u : (uint32_t)(s.l_s - 32 - from);
    auto mask_s = [&](int r0, Block &sc) __attribute__((always_inline)) {
        if ((uint32_t)(r0 - whole_from) > whole_span) {
            const bool diag = s.causal && (jw0 + C::KW - 1 > (int)s.s0 + r0);
            const int end = min(s.l_s - r0, 32) - 4 * g;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int first = diag ? max(min(jw0 + 16 * j + lk - (int)s.s0 - r0 - 4 * g, 64), 0) : 0;
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (16 * i + v < first || 16 * i + v >= end) sc.v[i][j][v] = -INFINITY;
            }
        }
    };
    // B for halves [h0, h1) of elements, element e = (i, j, v) = (e / (4 NJ), e / 4 % NJ, e % 4): P = 2^(c * (S - lse*sqrt(d))), dS = P * (dP - D);
    // finished pairs are rounded to bf16 into the operand fragments of C: slots 4 i + v of key block j.
    // (Exponent, exponential and the multiplies that consume it one element apart, half an element at a time, and a decision's pieces
    // likewise, as in the dQ workgroups.)
    // (dropout: `sv_b` are B's start values, from which the row keys and -D of four rows come ahead of the first of them)
    u32x4 rk4;
    f32x4 nd4;
    uint32_t r1, r2;
    float kept;                 // the weight in front of finish(), or 0
    auto load_keys = [&](int sv_b, int i) __attribute__((always_inline)) {
        if constexpr (DROP) rk4 = *reinterpret_cast<const u32x4 *>(smem + sv_b + SV_R + i * 64);
    };
    auto load_d = [&](int sv_b, int i) __attribute__((always_inline)) {
        if constexpr (DROP) nd4 = *reinterpret_cast<const f32x4 *>(smem + sv_b + SV_D + i * 64);
    };
    auto round1 = [&](int e) __attribute__((always_inline)) {
        if constexpr (DROP) r1 = drop_round1(rk4[e & 3], drop_ck[e / 4 % NJ]);
    };
    auto choose = [&](float p) __attribute__((always_inline)) {
        if constexpr (DROP) kept = drop_decide(r2, dr.thr) ? p : 0.f;
    };
    auto b_elems = [&](int sv_b, Block &sc, Block &dp, int h0, int h1, Frag<bf16_t> (&pf)[NJ],
                       Frag<bf16_t> (&df)[NJ]) __attribute__((always_inline)) {
        auto finish = [&](int e) __attribute__((always_inline)) {           // sc holds P by now
            const int i = e / (4 * NJ), j = e / 4 % NJ, v = e & 3;
            f32x4 &p4 = sc.v[i][j], &d4 = dp.v[i][j];
            if constexpr (DROP) {
                d4[v] = fmaf(kept, d4[v], p4[v] * nd4[v]);
                p4[v] = kept;
            } else {
                d4[v] = p4[v] * d4[v];
            }
            if (v & 1) {
                pf[j].v[4 * i + v - 1] = (bf16_t)p4[v - 1]; pf[j].v[4 * i + v] = (bf16_t)p4[v];
                df[j].v[4 * i + v - 1] = (bf16_t)d4[v - 1]; df[j].v[4 * i + v] = (bf16_t)d4[v];
            }
        };
#pragma unroll
        for (int h = h0; h < h1; ++h) {
            const int e = h / 2, n = e + 1;
            if (h % 2 == 0) {
                f32x4 &p4 = sc.v[e / (4 * NJ)][e / 4 % NJ], &n4 = sc.v[n / (4 * NJ) % 2][n / 4 % NJ];
                if (e == 0) {
                    p4[0] = p4[0] * c;
                    load_d(sv_b, 0);
                    round1(0);
                }
                const float next = n < NE ? n4[n & 3] * c : 0.f;
                p4[e & 3] = fast_exp2(p4[e & 3]);
                if (n < NE) n4[n & 3] = next;
                if constexpr (DROP) {
                    if (e > 0) choose(sc.v[(e - 1) / (4 * NJ)][(e - 1) / 4 % NJ][(e - 1) & 3]);
                    r2 = drop_round2(r1);
                }
            } else {
                if (e > 0) finish(e - 1);
                if (n < NE) round1(n);
                if (n == 4 * NJ - 1) load_keys(sv_b, 1);                // (the four before are done with)
                if (e == 4 * NJ) load_d(sv_b, 1);
                if (n == NE) {
                    choose(sc.v[1][NJ - 1][3]);
                    finish(e);
                }
            }
        }
    };
    // One pipeline step.  A: half qb_a of its tile into (sc_a, dp_a), from the start values in sv_l and sv_d.  B: (sc_b, dp_b),
    // first row r0_b, packing into (pf_b, df_b).  C: half qb_c of its tile from (pf_c, df_c) into dk, dv.  Per unit 2 NJ matrix
    // instructions of C and 2 NJ of A (A first in the last unit), each pair on one operand fragment; after each come the B
    // elements that fall to its slot.
    // Everything read from LDS is requested well before its use: operand fragments one unit ahead;
    // for the next step (halves qb_an and qb_cn) this step's last unit requests the fragments of both's first unit and the start
    // values of A's accumulators.  `mid` runs before those last requests: the even steps put the loop's barrier there, because
    // the next step's A block may lie in the tile that the barrier publishes, and move the addresses on.
    Frag<bf16_t> cq[2], cg[2], aq[2], ag[2];
    auto step = [&](auto has_a, auto has_b, auto has_c, int qb_a, Block &sc_a, Block &dp_a, int sv_b, int r0_b, Block &sc_b,
                    Block &dp_b, Frag<bf16_t> (&pf_b)[NJ], Frag<bf16_t> (&df_b)[NJ], int qb_c, Frag<bf16_t> (&pf_c)[NJ],
                    Frag<bf16_t> (&df_c)[NJ], int qb_an, int qb_cn, auto &&mid) __attribute__((always_inline)) {
        constexpr bool HA = decltype(has_a)::value, HB = decltype(has_b)::value, HC = decltype(has_c)::value;
        constexpr int PU = 4 * NJ, NS = PU * NU;        // slots per unit and in all; the elements of B spread over them
        static_assert(NU % 2 == 0, "fragment double buffers assume an even number of units");
        auto b_slot = [&](int slot) __attribute__((always_inline)) {
            if (HB) {
                const int h0 = slot * 2 * NE / NS, h1 = (slot + 1) * 2 * NE / NS;
                if (h0 == h1) return;
                __builtin_amdgcn_sched_barrier(0);
                b_elems(sv_b, sc_b, dp_b, h0, h1, pf_b, df_b);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // B's inputs pass through an empty asm here: its arithmetic depends on nothing else in this
        // step, and the compiler would otherwise move all of it out of the step, in one lump
        if (HB) {
            load_keys(sv_b, 0);
            mask_s(r0_b, sc_b);
#pragma unroll
            for (int n = 0; n < 2 * NJ; ++n) asm volatile("" : "+v"(sc_b.v[n / NJ][n % NJ]), "+v"(dp_b.v[n / NJ][n % NJ]));
        }
        auto do_a = [&](int u, int slot) __attribute__((always_inline)) {
            const int i = u % 2, ks = u / 2;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (HA) sc_a.v[i][j] = mma16(aq[u & 1], kf[ks][j], ks == 0 ? sv_l[i] : sc_a.v[i][j]);
                b_slot(slot + j);
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (HA) dp_a.v[i][j] = mma16(ag[u & 1], vf[ks][j], ks == 0 ? (DROP ? zero4 : sv_d[i]) : dp_a.v[i][j]);
                b_slot(slot + NJ + j);
            }
        };
        auto do_c = [&](int u, int slot) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (HC) dv[u][j] = mma16(cg[u & 1], pf_c[j], dv[u][j]);
                b_slot(slot + j);
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (HC) dk[u][j] = mma16(cq[u & 1], df_c[j], dk[u][j]);
                b_slot(slot + NJ + j);
            }
        };
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (u + 1 < NU) {
                if (HC) load_c(qb_c, u + 1, cq[(u + 1) & 1], cg[(u + 1) & 1]);
                if (HA) load_a(qb_a, u + 1, aq[(u + 1) & 1], ag[(u + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                wait_lds<(HC ? 4 : 0) + (HA ? 2 : 0)>();            // this unit's are there (one wait, not one per fragment)
                __builtin_amdgcn_sched_barrier(0);
                do_c(u, PU * u);
                do_a(u, PU * u + 2 * NJ);
            } else {
                // last unit: A first, so that its results are there when the next step's B wants them
                do_a(u, PU * u);
                mid();
                load_c(qb_cn, 0, cq[0], cg[0]);
                load_a(qb_an, 0, aq[0], ag[0]);
                init_load(qb_an);
                __builtin_amdgcn_sched_barrier(0);
                do_c(u, PU * u + 2 * NJ);
            }
        }
        // ... and its results through another one, so that it is not sunk below the step either
        if (HB)
#pragma unroll
            for (int j = 0; j < NJ; ++j) asm volatile("" : "+v"(pf_b[j].v), "+v"(df_b[j].v));
    };
    using std::true_type;
    using std::false_type;

    // ---- pipeline.  Block g of this workgroup = rows rq_begin + 32 g ..; tile t = blocks 2t, 2t+1.
    if (KG == 1 || T > 0) issue_next(ring);
    advance();
    if (T > 1) issue_next(ring + C::SLOT);
    advance();
    if constexpr (OWN) {
        float *const own = reinterpret_cast<float *>(own_values);
        const int n = s.l_s - rq_begin;
        for (int i = n + tid; i < (all_tiles + 1) * C::BQ; i += KG * C::NT) {    // rows past the segment, whose weights are 0: any finite values
            own[i] = own[C::OWN_ROWS + i] = 0.f;
            if constexpr (DROP) own[2 * C::OWN_ROWS + i] = 0.f;
        }
        const int64_t first = ((int64_t)b * s.l_s + rq_begin) * ld + (int64_t)h * D;
        neg_row_dots<D, KG * C::NT>(out + first, dO + first, lse + (int64_t)bh * s.l_s + rq_begin, ld, n, tid, [&](int i, float nd, float l) {
            own[i] = -l * sqrt_d;
            own[C::OWN_ROWS + i] = DROP ? nd / dr.scale : nd;
            if constexpr (DROP)
                reinterpret_cast<uint32_t *>(own)[2 * C::OWN_ROWS + i] = drop_row_key(dr.seed_lo, (uint32_t)bh, (uint32_t)(s.s0 + rq_begin + i));
        });
    }
    wait_vmem_all();
    __syncthreads();

    if (KG == 1 || T > 0) {
        Block sc0, dp0, sc1, dp1;                       // even / odd blocks
        Frag<bf16_t> pf0[NJ], df0[NJ], pf1[NJ], df1[NJ];
        // step -1: A(0) alone (leaves the first loop step's C operands in cq[0], cg[0]).  That step has
        // no C(-1): it multiplies zeros with tile 0 instead.
        auto nothing = [] {};
        load_a(0, 0, aq[0], ag[0]);
        init_load(0);
        step(true_type{}, false_type{}, false_type{}, 0, sc0, dp0, 0, 0, sc1, dp1, pf0, df0, 0, pf1, df1, 1, 1, nothing);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) { pf1[j].v[e] = (bf16_t)0.f; df1[j].v[e] = (bf16_t)0.f; }

        // ring slots (bytes): of tile t, of the next, the one that takes the tile after that (tile t - 1's); C's way to tile t
        int cur = 0, nxt = C::SLOT, prv = 2 * C::SLOT, c_step = 0;
        int r0 = rq_begin + row_base;
#pragma nounroll    // (unrolled, two groups' registers spill: 84 spills against none)
        for (int t = 0; t < T; ++t) {
            const int sv_b = sv_at;                     // (dropout: B's rows, of tile t)
            // even step g = 2t: A(2t+1) [tile t, second half], B(2t), C(2t-1) [tile t-1, second half;
            // for t = 0 tile 0, times zero]
            // Before its last requests (which may touch tile t+1): tile t+1's loads, issued one iteration
            // ago, have landed for this wavefront; after the barrier for all, and every wavefront has
            // requested its last operands from tile t-1, whose slot takes tile t+2.
            step(true_type{}, true_type{}, true_type{}, 1, sc1, dp1, sv_b, r0, sc0, dp0, pf0, df0, 1, pf1, df1, 0, 0, [&] {
                wait_vmem_all();
                __syncthreads();
                issue_next(ring + prv);
#pragma unroll
                for (int ks = 0; ks < NU / 2; ++ks) a_at[ks] += nxt - cur;
#pragma unroll
                for (int db = 0; db < NU; ++db) t_at[db] += c_step;
                sv_at += OWN ? C::BQ * 4 : nxt - cur;
            });
            // odd step g = 2t+1: A(2t+2) [tile t+1, first half; past the end of whatever its slot holds, result unused],
            // B(2t+1), C(2t) [tile t, first half]
            step(true_type{}, true_type{}, true_type{}, 0, sc0, dp0, sv_b + 32 * 4, r0 + 32, sc1, dp1, pf1, df1, 0, pf0, df0, 1, 1, nothing);
            advance();
            c_step = nxt - cur;
            const int used = cur;
            cur = nxt, nxt = prv, prv = used;
            r0 += C::BQ;
        }
        // step 2T: C(2T-1) [tile T-1, second half] alone
        step(false_type{}, false_type{}, true_type{}, 0, sc0, dp0, 0, 0, sc0, dp0, pf0, df0, 1, pf1, df1, 0, 1, nothing);
    }
    if (KG > 1)
        for (int t = max(T, 0); t < iters; ++t) __syncthreads();       // the barriers of the group that has more tiles

    // the ring is free once every wavefront has made its last reads and the last, redundant prefetches have landed
    wait_vmem_all();
    __syncthreads();
    {
        // (a buffer per wavefront for its finished tile, see store_key_rows)
        char *buf = smem + all_waves * (C::KW * D * 4);
        const int64_t off = kv_base + (int64_t)jw0 * ld;
        const int rows_ok = min(s.l_x - jw0, C::KW);
        const float m = DROP ? dr.scale : 1.f;          // of the kept weights: applied to their sums
        if constexpr (KG == 1) {
            store_key_rows16<D, NJ>(buf, dk, m / sqrt_d, dk_part + off, ld, rows_ok, lane);
            store_key_rows16<D, NJ>(buf, dv, m, dv_part + off, ld, rows_ok, lane);
        } else {
            // The groups' sums meet in LDS: the first finishes dV, the second dK, adding in group order.  What a wavefront
            // reads was written for it alone, into the buffer that is its own from then on.
            static_assert(KG == 2 && D == 64 && NJ == 2, "");
            char *const theirs = smem + (all_waves ^ C::WAVES) * (32 * D * 4);
            f32x4 sum[NU][2];
#pragma unroll
            for (int u = 0; u < 2 * NU; ++u)
                *reinterpret_cast<f32x4 *>(theirs + u * 1024 + lane * 16) = group == 0 ? dk[u / 2][u % 2] : dv[u / 2][u % 2];
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 2 * NU; ++u)
                sum[u / 2][u % 2] = (group == 0 ? dv[u / 2][u % 2] : dk[u / 2][u % 2]) + *reinterpret_cast<const f32x4 *>(buf + u * 1024 + lane * 16);
            store_key_rows16<D, NJ>(buf, sum, group == 0 ? m : m / sqrt_d, (group == 0 ? dv_part : dk_part) + off, ld, rows_ok, lane);
        }
    }
}

// dK/dV for a segment of at most 64 query rows (the segment length the paper's largest runs leave
// one GPU): every key tile then meets ONE Q/dO tile, and the pipeline above would spend most of its
// steps on its start and its end.  Here a workgroup loads that tile once and walks KT_PER_WG key tiles
// with it, one 32-key block per wavefront as above: both 32-row blocks' S and dP, then their weights,
// then dV^T and dK^T, in program order; the next key tile's K and V rows are requested from memory
// before the current one is computed.  After the first barrier the wavefronts never meet again.
constexpr int kSkinnyTilesPerWg = 4;
template <int D>
__device__ __forceinline__ void bwd_dkv_skinny_body(char *smem, const SegShape &s, const bf16_t *__restrict__ q,
                                                    const bf16_t *__restrict__ k, const bf16_t *__restrict__ v,
                                                    const bf16_t *__restrict__ out, const bf16_t *__restrict__ dO,
                                                    const float *__restrict__ lse, float *__restrict__ dk_part,
                                                    float *__restrict__ dv_part, int bh, int tile_group)
{
    using C = DkvBf16Cfg<D>;
    using Tile = typename C::Tile;
    constexpr int NU = C::NU;
    static_assert(C::BQ == kSkinnyRows, "one Q/dO tile holds the whole segment");

    const int tid = threadIdx.x, lane = tid & 63, lq = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = bh / s.H, h = bh % s.H;
    const int64_t ld = (int64_t)s.H * D;
    const int64_t kv_base = (int64_t)b * s.l_x * ld + (int64_t)h * D;
    const int n_key_tiles = (s.l_x + C::BKV - 1) / C::BKV;
    const int kt0 = tile_group * kSkinnyTilesPerWg, kt1 = min(kt0 + kSkinnyTilesPerWg, n_key_tiles);
    // key tiles from kt_vis on are seen by no query of the segment
    const int kt_vis = s.causal ? (int)min<int64_t>((s.s0 + s.l_s + C::BKV - 1) / C::BKV, n_key_tiles) : n_key_tiles;

    // ---- the segment's Q/dO tile and start values (slot 0), by all four wavefronts
    if (kt0 < kt_vis) {
        uint32_t off[Tile::NI];
        Tile::pair_offsets(off, ld, s.l_s, wave, lane);
        const bf16_t *qbase = q + (int64_t)b * s.l_s * ld + (int64_t)h * D;
        const bf16_t *gbase = dO + (int64_t)b * s.l_s * ld + (int64_t)h * D;
        Tile::issue_pair(Tile::pair_base(qbase), Tile::pair_base(gbase), off, off, smem, wave);
    }
    auto load_kv = [&](int kt, Frag<bf16_t> (&kf)[NU], Frag<bf16_t> (&vf)[NU]) __attribute__((always_inline)) {
        const int jj = kt * C::BKV + wave * C::KW + lq;
        const int64_t off = kv_base + (int64_t)min(jj, s.l_x - 1) * ld + hh * 8;
#pragma unroll
        for (int kb = 0; kb < NU; ++kb) {
            kf[kb] = load_frag<bf16_t>(k + off + kb * 16);
            vf[kb] = load_frag<bf16_t>(v + off + kb * 16);
        }
    };
    Frag<bf16_t> kf[NU], vf[NU], kf_n[NU], vf_n[NU];
    if (kt0 < kt_vis) {
        load_kv(kt0, kf, vf);
        const int64_t first = (int64_t)b * s.l_s * ld + (int64_t)h * D;
        for (int i = s.l_s + tid; i < C::BQ; i += C::NT)            // rows past the segment, whose weights are 0
            reinterpret_cast<float *>(smem + C::OFF_L)[i] = reinterpret_cast<float *>(smem + C::OFF_D)[i] = 0.f;
        neg_row_dots<D>(out + first, dO + first, lse + (int64_t)bh * s.l_s, ld, s.l_s, tid, [&](int i, float nd, float l) {
            reinterpret_cast<float *>(smem + C::OFF_L)[i] = -l * sqrtf((float)D);
            reinterpret_cast<float *>(smem + C::OFF_D)[i] = nd;
        });
    }
    wait_vmem_all();
    __syncthreads();

    int a_off[NU], t_off[D / 32];
#pragma unroll
    for (int kb = 0; kb < NU; ++kb) a_off[kb] = Tile::chunk_offset(lq, 2 * kb + hh);
#pragma unroll
    for (int db = 0; db < D / 32; ++db) t_off[db] = tr_lane_offset_sw<D>(lane, db);
    const float sqrt_d = sqrtf((float)D);
    const float c = kLog2e / sqrt_d, scale = 1.f / sqrt_d;
    const int n_blocks = s.l_s > 32 ? 2 : 1;            // 32-row blocks that hold rows of the segment

    for (int kt = kt0; kt < kt1; ++kt) {
        const int j0 = kt * C::BKV;
        if (kt >= kt_vis) {
            // no query of the segment sees this tile: its partial rows are zero, or stay unwritten
            if (s.skip_tail) return;
            constexpr int F4 = D / 4;
            const f32x4 z = {0.f, 0.f, 0.f, 0.f};
            for (int i = tid; i < C::BKV * F4; i += C::NT) {
                const int row = j0 + i / F4, c4 = (i % F4) * 4;
                if (row < s.l_x) {
                    *reinterpret_cast<f32x4 *>(dk_part + kv_base + (int64_t)row * ld + c4) = z;
                    *reinterpret_cast<f32x4 *>(dv_part + kv_base + (int64_t)row * ld + c4) = z;
                }
            }
            continue;
        }
        const bool more = kt + 1 < kt1 && kt + 1 < kt_vis;
        if (more) load_kv(kt + 1, kf_n, vf_n);          // in flight while this tile is computed

        const int jw0 = j0 + wave * C::KW, j = jw0 + lq;
        f32x16 dk[D / 32], dv[D / 32];
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) { dk[db][e] = 0.f; dv[db][e] = 0.f; }
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            if (qb < n_blocks) {
                const int r0 = 32 * qb;
                // S and dP of the block, accumulators starting at -lse*sqrt(d) and -D of their rows (element
                // e of this lane is row 8*(e/4) + 4*hh + e%4), masked elements at -inf
                f32x16 sc, dp;
#pragma unroll
                for (int e4 = 0; e4 < 4; ++e4) {
                    const f32x4 l4 = *reinterpret_cast<const f32x4 *>(smem + C::OFF_L + (r0 + 8 * e4 + 4 * hh) * 4);
                    const f32x4 d4 = *reinterpret_cast<const f32x4 *>(smem + C::OFF_D + (r0 + 8 * e4 + 4 * hh) * 4);
#pragma unroll
                    for (int i = 0; i < 4; ++i) { sc[4 * e4 + i] = l4[i]; dp[4 * e4 + i] = d4[i]; }
                }
                {
                    const bool diag = s.causal && (jw0 + C::KW - 1 > (int)s.s0 + r0);
                    if (diag || r0 + 32 > s.l_s) {
                        const int first = diag ? max(min(j - (int)s.s0 - r0 - 4 * hh, 64), 0) : 0;
                        const int end = min(s.l_s - r0, 32) - 4 * hh;
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            const int rr = 8 * (e >> 2) + (e & 3);
                            if (rr < first || rr >= end) sc[e] = -INFINITY;
                        }
                    }
                }
#pragma unroll
                for (int kb = 0; kb < NU; ++kb) {
                    const char *p = smem + r0 * (D * 2) + a_off[kb];
                    const Frag<bf16_t> fq = load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(p));
                    const Frag<bf16_t> fg = load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(p + C::OFF_G));
                    sc = mma(fq, kf[kb], sc);
                    dp = mma(fg, vf[kb], dp);
                }
                // weights: P = 2^(c * (S - lse*sqrt(d))), dS = P * (dP - D), rounded to bf16 operands
                Frag<bf16_t> pf[2], df[2];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float pw = fast_exp2(sc[e] * c);
                    pf[e >> 3].v[e & 7] = (bf16_t)pw;
                    df[e >> 3].v[e & 7] = (bf16_t)(pw * dp[e]);
                }
                // dV^T += dO^T P, dK^T += Q^T dS
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const int half = u / (D / 32), db = u % (D / 32);
                    const Frag<bf16_t> fq = load_frag_tr_sw<D>(smem, (qb * 2 + half) * 16, t_off[db]);
                    const Frag<bf16_t> fg = load_frag_tr_sw<D>(smem + C::OFF_G, (qb * 2 + half) * 16, t_off[db]);
                    dv[db] = mma(fg, pf[half], dv[db]);
                    dk[db] = mma(fq, df[half], dk[db]);
                }
            }
        }
        {   // (slots 1 and 2 of the ring are never used here: a staging buffer per wavefront)
            char *buf = smem + C::SLOT + wave * (32 * D * 4);
            const int64_t off = kv_base + (int64_t)jw0 * ld;
            const int rows_ok = min(s.l_x - jw0, C::KW);
            store_key_rows<D>(buf, dk, scale, dk_part + off, ld, rows_ok, lane);
            store_key_rows<D>(buf, dv, 1.f, dv_part + off, ld, rows_ok, lane);
        }
        if (more) {
#pragma unroll
            for (int kb = 0; kb < NU; ++kb) { kf[kb] = kf_n[kb]; vf[kb] = vf_n[kb]; }
        }
    }
}

// ------------------------------------------------------------------------------- dQ, dK and dV in one pass
// Segments of at most 128 rows with many heads and keys: all three gradients from ONE read of K and V.  The traffic is
// all that such a backward is (25,000 visible keys, 32 heads: 205 MB read, 410 MB of partials written, 122 us), and with
// workgroups of their own for dQ and for dK/dV the reads come twice and the dQ workgroups, half of whose wavefronts have no
// rows, take as long as the others (171 us; here 104).  A workgroup owns one (batch*head, split) and walks the split's
// 128-key tiles; each wavefront takes a 32-key block of its own at a time and meets the others only at the start and
// at the end:
//   * Its K block travels global -> LDS (4 KB, double-buffered, private to the wavefront: plain reads for S, transposing
//     ones for dQ), its V block through a slot of its own into registers; both a block ahead.
//   * S and dP (lane = key) give the operands of dV^T and dK^T as in bwd_dkv_body; the same operands
//     exchanged give S^T and dP^T (lane = query), whose weights are the second operand of dQ^T += K^T dS^T as in
//     bwd_dq_body.  Computing the weights twice is cheaper here than turning them round through LDS.
//   * dK and dV are made 32 columns at a time and leave at once through the K slot just used up.
//   * dQ stays in accumulators; the four wavefronts' are added up at the end, in wavefront order.
// QB = 32-row blocks of the segment.  With two the program order is fixed, so that 256 registers and with them two
// workgroups per compute unit suffice; with three or four a wavefront has 512 and the compiler overlaps the blocks
// (100 rows: 163 -> 157 us).
template <int D, int QB_>
struct SkinnyCfg {
    static constexpr int QB = QB_, ROWS = 32 * QB, NT = 256, BKV = 128, NU = D / 16;
    using QTile = DirectTile<D, ROWS>;
    using KTile = DirectTile<D, 32, 1>;
    // Q tile, dO tile, start values as in a ring slot of DkvBf16Cfg; then two K slots and a V slot per wavefront
    static constexpr int OFF_G = QTile::BYTES, OFF_L = 2 * QTile::BYTES, OFF_D = OFF_L + ROWS * 4, OFF_K = (OFF_D + ROWS * 4 + 1023) / 1024 * 1024;
    // (the four wavefronts' slots also hold two wavefronts' dQ at the end)
    static constexpr int SLOTS = 12 * KTile::BYTES, HAND = 2 * QB * (D / 32) * 4096;
    static constexpr int SMEM = OFF_K + (SLOTS > HAND ? SLOTS : HAND);
};

// One accumulator block, 32 keys x 32 columns, through `buf` (4 KB) to rows of `dst`: 128 bytes of 8 keys per instruction
template <int D>
__device__ __forceinline__ void store_key_columns(char *buf, const f32x16 &g, float scale, float *__restrict__ dst, int64_t ld, int rows_ok,
                                                  int lane)
{
    const int lq = lane & 31, hh = lane >> 5;
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4)
        *reinterpret_cast<f32x4 *>(buf + lq * 128 + (((2 * e4 + hh) ^ (lq & 7)) * 16)) =
            f32x4{g[4 * e4] * scale, g[4 * e4 + 1] * scale, g[4 * e4 + 2] * scale, g[4 * e4 + 3] * scale};
    const int c = lane & 7, row = lane >> 3;
    const uint32_t at = ((uint32_t)row * (uint32_t)ld + (uint32_t)c * 4u) * 4u;        // (8 rows of at most 2^23 floats)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f32x4 val = *reinterpret_cast<const f32x4 *>(buf + (i * 8 + row) * 128 + ((c ^ row) * 16));
        if (i * 8 + row < rows_ok) __builtin_nontemporal_store(val, reinterpret_cast<f32x4 *>(reinterpret_cast<char *>(dst + (int64_t)(i * 8) * ld) + at));
    }
}

template <int D, int QB>
__global__ __launch_bounds__(256, QB == 2 ? 2 : 1) void bwd_skinny_bf16_kernel(
    SegShape s, const bf16_t *__restrict__ q, const bf16_t *__restrict__ k, const bf16_t *__restrict__ v,
    const bf16_t *__restrict__ out, const bf16_t *__restrict__ dO, const float *__restrict__ lse, bf16_t *__restrict__ dq,
    float *__restrict__ dq_part, float *__restrict__ dk_part, float *__restrict__ dv_part, int n_splits)
{
    using C = SkinnyCfg<D, QB>;
    using QTile = typename C::QTile;
    using KTile = typename C::KTile;
    constexpr int NU = C::NU, DB = D / 32;
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    int bh, split;
    if (!xcd_item(blockIdx.x, s.B * s.H, n_splits, false, bh, split)) return;
    const int tid = threadIdx.x, lane = tid & 63, lq = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = bh / s.H, h = bh % s.H;
    const int64_t ld = (int64_t)s.H * D;
    const int64_t kv_base = (int64_t)b * s.l_x * ld + (int64_t)h * D, q_base = (int64_t)b * s.l_s * ld + (int64_t)h * D;
    const int n_key_tiles = (s.l_x + C::BKV - 1) / C::BKV;
    // key tiles from kt_vis on are seen by no query of the segment
    const int kt_vis = s.causal ? (int)min<int64_t>((s.s0 + s.l_s + C::BKV - 1) / C::BKV, n_key_tiles) : n_key_tiles;
    const int kt0 = (int)((int64_t)kt_vis * split / n_splits), kt1 = (int)((int64_t)kt_vis * (split + 1) / n_splits);

    char *const k_slots = smem + C::OFF_K + wave * 3 * KTile::BYTES, *const v_slot = k_slots + 2 * KTile::BYTES;
    // (a load instruction's rows start at a multiple of 8, the permutation goes by row % 16: one offset for the even ones, one for the odd)
    static_assert(D == 64, "");
    uint32_t offK[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        offK[i] = ((uint32_t)(lane / 8) * (uint32_t)ld + (uint32_t)((lane % 8) ^ tile_swizzle<D>(8 * i + lane / 8)) * 8u) * 2u;
    // the wavefront's block of key tile kt: rows past the sequence re-read its last row, are masked and never stored
    auto load_kv = [&](int kt, int slot) __attribute__((always_inline)) {
        const int jw0 = kt * C::BKV + wave * 32, j_first = min(jw0, s.l_x - 1);
        const int64_t at = kv_base + (int64_t)j_first * ld;
        char *const dst = k_slots + slot * KTile::BYTES;
        if (jw0 + 32 <= s.l_x) {
#pragma unroll
            for (int i = 0; i < KTile::NI; ++i) {
                lds_dma<16>(k + at + (int64_t)(8 * i) * ld, offK[i & 1], dst + i * 1024);
                lds_dma<16>(v + at + (int64_t)(8 * i) * ld, offK[i & 1], v_slot + i * 1024);
            }
        } else {
            uint32_t off[KTile::NI];
            KTile::offsets(off, ld, s.l_x - j_first, 0, lane);
            lds_dma_n<KTile::NI, 1024>(k + at, off, dst);
            lds_dma_n<KTile::NI, 1024>(v + at, off, v_slot);
        }
    };

    // ---- the segment's rows: Q and dO tile, start values; this lane's row of either block for the transposed products
    {
        uint32_t off[QTile::NI];
        QTile::offsets(off, ld, s.l_s, wave, lane);
#pragma unroll
        for (int i = 0; i < QTile::NI; ++i) {
            lds_dma<16>(q + q_base, off[i], smem + wave * 1024 + i * 4096);
            lds_dma<16>(dO + q_base, off[i], smem + C::OFF_G + wave * 1024 + i * 4096);
        }
    }
    if (kt0 < kt1) load_kv(kt0, 0);
    {
        float *const L = reinterpret_cast<float *>(smem + C::OFF_L), *const Dn = reinterpret_cast<float *>(smem + C::OFF_D);
        for (int i = s.l_s + tid; i < C::ROWS; i += C::NT) { L[i] = -INFINITY; Dn[i] = 0.f; }   // rows past the segment: weights exactly 0
        neg_row_dots<D>(out + q_base, dO + q_base, lse + (int64_t)bh * s.l_s, ld, s.l_s, tid, [&](int i, float nd, float l) {
            L[i] = -l * sqrtf((float)D);
            Dn[i] = nd;
        });
    }
    wait_vmem_all();
    __syncthreads();

    const float sqrt_d = sqrtf((float)D), c = kLog2e / sqrt_d, scale = 1.f / sqrt_d;
    float L2[C::QB], nd[C::QB];
#pragma unroll
    for (int qb = 0; qb < C::QB; ++qb) {
        const int r = 32 * qb + lq;
        L2[qb] = -reinterpret_cast<const float *>(smem + C::OFF_L)[r] * c;
        nd[qb] = reinterpret_cast<const float *>(smem + C::OFF_D)[r];
    }
    int a_off[NU], t_off[DB];
#pragma unroll
    for (int kb = 0; kb < NU; ++kb) a_off[kb] = QTile::chunk_offset(lq, 2 * kb + hh);
#pragma unroll
    for (int db = 0; db < DB; ++db) t_off[db] = tr_lane_offset_sw<D>(lane, db);

    f32x16 acc[C::QB][DB];
#pragma unroll
    for (int qb = 0; qb < C::QB; ++qb)
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[qb][db][e] = 0.f;

    for (int kt = kt0; kt < kt1; ++kt) {
        const int slot = (kt - kt0) & 1;
        char *const kblk = k_slots + slot * KTile::BYTES;
        // The block's loads have landed: of what was issued after them, 16 stores at most are still on their way (every
        // block but a sequence's last stores all its rows).
        if (kt > kt0) wait_vmem<16>();
        const int jw0 = kt * C::BKV + wave * 32, j = jw0 + lq;
        Frag<bf16_t> kf[NU], vf[NU];
#pragma unroll
        for (int kb = 0; kb < NU; ++kb) {
            kf[kb] = load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(kblk + a_off[kb]));
            vf[kb] = load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(v_slot + a_off[kb]));
        }
        if (kt + 1 < kt1) {
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");       // V is in registers: its slot takes the next block's
            load_kv(kt + 1, slot ^ 1);
        }
        Frag<bf16_t> pf[C::QB][2], df[C::QB][2];
#pragma unroll
        for (int qb = 0; qb < C::QB; ++qb) {
            const int r0 = 32 * qb;
            const char *const qt = smem + r0 * (D * 2);
            const bool diag = s.causal && jw0 + 31 > (int)s.s0 + r0;
            if constexpr (QB == 2) __builtin_amdgcn_sched_barrier(0);
            // ---- lane = key: the operands P and dS of dV^T and dK^T
            {
                f32x16 sc, dp;
#pragma unroll
                for (int e4 = 0; e4 < 4; ++e4) {
                    const f32x4 l4 = *reinterpret_cast<const f32x4 *>(smem + C::OFF_L + (r0 + 8 * e4 + 4 * hh) * 4);
                    const f32x4 d4 = *reinterpret_cast<const f32x4 *>(smem + C::OFF_D + (r0 + 8 * e4 + 4 * hh) * 4);
#pragma unroll
                    for (int i = 0; i < 4; ++i) { sc[4 * e4 + i] = l4[i]; dp[4 * e4 + i] = d4[i]; }
                }
                if (diag) {
                    const int first = max(min(j - (int)s.s0 - r0 - 4 * hh, 64), 0);
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (8 * (e >> 2) + (e & 3) < first) sc[e] = -INFINITY;
                }
#pragma unroll
                for (int kb = 0; kb < NU; ++kb) {
                    sc = mma(load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(qt + a_off[kb])), kf[kb], sc);
                    dp = mma(load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(qt + C::OFF_G + a_off[kb])), vf[kb], dp);
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float pw = fast_exp2(sc[e] * c);
                    pf[qb][e >> 3].v[e & 7] = (bf16_t)pw;
                    df[qb][e >> 3].v[e & 7] = (bf16_t)(pw * dp[e]);
                }
            }
            if constexpr (QB == 2) asm volatile("" : : : "memory");     // (the row operands are read again, not kept)
            // ---- lane = query: dQ^T += K^T dS^T
            {
                f32x16 sc, dp;
                float nd_here = nd[qb];
                if constexpr (QB == 2) asm volatile("" : "+v"(nd_here));       // (so that the start values are made here, not kept in 16 registers)
#pragma unroll
                for (int e = 0; e < 16; ++e) { sc[e] = 0.f; dp[e] = nd_here; }
#pragma unroll
                for (int kb = 0; kb < NU; ++kb) {
                    sc = mma(kf[kb], load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(qt + a_off[kb])), sc);
                    dp = mma(vf[kb], load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(qt + C::OFF_G + a_off[kb])), dp);
                }
                if (diag || jw0 + 32 > s.l_x) {
                    const int last = s.causal ? min((int)s.s0 + r0 + lq, s.l_x - 1) : s.l_x - 1;
                    const int rel = max(min(last - jw0 - 4 * hh, 64), -1);
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (8 * (e >> 2) + (e & 3) > rel) sc[e] = -INFINITY;
                }
                Frag<bf16_t> dt[2];
#pragma unroll
                for (int e = 0; e < 16; ++e) dt[e >> 3].v[e & 7] = (bf16_t)(fast_exp2(sc[e] * c - L2[qb]) * dp[e]);
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const int half = u / DB, db = u % DB;
                    acc[qb][db] = mma(load_frag_tr_sw<D>(kblk, half * 16, t_off[db]), dt[half], acc[qb][db]);
                }
            }
        }
        if constexpr (QB == 2) __builtin_amdgcn_sched_barrier(0);
        // ---- dV^T += dO^T P, dK^T += Q^T dS, a column block at a time, each written at once
        const int64_t off = kv_base + (int64_t)jw0 * ld;
        auto finish = [&](const char *tile, const Frag<bf16_t> (&w)[C::QB][2], int db, float f, float *dst) __attribute__((always_inline)) {
            f32x16 g;
#pragma unroll
            for (int e = 0; e < 16; ++e) g[e] = 0.f;
#pragma unroll
            for (int qb = 0; qb < C::QB; ++qb)
#pragma unroll
                    for (int half = 0; half < 2; ++half) g = mma(load_frag_tr_sw<D>(tile, (qb * 2 + half) * 16, t_off[db]), w[qb][half], g);
            store_key_columns<D>(kblk, g, f, dst + off + db * 32, ld, s.l_x - jw0, lane);
            if constexpr (QB == 2) __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            finish(smem, df, db, scale, dk_part);
            finish(smem + C::OFF_G, pf, db, 1.f, dv_part);
        }
    }

    // ---- key tiles that no query sees, dealt out among the splits: zeros, or nothing if the caller asked for that
    if (!s.skip_tail) {
        constexpr int F4 = D / 4;
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        for (int kt = kt_vis + split; kt < n_key_tiles; kt += n_splits)
            for (int i = tid; i < C::BKV * F4; i += C::NT) {
                const int row = kt * C::BKV + i / F4, c4 = (i % F4) * 4;
                if (row < s.l_x) {
                    __builtin_nontemporal_store(z, reinterpret_cast<f32x4 *>(dk_part + kv_base + (int64_t)row * ld + c4));
                    __builtin_nontemporal_store(z, reinterpret_cast<f32x4 *>(dv_part + kv_base + (int64_t)row * ld + c4));
                }
            }
    }

    // ---- dQ: waves 2 and 3 hand theirs to 0 and 1, then 1 to 0 (the K slots are free once everybody is here)
    constexpr int BLOCKS = C::QB * DB;
    auto hand = [&](int region, int blk, int e4) __attribute__((always_inline)) {
        return reinterpret_cast<f32x4 *>(smem + C::OFF_K + ((region * BLOCKS + blk) * 4 + e4) * 1024 + lane * 16);
    };
#pragma unroll
    for (int step = 2; step >= 1; step >>= 1) {
        __syncthreads();
        if (wave >= step && wave < 2 * step) {
#pragma unroll
            for (int blk = 0; blk < BLOCKS; ++blk)
#pragma unroll
                for (int e4 = 0; e4 < 4; ++e4) {
                    const f32x16 &a = acc[blk / DB][blk % DB];
                    *hand(wave - step, blk, e4) = f32x4{a[4 * e4], a[4 * e4 + 1], a[4 * e4 + 2], a[4 * e4 + 3]};
                }
        }
        __syncthreads();
        if (wave < step) {
#pragma unroll
            for (int blk = 0; blk < BLOCKS; ++blk)
#pragma unroll
                for (int e4 = 0; e4 < 4; ++e4) {
                    const f32x4 other = *hand(wave, blk, e4);
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[blk / DB][blk % DB][4 * e4 + i] += other[i];
                }
        }
    }
    if (wave > 0) return;
#pragma unroll
    for (int qb = 0; qb < C::QB; ++qb) {
        const int r = 32 * qb + lq;
        if (r >= s.l_s) continue;
        const int64_t off = ((int64_t)b * s.l_s + r) * ld + (int64_t)h * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                f32x4 val;
#pragma unroll
                for (int i = 0; i < 4; ++i) val[i] = acc[qb][db][4 * e4 + i] * scale;
                const int col = db * 32 + 8 * e4 + 4 * hh;
                if (n_splits == 1) *reinterpret_cast<bf16x4 *>(dq + off + col) = pack4(val[0], val[1], val[2], val[3]);
                else *reinterpret_cast<f32x4 *>(dq_part + (int64_t)split * s.B * s.l_s * ld + off + col) = val;
            }
    }
}

// Splits of the one-pass kernel, 0 where dQ and dK/dV workgroups of their own are the better ones.  Segments of up to 64
// rows run two workgroups per compute unit, longer ones (96 or 128 rows' accumulators) one, and a count that fills the
// chip once is taken, with two tiles per workgroup at least -- three where they share compute units.  Times in us:
//   here   a workgroup takes 3.3, 5.0 or 5.6 per 128-key tile (64, 96, 128 rows) and 9 to 12 besides, and the rows that no
//          query sees are zero-filled at the end (6.2 MB per us);
//   there  9, and the longer of a dQ workgroup's walk (`dq_tiles` of 64 keys) and the dK/dV tiles of all heads, with which
//          the zeros (5 MB per us) overlap in part.
// On 1080 launches (20..128 rows, 1000..50,000 keys, 4..128 heads, an eighth to all of the keys seen, zeros written or not) the
// choice costs 0.9 % over the better one of the two on average; always one pass 17 %, never 11 %.  32 heads of 58 rows against 25,056 keys: 171 -> 104 us, of 100: 209 -> 157.
// Without dropout and for d = 64 only: at d = 128 the slots alone take 96 KB and dQ's accumulators twice the registers, so that
// one workgroup per compute unit is left even at 64 rows; that kernel has not been written.
int skinny_splits(const SegShape &s, bool with_drop, int elem_bytes, int most, int dq_tiles)
{
    if (elem_bytes != 2 || with_drop || s.d != 64 || s.l_s > 128) return 0;
    const int64_t bhs = (int64_t)s.B * s.H, seen = s.causal ? (s.s0 + s.l_s < s.l_x ? s.s0 + s.l_s : (int64_t)s.l_x) : (int64_t)s.l_x;
    const int64_t tiles = (seen + 127) / 128;
    const bool two = s.l_s <= 64;
    int64_t n = std::min<int64_t>(256 / bhs, (tiles + 1) / 2);
    if (two) n = std::max(n, std::min<int64_t>(512 / bhs, tiles / 3));
    n = std::min<int64_t>(n, most);
    if (n < 1) return 0;
    const double walk = (double)((tiles + n - 1) / n), all = (double)(tiles * bhs);
    const double zeros = s.skip_tail ? 0.0 : (double)(s.l_x - seen) * bhs * s.d * 8.0 / 5.0e6;
    const double here = (two ? 9.0 + 3.3 * walk : s.l_s <= 96 ? 10.0 + 5.0 * walk : 12.0 + 5.6 * walk) + 0.8 * zeros;
    const double there = 9.0 + std::max(std::hypot((two ? 0.025 : 0.035) * all, zeros), 0.8 * dq_tiles);
    return here < there ? (int)n : 0;
}

int dq_bf16_rows_per_workgroup(int d) { return d == 64 ? DqBf16Cfg<64>::BR : DqBf16Cfg<128>::BR; }

// ------------------------------------------------------------------------------------------ launch
// Start values of the dK/dV accumulators, per query row: -D = -rowsum(dO * out) and -lse * sqrt(d).
// One 16-byte chunk of a row per thread, D/8 consecutive lanes per row.
// (dropout: -D (1 - p), and the generator's key of the row, for the dK/dV workgroups.)
template <int D, bool DROP>
__global__ __launch_bounds__(256) void bwd_prep_bf16_kernel(SegShape s, DropArgs dr, const bf16_t *__restrict__ out,
                                                            const bf16_t *__restrict__ dO, const float *__restrict__ lse,
                                                            float *__restrict__ Dn, float *__restrict__ Ls,
                                                            uint32_t *__restrict__ row_key)
{
    constexpr int CPR = D / 8;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t rows = (int64_t)s.B * s.l_s * s.H;
    const int64_t row = min(idx / CPR, rows - 1);       // memory order [b][r][h]; whole lane groups stay in range
    const int cpos = (int)(idx % CPR);
    const float nd = neg_row_dot<D>(load_frag<bf16_t>(dO + row * D + cpos * 8), load_frag<bf16_t>(out + row * D + cpos * 8));
    if (cpos == 0 && idx / CPR < rows) {
        const int h = (int)(row % s.H), r = (int)((row / s.H) % s.l_s), b = (int)(row / ((int64_t)s.H * s.l_s));
        const int64_t o_idx = ((int64_t)b * s.H + h) * s.l_s + r;
        Dn[o_idx] = DROP ? nd / dr.scale : nd;
        Ls[o_idx] = -lse[o_idx] * sqrtf((float)D);
        if constexpr (DROP) row_key[o_idx] = drop_row_key(dr.seed_lo, (uint32_t)(b * s.H + h), (uint32_t)(s.s0 + r));
    }
}

// dQ and dK/dV in one launch: the two kinds of workgroup do not depend on each other, so together
// they fill the chip better than one after the other (each alone ends in a tail of part-filled
// compute units, and short segments are mostly tail).  Workgroups [0, n_dq) take the (batch*head,
// query tile, key split) triples of dQ -- with few key splits they are the longest of the launch
// and start first -- and the rest the (batch*head, key tile) pairs of dK/dV.  Both parts are laid
// out in XCD order (xcd_item): an XCD works on one head at a time, whose workgroups share that
// head's K, V, Q and dO in its L2; within a head the longest workgroups come first (last query
// tiles; first key tiles, the zero-fill ones last).
// SKINNY: segments of at most 64 rows that do not take the one-pass kernel, whose dK/dV workgroups take kSkinnyTilesPerWg key tiles each
// (n_key_tiles then counts those groups).
// OWN: no preprocess kernel ran, every workgroup computes what it needs of D itself (bwd_own_values).
// KG = 2: a workgroup is two groups of four wavefronts, with tiles of their own in LDS, that walk half the key tiles (dQ) or query
// tiles (dK/dV) each and add their sums up in LDS, in group order.  As many wavefronts per compute unit as two workgroups
// of one group, each with half the walk: for launches that leave compute units idle or wait for their longest walk (pick_bwd_plan).
// NJ: blocks of 16 keys or query rows per wavefront.  One instead of two: eight wavefronts of 16 rows instead of four of 32, in half
// the registers, so that a SIMD has two of them (at D = 64: two where there is one workgroup per compute unit) and the matrix instructions of
// one run beside the vector work of the other;
// but every operand read from LDS feeds one instruction instead of two.  See bwd_narrow.
template <int D, bool DROP, bool OWN, bool SKINNY = false, int KG = 1, int NJ = 2>
__global__ __launch_bounds__(64 * (8 / NJ) * KG, D == 64 || NJ == 1 ? 2 : 1) void bwd_main_bf16_kernel(
    SegShape s, DropArgs dr, const bf16_t *__restrict__ q, const bf16_t *__restrict__ k, const bf16_t *__restrict__ v,
    const bf16_t *__restrict__ out, const bf16_t *__restrict__ dO, const float *__restrict__ lse,
    const float *__restrict__ Ls, const float *__restrict__ Dn, const uint32_t *__restrict__ row_key, bf16_t *__restrict__ dq,
    float *__restrict__ dq_part, float *__restrict__ dk_part, float *__restrict__ dv_part, int n_splits, int n_dq, int n_q_tiles,
    int n_key_tiles)
{
    using DkvC = DkvBf16Cfg<D, DROP, NJ>;
    constexpr int SMEM_DQ = KG * DqBf16Cfg<D, NJ>::group_lds(DROP);
    constexpr int SMEM_DKV = KG * DkvC::RING * DkvC::SLOT + (OWN && !SKINNY ? DkvC::OWN_BYTES : 0);
    constexpr int SMEM = SMEM_DQ > SMEM_DKV ? SMEM_DQ : SMEM_DKV;
    __shared__ __attribute__((aligned(1024))) char smem[SMEM];
    const int bhs = s.B * s.H;
    const int id = blockIdx.x;
    int bh, inner;
    if (id >= n_dq) {
        if (!xcd_item(id - n_dq, bhs, n_key_tiles, s.causal, bh, inner)) return;
        if constexpr (SKINNY) bwd_dkv_skinny_body<D>(smem, s, q, k, v, out, dO, lse, dk_part, dv_part, bh, inner);
        else bwd_dkv_body<D, DROP, OWN, KG, NJ>(smem, s, dr, q, k, v, out, dO, lse, Ls, Dn, row_key, dk_part, dv_part, bh, inner);
    } else {
        if (!xcd_item(id, bhs, n_q_tiles * n_splits, s.causal && s.s0 < s.l_s, bh, inner)) return;
        bwd_dq_body<D, DROP, OWN, KG, NJ>(smem, s, dr, q, k, v, out, dO, lse, Dn, dq, dq_part, n_splits, inner % n_q_tiles, n_q_tiles, bh,
                                  inner / n_q_tiles);
    }
}

template <int QB>
static hipError_t launch_skinny(const SegShape &s, const bf16_t *q, const bf16_t *k, const bf16_t *v, const bf16_t *out, const float *lse,
                                const bf16_t *dO, bf16_t *dq, float *dk_part, float *dv_part, const Workspace &ws, int n_splits,
                                hipStream_t st)
{
    using C = SkinnyCfg<64, QB>;
    const auto kernel = bwd_skinny_bf16_kernel<64, QB>;
    static DeviceOnce once;
    if (const hipError_t e = allow_lds(kernel, C::SMEM, once); e != hipSuccess) return e;
    TimedLaunch tl(K_BWD_SKINNY_BF16, st);
    hipLaunchKernelGGL(kernel, dim3((unsigned)xcd_grid(s.B * s.H, n_splits)), dim3(256), C::SMEM, st, s, q, k, v, out, dO, lse, dq, ws.dq_part,
                       dk_part, dv_part, n_splits);
    return hipGetLastError();
}

template <int D>
static hipError_t launch_bwd_bf16_d(const SegShape &s, const DropArgs &drop, const bf16_t *q, const bf16_t *k,
                                    const bf16_t *v, const bf16_t *out, const float *lse, const bf16_t *dO, bf16_t *dq,
                                    float *dk_part, float *dv_part, const Workspace &ws, const BwdLaunch &plan, hipStream_t st)
{
    hipError_t e;
    const bool with_drop = drop.thr != 0, own = plan.own, skinny = plan.skinny;
    const int n_splits = plan.splits, groups = plan.groups;
    if constexpr (D == 64) {
        if (plan.one_pass)
            return s.l_s <= 64 ? launch_skinny<2>(s, q, k, v, out, lse, dO, dq, dk_part, dv_part, ws, n_splits, st)
                 : s.l_s <= 96 ? launch_skinny<3>(s, q, k, v, out, lse, dO, dq, dk_part, dv_part, ws, n_splits, st)
                               : launch_skinny<4>(s, q, k, v, out, lse, dO, dq, dk_part, dv_part, ws, n_splits, st);
    }
    if (!own) {
        const int64_t items = (int64_t)s.B * s.l_s * s.H * (D / 8);
        const dim3 grid((unsigned)((items + 255) / 256));
        TimedLaunch tl(K_BWD_PREP_BF16, st);
        const auto kernel = with_drop ? bwd_prep_bf16_kernel<D, true> : bwd_prep_bf16_kernel<D, false>;
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, s, drop, out, dO, lse, ws.D, ws.Ls, ws.row_key);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const int n_q_tiles = (s.l_s + DqBf16Cfg<D>::BR - 1) / DqBf16Cfg<D>::BR;
    int n_key_tiles = (s.l_x + DkvBf16Cfg<D>::BKV - 1) / DkvBf16Cfg<D>::BKV;
    if (skinny) n_key_tiles = (n_key_tiles + kSkinnyTilesPerWg - 1) / kSkinnyTilesPerWg;      // groups of key tiles
    const int n_dq = xcd_grid(s.B * s.H, n_q_tiles * n_splits), n_dkv = xcd_grid(s.B * s.H, n_key_tiles);
    // (own start values for 65 to 512 rows: at d = 128 in narrow launches only -- the others have over 32 walks of 64 rows per compute unit,
    // where bwd_own_values, at 1.5 us per 64 rows and round of workgroups, says no)
    auto kernel = skinny      ? bwd_main_bf16_kernel<D, false, true, true>
                  : with_drop ? (own ? bwd_main_bf16_kernel<D, true, true> : bwd_main_bf16_kernel<D, true, false>)
                              : bwd_main_bf16_kernel<D, false, false>;
    if constexpr (D == 64) {
        if (own && !with_drop && !skinny) kernel = bwd_main_bf16_kernel<D, false, true>;
        if (groups == 2)
            kernel = with_drop ? (own ? bwd_main_bf16_kernel<D, true, true, false, 2> : bwd_main_bf16_kernel<D, true, false, false, 2>)
                               : (own ? bwd_main_bf16_kernel<D, false, true, false, 2> : bwd_main_bf16_kernel<D, false, false, false, 2>);
    }
    unsigned threads = 256 * groups;
    if (plan.narrow) {
        kernel = with_drop ? (own ? bwd_main_bf16_kernel<D, true, true, false, 1, 1> : bwd_main_bf16_kernel<D, true, false, false, 1, 1>)
                           : (own ? bwd_main_bf16_kernel<D, false, true, false, 1, 1> : bwd_main_bf16_kernel<D, false, false, false, 1, 1>);
        threads = 512;
    }
    TimedLaunch tl(K_BWD_MAIN_BF16, st);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(n_dkv + n_dq)), dim3(threads), 0, st, s, drop, q, k, v, out, dO, lse, ws.Ls, ws.D, ws.row_key,
                       dq, ws.dq_part, dk_part, dv_part, n_splits, n_dq, n_q_tiles, n_key_tiles);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return hipSuccess;
}

// accumulator start values (with dropout also the rows' generator keys), then dQ and dK/dV in one
// launch; the caller runs the dQ split merge
hipError_t launch_bwd_bf16_main(const SegShape &s, const DropArgs &drop, const bf16_t *q, const bf16_t *k,
                                const bf16_t *v, const bf16_t *out, const float *lse, const bf16_t *dO, bf16_t *dq,
                                float *dk_part, float *dv_part, const Workspace &ws, const BwdLaunch &plan, hipStream_t st)
{
    if (s.d == 64) return launch_bwd_bf16_d<64>(s, drop, q, k, v, out, lse, dO, dq, dk_part, dv_part, ws, plan, st);
    return launch_bwd_bf16_d<128>(s, drop, q, k, v, out, lse, dO, dq, dk_part, dv_part, ws, plan, st);
}

} // namespace lss
