// Tuned bf16 forward of Eq. 2 (Section 3, Principle 3) for gfx950.
//
// S^T = K Q^T with one query per lane, then O^T += V^T P^T with P^T fed straight from the S^T registers.  The keys are
// walked in blocks of 32 (two per 64-key K/V tile).  Per block g three stages:
//     A(g): S^T product (matrix),  B(g): weights P^T (vector: exp, row sum, bf16 packing),
//     C(g): O^T product (matrix).
// A wavefront issues in order, and vector work costs it several times the issue time of a matrix
// instruction, so the stages are software-pipelined: step g issues the matrix instructions of
// A(g+1) and C(g-1) with the vector work of B(g) spread between them.  K/V tiles travel
// global -> LDS directly (no registers in between), a full loop iteration ahead, into two unpadded, swizzled
// slots each; V is read transposed by DS_READ_B64_TR_B16.
//
// A workgroup is RB wavefronts of 32 query rows, or KG such groups that have a part of the keys each and tiles of their own
// in LDS, and meet there at the end: what fills the chip in launches of few rows without partial results in memory and
// a launch to merge them, and shortens the walk that each wavefront is alone with.  Between backward passes, 8 x 2 heads of 1024
// rows behind 0, 2048 and 4096 others: 128-row workgroups with the best split and its merge 21.1, 29.6 and 38.2 us, 64 rows in two
// groups 14.9, 27.4 and 38.2, 128 rows in two groups 18.4, 28.5 and 35.9; 4 heads of 256 rows behind 512: 11.3, 9.7 and 12.4.  Four groups
// of one or two row blocks (d = 64) go on where that leaves off (figures: pick_fwd_plan).  Large
// launches keep one group (64 heads of 4096 rows: 1692 us, in two groups
// 1829): three workgroups per compute unit hide each other's waits.  The form is chosen per launch (pick_fwd_plan).
//
// Softmax: B subtracts the running maximum m as it stands (no pass over the block first).  Only
// when the block's weights of some row add up to more than 2^8 -- so no weight can be larger
// without this being noticed: a score well above m, or a row seeing its first key -- does a rare,
// wavefront-uniform fix-up raise m to the exact maximum, rescale the row sum and the accumulator,
// and redo the block's weights.  The final division by the row sum, which uses the same m, makes
// the result independent of when m was raised.
#include "lss_bf16.h"
#include <type_traits>
#include "lss_kernels.h"

namespace lss {

template <int D, int RB_, int KG_>
struct FwdBf16Cfg {
    // KG groups of RB wavefronts share the query rows (32 per wavefront of a group) and have a part of the keys each.
    static constexpr int RB = RB_, KG = KG_, WAVES = RB * KG, RW = 32, BR = RB * RW, BC = 64, NT = 64 * WAVES;
    static constexpr int NU = D / 16;                   // operand steps of the S^T product; same for O^T
    using Tile = DirectTile<D, BC, RB>;
    // A group's LDS: two pair slots, slot p a K tile (number p mod 2) and after it a V tile (number p + 1 mod 2): K is
    // loaded one tile further ahead than V and done with one tile earlier, so that two tiles of each are enough.
    static constexpr int OFF_V = Tile::BYTES, PAIR = 2 * Tile::BYTES, RING = 2 * PAIR;
    // (dropout: behind them, the column keys of the last four tiles issued, 64 each)
    static constexpr int group_lds(bool drop) { return RING + (drop ? 4 * BC * 4 : 0); }
    // what the groups hand each other at the end: accumulators in chunks of 16 bytes per lane; maximum and row sum
    static constexpr int UNITS = D / 8, HAND_ML = WAVES * UNITS * 1024, HAND = KG > 1 ? HAND_ML + WAVES * 512 : 0;
    static constexpr int lds(bool drop) { return KG * group_lds(drop) > HAND ? KG * group_lds(drop) : HAND; }
    static constexpr float kMaxBlockSum = 256.0f;       // 2^8: largest sum of a lane's weights of one block without a fix-up
};

// DROP: dropout on the weights (Section 2.2): the weight that multiplies V is dropped or (the finished sum) scaled by
// 1 / (1 - p) according to drop_keep() of (seed, batch*head, global row, key); row sum and lse are
// those of the softmax.
template <int D, bool DROP, int RB, int KG>
__global__ __launch_bounds__(64 * RB * KG, D == 64 ? 2 : 1) void fwd_bf16_kernel(SegShape s, DropArgs dr, const bf16_t *__restrict__ q,
                                                                       const bf16_t *__restrict__ k,
                                                                       const bf16_t *__restrict__ v,
                                                                       bf16_t *__restrict__ out, float *__restrict__ lse,
                                                                       float *__restrict__ o_part,
                                                                       float *__restrict__ lse_part, int n_splits, int n_q_tiles)
{
    using C = FwdBf16Cfg<D, RB, KG>;
    using Tile = typename C::Tile;
    constexpr int NU = C::NU;
    __shared__ __attribute__((aligned(1024))) char smem[C::lds(DROP)];

    const int tid = threadIdx.x, lane = tid & 63, lq = lane & 31, hh = lane >> 5;
    const int all_waves = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = KG > 1 ? all_waves / RB : 0, wave = KG > 1 ? all_waves % RB : all_waves;      // wave: within the group
    char *const ring = smem + group * C::group_lds(DROP);
    // 1-D grid in XCD order (xcd_item): one head at a time per XCD, whose workgroups share its K and
    // V in that XCD's L2.  Within a head: query tiles, last first -- under the causal mask the last
    // tiles see the most keys, and starting the longest workgroups first shortens the tail of the
    // launch -- then key splits.
    const int bhs = s.B * s.H;
    int bh, inner;
    if (!xcd_item(blockIdx.x, bhs, n_q_tiles * n_splits, s.causal && s.s0 < s.l_s, bh, inner)) return;
    const int b = bh / s.H, h = bh % s.H;
    const int q_tile = inner % n_q_tiles, split = inner / n_q_tiles;
    const int r0 = (n_q_tiles - 1 - q_tile) * C::BR;
    const int rw0 = r0 + wave * C::RW;                  // first row of this wavefront
    const int64_t ld = (int64_t)s.H * D;

    const int r_last = min(r0 + C::BR, s.l_s) - 1;
    const int kv_end = s.causal ? (int)min<int64_t>(s.l_x, s.s0 + r_last + 1) : s.l_x;
    const int n_tiles = (kv_end + C::BC - 1) / C::BC;
    const int per = (n_tiles + n_splits - 1) / n_splits;
    const int s_begin = split * per, s_tiles = max(min(n_tiles, s_begin + per) - s_begin, 0);
    // this group's tiles; the first group has `iters` of them, the last ones fewer or none
    const int iters = KG > 1 ? (s_tiles + KG - 1) / KG : s_tiles;
    const int t_begin = s_begin + group * iters, T = KG > 1 ? max(min(s_tiles - group * iters, iters), 0) : s_tiles;

    // this lane's query row (column of the S^T tile); rows past the segment re-read its last row
    // (unconditional loads), are computed like any other and never stored
    const int r = rw0 + lq;
    const bool row_ok = r < s.l_s;
    Frag<bf16_t> qf[NU];
    {
        const bf16_t *qp = q + ((int64_t)b * s.l_s + min(r, s.l_s - 1)) * ld + (int64_t)h * D + hh * 8;
#pragma unroll
        for (int kb = 0; kb < NU; ++kb) qf[kb] = load_frag<bf16_t>(qp + kb * 16);
    }
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 o[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db) o[db] = zero16;
    float m = -INFINITY, l = 0.f;                       // running maximum (log2 domain); this lane's half of the row sum
    float m_sub = -1e30f;                               // what B subtracts: m, or as long as the row has seen no key a huge negative number
    const float c = kLog2e / sqrtf((float)D);

    if (s_tiles > 0) {
        const bf16_t *kbase = k + (int64_t)b * s.l_x * ld + (int64_t)h * D;
        const bf16_t *vbase = v + (int64_t)b * s.l_x * ld + (int64_t)h * D;

        // dropout: this lane's row key; the column seed; the column keys of tile t (global tile index)
        // are computed once, by one wavefront when the tile's loads are issued, into quarter t % 4 of
        // a small ring behind the tiles -- published by the same barrier as the tile
        uint32_t drop_rk = 0u, drop_cs = 0u;
        if (DROP) { drop_rk = drop_row_key(dr.seed_lo, (uint32_t)bh, (uint32_t)(s.s0 + r)); drop_cs = drop_col_seed(dr.seed_hi); }
        char *const ck_ring = ring + C::RING;

        // ---- tile loads, by all wavefronts of the group.  No branch and few scalar instructions on purpose: a branch inside a
        // pipeline step splits it into basic blocks, and the vector work that was meant to sit between the step's matrix
        // instructions is then moved behind the branch in one lump; addresses move on between the iterations instead.
        uint32_t offK[Tile::NI], offV[Tile::NI], offD[Tile::NI];    // this lane's global offsets within the next K and V tile; and
        Tile::pair_offsets(offK, ld, C::BC, wave, lane);            // what must be added to them in the sequence's last, partial
        const int t_part = s.l_x % C::BC ? s.l_x / C::BC : -1;     // tile (rows past the end re-read the last row)
        {
            uint32_t offL[Tile::NI];
            Tile::pair_offsets(offL, ld, t_part >= 0 ? s.l_x % C::BC : C::BC, wave, lane);
#pragma unroll
            for (int i = 0; i < Tile::NI; ++i) { offD[i] = offL[i] - offK[i]; offV[i] = offK[i]; }
        }
        const uint32_t tile_bytes = (uint32_t)(C::BC * ld * 2);
        // the next tile of K to load, and of V, one behind; past the group's last one that one again
        const int t_last = t_begin + max(T, 1) - 1;
        int k_tile_next = t_begin, v_tile_next = t_begin;
        const char *k_next = tile_ptr(Tile::pair_base(kbase), t_begin, tile_bytes), *v_next = tile_ptr(Tile::pair_base(vbase), t_begin, tile_bytes);
        auto to_part = [&](int t, uint32_t (&off)[Tile::NI]) __attribute__((always_inline)) {
            if (t == t_part)
#pragma unroll
                for (int i = 0; i < Tile::NI; ++i) off[i] += offD[i];
        };
        to_part(k_tile_next, offK);
        to_part(v_tile_next, offV);
        auto advance_k = [&] {
            if (k_tile_next < t_last) { ++k_tile_next; k_next += tile_bytes; to_part(k_tile_next, offK); }
        };
        auto advance_v = [&] {
            if (v_tile_next < t_last) { ++v_tile_next; v_next += tile_bytes; to_part(v_tile_next, offV); }
        };
        // Iteration t's loads, behind its barrier: K of tile t + 2 in the place of tile t's, whose last rows have been read
        // by then, and V of tile t + 1 in the place of tile t - 1's.  (Past the end a tile is loaded once more: K where it
        // lies already or where nobody reads any more, V where nobody reads any more.)
        auto issue_next = [&](char *pair_slot) __attribute__((always_inline)) {
            static_assert(C::OFF_V == Tile::BYTES, "V tile follows K tile");
            Tile::issue_pair(k_next, v_next, offK, offV, pair_slot, wave);
            if (DROP && wave == 0)
                reinterpret_cast<uint32_t *>(ck_ring)[(k_tile_next & 3) * C::BC + lane] = drop_col_key(drop_cs, (uint32_t)(k_tile_next * C::BC + lane));
        };

        // ---- this lane's LDS addresses (bytes from smem) in the K tile that A and in the V tile that C reads next; they move to
        // the next tile once per iteration, to the other pair slot and back
        const int ring_at = group * C::group_lds(DROP);
        int a_at[NU];                                   // A-operand chunk of row lq for operand step kb
#pragma unroll
        for (int kb = 0; kb < NU; ++kb) a_at[kb] = ring_at + Tile::chunk_offset(lq, 2 * kb + hh);
        int t_at[D / 32][2];                            // transposed reads, column block db: either read's
#pragma unroll
        for (int db = 0; db < D / 32; ++db) {
            const int off = tr_lane_offset_sw<D>(lane, db);
            t_at[db][0] = ring_at + C::OFF_V + off;
            t_at[db][1] = ring_at + C::OFF_V + (off ^ 48);
        }

        // ---- stage pieces.  `kb2`: which half of the tile, a block of 32 keys.
        auto load_a = [&](int kb2, int kb, Frag<bf16_t> &fk) __attribute__((always_inline)) {
            fk = load_frag<bf16_t>(reinterpret_cast<const bf16_t *>(smem + a_at[kb] + kb2 * 32 * (D * 2)));
        };
        auto load_c = [&](int kb2, int u, Frag<bf16_t> &fv) __attribute__((always_inline)) {
            const int half = u / (D / 32), db = u % (D / 32);
            fv = load_frag_tr_sw<D>(smem, (kb2 * 2 + half) * 16, t_at[db][0], t_at[db][1]);
        };
        // Where the causal diagonal or the end of the sequence crosses a block (first key jb), the
        // masked elements of its finished S^T accumulator are set to -inf, which B turns into weight
        // 0: keys after the lane's row, and keys past the sequence (whose loads re-read its last
        // row).  C-tile element e of this lane is key 8*(e/4) + 4*hh + e%4 of the block.
        // (positions are below 2^30, checked on the host: one 32-bit scalar compare, no vector work per step)
        const int last_whole = min(s.causal ? (int)s.s0 + rw0 - 31 : s.l_x, s.l_x - 32);       // blocks from here on need no mask
        auto mask_s = [&](int jb, f32x16 &sc) __attribute__((always_inline)) {
            if (jb > last_whole) {
                const int last = s.causal ? min((int)s.s0 + r, s.l_x - 1) : s.l_x - 1;
                const int rel = max(min(last - jb - 4 * hh, 64), -1);
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (8 * (e >> 2) + (e & 3) > rel) sc[e] = -INFINITY;
            }
        };
        // B for the pairs [n0, n1) of elements 2 n, 2 n + 1: weight = 2^(c * S - m); the pair is added to the row sum
        // and rounded to bf16 into the operand fragment of C.  What a pair's instructions wait for was made with the pair before:
        // its exponents come a pair ahead of its exponentials, sum and rounding a pair behind.
        // A row that has seen no key yet (m = -inf) subtracts a huge negative number instead (m_sub), so that
        // any real score gives weight +inf and forces the fix-up, while masked scores still give 0.
        // Dropout: a decision is a chain of eight instructions, which goes over three pairs' slots: first round a pair ahead of the exponential,
        // second beside it, the rest a pair behind.  (All in one slot, with two conversions and a permutation per pair and the keys read when they
        // were due: 16 heads x 2 of 4096 rows behind 16384, 1212 us; 1134 so.)
        u32x4 ck4;      // the column keys of four consecutive elements: element e of this lane is key jb + 8 (e / 4) + 4 hh + e % 4
        uint32_t r1_0, r1_1, r2_0, r2_1;
        float x0, x1, p0, p1;
        auto load_keys = [&](int jb, int e) __attribute__((always_inline)) {
            if (DROP) ck4 = *reinterpret_cast<const u32x4 *>(ck_ring + (((jb >> 6) & 3) * C::BC + (jb & 63) + 8 * (e >> 2) + 4 * hh) * 4);
        };
        auto round1 = [&](int e) __attribute__((always_inline)) {
            r1_0 = drop_round1(drop_rk, ck4[e & 3]);
            r1_1 = drop_round1(drop_rk, ck4[(e & 3) + 1]);
        };
        auto b_pairs = [&](const f32x16 &sc, int jb, int n0, int n1, float &psum, Frag<bf16_t> (&pf)[2])
            __attribute__((always_inline)) {
            auto finish = [&](int e) __attribute__((always_inline)) {       // p0, p1: the weights of elements e, e + 1
                psum += p0;
                psum += p1;
                if (DROP) {
                    p0 = drop_decide(r2_0, dr.thr) ? p0 : 0.f;
                    p1 = drop_decide(r2_1, dr.thr) ? p1 : 0.f;
                    asm("" : "+v"(p0), "+v"(p1));       // (or each is rounded by itself ahead of the choice: five instructions for three)
                }
                pf[e >> 3].v[e & 7] = (bf16_t)p0; pf[e >> 3].v[(e & 7) + 1] = (bf16_t)p1;
            };
#pragma unroll
            for (int n = n0; n < n1; ++n) {
                if (n == 0) {
                    x0 = sc[0] * c - m_sub; x1 = sc[1] * c - m_sub;
                    if (DROP) round1(0);
                }
                const float e0 = fast_exp2(x0), e1 = fast_exp2(x1);
                if (n < 7) { x0 = sc[2 * n + 2] * c - m_sub; x1 = sc[2 * n + 3] * c - m_sub; }
                if (n > 0) finish(2 * n - 2);
                if (DROP) {
                    r2_0 = drop_round2(r1_0);
                    r2_1 = drop_round2(r1_1);
                    if (n < 7) round1(2 * n + 2);
                    if (n % 2 == 0 && n < 6) load_keys(jb, 2 * n + 4);     // (the four before are done with)
                }
                p0 = e0, p1 = e1;
                if (n == 7) finish(14);
            }
        };
        // The fix-up: raise m to the exact maximum over what the row has seen including this block,
        // rescale what was accumulated under the old m (row sum l0 before this block; accumulator,
        // to which this block has not been added yet) and redo the block's weights.
        auto fixup = [&](const f32x16 &sc, int jb, float l0, Frag<bf16_t> (&pf)[2]) __attribute__((always_inline)) {
            float mx = -INFINITY;
#pragma unroll
            for (int e = 0; e < 16; ++e) mx = fmaxf(mx, sc[e]);
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m, mx * c);
            const float alpha = (m == -INFINITY) ? 0.f : fast_exp2(m - m_new);
            m = m_new;
            m_sub = m == -INFINITY ? -1e30f : m;
            l = l0 * alpha;
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) o[db][e] *= alpha;
            load_keys(jb, 0);
            b_pairs(sc, jb, 0, 8, l, pf);
        };

        // One pipeline step.  A: half kb2_a of its tile into sc_a.  B: sc_b, first key jb_b, packing
        // into pf_b.  C: half kb2_c of its tile from pf_c into o.  Per unit the matrix instructions
        // go C, A (A, C in the last unit); after each one come the B elements that fall to its slot.  Operand fragments are
        // read from LDS one unit ahead of their use; those of the first unit by the step before
        // (ak[0], cv[0] on entry), and this step leaves there those of the next step: halves kb2_an and kb2_cn.  `mid` runs
        // before those last reads: the even steps put the loop's barrier there, because the next step's blocks may lie in the
        // tile that the barrier publishes, and move the addresses on.
        Frag<bf16_t> ak[2], cv[2];
        auto step = [&](auto has_a, auto has_b, auto has_c, int kb2_a, f32x16 &sc_a, f32x16 &sc_b,
                        int jb_b, Frag<bf16_t> (&pf_b)[2], int kb2_c, Frag<bf16_t> (&pf_c)[2], int kb2_an, int kb2_cn, auto &&mid)
            __attribute__((always_inline)) {
            constexpr bool HA = decltype(has_a)::value, HB = decltype(has_b)::value, HC = decltype(has_c)::value;
            constexpr int NS = 2 * NU;                  // slots; the 8 element pairs of B spread over them
            static_assert(NU % 2 == 0, "fragment double buffers assume an even number of units");
            const float l0 = l;
            auto b_slot = [&](int slot) __attribute__((always_inline)) {
                if (HB) {
                    __builtin_amdgcn_sched_barrier(0);
                    b_pairs(sc_b, jb_b, slot * 8 / NS, (slot + 1) * 8 / NS, l, pf_b);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            if (HB) {
                load_keys(jb_b, 0);
                mask_s(jb_b, sc_b);
                // B's inputs pass through an empty asm here: its arithmetic depends on nothing else in
                // this step, and the compiler would otherwise move all of it out of the step, in one lump
                asm volatile("" : "+v"(sc_b));
            }
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int half = u / (D / 32), db = u % (D / 32);
                if (u + 1 < NU) {
                    if (HC) load_c(kb2_c, u + 1, cv[(u + 1) & 1]);
                    if (HA) load_a(kb2_a, u + 1, ak[(u + 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    wait_lds<(HC ? 2 : 0) + (HA ? 1 : 0)>();        // this unit's are there
                    __builtin_amdgcn_sched_barrier(0);
                    if (HC) o[db] = mma(cv[u & 1], pf_c[half], o[db]);
                    b_slot(2 * u);
                    if (HA) sc_a = mma(ak[u & 1], qf[u], u == 0 ? zero16 : sc_a);
                    b_slot(2 * u + 1);
                } else {
                    // last unit: A first, so that its result is there when the next step's B wants it
                    if (HA) sc_a = mma(ak[u & 1], qf[u], sc_a);
                    b_slot(2 * u);
                    mid();
                    load_c(kb2_cn, 0, cv[0]);
                    load_a(kb2_an, 0, ak[0]);
                    __builtin_amdgcn_sched_barrier(0);
                    if (HC) o[db] = mma(cv[u & 1], pf_c[half], o[db]);
                    b_slot(2 * u + 1);
                }
            }
            if (HB) {
                // ... and its results through another one, so that it is not sunk below the step either
                asm volatile("" : "+v"(pf_b[0].v), "+v"(pf_b[1].v), "+v"(l));
                if (__any(!(l - l0 <= C::kMaxBlockSum))) fixup(sc_b, jb_b, l0, pf_b);
            }
        };
        using std::true_type;
        using std::false_type;

        // ---- pipeline.  Block g = keys (t_begin + g/2) * 64 + (g%2) * 32 ..; tile t = blocks 2t, 2t+1.
        if (T > 0) {
            issue_next(ring);                           // (K of tile 0; its V here is overwritten before anybody reads it)
            advance_k();
            issue_next(ring + C::PAIR);
            advance_k();
            advance_v();
        }
        wait_vmem_all();
        __syncthreads();

        if (rw0 >= s.l_s) {
            // None of this wavefront's rows exists (a partly filled last query tile): it only keeps moving
            // tiles and meeting the loop's barriers.
            for (int t = 0; t < T; ++t) {
                wait_vmem_all();
                __syncthreads();
                issue_next(ring + (t & 1) * C::PAIR);
                advance_k();
                advance_v();
            }
        } else if (T > 0) {
            f32x16 sc0, sc1;                            // even / odd blocks
            Frag<bf16_t> pf0[2], pf1[2];
            // step -1: A(0) alone.  The first loop step has no C(-1): it multiplies zeros with tile 0 instead.
            load_a(0, 0, ak[0]);
            auto nothing = [] {};
            step(true_type{}, false_type{}, false_type{}, 0, sc0, sc1, 0, pf0, 0, pf1, 1, 1, nothing);
#pragma unroll
            for (int half = 0; half < 2; ++half)
#pragma unroll
                for (int e = 0; e < 8; ++e) pf1[half].v[e] = (bf16_t)0.f;

            // the pair slot (bytes) of K of tile t and V of tile t - 1, and the way to that of K of t + 1 and V of t
            int slot = 0, other = C::PAIR;
            int j0 = t_begin * C::BC;
            for (int t = 0; t < T; ++t) {
                // even step g = 2t: A(2t+1) [tile t, second half], B(2t), C(2t-1) [tile t-1, second half;
                // for t = 0 V of tile 0, which lies in both slots, times zero]
                // Before its last reads (which may touch tile t+1): K of tile t+1 and V of tile t, issued one iteration
                // ago, have landed for this wavefront; after the barrier for all, and every wavefront has
                // requested its last operands from K of tile t and V of tile t-1.
                step(true_type{}, true_type{}, true_type{}, 1, sc1, sc0, j0, pf0, 1, pf1, 0, 0, [&] {
                    wait_vmem_all();
                    __syncthreads();
                    issue_next(ring + slot);
#pragma unroll
                    for (int kb = 0; kb < NU; ++kb) a_at[kb] += other;
#pragma unroll
                    for (int db = 0; db < D / 32; ++db) { t_at[db][0] += other; t_at[db][1] += other; }
                });
                // odd step g = 2t+1: A(2t+2) [tile t+1, first half; past the end of whatever its slot holds, result unused],
                // B(2t+1), C(2t) [tile t, first half]
                step(true_type{}, true_type{}, true_type{}, 0, sc0, sc1, j0 + 32, pf1, 0, pf0, 1, 1, nothing);
                advance_k();
                advance_v();
                slot += other, other = -other;
                j0 += C::BC;
            }
            // step 2T: C(2T-1) [tile T-1, second half] alone
            step(false_type{}, false_type{}, true_type{}, 0, sc0, sc0, 0, pf0, 1, pf1, 0, 1, nothing);
        }
        if (KG > 1)
            for (int t = T; t < iters; ++t) __syncthreads();           // the barriers of the groups that have more tiles
        wait_vmem_all();                                // the last, redundant prefetches must land before the workgroup's LDS is given away
    }

    // this lane's row of the result: column group u, columns 8 u + 4 hh .. + 3 (a split's normalised output travels to the
    // merge kernel in fp32: rounded to bf16 once, there)
    const int64_t part_row = ((int64_t)split * bhs + bh) * s.l_s + r;
    auto put = [&](int u, const f32x4 &val) __attribute__((always_inline)) {
        if (n_splits == 1)
            *reinterpret_cast<bf16x4 *>(out + ((int64_t)b * s.l_s + r) * ld + (int64_t)h * D + 8 * u + 4 * hh) = pack4(val[0], val[1], val[2], val[3]);
        else *reinterpret_cast<f32x4 *>(o_part + part_row * D + 8 * u + 4 * hh) = val;
    };
    auto put_lse = [&](float v) {
        if (n_splits == 1) lse[(int64_t)bh * s.l_s + r] = v;
        else lse_part[part_row] = v;
    };
    const float l_own = l + __shfl_xor(l, 32);
    const float kept = DROP ? dr.scale : 1.f;           // of the kept weights: applied to their sum
    if constexpr (KG == 1) {
        const float inv = l_own > 0.f ? kept / l_own : 0.f;
        if (!row_ok) return;
        if (hh == 0) put_lse(l_own > 0.f ? (m + log2f(l_own)) * kLn2 : -INFINITY);
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4)
                put(db * 4 + e4, f32x4{o[db][4 * e4] * inv, o[db][4 * e4 + 1] * inv, o[db][4 * e4 + 2] * inv, o[db][4 * e4 + 3] * inv});
    } else {
        // The groups' results meet in LDS, where the tiles were: group g adds up its share of the columns, in group order,
        // weighted to the rows' maximum over all groups.
        auto hand = [&](int g, int u) { return reinterpret_cast<f32x4 *>(smem + ((g * RB + wave) * C::UNITS + u) * 1024 + lane * 16); };
        auto hand_ml = [&](int g) { return reinterpret_cast<float *>(smem + C::HAND_ML + (g * RB + wave) * 512 + lane * 8); };
        __syncthreads();
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4)
                *hand(group, db * 4 + e4) = f32x4{o[db][4 * e4], o[db][4 * e4 + 1], o[db][4 * e4 + 2], o[db][4 * e4 + 3]};
        hand_ml(group)[0] = m;
        hand_ml(group)[1] = l_own;
        __syncthreads();
        if (!row_ok) return;
        float mg[KG], m_all = -INFINITY, l_all = 0.f;
#pragma unroll
        for (int g = 0; g < KG; ++g) { mg[g] = hand_ml(g)[0]; m_all = fmaxf(m_all, mg[g]); }
#pragma unroll
        for (int g = 0; g < KG; ++g) {
            mg[g] = mg[g] == -INFINITY ? 0.f : fast_exp2(mg[g] - m_all);       // from here on: its weight
            l_all += mg[g] * hand_ml(g)[1];
        }
        const float inv = l_all > 0.f ? kept / l_all : 0.f;
        if (group == 0 && hh == 0) put_lse(l_all > 0.f ? (m_all + log2f(l_all)) * kLn2 : -INFINITY);
        constexpr int PER = C::UNITS / KG;
        static_assert(C::UNITS % KG == 0, "");
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int u = group * PER + i;
            f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int g = 0; g < KG; ++g) {
                const f32x4 v = *hand(g, u);
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] += mg[g] * v[e];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] *= inv;
            put(u, sum);
        }
    }
}

int fwd_bf16_rows_per_workgroup(int d) { return d == 64 ? 128 : 256; }

template <int D, int RB, int KG>
static hipError_t launch_fwd_main(const SegShape &s, const DropArgs &drop, const bf16_t *q, const bf16_t *k,
                                  const bf16_t *v, bf16_t *out, float *lse, const Workspace &ws, int n_splits, hipStream_t st)
{
    using C = FwdBf16Cfg<D, RB, KG>;
    const int n_q_tiles = (s.l_s + C::BR - 1) / C::BR;
    dim3 grid((unsigned)xcd_grid(s.B * s.H, n_q_tiles * n_splits));
    auto kernel = fwd_bf16_kernel<D, false, RB, KG>;
    if (drop.thr != 0) {
        if constexpr (D == 64 && RB == 4 && KG == 2) return hipErrorInvalidConfiguration;      // (pick_fwd_plan: never with dropout)
        else kernel = fwd_bf16_kernel<D, true, RB, KG>;
    }
    TimedLaunch tl(K_FWD_BF16, st);
    hipLaunchKernelGGL(kernel, grid, dim3(C::NT), 0, st, s, drop, q, k, v, out, lse, ws.o_part, ws.lse_part, n_splits, n_q_tiles);
    return hipGetLastError();
}

hipError_t launch_fwd_bf16_main(const SegShape &s, const DropArgs &drop, const bf16_t *q, const bf16_t *k,
                                const bf16_t *v, bf16_t *out, float *lse, const Workspace &ws, const FwdPlan &plan, hipStream_t st)
{
    if (s.d == 64) {
        switch (plan.form) {
        case FWD_2x2: return launch_fwd_main<64, 2, 2>(s, drop, q, k, v, out, lse, ws, plan.splits, st);
        case FWD_4x2: return launch_fwd_main<64, 4, 2>(s, drop, q, k, v, out, lse, ws, plan.splits, st);
        case FWD_2x4: return launch_fwd_main<64, 2, 4>(s, drop, q, k, v, out, lse, ws, plan.splits, st);
        case FWD_1x4: return launch_fwd_main<64, 1, 4>(s, drop, q, k, v, out, lse, ws, plan.splits, st);
        default: return launch_fwd_main<64, 4, 1>(s, drop, q, k, v, out, lse, ws, plan.splits, st);
        }
    }
    if (plan.form == FWD_4x2) return launch_fwd_main<128, 4, 2>(s, drop, q, k, v, out, lse, ws, plan.splits, st);
    return launch_fwd_main<128, 8, 1>(s, drop, q, k, v, out, lse, ws, plan.splits, st);
}

} // namespace lss
