// Backward of Eq. 2 (Section 3, Principle 3) for one segment.  With P the softmax weights
// recomputed from lse, dP = dO V^T and D[r] = dO[r] . out[r] (= sum_j P dP):
//     dS = P * (dP - D);   dQ = dS K / sqrt(d);   dK_part = dS^T Q / sqrt(d);   dV_part = P^T dO.
// With dropout on the weights (template flag DROP; mask M = keep / (1 - p), out = (P * M) V): dP is
// replaced by M * dP and dV_part = (P * M)^T dO; D = dO . out still equals sum_j P (M dP).
// dK_part/dV_part hold this segment's contribution only; their sum over segments is the
// arithmetic of the reduce-scatter of Fig. 2(v).
//
// The dQ workgroups (query-tile owned, split over key ranges) and the dK/dV workgroups (key-tile owned) share one
// launch (lss_bwd_bf16.hip, lss_f32.hip); here are the fp32 path's D = rowsum(dO * out), the merge of the
// dQ splits, and the launch sequence.  No atomics.
#include "lss_bwd_plan.h"
#include "lss_common.h"
#include "lss_kernels.h"
#include <algorithm>

namespace lss {

// ---------------------------------------------------------------- D = rowsum(dO * out)
template <typename T, int D>
__global__ __launch_bounds__(256) void bwd_rowdot_kernel(SegShape s, const T *__restrict__ out,
                                                         const T *__restrict__ dO, float *__restrict__ Dv)
{
    // 16 lanes per (b, r, h) row, each D/16 consecutive elements
    constexpr int PER = D / 16;
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t row = gid >> 4;          // (b * l_s + r) * H + h
    const int sub = (int)(gid & 15);
    const int64_t rows = (int64_t)s.B * s.l_s * s.H;
    float acc = 0.f;
    if (row < rows) {
        const T *o = out + row * D + sub * PER, *g = dO + row * D + sub * PER;
#pragma unroll
        for (int i = 0; i < PER; ++i) acc += (float)o[i] * (float)g[i];
    }
    acc += __shfl_xor(acc, 8);
    acc += __shfl_xor(acc, 4);
    acc += __shfl_xor(acc, 2);
    acc += __shfl_xor(acc, 1);
    if (row < rows && sub == 0) {
        const int64_t h = row % s.H, br = row / s.H, r = br % s.l_s, b = br / s.l_s;
        Dv[(b * s.H + h) * s.l_s + r] = acc;
    }
}

// dq = sum over splits, in split order.  MAXS: compile-time bound of n_splits, so that a thread's loads are in flight together
// (58 rows, 32 heads, 16 splits: 6.5 us in a loop over the splits, now 5.4; two splits: 4.9 either way).
template <typename T, int MAXS>
__global__ __launch_bounds__(256) void bwd_dq_merge_kernel(const float *__restrict__ dq_part, int n_splits,
                                                           int64_t n4, T *__restrict__ dq)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n4) return;
    f32x4 part[MAXS];
#pragma unroll
    for (int sp = 0; sp < MAXS; ++sp)
        part[sp] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(dq_part + ((sp < n_splits ? sp : n_splits - 1) * n4 + i) * 4));
    f32x4 acc = part[0];
#pragma unroll
    for (int sp = 1; sp < MAXS; ++sp)
        if (sp < n_splits) acc += part[sp];
    if constexpr (sizeof(T) == 2) *reinterpret_cast<bf16x4 *>(dq + i * 4) = bf16x4{(bf16_t)acc[0], (bf16_t)acc[1], (bf16_t)acc[2], (bf16_t)acc[3]};
    else *reinterpret_cast<f32x4 *>(dq + i * 4) = acc;
}

// (bf16 with at most 64 rows, and at d = 128 the base of pick_splits; see pick_bwd_plan in lss_bwd_plan.h for d = 64)
// The dQ workgroups share their launch with the dK/dV ones and need not fill the chip alone: keys are split so far that
// a dQ workgroup does not outlast the rest of the launch, never further than the workspace was sized for.  In 64-key
// tiles of dQ, of which a lone workgroup takes one per 1.0 us (d = 64) or 1.4 us (d = 128):
//   * A launch that leaves compute units idle splits until it fills them (l_x = 1024 in segments of 256, last one:
//     21.0 us with one range, 15.3 with three), in ranges of at least four tiles that take no less than a dK/dV
//     workgroup's walk over the queries, 1.35 per 64 of them.  Workgroups that only zero-fill count a quarter.
//   * Otherwise a range may be half as long again as the launch would take at full balance (the dK/dV and dQ tiles a
//     compute unit works off per us, and the zero-filled rows), but 24 to 64 tiles: 130 rows against 13,000 keys
//     take 54 us in ranges of 51 tiles and 38 in ranges of 26; in longer launches shorter ranges gain nothing.
//     Where one workgroup fills a compute unit (d = 128), a launch that fits the chip keeps fitting it.
static int pick_dq_splits(const SegShape &s, int most)
{
    const int rows_per_wg = dq_rows_per_wg(2, s.d);
    if (most <= 1) return 1;
    const int64_t bhs = (int64_t)s.B * s.H, seen = s.causal ? (s.s0 + s.l_s < s.l_x ? s.s0 + s.l_s : (int64_t)s.l_x) : (int64_t)s.l_x;
    const int64_t tiles = (seen + 63) / 64;                                     // key tiles of a query tile
    const int64_t dq_wgs = bhs * ((s.l_s + rows_per_wg - 1) / rows_per_wg), dkv_wgs = bhs * ((seen + 127) / 128);
    int64_t want = 1;
    struct Rate { double tile_us, dkv, dq; };
    const Rate rate = s.d == 64 ? Rate{1.0, 0.74, 1.25} : Rate{1.4, 0.5, 0.7};
    const double q_tiles = (double)((s.l_s + 63) / 64), walk = s.l_s <= 64 ? 8.0 : 1.35 * q_tiles;
    const double us = ((double)dkv_wgs * q_tiles / rate.dkv + (double)dq_wgs * tiles / rate.dq) / 256.0 +
                      (double)(s.l_x - seen) * bhs * s.d * 8.0 / 5.5e6;
    double longest = 1.5 * us / rate.tile_us;
    if (longest < 24.0) longest = 24.0;
    if (longest < walk) longest = walk;
    if (longest > 64.0) longest = 64.0;
    want = (int64_t)ceil((double)tiles / longest);
    const int64_t idle = (256 - dkv_wgs - (s.l_x - seen) * bhs / 512) / dq_wgs, fill = (int64_t)((double)tiles / (walk > 4.0 ? walk : 4.0));
    if (idle >= want) want = fill <= want ? want : idle < fill ? idle : fill;
    else if (s.d == 128 && idle >= 1) want = idle;
    return (int)(want < 1 ? 1 : want > most ? most : want);
}

// float, and bf16 at d = 128 with more than 64 rows: a launch takes about, in us,
//     start + (longest^6 + balance^6)^(1/6) + zeros + merge
// as in pick_bwd_plan: the longer of a dQ workgroup's walk over its 64-key tiles and a dK/dV workgroup's over the 64-row query tiles
// (half the time where two wavefronts share a key block), slower as two workgroups share a compute unit; all walks over 256 compute units,
// and a part of a last dK/dV walk where the launch takes more than one round.
// float: fitted to 290 launches (30 .. 12,661 rows, 512 .. 22,136 keys, 2 .. 32 heads, 1 .. 16 splits, after a forward call each).
// Ranges of 16 tiles, what every launch had, are the base, left where the estimate of shorter ones is 5 % better or of longer ones 15 %: launches
// took 12 % more with them on average (4 heads of 100 rows against 1000 keys 66 us, in four ranges 26), the choice costs 5 % over the best.
// bf16: fitted to 104 such launches, base the count of pick_dq_splits, 5 % either way: launches take 4.4 % less time than with that one
// on average (2 heads of 2214 rows against 10,610 keys 239 us, 130 now; 8 of 162 against 1162: 36 and 26), the choice costs 4 % over the best.
static int pick_splits(const SegShape &s, int most, int elem_bytes)
{
    struct Cost { double start, dq_us, dq_more, dkv_us, dkv_halves_us, dkv_more, dkv_slow, rate, last, zeros_rate, merge, merge_bytes, merge_rate; };
    static const Cost f64 = {4.3, 3.95, 0.0, 6.8, 3.3, 0.2, 0.136, 0.717, 0.36, 5.0, 3.0, 4.0, 1.1},
                      f128 = {0.0, 7.0, 0.6, 7.8, 7.8, 1.5, 0.0, 0.97, 0.58, 5.0, 3.0, 4.0, 1.5},
                      b128 = {7.4, 1.305, 0.58, 1.42, 1.42, 2.6, 0.0, 1.243, 0.28, 9.0, 1.8, 2.0, 1.08};
    const bool is_float = elem_bytes == 4;
    const Cost &c = !is_float ? b128 : s.d == 64 ? f64 : f128;
    const double bhs = (double)s.B * s.H, room = s.d == 64 ? 512.0 : 256.0;      // workgroups that fit the chip
    const int64_t seen = s.causal && s.s0 + s.l_s < s.l_x ? s.s0 + s.l_s : (int64_t)s.l_x, first = s.causal ? s.s0 + (s.l_s < 128 ? s.l_s : 128) : (int64_t)s.l_x;
    const int64_t tiles = (seen + 63) / 64, q_tiles = (s.l_s + 63) / 64, dq_tiles = (s.l_s + 127) / 128;
    const double mean_tiles = 0.5 * (double)(((first < seen ? first : seen) + 63) / 64 + tiles);
    const double zeros_mb = (double)(s.l_x - seen) * bhs * s.d * 8e-6, dq_m = bhs * s.l_s * s.d * 1e-6;
    auto estimate = [&](int sp) {
        const bool halves = is_float && f32_bwd_halves(s, sp);
        const int64_t keys = halves ? 64 : 128, key_tiles = (seen + keys - 1) / keys;
        const int64_t full = s.causal && s.s0 / keys < key_tiles ? s.s0 / keys : key_tiles;     // key tiles that all rows see; the others half of them
        const double dkv_us = halves ? c.dkv_halves_us : c.dkv_us, n_dq = (double)dq_tiles * bhs * sp, n_dkv = (double)key_tiles * bhs, N = n_dq + n_dkv;
        const double shared = N < 256.0 ? 0.0 : N > 512.0 ? 1.0 : N / 256.0 - 1.0;
        const double dq = ((double)((tiles + sp - 1) / sp) + c.dq_more) * c.dq_us, dkv = ((double)q_tiles + c.dkv_more) * dkv_us;
        const double longest = (dq > dkv ? dq : dkv) * (1.0 + c.dkv_slow * shared);
        double balance = c.rate / 256.0 * (((double)dq_tiles * bhs * mean_tiles + n_dq * c.dq_more) * c.dq_us +
                                           (bhs * ((double)full + 0.5 * (double)(key_tiles - full)) * (double)q_tiles + n_dkv * c.dkv_more) * dkv_us);
        if (N > room) balance += c.last * dkv;
        const double t = c.start + larger_or_both(longest, balance) + zeros_mb / c.zeros_rate;
        return sp > 1 ? t + c.merge + dq_m * (2 * sp + 1) * c.merge_bytes / c.merge_rate : t;
    };
    const int base = is_float ? (int)std::min<int64_t>((tiles + 15) / 16, most) : pick_dq_splits(s, most);
    const double base_t = estimate(base);
    int best = base;
    double best_t = base_t;
    for (int sp = 1; sp <= most; ++sp) {
        if (sp == base) continue;
        const double t = estimate(sp);
        if (t < (sp < base && is_float ? 0.85 : 0.95) * base_t && t < best_t) { best_t = t; best = sp; }
    }
    return best;
}

BwdLaunch plan_bwd(const SegShape &s, bool with_drop, int elem_bytes, bool may_own)
{
    const int most = choose_splits(s.l_s, s.l_x, s.B, s.H, dq_rows_per_wg(elem_bytes, s.d));
    if (elem_bytes == 4) return {pick_splits(s, most, elem_bytes), 1, false, false, false, false};
    const BwdPlan plan = s.l_s <= kSkinnyRows ? BwdPlan{pick_dq_splits(s, most), 1}
                         : s.d == 128         ? BwdPlan{pick_splits(s, most, elem_bytes), 1}
                                              : pick_bwd_plan(s, with_drop, most, may_own);
    const int64_t seen = s.causal && s.s0 + s.l_s < s.l_x ? s.s0 + s.l_s : (int64_t)s.l_x;
    const int dq_tiles = (int)(((seen + 63) / 64 + plan.splits - 1) / plan.splits + plan.groups - 1) / plan.groups;
    const int one_pass = may_own ? skinny_splits(s, with_drop, elem_bytes, most, dq_tiles) : 0;
    if (one_pass > 0) return {one_pass, 1, true, true, false, false};
    const bool own = may_own && bwd_own_values(s, plan.splits, plan.groups), skinny = own && !with_drop && s.l_s <= kSkinnyRows;
    return {plan.splits, plan.groups, false, own, skinny, !skinny && bwd_narrow(s, plan.splits, plan.groups, with_drop)};
}

template <typename T, int D>
static hipError_t launch_bwd_d(const SegShape &s, const DropArgs &dr, const T *q, const T *k, const T *v, const T *out,
                               const float *lse, const T *dO, T *dq, float *dk_part, float *dv_part,
                               const Workspace &ws, hipStream_t st)
{
    hipError_t e;
    // Gradients may be written over `out`, which nothing reads afterwards.  Workgroups that compute D themselves read all
    // rows of `out` while others write gradients: then a launch of its own reads it first.
    const size_t rows_bytes = (size_t)s.B * s.l_s * s.H * D * sizeof(T), part_bytes = (size_t)s.B * s.l_x * s.H * D * sizeof(float);
    const bool out_first = overlaps(dq, rows_bytes, out, rows_bytes) || overlaps(dk_part, part_bytes, out, rows_bytes) ||
                           overlaps(dv_part, part_bytes, out, rows_bytes);
    const BwdLaunch plan = plan_bwd(s, dr.thr != 0, (int)sizeof(T), !out_first);
    const int n_splits = plan.splits;
    if constexpr (sizeof(T) == 2) {
        if ((e = launch_bwd_bf16_main(s, dr, q, k, v, out, lse, dO, dq, dk_part, dv_part, ws, plan, st)) != hipSuccess) return e;
    } else {
        {
            const int64_t threads = (int64_t)s.B * s.l_s * s.H * 16;
            TimedLaunch tl(K_ROWDOT, st);
            hipLaunchKernelGGL((bwd_rowdot_kernel<T, D>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, s, out, dO, ws.D);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        if ((e = launch_bwd_f32_main(s, dr, q, k, v, lse, dO, dq, dk_part, dv_part, ws, n_splits, st)) != hipSuccess) return e;
    }
    if (n_splits > 1) {
        const int64_t n4 = (int64_t)s.B * s.l_s * s.H * D / 4;
        TimedLaunch tl(K_DQ_MERGE, st);
        const auto kernel = n_splits <= 2   ? bwd_dq_merge_kernel<T, 2>
                            : n_splits <= 4 ? bwd_dq_merge_kernel<T, 4>
                            : n_splits <= 8 ? bwd_dq_merge_kernel<T, 8>
                                            : bwd_dq_merge_kernel<T, 16>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, st, ws.dq_part, n_splits, n4, dq);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename T>
hipError_t launch_bwd(const SegShape &s, const DropArgs &dr, const T *q, const T *k, const T *v, const T *out,
                      const float *lse, const T *dO, T *dq, float *dk_part, float *dv_part, const Workspace &ws,
                      hipStream_t st)
{
    if (s.d == 64) return launch_bwd_d<T, 64>(s, dr, q, k, v, out, lse, dO, dq, dk_part, dv_part, ws, st);
    return launch_bwd_d<T, 128>(s, dr, q, k, v, out, lse, dO, dq, dk_part, dv_part, ws, st);
}

template hipError_t launch_bwd<bf16_t>(const SegShape &, const DropArgs &, const bf16_t *, const bf16_t *, const bf16_t *,
                                       const bf16_t *, const float *, const bf16_t *, bf16_t *, float *, float *,
                                       const Workspace &, hipStream_t);
template hipError_t launch_bwd<float>(const SegShape &, const DropArgs &, const float *, const float *, const float *,
                                      const float *, const float *, const float *, float *, float *, float *,
                                      const Workspace &, hipStream_t);

} // namespace lss
