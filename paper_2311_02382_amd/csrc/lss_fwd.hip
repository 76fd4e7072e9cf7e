// Forward of Eq. 2 (Section 3, Principle 3) for one segment: the number of key splits, the main kernel's launch
// (lss_fwd_bf16.hip, lss_f32.hip) and the merge of the splits' partial results.
#include "lss_common.h"
#include "lss_kernels.h"

namespace lss {

// Fixed-order merge of the split-KV partial results of one query row:
//   lse = log sum_s exp(lse_s),  out = sum_s exp(lse_s - lse) out_s.
// One thread per (b*H + h, r, group of 4 columns).
// MAXS: compile-time bound of n_splits (loop unrolling; all loads of a thread issued together)
template <typename T, int D, int MAXS>
__global__ __launch_bounds__(256) void fwd_merge_kernel(SegShape s, const float *__restrict__ o_part,
                                                        const float *__restrict__ lse_part, int n_splits,
                                                        T *__restrict__ out, float *__restrict__ lse)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t rows = (int64_t)s.B * s.H * s.l_s;
    if (idx >= rows * (D / 4)) return;
    const int64_t row = idx / (D / 4);
    const int c4 = (int)(idx % (D / 4)) * 4;
    // all loads of a thread are independent: issue them together, then combine in split order
    float l[MAXS];
    f32x4 part[MAXS];
#pragma unroll
    for (int sp = 0; sp < MAXS; ++sp) {
        const int spc = sp < n_splits ? sp : n_splits - 1;
        l[sp] = __builtin_nontemporal_load(lse_part + spc * rows + row);
        part[sp] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(o_part + (spc * rows + row) * D + c4));
    }
    float mx = -INFINITY;
#pragma unroll
    for (int sp = 0; sp < MAXS; ++sp)
        if (sp < n_splits) mx = fmaxf(mx, l[sp]);
    float sum = 0.f;
#pragma unroll
    for (int sp = 0; sp < MAXS; ++sp)
        if (sp < n_splits) sum += expf(l[sp] - mx);
    const float total = mx + logf(sum);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int sp = 0; sp < MAXS; ++sp)
        if (sp < n_splits) acc += expf(l[sp] - total) * part[sp];
    const int r = (int)(row % s.l_s);
    const int64_t bh = row / s.l_s;
    const int64_t b = bh / s.H, h = bh % s.H;
    T *dst = out + ((b * s.l_s + r) * s.H + h) * D + c4;
#pragma unroll
    for (int i = 0; i < 4; ++i) dst[i] = (T)acc[i];
    if (c4 == 0) lse[row] = total;
}

template <typename T, int D>
static hipError_t launch_fwd_d(const SegShape &s, const DropArgs &drop, const T *q, const T *k, const T *v, T *out,
                               float *lse, const Workspace &ws, hipStream_t st)
{
    // Under the causal mask a segment near the start of the sequence sees few keys: the split count
    // follows the keys this segment's query tiles see, within what the workspace has room for.
    hipError_t e;
    int n_splits;
    if constexpr (sizeof(T) == 2) {
        const FwdPlan plan = pick_fwd_plan(s, drop.thr != 0, ws.fwd_splits);
        n_splits = plan.splits;
        e = launch_fwd_bf16_main(s, drop, q, k, v, out, lse, ws, plan, st);
    } else {
        n_splits = pick_float_fwd_splits(s, ws.fwd_splits);
        e = launch_fwd_f32_main(s, drop, q, k, v, out, lse, ws, n_splits, st);
    }
    if (e != hipSuccess || n_splits == 1) return e;
    const int64_t items = (int64_t)s.B * s.H * s.l_s * (D / 4);
    {
        TimedLaunch tl(K_FWD_MERGE, st);
        const dim3 grid((unsigned)((items + 255) / 256)), block(256);
        if (n_splits <= 2)
            hipLaunchKernelGGL((fwd_merge_kernel<T, D, 2>), grid, block, 0, st, s, ws.o_part, ws.lse_part, n_splits, out, lse);
        else if (n_splits <= 4)
            hipLaunchKernelGGL((fwd_merge_kernel<T, D, 4>), grid, block, 0, st, s, ws.o_part, ws.lse_part, n_splits, out, lse);
        else if (n_splits <= 8)
            hipLaunchKernelGGL((fwd_merge_kernel<T, D, 8>), grid, block, 0, st, s, ws.o_part, ws.lse_part, n_splits, out, lse);
        else
            hipLaunchKernelGGL((fwd_merge_kernel<T, D, 16>), grid, block, 0, st, s, ws.o_part, ws.lse_part, n_splits, out, lse);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_fwd(const SegShape &s, const DropArgs &drop, const T *q, const T *k, const T *v, T *out, float *lse,
                      const Workspace &ws, hipStream_t st)
{
    if (s.d == 64) return launch_fwd_d<T, 64>(s, drop, q, k, v, out, lse, ws, st);
    return launch_fwd_d<T, 128>(s, drop, q, k, v, out, lse, ws, st);
}

template hipError_t launch_fwd<bf16_t>(const SegShape &, const DropArgs &, const bf16_t *, const bf16_t *, const bf16_t *,
                                       bf16_t *, float *, const Workspace &, hipStream_t);
template hipError_t launch_fwd<float>(const SegShape &, const DropArgs &, const float *, const float *, const float *, float *,
                                      float *, const Workspace &, hipStream_t);

} // namespace lss
