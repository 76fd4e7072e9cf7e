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
#include "lss_common.h"
#include "lss_kernels.h"

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

// dq = sum over splits, in split order.
template <typename T>
__global__ __launch_bounds__(256) void bwd_dq_merge_kernel(const float *__restrict__ dq_part, int n_splits,
                                                           int64_t n4, T *__restrict__ dq)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n4) return;
    f32x4 acc = *reinterpret_cast<const f32x4 *>(dq_part + i * 4);
    for (int sp = 1; sp < n_splits; ++sp) acc += *reinterpret_cast<const f32x4 *>(dq_part + (sp * n4 + i) * 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) dq[i * 4 + e] = (T)acc[e];
}

template <typename T, int D>
static hipError_t launch_bwd_d(const SegShape &s, const DropArgs &dr, const T *q, const T *k, const T *v, const T *out,
                               const float *lse, const T *dO, T *dq, float *dk_part, float *dv_part,
                               const Workspace &ws, hipStream_t st)
{
    hipError_t e;
    // The dQ workgroups share their launch with the dK/dV ones and need not fill the chip alone:
    // keys are split only so far that a dQ workgroup (64 key tiles at most, 16 of the slower float ones) does
    // not outlast the rest of the launch.  Never more splits than the workspace was sized for.
    int n_splits = choose_splits(s.l_s, s.l_x, s.B, s.H, dq_rows_per_wg((int)sizeof(T), D));
    const int64_t kv_extent = s.causal ? (s.s0 + s.l_s < s.l_x ? s.s0 + s.l_s : (int64_t)s.l_x) : (int64_t)s.l_x;
    constexpr int kMostKeys = 64 * (sizeof(T) == 2 ? 64 : 16);
    const int want = (int)((kv_extent + kMostKeys - 1) / kMostKeys);
    if (want < n_splits) n_splits = want < 1 ? 1 : want;
    if constexpr (sizeof(T) == 2) {
        if ((e = launch_bwd_bf16_main(s, dr, q, k, v, out, lse, dO, dq, dk_part, dv_part, ws, n_splits, st)) != hipSuccess)
            return e;
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
        hipLaunchKernelGGL((bwd_dq_merge_kernel<T>), dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, st,
                           ws.dq_part, n_splits, n4, dq);
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
