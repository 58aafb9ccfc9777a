// hgt_weights.h -- entries of HGT's folded per-relation weights, shared by the
// forward's and the backward's kernels: both form the segment queries from them,
// and the backward's scores have to match the forward's bit for bit.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace rgnn {

// Wf[r][j][n] = mu[r] scale sum_k Wq[t][j][k] Watt[r, i][n - i dk][k - i dk] over the k
// of n's head i, t = rel_dsttype[r]: the query projection folded into the
// reordered query weights.  idx = (r, j, n).
__device__ __forceinline__ float hgt_qp_fold_entry(int64_t idx, const float *Wq, const float *Watt, const float *mu,
                                                   float scale, const int32_t *rel_dsttype, int D, int heads)
{
    const int r = (int)(idx / (D * D)), j = (int)(idx / D % D), n = (int)(idx % D);
    const int dk = D / heads, i = n / dk;
    const float *wq = Wq + ((size_t)rel_dsttype[r] * D + j) * D + i * dk;
    const float *wa = Watt + (((size_t)r * heads + i) * dk + (n - i * dk)) * dk;
    float acc = 0.f;
#pragma unroll 16
    for (int k = 0; k < dk; ++k) acc = fmaf(wq[k], wa[k], acc);
    return mu[r] * scale * acc;
}

// Wmt[r][i dk + b][i dk + a] = Wmsg[r][i][a][b], 0 off the head blocks: the
// block-diagonal W_msg^T.  idx = (r, row, col).
__device__ __forceinline__ float hgt_msgT_entry(int64_t idx, const float *Wmsg, int D, int heads)
{
    const int r = (int)(idx / (D * D)), row = (int)(idx / D % D), col = (int)(idx % D);
    const int dk = D / heads, i = row / dk;
    if (col / dk != i) return 0.f;
    return Wmsg[(((size_t)r * heads + i) * dk + (col - i * dk)) * dk + (row - i * dk)];
}

// Wg[r][g][i dk + a] = sum_b Wa[t(r)][i dk + b][g] Wmsg[r, i][a][b].  idx = (r, g, n).
__device__ __forceinline__ float hgt_msg_fold_entry(int64_t idx, const float *Wa, const float *Wmsg,
                                                    const int32_t *rel_dsttype, int D, int heads)
{
    const int r = (int)(idx / (D * D)), g = (int)(idx / D % D), n = (int)(idx % D);
    const int dk = D / heads, i = n / dk;
    const float *wa = Wa + ((size_t)rel_dsttype[r] * D + i * dk) * D + g;
    const float *wm = Wmsg + (((size_t)r * heads + i) * dk + (n - i * dk)) * dk;
    float acc = 0.f;
#pragma unroll 16
    for (int b = 0; b < dk; ++b) acc = fmaf(wa[(size_t)b * D], wm[b], acc);
    return acc;
}

}  // namespace rgnn
