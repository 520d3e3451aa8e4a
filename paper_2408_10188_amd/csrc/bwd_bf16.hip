// Backward ring step on bf16 matrix cores, head_dim 128: dispatch of its two kernels and the
// small pre-pass they share.  No floating-point atomics, so results are bit-identical from run
// to run:
//
//  dq kernel   (query-stationary, like the forward): a wavefront owns 32 query rows, keeps Q,
//              dO (B operands) and the dQ^T accumulator in registers, streams K/V tiles:
//                S^T = K Q^T,  dP^T = V dO^T,  dS^T = P^T * (dP^T - delta),  dQ^T += K^T dS^T
//  dkdv kernel (key-stationary): a wavefront owns 32 keys of one KV head, keeps K, V (B
//              operands) and the dK^T, dV^T accumulators in registers, streams Q/dO tiles of
//              every query head of the group:
//                S = Q K^T,  dP = dO V^T,  P = exp(S - LSE),  dS = P * (dP - delta),
//                dV^T += dO^T P,  dK^T += Q^T dS
// Each recomputes S and dP (7 tile products in total instead of 5) in exchange for
// exclusive ownership of its outputs.
//
// Workspace of a backward call: [-LSE*log2e | -delta] padded to whole 64-row tiles (read by the dK/dV
// kernel, written by the dQ kernel or, without one, by bwd_stats_kernel), then the area for the partial dQ of cut
// query tiles and, later on the same stream, the partial dK / dV sums of split key tiles.
#include "common.h"

namespace mmsp {
namespace {

__global__ __launch_bounds__(256) void bwd_stats_kernel(const float* __restrict__ lse, const float* __restrict__ delta,
                                                        int64_t lse_hs, int row0, int n_rows, int padded,
                                                        float* __restrict__ nl2, float* __restrict__ ndl) {
  const int i = blockIdx.x * 256 + threadIdx.x, h = blockIdx.y;
  if (i >= padded) return;
  float n = -INFINITY, nd = 0.f;
  if (i < n_rows) {
    const float L = lse[(int64_t)h * lse_hs + row0 + i];
    n = L == -INFINITY ? -INFINITY : -L * kLog2e;      // a row that saw nothing: P = exp2(-inf) = 0
    nd = -delta[(int64_t)h * lse_hs + row0 + i];
  }
  nl2[(int64_t)h * padded + i] = n;
  ndl[(int64_t)h * padded + i] = nd;
}

}  // namespace

hipError_t launch_bwd_stats(const float* lse, const float* delta, int64_t lse_hs, int Hq, int row0, int n_rows,
                            float* nl2, float* ndl, hipStream_t stream) {
  const int padded = (int)tiles_of(n_rows) * 64;
  if (padded == 0) return hipSuccess;
  bwd_stats_kernel<<<dim3((padded + 255) / 256, Hq), dim3(256), 0, stream>>>(lse, delta, lse_hs, row0, n_rows, padded, nl2, ndl);
  return hipGetLastError();
}

int64_t bwd_bf16_workspace_bytes(int Hq, int64_t n_q) {
  return 2 * Hq * tiles_of(n_q) * 64 * (int64_t)sizeof(float) + bwd_dkdv_partial_bytes();
}

// A call that wants all three gradients has the dQ kernel write the row statistics, which its
// workgroups hold anyway: a launch less (4 to 5 us a step; 320 rows x 4 heads, two steps forward and
// backward: 120 -> 117 us).
hipError_t launch_bwd_bf16(const StepArgs& a, hipStream_t stream) {
  BwdWorkspace w;                                        // statistics, then the partial-sum area
  w.n_qtiles = (int32_t)tiles_of(a.n_q);
  w.nl2 = reinterpret_cast<float*>(a.ws);
  w.ndl = w.nl2 + (int64_t)a.Hq * w.n_qtiles * 64;
  w.partial = w.ndl + (int64_t)a.Hq * w.n_qtiles * 64;
  if (a.dq != nullptr) {
    const hipError_t e = launch_bwd_dq_bf16(a, a.dk != nullptr ? &w : nullptr, stream);
    if (e != hipSuccess || a.dk == nullptr) return e;
  } else {
    const hipError_t e = launch_bwd_stats(a.lse_final, a.delta, a.lse_hs, a.Hq, a.q_row0, a.n_q, w.nl2, w.ndl, stream);
    if (e != hipSuccess) return e;
  }
  return launch_bwd_dkdv_bf16(a, w, stream);
}

}  // namespace mmsp
