// HBM-bound helpers: the log-sum-exp merge of a partial into the running result, the cast of
// the running O to the io dtype, the backward row term delta = rowsum(dO * O), and the
// "nothing visible" fill.  All are one pass over dense [rows, Hq, d] data with 16-byte
// accesses; the [Hq, rows] statistics are tiny beside them.
#include "common.h"

namespace mmsp {
namespace {

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
  f32x2 x = {lo, hi};
  bf16x2 y = __builtin_convertvector(x, bf16x2);      // round to nearest even
  return __builtin_bit_cast(uint32_t, y);
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Where the 16 or 32 bytes of thread t lie: c-th piece of (row, head) rh; 2^shift pieces make one.  rows x heads is below 2^31
// (the fp32 tensors would not fit a GPU's memory otherwise).
struct Place {
  int c, h;
  int64_t r, off;                                       // row, first element
};
__device__ __forceinline__ Place place_of(int64_t t, int shift, int vec, int row0, const FastDiv& heads) {
  Place p;
  const uint32_t rh = (uint32_t)(t >> shift), r = rh / heads;
  p.c = (int)(t & ((1 << shift) - 1));
  p.h = (int)(rh - r * heads.d);
  p.r = (int64_t)r + row0;
  p.off = (((int64_t)row0 * heads.d + rh) << shift) * vec + p.c * vec;
  return p;
}

// One thread owns 4 consecutive d-elements of one (row, head), or 8 where only the cast to bf16 is wanted (16 bytes written
// by a thread instead of 8: 8192 x 28 heads 26.9 -> 24.9 us; a merge of 8 reads 32 bytes a lane and takes 78.5 instead of 71.4 us).  The
// threads of a (row, head) (8, 16 or 32, aligned inside a wavefront) share one LSE pair; the lane with chunk 0
// writes the merged LSE after every lane of the wavefront has read the old one.
constexpr int merge_vec(bool merge, int out) { return !merge && out == 1 ? 8 : 4; }
template <bool kMerge, int kOut /*0 none, 1 bf16, 2 f32*/>
__global__ __launch_bounds__(256) void merge_kernel(float* __restrict__ o_acc, float* __restrict__ lse_acc,
                                                    const float* __restrict__ o_part,
                                                    const float* __restrict__ lse_part, void* __restrict__ o_final,
                                                    int64_t lse_hs, FastDiv heads, int shift, int row0, int64_t n_vec) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= n_vec) return;
  constexpr int kVec = merge_vec(kMerge, kOut), kN = kVec / 4;
  const Place at = place_of(t, shift, kVec, row0, heads);
  // Also read where the running LSE is -inf: a row whose scores held a NaN has LSE = -inf and O = NaN, which 0 * O keeps.
  float4 o[kN];
#pragma unroll
  for (int i = 0; i < kN; ++i) o[i] = *reinterpret_cast<const float4*>(o_acc + at.off + i * 4);
  if (kMerge) {
    const int64_t li = at.h * lse_hs + at.r;
    const float la = lse_acc[li], lp = lse_part[li];
    const float4 p = *reinterpret_cast<const float4*>(o_part + at.off);
    const float m = fmaxf(la, lp);
    float wa, wb, ln;
    if (m == -INFINITY) { wa = 0.f; wb = 0.f; ln = -INFINITY; }
    else {
      const float ea = __expf(la - m), eb = __expf(lp - m);   // exp(-inf) = 0 handles an empty side
      const float tot = ea + eb;
      wa = ea / tot; wb = eb / tot; ln = m + __logf(tot);
    }
    o[0].x = wa * o[0].x + wb * p.x; o[0].y = wa * o[0].y + wb * p.y;
    o[0].z = wa * o[0].z + wb * p.z; o[0].w = wa * o[0].w + wb * p.w;
    *reinterpret_cast<float4*>(o_acc + at.off) = o[0];
    if (at.c == 0) lse_acc[li] = ln;
  }
  if (kOut == 1) {
    uint32_t w[2 * kN];
#pragma unroll
    for (int i = 0; i < kN; ++i) { w[2 * i] = pack_bf16x2(o[i].x, o[i].y); w[2 * i + 1] = pack_bf16x2(o[i].z, o[i].w); }
    uint16_t* const out = reinterpret_cast<uint16_t*>(o_final) + at.off;
    if constexpr (kN == 2) *reinterpret_cast<uint4*>(out) = make_uint4(w[0], w[1], w[2], w[3]);
    else *reinterpret_cast<uint2*>(out) = make_uint2(w[0], w[1]);
  } else if (kOut == 2) {
    *reinterpret_cast<float4*>(reinterpret_cast<float*>(o_final) + at.off) = o[0];
  }
}

// delta: kVec elements per thread (8 bf16 or 4 f32 = 16 bytes of each operand); the d/kVec
// lanes of one (row, head) reduce with xor-shuffles.
template <bool kBf16>
__global__ __launch_bounds__(256) void delta_kernel(const void* __restrict__ o_final, const void* __restrict__ d_o,
                                                    float* __restrict__ delta, int64_t lse_hs, FastDiv heads, int shift,
                                                    int row0, int64_t n_vec) {
  constexpr int kVec = kBf16 ? 8 : 4;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool live = t < n_vec;
  const Place at = place_of(live ? t : 0, shift, kVec, row0, heads);   // 2^shift: 8, 16 or 32 lanes
  float s = 0.f;
  if (live) {
    if (kBf16) {
      const uint4 a = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(o_final) + at.off);
      const uint4 b = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(d_o) + at.off);
      s = bf16_lo(a.x) * bf16_lo(b.x) + bf16_hi(a.x) * bf16_hi(b.x) + bf16_lo(a.y) * bf16_lo(b.y) +
          bf16_hi(a.y) * bf16_hi(b.y) + bf16_lo(a.z) * bf16_lo(b.z) + bf16_hi(a.z) * bf16_hi(b.z) +
          bf16_lo(a.w) * bf16_lo(b.w) + bf16_hi(a.w) * bf16_hi(b.w);
    } else {
      const float4 a = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(o_final) + at.off);
      const float4 b = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(d_o) + at.off);
      s = a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w;
    }
  }
  for (int w = 1 << shift >> 1; w > 0; w >>= 1) s += __shfl_xor(s, w);
  if (live && at.c == 0) delta[at.h * lse_hs + at.r] = s;
}

__global__ __launch_bounds__(256) void fill_empty_kernel(float* __restrict__ o, float* __restrict__ lse,
                                                         int64_t lse_hs, FastDiv heads, int shift, int row0, int64_t n_vec) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= n_vec) return;
  const Place at = place_of(t, shift, 4, row0, heads);
  *reinterpret_cast<float4*>(o + at.off) = make_float4(0.f, 0.f, 0.f, 0.f);
  if (at.c == 0) lse[at.h * lse_hs + at.r] = -INFINITY;
}

__global__ __launch_bounds__(256) void zero_kernel(float4* __restrict__ p, int64_t n_vec) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n_vec) p[t] = make_float4(0.f, 0.f, 0.f, 0.f);
}

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

}  // namespace

hipError_t launch_zero_f32(float* p, int64_t n, hipStream_t stream) {
  const int64_t n_vec = n / 4;
  if (n_vec == 0) return hipSuccess;
  zero_kernel<<<grid_for(n_vec, 256), 256, 0, stream>>>(reinterpret_cast<float4*>(p), n_vec);
  return hipGetLastError();
}

hipError_t launch_fill_empty(float* o, float* lse, int64_t lse_hs, int Hq, int d, int row0, int n_rows,
                             hipStream_t stream) {
  const int64_t n_vec = (int64_t)n_rows * Hq * (d / 4);
  if (n_vec == 0) return hipSuccess;
  fill_empty_kernel<<<grid_for(n_vec, 256), 256, 0, stream>>>(o, lse, lse_hs, fast_div(Hq), __builtin_ctz(d / 4), row0, n_vec);
  return hipGetLastError();
}

hipError_t launch_merge(float* o_acc, float* lse_acc, const float* o_part, const float* lse_part, void* o_final,
                        int io_dtype, int64_t lse_hs, int Hq, int d, int row0, int n_rows, hipStream_t stream) {
  if (n_rows == 0) return hipSuccess;
  const bool merge = o_part != nullptr;
  const int out = o_final == nullptr ? 0 : (io_dtype == 0 ? 1 : 2), vec = merge_vec(merge, out), shift = __builtin_ctz(d / vec);
  const int64_t n_vec = (int64_t)n_rows * Hq * (d / vec);
  const dim3 g(grid_for(n_vec, 256)), b(256);
#define MMSP_MERGE(M, O) \
  merge_kernel<M, O><<<g, b, 0, stream>>>(o_acc, lse_acc, o_part, lse_part, o_final, lse_hs, fast_div(Hq), shift, row0, n_vec)
  if (merge) { if (out == 0) MMSP_MERGE(true, 0); else if (out == 1) MMSP_MERGE(true, 1); else MMSP_MERGE(true, 2); }
  else       { if (out == 1) MMSP_MERGE(false, 1); else if (out == 2) MMSP_MERGE(false, 2); }
#undef MMSP_MERGE
  return hipGetLastError();
}

hipError_t launch_delta(const void* o_final, const void* d_o, float* delta, int io_dtype, int64_t lse_hs, int Hq,
                        int d, int row0, int n_rows, hipStream_t stream) {
  const int vec = io_dtype == 0 ? 8 : 4;
  const int64_t n_vec = (int64_t)n_rows * Hq * (d / vec);
  if (n_vec == 0) return hipSuccess;
  const dim3 g(grid_for(n_vec, 256)), b(256);
  const int shift = __builtin_ctz(d / vec);
  if (io_dtype == 0) delta_kernel<true><<<g, b, 0, stream>>>(o_final, d_o, delta, lse_hs, fast_div(Hq), shift, row0, n_vec);
  else delta_kernel<false><<<g, b, 0, stream>>>(o_final, d_o, delta, lse_hs, fast_div(Hq), shift, row0, n_vec);
  return hipGetLastError();
}

}  // namespace mmsp
