// fp32 path (io_dtype = f32): true fp32 products and accumulation with accurate expf/logf, for
// the full-precision configuration whose tolerance (1e-5) rules out bf16 matrix cores.
//
// The calls are small (a few hundred rows), so what bounds them is the serial chain of one row and
// the wavefronts in flight, not a rate.  One thread per row walked all keys one after the other (256
// rows of 2 heads: 8 wavefronts on the chip, 2240 us for a two-step forward and backward pass).
// Here a workgroup owns 16 rows and its 8 wavefronts take every eighth block of 16 streamed rows, each
// with partial results of its own that meet in LDS at the end, so the loop has no barrier; the
// products run on v_mfma_f32_16x16x4_f32 (fp32 operands and accumulation) with operands loaded
// straight from memory: a block's rows are used once per wavefront, so LDS tiles would buy nothing.
// The same pass now takes 72 us (nine launches, the larger ones 9 to 19 us each for chains of two to four blocks per
// wavefront) and is closer to 64 bits (3.2e-7, was 5.8e-7).
//
// v_mfma_f32_16x16x4_f32, C[16x16] += A[16x4] B[4x16], lane L: A row L % 16, k = L / 16; B column L % 16,
// k = L / 16; C column L % 16, rows (L / 16) * 4 + i, i = 0..3.  Which k a slot stands for is free as long
// as A and B agree, and so is the order of C's rows, which makes every load a contiguous one:
//   first products (X Y^T, contraction over d):  slot L / 16 of step s is d = (L / 16) * D/4 + s, so a lane
//     holds D/4 consecutive elements of row L % 16 ("natural" rows);
//   second products (Z^T W, contraction over the streamed rows, W in C's layout): step i takes the rows
//     (L / 16) * 4 + i that C's register i holds, and C row r of d block b is d = r * D/16 + b, so a lane
//     holds D/16 consecutive elements of four rows ("transposed" rows).
#include "common.h"

namespace mmsp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kRows = 16;            // rows of a workgroup, and of a streamed block
constexpr int kWaves = 8;

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <int N>
__device__ __forceinline__ void load_floats(float (&x)[N], const float* p) {
#pragma unroll
  for (int i = 0; i < N / 4; ++i) {
    const float4 v = *reinterpret_cast<const float4*>(p + i * 4);
    x[4 * i] = v.x; x[4 * i + 1] = v.y; x[4 * i + 2] = v.z; x[4 * i + 3] = v.w;
  }
}

// X Y^T of two sets of natural rows, two chains of accumulation
template <int D>
__device__ __forceinline__ f32x4 first_product(const float (&x)[D / 4], const float (&y)[D / 4]) {
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
  for (int s = 0; s < D / 4; s += 2) { s0 = mfma16(x[s], y[s], s0); s1 = mfma16(x[s + 1], y[s + 1], s1); }
  return s0 + s1;
}

// acc[b] (d block b x columns) += Z^T W.  z[i]: transposed row (lane / 16) * 4 + i of the block; W is zero
// where a pair is hidden.  A hidden pair contributes nothing whatever its row holds, but 0 * inf in a
// matrix instruction would: a block with hidden pairs and values that are not finite is added term by term.
template <int D>
__device__ __forceinline__ void second_product(f32x4 (&acc)[D / 16], const float (&z)[4][D / 16], const f32x4& w, bool hidden,
                                               uint32_t seen /* bit i: pair i of this lane is visible */, int lane) {
  if (hidden) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int b = 0; b < D / 16; ++b) t = fmaf(z[i][b], 0.f, t);
    if (__any(t != 0.f)) {
      for (int r = 0; r < kRows; ++r) {                  // streamed row r: weight and visibility from lane (r / 4, column)
        const int src = (r >> 2) * 16 + (lane & 15), i = r & 3;
        const float wi = i == 0 ? w[0] : i == 1 ? w[1] : i == 2 ? w[2] : w[3];
        const float wr = __shfl(wi, src);
        const bool on = (__shfl((int)seen, src) >> i) & 1;
#pragma unroll
        for (int b = 0; b < D / 16; ++b) {
          const float zi = i == 0 ? z[0][b] : i == 1 ? z[1][b] : i == 2 ? z[2][b] : z[3][b];
#pragma unroll
          for (int k = 0; k < 4; ++k) {                  // C row (lane / 16) * 4 + k: its elements are in lane (r / 4, that row)
            const float zr = __shfl(zi, (r >> 2) * 16 + (lane >> 4) * 4 + k);
            if (on) acc[b][k] = fmaf(wr, zr, acc[b][k]);
          }
        }
      }
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int b = 0; b < D / 16; ++b) acc[b] = mfma16(z[i][b], w[i], acc[b]);
}

// A wavefront's share of the result, [16 columns][D] in LDS (rows padded against bank conflicts)
template <int D>
__device__ __forceinline__ void store_partial(float* part, const f32x4 (&acc)[D / 16], int lane) {
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int b = 0; b < D / 16; b += 4) {
      float* p = part + (lane & 15) * (D + 4) + ((lane >> 4) * 4 + k) * (D / 16) + b;
      *reinterpret_cast<float4*>(p) = make_float4(acc[b][k], acc[b + 1][k], acc[b + 2][k], acc[b + 3][k]);
    }
}

template <int D>
constexpr int kPartFloats = kRows * (D + 4);

// sum over the wavefronts of float4 `item` (column item / (D/4)) of the result
template <int D>
__device__ __forceinline__ float4 sum_partials(const float* parts, int item) {
  const float* p = parts + item / (D / 4) * (D + 4) + item % (D / 4) * 4;
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const float4 y = *reinterpret_cast<const float4*>(p + w * kPartFloats<D>);
    x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w;
  }
  return x;
}

template <int D>
__global__ __launch_bounds__(64 * kWaves) void fwd_f32_kernel(StepArgs a) {
  __shared__ __attribute__((aligned(16))) float parts[kWaves * kPartFloats<D>];
  __shared__ float ms[kWaves][kRows], ls[kWaves][kRows];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, col = lane & 15;
  const int row0 = blockIdx.x * kRows, h = blockIdx.y, kvh = h / a.group;
  const int rowc = min(row0 + col, a.n_q - 1);
  int lo, hi;
  key_interval_of_row(a, CuGlobal{a.cu}, rowc, lo, hi);
  const int lo_first = __builtin_amdgcn_readlane(lo, 0), hi_first = __builtin_amdgcn_readlane(hi, 0);
  const int lo_last = __builtin_amdgcn_readlane(lo, 15), hi_last = __builtin_amdgcn_readlane(hi, 15);
  const int kb0 = lo_first / kRows, kb1 = hi_last >= lo_first ? hi_last / kRows : kb0 - 1;

  float q[D / 4];
  load_floats(q, reinterpret_cast<const float*>(a.q) + (int64_t)(a.q_row0 + rowc) * a.q_ts + (int64_t)h * a.q_hs + g * (D / 4));
  const float* kb_ = reinterpret_cast<const float*>(a.k) + (int64_t)a.k_row0 * a.kv_ts + (int64_t)kvh * a.kv_hs;
  const float* vb_ = reinterpret_cast<const float*>(a.v) + (int64_t)a.k_row0 * a.kv_ts + (int64_t)kvh * a.kv_hs;
  auto load_k = [&](float (&x)[D / 4], int kb) {
    load_floats(x, kb_ + (int64_t)min(kb * kRows + col, a.n_k - 1) * a.kv_ts + g * (D / 4));
  };

  f32x4 acc[D / 16];
#pragma unroll
  for (int b = 0; b < D / 16; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;                          // l: this lane's share (its 4 of every 16 keys)
  float k[D / 4];
  if (kb0 + wave <= kb1) load_k(k, kb0 + wave);
  for (int kb = kb0 + wave; kb <= kb1; kb += kWaves) {
    float v[4][D / 16], k_next[D / 4];
#pragma unroll
    for (int i = 0; i < 4; ++i) load_floats(v[i], vb_ + (int64_t)min(kb * kRows + g * 4 + i, a.n_k - 1) * a.kv_ts + col * (D / 16));
    load_k(k_next, min(kb + kWaves, kb1));
    f32x4 s = first_product<D>(k, q);
    const bool hidden = kb * kRows < lo_last || kb * kRows + kRows - 1 > hi_first;
    uint32_t seen = 0;
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int key = kb * kRows + g * 4 + i;
      s[i] *= a.scale;
      if (key >= lo && key <= hi) { seen |= 1u << i; mx = fmaxf(mx, s[i]); }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float mn = fmaxf(m, mx);
    const float alpha = m == -INFINITY ? 0.f : expf(m - mn);
    const float ref = mn == -INFINITY ? 0.f : mn;        // nothing but scores of -inf so far
    f32x4 p;
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[i] = (seen >> i) & 1 ? expf(s[i] - ref) : 0.f;
      sum += p[i];
    }
    l = l * alpha + sum;
    m = mn;
#pragma unroll
    for (int b = 0; b < D / 16; ++b) acc[b] *= alpha;
    second_product<D>(acc, v, p, hidden, seen, lane);
#pragma unroll
    for (int i = 0; i < D / 4; ++i) k[i] = k_next[i];
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  store_partial<D>(parts + wave * kPartFloats<D>, acc, lane);
  if (g == 0) { ms[wave][col] = m; ls[wave][col] = l; }
  __syncthreads();

  // merge of the wavefronts' partial results, and with the running one
  for (int item = threadIdx.x; item < kRows * D / 4; item += 64 * kWaves) {
    const int r = item / (D / 4), i = row0 + r;
    if (i >= a.n_q) break;
    float mt = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) mt = fmaxf(mt, ms[w][r]);
    float lt = 0.f;
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    const float* p = parts + r * (D + 4) + item % (D / 4) * 4;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float f = ms[w][r] == -INFINITY ? (ls[w][r] == 0.f ? 0.f : 1.f) : expf(ms[w][r] - mt);
      const float4 y = *reinterpret_cast<const float4*>(p + w * kPartFloats<D>);
      lt = fmaf(f, ls[w][r], lt);
      o.x = fmaf(f, y.x, o.x); o.y = fmaf(f, y.y, o.y); o.z = fmaf(f, y.z, o.z); o.w = fmaf(f, y.w, o.w);   // 0 * NaN stays NaN
    }
    const float inv = lt > 0.f ? 1.f / lt : 0.f;
    const float lse_part = lt > 0.f ? mt + logf(lt) : -INFINITY;
    const int64_t row = a.q_row0 + i;
    float4* op = reinterpret_cast<float4*>(a.o + (row * a.Hq + h) * (int64_t)D) + item % (D / 4);
    float* lp = a.lse + (int64_t)h * a.lse_hs + row;
    float wa = 0.f, wb = inv, lse_new = lse_part;
    if (a.accumulate) {
      // the lanes of a row belong to one wavefront, which reads the running value before it is replaced below
      const float la = *lp;
      const float mm = fmaxf(la, lse_part);
      if (mm == -INFINITY) continue;                     // both empty: leave the running state
      const float ea = expf(la - mm), eb = expf(lse_part - mm);
      const float tot = ea + eb;
      wa = ea / tot; wb = eb / tot * inv;
      lse_new = mm + logf(tot);
      const float4 old = *op;
      o.x = wa * old.x + wb * o.x; o.y = wa * old.y + wb * o.y; o.z = wa * old.z + wb * o.z; o.w = wa * old.w + wb * o.w;
    } else {
      o.x *= wb; o.y *= wb; o.z *= wb; o.w *= wb;
    }
    *op = o;
    if (item % (D / 4) == 0) *lp = lse_new;
  }
}

// dQ of 16 query rows of one head; parts: kWaves * kPartFloats<D> floats
template <int D>
__device__ __forceinline__ void dq_rows(const StepArgs& a, float* parts, int row_block, int h) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, col = lane & 15;
  const int row0 = row_block * kRows, kvh = h / a.group;
  const int rowc = min(row0 + col, a.n_q - 1);
  int lo, hi;
  key_interval_of_row(a, CuGlobal{a.cu}, rowc, lo, hi);
  const int lo_first = __builtin_amdgcn_readlane(lo, 0), hi_first = __builtin_amdgcn_readlane(hi, 0);
  const int lo_last = __builtin_amdgcn_readlane(lo, 15), hi_last = __builtin_amdgcn_readlane(hi, 15);
  const int kb0 = lo_first / kRows, kb1 = hi_last >= lo_first ? hi_last / kRows : kb0 - 1;
  const int64_t row = a.q_row0 + rowc;
  float q[D / 4], d_o[D / 4];
  load_floats(q, reinterpret_cast<const float*>(a.q) + row * a.q_ts + (int64_t)h * a.q_hs + g * (D / 4));
  load_floats(d_o, reinterpret_cast<const float*>(a.d_o) + (row * a.Hq + h) * (int64_t)D + g * (D / 4));
  const float L = a.lse_final[(int64_t)h * a.lse_hs + row];
  const float Dl = a.delta[(int64_t)h * a.lse_hs + row];
  if (L == -INFINITY) { lo = a.n_k; hi = a.n_k - 1; }   // a row that saw nothing: P = 0
  const bool any_empty = __any(L == -INFINITY);
  const float* kb_ = reinterpret_cast<const float*>(a.k) + (int64_t)a.k_row0 * a.kv_ts + (int64_t)kvh * a.kv_hs;
  const float* vb_ = reinterpret_cast<const float*>(a.v) + (int64_t)a.k_row0 * a.kv_ts + (int64_t)kvh * a.kv_hs;

  f32x4 acc[D / 16];
#pragma unroll
  for (int b = 0; b < D / 16; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int kb = kb0 + wave; kb <= kb1; kb += kWaves) {
    float k[D / 4], v[D / 4], kt[4][D / 16];
    const int64_t nat = (int64_t)min(kb * kRows + col, a.n_k - 1) * a.kv_ts + g * (D / 4);
    load_floats(k, kb_ + nat);
    load_floats(v, vb_ + nat);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_floats(kt[i], kb_ + (int64_t)min(kb * kRows + g * 4 + i, a.n_k - 1) * a.kv_ts + col * (D / 16));
    const f32x4 s = first_product<D>(k, q), dp = first_product<D>(v, d_o);
    const bool hidden = any_empty || kb * kRows < lo_last || kb * kRows + kRows - 1 > hi_first;
    uint32_t seen = 0;
    f32x4 ds;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int key = kb * kRows + g * 4 + i;
      const bool on = key >= lo && key <= hi;
      ds[i] = on ? expf(s[i] * a.scale - L) * (dp[i] - Dl) : 0.f;
      seen |= (uint32_t)on << i;
    }
    second_product<D>(acc, kt, ds, hidden, seen, lane);
  }
  store_partial<D>(parts + wave * kPartFloats<D>, acc, lane);
  __syncthreads();
  for (int item = threadIdx.x; item < kRows * D / 4; item += 64 * kWaves) {
    const int i = row0 + item / (D / 4);
    if (i >= a.n_q) break;
    const float4 x = sum_partials<D>(parts, item);
    float4* p = reinterpret_cast<float4*>(a.dq + ((int64_t)(a.q_row0 + i) * a.Hq + h) * (int64_t)D) + item % (D / 4);
    float4 y = *p;
    y.x += a.scale * x.x; y.y += a.scale * x.y; y.z += a.scale * x.z; y.w += a.scale * x.w;
    *p = y;
  }
}

// dK and dV of 16 keys of one KV head; the wavefronts share out the (head of the group, query block) sequence.
// parts: 2 kWaves * kPartFloats<D> floats
template <int D>
__device__ __forceinline__ void dkdv_keys(const StepArgs& a, float* parts, int key_block, int kvh) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, col = lane & 15;
  const int key0 = key_block * kRows;
  const int keyc = min(key0 + col, a.n_k - 1);
  int lo, hi;
  row_interval_of_key(a, CuGlobal{a.cu}, keyc, lo, hi);
  const int lo_first = __builtin_amdgcn_readlane(lo, 0), hi_first = __builtin_amdgcn_readlane(hi, 0);
  const int lo_last = __builtin_amdgcn_readlane(lo, 15), hi_last = __builtin_amdgcn_readlane(hi, 15);
  const int qb0 = lo_first / kRows, n_qb = hi_last >= lo_first ? hi_last / kRows - qb0 + 1 : 0;
  float k[D / 4], v[D / 4];
  {
    const int64_t nat = (int64_t)(a.k_row0 + keyc) * a.kv_ts + (int64_t)kvh * a.kv_hs + g * (D / 4);
    load_floats(k, reinterpret_cast<const float*>(a.k) + nat);
    load_floats(v, reinterpret_cast<const float*>(a.v) + nat);
  }
  f32x4 dk[D / 16], dv[D / 16];
#pragma unroll
  for (int b = 0; b < D / 16; ++b) dk[b] = dv[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float* qb_ = reinterpret_cast<const float*>(a.q) + (int64_t)a.q_row0 * a.q_ts;
  const float* dob_ = reinterpret_cast<const float*>(a.d_o) + (int64_t)a.q_row0 * a.Hq * D;
  for (int e = wave; e < n_qb * a.group; e += kWaves) {
    const int h = kvh * a.group + e / n_qb, row0 = (qb0 + e % n_qb) * kRows;
    const float* qh = qb_ + (int64_t)h * a.q_hs;
    const float* doh = dob_ + (int64_t)h * D;
    float q[D / 4], d_o[D / 4];
    const int64_t rn = min(row0 + col, a.n_q - 1);
    load_floats(q, qh + rn * a.q_ts + g * (D / 4));
    load_floats(d_o, doh + rn * a.Hq * D + g * (D / 4));
    float L[4], Dl[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t st = (int64_t)h * a.lse_hs + a.q_row0 + min(row0 + g * 4 + i, a.n_q - 1);
      L[i] = a.lse_final[st];
      Dl[i] = a.delta[st];
    }
    const f32x4 s = first_product<D>(q, k), dp = first_product<D>(d_o, v);
    // at d = 128 the 256 registers hold the natural rows, then dO's transposed rows, then Q's, but no two of them
    if (D == 128) __builtin_amdgcn_sched_barrier(0);
    float zt[4][D / 16];
#pragma unroll
    for (int i = 0; i < 4; ++i) load_floats(zt[i], doh + (int64_t)min(row0 + g * 4 + i, a.n_q - 1) * a.Hq * D + col * (D / 16));
    bool hidden = row0 < lo_last || row0 + kRows - 1 > hi_first;
    uint32_t seen = 0;
    f32x4 p, ds;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = row0 + g * 4 + i;
      const bool on = r >= lo && r <= hi && L[i] != -INFINITY;
      p[i] = on ? expf(s[i] * a.scale - L[i]) : 0.f;
      ds[i] = on ? p[i] * (dp[i] - Dl[i]) : 0.f;
      seen |= (uint32_t)on << i;
    }
    hidden = hidden || __any(seen != 15u);
    second_product<D>(dv, zt, p, hidden, seen, lane);
    if (D == 128) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_floats(zt[i], qh + (int64_t)min(row0 + g * 4 + i, a.n_q - 1) * a.q_ts + col * (D / 16));
    second_product<D>(dk, zt, ds, hidden, seen, lane);
  }
  store_partial<D>(parts + wave * kPartFloats<D>, dk, lane);
  store_partial<D>(parts + (kWaves + wave) * kPartFloats<D>, dv, lane);
  __syncthreads();
  for (int t = threadIdx.x; t < 2 * kRows * D / 4; t += 64 * kWaves) {
    const int which = t / (kRows * D / 4), item = t % (kRows * D / 4), j = key0 + item / (D / 4);
    if (j >= a.n_k) continue;
    const float mul = which ? 1.f : a.scale;
    float4 x = sum_partials<D>(parts + which * kWaves * kPartFloats<D>, item);
    x.x *= mul; x.y *= mul; x.z *= mul; x.w *= mul;
    float4* p = reinterpret_cast<float4*>((which ? a.dv : a.dk) + ((int64_t)(a.k_row0 + j) * a.Hkv + kvh) * (int64_t)D) + item % (D / 4);
    if (a.accumulate) {
      const float4 y = *p;
      x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w;
    }
    *p = x;
  }
}

// dK or dV alone (parts: kWaves * kPartFloats<D> floats): a shorter chain per element, and registers to spare, so that the
// transposed rows are on their way before the first product needs anything.
template <int D, bool kDv>
__device__ __forceinline__ void grad_keys(const StepArgs& a, float* parts, int key_block, int kvh) {
  constexpr bool kDk = !kDv;
  constexpr int kNat = kDk ? D / 4 : 4;                 // V and dO in natural rows: for dK only
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, col = lane & 15;
  const int key0 = key_block * kRows;
  const int keyc = min(key0 + col, a.n_k - 1);
  int lo, hi;
  row_interval_of_key(a, CuGlobal{a.cu}, keyc, lo, hi);
  const int lo_first = __builtin_amdgcn_readlane(lo, 0), hi_first = __builtin_amdgcn_readlane(hi, 0);
  const int lo_last = __builtin_amdgcn_readlane(lo, 15), hi_last = __builtin_amdgcn_readlane(hi, 15);
  const int qb0 = lo_first / kRows, n_qb = hi_last >= lo_first ? hi_last / kRows - qb0 + 1 : 0;
  float k[D / 4], v[kNat];
  {
    const int64_t nat = (int64_t)(a.k_row0 + keyc) * a.kv_ts + (int64_t)kvh * a.kv_hs + g * (D / 4);
    load_floats(k, reinterpret_cast<const float*>(a.k) + nat);
    if constexpr (kDk) load_floats(v, reinterpret_cast<const float*>(a.v) + nat);
  }
  f32x4 acc[D / 16];
#pragma unroll
  for (int b = 0; b < D / 16; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float* qb_ = reinterpret_cast<const float*>(a.q) + (int64_t)a.q_row0 * a.q_ts;
  const float* dob_ = reinterpret_cast<const float*>(a.d_o) + (int64_t)a.q_row0 * a.Hq * D;
  for (int e = wave; e < n_qb * a.group; e += kWaves) {
    const int h = kvh * a.group + e / n_qb, row0 = (qb0 + e % n_qb) * kRows;
    const float* qh = qb_ + (int64_t)h * a.q_hs;
    const float* doh = dob_ + (int64_t)h * D;
    float zt[4][D / 16];
    auto load_transposed = [&](const float* x, int64_t row_stride) {
#pragma unroll
      for (int i = 0; i < 4; ++i) load_floats(zt[i], x + (int64_t)min(row0 + g * 4 + i, a.n_q - 1) * row_stride + col * (D / 16));
    };
    float q[D / 4], d_o[kNat];
    const int64_t rn = min(row0 + col, a.n_q - 1);
    load_floats(q, qh + rn * a.q_ts + g * (D / 4));
    if constexpr (kDk) load_floats(d_o, doh + rn * a.Hq * D + g * (D / 4));
    float L[4], Dl[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t st = (int64_t)h * a.lse_hs + a.q_row0 + min(row0 + g * 4 + i, a.n_q - 1);
      L[i] = a.lse_final[st];
      if constexpr (kDk) Dl[i] = a.delta[st];
    }
    if constexpr (kDk) load_transposed(qh, a.q_ts);
    else load_transposed(doh, (int64_t)a.Hq * D);
    const f32x4 s = first_product<D>(q, k);
    f32x4 dp = {0.f, 0.f, 0.f, 0.f};
    if constexpr (kDk) dp = first_product<D>(d_o, v);
    bool hidden = row0 < lo_last || row0 + kRows - 1 > hi_first;
    uint32_t seen = 0;
    f32x4 p, ds;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = row0 + g * 4 + i;
      const bool on = r >= lo && r <= hi && L[i] != -INFINITY;
      p[i] = on ? expf(s[i] * a.scale - L[i]) : 0.f;
      ds[i] = on ? p[i] * (dp[i] - Dl[i]) : 0.f;
      seen |= (uint32_t)on << i;
    }
    hidden = hidden || __any(seen != 15u);
    second_product<D>(acc, zt, kDv ? p : ds, hidden, seen, lane);
  }
  store_partial<D>(parts + wave * kPartFloats<D>, acc, lane);
  __syncthreads();
  for (int item = threadIdx.x; item < kRows * D / 4; item += 64 * kWaves) {
    const int j = key0 + item / (D / 4);
    if (j >= a.n_k) continue;
    const float mul = kDv ? 1.f : a.scale;
    float4 x = sum_partials<D>(parts, item);
    x.x *= mul; x.y *= mul; x.z *= mul; x.w *= mul;
    float4* p = reinterpret_cast<float4*>((kDv ? a.dv : a.dk) + ((int64_t)(a.k_row0 + j) * a.Hkv + kvh) * (int64_t)D) + item % (D / 4);
    if (a.accumulate) {
      const float4 y = *p;
      x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w;
    }
    *p = x;
  }
}

enum Roles { kRowsOnly, kRowsAndKeys, kRowsAndSplitKeys };

// The first workgroups take key blocks (the longest chains; kRowsAndSplitKeys: n_keys for dK, then n_keys for dV), the others query blocks.
template <int D, Roles kRoles>
__global__ __launch_bounds__(64 * kWaves) void bwd_f32_kernel(StepArgs a, int n_keys) {
  __shared__ __attribute__((aligned(16))) float parts[(kRoles == kRowsAndKeys ? 2 : 1) * kWaves * kPartFloats<D>];
  int b = blockIdx.y * gridDim.x + blockIdx.x;           // roles apart: (blocks, heads), which one dimension need not hold (2^32 threads)
  const int kb = (a.n_k + kRows - 1) / kRows, qb = (a.n_q + kRows - 1) / kRows;
  if constexpr (kRoles == kRowsAndKeys) {
    if (b < n_keys) return dkdv_keys<D>(a, parts, b % kb, b / kb);
    b -= n_keys;
  }
  if constexpr (kRoles == kRowsAndSplitKeys) {
    if (b < n_keys) return grad_keys<D, false>(a, parts, b % kb, b / kb);
    b -= n_keys;
    if (b < n_keys) return grad_keys<D, true>(a, parts, b % kb, b / kb);
    b -= n_keys;
  }
  dq_rows<D>(a, parts, b % qb, b / qb);
}

// All gradients need only what the forward left, so one launch serves them where the chip has room for all workgroups at once, and with room
// to spare dK and dV are workgroups of their own: both need S, but what bounds them is the chain of loads and products of an
// element, and that is shorter for one result.  Measured at d = 128, us as two launches / one launch / one with dK and dV
// apart: 2/1 heads 256 x 256 causal 48.9 / 33.3 / 25.4, 4/1 800 x 800 (50 key blocks, 300 workgroups) 210 / 177 / 131;
// 8/8 128 x 256 (128 key blocks, 320 workgroups) 31 / 20 / 25, 256 x 256 (384) 37 / 22 / 27, 800 x 800 (1200) 138 / - / 151.
template <int D>
hipError_t launch_bwd(const StepArgs& a, hipStream_t stream) {
  const dim3 row_blocks((a.n_q + kRows - 1) / kRows, a.Hq), key_blocks((a.n_k + kRows - 1) / kRows, a.Hkv);
  const int64_t n_dq = a.dq != nullptr ? (int64_t)row_blocks.x * a.Hq : 0;
  const int64_t n_keys = a.dk != nullptr ? (int64_t)key_blocks.x * a.Hkv : 0;
  const int64_t n_cu = cu_count();
  const dim3 b(64 * kWaves);
  const int64_t apart = n_dq + 2 * n_keys;
  if (n_keys > 0 && (apart <= n_cu || (apart <= n_cu * 5 / 4 && n_keys <= n_cu / 4))) {
    bwd_f32_kernel<D, kRowsAndSplitKeys><<<dim3((unsigned)apart), b, 0, stream>>>(a, (int)n_keys);
    return hipGetLastError();
  }
  if (n_dq > 0 && n_keys > 0 && n_dq + n_keys <= n_cu) {
    bwd_f32_kernel<D, kRowsAndKeys><<<dim3((unsigned)(n_dq + n_keys)), b, 0, stream>>>(a, (int)n_keys);
    return hipGetLastError();
  }
  if (n_dq > 0) bwd_f32_kernel<D, kRowsOnly><<<row_blocks, b, 0, stream>>>(a, 0);
  if (n_keys > 0) bwd_f32_kernel<D, kRowsAndKeys><<<key_blocks, b, 0, stream>>>(a, (int)n_keys);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fwd_f32(const StepArgs& a, hipStream_t stream) {
  const dim3 g((a.n_q + kRows - 1) / kRows, a.Hq), b(64 * kWaves);
  if (a.d == 64) fwd_f32_kernel<64><<<g, b, 0, stream>>>(a);
  else fwd_f32_kernel<128><<<g, b, 0, stream>>>(a);
  return hipGetLastError();
}

hipError_t launch_bwd_f32(const StepArgs& a, hipStream_t stream) { return a.d == 64 ? launch_bwd<64>(a, stream) : launch_bwd<128>(a, stream); }

}  // namespace mmsp
