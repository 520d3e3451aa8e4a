// Cutting the key range of query-stationary kernels (forward, dQ) into several workgroups per query tile,
// and the kernels that combine the partial results.
//
// A workgroup owns up to 256 or 128 (row, head) pairs of one KV head and takes a CU for as long as it needs for all its keys, so a
// block of few rows leaves most of the chip idle: 203 rows x 28 / 4 heads are 24 workgroups of 256 on 256 CUs, 783 us for 32768
// keys with the final cast.  With the keys cut in ranges, each storing its partial result in the caller's workspace, the same
// two calls take 107 us.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "common.h"

namespace mmsp {
namespace {

// (O, LSE) of a row = log-sum-exp merge of its partial results, and with the running one when accumulate.  32 threads
// take 4 elements of d each; kGroups of them share out the ranges of a (row, head), so that a chain of dependent loads and sums is
// nsplit / kGroups long, and meet in LDS.
template <int kGroups>
__global__ __launch_bounds__(256) void fwd_combine_kernel(const float* __restrict__ part_o, const float* __restrict__ part_lse, int nsplit,
                                                          int n_q, int Hq, int row0, float* __restrict__ o, float* __restrict__ lse,
                                                          int64_t lse_hs, bool accumulate) {
  constexpr int kRows = 8 / kGroups;                    // (row, head)s of a workgroup
  __shared__ float4 xs[8][32];
  __shared__ float ms[8], ts[8];
  const int c = threadIdx.x & 31, team = threadIdx.x >> 5, g = team % kGroups;
  const int64_t n = (int64_t)n_q * Hq, rh = (int64_t)blockIdx.x * kRows + team / kGroups;
  const bool live = rh < n;
  const int h = (int)(rh % Hq);
  const int64_t r = rh / Hq;
  float m = -INFINITY, tot = 0.f;
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
  if (live) {
    const float* pl = part_lse + (int64_t)h * n_q + r;
    const float4* po = reinterpret_cast<const float4*>(part_o) + rh * 32 + c;
    bool nan = false;
#pragma unroll 4
    for (int s = g; s < nsplit; s += kGroups) {
      const float L = pl[s * n];
      m = fmaxf(m, L);
      nan |= L != L;
    }
    const bool nothing = m == -INFINITY;
#pragma unroll 4
    for (int s = g; s < nsplit; s += kGroups) {
      const float w = nothing ? 1.f : __expf(pl[s * n] - m);   // nothing: the sum of zeros, or the NaN of 0 * inf in V
      const float4 y = po[s * n * 32];                   // an empty range has stored zeros
      tot += w;
      x.x += w * y.x; x.y += w * y.y; x.z += w * y.z; x.w += w * y.w;
    }
    if (nan) m = NAN;
  }
  xs[team][c] = x;
  if (c == 0) { ms[team] = m; ts[team] = tot; }
  __syncthreads();
  if (!live || g != 0) return;
  float4* op = reinterpret_cast<float4*>(o) + ((r + row0) * Hq + h) * 32 + c;
  float* lp = lse + (int64_t)h * lse_hs + r + row0;
  const float la = accumulate ? *lp : -INFINITY;         // all lanes of the 32 read it before lane 0 replaces it: they lie in one wavefront
  m = la;
  bool nan = false;
  for (int k = 0; k < kGroups; ++k) {
    const float L = ms[team + k];
    m = fmaxf(m, L);
    nan |= L != L;
  }
  if (nan) {                                             // as a workgroup that has all keys leaves such a row
    if (accumulate && la == -INFINITY) return;
    *op = make_float4(NAN, NAN, NAN, NAN);
    if (c == 0 && !accumulate) *lp = -INFINITY;
    return;
  }
  const bool nothing = m == -INFINITY;
  if (nothing && accumulate) return;                     // both empty: leave the running state
  tot = 0.f;
  x = make_float4(0.f, 0.f, 0.f, 0.f);
  if (accumulate) {
    const float w = __expf(la - m);                      // exp(-inf) = 0
    const float4 y = *op;
    tot = w;
    x.x = w * y.x; x.y = w * y.y; x.z = w * y.z; x.w = w * y.w;
  }
  for (int k = 0; k < kGroups; ++k) {
    const float w = nothing ? 1.f : __expf(ms[team + k] - m);
    const float4 y = xs[team + k][c];
    tot += w * ts[team + k];
    x.x += w * y.x; x.y += w * y.y; x.z += w * y.z; x.w += w * y.w;
  }
  const float inv = nothing ? 1.f : 1.f / tot;
  x.x *= inv; x.y *= inv; x.z *= inv; x.w *= inv;
  *op = x;
  if (c == 0) *lp = nothing ? -INFINITY : m + __logf(tot);
}

// dq[rows of the block] += sum of the partial results.  A launch of few rows has too few wavefronts to hide a load behind
// another one's, so the loads of a batch are all on their way before the first sum; the batches are powers of two, so that a small count waits no
// longer than it has to (28/4 heads, 16 x 32768: 30.1 us four at a time, 28.4 so; 16 x 32768 with documents of 60 to 300 rows, 13 ranges that
// hold little: 14.3 and 12.2; 16 x 1000: 13.5 and 13.7, with the last batch under conditions 13.9).
__global__ __launch_bounds__(256) void dq_combine_kernel(const float* __restrict__ part, int nsplit, int64_t n4, float* __restrict__ dq) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= n4) return;
  const float4* p = reinterpret_cast<const float4*>(part) + t;
  float4* out = reinterpret_cast<float4*>(dq) + t;
  float4 x = *out;
  int s0 = 0;
  auto add_up = [&](auto count) {                       // the next partial results, all on their way at once
    constexpr int n = decltype(count)::value;
    float4 y[n];
#pragma unroll
    for (int j = 0; j < n; ++j) y[j] = p[(s0 + j) * n4];
#pragma unroll
    for (int j = 0; j < n; ++j) { x.x += y[j].x; x.y += y[j].y; x.z += y[j].z; x.w += y[j].w; }
    s0 += n;
  };
  while (s0 + 16 <= nsplit) add_up(std::integral_constant<int, 16>());
  if (s0 + 8 <= nsplit) add_up(std::integral_constant<int, 8>());
  if (s0 + 4 <= nsplit) add_up(std::integral_constant<int, 4>());
  if (s0 + 2 <= nsplit) add_up(std::integral_constant<int, 2>());
  if (s0 < nsplit) add_up(std::integral_constant<int, 1>());
  *out = x;
}

}  // namespace

int cu_count() {
  static std::atomic<int> cu_of_device[64] = {};        // 0 = not asked yet; the count never changes for a device
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 64) n = cu_of_device[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    if (dev >= 0 && dev < 64) cu_of_device[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

// Mean length of the documents up to the block's last position: exact for a whole sequence, too short for its earlier
// parts (n_docs counts the later documents too).
double mean_document(const StepArgs& a) {
  return (double)std::max(0, std::max(a.q_pos0 + a.n_q, a.k_pos0 + a.n_k)) / a.n_docs;
}

// Whether workgroups may rank their tiles (heaviest_first).  Every workgroup pays for it, the more the more tiles there
// are, and what it saves at the end of a launch is about one tile's work, so it is done
//  * from 1.2 rounds of workgroups (within one all start together) to max_rounds (the ends of many average out);
//  * where the rows of an average document, times the heads that a tile takes, outweigh rounds x tiles.
// Packs of clips of 200..4700 / 300..2500 / 100..1200 / 60..300 tokens, time without ranking over time with it:
//   forward, 7/1   79 tiles (2.2 rounds)  1.19 1.12 1.11 0.95   200 tiles (5.5)  1.04 0.97 0.92 0.83
//   forward, 28/4  16 tiles (1.75)        0.97 1.17 1.06 0.93   80 tiles (8.8)   0.97 0.95 0.92 0.89
//   dK/dV, 28/4    160 tiles (2.5)        1.30 1.49 1.23 1.07   510 tiles (8)    1.00 0.95 0.95 0.90
//   dK/dV, 4/2     260 tiles (2)          1.21 1.38 1.06 0.80   510 tiles (4)    1.04 1.00 0.87 0.72
int32_t may_rank(const StepArgs& a, int n_tiles, int n_blocks, int heads_per_tile, int max_rounds) {
  if (a.cu == nullptr || a.n_docs < 2 || a.n_docs > kMaxLocalDocs || n_tiles < 3 || n_tiles > kMaxRanked) return 0;
  const double rounds = (double)n_blocks / cu_count();
  if (rounds < 1.2 || rounds > max_rounds) return 0;
  return heads_per_tile * mean_document(a) >= (heads_per_tile > 1 ? 200. : 400.) + rounds * n_tiles;
}

// How a grid smaller than the chip is spread over it: by workgroups of 4 instead of 8 wavefronts (twice as many, each with half of
// the rows and the SIMDs to itself: 64 keys take 0.89 us instead of 1.2 in the forward, 1.15 instead of 1.6 in the dQ kernel) and by
// cutting the keys into ranges.  Taken is what minimises an estimate in us of the launch and of the combining pass (a launch, and every
// partial result written and read at about 4 TB/s).  A workgroup takes its tiles' time and the time to load Q and the first tiles and to store its result.  The
// launch lasts as long as its first, heaviest workgroup, or as the sum over all CUs and the part of a last round that stays empty, filled with its
// lightest: whole rounds where all rows see the same keys, nothing where the first see none.  Measured, 32 rows of 28/4 heads
// on 8192 keys, uncut: 162 us with 8 wavefronts, 122 with 4.  7/1 heads, 4961 x 4961 causal, 8 wavefronts: 103.8 us uncut (136 workgroups), 73.3
// in three ranges, which whole rounds of the heaviest took for slower; over 8302 forward and dQ blocks without documents of 24 to 8192 rows the
// choice takes 1.8 % longer than the best one measured in the mean, 4.0 with whole rounds.
// With a few documents the same holds (7/1 heads, 5651 x 5651, documents of 5000 and 651: 117.9 us uncut, 82.4 in three ranges; of 6457 forward blocks 508 are more than 3 %
// faster for it, 36 slower); many end one another's tiles at random, and a cut between short ones costs (8/8 heads, 5553 x 5553, 28 documents, dQ: 27 and 35 us).
// Documents shorten the visible keys by an amount the host does not know; taken are `mean_documents` documents
// of the mean length (the block's last position / n_docs), see the callers.  A cut that the documents leave with empty ranges
// costs 5 to 10 us; half of all keys, whatever n_docs, was such a cut for every block of short documents (100 rows on
// 8192 keys, 28/4 heads, documents of 60..300: forward 16 us uncut, 25 us cut, 14.6 us by this rule, which does not cut).
// At most bwd_dkdv_partial_bytes() are used, so that a workspace larger than asked for changes no result.
// Blocks so small that uncut tiles of 128 leave half of the CUs idle are cut into tiles of 64 to 8 rows, whose spare wavefronts help
// to move tiles: what a launch of one or two key tiles takes is the reading and writing of the rows of one workgroup.  28/4 heads,
// 48 x 48 causal, tiles of 128 / 32 / 8 rows: forward 8.3 / 7.8 / 7.4 us, merging 10.1 / 9.6 / 8.6, dQ 9.5 / 8.5 / 7.3 (fewer than 8 gain nothing
// more); 4/2 heads, 128 x 128: 9.3 / 8.7 / 8.2, 11.0 / 10.4 / 9.5, 10.7 / 9.6 / 8.3.
KeyRanges pick_key_ranges(const StepArgs& a, double tile_us, int64_t bytes_per_range, int64_t room, double mean_documents) {
  room = std::min(room, bwd_dkdv_partial_bytes());
  const double tile[2] = {tile_us, .73 * tile_us};
  constexpr double kStart[2] = {6., 5.}, kLaunch = 5., kBytesPerUs = 4.2e6;
  constexpr int kMaxRanges = 64;
  const int n_cu = cu_count();
  const int64_t rows = (int64_t)a.n_q * a.group;        // of one KV head
  const int64_t blocks[2] = {(rows + 255) / 256 * a.Hkv, (rows + 127) / 128 * a.Hkv};
  KeyRanges best = {8, 1, 256};
  if (blocks[0] >= n_cu || bytes_per_range <= 0) return best;
  int64_t keys = a.n_k;
  if (a.mask == 1) keys = std::max<int64_t>(0, std::min<int64_t>(keys, (int64_t)a.q_pos0 + a.n_q - a.k_pos0));
  if (a.cu != nullptr) keys = std::min(keys, (int64_t)(mean_documents * mean_document(a)));
  const double tiles = (double)((keys + 63) / 64);        // of the heaviest workgroup; of the lightest, and on average:
  double least = tiles, mean = tiles;
  if (a.mask == 1 && (a.cu == nullptr || a.n_docs <= 8)) {
    const int64_t first = (int64_t)a.q_pos0 + 1 - a.k_pos0, all = std::max<int64_t>(0, std::min<int64_t>(a.n_q, first + a.n_q - 1 - a.n_k));   // keys before the first row, rows behind all keys
    least = (double)((std::max<int64_t>(0, std::min(keys, first)) + 63) / 64);
    mean = tiles - (double)(a.n_q - all) / a.n_q * (tiles - least) / 2;
  }
  const int most = std::max(1, (int)std::min<int64_t>({kMaxRanges, room / bytes_per_range, (int64_t)(tiles / 4)}));
  double best_cost = 1e300;
  for (int w = 0; w < 2; ++w)
    for (int n = 1; n <= most; ++n) {
      auto us = [&](double t) { return t / n * tile[w] + kStart[w]; };
      const double rounds = (double)(blocks[w] * n) / n_cu, empty = (double)((blocks[w] * n + n_cu - 1) / n_cu) - rounds;
      const double cost = std::max(us(tiles), rounds * us(mean) + empty * us(least)) +
                          (n > 1 ? kLaunch + 2. * n * (double)bytes_per_range / kBytesPerUs : 0.);
      if (cost < best_cost) { best = {w ? 4 : 8, n, w ? 128 : 256}; best_cost = cost; }
    }
  if (best.waves == 4 && best.count == 1)
    while (best.rows > 8 && (rows + best.rows / 2 - 1) / (best.rows / 2) * a.Hkv <= n_cu) best.rows /= 2;
  return best;
}

hipError_t launch_fwd_combine(const StepArgs& a, const float* part_o, const float* part_lse, int nsplit, hipStream_t stream) {
  const int64_t n = (int64_t)a.n_q * a.Hq;
  if (nsplit >= 8)
    fwd_combine_kernel<8><<<dim3((unsigned)n), dim3(256), 0, stream>>>(part_o, part_lse, nsplit, a.n_q, a.Hq, a.q_row0, a.o, a.lse, a.lse_hs, a.accumulate);
  else
    fwd_combine_kernel<2><<<dim3((unsigned)((n + 3) / 4)), dim3(256), 0, stream>>>(part_o, part_lse, nsplit, a.n_q, a.Hq, a.q_row0, a.o, a.lse, a.lse_hs, a.accumulate);
  return hipGetLastError();
}

hipError_t launch_dq_combine(const StepArgs& a, const float* part, int nsplit, hipStream_t stream) {
  const int64_t n4 = (int64_t)a.n_q * a.Hq * 32;
  dq_combine_kernel<<<dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, stream>>>(part, nsplit, n4, a.dq + (int64_t)a.q_row0 * a.Hq * 128);
  return hipGetLastError();
}

}  // namespace mmsp
