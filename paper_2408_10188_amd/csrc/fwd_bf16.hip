// Forward ring step on bf16 matrix cores, head_dim 128.
//
// The query rows of the heads that share a KV head are one list of (row, head) pairs, head fastest: row i of the
// list is query row i / group of head i % group.  A workgroup owns up to kWaves * 32 rows of the list, a wavefront
// 32: their Q (MFMA B operands, 32 VGPRs), the O^T accumulator (128 d x 32 rows, 64 VGPRs) and the softmax statistics stay
// in registers for the whole call.  K and V tiles of 64 keys stream through two four-slot LDS rings
// filled by asynchronous global->LDS copies straight from the caller's tensors (one natural-orientation
// copy each; V is read back transposed by ds_read_b64_tr_b16).
//   S^T[key][row] = K . Q^T            (A = K tile from LDS, B = Q registers)
//   online softmax down the key axis, which is in-lane in S^T's register layout
//   O^T[d][row]  += V^T . P^T          (A = V tile read transposed, B = P^T straight from registers)
//
// One matrix instruction occupies a SIMD's matrix pipe for 32 cycles.  With two wavefronts on the SIMD four ordinary
// vector instructions fit beside it (measured: 34 cycles each with four, 40 with five; an exponential
// counts double), with one wavefront two (35; 26 + 4.2 n beyond).  The loop is therefore software-pipelined inside
// every wavefront: while the matrix pipe works on P.V of tile t-1 the vector units take the
// first half of the exponentials of tile t, and while it works on S of tile t+1 they take the
// second half.  The operand of every matrix instruction is read from LDS four instructions ahead, across
// phases and tiles: the workgroup's one barrier per tile stands in the middle of a phase, so that what is
// read ahead around it has landed before.  The interleaving is written out step by step (one matrix
// instruction per step) and pinned with empty asm statements and scheduling barriers.
// Tiles wholly outside every row's visible key interval are skipped; only tiles that cut an
// interval boundary (the causal diagonal, a document start) pay for masking.
#include <type_traits>

#include "mfma_tiles.h"

namespace mmsp {
namespace {

constexpr int kBN = 64;            // keys per tile

enum Result { kStore, kMerge, kPartial };

// n_items: work items per KV head, tiles of tile_rows <= kWaves * 32 rows of its list (x nsplit ranges of their keys).
// kPartial: nsplit workgroups share the key tiles of every query tile, each stores its (O, LSE) in
// part_o [nsplit][n_q][Hq][128] and part_lse [nsplit][Hq][n_q] for launch_fwd_combine.
template <int kWaves, Result kResult>
__global__ __launch_bounds__(512, 2) void fwd_bf16_kernel(StepArgs a, int n_items, int tile_rows, int xcd_bits, int nsplit, float* part_o,
                                                                           float* part_lse) {
  constexpr int kBM = 32 * kWaves;                      // most rows of a workgroup
  constexpr int kCopies = 16 / kWaves;
  constexpr int kDepth = 4;                              // LDS operand reads in flight
  // Tile t lives in slot (t - first) % 4 of its ring; slots are selected at compile time (the loop is unrolled four
  // tiles deep).  LDS map: the four V slots, then the four K slots.  An LDS instruction's immediate
  // offset reaches 64 KiB, so the K reads go through per-lane base registers that already hold the K
  // region's start (ka below) and no read needs an address addition of its own.
  constexpr int kKRegion = 4 * kTileGBytes;
  __shared__ __attribute__((aligned(1024))) char lds[8 * kTileGBytes];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);   // the same value in a scalar register (LDS targets of the copies)
  const int half = lane >> 5, col = lane & 31;

  // Workgroup -> (KV head, row tile).  Workgroups are dealt round-robin to the 8 XCDs; the
  // ones that land on the same XCD work on the same KV head so its K/V block stays in that
  // XCD's L2.  Later (heavier under the causal mask) tiles go first.
  int kvh = blockIdx.x, tile;
  if (xcd_bits >= 0) {                                  // 2^xcd_bits XCDs per KV head
    kvh = (blockIdx.x & 7) >> xcd_bits;
    tile = (blockIdx.x >> 3 << xcd_bits) + (blockIdx.x & ((1 << xcd_bits) - 1));
    if (tile >= n_items) return;
  } else {
    tile = blockIdx.x / a.Hkv;
    kvh = blockIdx.x - tile * a.Hkv;
  }
  tile = n_items - 1 - tile;
  int split = 0;
  if (kResult == kPartial) {                                       // an item is a range of a tile's keys
    const int item = tile;
    tile = item / nsplit;
    split = item - tile * nsplit;
  }
  const CuLocal cu = local_cu(a, reinterpret_cast<int32_t*>(lds + 8192), 64 * kWaves);
  if (a.rank) {                                         // n_items counts whole blocks of kBM query rows: `group` tiles each
    int block = tile / a.group;
    const int n_blocks = (a.n_q + kBM - 1) / kBM, sub = tile - block * a.group;
    if (worth_ranking(a, cu, a.q_pos0, a.q_pos0 + a.n_q - 1))
      block = heaviest_first(n_blocks - 1 - block, n_blocks, 64 * kWaves, reinterpret_cast<int*>(lds), [&](int i) { return key_tiles_of_rows(a, cu, i * kBM, kBM); });
    tile = block * a.group + sub;
  }
  const int n_rows = a.n_q * a.group, tile_row0 = tile * tile_rows;
  if (tile_row0 >= n_rows) return;
  const int row_end = min(tile_row0 + tile_rows, n_rows);
  const int row = tile_row0 + wave * 32 + col;          // this lane's row of the list
  const bool live = row < row_end;
  const int rowc = min(row, row_end - 1);
  const int q_row = row_of_pair(a, rowc), h = kvh * a.group + rowc - q_row * a.group;

  // visible key interval of this lane's row, and of the workgroup / wavefront extremes
  int lo, hi;
  key_interval_of_row(a, cu, q_row, lo, hi);
  int t_lo, t_hi, dummy;
  key_interval_of_row(a, cu, row_of_pair(a, tile_row0), t_lo, dummy);
  key_interval_of_row(a, cu, row_of_pair(a, row_end - 1), dummy, t_hi);
  // wavefront: smallest and largest lo and hi, those of its first and last row
  const int w_lo_min = __builtin_amdgcn_readlane(lo, 0), w_hi_min = __builtin_amdgcn_readlane(hi, 0);
  const int w_lo_max = __builtin_amdgcn_readlane(lo, 31), w_hi_max = __builtin_amdgcn_readlane(hi, 31);
  if (lo > hi) lo = hi = INT32_MAX;                      // a row that sees nothing: every key differs from lo by more than hi - lo
  if (cu.copied) __syncthreads();                        // the tile copies may overwrite cu_seqlens
  int kt0 = t_lo / kBN, kt1 = t_hi >= t_lo ? t_hi / kBN : kt0 - 1;   // inclusive tile range
  if (kResult == kPartial) {                                              // this workgroup's share of the tiles
    const int total = max(kt1 - kt0 + 1, 0), first = kt0;
    kt0 = first + (int)((int64_t)total * split / nsplit);
    kt1 = first + (int)((int64_t)total * (split + 1) / nsplit) - 1;
  }
  // wavefront-uniform values that divisions have left in vector registers
  kt0 = __builtin_amdgcn_readfirstlane(kt0);
  kt1 = __builtin_amdgcn_readfirstlane(kt1);
  kvh = __builtin_amdgcn_readfirstlane(kvh);
  // Iterations this wavefront has work in: from the one that computes S of its first tile to the one
  // that multiplies P of its last.  Outside them it only helps to move tiles, which leaves the SIMD
  // to the wavefront it shares it with (documents shorter than a tile's rows, rows past the end of the list).
  const bool w_any = w_lo_min <= w_hi_max && tile_row0 + wave_s * 32 < row_end;
  int t_first = w_any ? max(w_lo_min / kBN - 1, kt0) : 1 << 30, t_last = w_any ? w_hi_max / kBN + 1 : -1;
  // In vector registers on purpose: branches on them are then mask changes that the register allocator takes in its
  // stride, where the same branches as jumps make it spill the accumulators.
  asm volatile("" : "+v"(t_first), "+v"(t_last));

  // The loop takes four tiles per trip; the ones that are missing in the first trip are before the first tile.
  const bool any_tile = kt0 <= kt1;
  const int j0 = -(kt1 - kt0 + 1) & 3;                   // tile kt0 lives in slot j0, the last tile in slot 3

  // ---- asynchronous tile fetch ----
  const int64_t kv_off = ((int64_t)a.k_row0 * a.kv_ts + (int64_t)kvh * a.kv_hs) * 2;
  const char* const k_first = reinterpret_cast<const char*>(a.k) + kv_off;
  const char* const v_first = reinterpret_cast<const char*>(a.v) + kv_off;
  TileCopier<kCopies> copier;
  copier.init(lds, a.kv_ts, a.n_k, kt1, wave, lane);
  auto fetch = [&](const char* first, int t, int slot_offset) {
    const auto x = copier.tile(first, t);
#pragma unroll
    for (int i = 0; i < kCopies; ++i) copier.copy_to(x, i, slot_offset);
  };
  if (any_tile) {
    fetch(k_first, kt0, kKRegion + j0 * kTileGBytes);
    fetch(v_first, kt0, j0 * kTileGBytes);
    if (kt0 < kt1) fetch(k_first, kt0 + 1, kKRegion + ((j0 + 1) & 3) * kTileGBytes);
    // the first iteration multiplies an all-zero P with "the tile before the first": finite zeros
    for (int i = tid * 16; i < kTileGBytes; i += 64 * kWaves * 16) *reinterpret_cast<u32x4*>(lds + ((j0 + 3) & 3) * kTileGBytes + i) = mk4(0u, 0u, 0u, 0u);
  }

  // Q as B operands: k-step ks covers d = ks*16 .. +16, this lane holds 8 of them
  u32x4 qreg[8];
  {
    const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.q) + (int64_t)(a.q_row0 + q_row) * a.q_ts +
                         (int64_t)h * a.q_hs + half * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) qreg[i] = *reinterpret_cast<const u32x4*>(qp + i * 16);
  }
  // Wait for Q and the first tiles here, once.  Left to the compiler, the wait for the last of Q's loads would stand inside the
  // loop, where the same counter holds the tile copies that have just been issued.
#pragma unroll
  for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(qreg[i]));

  f32x16 oacc[4];
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
  // Softmax state.  m_ref is the raw-score reference the exponentials are taken against.  It
  // is the maximum of the first tile the row sees and moves only when a later tile's sum shows that
  // its maximum has grown by more than kLazy in the exponent, so the steady loop takes no maxima
  // and its exponentials need not wait for one.
  constexpr float kLazy = 8.f;
  constexpr float kSumLimit = 32.f * 256.f;              // 32 keys per lane and tile, 2^kLazy each
  float m_ref = -INFINITY;
  float neg_mc = 0.f;        // -m_ref * c  (0 while m_ref = -inf, so masked scores give exp2(-inf) = 0)
  float l = 0.f;             // this lane's share of the row sum (its 32 of every 64 keys)
  const float c = a.scale * kLog2e;
  const float lazy_raw = kLazy / c;

  // LDS read addresses inside a tile, fixed for the whole call; the K region's start is part of ka, kept opaque
  int ka[4], va[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    ka[i] = tile_g_nat(lane, i) + kKRegion;
    va[i] = tile_g_tr(lane, i);
    asm volatile("" : "+v"(ka[i]), "+v"(va[i]));
  }
  // operand of matrix instruction n (0..15) of S: k-step n / 2, keys (n & 1) * 32 .. +32;  of P.V: d block n & 3, keys (n >> 2) * 16 .. +16
  auto read_k = [&](int n, int slot) {
    return *reinterpret_cast<const u32x4*>(lds + ka[n >> 2] + (slot * kTileGBytes + ((n >> 1) & 1) * 32 + (n & 1) * kTileGRows32));
  };
  auto read_v = [&](int n, int slot) {
    const char* p = lds + va[n & 3] + (slot * kTileGBytes + (n >> 2) * kTileGRows16);
    const u32x2 v0 = lds_read_tr(p), v1 = lds_read_tr(p + kTileGRows8);
    return mk4(v0.x, v0.y, v1.x, v1.y);
  };

  f32x16 s[2][2];            // S^T of the tile whose softmax is being taken and of the next one (by the parity of the slot): two 32-key blocks
  u32x4 pb[4];               // P^T of the previous tile, packed as the B operands of its four k-steps
#pragma unroll
  for (int g = 0; g < 4; ++g) pb[g] = mk4(0u, 0u, 0u, 0u);
  u32x4 op[kDepth];          // operands of the next matrix instructions

  auto apply_mask = [&](f32x16 (&x)[2], int k0) {
    const int from_lo = k0 + half * 4 - lo;
    const uint32_t range = (uint32_t)(hi - lo);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if ((uint32_t)(from_lo + (kb * 32 + (i >> 2) * 8 + (i & 3))) > range) x[kb][i] = -INFINITY;
  };
  auto row_maximum = [&](const f32x16 (&x)[2]) {        // of the tile's scores, over both lanes of a row
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, x[kb][i]);
    return fmaxf(mx, __shfl_xor(mx, 32));
  };

#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int i = 0; i < 16; ++i) s[0][kb][i] = 0.f;
  if (any_tile) {
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0), lgkmcnt(0): the first tiles have landed, the zeros are written
    lds_barrier();
    if (kt0 + 2 <= kt1) fetch(k_first, kt0 + 2, kKRegion + ((j0 + 2) & 3) * kTileGBytes);
    if (kt0 + 1 <= kt1) fetch(v_first, kt0 + 1, ((j0 + 1) & 3) * kTileGBytes);
    if (kt0 + 3 <= kt1) fetch(k_first, kt0 + 3, kKRegion + ((j0 + 3) & 3) * kTileGBytes);
    u32x4 first[16];                                    // all operands at once: nothing else needs registers yet
#pragma unroll
    for (int n = 0; n < 16; ++n) first[n] = read_k(n, j0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 0; n < 16; ++n) s[0][n & 1] = mfma32(first[n], qreg[n >> 1], s[0][n & 1]);
    // The first tile's maximum is the reference of the rows that see it.  Left to the loop, it costs a second round of
    // exponentials (28/4 heads, 256 x 64: 12.7 us against 12.1, 2048 x 192: 18.8 against 18.2; a maximum in every
    // iteration took 12.3 and 18.4).
    const int k0 = kt0 * kBN;
    if (k0 < w_lo_max || k0 + kBN - 1 > w_hi_min) apply_mask(s[0], k0);
    m_ref = row_maximum(s[0]);
    if (m_ref != -INFINITY) neg_mc = -m_ref * c;
  }
  s[1][0] = s[0][0];
  s[1][1] = s[0][1];

  // One iteration: tile t in slot k, its scores in s[k & 1].  V(t-1) and K(t+1) are in the slots before and after.
  auto iteration = [&](auto slot_constant, int t) {
    constexpr int k = decltype(slot_constant)::value;
    constexpr int kPrev = (k + 3) & 3, kNext = (k + 1) & 3, kAfter = (k + 2) & 3;
    f32x16 (&sc)[2] = s[k & 1], (&sn)[2] = s[(k + 1) & 1];
    if (t < kt0) return;                                // before the first tile
    // Own copies of every group but the newest have landed: K(t+1) and K(t+2), V(t); after the barrier everybody's have,
    // and everybody is done with K(t) and V(t-2), whose slots are refilled with K(t+4) and V(t+2).  Every iteration issues one
    // whole group (past the end it fetches the last tile again, into slots nobody reads any
    // more), so the wait is the same constant everywhere.
    auto hand_over = [&]() {
      __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * kCopies));
      lds_barrier();
    };
    if (t < t_first || t > t_last) {
      hand_over();
      fetch(v_first, t + 2, kAfter * kTileGBytes);
      fetch(k_first, t + 4, kKRegion + k * kTileGBytes);
      return;
    }

    const int k0 = t * kBN;
    if (t == t_first) {
#pragma unroll
      for (int n = 0; n < kDepth; ++n) op[n] = read_v(n, kPrev);
    }
    // ---- mask (only tiles that cut an interval boundary; the first has its mask already) ----
    if (t != kt0 && (k0 < w_lo_max || k0 + kBN - 1 > w_hi_min)) apply_mask(sc, k0);
    __builtin_amdgcn_sched_barrier(0);

    // Each step below is one MFMA with the reads that feed the MFMA four steps later and its share
    // of the vector work; MMSP_STEP_END pins the values so that neither the optimiser nor the
    // instruction scheduler moves work from one step to another.
#define MMSP_PIN(x) asm volatile("" : "+v"(x))
#define MMSP_STEP_END() __builtin_amdgcn_sched_barrier(0)

    // ================= phase 1: O^T += V(t-1)^T P(t-1)^T  beside the first half of the exponentials of tile t =================
    // (the first iteration multiplies an all-zero P with a slot of zeros)
    uint32_t w[16];          // P^T of tile t, two keys per word
    float ps[4];             // fp32 sums of the unrounded P (LSE needs 1e-3)
    auto exp_item = [&](int j) {                        // keys 2j, 2j+1 of the lane's 32
      const f32x16& sv = sc[j >> 3];
      const int e = (j & 7) * 2;
      const float p0 = __builtin_amdgcn_exp2f(fmaf(sv[e], c, neg_mc));
      const float p1 = __builtin_amdgcn_exp2f(fmaf(sv[e + 1], c, neg_mc));
      ps[e & 3] = j < 2 ? p0 : ps[e & 3] + p0;
      ps[(e + 1) & 3] = j < 2 ? p1 : ps[(e + 1) & 3] + p1;
      w[j] = pack2(p0, p1);
      MMSP_PIN(ps[e & 3]); MMSP_PIN(ps[(e + 1) & 3]); MMSP_PIN(w[j]);
    };
    // The iteration's copies, spread over the steps after the hand-over: issued in a row, right behind the barrier and by all
    // wavefronts at once, they hold up each other and the matrix instructions behind them (4096 x 8192 rows, 28/4 heads: 407 against 396 thousand cycles).
    const auto v_next = copier.tile(v_first, t + 2), k_next = copier.tile(k_first, t + 4);
    auto copy_beside = [&](int step) {
      constexpr int kFirst = 9, kEvery = 24 / (2 * kCopies);
      if (step < kFirst || (step - kFirst) % kEvery != 0) return;
      const int n = (step - kFirst) / kEvery;
      if (n < kCopies) copier.copy(v_next, n, kAfter * kTileGBytes);
      else copier.copy(k_next, n - kCopies, kKRegion + k * kTileGBytes);
    };
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int db = i & 3;
      if (i == 7) hand_over();                          // K(t+1) is read from step 16 - kDepth on
      oacc[db] = mfma32(op[i % kDepth], pb[i >> 2], oacc[db]);
      op[i % kDepth] = i + kDepth < 16 ? read_v(i + kDepth, kPrev) : read_k(i + kDepth - 16, kNext);
      copy_beside(i);
      if (i & 1) exp_item(i >> 1);                      // exponentials of keys 0..15 of the lane
      MMSP_PIN(oacc[db]);
      MMSP_STEP_END();
    }

    // ================= phase 2: S^T of tile t+1  beside  the remaining exponentials of tile t =================
    // (after the last tile the product runs on whatever the slot holds and is never used)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int kb = i & 1;
      if (i < 2) {
#pragma unroll
        for (int e = 0; e < 16; ++e) sn[kb][e] = 0.f;
      }
      sn[kb] = mfma32(op[i % kDepth], qreg[i >> 1], sn[kb]);
      op[i % kDepth] = i + kDepth < 16 ? read_k(i + kDepth, kNext) : read_v(i + kDepth - 16, k);
      copy_beside(16 + i);
      if ((i & 1) == 0) exp_item(8 + (i >> 1));
      MMSP_PIN(sn[kb]);
      MMSP_STEP_END();
    }
    float tile_sum = (ps[0] + ps[1]) + (ps[2] + ps[3]);  // this lane's share of the tile's row sum
    MMSP_STEP_END();
    // ---- the reference (rare: the first tile a row sees if that is not the workgroup's, later ones whose maximum outgrew it) ----
    // A score above m_ref by more than kLazy in the exponent shows in the lane's sum of 32 terms:
    // while the sum is below 32 * 2^kLazy no P exceeds that, so neither P (bf16 has float's range)
    // nor the sums lose anything, and the maximum itself is never needed.  Otherwise the reference
    // moves to the tile's maximum and the tile's exponentials, whose scores are still here, are
    // taken again.  Both lanes of a row (its two halves of the keys) decide alike.
    if (__any(tile_sum > kSumLimit || (m_ref == -INFINITY && lo < k0 + kBN && hi >= k0))) {
      const float mx = row_maximum(sc);
      const bool moved = mx > m_ref + lazy_raw;
      const float m_new = moved ? mx : m_ref;
      const float alpha = moved ? __builtin_amdgcn_exp2f((m_ref - m_new) * c) : 1.f;   // m_ref = -inf -> 0
      m_ref = m_new;
      neg_mc = m_new == -INFINITY ? 0.f : -m_new * c;
      l *= alpha;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[db][i] *= alpha;
#pragma unroll
      for (int j = 0; j < 16; ++j) exp_item(j);
      tile_sum = (ps[0] + ps[1]) + (ps[2] + ps[3]);
    }
    l += tile_sum;
    MMSP_STEP_END();
#pragma unroll
    for (int g = 0; g < 4; ++g) pb[g] = mk4(w[4 * g], w[4 * g + 1], w[4 * g + 2], w[4 * g + 3]);
  };
#undef MMSP_PIN
#undef MMSP_STEP_END

  for (int t = kt0 - j0; t <= kt1; t += 4) {
    iteration(std::integral_constant<int, 0>(), t);
    iteration(std::integral_constant<int, 1>(), t + 1);
    iteration(std::integral_constant<int, 2>(), t + 2);
    iteration(std::integral_constant<int, 3>(), t + 3);
  }

  // Where the results go, and for a merge the running ones.  They are read here, beside the last product and the drain of the copies:
  // a launch of few tiles has nothing later to hide their latency (28/4 heads, 64 x 64: 10.2 us read behind the barrier, 9.4 here).
  float* const out = kResult == kPartial ? part_o + (int64_t)split * a.n_q * a.Hq * 128 : a.o + (int64_t)a.q_row0 * a.Hq * 128;
  auto result_at = [&](int list_row) {                   // where this lane's 16 bytes of a row of the list go
    return reinterpret_cast<float4*>(out + ((int64_t)row_of_pair(a, list_row) * (a.Hq - a.group) + kvh * a.group + list_row) * 128) + col;
  };
  const int row_up = tile_row0 + wave * 32 + half;       // this half of the wavefront takes every other row from here on
  float* const lp = kResult == kPartial ? part_lse + ((int64_t)split * a.Hq + h) * a.n_q + q_row : a.lse + (int64_t)h * a.lse_hs + a.q_row0 + q_row;
  float la = -INFINITY;
  float4 old[16];
  if (kResult == kMerge) {
    if (live) la = *lp;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (row_up + 2 * i < row_end) old[i] = *result_at(row_up + 2 * i);
  }
  __builtin_amdgcn_sched_barrier(0);

  if (any_tile) {            // O^T += V^T P^T of the last tile
    if (t_first <= kt1 && t_last >= kt1) {
#pragma unroll
      for (int n = 0; n < 16; ++n) {
        oacc[n & 3] = mfma32(op[n % kDepth], pb[n >> 2], oacc[n & 3]);
        if (n + kDepth < 16) op[n % kDepth] = read_v(n + kDepth, 3);
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);                   // the copies issued past the end have landed, everybody is done with the tiles:
  lds_barrier();                                        // the result can pass through LDS
  const float m = m_ref;

  // ---- epilogue ----
  l += __shfl_xor(l, 32);
  const bool empty = !(l > 0.f);
  const float inv = empty ? 0.f : 1.f / l;
  // A row of NaNs reports LSE = -inf, a range's share of one NaN: the combining pass has to tell it from an empty range.
  const float lse_part = (kResult == kPartial ? l == 0.f : empty) ? -INFINITY : (m * c + __builtin_amdgcn_logf(l)) * kLn2;   // v_log_f32 is log2
  float wa = 0.f, wb = inv;
  constexpr float kSkip = -1.f;                          // in the place of a weight, which is never negative: leave the row alone
  if (live) {
    float lse_new = lse_part;
    if (kResult == kMerge) {
      const float mm = fmaxf(la, lse_part);
      const float ea = __expf(la - mm), eb = __expf(lse_part - mm);
      const float tot = ea + eb;
      wa = mm == -INFINITY ? kSkip : ea / tot;          // both sides empty: the running result stays
      wb = eb / tot * inv;
      lse_new = mm + __logf(tot);
    }
    if (half == 0 && wa != kSkip) *lp = lse_new;
  }
  float* const weights = reinterpret_cast<float*>(lds + kWaves * kResultBytes) + wave * 32;
  if (kResult == kMerge && half == 0) weights[col] = wa;
  char* const area = lds + wave * kResultBytes;
  result_to_lds(area, oacc, wb, half, col);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int rr = 2 * i + half;
    float4 o = result_chunk(area, rr, col);
    bool on = row_up + 2 * i < row_end;
    if (kResult == kMerge) {
      const float w = weights[rr];
      on = on && w != kSkip;
      o.x += w * old[i].x; o.y += w * old[i].y; o.z += w * old[i].z; o.w += w * old[i].w;
    }
    if (on) *result_at(row_up + 2 * i) = o;
  }
}

}  // namespace

namespace {

template <int kWaves>
hipError_t launch(StepArgs a, const KeyRanges& r, hipStream_t stream) {
  constexpr int kBM = 32 * kWaves;
  const int n_blocks_q = (a.n_q + kBM - 1) / kBM, nsplit = r.count;
  a.rank = may_rank(a, n_blocks_q, n_blocks_q * nsplit * a.Hq, 1, 5);
  const int rows = a.rank ? kBM : r.rows;
  const int n_items = (a.rank ? n_blocks_q * a.group : (int)(((int64_t)a.n_q * a.group + rows - 1) / rows)) * nsplit;
  int xcd_bits = -1, n_blocks = n_items * a.Hkv;
  if (8 % a.Hkv == 0) {
    xcd_bits = __builtin_ctz(8 / a.Hkv);
    n_blocks = 8 * ((n_items + (1 << xcd_bits) - 1) >> xcd_bits);
  }
  const dim3 g(n_blocks), b(64 * kWaves);
  if (nsplit > 1) {
    float* part_o = reinterpret_cast<float*>(a.ws);
    float* part_lse = part_o + (int64_t)nsplit * a.n_q * a.Hq * 128;
    fwd_bf16_kernel<kWaves, kPartial><<<g, b, 0, stream>>>(a, n_items, rows, xcd_bits, nsplit, part_o, part_lse);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_fwd_combine(a, part_o, part_lse, nsplit, stream);
  }
  if (a.accumulate) fwd_bf16_kernel<kWaves, kMerge><<<g, b, 0, stream>>>(a, n_items, rows, xcd_bits, 1, nullptr, nullptr);
  else fwd_bf16_kernel<kWaves, kStore><<<g, b, 0, stream>>>(a, n_items, rows, xcd_bits, 1, nullptr, nullptr);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fwd_bf16(const StepArgs& a, hipStream_t stream) {
  const int n_blocks_q = (a.n_q + 255) / 256;
  // The slowest query tile counts: one tile lies anywhere in a document, of eight one lies late in a long one.
  const double mean_documents = 1. + (n_blocks_q < 8 ? n_blocks_q - 1 : 7) / 7.;
  const KeyRanges r = pick_key_ranges(a, 1.2, (int64_t)a.n_q * a.Hq * 129 * sizeof(float), a.ws_bytes, mean_documents);
  return r.waves == 4 ? launch<4>(a, r, stream) : launch<8>(a, r, stream);
}

}  // namespace mmsp
