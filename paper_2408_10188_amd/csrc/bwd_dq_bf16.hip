// Backward ring step, dQ kernel (query-stationary) on bf16 matrix cores, head_dim 128.
//
// Same skeleton as the forward kernel: the query rows of the heads that share a KV head are one list of (row, head)
// pairs, a workgroup owns up to kWaves * 32 of them, a wavefront 32: their Q and dO (MFMA
// B operands), the dQ^T accumulator (128 d x 32 rows) and the two row statistics (-LSE*log2e,
// delta) stay in registers for the whole call.  64-key tiles of K and V stream through two four-slot
// LDS rings filled by asynchronous global->LDS copies straight from the caller's tensors (natural
// orientation; the third product reads K back transposed with ds_read_b64_tr_b16).
//   S^T[key][row]  = K . Q^T            P^T = exp2(S^T * c - LSE*log2e)   (final LSE: no running max)
//   dP^T[key][row] = V . dO^T           dS^T = P^T * (dP^T - delta)
//   dQ^T[d][row]  += K^T . dS^T         (B operand = dS^T straight from registers)
// S and dP are recomputed here although the dK/dV kernel computes them too: that buys exclusive
// ownership of dQ, hence no floating-point atomics and bit-reproducible results.
//
// The loop is software-pipelined over blocks of 32 keys: while the matrix pipe computes S and dP of the next block
// (phase A, 16 instructions) the vector units turn those of this block into dS, which phase B (8 instructions) multiplies
// with K^T.  The operand of every matrix instruction is read from LDS four instructions ahead, across
// phases and tiles; the workgroup's one barrier per tile stands in the middle of a phase.
#include <type_traits>

#include "mfma_tiles.h"

namespace mmsp {
namespace {

constexpr int kBN = 64;            // keys per tile

// n_items: work items per KV head, tiles of tile_rows <= kWaves * 32 rows of its list (x nsplit ranges of their keys).
// kPartial: nsplit workgroups share the key tiles of every row tile, each stores its share of dQ in
// part [nsplit][n_q][Hq][128] for launch_dq_combine.
// The launch bound of 512 holds for four wavefronts too: with fewer the compiler would use the accumulation registers
// that a lone wavefront per SIMD has, and copy every S and dP out of them.
template <int kWaves, bool kPartial>
__global__ __launch_bounds__(512, 2) void bwd_dq_bf16_kernel(StepArgs a, int n_items, int tile_rows, int xcd_bits, int nsplit, float* part,
                                                             BwdWorkspace stats) {
  constexpr int kBM = 32 * kWaves;                      // most rows of a workgroup
  constexpr int kCopies = 16 / kWaves;
  constexpr int kDepth = 4;                              // LDS operand reads in flight
  // LDS map: the four K slots, then the four V slots; slots are selected at compile time (the loop is unrolled four tiles
  // deep).  An LDS instruction's immediate offset reaches 64 KiB, so the V reads go through per-lane base registers that
  // already hold the V region's start (va below).
  constexpr int kVRegion = 4 * kTileGBytes;
  __shared__ __attribute__((aligned(1024))) char lds[8 * kTileGBytes];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, col = lane & 31;

  // workgroup -> (KV head, row tile): the workgroups of a KV head share an XCD, later (heavier
  // under the causal mask) tiles first
  int kvh, tile;
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
  if (kPartial) {                                       // an item is a range of a tile's keys
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
    tile = __builtin_amdgcn_readfirstlane(block * a.group + sub);
  }
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int n_rows = a.n_q * a.group, tile_row0 = tile * tile_rows;
  if (tile_row0 >= n_rows) return;
  const int row_end = min(tile_row0 + tile_rows, n_rows);
  const int row = tile_row0 + wave * 32 + col;          // this lane's row of the list
  const bool live = row < row_end;
  const int rowc = min(row, row_end - 1);
  const int q_row = row_of_pair(a, rowc), h = kvh * a.group + rowc - q_row * a.group;

  int lo, hi;
  key_interval_of_row(a, cu, q_row, lo, hi);
  int t_lo, t_hi, dummy;
  key_interval_of_row(a, cu, row_of_pair(a, tile_row0), t_lo, dummy);
  key_interval_of_row(a, cu, row_of_pair(a, row_end - 1), dummy, t_hi);
  // wavefront: smallest and largest lo and hi, those of its first and last row
  const int w_lo_min = __builtin_amdgcn_readlane(lo, 0), w_hi_min = __builtin_amdgcn_readlane(hi, 0);
  const int w_lo_max = __builtin_amdgcn_readlane(lo, 31), w_hi_max = __builtin_amdgcn_readlane(hi, 31);
  if (lo > hi) lo = hi = INT32_MAX;                      // a row that sees nothing: every key differs from lo by more than hi - lo
  const int lane_lo = lo - half * 4;                     // this lane's keys are 4 half + 0..3 of every 8
  const uint32_t range = (uint32_t)(hi - lo);
  if (cu.copied) __syncthreads();                        // the tile copies may overwrite cu_seqlens
  int kt0 = t_lo / kBN, kt1 = t_hi >= t_lo ? t_hi / kBN : kt0 - 1;   // inclusive tile range
  if (kPartial) {                                              // this workgroup's share of the tiles
    const int total = max(kt1 - kt0 + 1, 0), first = kt0;
    kt0 = first + (int)((int64_t)total * split / nsplit);
    kt1 = first + (int)((int64_t)total * (split + 1) / nsplit) - 1;
  }
  // wavefront-uniform values that divisions have left in vector registers
  kt0 = __builtin_amdgcn_readfirstlane(kt0);
  kt1 = __builtin_amdgcn_readfirstlane(kt1);
  kvh = __builtin_amdgcn_readfirstlane(kvh);
  // Tiles that one of this wavefront's rows sees.  Outside them it only helps to move tiles, which leaves the SIMD
  // to the wavefront it shares it with (documents shorter than a tile's rows, rows past the end of the list).
  const bool w_any = w_lo_min <= w_hi_max && tile_row0 + wave * 32 < row_end;
  const int t_last = w_hi_max / kBN;
  int t_first = w_any ? max(w_lo_min / kBN, kt0) : 1 << 30;
  const uint32_t t_span = w_any && t_last > t_first ? t_last - t_first : 0;
  if (t_last < t_first) t_first = 1 << 30;               // nothing in this workgroup's range
  // In a vector register on purpose: branches on it are then mask changes that the register allocator takes in its
  // stride, where the same branches as jumps make it spill the accumulators.
  asm volatile("" : "+v"(t_first));

  // The loop takes four tiles per trip; the ones that are missing in the first trip are before the first tile.
  const bool any_tile = kt0 <= kt1;
  const int j0 = -(kt1 - kt0 + 1) & 3;                   // tile kt0 lives in slot j0, the last tile in slot 3

  // ---- asynchronous tile fetch ----
  const int64_t kv_off = ((int64_t)a.k_row0 * a.kv_ts + (int64_t)kvh * a.kv_hs) * 2;
  const char* const k_first = reinterpret_cast<const char*>(a.k) + kv_off;
  const char* const v_first = reinterpret_cast<const char*>(a.v) + kv_off;
  TileCopier<kCopies> copier;
  copier.init(lds, a.kv_ts, a.n_k, kt1, wave, lane);
  auto fetch = [&](int t, int slot) {
    const auto k = copier.tile(k_first, t), v = copier.tile(v_first, t);
#pragma unroll
    for (int i = 0; i < kCopies; ++i) copier.copy_to(k, i, slot * kTileGBytes);
#pragma unroll
    for (int i = 0; i < kCopies; ++i) copier.copy_to(v, i, kVRegion + slot * kTileGBytes);
  };
  if (any_tile) {
    fetch(kt0, j0);
    if (kt0 < kt1) fetch(kt0 + 1, (j0 + 1) & 3);
  }

  // Q and dO as B operands: k-step ks covers d = ks*16 .. +16, this lane holds 8 of them
  const int64_t r = a.q_row0 + q_row;
  u32x4 qreg[8], doreg[8];
  {
    const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.q) + r * a.q_ts + (int64_t)h * a.q_hs + half * 8;
    const uint16_t* dp = reinterpret_cast<const uint16_t*>(a.d_o) + (r * a.Hq + h) * 128 + half * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      qreg[ks] = *reinterpret_cast<const u32x4*>(qp + ks * 16);
      doreg[ks] = *reinterpret_cast<const u32x4*>(dp + ks * 16);
    }
  }
  const float L = a.lse_final[(int64_t)h * a.lse_hs + r];
  const float Dl = a.delta[(int64_t)h * a.lse_hs + r];
  // Wait for these loads here, once.  Left to the compiler, the wait for the last of them stands at their use inside the loop,
  // where the same counter holds the tile copies that have just been issued.
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) asm volatile("" : "+v"(qreg[ks]), "+v"(doreg[ks]));
  float neg_l2 = L == -INFINITY ? -INFINITY : -L * kLog2e;   // a row that saw nothing: P = 0
  const float c = a.scale * kLog2e;
  // Row statistics for the dK/dV kernel that follows; rows up to the next whole 64 count as rows that saw nothing.
  if (stats.nl2 != nullptr && split == 0) {
    const int padded = stats.n_qtiles * 64;
    if (live && half == 0) {
      stats.nl2[(int64_t)h * padded + q_row] = neg_l2;
      stats.ndl[(int64_t)h * padded + q_row] = -Dl;
    }
    if (row_end == n_rows) {                            // the padding of every head of the group: the last tile's workgroup
      for (int i = tid; i < (padded - a.n_q) * a.group; i += 64 * kWaves) {
        const int pad = row_of_pair(a, i);
        const int64_t at = (int64_t)(kvh * a.group + i - pad * a.group) * padded + a.n_q + pad;
        stats.nl2[at] = -INFINITY;
        stats.ndl[at] = 0.f;
      }
    }
  }

  // dP's accumulator starts from -delta (one value per lane: a lane holds one row), so dP - delta
  // needs no subtraction: 32 vector instructions a tile.
  f32x16 ndl;
#pragma unroll
  for (int i = 0; i < 16; ++i) ndl[i] = -Dl;
  asm volatile("" : "+v"(ndl), "+v"(neg_l2));

  f32x16 dq[4];
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) dq[db][i] = 0.f;

  // LDS read addresses inside a tile, fixed for the whole call; the V region's start is part of va, kept opaque
  int ka[4], va[4], ta[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    ka[i] = tile_g_nat(lane, i);
    va[i] = ka[i] + kVRegion;
    ta[i] = tile_g_tr(lane, i);
    asm volatile("" : "+v"(ka[i]), "+v"(va[i]), "+v"(ta[i]));
  }
  // operand i (0..15) of S (even, K) and dP (odd, V) of the 32 keys from row 32 blk of a slot's tile
  auto read_nat = [&](int i, int blk, int slot) {
    const int at = slot * kTileGBytes + ((i >> 1) & 1) * 32 + blk * kTileGRows32;
    return *reinterpret_cast<const u32x4*>(lds + ((i & 1) ? va[i >> 2] : ka[i >> 2]) + at);
  };
  // operand i (0..7) of dQ: d block i & 3, keys 16 (i >> 2) .. +16 of the block
  auto read_tr = [&](int i, int blk, int slot) {
    const char* p = lds + ta[i & 3] + (slot * kTileGBytes + (blk * 2 + (i >> 2)) * kTileGRows16);
    const u32x2 v0 = lds_read_tr(p), v1 = lds_read_tr(p + kTileGRows8);
    return mk4(v0.x, v0.y, v1.x, v1.y);
  };

  f32x16 s[2], dp[2];        // S and dP - delta of the tile's two blocks (the second one's, later the next tile's first, in progress)
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) { s[b][i] = 0.f; dp[b][i] = 0.f; }
  u32x4 op[kDepth];          // operands of the next matrix instructions

  if (any_tile) {
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0), lgkmcnt(0): the first two tiles have landed
    lds_barrier();
    if (kt0 + 2 <= kt1) fetch(kt0 + 2, (j0 + 2) & 3);
  }

  auto iteration = [&](auto slot_constant, int t) {
    constexpr int k = decltype(slot_constant)::value;
    constexpr int kNext = (k + 1) & 3, kRefill = (k + 3) & 3;
    if (t < kt0) return;                                // before the first tile
    // Own copies of every group but the newest have landed: tile t+1; after the barrier everybody's have,
    // and everybody is done with tile t-1, whose slot is refilled with tile t+3.  Every iteration issues one
    // whole group (past the end it fetches the last tile again, into a slot nobody reads any
    // more), so the wait is the same constant everywhere.
    auto hand_over = [&]() {
      __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * kCopies));
      lds_barrier();
    };
    int first = t_first;
    asm volatile("" : "+v"(first));                     // or the compiler keeps t - t_first of every slot in a register of its own
    if ((uint32_t)(t - first) > t_span) {
      hand_over();
      fetch(t + 3, kRefill);
      return;
    }
#define MMSP_PIN(x) asm volatile("" : "+v"(x))
#define MMSP_STEP_END() __builtin_amdgcn_sched_barrier(0)
    // operand n of the iteration's 48 matrix instructions (48 .. : the next iteration's first)
    auto operand = [&](int n) {
      if (n >= 48) return read_nat(n - 48, 1, kNext);
      if (n < 16) return read_nat(n, 1, k);
      if (n < 24) return read_tr(n - 16, 0, k);
      if (n < 40) return read_nat(n - 24, 0, kNext);
      return read_tr(n - 40, 1, k);
    };
    const int k0 = t * kBN;
    if (t == first) {                                   // S and dP of the first block a row of the wavefront may see
      u32x4 next[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) next[i] = read_nat(i, 0, k);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const u32x4 o = next[i & 7];
        if (i + 8 < 16) next[i & 7] = read_nat(i + 8, 0, k);
        if (i == 0) {
#pragma unroll
          for (int e = 0; e < 16; ++e) s[0][e] = 0.f;
        }
        if ((i & 1) == 0) s[0] = mfma32(o, qreg[i >> 1], s[0]);
        else dp[0] = mfma32(o, doreg[i >> 1], i == 1 ? ndl : dp[0]);
        MMSP_STEP_END();
      }
#pragma unroll
      for (int n = 0; n < kDepth; ++n) op[n] = operand(n);
    }
    MMSP_STEP_END();
    // The iteration's copies, spread over the steps after the hand-over.
    const auto k_next = copier.tile(k_first, t + 3), v_next = copier.tile(v_first, t + 3);
    auto copy_beside = [&](int step) {
      constexpr int kFirst = 9, kEvery = 36 / (2 * kCopies);
      if (step < kFirst || (step - kFirst) % kEvery != 0) return;
      const int n = (step - kFirst) / kEvery;
      if (n < kCopies) copier.copy(k_next, n, kRefill * kTileGBytes);
      else if (n < 2 * kCopies) copier.copy(v_next, n - kCopies, kVRegion + kRefill * kTileGBytes);
    };

#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      f32x16 &sc = s[blk], &dc = dp[blk], &sn = s[blk ^ 1], &dn = dp[blk ^ 1];
      const int b0 = k0 + blk * 32;                     // first key of the block
      if (b0 < w_lo_max || b0 + 31 > w_hi_min) {
        const int from_lo = b0 - lane_lo;
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if ((uint32_t)(from_lo + ((i >> 2) * 8 + (i & 3))) > range) sc[i] = -INFINITY;
      }
      MMSP_STEP_END();
      // ---- phase A: S, dP - delta of the following block beside dS of this one ----
      uint32_t w[8];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int n = blk * 24 + i;
        if (n == 7) hand_over();
        if (i == 0) {
#pragma unroll
          for (int e = 0; e < 16; ++e) sn[e] = 0.f;
        }
        if ((i & 1) == 0) { sn = mfma32(op[n % kDepth], qreg[i >> 1], sn); }
        else { dn = mfma32(op[n % kDepth], doreg[i >> 1], i == 1 ? ndl : dn); }
        op[n % kDepth] = operand(n + kDepth);
        copy_beside(n);
        if (i & 1) {                                    // dS of keys 2j, 2j+1 of the lane's 16
          const int j = i >> 1;
          const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[2 * j], c, neg_l2));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[2 * j + 1], c, neg_l2));
          w[j] = pack2(p0 * dc[2 * j], p1 * dc[2 * j + 1]);
          MMSP_PIN(w[j]);
        }
        if ((i & 1) == 0) MMSP_PIN(sn); else MMSP_PIN(dn);
        MMSP_STEP_END();
      }
      const u32x4 ds0 = mk4(w[0], w[1], w[2], w[3]), ds1 = mk4(w[4], w[5], w[6], w[7]);
      // ---- phase B: dQ^T += K^T dS^T ----
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int n = blk * 24 + 16 + i, db = i & 3;
        dq[db] = mfma32(op[n % kDepth], i < 4 ? ds0 : ds1, dq[db]);
        op[n % kDepth] = operand(n + kDepth);
        copy_beside(n);
        MMSP_PIN(dq[db]);
        MMSP_STEP_END();
      }
    }
#undef MMSP_PIN
#undef MMSP_STEP_END
  };

  for (int t = kt0 - j0; t <= kt1; t += 4) {
    iteration(std::integral_constant<int, 0>(), t);
    iteration(std::integral_constant<int, 1>(), t + 1);
    iteration(std::integral_constant<int, 2>(), t + 2);
    iteration(std::integral_constant<int, 3>(), t + 3);
  }
  // lane, half and column anew: kept from above they would take registers that the loop is short of
  const int lane_e = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), half_e = lane_e >> 5, col_e = lane_e & 31;
  float* const out = kPartial ? part + (int64_t)split * a.n_q * a.Hq * 128 : a.dq + (int64_t)a.q_row0 * a.Hq * 128;
  auto result_at = [&](int list_row) {                   // where this lane's 16 bytes of a row of the list go
    return reinterpret_cast<float4*>(out + ((int64_t)row_of_pair(a, list_row) * (a.Hq - a.group) + kvh * a.group + list_row) * 128) + col_e;
  };
  const int row_up = tile_row0 + wave_s * 32 + half_e;   // this half of the wavefront takes every other row from here on
  float4 old[16];
  if (!kPartial) {                                       // on their way before the drain of the copies (28/4 heads, 64 x 64: 10.0 us behind it, 8.9 here)
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (row_up + 2 * i < row_end) old[i] = *result_at(row_up + 2 * i);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);                   // the copies issued past the end have landed, everybody is done with the tiles:
  lds_barrier();                                        // the result can pass through LDS
  char* const area = lds + wave_s * kResultBytes;
  result_to_lds(area, dq, a.scale, half_e, col_e);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    float4 o = result_chunk(area, 2 * i + half_e, col_e);
    if (!kPartial) { o.x += old[i].x; o.y += old[i].y; o.z += old[i].z; o.w += old[i].w; }
    if (row_up + 2 * i < row_end) *result_at(row_up + 2 * i) = o;
  }
}

template <int kWaves>
hipError_t launch(StepArgs a, const BwdWorkspace& st, const KeyRanges& r, float* part, hipStream_t stream) {
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
    bwd_dq_bf16_kernel<kWaves, true><<<g, b, 0, stream>>>(a, n_items, rows, xcd_bits, nsplit, part, st);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_dq_combine(a, part, nsplit, stream);
  }
  bwd_dq_bf16_kernel<kWaves, false><<<g, b, 0, stream>>>(a, n_items, rows, xcd_bits, 1, nullptr, st);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_bwd_dq_bf16(const StepArgs& a, const BwdWorkspace* stats_out, hipStream_t stream) {
  const BwdWorkspace no_stats = {nullptr, nullptr, nullptr, 0}, st = stats_out != nullptr ? *stats_out : no_stats;
  // the partial results lie where the dK/dV kernel, later on the same stream, keeps its own
  const int64_t stats = bwd_bf16_workspace_bytes(a.Hq, a.n_q) - bwd_dkdv_partial_bytes();
  // Two documents' keys for any number of query tiles (the forward: one to two): a tile costs more here, so a cut pays sooner.
  const KeyRanges r = pick_key_ranges(a, 1.6, (int64_t)a.n_q * a.Hq * 128 * sizeof(float), a.ws_bytes - stats, 2.);
  float* part = reinterpret_cast<float*>(a.ws + stats);
  return r.waves == 4 ? launch<4>(a, st, r, part, stream) : launch<8>(a, st, r, part, stream);
}

}  // namespace mmsp
