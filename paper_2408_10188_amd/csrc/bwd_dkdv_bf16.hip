// Backward ring step, dK/dV kernel (key-stationary) on bf16 matrix cores, head_dim 128.
//
// Workgroup = 4 wavefronts (one per SIMD, the whole 512-entry register file each) = 128 keys of
// one KV head.  A wavefront owns 32 keys and keeps their K and V rows (MFMA B operands) and the
// two accumulators dK^T, dV^T (128 d x 32 keys each) in registers for the whole call.  64-row
// tiles of Q and dO of every query head of the group stream through a four-slot LDS ring filled
// by asynchronous global->LDS copies straight from the caller's tensors (natural orientation;
// the second products read them back transposed with ds_read_b64_tr_b16), the per-row
// statistics (-LSE*log2e, delta) from padded copies in the workspace.  Per 32-row block:
//   S = Q K^T,  dP = dO V^T            (A = Q / dO rows from LDS, B = K / V registers)
//   P = exp2(S*c - LSE*log2e),  dS = P * (dP - delta)
//   dV^T += dO^T P,  dK^T += Q^T dS    (A = dO / Q read transposed, B = P / dS straight from registers)
// Nothing passes between wavefronts, so the only workgroup barrier is the one that hands a ring
// slot over, once per tile.
//
// A matrix instruction keeps the SIMD's matrix pipe busy for 32 cycles but its issue port for
// about 8, so a wavefront keeps the pipe full on its own if independent vector and LDS
// instructions are interleaved with the matrix instructions in program order.  The loop is
// software-pipelined over blocks: while the pipe computes S and dP of block b+1 the vector units
// turn dP of block b into dS; while it accumulates dV and dK of block b they take the exponentials
// of block b+1.  The operand of every matrix instruction is read from LDS four instructions ahead.
#include <algorithm>
#include <type_traits>

#include "mfma_tiles.h"

namespace mmsp {
namespace {

constexpr int kKeys = 128;          // keys per workgroup
constexpr int kBQ = 64;             // query rows per streamed tile
constexpr int kWaves = 4;
constexpr int kCopies = 16 / kWaves;            // 1 KiB copies per wavefront and 16 KiB tile
constexpr int kGroup = 2 * kCopies + 1;         // copies per wavefront and ring slot: Q, dO, one statistics row
constexpr int kDepth = 4;                        // LDS operand reads in flight ahead of the matrix instructions (power of two)

#define MMSP_PIN(x) asm volatile("" : "+v"(x))
#define MMSP_PIN_ACC(x) asm volatile("" : "+a"(x))     // keeps an accumulator in the AGPR half of the register file
#define MMSP_STEP_END() __builtin_amdgcn_sched_barrier(0)

// The first products (S, dP) as inline assembly: their results are consumed by vector
// instructions, so they belong in the VGPR half of the register file, but the compiler puts every
// accumulator of a function that uses AGPRs into AGPRs and then copies the 64 results of a tile
// back one v_accvgpr_read each.  Of the 518 instructions of a tile those copies and the 32
// subtractions of delta (now the accumulator's start value) were 96.  The compiler does not know
// that these are matrix instructions, so the waits it would insert are the caller's:
//  * no vector instruction may write an operand in the two wait states before.  A comes straight from
//    an LDS read, B (AGPRs) never changes, and the accumulator input of dP, read from LDS too, is pinned before
//    the S product that precedes its first use, so that copies the compiler may need come before that product;
//  * a result may be read by a vector instruction only behind four more matrix instructions
//    (each holds the issue of the next for its eight passes; nineteen wait states are required), or behind
//    MMSP_RESULT_WAIT: MMSP_PIN of the result at that place keeps earlier readers out.
__device__ __forceinline__ void mfma32_v_first(f32x16& d, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "a"(b));
}
__device__ __forceinline__ void mfma32_v(f32x16& d, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b));
}
#define MMSP_RESULT_WAIT(x) asm volatile("s_nop 15\n\ts_nop 7" : "+v"(x))

// kMask = false: the host has checked that every (query, key) pair of the block is visible and
// that n_q is a multiple of the tile length, so no tile needs masking.
// nsplit > 1: the (query tile, head) sequence of every key tile is dealt out to nsplit
// workgroups, which store their partial dK / dV into w.partial for dkdv_reduce_kernel to sum
// (used when one workgroup per key tile would leave CUs idle or unevenly loaded).
// kAdd: add to dk and dv (nsplit is 1; the reduction does it otherwise).
template <bool kMask, bool kAdd>
__global__ __launch_bounds__(64 * kWaves, 1) void bwd_dkdv_bf16_kernel(StepArgs a, BwdWorkspace w, int n_kt, int xcd_per_kv,
                                                                       int nsplit, int rotate) {
  // LDS map: four Q tile slots in [0, 64 KiB), four dO tile slots in [64 KiB, 128 KiB), then the four
  // statistics slots.  Slots are selected at compile time (the loop is unrolled four tiles deep).
  // An LDS instruction's immediate offset reaches 64 KiB: reads of the upper regions go through
  // per-lane base registers that already hold the region's start (na_o, ta_o, so_st below), so
  // that no read needs an address addition of its own.
  constexpr int kQRegion = 0, kORegion = 4 * kTileBytes, kStRegion = 8 * kTileBytes;
  __shared__ __attribute__((aligned(1024))) char lds[kStRegion + 4 * 512];
  char* const qs0 = lds + kQRegion;                     // Q tiles, TileS
  char* const qs1 = qs0 + kTileBytes;
  char* const qs2 = qs1 + kTileBytes;
  char* const qs3 = qs2 + kTileBytes;
  char* const os0 = lds + kORegion;                     // dO tiles, TileS
  char* const os1 = os0 + kTileBytes;
  char* const os2 = os1 + kTileBytes;
  char* const os3 = os2 + kTileBytes;
  float* const st0 = reinterpret_cast<float*>(lds + kStRegion);   // [0,64) -LSE*log2e, [64,128) -delta
  float* const st1 = st0 + 128;
  float* const st2 = st1 + 128;
  float* const st3 = st2 + 128;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);   // the same value in a scalar register (LDS targets of the copies)
  const int half = lane >> 5, col = lane & 31;

  int kvh, item;                    // item = key tile * nsplit + range
  if (xcd_per_kv > 0) {             // workgroups of one KV head share an XCD (its L2 then serves the Q/dO stream once)
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    kvh = xcd / xcd_per_kv;
    item = slot * xcd_per_kv + (xcd % xcd_per_kv);
    if (item >= n_kt * nsplit) return;
  } else {
    item = blockIdx.x / a.Hkv;      // heavy tiles of every KV head first
    kvh = blockIdx.x - item * a.Hkv;
  }
  int kt = item / nsplit;
  const int split = (item - kt * nsplit + rotate * kt) % nsplit;
  const CuLocal cu = local_cu(a, reinterpret_cast<int32_t*>(lds + 8192), 64 * kWaves);
  if (kMask && worth_ranking(a, cu, a.k_pos0, a.k_pos0 + a.n_k - 1))
    kt = heaviest_first(kt, n_kt, 64 * kWaves, reinterpret_cast<int*>(lds), [&](int i) { return query_tiles_of_keys(a, cu, i * kKeys, kKeys); });
  kt = __builtin_amdgcn_readfirstlane(kt);
  const int tile_key0 = kt * kKeys;
  const int key = tile_key0 + wave * 32 + col;           // block-relative key of this lane
  const int keyc = min(key, a.n_k - 1);                  // a lane past the end repeats the last key: a column of its own that nobody stores

  int rlo, rhi;                                          // query rows that see this lane's key
  row_interval_of_key(a, cu, keyc, rlo, rhi);
  const int w_hi_min = __builtin_amdgcn_readlane(rhi, 0);    // first and last key of the wavefront
  const int w_lo_max = __builtin_amdgcn_readlane(rlo, 31);
  int t_lo, t_hi, dummy;
  row_interval_of_key(a, cu, tile_key0, t_lo, dummy);
  row_interval_of_key(a, cu, min(tile_key0 + kKeys, a.n_k) - 1, dummy, t_hi);
  if (cu.copied) __syncthreads();                        // the tile copies may overwrite cu_seqlens
  // wavefront-uniform values, pinned to scalar registers so that the loop control is scalar too
  t_lo = __builtin_amdgcn_readfirstlane(t_lo);
  t_hi = __builtin_amdgcn_readfirstlane(t_hi);
  const int qt0 = t_lo / kBQ, qt1 = t_hi >= t_lo ? t_hi / kBQ : qt0 - 1;
  const int ntiles = qt1 - qt0 + 1;
  // this workgroup's share of the (query tile, head of the group) sequence: elements split,
  // split + nsplit, ...  (interleaved rather than contiguous, so that the workgroups of a key
  // tile, and of neighbouring key tiles, walk the Q / dO tiles at the same place and pace and
  // share them in L2).  Sequence order: query tiles from the last visible one downwards, the
  // heads of the group inside a tile: under a causal or document mask the key tiles that share
  // an XCD see query ranges with different starts but a common end.
  int niter = 0;
  if (ntiles > 0) {
    const int total = ntiles * a.group;
    niter = total > split ? (total - split + nsplit - 1) / nsplit : 0;
  }
  if (kAdd && niter == 0) return;                          // nothing visible, nothing to add

  const float c = a.scale * kLog2e;

  f32x16 dv[4], dk[4];                                   // dV^T, dK^T: 128 d x 32 keys
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) { dv[db][i] = 0.f; dk[db][i] = 0.f; }

  // The results pass through LDS: into the partial result of this range, summed by dkdv_reduce_kernel, or where they belong.
  // Each store takes two whole rows; workgroups take the rows in different orders.  They end at the same time and their tiles lie at
  // distances of a power of two, so that in one order all of them write to a few memory channels at a time (4/2 heads,
  // 1000 x 2000, eight shares, 256 workgroups: 36.3 us in one order, 32.5 in several).  The i-th store takes rows turn ^ 2 i, in LDS at
  // addresses that an exclusive or turns into each other.
  const int turn = (2 * (7 * kt + 5 * split + 3 * kvh) & 31) + half, keys_up = a.n_k - (tile_key0 + wave_s * 32);
  int64_t rows[2];                                       // the wavefront's first row of dK and of dV, bytes from the pointer below
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    const int64_t first = nsplit > 1 ? ((int64_t)(which ? nsplit : 0) + split) * n_kt * kKeys : a.k_row0;
    rows[which] = ((first + tile_key0 + wave_s * 32) * a.Hkv + kvh) * 512;
    asm volatile("" : "+s"(rows[which]));                // or it is computed anew for every store
  }
  auto result_at = [&](int which, int i) {               // where this lane's 16 bytes of the i-th store go
    char* const out = reinterpret_cast<char*>(nsplit > 1 ? w.partial : which ? a.dv : a.dk) + rows[which];
    return reinterpret_cast<float4*>(out + ((uint32_t)(turn ^ 2 * i) * (uint32_t)(a.Hkv * 512) + col * 16));
  };
  auto each_store = [&](auto f) {
    if (keys_up >= 32) {
#pragma unroll
      for (int n = 0; n < 32; ++n) f(n >> 4, n & 15);
    } else {
#pragma unroll
      for (int n = 0; n < 32; ++n)
        if ((turn ^ 2 * (n & 15)) < keys_up) f(n >> 4, n & 15);
    }
  };
  float4 old[2][16];

  if (niter > 0) {
    // ---- asynchronous tile fetch: cursor over the (head of the group, query tile) sequence ----
    const char* qbase = reinterpret_cast<const char*>(a.q) + ((int64_t)a.q_row0 * a.q_ts + (int64_t)kvh * a.group * a.q_hs) * 2;
    const char* dobase = reinterpret_cast<const char*>(a.d_o) + ((int64_t)a.q_row0 * a.Hq + (int64_t)kvh * a.group) * 256;
    const int64_t q_tile_bytes = (int64_t)kBQ * a.q_ts * 2, do_tile_bytes = (int64_t)kBQ * a.Hq * 256;
    const int64_t q_head_bytes = (int64_t)a.q_hs * 2;
    const int64_t st_head_bytes = (int64_t)w.n_qtiles * kBQ * 4;
    const char* stat_src = reinterpret_cast<const char*>((wave_s & 1) ? w.ndl : w.nl2) + (int64_t)kvh * a.group * st_head_bytes;
    const DmaOffs<kCopies> qoff_full = dma_s_offsets<kCopies>(a.q_ts, kBQ, wave, lane);
    const DmaOffs<kCopies> dooff_full = dma_s_offsets<kCopies>((int64_t)a.Hq * 128, kBQ, wave, lane);
    // the last query tile of the block may be ragged: rows past the end repeat the last row
    const int qt_ragged = a.n_q % kBQ != 0 ? a.n_q / kBQ : -1;
    const DmaOffs<kCopies> qoff_ragged = dma_s_offsets<kCopies>(a.q_ts, qt_ragged >= 0 ? a.n_q % kBQ : kBQ, wave, lane);
    const DmaOffs<kCopies> dooff_ragged = dma_s_offsets<kCopies>((int64_t)a.Hq * 128, qt_ragged >= 0 ? a.n_q % kBQ : kBQ, wave, lane);
    // Element the next fetch takes, and where its Q / dO / statistics rows start.  The three
    // addresses are wavefront-uniform and move by additions only.
    int f_hg = split % a.group, f_qt = qt1 - split / a.group, f_it = 0;
    const char* f_q = qbase + f_hg * q_head_bytes + f_qt * q_tile_bytes;
    const char* f_do = dobase + f_hg * 256 + f_qt * do_tile_bytes;
    const char* f_st = stat_src + f_hg * st_head_bytes + f_qt * (kBQ * 4);
    const int64_t step_q = nsplit * q_head_bytes, wrap_q = a.group * q_head_bytes + q_tile_bytes;
    const int64_t step_do = nsplit * 256, wrap_do = a.group * 256 + do_tile_bytes;
    const int64_t step_st = nsplit * st_head_bytes, wrap_st = a.group * st_head_bytes + kBQ * 4;
    // A fetch is issued in 2 kCopies + 1 pieces (one copy instruction each) so that the loop can
    // spread them between its matrix instructions: a copy holds up the issuing wavefront while
    // the memory pipeline accepts it, and with one wavefront per SIMD nobody else fills that gap.
    struct Fetch { const char* q; const char* d_o; const char* st; bool ragged; };
    auto fetch_begin = [&]() {
      Fetch f;
      f.q = f_q; f.d_o = f_do; f.st = f_st;
      f.ragged = kMask && f_qt == qt_ragged;              // without a mask n_q is a multiple of the tile
      if (f_it + 1 < niter) {                           // past the end the last tile is fetched again (into a free slot)
        ++f_it;
        f_hg += nsplit; f_q += step_q; f_do += step_do; f_st += step_st;
        while (f_hg >= a.group) { f_hg -= a.group; --f_qt; f_q -= wrap_q; f_do -= wrap_do; f_st -= wrap_st; }
      }
      return f;
    };
    auto fetch_piece = [&](const Fetch& f, int piece, char* qdst, char* odst, float* sdst) {
      constexpr int W = 16 / kCopies;
      if (piece < kCopies) {
        dma16(f.q, f.ragged ? qoff_ragged.o[piece] : qoff_full.o[piece], qdst, (wave_s + piece * W) * 1024);
      } else if (piece < 2 * kCopies) {
        const int p = piece - kCopies;
        dma16(f.d_o, f.ragged ? dooff_ragged.o[p] : dooff_full.o[p], odst, (wave_s + p * W) * 1024);
      } else {
        dma4(f.st, (uint32_t)lane * 4, sdst, (wave_s & 1) * 256);   // even wavefronts fetch -LSE*log2e, odd ones -delta
      }
    };
    auto fetch = [&](char* qdst, char* odst, float* sdst) {
      const Fetch f = fetch_begin();
#pragma unroll
      for (int piece = 0; piece < kGroup; ++piece) fetch_piece(f, piece, qdst, odst, sdst);
    };
    fetch(qs0, os0, st0);
    // K and V rows of this lane's key as B operands (k index along d), on their way together with the first tile
    u32x4 kreg[8], vreg[8];
    {
      const int64_t off = (int64_t)(a.k_row0 + keyc) * a.kv_ts + (int64_t)kvh * a.kv_hs + half * 8;
      const uint16_t* pk = reinterpret_cast<const uint16_t*>(a.k) + off;
      const uint16_t* pv = reinterpret_cast<const uint16_t*>(a.v) + off;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        kreg[ks] = *reinterpret_cast<const u32x4*>(pk + ks * 16);
        vreg[ks] = *reinterpret_cast<const u32x4*>(pv + ks * 16);
      }
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) { MMSP_PIN_ACC(kreg[ks]); MMSP_PIN_ACC(vreg[ks]); }   // landed before the other tiles' copies are counted; AGPRs
    }
    fetch(qs1, os1, st1);
    fetch(qs2, os2, st2);

    // LDS read offsets inside a tile, fixed for the whole call: natural operand k-step ks (rows
    // +32 -> +8192 bytes); transposed operand of d block db, first / second read (16 rows further
    // -> +4096 bytes)
    int na[8], ta[4][2];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) na[ks] = tile_s_offset(col, ks * 2 + half);
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      ta[db][0] = tile_s_tr_offset(lane, db, 0);
      ta[db][1] = tile_s_tr_offset(lane, db, 1);
    }
    const int so = half * 4;                             // statistics of rows (i/4)*8 + half*4 + i%4: float4 at so + 8 g4
    // the same per-lane offsets with the start of the dO / statistics region added, kept opaque so
    // that the compiler uses them as bases instead of rebuilding them from na / ta
    int na_o[8], ta_o[4][2], so_st = so * 4 + kStRegion;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) { na_o[ks] = na[ks] + kORegion; asm volatile("" : "+v"(na_o[ks])); }
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      ta_o[db][0] = ta[db][0] + kORegion; asm volatile("" : "+v"(ta_o[db][0]));
      ta_o[db][1] = ta[db][1] + kORegion; asm volatile("" : "+v"(ta_o[db][1]));
    }
    asm volatile("" : "+v"(so_st));
    auto stat4 = [&](const float* slot, int first_float) {   // float4 of this lane's rows, first_float = offset inside the slot
      return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(slot) - kStRegion + so_st + first_float * 4);
    };

    // (head of the group, query tile) of the tile being computed
    int c_hg = split % a.group, c_qt = qt1 - split / a.group;

    // Software pipeline state carried from block to block.
    f32x16 s_nx, dp_nx;          // S and dP - delta of the next block (first products, being accumulated)
    f32x16 p_cur, dp_cur;        // P (fp32) and dP - delta of the current block
    u32x4 pb0, pb1;              // P of the current block packed as B operands (rows 0..15, 16..31)
    u32x4 oq[kDepth];            // LDS operands in flight, kDepth matrix instructions deep

    // Operand n of a tile body (one per matrix instruction), read four instructions ahead:
    //   n =  0..15  phase A of block 0: S / dP of block 1      natural rows 32..63 of this tile (Q even n, dO odd n)
    //   n = 16..31  phase B of block 0: dV / dK of block 0     transposed rows 0..31 (dO even n, Q odd n)
    //   n = 32..47  phase A of block 1: S / dP of the next tile's block 0   natural rows 0..31 of the next tile
    //   n = 48..63  phase B of block 1: dV / dK of block 1     transposed rows 32..63
    //   n = 64 ...  = the first operands of the next tile body (whose "this tile" is our next tile)
    auto operand = [&](int n, const char* cq, const char* co, const char* nq, const char* no) -> u32x4 {
      if (n >= 64) { n -= 64; cq = nq; co = no; }
      const int ph = n >> 4, i = n & 15;
      if ((ph & 1) == 0) {                               // natural: k-step i / 2, Q for S (even), dO for dP (odd)
        const int at = ph == 0 ? 8192 : 0;
        if (i & 1) return *reinterpret_cast<const u32x4*>((ph == 0 ? co : no) - kORegion + na_o[i >> 1] + at);
        return *reinterpret_cast<const u32x4*>((ph == 0 ? cq : nq) + na[i >> 1] + at);
      }
      // transposed: i = 8 t' + 2 db + (0: dO^T for dV, 1: Q^T for dK)
      const int tq = i >> 3, db = (i >> 1) & 3, g = (ph == 1 ? 0 : 2) + tq;
      u32x2 v0, v1;
      if (i & 1) {
        v0 = lds_read_tr(cq + ta[db][0] + g * 4096);
        v1 = lds_read_tr(cq + ta[db][1] + g * 4096);
      } else {
        v0 = lds_read_tr(co - kORegion + ta_o[db][0] + g * 4096);
        v1 = lds_read_tr(co - kORegion + ta_o[db][1] + g * 4096);
      }
      return mk4(v0.x, v0.y, v1.x, v1.y);
    };

    auto apply_mask = [&](f32x16& x, int q0) {           // q0: first row of the block
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int qrow = q0 + (i >> 2) * 8 + half * 4 + (i & 3);
        x[i] = (qrow < rlo || qrow > rhi) ? -INFINITY : x[i];
      }
    };
    // start value of dP's accumulator: -delta of the block's rows, read from LDS into its registers
    auto load_ndl = [&](f32x16& x, const float* slot, int row0) {
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const float4 d = stat4(slot, 64 + row0 + g4 * 8);
        x[g4 * 4 + 0] = d.x; x[g4 * 4 + 1] = d.y; x[g4 * 4 + 2] = d.z; x[g4 * 4 + 3] = d.w;
      }
    };
    auto needs_mask = [&](int q0) { return kMask && (q0 < w_lo_max || q0 + 31 > w_hi_min); };

    // ---- prologue: S, dP and P of the first block ----
    __builtin_amdgcn_s_waitcnt(0x0F70 | ((2 * kGroup) & 15) | (((2 * kGroup) >> 4) << 14));   // vmcnt(2 kGroup): the first tile has landed (two newer groups may be in flight)
    lds_barrier();
    {
      load_ndl(dp_nx, st0, 0);
      MMSP_PIN(dp_nx);
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        const u32x4 oq_ = *reinterpret_cast<const u32x4*>(qs0 + na[ks]), oo_ = *reinterpret_cast<const u32x4*>(os0 + na[ks]);
        if (ks == 0) mfma32_v_first(s_nx, oq_, kreg[ks]);
        else mfma32_v(s_nx, oq_, kreg[ks]);
        mfma32_v(dp_nx, oo_, vreg[ks]);
      }
      MMSP_RESULT_WAIT(s_nx);
      MMSP_RESULT_WAIT(dp_nx);
      if (needs_mask(c_qt * kBQ)) apply_mask(s_nx, c_qt * kBQ);
      uint32_t pw[8];
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const float4 nl = *reinterpret_cast<const float4*>(st0 + so + g4 * 8);
        p_cur[g4 * 4 + 0] = __builtin_amdgcn_exp2f(fmaf(s_nx[g4 * 4 + 0], c, nl.x));
        p_cur[g4 * 4 + 1] = __builtin_amdgcn_exp2f(fmaf(s_nx[g4 * 4 + 1], c, nl.y));
        p_cur[g4 * 4 + 2] = __builtin_amdgcn_exp2f(fmaf(s_nx[g4 * 4 + 2], c, nl.z));
        p_cur[g4 * 4 + 3] = __builtin_amdgcn_exp2f(fmaf(s_nx[g4 * 4 + 3], c, nl.w));
        pw[g4 * 2] = pack2(p_cur[g4 * 4 + 0], p_cur[g4 * 4 + 1]);
        pw[g4 * 2 + 1] = pack2(p_cur[g4 * 4 + 2], p_cur[g4 * 4 + 3]);
      }
      pb0 = mk4(pw[0], pw[1], pw[2], pw[3]);
      pb1 = mk4(pw[4], pw[5], pw[6], pw[7]);
      dp_cur = dp_nx;
      load_ndl(dp_nx, st0, 32);
    }

    // One tile: four phases of 16 matrix instructions.  cq / co / cs: this tile's slot, nq / no / ns:
    // the next tile's, rq / ro / rs: the slot to refill (three tiles ahead).
    auto body = [&](bool first, const char* cq, const char* co, const float* cs, const char* nq, const char* no, const float* ns,
                    char* rq, char* ro, float* rs) {
      // Own copies of every group but the newest have landed; after the barrier everybody's have
      // (this tile's and the next one's), and everybody is done with the slot about to be refilled.
      __builtin_amdgcn_s_waitcnt(0x0F70 | kGroup);
      lds_barrier();
      const Fetch fx = fetch_begin();
      const int q0 = c_qt * kBQ;
      c_hg += nsplit;
      while (c_hg >= a.group) { c_hg -= a.group; --c_qt; }
      const int q0_next = c_qt * kBQ;                    // first row of the next tile (unused after the last)
      if (first) {
#pragma unroll
        for (int n = 0; n < kDepth; ++n) oq[n] = operand(n, cq, co, nq, no);
      }
      MMSP_STEP_END();

#pragma unroll
      for (int ph = 0; ph < 4; ++ph) {
        const int blk = ph >> 1;                         // block of this tile the phase works for
        if ((ph & 1) == 0) {
          // ---- phase A: S, dP - delta of the following block beside dS of block blk ----
          uint32_t sw[8];
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int n = ph * 16 + i, ks = i >> 1;
            u32x4 op = oq[n & (kDepth - 1)];
            MMSP_PIN(op);
            if (i == 0) MMSP_PIN(dp_nx);
            if (i == 0) mfma32_v_first(s_nx, op, kreg[0]);
            else if ((i & 1) == 0) mfma32_v(s_nx, op, kreg[ks]);
            else mfma32_v(dp_nx, op, vreg[ks]);
            oq[n & (kDepth - 1)] = operand(n + kDepth, cq, co, nq, no);
            if (n % 7 == 3 && n / 7 < kGroup) fetch_piece(fx, n / 7, rq, ro, rs);
            if (i >= 4 && i < 12) {                      // dS of rows 2j, 2j+1 of the lane's 16 (one pair per step)
              const int j = i - 4, e = 2 * j;
              sw[j] = pack2(p_cur[e] * dp_cur[e], p_cur[e + 1] * dp_cur[e + 1]);
              MMSP_PIN(sw[j]);
            }
            MMSP_STEP_END();
          }
          // hand over: the packed dS of block blk feeds phase B; S / dP of the following block become current
          const u32x4 ds0 = mk4(sw[0], sw[1], sw[2], sw[3]), ds1 = mk4(sw[4], sw[5], sw[6], sw[7]);
          const int q0_f = blk == 0 ? q0 + 32 : q0_next;  // first row of the following block
          if (needs_mask(q0_f)) {
            MMSP_RESULT_WAIT(s_nx);
            apply_mask(s_nx, q0_f);
          }
          MMSP_STEP_END();
          // ---- phase B: dV, dK of block blk beside P of the following block ----
          const float* fs = blk == 0 ? cs + 32 : ns;     // -LSE*log2e of the following block's rows
          float4 nl[4];
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4) nl[g4] = stat4(fs, g4 * 8);
          uint32_t pw[8];
          f32x16 p_nx, dp_ld;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int n = (ph + 1) * 16 + i, tq = i >> 3, db = (i >> 1) & 3;
            u32x4 op = oq[n & (kDepth - 1)];
            MMSP_PIN(op);
            if ((i & 1) == 0) dv[db] = mfma32(op, tq ? pb1 : pb0, dv[db]);
            else dk[db] = mfma32(op, tq ? ds1 : ds0, dk[db]);
            oq[n & (kDepth - 1)] = operand(n + kDepth, cq, co, nq, no);
            if (n % 7 == 3 && n / 7 < kGroup) fetch_piece(fx, n / 7, rq, ro, rs);
            if (i == 4) { MMSP_PIN(s_nx); MMSP_PIN(dp_nx); }   // four matrix instructions behind the last first product
            if (i == 12) load_ndl(dp_ld, ns, blk * 32);  // for the block after the following one
            if (i >= 4 && i < 12) {                      // P of rows 2j, 2j+1
              const int j = i - 4, e = 2 * j;
              const float n0 = (e & 3) == 0 ? nl[e >> 2].x : nl[e >> 2].z;
              const float n1 = (e & 3) == 0 ? nl[e >> 2].y : nl[e >> 2].w;
              p_nx[e] = __builtin_amdgcn_exp2f(fmaf(s_nx[e], c, n0));
              p_nx[e + 1] = __builtin_amdgcn_exp2f(fmaf(s_nx[e + 1], c, n1));
              pw[j] = pack2(p_nx[e], p_nx[e + 1]);
              MMSP_PIN(pw[j]);
            }
            if ((i & 1) == 0) MMSP_PIN_ACC(dv[db]); else MMSP_PIN_ACC(dk[db]);
            MMSP_STEP_END();
          }
          pb0 = mk4(pw[0], pw[1], pw[2], pw[3]);
          pb1 = mk4(pw[4], pw[5], pw[6], pw[7]);
          p_cur = p_nx;
          dp_cur = dp_nx;
          dp_nx = dp_ld;
          MMSP_STEP_END();
        }
      }
    };

    // Four tiles per trip so that every slot is a compile-time constant; the steady-state loop
    // has no conditional bodies.
    int it = 0;
    for (; it + 3 < niter; it += 4) {
      body(it == 0, qs0, os0, st0, qs1, os1, st1, qs3, os3, st3);
      body(false, qs1, os1, st1, qs2, os2, st2, qs0, os0, st0);
      body(false, qs2, os2, st2, qs3, os3, st3, qs1, os1, st1);
      body(false, qs3, os3, st3, qs0, os0, st0, qs2, os2, st2);
    }
    if (it < niter) {
      body(it == 0, qs0, os0, st0, qs1, os1, st1, qs3, os3, st3);
      if (it + 1 < niter) body(false, qs1, os1, st1, qs2, os2, st2, qs0, os0, st0);
      if (it + 2 < niter) body(false, qs2, os2, st2, qs3, os3, st3, qs1, os1, st1);
    }
    // What is added to is read here, all of it at once, beside the drain of the copies: a launch of few tiles has nothing later to hide
    // the latency (4/2 heads, 32 x 32: 18.2 us with dK's and then dV's read behind the barrier, 13.7 here).
    if (kAdd) each_store([&](int which, int i) { old[which][i] = *result_at(which, i); });
    __builtin_amdgcn_s_waitcnt(0x0F70);                  // the copies issued past the end have landed
  }

  lds_barrier();                                         // everybody is done with the tiles: the results can pass through LDS
  char* const area = lds + wave * 2 * kResultBytes;
  const int chunk = turn * 512 + ((col ^ turn) << 4);
  result_to_lds(area, dk, a.scale, half, col);
  result_to_lds(area + kResultBytes, dv, 1.f, half, col);
  each_store([&](int which, int i) {
    float4 o = *reinterpret_cast<const float4*>(area + which * kResultBytes + (chunk ^ i * (2 * 512 + 2 * 16)));   // result_chunk of that row
    if (kAdd) { o.x += old[which][i].x; o.y += old[which][i].y; o.z += old[which][i].z; o.w += old[which][i].w; }
    *result_at(which, i) = o;
  });
}
#undef MMSP_PIN
#undef MMSP_PIN_ACC
#undef MMSP_STEP_END

// out[i] (+)= sum over the nsplit partial slots, for the n4 float4 of dK (blockIdx.y = 0) or dV (1).
__global__ __launch_bounds__(256) void dkdv_reduce_kernel(const float* __restrict__ partial, int nsplit, int64_t slot_elems,
                                                          float* __restrict__ dk, float* __restrict__ dv, int64_t n4,
                                                          bool accumulate) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n4) return;
  const float* src = partial + (int64_t)blockIdx.y * nsplit * slot_elems + i * 4;
  float4* dst = reinterpret_cast<float4*>(blockIdx.y ? dv : dk) + i;
  float4 x = accumulate ? *dst : make_float4(0.f, 0.f, 0.f, 0.f);
  auto add_up = [&](auto all, int s0) {                 // the partial results from s0 on, at most eight
    float4 p[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (all || s0 + j < nsplit) p[j] = *reinterpret_cast<const float4*>(src + (s0 + j) * slot_elems);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (all || s0 + j < nsplit) { x.x += p[j].x; x.y += p[j].y; x.z += p[j].z; x.w += p[j].w; }
  };
  int s0 = 0;
  for (; s0 + 8 <= nsplit; s0 += 8) add_up(std::true_type(), s0);
  if (s0 < nsplit) add_up(std::false_type(), s0);        // all on their way at once too: 28/4 heads, 50 x 50, seven shares 16.2 -> 15.0 us
  *dst = x;
}

}  // namespace

// The partial-sum area holds this many key tiles' dK and dV.
constexpr int kSplitMaxBlocks = 512;
constexpr int kSplitMaxRanges = 32;

int64_t bwd_dkdv_partial_bytes() { return 2LL * kSplitMaxBlocks * kKeys * 128 * (int64_t)sizeof(float); }

// What the key tiles of a launch have to do, in elements (64 rows of one head), heaviest first: `full` tiles of `most`, then tiles
// falling evenly to `least`; the rest sees nothing.
struct TileWork { int tiles, full, seen; double most, least; };

// Estimated us of the launch with n shares per tile.  A workgroup takes kElement for each of its elements and as much as kStart (kEmpty: without
// any) of them to begin and to store its result; the launch lasts as long as its longest chain of workgroups, or as the sum over all CUs.  Workgroups go
// to XCDs and shader engines in turn and wait for a CU of theirs, so that workgroup n_cu + k follows one a thirty-second
// further up, not the one that ends first (7/1 heads, 1500 rows behind 10000, three shares: 270 workgroups, the last 14 of them short,
// 154 us; in order of the ends they would take 126).  The reduction costs a launch, and every partial result is written and read.
static double dkdv_us(const TileWork& w, int n_kv_heads, int n, int n_cu) {
  constexpr double kElement = 1.2, kStart = 7., kEmpty = 2., kFixed = 8., kLaunch = 2.2, kMegabyte = .34;
  const int step = n_cu / 8, per_tile = n_kv_heads * n, blocks = w.tiles * per_tile;
  const double fall = (w.least - w.most) / std::max(1, w.seen - w.full), per_n = 1. / n;
  auto workgroup = [&](int i) {
    if (i >= blocks) return 0.;
    const int t = i / per_tile;
    if (t >= w.seen) return kEmpty;
    return (int)((w.most + fall * std::max(0, t - w.full + 1)) * per_n + (1. - 1e-9)) + kStart;   // rounded up
  };
  const double elements = n_kv_heads * (w.full * w.most + (w.seen - w.full) * (w.most + w.least) / 2);
  double longest = std::max(workgroup(0), (elements + per_tile * (w.seen * kStart + (w.tiles - w.seen) * kEmpty)) / n_cu);
  if (blocks > n_cu) {
    const int last = (std::min(blocks, 2 * n_cu) - 1 - n_cu) / step;
    for (int x : {0, last / 2, last}) longest = std::max(longest, workgroup(std::max(0, n_cu - step - step * x)) + workgroup(n_cu + step * x));
  }
  const double megabytes = 2e-6 * kKeys * 128 * sizeof(float) * blocks;
  return kFixed + kElement * longest + (n > 1 ? kLaunch + kMegabyte * megabytes : 0.);
}

// Into how many shares a key tile's (query tile, head) sequence is dealt.  Without documents, or with one, the host knows what every key
// tile sees; of several it knows only how many there are, and one long document wants another count than many of the mean length.
// So the count that gives every CU one workgroup (two where tiles differ), at most eight, is left only for one that the estimate finds
// faster, by 3 %, or with several documents by 10 % both if one of them holds everything and if the longest is twice the mean.
// Measured with every count up to 32: 4434 blocks without documents (5 arrangements of heads, 40 to 5000 rows on 40 to 17000 keys, with
// and without a causal mask) take 1.2 % longer than with their best count in the mean, 62 blocks of packs as synth.py draws
// them 2.9 %; 1265 with made-up documents (clips of 60 to 300 tokens, longer ones, one long first or last, few rows behind many keys) 6 %, where
// a rule that trusts the mean length takes 14 % and up to 2.9 times as long.  us by count:
//   28/4 heads, 760 x 1520:               1: 117  2: 73  3: 56  4: 52  5: 49  6: 68 (288 workgroups)
//   8/8 heads, 320 x 640:                 1: 17  2: 21  4: 25  6: 28
//   28/4 heads, 1000 rows behind 3000:    1: 163  2: 113  3: 141  4: 125 (nearly all tiles see all rows: whole rounds)
//   7/1 heads, 2500 x 2500 causal:        1: 357  4: 108  8: 68  16: 51  24: 57
//   4/2 heads, 4000 x 4000, documents:    one long 1: 221  2: 124  4: 79  8: 72;  clips of 60 to 300 1: 35  2: 33  4: 31  8: 49
static int pick_shares(const StepArgs& a, int n_kt) {
  const int base = n_kt * a.Hkv, q_tiles = (int)tiles_of(a.n_q), n_cu = cu_count();
  const int limit = (int)std::min<int64_t>({kSplitMaxRanges, kSplitMaxBlocks / base, (int64_t)q_tiles * a.group});
  if (limit <= 1) return 1;
  const bool even = a.mask == 0 && a.cu == nullptr;
  TileWork w[2];
  int n_w = 1;
  w[0] = {n_kt, n_kt, n_kt, (double)q_tiles * a.group, (double)q_tiles * a.group};
  const int64_t behind = (int64_t)a.q_pos0 - a.k_pos0;   // keys that lie before the first row
  if (a.mask == 1) {
    w[0].seen = (int)std::max<int64_t>(0, std::min<int64_t>(n_kt, (behind + a.n_q + kKeys - 1) / kKeys));
    w[0].full = std::min<int64_t>(w[0].seen, behind >= 0 ? behind / kKeys + 1 : 0);
    const int64_t hidden = std::min<int64_t>(a.n_q - 1, std::max<int64_t>(0, (int64_t)(w[0].seen - 1) * kKeys - behind));
    w[0].least = (double)(q_tiles - hidden / kBQ) * a.group;
  }
  const bool guess = a.cu != nullptr && a.n_docs > 1;
  if (guess) {
    const double mean = mean_document(a);
    const int before = (int)std::max(0., std::min((behind - mean) / kKeys, (double)n_kt));   // tiles of earlier documents
    n_w = 2;
    w[1] = {n_kt, 0, std::max(1, w[0].seen - before), std::min<double>(q_tiles, 2. * mean / kBQ + 2.) * a.group, std::min(q_tiles, 2) * (double)a.group};
  }
  const int fill = std::max(1, std::min({(even ? n_cu : 2 * n_cu) / base, 8, limit}));
  double with_fill[2];
  for (int k = 0; k < n_w; ++k) with_fill[k] = dkdv_us(w[k], a.Hkv, fill, n_cu);
  int best = fill;
  double best_ratio = guess ? .9 : .97;
  for (int n = 1; n <= limit; ++n) {
    double ratio = 0.;
    for (int k = 0; k < n_w && ratio < best_ratio; ++k) ratio = std::max(ratio, dkdv_us(w[k], a.Hkv, n, n_cu) / with_fill[k]);
    if (ratio < best_ratio) { best = n; best_ratio = ratio; }
  }
  return best;
}

// Workgroups go to XCDs in turn, so that with an even number of shares an XCD of several that serve a KV head gets the same shares of every key
// tile, with an odd one others from tile to tile.  The first way reads the Q and dO rows of a share into one L2 only, the second does not make
// all its workgroups wait for the same rows at once, which counts while a share is short: 28/4 heads, 747 x 373, 16 shares 31.5 us, 17 27.9;
// 4/2 heads, 2689 x 1344, 8 shares 39.5, 9 34.8.  Rotated by the tile's number an even number of short shares behaves as an odd one (28.6 and 35.3 us;
// an odd number would behave as an even one).  From some 16 elements on both take the same time (7/1 heads, 4096 x 4096 causal, 8 shares of 56: 96.4 and 96.2), and
// the first way reads less: 7/1 heads, 8192 x 8192 causal, 8 shares.
static int rotate_shares(const StepArgs& a, int xcd_per_kv, int nsplit) {
  if (xcd_per_kv < 2 || nsplit % 2 != 0) return 0;
  double tiles = (double)tiles_of(a.n_q);
  if (a.cu != nullptr) tiles = std::min(tiles, 2. * mean_document(a) / kBQ + 2.);
  return tiles * a.group <= 16. * nsplit;
}

hipError_t launch_bwd_dkdv_bf16(const StepArgs& args, const BwdWorkspace& w, hipStream_t stream) {
  StepArgs a = args;
  const int n_kt = (a.n_k + kKeys - 1) / kKeys;
  const bool no_mask = a.mask == 0 && a.cu == nullptr && a.n_q % kBQ == 0;
  const int nsplit = pick_shares(a, n_kt);
  const int n_items = n_kt * nsplit;
  a.rank = may_rank(a, n_kt, n_items * a.Hkv, a.group, 7);
  int xcd_per_kv = 0, n_blocks = n_items * a.Hkv;
  if (8 % a.Hkv == 0) {
    xcd_per_kv = 8 / a.Hkv;
    n_blocks = 8 * ((n_items + xcd_per_kv - 1) / xcd_per_kv);
  }
  const bool add = a.accumulate && nsplit == 1;
  const auto kernel = no_mask ? (add ? bwd_dkdv_bf16_kernel<false, true> : bwd_dkdv_bf16_kernel<false, false>)
                              : (add ? bwd_dkdv_bf16_kernel<true, true> : bwd_dkdv_bf16_kernel<true, false>);
  kernel<<<dim3(n_blocks), dim3(64 * kWaves), 0, stream>>>(a, w, n_kt, xcd_per_kv, nsplit, rotate_shares(a, xcd_per_kv, nsplit));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || nsplit == 1) return e;
  const int64_t n4 = (int64_t)a.n_k * a.Hkv * 32;
  const int64_t first = (int64_t)a.k_row0 * a.Hkv * 128;
  dkdv_reduce_kernel<<<dim3((unsigned)((n4 + 255) / 256), 2), dim3(256), 0, stream>>>(
      w.partial, nsplit, (int64_t)n_kt * kKeys * a.Hkv * 128, a.dk + first, a.dv + first, n4, a.accumulate);
  return hipGetLastError();
}

}  // namespace mmsp
