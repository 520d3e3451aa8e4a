// Shared declarations of the HIP side: kernel argument block, visibility bounds, and the
// launcher prototypes the C-ABI layer dispatches to.  gfx950 only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mmsp {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Everything a kernel needs to know about one call.  Row counts and positions are
// validated on the host to fit in int32.
struct StepArgs {
  // tensors (device)
  const void* q;  const void* k;  const void* v;
  const void* d_o;              // backward only
  float* o;  float* lse;        // forward outputs / running state
  const float* lse_final;  const float* delta;   // backward inputs
  float* dq;  float* dk;  float* dv;             // backward outputs
  const int32_t* cu;            // cu_seqlens or nullptr
  // shape
  int32_t Hq, Hkv, group, d;
  uint32_t group_magic;         // set_group()
  int64_t q_ts, q_hs, kv_ts, kv_hs, lse_hs;
  float scale;
  // block
  int32_t q_row0, n_q, k_row0, n_k, q_pos0, k_pos0;
  int32_t mask;                 // 0 full, 1 causal-diag
  int32_t n_docs;
  int32_t accumulate;           // fwd: merge into running state; bwd: add to dk/dv
  char* ws;                     // caller's workspace (bf16; nullptr or too small for a cut: no cut)
  int64_t ws_bytes;
  int32_t rank;                 // bf16 kernels: whether workgroups may rank their tiles (may_rank)
};

// Division of 0 <= i < 2^31 by a number the host knows.  The rounded-up reciprocal exceeds 1 / d by at most 2^-32, so the
// product's upper half is the quotient or, at most, one more.  (A division of two runtime integers is some 35 dependent
// instructions, of 64-bit ones over a hundred.)
struct FastDiv {
  uint32_t d, magic;                                    // magic: floor(2^32 / d) + 1, 0 for d = 1
};
inline FastDiv fast_div(int64_t d) { return {(uint32_t)d, d > 1 ? (uint32_t)((1ull << 32) / (uint64_t)d) + 1 : 0}; }
__device__ __forceinline__ uint32_t operator/(uint32_t i, const FastDiv& f) {
  if (f.magic == 0) return i;
  const uint32_t q = __umulhi(i, f.magic);
  return q - (q * f.d > i ? 1u : 0u);
}

// Heads per KV head; the row of pair i of a KV head's (row, head) list.
inline void set_group(StepArgs& a, int group) {
  a.group = group;
  a.group_magic = fast_div(group).magic;
}
__device__ __forceinline__ int row_of_pair(const StepArgs& a, int i) { return (int)((uint32_t)i / FastDiv{(uint32_t)a.group, a.group_magic}); }

// Workspace views of one backward call (all inside the caller's workspace).
struct BwdWorkspace {
  float* nl2;          // -LSE*log2e, [Hq][n_qtiles*64], -inf where LSE = -inf and in the padding
  float* ndl;          // -delta,     [Hq][n_qtiles*64], 0 in the padding
  float* partial;      // bwd_dkdv_partial_bytes(): partial dQ of cut query tiles, then dK and dV of split key tiles
  int32_t n_qtiles;
};

__host__ __device__ inline int64_t tiles_of(int64_t rows) { return (rows + 63) / 64; }

// Where a kernel reads cu_seqlens from: memory, or LDS that its workgroup has copied it to.  The searches below
// are chains of dependent reads, about 0.4 us each from memory and a tenth of that from LDS; a
// workgroup makes three of them before its first copy is issued, and one per tile that it ranks.
struct CuGlobal {
  const int32_t* p;
  __device__ __forceinline__ int operator[](int i) const { return p[i]; }
};
struct CuLocal {
  const int32_t* p;
  const int32_t* in_lds;
  bool copied;
  __device__ __forceinline__ int operator[](int i) const { return copied ? in_lds[i] : p[i]; }
};
constexpr int kMaxLocalDocs = 1023;                     // 4 KiB of LDS
// Copies cu_seqlens to `lds` (kMaxLocalDocs + 1 ints) if it fits; every thread of the workgroup calls it.
__device__ __forceinline__ CuLocal local_cu(const StepArgs& a, int32_t* lds, int n_threads) {
  const bool copied = a.cu != nullptr && a.n_docs <= kMaxLocalDocs;
  if (copied) {
    for (int i = threadIdx.x; i <= a.n_docs; i += n_threads) lds[i] = a.cu[i];
    __syncthreads();
  }
  return CuLocal{a.cu, lds, copied};
}

// Visible key interval [lo, hi] (indices inside the block's key range, already clipped to
// [0, n_k-1]) of the query row with block-relative index i.  Empty when lo > hi.
// A pair is visible iff the key position is <= the query position (causal-diag only) and
// both positions lie in the same cu_seqlens document (when given).
template <class Cu>
__device__ __forceinline__ void key_interval_of_row(const StepArgs& a, const Cu& cu, int i, int& lo, int& hi) {
  const int p = a.q_pos0 + i;
  int lo_pos = INT32_MIN / 2, hi_pos = INT32_MAX / 2;
  if (a.mask == 1) hi_pos = p;
  if (a.cu != nullptr) {
    // largest k with cu[k] <= p
    int L = 0, R = a.n_docs;          // invariant: cu[L] <= p (if p >= 0) < cu[R] (if inside)
    // positions outside every document see nothing; the empty intervals are chosen so that
    // lo and hi stay non-decreasing in the row index
    if (p < cu[0]) { lo = 0; hi = -1; return; }
    if (p >= cu[a.n_docs]) { lo = a.n_k; hi = a.n_k - 1; return; }
    while (R - L > 1) { int m = (L + R) >> 1; if (cu[m] <= p) L = m; else R = m; }
    lo_pos = max(lo_pos, cu[L]);
    hi_pos = min(hi_pos, cu[L + 1] - 1);
  }
  lo = max(0, lo_pos - a.k_pos0);
  hi = min(a.n_k - 1, hi_pos - a.k_pos0);
}

// Mirror image: interval [lo, hi] of block-relative query rows that see the key with
// block-relative index j (clipped to [0, n_q-1]).
template <class Cu>
__device__ __forceinline__ void row_interval_of_key(const StepArgs& a, const Cu& cu, int j, int& lo, int& hi) {
  const int p = a.k_pos0 + j;
  int lo_pos = INT32_MIN / 2, hi_pos = INT32_MAX / 2;
  if (a.mask == 1) lo_pos = p;
  if (a.cu != nullptr) {
    int L = 0, R = a.n_docs;
    if (p < cu[0]) { lo = 0; hi = -1; return; }
    if (p >= cu[a.n_docs]) { lo = a.n_q; hi = a.n_q - 1; return; }
    while (R - L > 1) { int m = (L + R) >> 1; if (cu[m] <= p) L = m; else R = m; }
    lo_pos = max(lo_pos, cu[L]);
    hi_pos = min(hi_pos, cu[L + 1] - 1);
  }
  lo = max(0, lo_pos - a.q_pos0);
  hi = min(a.n_q - 1, hi_pos - a.q_pos0);
}

// Workgroups are dispatched in index order as CUs come free, so the heaviest should come first.  Without
// documents the index order does that by itself (work falls or rises steadily under a causal mask); documents
// shorter than the block restart the triangle at every boundary, and heavy tiles that start last leave most CUs
// waiting for them.  The host does not know the documents, so every workgroup ranks the n tiles by itself:
// the index of the tile with the want-th most work (work(i) < 2^20; earlier tiles first among equals).
// That costs every workgroup some us, the more the more tiles there are; when it pays: may_rank.
// scratch: LDS of at least kMaxRanked + 1 ints, free to be overwritten when the function returns.
constexpr int kMaxRanked = 512;
template <class Work>
__device__ __forceinline__ int heaviest_first(int want, int n, int n_threads, int* scratch, Work work) {
  for (int i = threadIdx.x; i < n; i += n_threads) scratch[i] = work(i) * kMaxRanked + (kMaxRanked - 1 - i);
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += n_threads) {
    const int mine = scratch[i];
    int rank = 0;
    for (int j = 0; j < n; ++j) rank += scratch[j] > mine;
    if (rank == want) scratch[kMaxRanked] = i;
  }
  __syncthreads();
  const int found = __builtin_amdgcn_readfirstlane(scratch[kMaxRanked]);
  __syncthreads();
  return found;
}

// Whether ranking tiles over the positions [first, last] can change their order.
template <class Cu>
__device__ __forceinline__ bool worth_ranking(const StepArgs& a, const Cu& cu, int first, int last) {
  if (!a.rank) return false;
  if (first < cu[0] || last >= cu[a.n_docs]) return true;
  int L = 0, R = a.n_docs;
  while (R - L > 1) { int m = (L + R) >> 1; if (cu[m] <= first) L = m; else R = m; }
  return last >= cu[L + 1];                             // positions of one document: sorted already
}

// Key tiles of 64 that a query tile of n rows visits / query tiles of 64 that a key tile visits.
template <class Cu>
__device__ __forceinline__ int key_tiles_of_rows(const StepArgs& a, const Cu& cu, int row0, int n) {
  int lo, hi, dummy;
  key_interval_of_row(a, cu, row0, lo, dummy);
  key_interval_of_row(a, cu, min(row0 + n, a.n_q) - 1, dummy, hi);
  return hi >= lo ? min(hi / 64 - lo / 64 + 1, (1 << 20) - 1) : 0;
}
template <class Cu>
__device__ __forceinline__ int query_tiles_of_keys(const StepArgs& a, const Cu& cu, int key0, int n) {
  int lo, hi, dummy;
  row_interval_of_key(a, cu, key0, lo, dummy);
  row_interval_of_key(a, cu, min(key0 + n, a.n_k) - 1, dummy, hi);
  return hi >= lo ? min(hi / 64 - lo / 64 + 1, (1 << 20) - 1) : 0;
}

// ---- launchers (each enqueues on `stream` and returns hipGetLastError()) ----
hipError_t launch_fill_empty(float* o, float* lse, int64_t lse_hs, int Hq, int d,
                             int row0, int n_rows, hipStream_t stream);
hipError_t launch_zero_f32(float* p, int64_t n /* multiple of 4, p 16-byte aligned */, hipStream_t stream);
hipError_t launch_merge(float* o_acc, float* lse_acc, const float* o_part, const float* lse_part,
                        void* o_final, int io_dtype, int64_t lse_hs, int Hq, int d,
                        int row0, int n_rows, hipStream_t stream);
hipError_t launch_delta(const void* o_final, const void* d_o, float* delta, int io_dtype,
                        int64_t lse_hs, int Hq, int d, int row0, int n_rows, hipStream_t stream);

// Padded per-row statistics of the backward: nl2 = -LSE*log2e (or -inf), ndl = -delta.
hipError_t launch_bwd_stats(const float* lse, const float* delta, int64_t lse_hs, int Hq, int row0, int n_rows,
                            float* nl2, float* ndl, hipStream_t stream);

// Query tiles whose key range is cut into several workgroups (forward, dQ), see split.hip.
int cu_count();
double mean_document(const StepArgs& a);
int32_t may_rank(const StepArgs& a, int n_tiles, int n_blocks, int heads_per_tile, int max_rounds);
struct KeyRanges { int waves, count, rows; };           // wavefronts of a workgroup, workgroups that share a tile's keys, rows of a tile
KeyRanges pick_key_ranges(const StepArgs& a, double tile_us, int64_t bytes_per_range, int64_t room, double mean_documents);
hipError_t launch_fwd_combine(const StepArgs& a, const float* part_o, const float* part_lse, int nsplit, hipStream_t stream);
hipError_t launch_dq_combine(const StepArgs& a, const float* part, int nsplit, hipStream_t stream);

hipError_t launch_bwd_dkdv_bf16(const StepArgs& a, const BwdWorkspace& w, hipStream_t stream);
int64_t bwd_bf16_workspace_bytes(int Hq, int64_t n_q);
int64_t bwd_dkdv_partial_bytes();
// stats: where to write the padded row statistics on the way, or nullptr
hipError_t launch_bwd_dq_bf16(const StepArgs& a, const BwdWorkspace* stats, hipStream_t stream);

hipError_t launch_zigzag_gather(const void* seq, void* shards, int64_t T, int N, int64_t row_bytes, hipStream_t stream);
hipError_t launch_zigzag_scatter(const void* shards, void* seq, int64_t T, int N, int64_t row_bytes, hipStream_t stream);
hipError_t launch_swap_outer(const void* src, void* dst, int64_t A, int64_t B, int64_t row_bytes, hipStream_t stream);

hipError_t launch_fwd_f32(const StepArgs& a, hipStream_t stream);
hipError_t launch_bwd_f32(const StepArgs& a, hipStream_t stream);
hipError_t launch_fwd_bf16(const StepArgs& a, hipStream_t stream);
hipError_t launch_bwd_bf16(const StepArgs& a, hipStream_t stream);

}  // namespace mmsp
