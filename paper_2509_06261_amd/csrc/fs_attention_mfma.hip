// MFMA split-K paged decode-attention kernel for gfx950 (head_dim 64, 128 or 256, all four KV formats).
//
// FineServe Sec. 2.1: the decode phase re-reads the whole KV cache for every generated token and is bound by
// memory bandwidth; Sec. 2.3 / 5.1: the cache is reached through each model's own block table over the
// shared slab pool.  The tile machinery (loads, dequantization around the MFMAs, online softmax) is in
// fs_mfma_tiles.h; this file holds the work decomposition:
//   a persistent grid of independent waves: each wave draws work items (sequence, split, KV head) from the
//   queue, streams the split's 32-token tiles with a private online-softmax state and writes the output (or
//   the split's partial record) straight from its accumulators.  No wave waits for another.
//   An item's record carries its sequence's length, so the only look-up between a queue ticket and the item's
//   first K/V requests is the record, then the block-table entries.
// Launches whose sequences need no fine splitting take mfma_direct_kernel instead: one workgroup per (sequence, split,
// KV head), no queue (plan_direct decides).
#include "fs_mfma_tiles.h"

namespace fs {
namespace {

// What the wave knows about an item before its tiles stream (all wave-uniform): the record's fields, the runs
// [v0, v1) it covers and the blocks k0 .. k0 + nb - 1 they lie in.
struct ItemPlan {
  int b, seq, chunk, head, len;
  uint32_t local;  // the item's index within its batch: where its partial record goes
  int v0, v1, k0, nb;
};

// rec: lane l < 8 holds dword l of the item's record (see make_rec).
__device__ __forceinline__ ItemPlan plan_item(const MultiArgs& A, uint32_t rec) {
  ItemPlan P;
  const int x = (int)__builtin_amdgcn_readlane(rec, 0);
  P.b = x & 15;
  P.head = x >> 4;
  P.seq = (int)__builtin_amdgcn_readlane(rec, 1);
  P.chunk = (int)__builtin_amdgcn_readlane(rec, 2);
  P.local = __builtin_amdgcn_readlane(rec, 3);
  P.len = (int)__builtin_amdgcn_readlane(rec, 4);
  const ItemRange r = item_range(A.b[P.b], P.seq, P.chunk, P.len);
  P.v0 = r.v0;
  P.v1 = r.v1;
  P.k0 = r.k0;
  P.nb = r.nb;
  return P;
}

constexpr int kTabRegs = 4;  // an item touches at most 64 * kTabRegs blocks (the host caps the item size accordingly)

// The item's block-table entries: entry i goes to register i / 64 of lane i % 64.
__device__ __forceinline__ void load_entries(const MultiArgs& A, const ItemPlan& P, int lane, int32_t (&tab)[kTabRegs]) {
  const DevBatch& B = A.b[P.b];
  const int32_t* t = B.tables + (int64_t)P.seq * B.max_blocks + P.k0;
#pragma unroll
  for (int q = 0; q < kTabRegs; ++q) tab[q] = lane + 64 * q < P.nb ? t[lane + 64 * q] : 0;
}

// Head-chunk addresses of the item's blocks into this wave's LDS table (see fill_table).
__device__ __forceinline__ void store_table(const MultiArgs& A, const ItemPlan& P, int lane, const int32_t (&tab)[kTabRegs],
                                            uint64_t* s_ptr) {
  const DevBatch& B = A.b[P.b];
  const uint8_t* head_base = B.layer_base + (uint64_t)P.head * B.g.head_chunk;
#pragma unroll
  for (int q = 0; q < kTabRegs; ++q)
    if (lane + 64 * q < P.nb)
      s_ptr[lane + 64 * q] = reinterpret_cast<uint64_t>(head_base + (uint64_t)checked_block(tab[q], B.n_blocks, A.header) * B.g.block_budget);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One work item is processed by ONE wave in two steps: stream_item runs all tiles of the split through the wave's
// private online-softmax state; finish_item writes the output (or the split's partial record) straight from the
// accumulator registers.  Waves never synchronise with each other.  (Two steps, so that the tile loops of the
// eight format / group variants do not carry the output code's registers; the state has the same shape for all.)
// s_ptr: this wave's LDS table of head-chunk addresses, already holding the item's blocks.
template <int DT, int GP, int HD>
__device__ __forceinline__ void stream_item(const MultiArgs& A, const ItemPlan& P, uint64_t* s_ptr, StateT<HD>& st) {
  const int seq = P.seq, head = P.head;
  const DevBatch& B = A.b[P.b];
  const DevGeom& g = B.g;
  // The lane index is made opaque per item: otherwise the compiler hoists every variant's lane-dependent
  // constants out of the kernel's item loop, where they stay live across all other variants and push the
  // tile loops into spilling.
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int j = lane >> 4, c = lane & 15;
  const int G = B.G;

  ItemCtx X;
  X.T = g.T;
  X.R = B.R;
  X.r_magic = B.r_magic;
  X.len = P.len;
  X.len_u = P.len;
  X.v_end = P.v1;
  X.k0 = P.k0;
  X.chunk_ptr = s_ptr;

  // Q operand and per-head constants
  u32x4 qb[HD / 32];
  float qsum;
  load_q<DT, true, HD>(B.q + ((int64_t)seq * B.n_q + head * G + c) * HD, c < G, j, qb, qsum);
  if constexpr (Fmt<DT, HD>::kParBytes != 0) {
    qsum += __shfl_xor(qsum, 16, 64);
    qsum += __shfl_xor(qsum, 32, 64);
    if constexpr (GP == 4) qsum = __shfl(qsum, c & 3, 64);  // of the head this lane exponentiates
  }
  float alpha = B.sm_scale * kLog2e;
  if (DT == FS_KV_FP8_E4M3) alpha *= B.k_scale[head];

#pragma unroll
  for (int e = 0; e < HD / 16; ++e) st.acc[e] = float4v{0.f, 0.f, 0.f, 0.f};
  st.m = kNoReference;
  st.l = 0.f;
  st.zc = 0.f;

  if constexpr (DT == FS_KV_INT8) {
    if (B.stream_v) return stream_tiles<DT, GP, HD, true, true>(X, g, P.v0, qb, qsum, alpha, st, j, c);
  }
  stream_tiles<DT, GP, HD, true>(X, g, P.v0, qb, qsum, alpha, st, j, c);
}

// Per-head sums over the lanes of the head.
template <int DT, int GP, int HD>
__device__ __forceinline__ void reduce_sums(StateT<HD>& st) {
  if constexpr (GP == 4) {
    st.l += __shfl_xor(st.l, 4, 64);
    st.l += __shfl_xor(st.l, 8, 64);
  }
  st.l += __shfl_xor(st.l, 16, 64);
  st.l += __shfl_xor(st.l, 32, 64);
  if constexpr (Fmt<DT, HD>::kParBytes != 0) {
    if constexpr (GP == 4) {
      st.zc += __shfl_xor(st.zc, 4, 64);
      st.zc += __shfl_xor(st.zc, 8, 64);
    }
    st.zc += __shfl_xor(st.zc, 16, 64);
    st.zc += __shfl_xor(st.zc, 32, 64);
  }
}

// Accumulator row r of this lane, dequantized (not divided by the sum).
template <int DT, int HD>
__device__ __forceinline__ void output_row(const StateT<HD>& st, int r, float Z, float v_static, float (&o)[HD / 16]) {
#pragma unroll
  for (int e = 0; e < HD / 16; ++e) {
    o[e] = column_value<DT>(st.acc, e, r);
    if constexpr (Fmt<DT, HD>::kParBytes != 0) o[e] += Z;
    o[e] *= v_static;
  }
}

// part_off: the batches' offsets into the partial buffer (the workspace header's words, copied to LDS once per
// workgroup: read from memory here they would be one more round trip in front of every item's stores).
template <int DT, int GP, int HD>
__device__ __forceinline__ void finish_item(const MultiArgs& A, const ItemPlan& P, StateT<HD>& st, const uint64_t* part_off) {
  constexpr int NE = HD / 16;  // output columns of this lane (column_of)
  const int b = P.b, seq = P.seq, head = P.head;
  const DevBatch& B = A.b[b];
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int j = lane >> 4, c = lane & 15;
  const int G = B.G;
  const int n_chunks = n_splits(B, seq, P.len);
  const uint64_t part_base = part_off[b] + (uint64_t)P.local * (uint64_t)B.part_stride;  // local: index within the batch
  if (n_chunks > 1 && part_base + (uint64_t)B.part_stride > A.part_capacity) {  // wave-uniform
    // the workspace was sized for shorter sequences: reported, the item's record is not written
    if (lane == 0) atomicOr(A.header + kHdrStatus, 2u);
    return;
  }

  // ---- output: rows h < G straight from the accumulators ----
  reduce_sums<DT, GP, HD>(st);
  const float v_static = DT == FS_KV_FP8_E4M3 ? B.v_scale[head] : 1.0f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int h = 4 * j + r;  // accumulator row r of this lane; its m, l, zc live in lane c = h
    const float L = __shfl(st.l, h, 64), M = __shfl(st.m, h, 64), Z = __shfl(st.zc, h, 64);
    if (h < G) {
      float o[NE];
      output_row<DT, HD>(st, r, Z, v_static, o);
      const int qh = head * G + h;
      if (n_chunks == 1) {
        const float inv = 1.0f / L;
        uint32_t w[NE / 2];
#pragma unroll
        for (int q = 0; q < NE / 2; ++q) {
          const half2v hv = {(_Float16)(o[2 * q] * inv), (_Float16)(o[2 * q + 1] * inv)};
          w[q] = h2u(hv);
        }
        _Float16* orow = B.out + ((int64_t)seq * B.n_q + qh) * HD;
        if constexpr (NE == 4) {
          *reinterpret_cast<u32x2*>(orow + column_of<DT, HD>(c, 0)) = u32x2{w[0], w[1]};
        } else {
#pragma unroll
          for (int q = 0; q < NE / 8; ++q)
            *reinterpret_cast<u32x4*>(orow + column_of<DT, HD>(c, 8 * q)) = u32x4{w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]};
        }
        if (c == 0 && B.lse) B.lse[(int64_t)seq * B.n_q + qh] = (M + __builtin_amdgcn_logf(L)) * kLn2;
      } else {
        float* pr = A.partials + part_base + (uint64_t)h * (HD + 2);
        // (a row starts at a multiple of 8 bytes: part_stride and HD + 2 are even)
#pragma unroll
        for (int e = 0; e < NE; e += 2) *reinterpret_cast<float2*>(pr + column_of<DT, HD>(c, e)) = float2{o[e], o[e + 1]};
        if (c == 0) {
          pr[HD] = M * kLn2;  // partial records keep the reference in natural-log units
          pr[HD + 1] = L;
        }
      }
    }
  }
}

// The state of a wave as the partial records of its G heads, rec[h (HD + 2)] in LDS: unnormalized output row,
// reference (natural-log units), sum.
template <int DT, int GP, int HD>
__device__ __forceinline__ void leave_records(const MultiArgs& A, const ItemPlan& P, StateT<HD>& st, float* rec) {
  constexpr int NE = HD / 16;
  const DevBatch& B = A.b[P.b];
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int j = lane >> 4, c = lane & 15;
  reduce_sums<DT, GP, HD>(st);
  const float v_static = DT == FS_KV_FP8_E4M3 ? B.v_scale[P.head] : 1.0f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int h = 4 * j + r;
    const float L = __shfl(st.l, h, 64), M = __shfl(st.m, h, 64), Z = __shfl(st.zc, h, 64);
    if (h < B.G) {
      float* pr = rec + h * (HD + 2);
      float o[NE];
      output_row<DT, HD>(st, r, Z, v_static, o);
#pragma unroll
      for (int e = 0; e < NE; e += 2) *reinterpret_cast<float2*>(pr + column_of<DT, HD>(c, e)) = float2{o[e], o[e + 1]};
      if (c == 0) *reinterpret_cast<float2*>(pr + HD) = float2{M * kLn2, L};
    }
  }
}

// step 0: stream_item, step 1: finish_item, step 2: stream_item and leave_records
template <int STEP, int GP, int HD>
__device__ __forceinline__ void dispatch_dtype(const MultiArgs& A, const ItemPlan& P, uint64_t* s_ptr, StateT<HD>& st,
                                               const uint64_t* part_off, float* rec) {
  switch (A.b[P.b].g.dtype) {
#define FS_STEP(DT)                                                       \
  if constexpr (STEP == 0) stream_item<DT, GP, HD>(A, P, s_ptr, st);      \
  else if constexpr (STEP == 1) finish_item<DT, GP, HD>(A, P, st, part_off); \
  else {                                                                  \
    StateT<HD> own;                                                       \
    stream_item<DT, GP, HD>(A, P, s_ptr, own);                            \
    leave_records<DT, GP, HD>(A, P, own, rec);                            \
  }                                                                       \
  break
    case FS_KV_FP16: FS_STEP(FS_KV_FP16);
    case FS_KV_FP8_E4M3: FS_STEP(FS_KV_FP8_E4M3);
    case FS_KV_INT8: FS_STEP(FS_KV_INT8);
    default: FS_STEP(FS_KV_INT4);
#undef FS_STEP
  }
}

template <int STEP, int HD>
__device__ __forceinline__ void dispatch_item(const MultiArgs& A, const ItemPlan& P, uint64_t* s_ptr, StateT<HD>& st,
                                              const uint64_t* part_off, float* rec = nullptr) {
  if (A.b[P.b].G <= 4) dispatch_dtype<STEP, 4, HD>(A, P, s_ptr, st, part_off, rec);
  else dispatch_dtype<STEP, 16, HD>(A, P, s_ptr, st, part_off, rec);
}

// One kernel per head_dim (every batch of a launch has the same one).
template <int HD>
__global__ __launch_bounds__(kThreads, mfma_wgs_per_cu(HD)) void mfma_attention_kernel(MultiArgs A, int table_entries) {
  extern __shared__ uint64_t smem64[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint64_t* s_ptr = smem64 + (size_t)wave * table_entries;
  __shared__ uint64_t s_part_off[kMaxBatches];
  if (threadIdx.x < kMaxBatches) s_part_off[threadIdx.x] = reinterpret_cast<const uint64_t*>(A.header + kHdrPartOff)[threadIdx.x];
  __syncthreads();
  const uint32_t total = A.header[kHdrTotalItems];
#ifdef FS_TIMELINE
  const uint64_t tl_start = wall_clock64();
  uint64_t tl_items = 0;
#endif
  // Every wave is its own worker and draws its items from kDecodePools ticket counters: pool p holds the items
  // p, p + kDecodePools, ... of the queue.  Waves that get short items, or sit on a faster compute unit, simply
  // draw more often; with a fixed deal (wave w takes items w, w + n_workers, ...) the slowest wave was
  // measured to finish a quarter later than the median one.  One counter for all items is no option: an
  // address serves an atomic every ~11 ns when idle and several times slower under streaming load, which
  // was measured to bound the kernel (and still to cost short launches a tenth with 8 counters); 64 do not.
  // A wave takes its tickets from the pools in turn (its k-th from pool w + k), so all counters advance at
  // about the same rate and the grid as a whole walks the queue roughly front to back: the large items of the
  // queue's front are all under way before its small last items are handed out.  (With a home pool per wave that
  // was emptied before the wave looked elsewhere, the pools drifted apart and the slowest pool's large items
  // started when the others were done: waves idled 5 % of the launch at its end, against 3.5 %.)
  // Once a wave meets an empty pool the launch is in its last few per cent.  From then on the wave looks at all
  // counters at once (lane p reads pool p's) and picks the pool of a random one of the items that are left, so
  // pools that lag get helpers in proportion to what they still hold, and stays there until that pool is
  // empty too.  It leaves only when every pool is past its last item.
  // The next ticket is drawn before the current item is processed, so the atomic's latency is not waited for
  // between items; a wave's first ticket needs no draw at all (the work-list kernel starts the counters past the
  // pools' first waves), which takes one round trip off the start of every launch.
  static_assert(kDecodePools <= 64, "one pool per lane in the look at all counters");
  const uint32_t worker = blockIdx.x * kWaves + wave;
  uint32_t pool = worker % kDecodePools;
  uint32_t ticket = worker / kDecodePools;
  bool in_turn = true;                            // false once an empty pool was met
  uint32_t rng = worker * 2654435761u + 0x9e3779b9u;  // wave-uniform
  constexpr uint32_t kNone = 0xffffffffu;
  auto draw = [&]() {
    if (lane == 0) ticket = atomicAdd(A.header + kHdrPools + pool * kPoolStride, 1u);
  };
  // the item the drawn ticket stands for, or kNone once every pool is empty (then no ticket is outstanding)
  auto resolve = [&]() -> uint32_t {
    for (;;) {
      const uint32_t item = pool + kDecodePools * __builtin_amdgcn_readfirstlane(ticket);
      if (item < total) return item;
      // this pool is empty: what do the others hold?  (the counters only grow)
      in_turn = false;
      const uint32_t cnt = lane < kDecodePools ? __hip_atomic_load(A.header + kHdrPools + lane * kPoolStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
      const uint32_t held = lane < kDecodePools && (uint32_t)lane < total ? (total - lane + kDecodePools - 1) / kDecodePools : 0u;
      uint32_t incl = held > cnt ? held - cnt : 0u;  // items left in pool `lane`, then their inclusive sum over the lanes
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(incl, off, 64);
        if (lane >= off) incl += t;
      }
      const uint32_t left = __builtin_amdgcn_readlane(incl, 63);
      if (left == 0) return kNone;  // every pass finds fewer items left or takes one
      rng = rng * 1664525u + 1013904223u;
      const uint32_t k = (uint32_t)(((uint64_t)rng * (uint64_t)left) >> 32);  // one of the items left, uniformly
      pool = (uint32_t)__builtin_ctzll(__ballot(incl > k));                    // the pool it lies in (wave-uniform)
      draw();
    }
  };
  auto load_rec = [&](uint32_t item) -> uint32_t {
    return lane < 8 ? reinterpret_cast<const uint32_t*>(A.item_list + 2 * (size_t)item)[lane] : 0u;
  };
  for (;;) {
    const uint32_t item = resolve();
    if (item == kNone) break;  // every wave leaves here, once all pools are empty
#ifdef FS_TIMELINE
    const uint64_t tl_begin = wall_clock64();
#endif
    if (in_turn) pool = (pool + 1) % kDecodePools;
    draw();                    // the next ticket, answered while this item streams
    const ItemPlan P = plan_item(A, load_rec(item));
    int32_t tab[kTabRegs];
    load_entries(A, P, lane, tab);
    store_table(A, P, lane, tab, s_ptr);
#ifdef FS_TIMELINE
    const uint64_t tl_table = wall_clock64();
    ++tl_items;
#endif
    StateT<HD> st;
    dispatch_item<0, HD>(A, P, s_ptr, st, s_part_off);
#ifdef FS_TIMELINE
    const uint64_t tl_tiles = wall_clock64();
#endif
    dispatch_item<1, HD>(A, P, s_ptr, st, s_part_off);
#ifdef FS_TIMELINE
    if (lane == 0 && item < kTimelineItems) {
      uint64_t* row = A.timeline + 8 * (kTimelineWaves + item);
      row[0] = tl_begin;
      row[1] = tl_table;
      row[2] = tl_tiles;
      row[3] = wall_clock64();
      row[4] = (uint64_t)(blockIdx.x * kWaves + wave) | ((uint64_t)P.b << 32) | ((uint64_t)tier_of(A.b[P.b], P.seq) << 40);
      row[5] = (uint64_t)(P.v1 - P.v0) | ((uint64_t)P.seq << 32);
    }
#endif
  }
#ifdef FS_TIMELINE
  if (lane == 0 && blockIdx.x * kWaves + wave < kTimelineWaves) {
    uint64_t* row = A.timeline + 8 * (blockIdx.x * kWaves + wave);
    row[0] = tl_start;
    row[1] = wall_clock64();
    row[2] = tl_items;
    row[3] = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7;  // hwreg(HW_REG_XCC_ID, 0, 4)
  }
#endif
}

// ---- Direct launches: one workgroup per (sequence, split, KV head), no work list ------------------------------------
// The grid itself is the queue: the hardware hands workgroups out in order as compute units fall free.  A workgroup finds
// its item from its index, requests the sequence's length and the item's block-table entries together, its four waves
// stream a quarter of the item's tiles each and leave their records in LDS, where the workgroup merges them: into the
// output if the sequence has one split, into a partial record for direct_combine_kernel otherwise.
// What it saves over the work list: the preparation launch, tickets, item records, most partial records, and the combine
// wherever a sequence has one split.  Eight sequences of up to 256 tokens, 4 KV heads of 64: 19.3 -> 8.3 us; 64 FP16
// sequences of 512 - 4096 tokens, 8 KV heads of 128: 128 - 139 -> 105 - 115 us (5.3 - 5.8 TB/s); 128 FP8 sequences of
// 3000 - 4000 tokens: 184 - 202 -> 147 - 153 us; five FP8 sequences of 9000 - 32768: 56 -> 42 us.
// The status word has nobody to clear it before the launch: the items report to a word that nobody reads, and workgroup
// 0 does nothing but judge the whole call and write the word.
constexpr int kEntriesPerThread = kDirectEntries / kThreads;

typedef int32_t entries4 __attribute__((ext_vector_type(4), aligned(4)));  // (a table's rows are aligned to an entry only)

// Status of the call: bit 0 for a length out of range, bit 2 for a block-table entry outside the pool inside a length.
__device__ __forceinline__ void direct_status(const DirectArgs& D, uint32_t* status) {
  const MultiArgs& A = D.m;
  __shared__ uint32_t s_flags;
  if (threadIdx.x == 0) s_flags = 0;
  __syncthreads();
  // as many neighbouring threads per sequence as there are for all of them
  int per = kThreads;
  while (per > 1 && per * A.n_seq_total > kThreads) per >>= 1;
  uint32_t flags = 0;
  for (int i = threadIdx.x / per; i < A.n_seq_total; i += kThreads / per) {
    int b = 0;
    while (b + 1 < A.n_batches && i >= A.b[b + 1].seq_first) ++b;
    const DevBatch& B = A.b[b];
    const int seq = i - B.seq_first;
    const int max_len = (int)min((int64_t)B.max_blocks * B.g.T, (int64_t)0x7fffffff);
    int len = B.seq_lens[seq];
    if (len < 1 || len > max_len) flags |= 1u;
    len = len < 1 ? 1 : min(len, max_len);
    const int nb = (len + B.g.T - 1) / B.g.T;
    const int32_t* table = B.tables + (int64_t)seq * B.max_blocks;
    // four entries per load: with a thread per sequence neighbouring lanes read different lines, and it is the loads in flight
    // that count (the whole call, an entry per load: 512 INT4 sequences of 400 entries 121 us, 77 now; 1024 FP16 ones of 64
    // entries 44 and 29)
#pragma unroll 4
    for (int k = 4 * (threadIdx.x % per); k + 4 <= nb; k += 4 * per) {
      const entries4 e = *reinterpret_cast<const entries4*>(table + k);
#pragma unroll
      for (int q = 0; q < 4; ++q) flags |= (uint32_t)e[q] < B.n_blocks ? 0u : 4u;
    }
    for (int k = (nb & ~3) + threadIdx.x % per; k < nb; k += per) flags |= (uint32_t)table[k] < B.n_blocks ? 0u : 4u;
  }
  if (flags) atomicOr(&s_flags, flags);
  __syncthreads();
  if (threadIdx.x == 0) *status = s_flags;
}

// Merges the four waves' records into the output (whole) or into the item's partial record.  SEGMENTS: the item has several
// segments; `before` holds the references and sums of those already merged into the partial record (null: none), `after`
// takes the new ones (null: the last segment, they go to the record).  Elements of the record are written and read again by
// the same thread.
template <int HD, bool SEGMENTS>
__device__ __forceinline__ void merge_records(const MultiArgs& A, const ItemPlan& P, const float* s_rec, bool whole, float* part,
                                              const float2* before, float2* after) {
  const DevBatch& B = A.b[P.b];
  const int G = B.G;
  for (int i = threadIdx.x; i < G * (HD / 2); i += kThreads) {
    const int h = i / (HD / 2), d = 2 * (i % (HD / 2));
    float2 ml0{-INFINITY, 0.f}, v0{0.f, 0.f};
    if constexpr (SEGMENTS) {
      if (before) {
        ml0 = before[h];
        v0 = *reinterpret_cast<const float2*>(part + h * (HD + 2) + d);
      }
    }
    float M = ml0.x;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, s_rec[(w * G + h) * (HD + 2) + HD]);
    float L = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float* pr = s_rec + (w * G + h) * (HD + 2);
      const float2 ml = *reinterpret_cast<const float2*>(pr + HD);
      if (ml.x != -INFINITY) {  // (a wave without tokens left no row; one with a NaN logit has a NaN sum, which goes on)
        const float x = expf(ml.x - M);
        const float2 v = *reinterpret_cast<const float2*>(pr + d);
        L += ml.y * x;
        o0 += v.x * x;
        o1 += v.y * x;
      }
    }
    if constexpr (SEGMENTS) {
      if (before) {
        const float x = expf(ml0.x - M);
        L += ml0.y * x;
        o0 += v0.x * x;
        o1 += v0.y * x;
      }
    }
    if (whole) {
      const float inv = 1.0f / L;
      const int64_t row = (int64_t)P.seq * B.n_q + P.head * G + h;
      const half2v hv = {(_Float16)(o0 * inv), (_Float16)(o1 * inv)};
      *reinterpret_cast<uint32_t*>(B.out + row * HD + d) = h2u(hv);
      if (d == 0 && B.lse) B.lse[row] = M + logf(L);
    } else {
      *reinterpret_cast<float2*>(part + h * (HD + 2) + d) = float2{o0, o1};
      if (d == 0) {
        if (SEGMENTS && after) after[h] = float2{M, L};
        else *reinterpret_cast<float2*>(part + h * (HD + 2) + HD) = float2{M, L};
      }
    }
  }
}

template <int HD>
__global__ __launch_bounds__(kThreads, mfma_wgs_per_cu(HD)) void mfma_direct_kernel(DirectArgs D, uint32_t* status) {
  extern __shared__ uint64_t s_tab[];
  __shared__ float2 s_before[2][16];
  if (blockIdx.x == 0) {
    direct_status(D, status);
    return;
  }
  const MultiArgs& A = D.m;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* s_rec = reinterpret_cast<float*>(s_tab + D.entries);
  ItemPlan P;
  uint32_t local = direct_index(D, blockIdx.x - 1);
  P.b = direct_batch(D, local);
  const DevBatch& B = A.b[P.b];
  const DirectItem item = direct_item(D, P.b, local);
  P.head = item.head;
  P.chunk = item.split;
  P.seq = item.seq;
  P.local = local;
  const int max_len = (int)min((int64_t)B.max_blocks * B.g.T, (int64_t)0x7fffffff);
  const int32_t* table = B.tables + (int64_t)P.seq * B.max_blocks;
  const uint8_t* head_base = B.layer_base + (uint64_t)P.head * B.g.head_chunk;
  const int G = B.G;
  float* rec = s_rec + wave * G * (HD + 2);
  auto record = [&] { return A.partials + D.part_off[P.b] + (uint64_t)item.rec * (uint64_t)A.b[P.b].part_stride; };
  float* part = record();
  DirectRange r{P.chunk * B.chunk_runs, 0};
  bool whole = false;
  // one turn per segment of the item (see direct_segment_end): nearly always one
  for (int turn = 0;; ++turn) {
    // the block-table entries do not wait for the length: the segment's first run, and so its first block, is known
    P.k0 = div_runs(r.v0, B.R, B.r_magic);
    int32_t tab[kEntriesPerThread];
#pragma unroll
    for (int q = 0; q < kEntriesPerThread; ++q) {
      const int i = (int)threadIdx.x + kThreads * q;
      tab[q] = i < D.entries && P.k0 + i < B.max_blocks ? table[P.k0 + i] : 0;
    }
    if (turn == 0) {
      int len = __builtin_amdgcn_readfirstlane(B.seq_lens[P.seq]);
      len = len < 1 ? 1 : min(len, max_len);
      P.len = len;
      const int runs = n_runs(len, B.g.T, B.R);
      r = direct_range(D, P.b, P.chunk, runs);
      if (r.v0 >= r.v1) return;  // (uniform: a split past the sequence's end)
      whole = direct_splits_of(D, P.b, runs) == 1;
    }
    const int end = direct_segment_end(D, P.b, r.v0, r.v1);
    P.nb = div_runs(end - 1, B.R, B.r_magic) - P.k0 + 1;
    const int share = ((end - r.v0 + 3) / 4 + kWaves - 1) / kWaves * 4;  // runs per wave: whole tiles
    P.v0 = r.v0 + wave * share;
    P.v1 = min(end, P.v0 + share);
    if (turn) __syncthreads();  // (every wave is through with the last segment's table and records)
#pragma unroll
    for (int q = 0; q < kEntriesPerThread; ++q) {
      const int i = (int)threadIdx.x + kThreads * q;
      if (i < P.nb) s_tab[i] = reinterpret_cast<uint64_t>(head_base + (uint64_t)checked_block(tab[q], B.n_blocks, A.header) * B.g.block_budget);
    }
    __syncthreads();
    if (P.v0 < P.v1) {  // wave-uniform
      StateT<HD> unused;
      dispatch_item<2, HD>(A, P, s_tab, unused, nullptr, rec);
    } else if (lane < G) {
      *reinterpret_cast<float2*>(rec + lane * (HD + 2) + HD) = float2{-INFINITY, 0.f};
    }
    __syncthreads();
    const bool last = end == r.v1;
    // (Above head_dim 64 the record's place is looked up here: kept over the tiles it pushes out their scalars.  At 64 the smallest
    // calls are faster with it looked up in front: one sequence of 100 tokens 6.05 us, 6.15 like this.)
    if constexpr (HD > 64) {
      asm volatile("" : "+s"(P.b));
      part = record();
    }
    if (turn == 0 && last) merge_records<HD, false>(A, P, s_rec, whole, part, nullptr, nullptr);
    else merge_records<HD, true>(A, P, s_rec, false, part, turn ? s_before[turn & 1] : nullptr, last ? nullptr : s_before[(turn + 1) & 1]);
    if (last) return;
    r.v0 = end;
  }
}

}  // namespace

// Shapes this kernel covers: head_dim 64, 128 or 256, at least 8 tokens per block (a run of 8 slots fits a block),
// and run indices small enough for the multiply-high division by R.
bool mfma_supports(const DevBatch& b) {
  if ((b.g.D != 64 && b.g.D != 128 && b.g.D != 256) || b.g.T < 8 || b.G > 16) return false;
  const uint64_t max_tok = (uint64_t)b.max_blocks * (uint64_t)b.g.T;
  const uint64_t max_run = (uint64_t)b.max_blocks * (uint64_t)b.R + 8;
  return max_tok < (1ull << 31) && max_run * (uint64_t)b.R < (1ull << 32);
}

hipError_t launch_mfma(const MultiArgs& A, int n_workgroups, hipStream_t s) {
  // LDS: per wave one 8-byte address per block of the largest split (+ slack)
  int entries = 0;
  for (int i = 0; i < A.n_batches; ++i) entries = std::max(entries, A.b[i].chunk_runs / A.b[i].R + 4);
  const size_t smem = (size_t)kWaves * entries * sizeof(uint64_t);
  switch (A.b[0].g.D) {  // (the caller checked that all batches share it)
    case 64: hipLaunchKernelGGL(mfma_attention_kernel<64>, dim3(n_workgroups), dim3(kThreads), smem, s, A, entries); break;
    case 128: hipLaunchKernelGGL(mfma_attention_kernel<128>, dim3(n_workgroups), dim3(kThreads), smem, s, A, entries); break;
    default: hipLaunchKernelGGL(mfma_attention_kernel<256>, dim3(n_workgroups), dim3(kThreads), smem, s, A, entries); break;
  }
  return hipGetLastError();
}

hipError_t launch_mfma_direct(const DirectArgs& args, hipStream_t s) {
  DirectArgs D = args;
  int heads = 0;
  uint32_t items = 0;
  for (int i = 0; i < D.m.n_batches; ++i) {
    heads = std::max(heads, (int)D.m.b[i].G);
    items += D.items[i];
  }
  const int hd = D.m.b[0].g.D;
  const size_t smem = (size_t)D.entries * sizeof(uint64_t) + (size_t)kWaves * heads * (hd + 2) * sizeof(float);
  uint32_t* status = D.m.header + kHdrStatus;
  D.m.header += kHdrIgnored - kHdrStatus;
  static_assert(kThreads * ((uint64_t)kDirectMaxItems + 1) < 1ull << 32, "threads of the grid");
  void (*const kern)(DirectArgs, uint32_t*) = hd == 64 ? mfma_direct_kernel<64> : hd == 128 ? mfma_direct_kernel<128> : mfma_direct_kernel<256>;
  if (smem > 64 * 1024) {  // (head_dim 256 with 15 or 16 query heads per KV head: has to be granted per kernel)
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(items + 1), dim3(kThreads), smem, s, D, status);
  return hipGetLastError();
}

}  // namespace fs
