// MFMA paged prefill (chunked prefill) attention kernel for gfx950 (head_dim 64, 128 and 256, all four KV formats).
//
// FineServe Sec. 2.1: the prefill phase processes the prompt's tokens, each attending to the tokens up to
// itself; Sec. 2.3: it is the compute-intensive phase; Sec. 4.2 schedules it in chunks.  Here a chunk's
// keys and values are first appended to the slab pool (fs_kv_append), then every query row of the chunk
// attends to the cached tokens 0..its own position, read from the pool exactly as decode attention reads
// them (same dequantization), through the sequence's block table (Sec. 5.1).
//
// Work decomposition: a work item is (sequence, KV head, tile of query tokens); the 16 logit columns of the
// MFMAs (see fs_mfma_tiles.h) are (query token, query head of the group) pairs, 16 / G tokens per block of 16
// columns.  One wave streams the cached tokens 0 .. last position of the tile once for all its columns;
// causality is a per-column sequence length, so only the tiles on the diagonal pay for masking.  Three kernels:
// prefill_kernel keeps one block of 16 columns per wave (two waves per SIMD); prefill_wide_kernel 2 or 4
// blocks (one wave per SIMD): a tile's K and V rows are then loaded, unpacked and transposed once for 32 or 64
// columns; prefill_wg_kernel (the default at head_dim 64 and 128) lets the waves of a workgroup share every unpacked
// K/V fragment through LDS.  Items of one (sequence, head) are neighbours in the queue (or, in the workgroup kernels,
// a number of heads apart that brings them to the same XCD), longest first, so that the waves streaming the same keys and
// values run side by side and share them through the L2.  Waves draw items from the same pooled ticket counters as the decode kernel.  A long context is
// streamed in segments, the wave's block-address table being refilled per segment.
#include <cstdlib>

// Prefill re-reads every K/V row once per query tile of its (sequence, head) -- from the L2 and the memory-side
// cache after the first time -- so its loads carry no non-temporal hint (decode, which reads every row once, hints
// its V loads; with the hint here config 2's prefill ran 6 % slower, 739 against 783 TFLOP/s on one box).
#define FS_NT_V 0
#include "fs_mfma_tiles.h"
#include "fs_prefill_index.h"

namespace fs {
namespace {

struct PrefillArgs {
  DevBatch b;                // geometry and the batch's pointers (q, tables, seq_lens, out, lse, FP8 scales)
  const int32_t* q_offsets;  // [n_seq + 1] first query row of each sequence's chunk
  uint32_t* header;          // workspace header: status word and the pools' ticket counters (layout of fs_attention.h)
  uint32_t* tile_first;      // [n_seq + 1] first query tile of each sequence
  int32_t tpt;               // query tokens per block of 16 logit columns: 16 / G
  int32_t ncb;               // column blocks per work item (1: prefill_kernel; 2, 4: prefill_wide_kernel)
  int32_t seg_runs;          // runs of 8 token slots streamed per refill of the block-address table (multiple of 4)
  int32_t table_entries;     // LDS table entries per wave
  int32_t n_rows;            // query rows in q / out (host value: every row index is clamped into it)
  int32_t tf_cache;          // workgroup kernels: 1 = tile_first is copied into LDS at kernel start, 2 = every workgroup
                             // scans (and sorts) the sequences itself (see scan_sequences)
  int32_t whole_runs;        // 1 = tokens per block is a multiple of 8: no eight tokens from a multiple of 8 on cross a block
  int32_t seg_tokens;        // workgroup kernels: tokens streamed per refill of the block-address table (multiple of 128)
  uint32_t t_magic;          // workgroup kernels: for the division by the tokens per block (block_of, fs_prefill_index.h)
  int32_t chunk_shift;       // workgroup kernels: log2 of the consecutive work items that go to one XCD
  int32_t kv_shift;          // workgroup kernels: log2 of the groups of waves that share an item's context (merge_groups) ...
  int32_t group_len;         // ... in launches with a sequence of at least this many tokens (see scan_sequences)
  int32_t by_tile;           // workgroup kernels: 1 = items in the order of decode_item_by_tile
  int32_t direct;            // workgroup kernels: 1 = no preparation ran and no tickets are drawn (see "Direct launches")
  int32_t plan_items;        // workgroup kernel with split items: places for items in the plan (a multiple of eight, see SplitPlan)
  uint8_t* pieces;           // ... its counters and partial results in the workspace (see "Split items")
#ifdef FS_TIMELINE
  uint64_t* timeline;        // (timeline build) clock readings of the workgroup kernels, at the end of the workspace
#endif
};

// Timeline build (-DFS_TIMELINE, bench_timeline.py; never the product library): the workgroup kernels leave clock
// readings at the end of the workspace, which fs_prefill_workspace_bytes then includes.  Rows of eight 64-bit words:
// kPfTimelineGroups rows of workgroups (start, end, items, XCD, then the items' summed phases: entry -> address table
// in LDS, -> first sub-tiles staged, -> last step done, -> output written), then kPfTimelineItems rows of work items
// by item index (begin, end, sequence << 32 | KV head << 20 | query tile, workgroup | draw-and-barriers time << 32).
#ifdef FS_TIMELINE
constexpr uint64_t kPfTimelineGroups = 1024, kPfTimelineItems = 1ull << 18;
constexpr uint64_t kPfTimelineBytes = 64 * (kPfTimelineGroups + kPfTimelineItems);
#endif

constexpr int kPrepThreads = 1024;

// Sequence i's clamped length, the query tokens it brings and their first row; raises bit 0 of `flags` for a length or
// chunk out of range.
struct SeqShape {
  int len, n_new, q0;
};
__device__ __forceinline__ SeqShape seq_shape(const PrefillArgs& P, int i, uint32_t& flags) {
  const DevBatch& B = P.b;
  const int max_len = (int)min((int64_t)B.max_blocks * B.g.T, (int64_t)0x7fffffff);
  SeqShape s;
  s.len = B.seq_lens[i];
  s.q0 = P.q_offsets[i];
  s.n_new = P.q_offsets[i + 1] - s.q0;
  if (s.len < 1 || s.len > max_len || s.n_new < 0 || s.n_new > s.len) {
    flags |= 1u;
    s.len = s.len < 1 ? 1 : min(s.len, max_len);
    s.n_new = s.n_new < 0 ? 0 : min(s.n_new, s.len);
  }
  return s;
}
__device__ __forceinline__ uint32_t shape_tiles(const PrefillArgs& P, const SeqShape& s, int ncb) {
  return (uint32_t)((s.n_new + P.tpt * ncb - 1) / (P.tpt * ncb));
}

// Query tiles per sequence -> tile_first (exclusive scan), validation flags, counter reset.  One workgroup.
__global__ __launch_bounds__(kPrepThreads) void prefill_prep_kernel(PrefillArgs P) {
  __shared__ uint32_t s_wave[kPrepThreads / 64];
  __shared__ uint32_t s_running;
  const DevBatch& B = P.b;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) {
    s_running = 0;
    P.header[kHdrStatus] = 0;
  }
  if (tid < kPools) P.header[kHdrPools + tid * kPoolStride] = 0;
  __syncthreads();
  for (int base = 0; base < B.n_seq; base += kPrepThreads) {
    const int i = base + tid;
    uint32_t v = 0;
    if (i < B.n_seq) {
      uint32_t flags = 0;
      v = shape_tiles(P, seq_shape(P, i, flags), P.ncb);
      if (flags) atomicOr(P.header + kHdrStatus, flags);
    }
    if (P.tf_cache == 2) break;  // (one round: every workgroup of the attention kernel scans for itself)
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t t = __shfl_up(incl, off, 64);
      if (lane >= off) incl += t;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    uint32_t before = s_running;
    for (int w = 0; w < wave; ++w) before += s_wave[w];
    if (i < B.n_seq) P.tile_first[i] = before + incl - v;
    __syncthreads();
    if (tid == kPrepThreads - 1) s_running = before + incl;
    __syncthreads();
  }
  if (tid == 0) P.tile_first[B.n_seq] = s_running;
}

template <int DT, int HD = kD>
__device__ void prefill_item(const PrefillArgs& P, int seq, int head, int qt, uint64_t* s_ptr) {
  constexpr int GP = 16;  // every logit column is live: one column per lane in the softmax
  const DevBatch& B = P.b;
  const DevGeom& g = B.g;
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));  // see the decode kernel: keeps lane constants out of the item loop
  const int j = lane >> 4, c = lane & 15;
  const int G = B.G;
  const int max_len = (int)min((int64_t)B.max_blocks * g.T, (int64_t)0x7fffffff);
  int len = B.seq_lens[seq];
  len = len < 1 ? 1 : min(len, max_len);
  int n_new = P.q_offsets[seq + 1] - P.q_offsets[seq];
  n_new = n_new < 0 ? 0 : min(n_new, len);
  const int r0 = qt * P.tpt;              // first query token of the tile within the chunk
  if (r0 >= n_new) return;                // (cannot happen with consistent inputs)
  const int first_pos = len - n_new + r0;  // its position in the sequence
  const int n_tok = min(P.tpt, n_new - r0);
  // column c = (query token c / G of the tile, query head c % G of the group)
  const int tok_c = c / G, hg_c = c - tok_c * G;
  const bool live = tok_c < n_tok;
  const int row_c = min(max(P.q_offsets[seq] + r0 + tok_c, 0), P.n_rows - 1);

  ItemCtx X;
  X.T = g.T;
  X.R = B.R;
  X.r_magic = B.r_magic;
  X.len_u = first_pos + n_tok;                  // the tile's last query sees this many tokens
  X.len = live ? first_pos + tok_c + 1 : 1;     // causality: a column sees the tokens up to its own position
  X.chunk_ptr = s_ptr;

  constexpr int NE = HD / 16;  // output columns NE c .. NE c + NE - 1 are this lane's
  u32x4 qb[HD / 32];
  float qsum;
  load_q<DT, true, HD>(B.q + ((int64_t)row_c * B.n_q + head * G + hg_c) * HD, live, j, qb, qsum);
  if constexpr (Fmt<DT>::kParBytes != 0) {
    qsum += __shfl_xor(qsum, 16, 64);
    qsum += __shfl_xor(qsum, 32, 64);
  }
  float alpha = B.sm_scale * kLog2e;
  if (DT == FS_KV_FP8_E4M3) alpha *= B.k_scale[head];

  StateT<HD> st;
#pragma unroll
  for (int e = 0; e < NE; ++e) st.acc[e] = float4v{0.f, 0.f, 0.f, 0.f};
  st.m = -INFINITY;
  st.l = 0.f;
  st.zc = 0.f;

  const int32_t* table = B.tables + (int64_t)seq * B.max_blocks;
  const uint8_t* head_base = B.layer_base + (uint64_t)head * g.head_chunk;
  const int n_run = n_runs(X.len_u, g.T, B.R);
  for (int v0 = 0; v0 < n_run; v0 += P.seg_runs) {
    X.v_end = min(n_run, v0 + P.seg_runs);
    X.k0 = div_runs(v0, B.R, B.r_magic);
    fill_table(s_ptr, table, head_base, g.block_budget, X.k0, div_runs(X.v_end - 1, B.R, B.r_magic) - X.k0 + 1, lane, B.n_blocks, P.header);
    stream_tiles<DT, GP, HD>(X, g, v0, qb, qsum, alpha, st, j, c);
  }

  // ---- output: per-column sums over the four lane groups, then the live rows straight from the accumulators ----
  st.l += __shfl_xor(st.l, 16, 64);
  st.l += __shfl_xor(st.l, 32, 64);
  if constexpr (Fmt<DT>::kParBytes != 0) {
    st.zc += __shfl_xor(st.zc, 16, 64);
    st.zc += __shfl_xor(st.zc, 32, 64);
  }
  const float v_static = DT == FS_KV_FP8_E4M3 ? B.v_scale[head] : 1.0f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int h = 4 * j + r;  // accumulator row r of this lane is logit column h; its m, l, zc live in lane c = h
    const float L = __shfl(st.l, h, 64), M = __shfl(st.m, h, 64), Z = __shfl(st.zc, h, 64);
    const int row_h = __shfl(row_c, h, 64);
    const int tok_h = h / G, hg_h = h - tok_h * G;
    if (tok_h < n_tok) {
      const float inv = 1.0f / L;
      uint32_t w[NE / 2];
#pragma unroll
      for (int q = 0; q < NE / 2; ++q) {
        float o[2];
#pragma unroll
        for (int z = 0; z < 2; ++z) {
          const int e = 2 * q + z;
          // integer formats: undo the 2^-24 of the subnormal encoding (and the 16 of INT4's odd code positions)
          const float f = DT == FS_KV_INT8 ? kTwo24 : (DT == FS_KV_INT4 ? ((e & 1) ? kTwo20 : kTwo24) : 1.0f);
          o[z] = st.acc[e][r] * f;
          if constexpr (Fmt<DT>::kParBytes != 0) o[z] += Z;
          o[z] *= v_static * inv;
        }
        const half2v hv = {(_Float16)o[0], (_Float16)o[1]};
        w[q] = h2u(hv);
      }
      const int64_t qrow = (int64_t)row_h * B.n_q + head * G + hg_h;
      _Float16* orow = B.out + qrow * HD + NE * c;
      if constexpr (NE == 4) {
        *reinterpret_cast<u32x2*>(orow) = u32x2{w[0], w[1]};
      } else {
#pragma unroll
        for (int q = 0; q < NE / 8; ++q)
          reinterpret_cast<u32x4*>(orow)[q] = u32x4{w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]};
      }
      if (c == 0 && B.lse) B.lse[qrow] = (M + __builtin_amdgcn_logf(L)) * kLn2;
    }
  }
}

// ---------------------------------------------------------------------------------------------------------
// Wide variant: NCB blocks of 16 logit columns per wave.  A tile's K rows are unpacked once and multiplied
// with NCB query operands, its V rows are unpacked and transposed once and multiplied with NCB weight
// operands; per-token parameters are broadcast once.  Only the softmax itself is per block.  The accumulators
// (NCB x 32 registers) take the place of a second resident wave: the kernel runs one wave per SIMD.
// ---------------------------------------------------------------------------------------------------------
// Makes the query operand's loads complete here, once per item.  Their first real use is an MFMA inside the
// tile loop; left pending until there, the compiler's wait-count bookkeeping must assume at the loop head that
// they may still be in flight, and its wait for them also waits for the K/V loads issued just before -- the
// very loads the loop is arranged to keep in flight across a whole step.
template <int KS>
__device__ __forceinline__ void settle_q(u32x4 (&q)[KS]) {
  uint32_t any = 0;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) any |= q[ks][0] | q[ks][1] | q[ks][2] | q[ks][3];
  asm volatile("" ::"v"(any));
}

template <int NCB, int HD = kD>
struct WgState {
  float4v acc[NCB][HD / 16];
  float m[NCB], l[NCB];
};
template <int NCB, int HD = kD>
struct WideState : WgState<NCB, HD> {
  float zc[NCB];  // (parameter formats) this lane's share of the zero-point term
};

// This file is compiled with VGPR-form MFMAs (-mllvm -amdgpu-mfma-vgpr-form, see build.py): accumulators, S^T
// results and operands all live in vector registers and the kernels use no AccVGPRs as MFMA operands.  With the
// default (accumulators in AccVGPRs, which the vector ALU cannot address) every S^T tile had to be read out with
// v_accvgpr_read before the softmax -- 16 of the ~100 vector instructions of a sub-tile -- and the rarely taken
// rescale of the accumulators needed explicit accvgpr moves in inline assembly to keep the register allocator
// from shuttling all of them between the register files on every tile.  256 vector registers per wave (two waves
// per SIMD) hold everything; measured against the AccVGPR build on one machine: + 10-14 % on every format.

// Moves the reference of column block cb (see the lazy online softmax of fs_mfma_tiles.h): tmax = this lane's
// largest logit of the tile for its column.
template <int DT, int NCB, int HD>
__device__ __forceinline__ void wide_move_reference(WideState<NCB, HD>& st, int cb, float tmax, int j) {
  tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
  tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
  const float m_new = fmaxf(st.m[cb], tmax);  // finite: token 0 is seen by every column
  if (__all(st.m[cb] == -INFINITY)) {         // the item's first tile: nothing accumulated yet, nothing to rescale
    st.m[cb] = m_new;
    return;
  }
  const float corr = __builtin_amdgcn_exp2f(st.m[cb] - m_new);
  st.l[cb] *= corr;
  if constexpr (Fmt<DT>::kParBytes != 0) st.zc[cb] *= corr;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float cr = __shfl(corr, 4 * j + r, 64);  // column h keeps its factor in lane c = h
#pragma unroll
    for (int e = 0; e < HD / 16; ++e) st.acc[cb][e][r] *= cr;
  }
  st.m[cb] = m_new;
}

// One 32-token tile for NCB column blocks.  Order of work: all S^T MFMAs; the logits and, on the tiles that
// need it, their masks; the column maxima and one (rare) reference check for all column blocks; per column
// block the exponentials; the P V MFMAs.  A tile is interior when its four runs are whole (8 slots each, none
// repeated) and every column of the item sees all 32 tokens (the tile ends at or before the item's first query
// token): nothing is masked there, and the mask code is one skipped branch that touches no accumulator.
template <int DT, int NCB>
__device__ __forceinline__ void wide_tile(const ItemCtx& X, const DevGeom& g, Tile<DT, 16>& t, const u32x4 (&qb)[NCB][4],
                                          const float (&qsum)[NCB], const int (&len_cb)[NCB], float alpha, int first_pos,
                                          int vb, int vb_next, int j, int c, WideState<NCB>& st) {
  using F = Fmt<DT>;
  // ---- S^T = K Q^T for every column block ----
  float4v s[NCB][2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    u32x4 a[4];
    k_operands<DT>(t.k[u], a);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      float4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) acc = mfma(a[ks], qb[cb][ks], acc);
      s[cb][u] = acc;
    }
  }
  issue_k<DT, 16>(X, vb_next, j, c, t);

  const RunLoc L = locate(X, vb, j);  // X.len == X.len_u here: L.hi == L.hi_u
  const bool interior = __all(L.lo == 0 && L.tok0 + 8 <= first_pos + 1);  // wave-uniform
  // per-token dequantization factors, prepared by the lane that loaded the token's parameters, broadcast once
  float ka[8], kb[8], va[8], vb2[8];
  if constexpr (F::kParBytes != 0) {
    float pa, pb;
    const float sc = f16lo(t.par[0]);
    const float zp = DT == FS_KV_INT4 ? f16hi(t.par[0]) : 128.0f;
    if (c < 8) {  // K: logit = alpha * sc * (2^24 * S_raw - zp * qsum)
      pa = alpha * kTwo24 * sc;
      pb = -alpha * sc * zp;
    } else {      // V: p' = p * sc, zero-point term -p * sc * zp
      const bool ok = (c & 7) >= L.lo && (c & 7) < L.hi_u;  // a slot past the sequence may hold any bit pattern
      pa = ok ? sc : 0.f;
      pb = ok ? -sc * zp : 0.f;
    }
    static_for(std::make_integer_sequence<int, 8>{}, [&](auto I) {
      constexpr int i = decltype(I)::value;
      ka[i] = row_bcast<i>(pa);
      kb[i] = row_bcast<i>(pb);
      va[i] = row_bcast<8 + i>(pa);
      vb2[i] = row_bcast<8 + i>(pb);
    });
  }
  // logits in the base-2 domain (parameter formats) or raw products (FP16, FP8: their one common factor
  // alpha > 0 is applied inside the exponential's argument)
  float x[NCB][8];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float v = s[cb][i >> 2][i & 3];
      if constexpr (F::kParBytes != 0) x[cb][i] = fmaf(v, ka[i], kb[i] * qsum[cb]);
      else x[cb][i] = v;
    }
  if (!interior) {
    if constexpr (DT == FS_KV_FP16 || DT == FS_KV_FP8_E4M3) {
      // slots past the sequence's end may hold NaN/Inf bit patterns; 0 * NaN would poison the MFMA
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int w = 0; w < F::kVBytes / 4; ++w) t.v[i][w] = i < L.hi_u ? t.v[i][w] : 0u;
    }
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const int hi = min(L.hi_u, len_cb[cb] - L.tok0);  // causality: this lane's column sees tokens < len_cb
      const uint32_t n_ok = (uint32_t)max(hi - L.lo, 0);
#pragma unroll
      for (int i = 0; i < 8; ++i) x[cb][i] = (uint32_t)(i - L.lo) < n_ok ? x[cb][i] : -INFINITY;
    }
  }
  // ---- column maxima; the lazily moved reference (see fs_mfma_tiles.h) is checked once for all blocks ----
  float tmax[NCB];
  bool need = false;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    float mx = fmaxf(fmaxf(x[cb][0], x[cb][1]), x[cb][2]);
    mx = fmaxf(fmaxf(mx, x[cb][3]), x[cb][4]);
    mx = fmaxf(fmaxf(mx, x[cb][5]), x[cb][6]);
    mx = fmaxf(mx, x[cb][7]);
    if constexpr (F::kParBytes == 0) mx *= alpha;
    tmax[cb] = mx;
    need |= mx - st.m[cb] > kTau;
  }
  if (__any(need)) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) wide_move_reference<DT>(st, cb, tmax[cb], j);
  }
  // ---- weights ----
  u32x4 pk[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    const float m = st.m[cb];
    if constexpr (F::kParBytes != 0) {
      float p[8], lsum = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float e = __builtin_amdgcn_exp2f(x[cb][i] - m);
        lsum += e;
        p[i] = e * va[i];
        st.zc[cb] = fmaf(e, vb2[i], st.zc[cb]);
      }
      st.l[cb] += lsum;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const half2v h = {(_Float16)p[2 * q], (_Float16)p[2 * q + 1]};
        pk[cb][q] = h2u(h);
      }
    } else {
      // the running sum is taken over the weights as the MFMA sees them (rounded to fp16)
      const half2v one = {(_Float16)1.0f, (_Float16)1.0f};
      float l = st.l[cb];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float e0 = __builtin_amdgcn_exp2f(fmaf(x[cb][2 * q], alpha, -m));
        const float e1 = __builtin_amdgcn_exp2f(fmaf(x[cb][2 * q + 1], alpha, -m));
        const half2v h = {(_Float16)e0, (_Float16)e1};
        pk[cb][q] = h2u(h);
        l = __builtin_amdgcn_fdot2(h, one, l, false);
      }
      st.l[cb] = l;
    }
  }
  // ---- V rows of the run -> B operands (8x8 in-register transpose), out += P V for every column block ----
  uint32_t vx[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i) v_unpack<DT>(t.v[i], vx[i]);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int reg = DT == FS_KV_INT4 ? (e & 3) : (e >> 1);
    const uint32_t sel = (DT == FS_KV_INT4 ? (e >> 2) : (e & 1)) ? 0x07060302u : 0x05040100u;
    u32x4 b;
#pragma unroll
    for (int q = 0; q < 4; ++q) b[q] = __builtin_amdgcn_perm(vx[2 * q + 1][reg], vx[2 * q][reg], sel);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) st.acc[cb][e] = mfma(pk[cb], b, st.acc[cb][e]);
  }
  issue_v<DT, 16>(X, g, vb_next, j, c, t);
}

// One work item of the wide variant: (sequence, KV head, NCB consecutive 16-column query tiles).
template <int DT, int NCB>
__device__ void prefill_item_wide(const PrefillArgs& P, int seq, int head, int qt, uint64_t* s_ptr) {
  const DevBatch& B = P.b;
  const DevGeom& g = B.g;
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int j = lane >> 4, c = lane & 15;
  const int G = B.G;
  const int max_len = (int)min((int64_t)B.max_blocks * g.T, (int64_t)0x7fffffff);
  int len = B.seq_lens[seq];
  len = len < 1 ? 1 : min(len, max_len);
  int n_new = P.q_offsets[seq + 1] - P.q_offsets[seq];
  n_new = n_new < 0 ? 0 : min(n_new, len);
  const int r0 = qt * P.tpt * NCB;  // first query token of the item within the chunk
  if (r0 >= n_new) return;
  const int first_pos = len - n_new + r0;
  const int n_tok = min(P.tpt * NCB, n_new - r0);
  const int tok_c = c / G, hg_c = c - tok_c * G;  // within a column block

  ItemCtx X;
  X.T = g.T;
  X.R = B.R;
  X.r_magic = B.r_magic;
  X.len_u = first_pos + n_tok;
  X.len = X.len_u;
  X.chunk_ptr = s_ptr;

  u32x4 qb[NCB][4];
  float qsum[NCB];
  int len_cb[NCB], row_cb[NCB];
  float alpha = B.sm_scale * kLog2e;
  if (DT == FS_KV_FP8_E4M3) alpha *= B.k_scale[head];
  WideState<NCB> st;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    const int tok = cb * P.tpt + tok_c;  // query token of this lane's column in block cb
    const bool live = tok_c < P.tpt && tok < n_tok;
    len_cb[cb] = live ? first_pos + tok + 1 : X.len_u;  // a dead column (q = 0, never written) sees everything
    row_cb[cb] = min(max(P.q_offsets[seq] + r0 + tok, 0), P.n_rows - 1);
    load_q<DT>(B.q + ((int64_t)row_cb[cb] * B.n_q + head * G + hg_c) * kD, live, j, qb[cb], qsum[cb]);
    settle_q(qb[cb]);
    if constexpr (Fmt<DT>::kParBytes != 0) {
      qsum[cb] += __shfl_xor(qsum[cb], 16, 64);
      qsum[cb] += __shfl_xor(qsum[cb], 32, 64);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) st.acc[cb][e] = float4v{0.f, 0.f, 0.f, 0.f};
    st.m[cb] = -INFINITY;
    st.l[cb] = 0.f;
    st.zc[cb] = 0.f;
  }

  const int32_t* table = B.tables + (int64_t)seq * B.max_blocks;
  const uint8_t* head_base = B.layer_base + (uint64_t)head * g.head_chunk;
  const int n_run = n_runs(X.len_u, g.T, B.R);
  constexpr int NBUF = Fmt<DT>::kRing;
  for (int v0 = 0; v0 < n_run; v0 += P.seg_runs) {
    X.v_end = min(n_run, v0 + P.seg_runs);
    X.k0 = div_runs(v0, B.R, B.r_magic);
    fill_table(s_ptr, table, head_base, g.block_budget, X.k0, div_runs(X.v_end - 1, B.R, B.r_magic) - X.k0 + 1, lane, B.n_blocks, P.header);
    // the ring of stream_tiles (fs_mfma_tiles.h), with the wide tile step
    const int n_tiles = (X.v_end - v0 + 3) >> 2;
    Tile<DT, 16> t[NBUF];
    static_for(std::make_integer_sequence<int, NBUF>{}, [&](auto Bi) {
      constexpr int bi = decltype(Bi)::value;
      issue_k<DT, 16>(X, v0 + bi * 4, j, c, t[bi]);
      issue_v<DT, 16>(X, g, v0 + bi * 4, j, c, t[bi]);
    });
    for (int k0 = 0; k0 < n_tiles; k0 += NBUF) {
      static_for(std::make_integer_sequence<int, NBUF>{}, [&](auto Bi) {
        constexpr int bi = decltype(Bi)::value;
        const int vb = v0 + (k0 + bi) * 4;
        wide_tile<DT, NCB>(X, g, t[bi], qb, qsum, len_cb, alpha, first_pos, vb, vb + NBUF * 4, j, c, st);
      });
    }
  }

  const float v_static = DT == FS_KV_FP8_E4M3 ? B.v_scale[head] : 1.0f;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    float l = st.l[cb], zc = st.zc[cb];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if constexpr (Fmt<DT>::kParBytes != 0) {
      zc += __shfl_xor(zc, 16, 64);
      zc += __shfl_xor(zc, 32, 64);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int h = 4 * j + r;  // accumulator row r of this lane is logit column h of block cb
      const float L = __shfl(l, h, 64), M = __shfl(st.m[cb], h, 64), Z = __shfl(zc, h, 64);
      const int row_h = __shfl(row_cb[cb], h, 64);
      const int tok_h = h / G, hg_h = h - tok_h * G;
      if (tok_h < P.tpt && cb * P.tpt + tok_h < n_tok) {
        const float inv = 1.0f / L;
        u32x4 w;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float o[2];
#pragma unroll
          for (int z = 0; z < 2; ++z) {
            const int e = 2 * q + z;
            const float f = DT == FS_KV_INT8 ? kTwo24 : (DT == FS_KV_INT4 ? ((e & 1) ? kTwo20 : kTwo24) : 1.0f);
            o[z] = st.acc[cb][e][r] * f;
            if constexpr (Fmt<DT>::kParBytes != 0) o[z] += Z;
            o[z] *= v_static * inv;
          }
          const half2v hv = {(_Float16)o[0], (_Float16)o[1]};
          w[q] = h2u(hv);
        }
        const int64_t qrow = (int64_t)row_h * B.n_q + head * G + hg_h;
        *reinterpret_cast<u32x4*>(B.out + qrow * kD + 8 * c) = w;
        if (c == 0 && B.lse) B.lse[qrow] = (M + __builtin_amdgcn_logf(L)) * kLn2;
      }
    }
  }
}

// Which items a ticket pool holds.  The query tiles of one (sequence, KV head) stream the same keys and values,
// and each of the chip's eight XCDs has an L2 of its own: a pair's tiles must run on ONE XCD, side by side, for
// its K/V to be fetched from memory once instead of once per XCD (measured on a 0.58 GB cache: 36 GB fetched
// per launch with the tiles dealt round-robin over all XCDs).  The item list (sequence-major, then head, then
// tile) is therefore cut into chunks of consecutive items, chunk k belongs to XCD k % 8, and the 8
// pools of an XCD (pool = 8 s + xcd) take that XCD's items s, s + 8, ... in order.  A wave's home pool is one
// of its own XCD's (the XCC_ID hardware register says which); pools of other XCDs are only visited when the
// home pool has run dry, at the end of the launch.
static_assert(kPools == 64, "pool = 8 * sub-pool + XCD");
// chunk = 2^shift items = the workers resident per XCD (wave-level items: 128 waves, workgroup-level items: 32)
constexpr uint32_t kWaveChunkShift = 7, kWgChunkShift = 5;
__device__ __forceinline__ uint32_t home_pool(uint32_t worker) {  // worker: index among the workers of its XCD
  const uint32_t xcd = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7;  // hwreg(HW_REG_XCC_ID, 0, 4)
  return (worker & 7) * 8 + xcd;
}

// tf: tile_first, in global memory or its copy in LDS (ten dependent look-ups: a round trip to memory each otherwise)
__device__ __forceinline__ bool decode_item(const PrefillArgs& P, const uint32_t* tf, uint32_t item, uint32_t H, int& seq,
                                            int& head, int& qt) {
  return fs::decode_item(tf, P.b.n_seq, item, H, seq, head, qt);
}

// Drawing work items until none is left.  A wave first empties its home pool; after that it looks at all 64
// counters at once (lane p reads pool p's), moves to a pool that still holds items -- one of its own XCD's if
// there is one -- and goes on.  It leaves only when every pool is past its last item, so every item is taken
// whatever the grid size and wherever the workgroups landed.  The next ticket is drawn before the current item
// is processed.
struct ItemDraw {
  uint32_t pool, ticket;
};
__device__ __forceinline__ ItemDraw first_draw(uint32_t* header, uint32_t worker, int lane) {
  ItemDraw d{home_pool(worker), 0u};
  if (lane == 0) d.ticket = atomicAdd(header + kHdrPools + d.pool * kPoolStride, 1u);
  return d;
}
// The drawn item (and the next ticket drawn), or false when every pool is empty.
__device__ __forceinline__ bool next_item(ItemDraw& d, uint32_t* header, uint32_t total, uint32_t shift, int lane,
                                          uint32_t& item) {
  for (;;) {
    item = pool_item(d.pool, __builtin_amdgcn_readfirstlane(d.ticket), shift);
    if (item < total) break;
    const uint32_t cnt = __hip_atomic_load(header + kHdrPools + lane * kPoolStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint64_t left = __ballot(pool_item((uint32_t)lane, cnt, shift) < total);  // wave-uniform; counters only grow
    if (left == 0) return false;
    const uint64_t own = left & (0x0101010101010101ull << (d.pool & 7));
    if (own) left = own;
    const uint32_t r = (d.pool + 1) & 63;  // the first such pool after the current one, cyclically
    const uint64_t rot = r ? (left >> r) | (left << (64 - r)) : left;
    d.pool = (r + (uint32_t)__builtin_ctzll(rot)) & 63;
    if (lane == 0) d.ticket = atomicAdd(header + kHdrPools + d.pool * kPoolStride, 1u);
  }
  if (lane == 0) d.ticket = atomicAdd(header + kHdrPools + d.pool * kPoolStride, 1u);
  return true;
}

// One kernel per KV format: the model's format is known at launch, and a kernel that holds a single format's
// tile code leaves the register allocator a far smaller problem than a run-time switch over all four.
// WPS = waves per SIMD the kernel is built for (its register budget: 512 / WPS).  (Measured: a second wave of the
// 32-column kernel gains nothing; its loads already saturate the compute unit's vector memory pipeline.)
template <int DT, int NCB, int WPS>
__global__ __launch_bounds__(kThreads, WPS) void prefill_wide_kernel(PrefillArgs P) {
  extern __shared__ uint64_t smem64[];
  const DevBatch& B = P.b;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint64_t* s_ptr = smem64 + (size_t)wave * P.table_entries;
  const uint32_t H = (uint32_t)B.g.H;
  const uint32_t total = P.tile_first[B.n_seq] * H;
  ItemDraw d = first_draw(P.header, (blockIdx.x >> 3) * kWaves + wave, lane);
  for (uint32_t item; next_item(d, P.header, total, kWaveChunkShift, lane, item);) {
    int seq, head, qt;
    if (!decode_item(P, P.tile_first, item, H, seq, head, qt)) continue;
    prefill_item_wide<DT, NCB>(P, seq, head, qt, s_ptr);
  }
}

// ---------------------------------------------------------------------------------------------------------
// Workgroup variant.  Counters of the wave-level kernels show the compute unit's vector memory pipeline busy
// 92 % of the time: every wave fetches every K/V byte of its item itself, four times per compute unit.  Here
// the four waves of a workgroup take four neighbouring query tiles (64 logit columns each) of one (sequence,
// KV head) and walk the keys and values together, 128 tokens per step: wave w fetches sub-tile w (32 tokens) of
// the step, unpacks it, transposes its V rows, and leaves the finished MFMA operand fragments -- exactly what
// it would have fed its own MFMAs -- in LDS; after a barrier every wave multiplies all four sub-tiles from
// LDS.  Global loads, unpacking and transposes per wave drop to a quarter; the fragments are written and read
// lane-contiguously (16 bytes per lane), free of bank conflicts.  Two stages alternate, so one barrier per
// step suffices: a stage is rewritten only after the barrier that follows its last readers.
// Stage layout: K fragments [sub-tile][u][k-step][lane] 16 B, V fragments [sub-tile][e][lane] 16 B, per token of the
// parameter formats two factors [sub-tile][K, V][32] 4 B (the pipelined kernel: parameters [sub-tile][lane] 4 B).
constexpr uint32_t kFrag = 64 * 16;  // one operand fragment of a wave
// K (and V) fragments of a sub-tile: two 16-token halves x HD / 32 k-steps (HD / 16 groups of 16 output columns)
constexpr int frags(int hd) { return hd / 16; }
// a stage of SUBS sub-tiles: K fragments, V fragments (8 KiB per sub-tile each at head_dim 128), parameters
constexpr uint32_t stage_v(int subs, int hd = kD) { return (uint32_t)(subs * frags(hd)) * kFrag; }
constexpr uint32_t stage_par(int subs, int hd = kD) { return 2 * stage_v(subs, hd); }
constexpr uint32_t stage_bytes(int subs, int hd = kD) { return stage_par(subs, hd) + (uint32_t)subs * 256; }
constexpr uint32_t kWgCtlBytes = 16;

template <int DT, int HD>
__device__ __forceinline__ void stage_k(uint8_t* stage, int sub, int lane, Tile<DT, 16, HD>& t) {  // (K fragments lead the stage)
  constexpr int KS = HD / 32;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    u32x4 a[KS];
    k_operands<DT, HD>(t.k[u], a);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      *reinterpret_cast<u32x4*>(stage + (uint32_t)(((sub * 2 + u) * KS + ks) * kFrag) + lane * 16) = a[ks];
  }
}
template <int DT, int SUBS, int HD>
__device__ __forceinline__ void stage_v(uint8_t* stage, int sub, int lane, bool clear, int live, Tile<DT, 16, HD>& t) {
  using F = Fmt<DT, HD>;
  if constexpr (DT == FS_KV_FP16 || DT == FS_KV_FP8_E4M3) {
    // slots past the sequence's end may hold NaN/Inf bit patterns; 0 * NaN would poison the MFMA
    if (clear) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int q = 0; q < F::kVWords; ++q) t.v[i][q] = i < live ? t.v[i][q] : 0u;
    }
  }
  uint32_t vx[8][F::kVRegs];
#pragma unroll
  for (int i = 0; i < 8; ++i) v_unpack<DT, HD>(t.v[i], vx[i]);
#pragma unroll
  for (int e = 0; e < F::kNE; ++e) {
    const int reg = DT == FS_KV_INT4 ? 4 * (e >> 3) + (e & 3) : (e >> 1);
    const uint32_t sel = (DT == FS_KV_INT4 ? ((e >> 2) & 1) : (e & 1)) ? 0x07060302u : 0x05040100u;
    u32x4 b;
#pragma unroll
    for (int q = 0; q < 4; ++q) b[q] = __builtin_amdgcn_perm(vx[2 * q + 1][reg], vx[2 * q][reg], sel);
    *reinterpret_cast<u32x4*>(stage + stage_v(SUBS, HD) + (uint32_t)((sub * F::kNE + e) * kFrag) + lane * 16) = b;
  }
  if constexpr (F::kParBytes != 0) *reinterpret_cast<uint32_t*>(stage + stage_par(SUBS, HD) + sub * 256 + lane * 4) = t.par[0];
}

// ---- Staged dequantization (INT8 / INT4) ----------------------------------------------------------------------
// The staging wave may as well leave *dequantized* fp16 operands in LDS: (code - zero point) * scale, rounded to
// fp16 -- what an engine that dequantizes in front of its matrix cores feeds them.  Every consumer wave then runs
// the FP16 tile code (no per-logit scale, no zero-point terms: less than half the vector instructions per logit),
// and the conversion is paid once per workgroup instead of once per wave.  The codes are made exact fp16
// integers first (0x6400 | n = 1024 + n); the offset and the (integer) zero point are subtracted exactly, the
// multiplication by the scale rounds once (relative 2^-12).
__device__ __forceinline__ half2v splat_lo(uint32_t w) { return u2h(__builtin_amdgcn_perm(w, w, 0x01000100u)); }
__device__ __forceinline__ half2v splat_hi(uint32_t w) { return u2h(__builtin_amdgcn_perm(w, w, 0x03020302u)); }

// per-token constants of the dequantization: par = {scale, zero point} (INT4) or {scale} (INT8).  The INT4 zero
// point is an integer 0..15 (the quantizer rounds it), so 1024 + zp and 1024 + 16 zp are exact in fp16 and the
// offset of the integer encoding and the zero point leave in ONE exact subtraction.
template <int DT>
struct Deq {
  half2v sc, sc16, off, off16;
  __device__ __forceinline__ explicit Deq(uint32_t par) {
    const half2v c16 = {(_Float16)16.0f, (_Float16)16.0f}, r16 = {(_Float16)0.0625f, (_Float16)0.0625f};
    const half2v k1024 = {(_Float16)1024.0f, (_Float16)1024.0f}, k1152 = {(_Float16)1152.0f, (_Float16)1152.0f};
    sc = splat_lo(par);
    sc16 = sc * r16;
    if constexpr (DT == FS_KV_INT4) {
      const half2v zp = splat_hi(par);
      off = zp + k1024;
      off16 = zp * c16 + k1024;
    } else {
      off = k1152;  // 1024 + 128: the stored byte is the code + 128 after the sign flip
      off16 = k1152;
    }
  }
};

// Four registers of 8 stored codes -> (code - zp) * scale as packed fp16 (the subtraction exact, the product
// rounded once).  INT8: register p holds elements (2p, 2p + 1).  INT4: register p holds codes (p, p + 4); the odd
// registers hold them 16-fold (the nibble stays where it is stored), which the scale / 16 takes out again: every
// position ends up a plain value, with fp16's whole range.
template <int DT>
__device__ __forceinline__ void dequant8(const uint32_t* w, const Deq<DT>& q, uint32_t (&x)[4]) {
  if constexpr (DT == FS_KV_INT8) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t u = w[h] ^ 0x80808080u;  // code + 128, unsigned
      const uint32_t r0 = __builtin_amdgcn_perm(0x64646464u, u, 0x04010400u);  // halves 1024 + 128 + code
      const uint32_t r1 = __builtin_amdgcn_perm(0x64646464u, u, 0x04030402u);
      x[2 * h] = h2u((u2h(r0) - q.off) * q.sc);
      x[2 * h + 1] = h2u((u2h(r1) - q.off) * q.sc);
    }
  } else {
    const uint32_t w0 = w[0], w8 = w0 >> 8;
    const uint32_t r0 = (w0 & 0x000F000Fu) | 0x64006400u, r1 = (w0 & 0x00F000F0u) | 0x64006400u;  // 1024 + n, 1024 + 16 n
    const uint32_t r2 = (w8 & 0x000F000Fu) | 0x64006400u, r3 = (w8 & 0x00F000F0u) | 0x64006400u;
    x[0] = h2u((u2h(r0) - q.off) * q.sc);
    x[1] = h2u((u2h(r1) - q.off16) * q.sc16);
    x[2] = h2u((u2h(r2) - q.off) * q.sc);
    x[3] = h2u((u2h(r3) - q.off16) * q.sc16);
  }
}

// ---- Token-addressed fetch of the workgroup kernels --------------------------------------------------------------------
// A sub-tile is 32 consecutive tokens of the sequence, wherever its blocks end: blocks of 60 or 31 tokens cost no repeated
// slots, no masks for them and no look-up of a run's place in every wave that multiplies the sub-tile (the wave-level kernels
// walk runs of eight slots that never cross a block).  The fetching lane pays: a row of K has its own block, and the eight
// rows of V may come from two.  Rows past the segment's last token are that token's again where blocks are no multiple of
// eight tokens; otherwise eight slots are always inside a block.  Either way those of V are cleared when they are staged.
// (us: 32 INT4 prompts of 512 - 4096 tokens in blocks of 60, GQA 4:1, 2273 -> 1946; 12 multi-head ones of 300 - 3000 in blocks
// of 46 720 -> 599; FP8 ones in blocks of 25 804 -> 542; 8 INT8 prompts of 2000 - 6000, GQA 8:1, blocks of 31, 2933 -> 2577;
// blocks of 16 or 32 tokens the same within 1 %.)
struct TokenCtx {
  const uint64_t* ptr;  // LDS: addresses of the blocks' layers from the segment's first block on
  uint64_t base_off;    // of the KV head
  int rel0;             // the segment's first token within its first block
  int last;             // the segment's last token, counted from its first one
  int T;
  uint32_t magic;
};
struct TokenPlace {
  gptr base;  // the head's chunk in the token's block
  int k, slot;
};
__device__ __forceinline__ TokenPlace place_token(const TokenCtx& X, int t) {
  TokenPlace p;
  const int rel = X.rel0 + t;
  p.k = block_of(rel, X.T, X.magic);
  p.slot = rel - p.k * X.T;
  p.base = (gptr)(X.ptr[p.k] + X.base_off);
  return p;
}

// K rows of the sub-tile from token tb of the segment on: row c of half-tile u is token 8 (c / 4) + 4 u + c % 4.
// kpar (PAR): their parameters
template <int DT, int HD, bool PAR>
__device__ __forceinline__ void fetch_k(const TokenCtx& X, const DevGeom& g, bool whole, int tb, int j, int c, Tile<DT, 16, HD>& t,
                                        uint32_t (&kpar)[2]) {
  using F = Fmt<DT, HD>;
  typedef typename KVec<F::kKLane>::type kvec;
  auto row = [&](const TokenPlace& p, int u) {
    const gptr at = p.base + (uint32_t)(p.slot * F::kRowBytes) + F::kKLane * j;
#pragma unroll
    for (int s = 0; s < F::kKLoads; ++s) t.k[u][s] = *reinterpret_cast<const FS_GLOBAL kvec*>(at + 4 * F::kKLane * s);
    if constexpr (PAR) {
      const gptr pp = p.base + 2u * g.kv_tile + (uint32_t)(p.slot * F::kParBytes);
      if constexpr (F::kParBytes == 2) kpar[u] = *reinterpret_cast<const FS_GLOBAL uint16_t*>(pp);
      else kpar[u] = *reinterpret_cast<const FS_GLOBAL uint32_t*>(pp);
    }
  };
  const int run = tb + 8 * (c >> 2);
  if (whole) {  // (uniform)
    TokenPlace p = place_token(X, min(run, X.last & ~7));
    p.slot += c & 3;
    row(p, 0);
    p.slot += 4;
    row(p, 1);
  } else {
#pragma unroll
    for (int u = 0; u < 2; ++u) row(place_token(X, min(run + 4 * u + (c & 3), X.last)), u);
  }
}

// V rows of the sub-tile: lane j takes tokens 8 j .. 8 j + 7; and its parameters: lane c those of token c % 8, K for c < 8
// (dequantizing staging does not use them), V for the others.
template <int DT, int HD>
__device__ __forceinline__ void fetch_v(const TokenCtx& X, const DevGeom& g, bool whole, int tb, int j, int c, Tile<DT, 16, HD>& t) {
  using F = Fmt<DT, HD>;
  const int run = tb + 8 * j;
  const RunRows R = run_rows(X.rel0, X.last, X.T, X.magic, run, whole);
  const TokenPlace p{(gptr)(X.ptr[R.k] + X.base_off), R.k, R.slot};
  if constexpr (F::kParBytes != 0) {  // parameters first: they are needed before the rows
    TokenPlace o = p;
    if (whole) o.slot += c & 7;
    else o = place_token(X, min(run + (c & 7), X.last));
    const gptr pp = o.base + 2u * g.kv_tile + ((c >> 3) ? g.par_tile : 0u) + (uint32_t)(o.slot * F::kParBytes);
    if constexpr (F::kParBytes == 2) t.par[0] = *reinterpret_cast<const FS_GLOBAL uint16_t*>(pp);
    else t.par[0] = *reinterpret_cast<const FS_GLOBAL uint32_t*>(pp);
  }
  const gptr p0 = p.base + g.kv_tile + (uint32_t)(p.slot * F::kRowBytes) + c * F::kVBytes;
  if (whole || __all(R.left >= 8 && R.most >= 7)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) load_v_row<DT, HD>(p0 + i * F::kRowBytes, t.v[i]);
  } else {
    const gptr p1 = (gptr)(X.ptr[R.k1] + X.base_off) + g.kv_tile + c * F::kVBytes - (uint32_t)(R.left * F::kRowBytes);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = min(i, R.most);
      load_v_row<DT, HD>((r < R.left ? p0 : p1) + (uint32_t)(r * F::kRowBytes), t.v[i]);
    }
  }
}

template <int DT>
__device__ __forceinline__ void stage_k_deq(uint8_t* stage, int sub, int lane, Tile<DT, 16>& t, const uint32_t (&kpar)[2]) {
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const Deq<DT> q(kpar[u]);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      // the 8 codes of k-step ks: INT8 two dwords of load ks >> 1, INT4 dword ks of the one load
      uint32_t w[2];
      if constexpr (DT == FS_KV_INT8) {
        w[0] = t.k[u][ks >> 1][2 * (ks & 1)];
        w[1] = t.k[u][ks >> 1][2 * (ks & 1) + 1];
      } else {
        w[0] = t.k[u][0][ks];
        w[1] = 0u;
      }
      uint32_t x[4];
      dequant8<DT>(w, q, x);
      const u32x4 a = {x[0], x[1], x[2], x[3]};
      *reinterpret_cast<u32x4*>(stage + (uint32_t)((sub * 8 + u * 4 + ks) * kFrag) + lane * 16) = a;
    }
  }
}

template <int DT, int SUBS>
__device__ __forceinline__ void stage_v_deq(uint8_t* stage, int sub, int lane, bool clear, int live, Tile<DT, 16>& t) {
  uint32_t vx[8][4];
  static_for(std::make_integer_sequence<int, 8>{}, [&](auto I) {
    constexpr int i = decltype(I)::value;
    // V parameters of slot i of the lane's run: held by lane 8 + i of the row
    const uint32_t par = __builtin_amdgcn_update_dpp(0u, t.par[0], 0x150 + 8 + i, 0xF, 0xF, false);
    const Deq<DT> q(par);
    dequant8<DT>(t.v[i], q, vx[i]);
  });
  // slots past the sequence's end may hold any codes and parameters (NaN / Inf after the conversion); 0 * NaN
  // would poison the MFMA
  if (clear) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) vx[i][q] = i < live ? vx[i][q] : 0u;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int reg = DT == FS_KV_INT4 ? (e & 3) : (e >> 1);
    const uint32_t sel = (DT == FS_KV_INT4 ? (e >> 2) : (e & 1)) ? 0x07060302u : 0x05040100u;
    u32x4 b;
#pragma unroll
    for (int q = 0; q < 4; ++q) b[q] = __builtin_amdgcn_perm(vx[2 * q + 1][reg], vx[2 * q][reg], sel);
    *reinterpret_cast<u32x4*>(stage + stage_v(SUBS) + (uint32_t)((sub * 8 + e) * kFrag) + lane * 16) = b;
  }
}

// ---- Staged integers (INT8 / INT4 where the codes stay exact) ---------------------------------------------------------
// The staging wave leaves code - zero point in LDS, an integer that fp16 holds exactly (INT4's odd code positions 16-fold:
// the query operand and the output take that out), and per token the two factors that remain, alpha times K's scale and V's
// scale, as floats.  A consumer multiplies a logit by the one and a weight by the other; there is no zero-point term on
// either side and nothing to broadcast between lanes (16 bytes of four tokens' factors per load).  With codes consumed as
// subnormals, offsets as rank-1 terms and parameters broadcast by DPP a sub-tile of two blocks took 72 vector instructions
// more.  (us: 24 INT8 prompts of 256 - 3000 tokens at head_dim 64, GQA 4:1, 869 -> 656, INT4 878 -> 683; three INT8 prompts
// of 500 - 700 at 128 40.8 -> 34.2; and the results are as near the definition as FP16's, 2.4e-4 where they were 3.8 - 5e-4.  At
// head_dim 256, where four waves stage everything, one INT4 prompt of 900 tokens lost 3 % by it, and is at 44.8 where it was 48.5
// before the accumulators were transposed.)
template <int DT>
__device__ __forceinline__ void int_codes(uint32_t w, half2v off, half2v off16, uint32_t (&x)[4]) {
  if constexpr (DT == FS_KV_INT8) {  // two registers: elements (0, 1), (2, 3)
    const uint32_t u = w ^ 0x80808080u;  // code + 128, unsigned
    x[0] = h2u(u2h(__builtin_amdgcn_perm(0x64646464u, u, 0x04010400u)) - off);  // 1024 + 128 + code
    x[1] = h2u(u2h(__builtin_amdgcn_perm(0x64646464u, u, 0x04030402u)) - off);
  } else {  // four: codes (p, p + 4), 16-fold in the odd ones
    const uint32_t w8 = w >> 8;
    x[0] = h2u(u2h((w & 0x000F000Fu) | 0x64006400u) - off);
    x[1] = h2u(u2h((w & 0x00F000F0u) | 0x64006400u) - off16);
    x[2] = h2u(u2h((w8 & 0x000F000Fu) | 0x64006400u) - off);
    x[3] = h2u(u2h((w8 & 0x00F000F0u) | 0x64006400u) - off16);
  }
}

template <int DT, int HD>
__device__ __forceinline__ void stage_k_int(uint8_t* stage, int sub, int lane, Tile<DT, 16, HD>& t, const uint32_t (&kpar)[2]) {
  constexpr int KS = HD / 32, W = Fmt<DT, HD>::kKLane / 4;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const Deq<DT> q(kpar[u]);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint32_t x[4];
      if constexpr (DT == FS_KV_INT8) {
        uint32_t y[4];
        int_codes<DT>(t.k[u][ks >> 1][2 * (ks & 1)], q.off, q.off16, x);
        int_codes<DT>(t.k[u][ks >> 1][2 * (ks & 1) + 1], q.off, q.off16, y);
        x[2] = y[0];
        x[3] = y[1];
      } else {
        int_codes<DT>(t.k[u][ks / W][ks % W], q.off, q.off16, x);
      }
      *reinterpret_cast<u32x4*>(stage + (uint32_t)(((sub * 2 + u) * KS + ks) * kFrag) + lane * 16) = u32x4{x[0], x[1], x[2], x[3]};
    }
  }
}

// live: as in stage_v (slots past the end may hold any codes and parameters)
template <int DT, int SUBS, int HD>
__device__ __forceinline__ void stage_v_int(uint8_t* stage, int sub, int lane, bool clear, int live, float alpha, Tile<DT, 16, HD>& t) {
  using F = Fmt<DT, HD>;
  constexpr int kPer = DT == FS_KV_INT8 ? 2 : 4;  // registers a word unpacks to
  uint32_t vx[8][kPer * F::kVWords];
  static_for(std::make_integer_sequence<int, 8>{}, [&](auto I) {
    constexpr int i = decltype(I)::value;
    const Deq<DT> q(__builtin_amdgcn_update_dpp(0u, t.par[0], 0x150 + 8 + i, 0xF, 0xF, false));
#pragma unroll
    for (int w = 0; w < F::kVWords; ++w) {
      uint32_t x[4];
      int_codes<DT>(t.v[i][w], q.off, q.off16, x);
#pragma unroll
      for (int z = 0; z < kPer; ++z) vx[i][kPer * w + z] = x[z];
    }
  });
  if (clear) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int q = 0; q < kPer * F::kVWords; ++q) vx[i][q] = i < live ? vx[i][q] : 0u;
  }
#pragma unroll
  for (int e = 0; e < F::kNE; ++e) {
    const int reg = DT == FS_KV_INT4 ? 4 * (e >> 3) + (e & 3) : (e >> 1);
    const uint32_t sel = (DT == FS_KV_INT4 ? ((e >> 2) & 1) : (e & 1)) ? 0x07060302u : 0x05040100u;
    u32x4 b;
#pragma unroll
    for (int q = 0; q < 4; ++q) b[q] = __builtin_amdgcn_perm(vx[2 * q + 1][reg], vx[2 * q][reg], sel);
    *reinterpret_cast<u32x4*>(stage + stage_v(SUBS, HD) + (uint32_t)((sub * F::kNE + e) * kFrag) + lane * 16) = b;
  }
  // the factors of token 8 j + c % 8: [K 32][V 32] floats
  const int j = lane >> 4, c = lane & 15;
  const float sc = f16lo(t.par[0]);
  const float f = c < 8 ? alpha * sc : ((c & 7) < live ? sc : 0.f);
  *reinterpret_cast<float*>(stage + stage_par(SUBS, HD) + sub * 256 + (c >> 3) * 128 + (8 * j + (c & 7)) * 4) = f;
}

// Column c's value combined over the four lanes j that hold its tokens (every lane of the column gets the result).
template <typename Op>
__device__ __forceinline__ float over_column(float x, Op op) {
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
  const u2 a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const u2 b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// The workgroup kernel keeps its accumulators transposed (rows = output elements, columns = logit columns): the V fragment is
// the A operand, the weights are the B operand.  A lane then holds elements of its own column only, the one whose logits it
// exponentiates, and moving the reference is a maximum over four lanes (row swaps on the vector ALU) and plain
// multiplications.  With the weights as the A operand a lane held four other columns, and the maximum and the factors came
// through LDS, three dependent round trips while the other waves waited at the step's barrier; and in most of an item's first
// sub-tiles some column of a wave moves its reference.  Each block of 16 columns moves on its own.  (us: 64 FP16 prompts of
// 512 - 4096 tokens, GQA 4:1, 3920 -> 3801; 32 such INT4 prompts 2369 -> 2271; 24 FP16 prompts of 256 - 3000 tokens at
// head_dim 64 625 -> 576; one of 777 tokens 27.7 -> 26.2.  A wider window than 2^kTau saves another 1 - 3 %, but the largest
// weights of a row are then no longer near 1, where fp16 holds them exactly, and the results are 6 - 14 % further from
// the definition.  Weights first and a check on their sum in the place of the maxima: slower wherever references move.)
// A little less than kTau: with it, blocks that move alone left results 0.5 % further from the definition than blocks that
// moved together (1 % of the time).
constexpr float kTauBlock = 2.5f;
template <int NCB, int HD>
__device__ __forceinline__ void wg_move_reference(WgState<NCB, HD>& st, int cb, float tmax) {
  const float m_new = fmaxf(st.m[cb], over_column(tmax, [](float a, float b) { return fmaxf(a, b); }));
  const float corr = __builtin_amdgcn_exp2f(st.m[cb] - m_new);
  st.l[cb] *= corr;
#pragma unroll
  for (int e = 0; e < HD / 16; ++e)
#pragma unroll
    for (int r = 0; r < 4; ++r) st.acc[cb][e][r] *= corr;
  st.m[cb] = m_new;
}

// One staged 32-token sub-tile for the wave's column blocks: wide_tile with the operands read from LDS.
// VPRE: V fragments requested in front of the softmax (registers permitting)
// SUM32: the running sum of an FP16 / FP8 column takes the weights before they are rounded to fp16 (twice the
// instructions of the dot product with ones), as the 16-column kernel does: for launches that kernel served before
// CUT: values of tokens that no column of a block sees do not reach the block's MFMAs: an Inf or NaN among them (an fp32
// value above 65504 is one in FP16) would turn weight 0 into NaN, in rows up to a sub-tile ahead of its token.  A tile code of
// its own for the sub-tiles on the diagonal: as a branch in the common one it cost a prompt of 777 tokens 27.4 -> 31.4 us.
template <int DT, int NCB, int SUBS, int VPRE, int HD, bool SUM32, bool CUT = false>
__device__ __forceinline__ void wg_tile(const uint8_t* stage, int sub, int tb, const u32x4 (&qb)[NCB][HD / 32],
                                        const int (&len_cb)[NCB], float alpha, int first_pos,
                                        int lane, int j, int c, WgState<NCB, HD>& st, int tpt = 0, int n_tok = 0) {
  using F = Fmt<DT, HD>;
  constexpr int KS = HD / 32;
  float4v s[NCB][2];
  // The wave raises its priority for its MFMA sections and drops it for the softmax: of the two waves of a SIMD
  // the one that feeds the matrix pipe goes first, the other's vector work fills in (+ 2.4-3.5 % measured).
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    u32x4 a[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      a[ks] = *reinterpret_cast<const u32x4*>(stage + (uint32_t)(((sub * 2 + u) * KS + ks) * kFrag) + lane * 16);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      float4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) acc = mfma(a[ks], qb[cb][ks], acc);
      s[cb][u] = acc;
    }
  }
  __builtin_amdgcn_s_setprio(0);
  // the first V fragments are requested now, in front of the softmax's vector work, so that the P V MFMAs do not
  // start by waiting for LDS
  u32x4 vpre[VPRE > 0 ? VPRE : 1];
#pragma unroll
  for (int e = 0; e < VPRE; ++e)
    vpre[e] = *reinterpret_cast<const u32x4*>(stage + stage_v(SUBS, HD) + (uint32_t)((sub * F::kNE + e) * kFrag) + lane * 16);
  // interior (uniform): every token of the sub-tile lies at or before the wave's first query token: nothing to mask
  const bool interior = sub_tile_interior(tb, first_pos);
  const int tok0 = tb + 8 * j;  // the lane's first token
  float ka[8], va[8];  // (parameter formats) the factors of the lane's eight tokens
  if constexpr (F::kParBytes != 0) {
    const uint8_t* const par = stage + stage_par(SUBS, HD) + sub * 256 + 32 * j;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float4v k4 = *reinterpret_cast<const float4v*>(par + 16 * h), v4 = *reinterpret_cast<const float4v*>(par + 128 + 16 * h);
#pragma unroll
      for (int z = 0; z < 4; ++z) {
        ka[4 * h + z] = k4[z];
        va[4 * h + z] = v4[z];
      }
    }
  }
  float x[NCB][8];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float v = s[cb][i >> 2][i & 3];
      if constexpr (F::kParBytes != 0) x[cb][i] = v * ka[i];
      else x[cb][i] = v;
    }
  if (!interior) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const int hi = len_cb[cb] - tok0;  // causality: this lane's column sees tokens < len_cb
#pragma unroll
      for (int i = 0; i < 8; ++i) x[cb][i] = i < hi ? x[cb][i] : -INFINITY;
    }
  }
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    float mx = fmaxf(fmaxf(x[cb][0], x[cb][1]), x[cb][2]);
    mx = fmaxf(fmaxf(mx, x[cb][3]), x[cb][4]);
    mx = fmaxf(fmaxf(mx, x[cb][5]), x[cb][6]);
    mx = fmaxf(mx, x[cb][7]);
    if constexpr (F::kParBytes == 0) mx *= alpha;
    if (__any(mx - st.m[cb] > kTauBlock)) wg_move_reference(st, cb, mx);
  }
  u32x4 pk[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    const float m = st.m[cb];
    if constexpr (F::kParBytes != 0) {
      float p[8], lsum = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float e = __builtin_amdgcn_exp2f(x[cb][i] - m);
        lsum += e;
        p[i] = e * va[i];
      }
      st.l[cb] += lsum;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const half2v h = {(_Float16)p[2 * q], (_Float16)p[2 * q + 1]};
        pk[cb][q] = h2u(h);
      }
    } else {
      const half2v one = {(_Float16)1.0f, (_Float16)1.0f};
      float l = st.l[cb];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float e0 = __builtin_amdgcn_exp2f(fmaf(x[cb][2 * q], alpha, -m));
        const float e1 = __builtin_amdgcn_exp2f(fmaf(x[cb][2 * q + 1], alpha, -m));
        const half2v h = {(_Float16)e0, (_Float16)e1};
        pk[cb][q] = h2u(h);
        if constexpr (SUM32) l += e0 + e1;
        else l = __builtin_amdgcn_fdot2(h, one, l, false);
      }
      st.l[cb] = l;
    }
  }
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int e = 0; e < F::kNE; ++e) {
    u32x4 b;
    if (e < VPRE) b = vpre[e];
    else b = *reinterpret_cast<const u32x4*>(stage + stage_v(SUBS, HD) + (uint32_t)((sub * F::kNE + e) * kFrag) + lane * 16);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      u32x4 seen = b;
      if constexpr (CUT) {
        int n = first_pos + min((cb + 1) * tpt, n_tok) - tok0;  // slots of this lane's run that the block sees
        if constexpr (NCB * HD > 128) asm volatile("" : "+v"(n));  // (masks made anew for each fragment: no registers to keep them in)
#pragma unroll
        for (int q = 0; q < 4; ++q) seen[q] &= (2 * q < n ? 0xFFFFu : 0u) | (2 * q + 1 < n ? 0xFFFF0000u : 0u);
      }
      st.acc[cb][e] = mfma(seen, pk[cb], st.acc[cb][e]);
    }
  }
}

// One work item of the workgroup variant: (sequence, KV head, NW x NCB consecutive 16-column query tiles): NW waves
// of NCB column blocks each walk K/V in steps of SUBS sub-tiles (32 tokens each).  With NW == SUBS every wave fetches
// and stages K and V of sub-tile w; with NW == 2 SUBS waves 0..SUBS-1 stage the K fragments of sub-tile w and the
// others the V fragments and parameters of sub-tile w - SUBS.  Built variants: 8 waves x 2 blocks, 4 sub-tiles per
// step, one workgroup per compute unit (two waves per SIMD, so that one's softmax runs under the other's MFMAs);
// 4 x 4, 4 sub-tiles (one wave per SIMD); 8 x 4 and 8 x 3 for large launches at head_dim 64; 8 x 1 for small launches, 8 x 2 in
// groups (GROUPS) for those behind long contexts; 4 x 1 with 2 sub-tiles per step at head_dim 256.
// (Another one -- 4 x 2 with 2 sub-tiles per step, two workgroups per
// compute unit -- passed its small cases but ended a full-size two-model run with the GPU faulted or hung; the
// cause was not found and the variant is no longer built.  What was particular to it is absent from the 4 x 1 kernel of
// head_dim 256: that one has a compute unit to itself (its two stages alone are 129 KiB of the 160), a wave has one column
// block, and its staging roles, fragment offsets and barriers are those of the 8-wave kernels, NW == 2 SUBS, with half the
// counts: fragment indices end at SUBS * HD / 16 on both sides, which is where stage_v and stage_par begin.)
// An item whose context was dealt to 2^kv_shift groups of waves (sub-tile s to group s mod 2^kv_shift): the waves of a query
// tile exchange their accumulators through LDS, where the stages were, and each finishes one part of them: with two groups a
// column block, with four half of one's output elements.  Every wave of the workgroup takes part.
template <int DT, int NW, int NCB, int HD>
__device__ __forceinline__ void merge_groups(const PrefillArgs& P, WgState<NCB, HD>& st, uint8_t* smem, int w, int lane, int head,
                                             int row0, int n_tok, float v_static) {
  constexpr int NE = HD / 16, N = NCB * NE;  // accumulator tiles of a wave
  static_assert(NW * (N * 1024 + NCB * 128) <= 2 * (int)stage_bytes(NW == 8 ? 4 : 2, HD), "the partial sums fit the stages");
  const DevBatch& B = P.b;
  const int j = lane >> 4, c = lane & 15;
  const int n_kv = 1 << P.kv_shift, n_q = NW >> P.kv_shift, size = N >> P.kv_shift;
  const int qg = w & (n_q - 1), kv = w / n_q;
  float4v* const s_acc = reinterpret_cast<float4v*>(smem);                       // [wave][tile][lane]
  float2* const s_ml = reinterpret_cast<float2*>(smem + NW * N * 1024);          // [wave][block][column]
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    st.l[cb] = over_column(st.l[cb], [](float a, float b) { return a + b; });
    if (j == 0) s_ml[(w * NCB + cb) * 16 + c] = float2{st.m[cb], st.l[cb]};
  }
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (i / size != kv) s_acc[(w * N + i) * 64 + lane] = st.acc[i / NE][i % NE];
  __syncthreads();
  const int tok_c = c / B.G, hg_c = c - tok_c * B.G;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    if ((cb * NE + NE - 1) / size < kv || cb * NE / size > kv) continue;  // (uniform) none of this block's tiles are this wave's
    float M = st.m[cb];
    for (int g = 0; g < n_kv; ++g) M = fmaxf(M, s_ml[((g * n_q + qg) * NCB + cb) * 16 + c].x);
    float L = 0.f;
    const float own = __builtin_amdgcn_exp2f(st.m[cb] - M);
#pragma unroll
    for (int e = 0; e < NE; ++e)
      if ((cb * NE + e) / size == kv) st.acc[cb][e] *= own;
    for (int g = 0; g < n_kv; ++g) {
      const int wg = g * n_q + qg;
      const float2 ml = s_ml[(wg * NCB + cb) * 16 + c];
      const float f = __builtin_amdgcn_exp2f(ml.x - M);
      L += f * ml.y;
      if (g == kv) continue;
#pragma unroll
      for (int e = 0; e < NE; ++e)
        if ((cb * NE + e) / size == kv) {
          const float4v x = s_acc[(wg * N + cb * NE + e) * 64 + lane];
#pragma unroll
          for (int r = 0; r < 4; ++r) st.acc[cb][e][r] += f * x[r];
        }
    }
    if (tok_c >= P.tpt || cb * P.tpt + tok_c >= n_tok) continue;
    const float inv = v_static / L;
    const int row = min(max(row0 + cb * P.tpt + tok_c, 0), P.n_rows - 1);
    const int64_t qrow = (int64_t)row * B.n_q + head * B.G + hg_c;
    _Float16* const orow = B.out + qrow * HD + 4 * NE * j;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      uint32_t wv[NE / 2];
#pragma unroll
      for (int q = 0; q < NE / 2; ++q) {
        const half2v hv = {(_Float16)(st.acc[cb][2 * q][r] * inv), (_Float16)(st.acc[cb][2 * q + 1][r] * (DT == FS_KV_INT4 ? 0.0625f * inv : inv))};
        wv[q] = h2u(hv);
      }
      if (NE == 8 && size == N / 2) {  // (uniform) a whole block
        *reinterpret_cast<u32x4*>(orow + NE * r) = u32x4{wv[0], wv[1], wv[NE / 2 - 2], wv[NE / 2 - 1]};
      } else {
#pragma unroll
        for (int q = 0; q < NE / 2; q += 2) {  // four or (head_dim 64 with four groups) two elements
          if (size >= 4) {
            if ((cb * NE + 2 * q) / size == kv) *reinterpret_cast<u32x2*>(orow + NE * r + 2 * q) = u32x2{wv[q], wv[q + 1]};
          } else {
            if ((cb * NE + 2 * q) / size == kv) *reinterpret_cast<uint32_t*>(orow + NE * r + 2 * q) = wv[q];
            if ((cb * NE + 2 * q + 2) / size == kv) *reinterpret_cast<uint32_t*>(orow + NE * r + 2 * q + 2) = wv[q + 1];
          }
        }
      }
    }
    if (j == 0 && B.lse && cb * NE / size == kv) B.lse[qrow] = (M + __builtin_amdgcn_logf(L)) * kLn2;
  }
  __syncthreads();  // (the next item's first stage goes where the partial sums are)
}

// ---------------------------------------------------------------------------------------------------------
// Split items.  In a launch of few items per compute unit the longest context, or the second round of a few items, decides:
// four FP8 chunks of 512 tokens behind 4700 - 14700 (256 items, one per unit) took 383 us, what 115 steps take although the mean
// is 76; now 300 (with no unit idle the chip's power bounds a step, 3.8 us against 3.3).  Such a launch lays its items' steps
// (128 tokens each, and two for an item's start) one after the other and cuts the row into equal ranges, one per workgroup
// (SplitPlan): an item that a cut divides is worked on in pieces by neighbouring workgroups, each of which leaves its
// accumulators, references and sums (fp32, as they stand in the registers) in the workspace and counts; whoever counts
// last adds the pieces up, in the order of the context whoever that is, and writes the rows.  Nobody waits for anybody.
// (One workgroup reads all pieces of an item, 1.5 us each; a piece stands for eight steps of 3 us or more that others took.)
// A counter is a 64-bit word in the workspace that nothing clears before the launch: the count stands behind a
// 48-bit mark without which the word reads as zero, and the last piece of an item takes the mark away again.
// ---------------------------------------------------------------------------------------------------------
static_assert(kSplitGroups <= 512, "a thread for every workgroup's whole items");  // (their pieces have a place: two each)
constexpr uint32_t kPieceBytes = 8 * (16 * 1024 + 2 * 128);  // 8 waves of 16 accumulator tiles and 2 x 16 references and sums
constexpr uint64_t kPieceMark = 0x9d3c5af16e870000ull;
constexpr uint64_t kPiecesBytes = 8ull * kSplitGroups + 2ull * kSplitGroups * kPieceBytes;
struct Piece {
  int step = 0, end = 0x7fffffff;  // of the item's steps
  uint32_t first = 0, n = 1;       // the first workgroup with a piece of this item, and how many have one
  uint32_t own = 0;                // which of them this is
  uint32_t* s_count = nullptr;     // a word of LDS
};
// The first piece of an item lies at the end of its workgroup's range, all others at the beginning of theirs.
__device__ __forceinline__ uint8_t* piece_at(const PrefillArgs& P, const Piece& p, uint32_t k) {
  return P.pieces + 8ull * kSplitGroups + (uint64_t)piece_place(p.first, k) * kPieceBytes;
}
// How many pieces of the item that begins in workgroup `at` have been left, this one included.
__device__ __forceinline__ uint32_t count_piece(const PrefillArgs& P, uint32_t at, uint32_t n) {
  unsigned long long* word = reinterpret_cast<unsigned long long*>(P.pieces) + at;
  unsigned long long old = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), next;
  uint32_t count;
  do {  // (as many rounds as other pieces of the item are being counted)
    count = (old & ~0xffffull) == kPieceMark ? (uint32_t)(old & 0xffff) + 1 : 1;
    next = count == n ? 0ull : kPieceMark | count;
  } while (!__hip_atomic_compare_exchange_strong(word, &old, next, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  return count;
}
// A pair of a piece's numbers, written to and read from where every XCD sees it (agent scope: past the XCDs' own L2s).  us, with a
// write-back of the L2 by every wave in front of the count -> like this: four FP8 chunks of 512 behind 3000 - 16384 379 -> 302, 300
// FP16 ones of 16 behind 200 - 4000 with one KV head 293 -> 126, 14 of 100 with 40 heads 441 -> 244.
typedef float float2v __attribute__((ext_vector_type(2)));
typedef unsigned long long Pair;
__device__ __forceinline__ void leave_pair(Pair* at, float x, float y) {
  __hip_atomic_store(at, (Pair)__float_as_uint(y) << 32 | __float_as_uint(x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2v take_pair(const Pair* at) {
  const Pair v = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return float2v{__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32))};
}
// Leaves the workgroup's piece; true: it was the last, and st holds the whole item (the sum in the lanes j = 0).  Every wave
// takes part; the result is uniform.
template <int NW, int NCB, int HD>
__device__ __forceinline__ bool merge_pieces(const PrefillArgs& P, const Piece& p, WgState<NCB, HD>& st, int w, int lane, int n_tok) {
  constexpr int NE = HD / 16, N = NCB * NE;
  static_assert(NW * (N * 1024 + NCB * 128) <= (int)kPieceBytes, "a piece has room");
  const int j = lane >> 4, c = lane & 15;
  auto acc_at = [&](uint32_t k) { return reinterpret_cast<Pair*>(piece_at(P, p, k)) + w * N * 128 + lane; };
  auto ml_at = [&](uint32_t k) { return reinterpret_cast<Pair*>(piece_at(P, p, k)) + NW * N * 128 + w * NCB * 16 + c; };
  // (A wave without query tokens has nothing to leave, in any of the item's pieces: chunks of 16 tokens keep one wave of eight.
  // 100 FP8 chunks of 16 behind 4000: 305 us with all waves' parts, 290 without those.)
  if (n_tok > 0) {
    Pair* const acc = acc_at(p.own);
    Pair* const ml = ml_at(p.own);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const float l = over_column(st.l[cb], [](float a, float b) { return a + b; });
      if (j == 0) leave_pair(ml + cb * 16, st.m[cb], l);
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int h = 0; h < 2; ++h) leave_pair(acc + ((cb * NE + e) * 2 + h) * 64, st.acc[cb][e][2 * h], st.acc[cb][e][2 * h + 1]);
    }
  }
  // Every wave waits until its own stores are done before it meets the barrier, which waits for none; then one counts.  (The
  // wait is what an agent-scope release has; its write-back is for plain stores, and none of a piece's are.)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) *p.s_count = count_piece(P, p.first, p.n);
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(*p.s_count) != p.n) return false;  // (the next piece's count lies behind barriers)
  if (n_tok == 0) return true;
  float M[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    M[cb] = take_pair(ml_at(0) + cb * 16)[0];
    for (uint32_t k = 1; k < p.n; ++k) M[cb] = fmaxf(M[cb], take_pair(ml_at(k) + cb * 16)[0]);
    st.l[cb] = 0.f;
#pragma unroll
    for (int e = 0; e < NE; ++e) st.acc[cb][e] = float4v{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll 1
  for (uint32_t k = 0; k < p.n; ++k) {
    const Pair* const acc = acc_at(k);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const float2v ml = take_pair(ml_at(k) + cb * 16);
      float2v x[NE][2];
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int h = 0; h < 2; ++h) x[e][h] = take_pair(acc + ((cb * NE + e) * 2 + h) * 64);
      const float f = __builtin_amdgcn_exp2f(ml[0] - M[cb]);
      st.l[cb] += f * ml[1];
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int r = 0; r < 4; ++r) st.acc[cb][e][r] += f * x[e][r >> 1][r & 1];
    }
  }
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    st.m[cb] = M[cb];
    if (j != 0) st.l[cb] = 0.f;
  }
  return true;
}

// smem: two stages, then the workgroup's block-address table.
// DEQ (INT8 / INT4 only): the staging waves dequantize, the tile code is the FP16 one.
// header: where a block-table entry outside the pool is reported.
// S: what the workgroup holds of the sequence it last worked on.  A sequence that fits one table segment has all its
// blocks' addresses in LDS (without the head, which is added at the use), so that an item of the same sequence as the one
// before starts with its first K/V fetch.
struct SeqHeld {
  int seq = -1;
  bool table = false;  // the address table holds all blocks of the sequence
};
template <int DT, int NW, int NCB, int SUBS, bool DEQ, int HD, bool SUM32, bool GROUPS, bool SPLIT = false>
__device__ void prefill_item_wg(const PrefillArgs& P, uint32_t* header, int seq, const SeqShape& shape, int head, int qt,
                                uint8_t* smem, uint64_t* s_tab, int w, SeqHeld& S, const Piece& piece = Piece{}) {
  static_assert(NW == SUBS || NW == 2 * SUBS, "staging roles");
#ifdef FS_TIMELINE
  uint64_t tl_ph[5] = {(uint64_t)wall_clock64(), 0, 0, 0, 0};
#endif
  static_assert(!DEQ || Fmt<DT>::kParBytes != 0, "staged dequantization is for the formats with per-token parameters");
  static_assert(!DEQ || HD == kD, "staged dequantization is written for head_dim 128");
  constexpr int NE = HD / 16;  // accumulator tiles of a column block: row 4 j + r of tile e is element NE (4 j + r) + e of column c
  constexpr int CDT = DEQ ? FS_KV_FP16 : DT;  // the format the consumer code sees
  // V fragments read ahead of the softmax: what the format's register budget leaves room for (two waves per SIMD)
  // (eight instead of four: a 4 x 512-token FP8 chunk step 429.5 -> 423 us, INT8 prompts 817 -> 811 us; FP16 would spill)
  constexpr int kVPre = NW != 8 ? 0 : (HD == kD && (DEQ || DT == FS_KV_FP8_E4M3) ? 8 : 4);
  const bool whole = P.whole_runs != 0;  // (uniform)
  const bool does_k = NW == SUBS || w < SUBS, does_v = NW == SUBS || w >= SUBS;  // wave-uniform staging roles
  const int sw = w % SUBS;                                                       // the sub-tile this wave stages
  const DevBatch& B = P.b;
  const DevGeom& g = B.g;
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int j = lane >> 4, c = lane & 15;
  const int G = B.G;
  if (seq != S.seq) S.table = false;  // (uniform)
  S.seq = seq;
  const int len = shape.len, n_new = shape.n_new;
  // groups of waves that share the context; the wave's query tile and its group
  const int kv_shift = GROUPS ? P.kv_shift : 0, n_kv = 1 << kv_shift;
  const int qg = GROUPS ? w & ((NW >> kv_shift) - 1) : w, kv = GROUPS ? w / (NW >> kv_shift) : 0;
  const int qw = P.tpt * NCB;                 // query tokens per wave
  const int q_wg = qw * (NW >> kv_shift);     // query tokens per item
  const int r0_wg = qt * q_wg;                // first query token of the item within the chunk
  if (r0_wg >= n_new) return;                 // (cannot happen with consistent inputs; uniform over the workgroup)
  const int n_tok_wg = min(q_wg, n_new - r0_wg);
  const int r0 = r0_wg + qg * qw;             // this wave's share
  const int n_tok = max(0, min(qw, n_tok_wg - qg * qw));
  const int first_pos = len - n_new + r0;
  const int tok_c = c / G, hg_c = c - tok_c * G;

  const int len_u = len - n_new + r0_wg + n_tok_wg;  // tokens that the workgroup's last query sees
  // (SPLIT) where the piece ends
  const int end_u = SPLIT && piece.end < (len_u + 32 * SUBS - 1) / (32 * SUBS) ? 32 * SUBS * piece.end : len_u;
  TokenCtx X;
  X.ptr = s_tab;
  X.base_off = (uint64_t)head * g.head_chunk;
  X.T = g.T;
  X.magic = P.t_magic;

  u32x4 qb[NCB][HD / 32];
  int len_cb[NCB], row_cb[NCB];
  float alpha = B.sm_scale * kLog2e;
  if (DT == FS_KV_FP8_E4M3) alpha *= B.k_scale[head];
  WgState<NCB, HD> st;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    const int tok = cb * P.tpt + tok_c;  // query token of this lane's column in block cb
    const bool live = tok_c < P.tpt && tok < n_tok;
    len_cb[cb] = live ? first_pos + tok + 1 : len_u;  // a dead column (q = 0, never written) sees everything
    row_cb[cb] = min(max(shape.q0 + r0 + tok, 0), P.n_rows - 1);
    float sum;  // (of no use here; without it the loads come out in another order, and one prompt of 777 tokens takes 24.5 -> 24.7 us)
    load_q<DT, !DEQ, HD>(B.q + ((int64_t)row_cb[cb] * B.n_q + head * G + hg_c) * HD, live, j, qb[cb], sum);
#pragma unroll
    for (int e = 0; e < NE; ++e) st.acc[cb][e] = float4v{0.f, 0.f, 0.f, 0.f};
    st.m[cb] = kNoReference;  // (a masked logit then weighs 0 from the start; with -inf it would be NaN)
    st.l[cb] = 0.f;
  }

  const int32_t* table = B.tables + (int64_t)seq * B.max_blocks;
  const int w_end = n_tok > 0 ? first_pos + n_tok : 0;  // tokens this wave's last query sees
  constexpr bool kCut = SUM32 && DT == FS_KV_FP16;  // (see wg_tile)
  int t0 = SPLIT ? 32 * SUBS * piece.step : 0;  // (and what is counted from it: multiples of 32)
  if (SPLIT && t0 > 0) S.table = false;
  do {
    const int n = min(end_u - t0, P.seg_tokens), k0 = t0 / g.T;
    X.rel0 = t0 - k0 * g.T;
    X.last = n - 1;
    if (!S.table) {  // (uniform)
      // the previous segment's (or item's) last barrier lies behind every use of the old table
      S.table = len <= P.seg_tokens && (!SPLIT || t0 == 0);  // one segment (t0 = 0): all of the sequence's blocks, for its next items
      const int nb = (X.rel0 + (S.table ? len : n) - 1) / g.T + 1;
      for (int i = threadIdx.x; i < nb; i += NW * 64)
        s_tab[i] = reinterpret_cast<uint64_t>(B.layer_base + (uint64_t)checked_block(table[k0 + i], B.n_blocks, header) * g.block_budget);
      __syncthreads();
    }
#ifdef FS_TIMELINE
    if (t0 == 0) tl_ph[1] = wall_clock64();
#endif
    const int n_super = (n + 32 * SUBS - 1) / (32 * SUBS);
    Tile<DT, 16, HD> t;
    uint32_t kpar[2] = {0u, 0u};  // (parameter formats) K parameters of the rows this lane stages
    // fetch / stage this wave's share of the sub-tile that starts at token tb of the segment
    auto fetch = [&](int tb) {
      if (does_k) fetch_k<DT, HD, Fmt<DT>::kParBytes != 0>(X, g, whole, tb, j, c, t, kpar);
      if (does_v) fetch_v<DT, HD>(X, g, whole, tb, j, c, t);
    };
    auto stage_to = [&](uint8_t* stage, int tb) {
      // V slots past the segment's last token are cleared whatever they hold -- the last token's rows again where blocks are no
      // multiple of eight tokens: weight 0 times its Inf made its own row NaN.
      const bool clear = n - tb < 32;  // (uniform)
      const int live = n - (tb + 8 * j);
      if constexpr (DEQ) {
        if (does_k) stage_k_deq<DT>(stage, sw, lane, t, kpar);
        if (does_v) stage_v_deq<DT, SUBS>(stage, sw, lane, clear, live, t);
      } else if constexpr (Fmt<DT>::kParBytes != 0) {
        if (does_k) stage_k_int<DT, HD>(stage, sw, lane, t, kpar);
        if (does_v) stage_v_int<DT, SUBS, HD>(stage, sw, lane, clear, live, alpha, t);
      } else {
        if (does_k) stage_k<DT, HD>(stage, sw, lane, t);
        if (does_v) stage_v<DT, SUBS, HD>(stage, sw, lane, clear, live, t);
      }
    };
    fetch(32 * sw);
    stage_to(smem, 32 * sw);
    __syncthreads();
#ifdef FS_TIMELINE
    if (t0 == 0) tl_ph[2] = wall_clock64();
#endif
    // the query operands' loads, issued before the table and the first K/V fetch, are collected here
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) settle_q(qb[cb]);
    for (int i = 0; i < n_super; ++i) {
      // next step's sub-tile of this wave; the segment's last step fetches and stages nothing (the wait in stage_to
      // is for this step's fetch alone, so the condition costs the compiler's wait counts nothing)
      const int tb_next = 32 * ((i + 1) * SUBS + sw);
      const bool more = i + 1 < n_super;  // wave-uniform
      if (more) fetch(tb_next);
      const uint8_t* stage = smem + (uint32_t)(i & 1) * stage_bytes(SUBS, HD);
      // A wave multiplies the sub-tiles that hold a token one of its queries sees: those past its diagonal (half of
      // the last step or two of an item, and all of them in a wave without query tokens: a ragged last item of a chunk,
      // chunks shorter than the workgroup's 16 NW / G tokens) are left out.  A loop bound, not a branch around the
      // tile: it costs the accumulators' registers nothing.  (64 FP16 prompts of 512 - 4096 tokens, GQA 4:1: 4126 ->
      // 3977 us; 12 INT4 multi-head prompts of 300 - 3000 tokens, whose items span two steps of diagonal: 840 -> 800 us.)
      const int ts = t0 + 32 * SUBS * i;  // the step's first token
      const int n_live = live_sub_tiles(w_end, ts, SUBS);
      // (sub-tiles that end at or before the first query's own token are seen by all of the wave's columns)
      const int n_seen = kCut ? min(n_live, max(first_pos + 1 - ts, 0) >> 5) : n_live;
#pragma unroll 1  // (unrolled by two: measured 0.5 % slower)
      for (int sub = kv; sub < n_seen; sub += n_kv)
        wg_tile<CDT, NCB, SUBS, kVPre, HD, SUM32>(stage, sub, ts + 32 * sub, qb, len_cb, alpha, first_pos, lane, j, c, st);
      if constexpr (kCut) {
#pragma unroll 1
        for (int sub = n_seen + ((kv - n_seen) & (n_kv - 1)); sub < n_live; sub += n_kv)
          wg_tile<CDT, NCB, SUBS, 0, HD, SUM32, true>(stage, sub, ts + 32 * sub, qb, len_cb, alpha, first_pos, lane, j, c,
                                                      st, P.tpt, n_tok);
      }
      uint8_t* next = smem + (uint32_t)((i + 1) & 1) * stage_bytes(SUBS, HD);
      if (more) stage_to(next, tb_next);
      __syncthreads();  // (also after the last step: the next staging overwrites what other waves may still read)
    }
  } while (next_segment(t0, end_u, P.seg_tokens));
#ifdef FS_TIMELINE
  tl_ph[3] = wall_clock64();
#endif
  const float v_static = DT == FS_KV_FP8_E4M3 ? B.v_scale[head] : 1.0f;
  if constexpr (SPLIT) {
    if (piece.n > 1) {  // (uniform)
      S.table = false;
      if (!merge_pieces<NW, NCB, HD>(P, piece, st, w, lane, n_tok)) return;
    }
  }
  if constexpr (GROUPS) {
    merge_groups<CDT, NW, NCB, HD>(P, st, smem, w, lane, head, shape.q0 + r0, n_tok, v_static);
    return;
  }
  if (n_tok == 0) return;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    auto sum = [](float a, float b) { return a + b; };
    const float l = over_column(st.l[cb], sum);
    if (tok_c >= P.tpt || cb * P.tpt + tok_c >= n_tok) continue;
    const float inv = 1.0f / l;
    const int64_t qrow = (int64_t)row_cb[cb] * B.n_q + head * G + hg_c;
    _Float16* const orow = B.out + qrow * HD + 4 * NE * j;
#pragma unroll
    for (int r = 0; r < 4; ++r) {  // row 4 j + r of the transposed accumulators e: element NE (4 j + r) + e of the column
      uint32_t wv[NE / 2];
#pragma unroll
      for (int q = 0; q < NE / 2; ++q) {
        float o[2];
#pragma unroll
        for (int z = 0; z < 2; ++z) {
          const int e = 2 * q + z;
          const float f = CDT == FS_KV_INT4 && (e & 1) ? 0.0625f : 1.0f;  // (INT4's odd code positions are staged 16-fold)
          o[z] = st.acc[cb][e][r] * (f * v_static * inv);
        }
        const half2v hv = {(_Float16)o[0], (_Float16)o[1]};
        wv[q] = h2u(hv);
      }
      if constexpr (NE == 4) {
        reinterpret_cast<u32x2*>(orow)[r] = u32x2{wv[0], wv[1]};
      } else {
#pragma unroll
        for (int q = 0; q < NE / 8; ++q)
          reinterpret_cast<u32x4*>(orow)[NE / 8 * r + q] = u32x4{wv[4 * q], wv[4 * q + 1], wv[4 * q + 2], wv[4 * q + 3]};
      }
    }
    if (j == 0 && B.lse) B.lse[qrow] = (st.m[cb] + __builtin_amdgcn_logf(l)) * kLn2;
  }
#ifdef FS_TIMELINE
  if (threadIdx.x == 0 && blockIdx.x < kPfTimelineGroups) {
    uint64_t* row = P.timeline + 8 * blockIdx.x;
    tl_ph[4] = wall_clock64();
    for (int k = 0; k < 4; ++k) row[4 + k] += tl_ph[k + 1] - tl_ph[k];
  }
#endif
}

// ---------------------------------------------------------------------------------------------------------
// Software-pipelined workgroup variant (4 waves x 64 columns, one wave per SIMD).  The compiler emits a tile's
// MFMAs and its softmax as separate bursts, and the step barrier keeps the waves of a SIMD in phase, so in the
// variants above the matrix cores idle during every softmax.  Here one wave overlaps the two itself: while the
// vector ALU exponentiates sub-tile s, the MFMAs of S^T for sub-tile s + 1 are issued between its instructions
// (block 1); while the MFMAs of P V for sub-tile s run, the vector ALU turns the new S^T into logits and column
// maxima (block 2); scheduling-group barriers pin the interleave (one MFMA, then a few vector instructions).
// The pipeline is restarted at every step (S^T of the step's first sub-tile runs alone; block 1 of the last
// sub-tile multiplies the step's first sub-tile again and discards it): carrying it across the step barrier
// would let a fast wave overwrite a stage that a slow wave still reads.
// ---------------------------------------------------------------------------------------------------------
template <int DT, int NCB>
struct Logits {
  float x[NCB][8];   // logits (parameter formats) or raw products (FP16, FP8)
  float tmax[NCB];   // column maxima, base-2 domain
  float va[8], vb2[8];  // parameter formats: per-token V factors for the weights of this sub-tile
};

// S^T accumulators -> logits, masks, column maxima.  Returns whether some column's reference must move.
template <int DT, int NCB, int SUBS>
__device__ __forceinline__ bool make_logits(const float4v (&s)[NCB][2], const uint8_t* stage, int sub, const ItemCtx& X,
                                            const float (&qsum)[NCB], const int (&len_cb)[NCB], float alpha, int first_pos,
                                            int vb, int lane, int c, const WideState<NCB>& st, Logits<DT, NCB>& out) {
  using F = Fmt<DT>;
  const RunLoc L = locate(X, vb, lane >> 4);
  const bool interior = __all(L.lo == 0 && L.tok0 + 8 <= first_pos + 1);  // wave-uniform
  float ka[8], kb[8];
  if constexpr (F::kParBytes != 0) {
    const uint32_t par = *reinterpret_cast<const uint32_t*>(stage + stage_par(SUBS) + sub * 256 + lane * 4);
    float pa, pb;
    const float sc = f16lo(par);
    const float zp = DT == FS_KV_INT4 ? f16hi(par) : 128.0f;
    if (c < 8) {
      pa = alpha * kTwo24 * sc;
      pb = -alpha * sc * zp;
    } else {
      const bool ok = (c & 7) >= L.lo && (c & 7) < L.hi_u;
      pa = ok ? sc : 0.f;
      pb = ok ? -sc * zp : 0.f;
    }
    static_for(std::make_integer_sequence<int, 8>{}, [&](auto I) {
      constexpr int i = decltype(I)::value;
      ka[i] = row_bcast<i>(pa);
      kb[i] = row_bcast<i>(pb);
      out.va[i] = row_bcast<8 + i>(pa);
      out.vb2[i] = row_bcast<8 + i>(pb);
    });
  }
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float v = s[cb][i >> 2][i & 3];
      if constexpr (F::kParBytes != 0) out.x[cb][i] = fmaf(v, ka[i], kb[i] * qsum[cb]);
      else out.x[cb][i] = v;
    }
  auto maxima = [&]() {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      float mx = fmaxf(fmaxf(out.x[cb][0], out.x[cb][1]), out.x[cb][2]);
      mx = fmaxf(fmaxf(mx, out.x[cb][3]), out.x[cb][4]);
      mx = fmaxf(fmaxf(mx, out.x[cb][5]), out.x[cb][6]);
      mx = fmaxf(mx, out.x[cb][7]);
      if constexpr (F::kParBytes == 0) mx *= alpha;
      out.tmax[cb] = mx;
    }
  };
  maxima();  // in the straight-line part, beside the caller's MFMAs; redone below on the rare masked tiles
  __builtin_amdgcn_sched_barrier(0);
  if (!interior) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const int hi = min(L.hi_u, len_cb[cb] - L.tok0);
      const uint32_t n_ok = (uint32_t)max(hi - L.lo, 0);
#pragma unroll
      for (int i = 0; i < 8; ++i) out.x[cb][i] = (uint32_t)(i - L.lo) < n_ok ? out.x[cb][i] : -INFINITY;
    }
    maxima();
  }
  bool need = false;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) need |= out.tmax[cb] - st.m[cb] > kTau;
  return need;
}

template <int DT>
__device__ void prefill_item_wgp(const PrefillArgs& P, int seq, int head, int qt, uint8_t* smem, uint64_t* s_tab, int w) {
  constexpr int NW = 4, NCB = 4, SUBS = 4;
  using F = Fmt<DT>;
  const DevBatch& B = P.b;
  const DevGeom& g = B.g;
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int j = lane >> 4, c = lane & 15;
  const int G = B.G;
  const int max_len = (int)min((int64_t)B.max_blocks * g.T, (int64_t)0x7fffffff);
  int len = B.seq_lens[seq];
  len = len < 1 ? 1 : min(len, max_len);
  int n_new = P.q_offsets[seq + 1] - P.q_offsets[seq];
  n_new = n_new < 0 ? 0 : min(n_new, len);
  const int qw = P.tpt * NCB;
  const int r0_wg = qt * qw * NW;
  if (r0_wg >= n_new) return;
  const int n_tok_wg = min(qw * NW, n_new - r0_wg);
  const int r0 = r0_wg + w * qw;
  const int n_tok = max(0, min(qw, n_tok_wg - w * qw));
  const int first_pos = len - n_new + r0;
  const int tok_c = c / G, hg_c = c - tok_c * G;

  ItemCtx X;
  X.T = g.T;
  X.R = B.R;
  X.r_magic = B.r_magic;
  X.len_u = len - n_new + r0_wg + n_tok_wg;
  X.len = X.len_u;
  X.chunk_ptr = s_tab;

  u32x4 qb[NCB][4];
  float qsum[NCB];
  int len_cb[NCB], row_cb[NCB];
  float alpha = B.sm_scale * kLog2e;
  if (DT == FS_KV_FP8_E4M3) alpha *= B.k_scale[head];
  WideState<NCB> st;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    const int tok = cb * P.tpt + tok_c;
    const bool live = tok_c < P.tpt && tok < n_tok;
    len_cb[cb] = live ? first_pos + tok + 1 : X.len_u;
    row_cb[cb] = min(max(P.q_offsets[seq] + r0 + tok, 0), P.n_rows - 1);
    load_q<DT>(B.q + ((int64_t)row_cb[cb] * B.n_q + head * G + hg_c) * kD, live, j, qb[cb], qsum[cb]);
    if constexpr (F::kParBytes != 0) {
      qsum[cb] += __shfl_xor(qsum[cb], 16, 64);
      qsum[cb] += __shfl_xor(qsum[cb], 32, 64);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) st.acc[cb][e] = float4v{0.f, 0.f, 0.f, 0.f};
    st.m[cb] = -INFINITY;
    st.l[cb] = 0.f;
    st.zc[cb] = 0.f;
  }

  const int32_t* table = B.tables + (int64_t)seq * B.max_blocks;
  const uint8_t* head_base = B.layer_base + (uint64_t)head * g.head_chunk;
  const int n_run = n_runs(X.len_u, g.T, B.R);
  for (int v0 = 0; v0 < n_run; v0 += P.seg_runs) {
    X.v_end = min(n_run, v0 + P.seg_runs);
    X.k0 = div_runs(v0, B.R, B.r_magic);
    {
      const int nb = div_runs(X.v_end - 1, B.R, B.r_magic) - X.k0 + 1;
      for (int i = threadIdx.x; i < nb; i += NW * 64)
        s_tab[i] = reinterpret_cast<uint64_t>(head_base + (uint64_t)checked_block(table[X.k0 + i], B.n_blocks, P.header) * g.block_budget);
      __syncthreads();
    }
    const int n_super = (X.v_end - v0 + 4 * SUBS - 1) / (4 * SUBS);
    Tile<DT, 16> t;
    issue_k<DT, 16>(X, v0 + 4 * w, j, c, t);
    issue_v<DT, 16>(X, g, v0 + 4 * w, j, c, t);
    stage_k<DT, kD>(smem, w, lane, t);
    {
      const int live = locate(X, v0 + 4 * w, j).hi_u;
      stage_v<DT, SUBS, kD>(smem, w, lane, !__all(live >= 8), live, t);
    }
    __syncthreads();
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) settle_q(qb[cb]);  // (issued before the table and the first K/V fetch)
    for (int i = 0; i < n_super; ++i) {
      const int vb_next = v0 + (i + 1) * 4 * SUBS + 4 * w;
      issue_k<DT, 16>(X, vb_next, j, c, t);
      issue_v<DT, 16>(X, g, vb_next, j, c, t);
      const uint8_t* stage = smem + (uint32_t)(i & 1) * stage_bytes(SUBS);
      const uint8_t* lane_base = stage + lane * 16;
      // ---- pipeline start: S^T and logits of the step's first sub-tile ----
      u32x4 kf[2][4];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) kf[u][ks] = *reinterpret_cast<const u32x4*>(lane_base + (uint32_t)((u * 4 + ks) * kFrag));
      float4v sn[NCB][2];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
          float4v a4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) a4 = mfma(kf[u][ks], qb[cb][ks], a4);
          sn[cb][u] = a4;
        }
      Logits<DT, NCB> cur;
      if (__any(make_logits<DT, NCB, SUBS>(sn, stage, 0, X, qsum, len_cb, alpha, first_pos, v0 + i * 4 * SUBS, lane, c, st, cur))) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) wide_move_reference<DT>(st, cb, cur.tmax[cb], j);
      }
#pragma unroll 1  // (unrolled by two: measured 0.5 % slower)
      for (int sub = 0; sub < SUBS; ++sub) {
        const int nsub = (sub + 1) & (SUBS - 1);  // after the last sub-tile: the first again, its result unused
        // ---- block 1: S^T of sub-tile nsub (MFMA) beside the exponentials of sub-tile sub (vector ALU) ----
        u32x4 vf[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) vf[e] = *reinterpret_cast<const u32x4*>(lane_base + stage_v(SUBS) + (uint32_t)((sub * 8 + e) * kFrag));
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int ks = 0; ks < 4; ++ks)
            kf[u][ks] = *reinterpret_cast<const u32x4*>(lane_base + (uint32_t)((nsub * 8 + u * 4 + ks) * kFrag));
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) {
            float4v a4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a4 = mfma(kf[u][ks], qb[cb][ks], a4);
            sn[cb][u] = a4;
          }
        u32x4 pk[NCB];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
          const float m = st.m[cb];
          if constexpr (F::kParBytes != 0) {
            float pw[8], lsum = 0.f;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              const float ex = __builtin_amdgcn_exp2f(cur.x[cb][q] - m);
              lsum += ex;
              pw[q] = ex * cur.va[q];
              st.zc[cb] = fmaf(ex, cur.vb2[q], st.zc[cb]);
            }
            st.l[cb] += lsum;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const half2v h = {(_Float16)pw[2 * q], (_Float16)pw[2 * q + 1]};
              pk[cb][q] = h2u(h);
            }
          } else {
            const half2v one = {(_Float16)1.0f, (_Float16)1.0f};
            float l = st.l[cb];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float e0 = __builtin_amdgcn_exp2f(fmaf(cur.x[cb][2 * q], alpha, -m));
              const float e1 = __builtin_amdgcn_exp2f(fmaf(cur.x[cb][2 * q + 1], alpha, -m));
              const half2v h = {(_Float16)e0, (_Float16)e1};
              pk[cb][q] = h2u(h);
              l = __builtin_amdgcn_fdot2(h, one, l, false);
            }
            st.l[cb] = l;
          }
        }
        // one MFMA, then a few vector instructions, 32 times
#pragma unroll
        for (int r = 0; r < 2 * NCB * 4; ++r) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
          __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);  // VALU
          __builtin_amdgcn_sched_group_barrier(0x400, 1, 0);  // transcendental
        }
        __builtin_amdgcn_sched_barrier(0);
        // ---- block 2: P V of sub-tile sub (MFMA) beside the logits of sub-tile nsub (vector ALU) ----
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) st.acc[cb][e] = mfma(pk[cb], vf[e], st.acc[cb][e]);
#pragma unroll
        for (int r = 0; r < 8 * NCB; ++r) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);  // MFMA
          __builtin_amdgcn_sched_group_barrier(0x002, 2, 1);  // VALU
        }
        const bool need = make_logits<DT, NCB, SUBS>(sn, stage, nsub, X, qsum, len_cb, alpha, first_pos,
                                                     v0 + (i * SUBS + nsub) * 4, lane, c, st, cur);
        if (sub + 1 < SUBS && __any(need)) {  // (the wrapped-around sub-tile's logits are discarded)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) wide_move_reference<DT>(st, cb, cur.tmax[cb], j);
        }
      }
      uint8_t* next = smem + (uint32_t)((i + 1) & 1) * stage_bytes(SUBS);
      stage_k<DT, kD>(next, w, lane, t);
      {
        const int live = locate(X, vb_next, j).hi_u;
        stage_v<DT, SUBS, kD>(next, w, lane, !__all(live >= 8), live, t);
      }
      __syncthreads();
    }
  }
  if (n_tok == 0) return;

  const float v_static = DT == FS_KV_FP8_E4M3 ? B.v_scale[head] : 1.0f;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    float l = st.l[cb], zc = st.zc[cb];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if constexpr (F::kParBytes != 0) {
      zc += __shfl_xor(zc, 16, 64);
      zc += __shfl_xor(zc, 32, 64);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int h = 4 * j + r;
      const float Lh = __shfl(l, h, 64), M = __shfl(st.m[cb], h, 64), Z = __shfl(zc, h, 64);
      const int row_h = __shfl(row_cb[cb], h, 64);
      const int tok_h = h / G, hg_h = h - tok_h * G;
      if (tok_h < P.tpt && cb * P.tpt + tok_h < n_tok) {
        const float inv = 1.0f / Lh;
        u32x4 wv;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float o[2];
#pragma unroll
          for (int z = 0; z < 2; ++z) {
            const int e = 2 * q + z;
            const float f = DT == FS_KV_INT8 ? kTwo24 : (DT == FS_KV_INT4 ? ((e & 1) ? kTwo20 : kTwo24) : 1.0f);
            o[z] = st.acc[cb][e][r] * f;
            if constexpr (F::kParBytes != 0) o[z] += Z;
            o[z] *= v_static * inv;
          }
          const half2v hv = {(_Float16)o[0], (_Float16)o[1]};
          wv[q] = h2u(hv);
        }
        const int64_t qrow = (int64_t)row_h * B.n_q + head * G + hg_h;
        *reinterpret_cast<u32x4*>(B.out + qrow * kD + 8 * c) = wv;
        if (c == 0 && B.lse) B.lse[qrow] = (M + __builtin_amdgcn_logf(Lh)) * kLn2;
      }
    }
  }
}

// ---- Direct launches ----------------------------------------------------------------------------------------------
// A launch with no more work items than compute units needs no queue: workgroup b takes one item, found from the
// sequences' tile counts, which every workgroup scans itself (as many sequences as it has threads, at most).  That
// saves the preparation kernel and the gap behind it.  What the preparation also does, the reset of the status word,
// cannot be ordered before other workgroups' reports without it, so the items report to a word that nobody reads (kHdrIgnored)
// and the workgroup of the last item -- the first tile of a head, its shortest -- judges the call as a whole when it is
// done: every length and chunk, and every block-table entry that the sequences with new tokens reach.
constexpr int kBlocks256 = 4;    // ... and of its item at head_dim 256
// Small launches with a long context deal it to two groups of waves, or four where even items of four blocks all find a
// compute unit.  The host does not know the lengths: over tables that can hold contexts long enough it launches the kernel that
// has both walks, and that kernel's scan of the sequences says which (scan_sequences).  The lines, for the longest sequence with
// new tokens; us with every launch forced to either side, items of 8 blocks whose waves all walk the whole context -> groups,
// FP16 / FP8 / INT8 / INT4, 8 KV heads x 4 of 128 unless said otherwise:
//   four groups: 2 x 100 tokens behind 600 21.4 -> 21.4 (FP16), behind 700 23.7 -> 22.9 / 22.4 -> 20.0 / 26.7 -> 23.2 / 25.4 -> 22.9, behind
//   1024 30.2 -> 26.1 / 28.5 -> 23.6 / 35.0 -> 28.1 / 32.9 -> 27.4; but a prompt of 400 15.9 -> 18.6 / 15.2 -> 16.8 / 17.1 -> 18.6 / 16.5 -> 18.7;
//   four groups, at most four blocks of columns a sequence, which leave half the waves of the other walk idle: 6 x 16 tokens
//   behind 700 20.0 -> 23.8 / 19.9 -> 20.8 / 21.9 -> 23.8 / 21.5 -> 23.6, 1024 25.0 -> 27.9 / 25.3 -> 24.1 / 29.4 -> 29.1 / 27.7 -> 28.0, 2048
//   42.2 -> 43.1 / 45.4 -> 35.8 / 52.6 -> 47.4 / 48.7 -> 43.8, 3072 59.3 -> 58.1 / 64.8 -> 48.1 / ...; FP16 at head_dim 64 (16 heads) 1024
//   21.0 -> 19.3;
//   two groups: a prompt of 777 24.9 -> 27.0 (FP16), 2 x 300 behind 1024 30.7 -> 32.5 / 28.8 -> 29.5 / 35.3 -> 34.7 / 33.2 -> 33.3, 1536
//   42.2 -> 42.7 / 39.3 -> 38.3 / 49.4 -> 46.9 / 46.2 -> 44.3, 2048 53.5 -> 52.7 / 49.8 -> 47.1 / 63.7 -> 58.8 / 59.1 -> 55.3.
// (The walk without groups is up to 5 % slower in that kernel than in its own for FP8 and INT4 -- a prompt of 400 tokens 14.8 ->
// 15.2, 15.8 -> 16.6 -- and the same for the others.)
constexpr int group_context(int kv_shift, int dtype, bool d64, bool few_columns) {
  if (kv_shift == 1) return dtype == FS_KV_FP16 ? 2048 : dtype == FS_KV_FP8_E4M3 ? 1536 : 1024;
  return !few_columns ? 640 : dtype == FS_KV_FP16 && !d64 ? 3072 : 1024;
}
constexpr int kSmallBlocks = 8;  // column blocks of the workgroup kernel's smaller item
// The launch's sequences in LDS, where every item's look-ups find them: longest context first, so that the queue ends
// with the shortest items (in the order of the call, 12 INT4 multi-head prompts of 300 - 3000 tokens left the workgroups
// idle for 107 of 885 us at the launch's end on the timeline build, 64 FP16 prompts of 512 - 4096 tokens for 172 of 4800;
// now 48 and 49).  The calls: 796 -> 754 us and 4075 - 4194 -> 3882 - 4110 us, 24 FP16 prompts of 256 - 3000 tokens at
// head_dim 64 646 -> 605 us.
struct SeqList {
  uint32_t* tf;     // [n_seq + 1] first query tile of the k-th longest sequence
  int32_t* seq;     // [n_seq] which sequence that is
  SeqShape* shape;  // [n_seq] by sequence
};
__device__ __forceinline__ SeqList seq_list(void* lds, int n_seq) {
  uint32_t* w = reinterpret_cast<uint32_t*>(lds);
  return SeqList{w, reinterpret_cast<int32_t*>(w + n_seq + 1), reinterpret_cast<SeqShape*>(w + 2 * n_seq + 1)};
}
constexpr uint32_t seq_list_bytes(int n_seq) { return (5u * (uint32_t)n_seq + 1) * 4; }

// Fills the list (n_seq <= threads of the workgroup); returns the number of query tiles.  s_tmp: n_seq + 16 words.
// GROUPS: *s_long says whether some sequence with new tokens is long enough for groups of waves; if none is, the tiles are
// those of items of kSmallBlocks (never more than the host counted).
template <bool GROUPS>
__device__ __forceinline__ uint32_t scan_sequences(const PrefillArgs& P, const SeqList& L, uint32_t* s_tmp, uint32_t* s_long) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = P.b.n_seq;
  uint32_t* s_wave = s_tmp + n;
  SeqShape s{0, 0, 0};
  if (n <= 64) {  // (uniform) one wave's work: no barrier but the last
    if (wave == 0) {
      uint32_t flags = 0;
      if (lane < n) s = seq_shape(P, lane, flags);
      int ncb = P.ncb;
      if constexpr (GROUPS) {
        const bool grouped = __ballot(s.n_new > 0 && s.len >= P.group_len) != 0;
        if (lane == 0) *s_long = grouped;
        ncb = grouped ? ncb : kSmallBlocks;
      }
      int rank = 0;
      for (int i = 0; i < n; ++i) {
        const int l = __builtin_amdgcn_readlane(s.len, i);
        rank += l > s.len || (l == s.len && i < lane);
      }
      const uint32_t v = lane < n ? shape_tiles(P, s, ncb) : 0u;
      uint32_t first = 0;  // tiles of the longer sequences
      for (int i = 0; i < n; ++i) {
        const uint32_t r = __builtin_amdgcn_readlane(rank, i), u = __builtin_amdgcn_readlane(v, i);
        first += (int)r < rank ? u : 0u;
      }
      if (lane < n) {
        L.shape[lane] = s;
        L.seq[rank] = lane;
        L.tf[rank] = first;
        if (rank == n - 1) L.tf[n] = first + v;
      }
    }
    __syncthreads();
    return L.tf[n];
  }
  if (tid < n) {
    uint32_t flags = 0;
    s = seq_shape(P, tid, flags);
    L.shape[tid] = s;
  }
  __syncthreads();
  if (tid < n) {
    int rank = 0, ncb = P.ncb;
    bool grouped = false;
    for (int i = 0; i < n; ++i) {
      const int l = L.shape[i].len;
      rank += l > s.len || (l == s.len && i < tid);
      if constexpr (GROUPS) grouped |= L.shape[i].n_new > 0 && l >= P.group_len;
    }
    if constexpr (GROUPS) {
      if (tid == 0) *s_long = grouped;
      ncb = grouped ? ncb : kSmallBlocks;
    }
    L.seq[rank] = tid;
    s_tmp[rank] = shape_tiles(P, s, ncb);
  }
  __syncthreads();
  uint32_t incl = tid < n ? s_tmp[tid] : 0u;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t u = __shfl_up(incl, off, 64);
    if (lane >= off) incl += u;
  }
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wave; ++w) before += s_wave[w];
  if (tid < n) L.tf[tid + 1] = before + incl;
  if (tid == 0) L.tf[0] = 0;
  __syncthreads();
  return L.tf[n];
}

// The plan of a launch with split items, in LDS: item i of the plan's order (XCD by XCD, an XCD's items in the order of a direct
// launch) has steps cum[i] .. cum[i + 1], workgroup k of that order the steps cut[k] .. cut[k + 1].
struct SplitPlan {
  uint32_t* cum;  // [plan_items + 1]
  uint32_t* cut;  // [workgroups + 1]
  uint16_t* order;     // [8][kSplitItems][workgroups / 8] whole items: XCD, round, workgroup of the XCD -> the XCD's item (0xffff: none) ...
  bool sorted = false; // ... where it has more of them than workgroups
  bool weighed = false;  // steps are those of weighed() (some tiles have all their waves, others less)
  uint32_t turns = 1;  // sequences whose tiles are dealt one from each in turn (see plan_item)
};
constexpr uint32_t split_plan_bytes(uint32_t plan_items) { return (plan_items + 1 + kSplitGroups + 1) * 4 + kSplitItems * kSplitGroups * 2; }
// Lays the plan (n = 8 per items, n <= plan_items, n > 0); false: the items stay whole, each workgroup taking its XCD's in turn.
// That is so where a range has fewer than eight steps, and where the busiest workgroup would not end late enough after the
// mean.  Both count an item's start as two steps (kItemStart): ranges of steps alone held more items where contexts are short, and
// 128 chunks of 16 behind 100 - 3000 took 238 us if cut, 207 with starts counted, 165 whole.  A cut costs its two workgroups an item's
// start and a piece written and read again (six steps in all), and workgroups that read the same context out of step share fewer of
// its lines in their L2.  Where the sequences bring one tile each, or the same number and no more than an XCD has workgroups (the plan
// then goes through the sequences tile by tile, and the ranges of a sequence's tiles begin at nearly the same of its steps), a
// sixteenth more is enough; a quarter elsewhere.  Forced to either side, whole -> cut, us by the busiest workgroup over the mean, FP16 /
// FP8 / INT4, 8 heads x 4: chunks of 16 behind 4000: 40 (68 over 42 steps) 186 -> 145 / 170 -> 127 / 182 -> 136, 80 (102 / 85) 285 -> 260 / 258 ->
// 230 / 277 -> 245, 88 (102 / 93) 291 -> 293 / 261 -> 257 / 279 -> 273, 128 (136 / 136) 388 -> 394 / 346 -> 353 / 371 -> 376; of 64 behind 1000 - 9000:
// 40 (72 / 52) 311 -> 282 / 255 -> 233 / 275 -> 242, 72 (107 / 93) 493 -> 494 / 401 -> 407 / 430 -> 419, 88 (127 / 114) 589 -> 600 / 483 -> 495 / 507 ->
// 515; of 512: 4 behind 1500 - 6000 (45 / 30) 171 -> 146 / 156 -> 136 / 170 -> 143, 6 behind 1500 (32 / 25) 129 -> 126 / 119 -> 116 / 128 -> 124; one
// prompt of 5000 tokens (62 / 55) 244 -> 249 / 224 -> 226 / 242 -> 243, of 4000 (34 / 32) 152 -> 192 / 136 -> 185 / 149 -> 193 (steps alone).
// A last tile's waves without tokens leave the others more of their SIMDs: where tiles differ in that, its steps weigh less (live_sixths;
// 32 chunks behind 4000, us of 26 - 32 / 40 / 48 / 64 tokens: FP16 106 - 113 / 141 / 150 / 169, FP8 91 at 32, 121 / 137 at 48 and 64).
// Whole items are dealt the first two rounds there and back over an XCD's workgroups and the others to whoever has least so far
// (snake, load_rank).  Where a sequence's tiles see mostly the same tokens, in their order: tiles of one sequence run side by side and find
// its lines in the XCD's L2.  Elsewhere -- prompts, whose tiles see from none to all -- by their steps, most first (item_rank).
// us, queue / by steps / by weighed steps / in order: chunks of 154, FP16, 24 behind 689 - 1054 94 / 111 / 103 / 88, 33 130 / 146 / 131 / 118, 33
// behind 1500 - 2500 252 / 268 / 257 / 229; of 100, 60 behind 600 - 1100 153 / 160 / 160 / 154; of 512, 16 behind 600 - 1500 170 / 160 / 160 /
// 155; prompts, five of 600 - 2000, 131 / 121 / 121 / 138.
// Against the ticket queue behind a preparation launch, us: one prompt of 3000
// 138 -> 104 / 128 -> 95 / 140 -> 102; 12 chunks of 300 behind 100 - 16000 705 -> 537 / 594 -> 450 / 664 -> 491; 40 of 64 behind 300 - 1200 79 ->
// 59 / 74 -> 56 / 78 -> 57; three prompts of 1200 - 2000 121 -> 99 (FP16), eight of 256 - 1000 71 -> 66 (FP8); three and four items per unit
// the same within 2 %.  A launch of an item per unit whose contexts are alike pays the plan's first look, 1 us of 55 - 75.
__device__ __forceinline__ SplitPlan split_plan(const SeqList& list, int n_seq, int plan_items) {  // (behind the list of sequences)
  uint32_t* const w = list.tf + 5 * n_seq + 1;
  return SplitPlan{w + kSplitGroups + 1, w, reinterpret_cast<uint16_t*>(w + kSplitGroups + 1 + plan_items + 1)};
}
template <int NT>
__device__ __forceinline__ bool lay_plan(const PrefillArgs& P, SplitPlan& plan, const SeqList& list, uint32_t* s_tmp, uint32_t total,
                                         int step_tokens, int ncb, int nw) {
  // Wave x lays XCD x's part; a lane has its items `lane` and, of more than 64, `lane + 64`.
  static_assert(NT == 512 && kSplitItems * kSplitGroups / 8 <= 128, "a wave for every XCD, two items a lane");
  const uint32_t lane = threadIdx.x & 63, x = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t per = (total + 7) / 8, n = 8 * per, groups = gridDim.x, slots = groups >> 3;
  const int q_wg = P.tpt * ncb * nw, halves = per > 64 ? 2 : 1;
  uint32_t* const cum = plan.cum + x * per + 1;
  auto settle = [] {  // (a wave's LDS operations complete in order; this keeps the compiler from turning them round)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  // the sequences: whether they bring the same number of tiles, and the tokens that the query tiles of one head see
  const uint32_t tiles = list.tf[1];
  bool same = true;
  bool full = false;  // some tile has all its waves
  float seen = 0.f, light = 0.f, behind = 0.f;  // (light: what waves without tokens take off that; behind: of it, before the new tokens)
  auto sixths = [&](int n_new, int qt) {
    const int tokens = min(n_new - qt * q_wg, q_wg), own = P.tpt * ncb;
    return live_sixths((uint32_t)((tokens + own - 1) / own), (uint32_t)nw);
  };
  for (int k = lane; k < P.b.n_seq; k += 64) {
    const uint32_t t = list.tf[k + 1] - list.tf[k];
    const SeqShape s = list.shape[list.seq[k]];
    same = same && t == tiles;
    if (t > 0) {
      const uint32_t w = sixths(s.n_new, (int)t - 1);
      full = full || t > 1 || w == 6;
      seen += (float)t * ((float)(s.len - s.n_new) + 0.5f * (float)(t - 1) * (float)q_wg) + (float)s.n_new;
      behind += (float)t * (float)(s.len - s.n_new);
      light += (float)s.len * (float)(6 - w) * (1.f / 6.f);
    }
  }
  plan.weighed = __any(full);  // (uniform; else all steps are short alike)
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    seen += __shfl_xor(seen, off, 64);
    behind += __shfl_xor(behind, off, 64);
  }
  const bool shared = 2.f * behind >= seen;  // (uniform) a sequence's tiles see mostly the same tokens
  const bool rows = P.by_tile && P.b.g.H % 8 == 0 && tiles * (uint32_t)(P.b.g.H / 8) <= slots;
  const bool even = __all(same) && (tiles == 1 || rows);  // (uniform)
  auto worth = [&](uint32_t mean, uint32_t busy) { return busy > mean + mean / (even ? 16 : 4) + 6; };
  plan.sorted = per > slots;
  if (!plan.sorted) {
    // An item a workgroup at most: none takes longer than the longest sequence's last tile, and the mean is known from below: enough
    // for the launches whose items are all alike.
    if (plan.weighed) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) light += __shfl_xor(light, off, 64);
      seen -= light;
    }
    const float mean = (0.9999f * seen * (float)P.b.g.H / (float)step_tokens + (float)(kItemStart * total)) / (float)groups;
    if (!worth((uint32_t)mean, (uint32_t)((list.shape[list.seq[0]].len - 1) / step_tokens + 1) + kItemStart)) return false;
  }
  uint32_t sum = 0, busy = 0;
#pragma unroll 1
  for (int h = 0; h < halves; ++h) {
    const uint32_t u = lane + 64 * h, item = u < per ? plan_item(P.by_tile, x * per + u, per, 1) : total;
    uint32_t steps = 0;
    int seq, head, qt;
    if (item < total && (P.by_tile ? fs::decode_item_by_tile(list.tf, P.b.n_seq, item, (uint32_t)P.b.g.H, seq, head, qt)
                                   : fs::decode_item(list.tf, P.b.n_seq, item, (uint32_t)P.b.g.H, seq, head, qt))) {
      const SeqShape s = list.shape[list.seq[seq]];
      steps = (uint32_t)(((int64_t)s.len - s.n_new + min((qt + 1) * q_wg, s.n_new) + step_tokens - 1) / step_tokens);
      if (plan.weighed) steps = weighed(steps, sixths(s.n_new, qt));
    }
    if (steps) steps += kItemStart;
    if (u < per) cum[u] = steps;
    sum += steps;
    busy = max(busy, steps);
  }
  settle();
  // what whole items would take the busiest workgroup, an item's start among it
  if (plan.sorted) {  // (uniform)
    uint32_t* const by_rank = s_tmp + 32 + x * 256;  // [128] steps, [128] items, [64] loads behind all of them
    uint32_t* const load = s_tmp + 32 + 8 * 256 + x * 64;
    bool falling = true;  // (so are one sequence's tiles, and sequences of one tile each)
    for (int h = 0; h < halves; ++h) {
      const uint32_t u = lane + 64 * h;
      if (u + 1 < per) falling = falling && cum[u] >= cum[u + 1];
    }
    falling = shared || __all(falling);
#pragma unroll 1
    for (int h = 0; h < halves; ++h) {
      const uint32_t u = lane + 64 * h;
      if (u >= per) continue;
      const uint32_t rank = falling ? u : item_rank(cum, per, u);
      by_rank[rank] = cum[u];
      by_rank[128 + rank] = u;
    }
    settle();
    busy = 0;
#pragma unroll 1
    for (uint32_t first = 0; first < per; first += slots) {
      load[lane] = busy;
      settle();
      // the first two rounds there and back, the others to whoever has least so far
      const uint32_t k = lane < slots ? lane : slots - 1;
      const uint32_t at = first < 2 * slots ? snake(first + k, slots) : first + load_rank(load, slots, k);
      if (lane < slots) {
        const bool has = at < per;
        plan.order[(x * kSplitItems + first / slots) * slots + lane] = has ? (uint16_t)by_rank[128 + at] : (uint16_t)0xffff;
        if (has) busy += by_rank[at];
      }
      settle();
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    sum += __shfl_xor(sum, off, 64);
    busy = max(busy, (uint32_t)__shfl_xor(busy, off, 64));
  }
  if (lane == 0) s_tmp[x] = sum, s_tmp[8 + x] = busy;
  __syncthreads();
  uint32_t steps = 0, before = 0;
#pragma unroll
  for (uint32_t k = 0; k < 8; ++k) {
    before += k < x ? s_tmp[k] : 0u;
    steps += s_tmp[k];
    busy = max(busy, s_tmp[8 + k]);
  }
  const uint32_t mean = steps / groups;
  if (mean < kSplitLeast || !worth(mean, busy)) return false;
  // running sums, the XCD's first step in front of them
  if (even && rows) plan.turns = (uint32_t)P.b.n_seq;
  uint32_t mine[2] = {0, 0};
  for (int h = 0; h < halves; ++h) {
    const uint32_t u = lane + 64 * h;
    if (u < per) mine[h] = cum[dealt(u, per, plan.turns)];
  }
  settle();
  for (int h = 0; h < halves; ++h) {
    const uint32_t u = lane + 64 * h;
    uint32_t incl = mine[h];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t up = __shfl_up(incl, off, 64);
      if ((int)lane >= off) incl += up;
    }
    if (u < per) cum[u] = before + incl;
    before += __shfl(incl, 63, 64);
  }
  if (threadIdx.x == 0) plan.cum[0] = 0;
  __syncthreads();
  for (uint32_t k = threadIdx.x; k <= groups; k += NT) plan.cut[k] = plan_cut(plan.cum, n, groups, k);
  __syncthreads();
  return true;
}

// Every sequence's share of the threads (a power of two, n_seq <= NT) reads its table, eight entries a thread in flight: one
// workgroup does this alone, at the launch's end where all are done at the same time.  us, a wave for a sequence after the other ->
// like this: 500 FP16 chunks of 8 behind 2000, one KV head, 171 -> 129; 510 INT4 ones behind 8000 403 -> 363.
template <int NT>
__device__ __forceinline__ void direct_status(const PrefillArgs& P, uint32_t* s_flags) {
  const DevBatch& B = P.b;
  if (threadIdx.x == 0) *s_flags = 0;
  __syncthreads();
  uint32_t flags = 0;
  int share = NT;
  while (share > 1 && share * B.n_seq > NT) share >>= 1;
  const int seq = threadIdx.x / share, own = threadIdx.x & (share - 1);
  if (seq < B.n_seq) {
    const SeqShape s = seq_shape(P, seq, flags);
    const int nb = s.n_new == 0 ? 0 : (s.len + B.g.T - 1) / B.g.T;
    const int32_t* table = B.tables + (int64_t)seq * B.max_blocks;
    for (int i = own; i < nb; i += 8 * share) {
      uint32_t most = 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) most = max(most, (uint32_t)table[min(i + k * share, nb - 1)]);
      flags |= most < B.n_blocks ? 0u : 4u;
    }
  }
  if (flags) atomicOr(s_flags, flags);
  __syncthreads();
  if (threadIdx.x == 0) P.header[kHdrStatus] = *s_flags;
}

// WPC = workgroups per compute unit the kernel is built for.  GROUPS: the groups' items, or -- where the scan finds no context
// long enough -- those of the small launches' kernel, one block per wave.
template <int DT, int NW, int NCB, int SUBS, int WPC, bool PIPE = false, bool DEQ = false, int HD = kD, bool SUM32 = false, bool GROUPS = false, bool SPLIT = false>
__global__ __launch_bounds__(NW * 64, WPC) void prefill_wg_kernel(PrefillArgs P) {
  extern __shared__ uint64_t smem64[];
  const DevBatch& B = P.b;
  uint8_t* smem = reinterpret_cast<uint8_t*>(smem64);
  uint64_t* s_tab = reinterpret_cast<uint64_t*>(smem + 2 * stage_bytes(SUBS, HD));
  uint32_t* s_ctl = reinterpret_cast<uint32_t*>(smem + 2 * stage_bytes(SUBS, HD) + (size_t)P.table_entries * 8);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t H = (uint32_t)B.g.H;
  uint32_t* s_tf = reinterpret_cast<uint32_t*>(smem + 2 * stage_bytes(SUBS, HD) + (size_t)P.table_entries * 8 + kWgCtlBytes);
  const bool direct = GROUPS || SPLIT || (!PIPE && P.direct);  // (uniform)
  uint32_t* const header = direct ? P.header + kHdrIgnored - kHdrStatus : P.header;
  const uint32_t* tf = P.tile_first;
  const SeqList list = seq_list(s_tf, B.n_seq);
  uint32_t total;
  const bool listed = GROUPS || SPLIT || (!PIPE && P.tf_cache == 2);  // (uniform; always so in a direct launch)
  if (listed) {
    total = __builtin_amdgcn_readfirstlane(scan_sequences<GROUPS>(P, list, reinterpret_cast<uint32_t*>(smem), s_ctl)) * H;
    tf = list.tf;
  } else {
    total = P.tile_first[B.n_seq] * H;
    if (P.tf_cache) {  // (uniform)
      for (int i = threadIdx.x; i <= B.n_seq; i += NW * 64) s_tf[i] = P.tile_first[i];
      __syncthreads();
      tf = s_tf;
    }
  }
#ifdef FS_TIMELINE
  const uint64_t tl_start = wall_clock64();
  uint64_t tl_items = 0;
#endif
  // the workgroup's work items
  auto items = [&](auto ncb_c, auto groups_c) __attribute__((always_inline)) {
    // direct: consecutive items, which stream the same keys and values, on one XCD (workgroups are dealt to the XCDs in
    // turn); workgroup b takes items (b % 8) per + b / 8, + slots, ... of its XCD's share
    const uint32_t per = (total + 7) / 8, slots = gridDim.x >> 3;  // (the host launches a multiple of eight)
    uint32_t u = blockIdx.x >> 3;
    ItemDraw d{0u, 0u};
    SeqHeld held;
    uint32_t turn = 0;
    Piece piece;
    // (SPLIT) the workgroup's range of steps, and the item that its next step belongs to
    uint32_t at = 0, end = 0, i_plan = 0, me = 0;
    SplitPlan plan = split_plan(list, B.n_seq, P.plan_items);
    bool split = false;
    if constexpr (SPLIT) {
      if (per > 0 && 8 * per <= (uint32_t)P.plan_items)
        split = __builtin_amdgcn_readfirstlane(lay_plan<NW * 64>(P, plan, list, reinterpret_cast<uint32_t*>(smem), total, 32 * SUBS, NCB, NW));
      __syncthreads();  // (the first stage goes where its scratch word is)
      if (split) {
        me = (blockIdx.x & 7) * slots + (blockIdx.x >> 3);
        at = __builtin_amdgcn_readfirstlane(plan.cut[me]);
        end = __builtin_amdgcn_readfirstlane(plan.cut[me + 1]);
        i_plan = __builtin_amdgcn_readfirstlane(item_of_step(plan.cum, 8 * per, at));
      }
      piece.s_count = s_ctl + 2;
    }
    if (wave == 0 && !direct) d = first_draw(P.header, blockIdx.x >> 3, lane);
    for (;;) {
#ifdef FS_TIMELINE
      const uint64_t tl_top = wall_clock64();
#endif
      uint32_t item;
      if (SPLIT && split) {
        if (at >= end) break;
        const uint32_t from = __builtin_amdgcn_readfirstlane(plan.cum[i_plan]), to = __builtin_amdgcn_readfirstlane(plan.cum[i_plan + 1]);
        item = plan_item(P.by_tile, i_plan, per, plan.turns);
        ++i_plan;
        if (to <= at) continue;  // (an item without steps)
        piece.step = at > from ? (int)(at - from - kItemStart) : 0;
        piece.end = to <= end ? 0x7fffffff : (int)(end - from - kItemStart);
        uint32_t last;
        piece_owners(plan.cut, me, from, to, piece.first, last);
        piece.first = __builtin_amdgcn_readfirstlane(piece.first);
        piece.n = __builtin_amdgcn_readfirstlane(last) - piece.first + 1;
        piece.own = me - piece.first;
        at = min(to, end);
      } else if (direct) {
        if constexpr (SPLIT) {  // (whoever had the longest item of one round has the shortest of the next)
          if (u - u % slots >= per) break;
          const uint32_t v = plan.sorted ? __builtin_amdgcn_readfirstlane((uint32_t)plan.order[(blockIdx.x & 7) * kSplitItems * slots + u]) : u;
          u += slots;
          if (v >= per) continue;
          item = P.by_tile ? 8 * v + (blockIdx.x & 7) : (blockIdx.x & 7) * per + v;
          if (item >= total) continue;
        } else {
          item = P.by_tile ? 8 * u + (blockIdx.x & 7) : (blockIdx.x & 7) * per + u;
          if (u >= per || item >= total) break;
          u += slots;
        }
      } else {
        if (wave == 0) {  // one wave draws for the workgroup
          const bool ok = next_item(d, P.header, total, (uint32_t)P.chunk_shift, lane, item);
          if (lane == 0) s_ctl[turn] = ok ? item : 0xffffffffu;
        }
        __syncthreads();
        // (an LDS load is not uniform to the compiler; the next draw writes the other word, the one after it lies behind
        // a barrier that every wave passes with this item in hand)
        item = __builtin_amdgcn_readfirstlane(s_ctl[turn]);
        turn ^= 1;
        if (item == 0xffffffffu) break;
      }
      int seq, head, qt;
      const int found = P.by_tile ? fs::decode_item_by_tile(tf, B.n_seq, item, H, seq, head, qt) : decode_item(P, tf, item, H, seq, head, qt);
      if (!__builtin_amdgcn_readfirstlane(found)) continue;  // (uniform, so that what lives across items stays scalar)
      uint32_t unused = 0;
      seq = __builtin_amdgcn_readfirstlane(listed ? list.seq[seq] : seq);
      SeqShape shape = listed ? list.shape[seq] : seq_shape(P, seq, unused);
      shape.len = __builtin_amdgcn_readfirstlane(shape.len);
      shape.n_new = __builtin_amdgcn_readfirstlane(shape.n_new);
      shape.q0 = __builtin_amdgcn_readfirstlane(shape.q0);
      // (the same in every lane; said so, the item's addresses and bounds live in scalar registers: FP16 needs no
      // scratch any more, and 64 prompts of 512 - 4096 tokens run 4232 -> 4126 us)
      head = __builtin_amdgcn_readfirstlane(head);
      qt = __builtin_amdgcn_readfirstlane(qt);
      if constexpr (SPLIT) {
        if (split && plan.weighed) {  // (steps of the plan -> steps of the item; the next piece's step comes of the same number)
          const int own = P.tpt * NCB, tokens = min(shape.n_new - qt * own * NW, own * NW);
          const uint32_t w = live_sixths((uint32_t)((tokens + own - 1) / own), NW);
          piece.step = (int)step_at((uint32_t)piece.step, w);
          if (piece.end != 0x7fffffff) piece.end = (int)step_at((uint32_t)piece.end, w);
        }
      }
#ifdef FS_TIMELINE
      const uint64_t tl_begin = wall_clock64();
#endif
      if constexpr (PIPE) prefill_item_wgp<DT>(P, seq, head, qt, smem, s_tab, wave);
      else prefill_item_wg<DT, NW, decltype(ncb_c)::value, SUBS, DEQ, HD, SUM32, decltype(groups_c)::value, SPLIT>(P, header, seq, shape, head, qt, smem, s_tab, wave, held, piece);
#ifdef FS_TIMELINE
      ++tl_items;
      if (threadIdx.x == 0 && item < kPfTimelineItems) {
        uint64_t* row = P.timeline + 8 * (kPfTimelineGroups + item);
        row[0] = tl_begin;
        row[1] = wall_clock64();
        row[2] = ((uint64_t)seq << 32) | ((uint64_t)head << 20) | (uint64_t)qt;
        row[3] = (uint64_t)blockIdx.x | ((tl_begin - tl_top) << 32);
      }
#endif
    }
  };
  if constexpr (GROUPS) {
    if (__builtin_amdgcn_readfirstlane(s_ctl[0])) items(std::integral_constant<int, NCB>{}, std::true_type{});
    else items(std::integral_constant<int, 1>{}, std::false_type{});
  } else {
    items(std::integral_constant<int, NCB>{}, std::false_type{});
  }
  if (direct) {
    const uint32_t last = total ? total - 1 : 0u, per = (total + 7) / 8, slots = gridDim.x >> 3, n = total ? per : 1u;
    if (blockIdx.x == (P.by_tile ? last % gridDim.x : (last % n % slots) * 8 + last / n)) direct_status<NW * 64>(P, reinterpret_cast<uint32_t*>(smem));
  }
#ifdef FS_TIMELINE
  if (threadIdx.x == 0 && blockIdx.x < kPfTimelineGroups) {
    uint64_t* row = P.timeline + 8 * blockIdx.x;
    row[0] = tl_start;
    row[1] = wall_clock64();
    row[2] = tl_items;
    row[3] = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7;  // hwreg(HW_REG_XCC_ID, 0, 4)
  }
#endif
}

// The 16-column kernel (HD: its tile code takes any of the three head_dims).
template <int HD>
__global__ __launch_bounds__(kThreads, mfma_wgs_per_cu(HD)) void prefill_kernel(PrefillArgs P) {
  extern __shared__ uint64_t smem64[];
  const DevBatch& B = P.b;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint64_t* s_ptr = smem64 + (size_t)wave * P.table_entries;
  const uint32_t H = (uint32_t)B.g.H;
  const uint32_t total = P.tile_first[B.n_seq] * H;
  ItemDraw d = first_draw(P.header, (blockIdx.x >> 3) * kWaves + wave, lane);
  for (uint32_t item; next_item(d, P.header, total, kWaveChunkShift, lane, item);) {
    int seq, head, qt;
    if (!decode_item(P, P.tile_first, item, H, seq, head, qt)) continue;
    switch (B.g.dtype) {
      case FS_KV_FP16: prefill_item<FS_KV_FP16, HD>(P, seq, head, qt, s_ptr); break;
      case FS_KV_FP8_E4M3: prefill_item<FS_KV_FP8_E4M3, HD>(P, seq, head, qt, s_ptr); break;
      case FS_KV_INT8: prefill_item<FS_KV_INT8, HD>(P, seq, head, qt, s_ptr); break;
      default: prefill_item<FS_KV_INT4, HD>(P, seq, head, qt, s_ptr); break;
    }
  }
}

uint64_t align256(uint64_t x) { return (x + 255) & ~255ull; }

}  // namespace
}  // namespace fs

using namespace fs;

#ifdef FS_TIMELINE
// (timeline build only) bytes of the clock readings at the end of a prefill workspace, and their layout
extern "C" uint64_t fs_prefill_timeline_bytes(uint64_t* group_rows, uint64_t* item_rows) {
  if (group_rows) *group_rows = kPfTimelineGroups;
  if (item_rows) *item_rows = kPfTimelineItems;
  return kPfTimelineBytes;
}
#endif

// The workspace: header and first tiles, which every launch needs, then the pieces of split items; a workspace that ends before
// these is served as well, with whole items.  (Timeline build: the readings lie at the end, and it has to be all there.)
static uint64_t pieces_at(int n_seq) { return align256(kHeaderBytes + 4ull * ((uint64_t)n_seq + 1)); }
#ifdef FS_TIMELINE
uint64_t fs_prefill_workspace_bytes(int n_seq) { return n_seq < 1 ? 0 : align256(pieces_at(n_seq) + kPiecesBytes) + kPfTimelineBytes; }
uint64_t fs_prefill_least_workspace_bytes(int n_seq) { return fs_prefill_workspace_bytes(n_seq); }
#else
uint64_t fs_prefill_workspace_bytes(int n_seq) { return n_seq < 1 ? 0 : pieces_at(n_seq) + kPiecesBytes; }
uint64_t fs_prefill_least_workspace_bytes(int n_seq) { return n_seq < 1 ? 0 : pieces_at(n_seq); }
#endif

int fs_prefill_attention(fs_pool* p, fs_model_t model, int layer, int n_q_heads, float sm_scale, const void* q,
                         const int32_t* block_tables, const int32_t* seq_lens, const int32_t* q_offsets,
                         const int32_t* q_offsets_host, int n_seq, int max_blocks, void* out, float* lse, void* workspace,
                         uint64_t workspace_bytes, void* stream) {
  if (!p || model < 0 || model >= kMaxModels || !p->models[model].in_use) {
    set_error("prefill attention: unknown pool or model");
    return FS_ERR_INVALID;
  }
  const Model& M = p->models[model];
  const fs_geometry_t& g = M.g;
  if (layer < 0 || layer >= g.n_layers || n_seq < 1 || max_blocks < 1 || !q || !block_tables || !seq_lens || !q_offsets ||
      !q_offsets_host || !out || n_q_heads < g.n_kv_heads || n_q_heads % g.n_kv_heads || !(sm_scale == sm_scale)) {
    set_error("prefill attention: invalid argument");
    return FS_ERR_INVALID;
  }
  if (((uintptr_t)q | (uintptr_t)out) & 15) {
    set_error("prefill attention: q and out must be 16-byte aligned");
    return FS_ERR_INVALID;
  }
  if (q_offsets_host[0] != 0) {
    set_error("prefill attention: q_offsets must start at 0");
    return FS_ERR_INVALID;
  }
  const int G = n_q_heads / g.n_kv_heads;
  if (G > 16) {
    set_error("prefill attention: more than 16 query heads per KV head");
    return FS_ERR_INVALID;
  }
  const int tpt = 16 / G;
  // (FS_OPT_PREFILL_COLUMN_BLOCKS chooses among variants that are built for head_dim 128: one setting for a pool must not
  // take its models of head_dim 64 and 256 off the kernel that suits their launches)
  const int ncb_env = g.head_dim == kD ? p->opt.prefill_ncb : 0;
  // the wide kernels fold the (positive) softmax scale into the exponential's argument; any other scale takes
  // the 16-column kernel, which does not
  const bool scale_ok = sm_scale > 0.f && sm_scale < INFINITY;
  // (head_dim 64: the 8-wave workgroup kernels or the 16-column kernel; 256: the 4-wave workgroup kernel of one block per
  // wave or the 16-column kernel)
  const bool d64 = g.head_dim == 64, d256 = g.head_dim == 256;
  int ncb = !scale_ok || (g.head_dim != kD && !d64 && !d256) ? 1 : (ncb_env ? ncb_env : 16);
  if (d256 && ncb == 16) ncb = kBlocks256;
  uint64_t tiles = 0;
  int kv_shift = 0, group_len = 0;
  auto count_tiles = [&](int blocks) {
    tiles = 0;
    for (int b = 0; b < n_seq; ++b) {
      const int64_t n_new = (int64_t)q_offsets_host[b + 1] - q_offsets_host[b];
      if (n_new < 0) return false;
      tiles += (uint64_t)((n_new + tpt * blocks - 1) / (tpt * blocks));
    }
    return true;
  };
  if (!count_tiles(ncb)) {
    set_error("prefill attention: q_offsets must not decrease");
    return FS_ERR_INVALID;
  }
  // By default the workgroup kernel with 16 blocks per item; with 8 blocks (eight waves of one block each) where even
  // those items all find a compute unit of their own: twice the units work, and a step takes little more than half the
  // time.  A prompt of 777 tokens, 8 KV heads x 4 of 128: 66 us in the 16-column kernel that served launches with fewer
  // items than compute units before, 27.5 us with 8 blocks (200 items); one of 1500 tokens: 137 us, 75 with 8 blocks
  // (376 items: some units take two), 60 with 16 (188 items).  (us, items of 16 -> of 8, FP16 / FP8 / INT4: one of 777 34.4 -> 24.4 / 31.7 ->
  // 23.0 / 36.4 -> 25.5, of 1000 41.3 -> 30.0 / 38.0 -> 28.3 / 44.1 -> 31.5; past an item of 8 per unit: of 1040 42.7 -> 34.0 / 39.0 -> 32.7 / 45.3 ->
  // 35.6, of 1200 47.7 -> 47.0 / 43.4 -> 44.2 / 51.6 -> 49.1, of 1750 65.3 -> 71.0 / 59.6 -> 67.4 / 71.5 -> 75.0, 4 of 400 24.7 -> 31.1 / 23.2 ->
  // 29.2 / 25.2 -> 31.3, 24 chunks of 64 behind 2000 85 -> 120 / 73 -> 104 / 87 -> 116.)
  if (ncb == 16 && !ncb_env && tiles * (uint64_t)g.n_kv_heads < (uint64_t)p->n_cu) {
    (void)count_tiles(kSmallBlocks);
    // (head_dim 64: too few items to matter stay with the 16-column kernel; two prompts of 100 and 600 tokens with 4 KV
    // heads: 29 us)
    if (tiles * (uint64_t)g.n_kv_heads <= (uint64_t)p->n_cu) ncb = d64 && tiles * (uint64_t)g.n_kv_heads < 64 ? 1 : kSmallBlocks;
    if (ncb != kSmallBlocks) (void)count_tiles(ncb);
    else if (n_seq <= 8 * 64) {  // (the workgroups list the sequences)
      const uint64_t at8 = tiles;
      (void)count_tiles(kSmallBlocks / 2);
      const int shift = tiles * (uint64_t)g.n_kv_heads <= (uint64_t)p->n_cu ? 2 : 1;
      int most = 0;
      for (int b = 0; b < n_seq; ++b) most = std::max(most, q_offsets_host[b + 1] - q_offsets_host[b]);
      group_len = group_context(shift, g.kv_dtype, d64, most <= 4 * tpt);
      if ((int64_t)max_blocks * g.tokens_per_block >= group_len) kv_shift = shift;
      if (kv_shift == 2) ncb = kSmallBlocks / 2;
      else tiles = at8;
    }
  }
  // head_dim 256: the workgroup kernel, one wave per SIMD, for FP16 and for launches of no more items than compute units
  // (and at least half as many); the other formats' larger launches have enough waves in the 16-column kernel, which
  // reads half the bytes per row.  12 prompts of 300 - 3000 tokens, 4 KV heads x 4: FP16 1541 -> 1176 us, but FP8 861 ->
  // 1089; one FP16 prompt of 900 tokens 95 -> 52.5 us.
  if (ncb == kBlocks256 && d256 && !ncb_env &&
      (tiles * (uint64_t)g.n_kv_heads < (uint64_t)p->n_cu / 2 ||
       (g.kv_dtype != FS_KV_FP16 && tiles * (uint64_t)g.n_kv_heads > (uint64_t)p->n_cu))) {
    ncb = 1;
    (void)count_tiles(ncb);
  }
  // head_dim 64: items of 32 blocks (FP16) or 24 (the other formats, whose staging needs the registers), four or three per
  // wave, where there are at least eight per compute unit and they are as full as those of 16: half or two thirds of the
  // staging and of the operand reads per product, but 1.65 or 1.35 times an item.  us, 8 heads x 4, items of 16 -> wide ones, prompts of
  // 256 - 3000 tokens, by wide items per unit: FP16 at 4 268 -> 261, 6 374 -> 369, 8 487 -> 471, 9 552 -> 506, 12 710 -> 647, 16 934 -> 856;
  // INT8 at 4 251 -> 267, 5 281 -> 302, 6 328 -> 323, 8 429 -> 404, 12 632 -> 596; INT4 at 6 343 -> 334, 8 452 -> 419; FP8 at 6 278 -> 272, 8 358 ->
  // 344; prompts of 5000 - 12000 at 8 FP16 1791 -> 1693, INT8 1628 -> 1550; 64 chunks of 64 tokens (half-empty items) 132 -> 152.
  if (d64 && ncb == 16 && !ncb_env) {
    const uint64_t at16 = tiles;
    const int wide = g.kv_dtype == FS_KV_FP16 ? 32 : 24;
    (void)count_tiles(wide);
    if (tiles * (uint64_t)g.n_kv_heads >= 8 * (uint64_t)p->n_cu && tiles * (uint64_t)wide <= at16 * 16 + at16 * 16 / 10) ncb = wide;
    else tiles = at16;
  }
  const int64_t n_rows = q_offsets_host[n_seq];
  if (tiles * (uint64_t)g.n_kv_heads > 0xfffffff0ull || n_rows > 0x7fffffff) {
    set_error("prefill attention: batch too large");
    return FS_ERR_INVALID;
  }
  if (g.kv_dtype == FS_KV_FP8_E4M3 && !M.d_k_scale) {
    set_error("prefill attention: FP8 model has no scales (fs_model_set_fp8_scales)");
    return FS_ERR_INVALID;
  }
  if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < fs_prefill_least_workspace_bytes(n_seq)) {
    set_error("prefill attention: workspace missing, not 256-byte aligned or too small (see fs_prefill_workspace_bytes)");
    return workspace && !((uintptr_t)workspace & 255) ? FS_ERR_NOMEM : FS_ERR_INVALID;
  }
  if (p->n_cu == 0) {
    set_error("prefill attention: pool has no HIP device");
    return FS_ERR_DEVICE;
  }
  PrefillArgs P{};
  DevBatch& B = P.b;
  B.g = dev_geom(g);
  B.layer_base = p->base + (uint64_t)layer * g.layer_bytes;
  B.q = (const _Float16*)q;
  B.tables = block_tables;
  B.seq_lens = seq_lens;
  B.out = (_Float16*)out;
  B.lse = lse;
  B.k_scale = M.d_k_scale ? M.d_k_scale + (size_t)layer * g.n_kv_heads : nullptr;
  B.v_scale = M.d_v_scale ? M.d_v_scale + (size_t)layer * g.n_kv_heads : nullptr;
  B.n_seq = n_seq;
  B.max_blocks = max_blocks;
  B.n_q = n_q_heads;
  B.G = G;
  B.sm_scale = sm_scale;
  B.R = (g.tokens_per_block + 7) / 8;
  B.r_magic = B.R == 1 ? 0u : (uint32_t)(((1ull << 32) + (uint64_t)B.R - 1) / (uint64_t)B.R);
  B.n_blocks = (uint32_t)(p->pool_bytes / g.block_budget);
  for (int t = 0; t < kTierSteps; ++t) B.tier_seq[t] = 0x7fffffff;  // (decode's split sizes: not used by prefill)
  B.ring_runs = 4;
  const bool generic = !mfma_supports(B);  // head_dim other than 64, 128 or 256, or blocks of fewer than 8 tokens
  if (generic && (g.head_dim & (g.head_dim - 1))) {
    set_error("prefill attention: head_dim must be a power of two");
    return FS_ERR_INVALID;
  }
  P.q_offsets = q_offsets;
  P.header = (uint32_t*)workspace;
  P.tile_first = (uint32_t*)((uint8_t*)workspace + kHeaderBytes);
#ifdef FS_TIMELINE
  P.timeline = (uint64_t*)((uint8_t*)workspace + fs_prefill_workspace_bytes(n_seq) - kPfTimelineBytes);
#endif
  P.tpt = tpt;
  P.ncb = ncb;
  P.kv_shift = kv_shift;
  P.group_len = group_len;
  P.seg_runs = prefill_seg_runs(B.R);
  P.seg_tokens = prefill_seg_tokens(g.tokens_per_block);
  P.t_magic = token_magic(g.tokens_per_block);
  P.table_entries = std::max(prefill_table_entries(P.seg_runs, B.R), P.seg_tokens / g.tokens_per_block + 3);
  P.n_rows = (int32_t)n_rows;
  P.whole_runs = (g.tokens_per_block & 7) == 0;
  if (n_rows == 0) return FS_OK;
  hipStream_t s = (hipStream_t)stream;
  (void)hipGetLastError();
  const uint64_t items = tiles * (uint64_t)g.n_kv_heads;
  const bool wg = ncb >= 16 || kv_shift || ncb == kSmallBlocks || (d256 && ncb == kBlocks256);
  // (FS_OPT_PREFILL_WAVES is about the launches that have a 16-block item per compute unit; a smaller launch by the
  // library's own choice keeps the integer codes exact and its sums over the unrounded weights, as the 16-column kernel that
  // served it before, and the 4-wave kernels are not built like that)
  const bool large = ncb_env || items >= (uint64_t)p->n_cu;
  const int nw = d256 || (p->opt.prefill_nw == 4 && ncb == 16 && !d64 && large) ? 4 : 8;
  // the workgroups list the sequences themselves while they have a thread for each; the per-sequence tile counts of more
  // go to LDS while they fit beside the stages (16 KiB: 4095 sequences)
  P.tf_cache = !wg || generic ? 0 : (nw == 8 || d256) && n_seq <= nw * 64 ? 2 : (uint64_t)n_seq + 1 <= 4096;
  // no more items than compute units: a direct launch (see "Direct launches")
  P.direct = P.tf_cache == 2 && items <= (uint64_t)p->n_cu;
  // Split items: up to four of 16 blocks per compute unit (the queue deals more as evenly: 3 prompts of 2000 - 6000 tokens, 3.8 per
  // unit, 509 us with either), where the tables can hold eight steps (the workgroups, who see the lengths, decide: see lay_plan)
  // and the workspace has room for the pieces.
  const bool deq_on = p->opt.prefill_deq || g.kv_dtype == FS_KV_FP16 || g.kv_dtype == FS_KV_FP8_E4M3;
  const uint32_t split_groups = std::min<uint32_t>(kSplitGroups, (uint32_t)p->n_cu & ~7u);
  const int64_t capacity = std::min<int64_t>((int64_t)max_blocks * g.tokens_per_block, 0x7fffffff);
  bool split = P.tf_cache == 2 && g.head_dim == kD && nw == 8 && ncb == 16 && !ncb_env && large && deq_on && split_groups >= 8 &&
               items <= kSplitItems * (uint64_t)split_groups && capacity >= 128 * (int64_t)kSplitLeast &&
               (uint64_t)(capacity / 128 + 2 + kItemStart) * items < (1ull << 31) &&  // (sums of steps)
               workspace_bytes >= fs_prefill_workspace_bytes(n_seq);
  P.plan_items = (int32_t)((items + 7) / 8 * 8);
  P.pieces = (uint8_t*)workspace + pieces_at(n_seq);
  const size_t smem_split = 2 * (size_t)stage_bytes(4, g.head_dim) + (size_t)P.table_entries * 8 + kWgCtlBytes + seq_list_bytes(n_seq) +
                            split_plan_bytes((uint32_t)P.plan_items);
  if (smem_split > 160 * 1024) split = false;
  if (split) P.direct = 1;
  hipError_t e = hipSuccess;
  if (!P.direct) {
    hipLaunchKernelGGL(prefill_prep_kernel, dim3(1), dim3(kPrepThreads), 0, s, P);
    e = hipGetLastError();
    if (e != hipSuccess) return device_error(e, "prefill prep launch");
  }
  if (generic) {
    // one workgroup per (query row, KV head) on the vector ALU: every shape the pool can hold
    MultiArgs A{};
    A.b[0] = B;
    A.header = P.header;
    A.n_batches = 1;
    const uint64_t work = (uint64_t)n_rows * (uint64_t)g.n_kv_heads;
    p->opt.last_prefill = 1 << 18;
    p->opt.last_items = 0;
    e = launch_generic_prefill(A, q_offsets, (int)n_rows, (int)std::min<uint64_t>(work, (uint64_t)p->n_cu * 8), s);
    if (e != hipSuccess) return device_error(e, "prefill launch (generic kernel)");
    return FS_OK;
  }
  p->opt.last_items = ncb | (kv_shift << 8);
  // waves per SIMD: the 16-column kernel runs two, the wider wave-level ones one
  const int wps = ncb == 1 ? mfma_wgs_per_cu(g.head_dim) : 1;
  // workgroup kernels: 16 blocks = 8 waves x 2 (default) or 4 x 4, 4 sub-tiles per step, one workgroup per compute unit
  const int subs = d256 ? 2 : 4, wpc = 1;
  const int n_wg = split ? (int)split_groups : P.direct ? (int)((items + 7) / 8 * 8) : wg ? (int)std::min<uint64_t>((uint64_t)p->n_cu * wpc, std::max<uint64_t>(items, 1))
                      : (int)std::min<uint64_t>((uint64_t)p->n_cu * wps, std::max<uint64_t>((items + kWaves - 1) / kWaves, 1));
  // (The other kernels, and other numbers of heads:) consecutive items -- the query tiles of one (sequence, head), which stream
  // the same K/V -- go to one XCD in chunks of 128 (a head of 8192 tokens in one piece: measured + 1.4 % over chunks of 32 on long prompts), of
  // fewer while that leaves an XCD less than eight chunks to balance with.
  P.chunk_shift = 7;
  while (P.chunk_shift > (int32_t)kWgChunkShift && (items >> P.chunk_shift) < 64) --P.chunk_shift;
  // Where the heads allow it (see decode_item_by_tile) the workgroup kernels take a sequence's tiles longest first over all its
  // heads, dealt to the XCDs in turn: head by head, a launch's last head began with its longest tile.  us, head by head -> by
  // tile: one FP16 prompt of 3000 tokens, GQA 4:1, 155 -> 139; two of 1107 and 2179 124 -> 114; four FP8 ones of 500 - 2000, GQA
  // 8:1, 194 -> 174; two of 7000 and 8000, 8 / 16 / 40 heads, 1114 -> 968 / 1098 -> 971 / 1449 -> 1309; 12 of 500 - 3500 the same within
  // 1.5 %; 4 heads: two of 7000 and 8000 594 -> 573, six FP8 ones of 11000 - 16000 4202 -> 4029, 48 of 500 - 3500 1129 -> 1136.
  // One or two heads put a head's tiles on eight or four XCDs, each of which fetches the context.  That pays while the launch's
  // end matters: 12 prompts (5 items per unit) 322 -> 314 / 324 -> 323, six FP8 ones of 11000 - 16000 (20) 4116 -> 3993 / 4151 -> 4001;
  // two of 7000 and 8000 (4) 568 -> 575 / 562 -> 575; but 48 of 500 - 3500 (23) 1105 -> 1120 / 1112 -> 1124 and 24 of 14000 - 16000 (87)
  // 21045 -> 21929 / 21370 -> 21957.
  // Launches that may split items take this order with any number of heads: head by head, the XCD with the longest contexts ended
  // long after the others, and whole items stay on their XCD there.  us, head by head -> by tile: 60 chunks of 16 behind 200 - 4000, 12
  // heads 239 -> 180, FP8 with 10 heads 189 -> 144; 12 prompts of 300 - 1500, 5 heads 75 -> 64; eight chunks of 1024 behind 976, 5 heads
  // 105 -> 110 (all three in the queue, behind a preparation launch: 192, 155, 86 and 142).
  P.by_tile = wg && (split || g.n_kv_heads % 8 == 0 || g.n_kv_heads == 4 || (g.n_kv_heads <= 2 && items <= 20 * (uint64_t)p->n_cu));
  if (P.by_tile) P.chunk_shift = 0;
  const size_t smem = split ? smem_split : wg ? 2 * (size_t)stage_bytes(subs, g.head_dim) + (size_t)P.table_entries * 8 + kWgCtlBytes +
                               (P.tf_cache == 2 ? seq_list_bytes(n_seq) : P.tf_cache ? (((size_t)n_seq + 1) * 4 + 15) / 16 * 16 : 0)
                         : (size_t)kWaves * P.table_entries * sizeof(uint64_t);
  if (wg) {
    void (*kern)(PrefillArgs) = nullptr;
#define FS_WG(DT)                                  \
  (nw == 8 ? prefill_wg_kernel<DT, 8, 2, 4, 1> \
           : (p->opt.prefill_pipe ? prefill_wg_kernel<DT, 4, 4, 4, 1, true> : prefill_wg_kernel<DT, 4, 4, 4, 1>))
    // (that kernel at head_dim 128 only)
    const bool deq = p->opt.prefill_deq && nw == 8 && ncb == 16 && !d64 && large;
    if (d256) {
      // Four waves of one block each (a wave's share of a sub-tile's K or V, 64 registers in FP16, and its accumulators
      // leave room for no second one), one wave per SIMD, 64 tokens per step
      switch (g.kv_dtype) {
        case FS_KV_FP16: kern = prefill_wg_kernel<FS_KV_FP16, 4, 1, 2, 1, false, false, 256, true>; break;
        case FS_KV_FP8_E4M3: kern = prefill_wg_kernel<FS_KV_FP8_E4M3, 4, 1, 2, 1, false, false, 256, true>; break;
        case FS_KV_INT8: kern = prefill_wg_kernel<FS_KV_INT8, 4, 1, 2, 1, false, false, 256, true>; break;
        default: kern = prefill_wg_kernel<FS_KV_INT4, 4, 1, 2, 1, false, false, 256, true>; break;
      }
    } else if (kv_shift) {
#define FS_WGKV(DT) \
  (d64 ? prefill_wg_kernel<DT, 8, 2, 4, 1, false, false, 64, true, true> : prefill_wg_kernel<DT, 8, 2, 4, 1, false, false, kD, true, true>)
      switch (g.kv_dtype) {
        case FS_KV_FP16: kern = FS_WGKV(FS_KV_FP16); break;
        case FS_KV_FP8_E4M3: kern = FS_WGKV(FS_KV_FP8_E4M3); break;
        case FS_KV_INT8: kern = FS_WGKV(FS_KV_INT8); break;
        default: kern = FS_WGKV(FS_KV_INT4); break;
      }
#undef FS_WGKV
    } else if (ncb == kSmallBlocks) {
      // (integer codes exact, as in the 16-column kernel that served these launches before)
#define FS_WG1(DT) \
  (d64 ? prefill_wg_kernel<DT, 8, 1, 4, 1, false, false, 64, true> : prefill_wg_kernel<DT, 8, 1, 4, 1, false, false, kD, true>)
      switch (g.kv_dtype) {
        case FS_KV_FP16: kern = FS_WG1(FS_KV_FP16); break;
        case FS_KV_FP8_E4M3: kern = FS_WG1(FS_KV_FP8_E4M3); break;
        case FS_KV_INT8: kern = FS_WG1(FS_KV_INT8); break;
        default: kern = FS_WG1(FS_KV_INT4); break;
      }
#undef FS_WG1
    } else if (d64) {
      // Integer codes enter the MFMAs exactly here, as in the 16-column kernel that served this head_dim before.
#define FS_WG64(DT, WIDE) \
  (ncb == 16 ? prefill_wg_kernel<DT, 8, 2, 4, 1, false, false, 64, true> : prefill_wg_kernel<DT, 8, WIDE, 4, 1, false, false, 64, true>)
      switch (g.kv_dtype) {
        case FS_KV_FP16: kern = FS_WG64(FS_KV_FP16, 4); break;
        case FS_KV_FP8_E4M3: kern = FS_WG64(FS_KV_FP8_E4M3, 3); break;
        case FS_KV_INT8: kern = FS_WG64(FS_KV_INT8, 3); break;
        default: kern = FS_WG64(FS_KV_INT4, 3); break;
      }
#undef FS_WG64
    } else if (split) {
#define FS_WGS(DT, DEQ) prefill_wg_kernel<DT, 8, 2, 4, 1, false, DEQ, kD, false, false, true>
      switch (g.kv_dtype) {
        case FS_KV_FP16: kern = FS_WGS(FS_KV_FP16, false); break;
        case FS_KV_FP8_E4M3: kern = FS_WGS(FS_KV_FP8_E4M3, false); break;
        case FS_KV_INT8: kern = FS_WGS(FS_KV_INT8, true); break;
        default: kern = FS_WGS(FS_KV_INT4, true); break;
      }
#undef FS_WGS
    } else switch (g.kv_dtype) {
      case FS_KV_FP16: kern = large ? FS_WG(FS_KV_FP16) : prefill_wg_kernel<FS_KV_FP16, 8, 2, 4, 1, false, false, kD, true>; break;
      case FS_KV_FP8_E4M3: kern = large ? FS_WG(FS_KV_FP8_E4M3) : prefill_wg_kernel<FS_KV_FP8_E4M3, 8, 2, 4, 1, false, false, kD, true>; break;
      case FS_KV_INT8: kern = deq ? prefill_wg_kernel<FS_KV_INT8, 8, 2, 4, 1, false, true> : FS_WG(FS_KV_INT8); break;
      default: kern = deq ? prefill_wg_kernel<FS_KV_INT4, 8, 2, 4, 1, false, true> : FS_WG(FS_KV_INT4); break;
    }
#undef FS_WG
    // more than 64 KiB of dynamic LDS has to be granted per kernel
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return device_error(e, "prefill LDS attribute");
    const bool deq_used = deq && (g.kv_dtype == FS_KV_INT8 || g.kv_dtype == FS_KV_INT4);
    p->opt.last_prefill = (kv_shift ? kSmallBlocks : std::min(ncb, 16)) | (nw << 8) | ((int64_t)deq_used << 16) | ((int64_t)(nw == 4 && p->opt.prefill_pipe) << 17);
    hipLaunchKernelGGL(kern, dim3(n_wg), dim3(nw * 64), smem, s, P);
  } else if (ncb == 1) {
    p->opt.last_prefill = 1;
    if (g.head_dim == 64) hipLaunchKernelGGL(prefill_kernel<64>, dim3(n_wg), dim3(kThreads), smem, s, P);
    else if (g.head_dim == 256) hipLaunchKernelGGL(prefill_kernel<256>, dim3(n_wg), dim3(kThreads), smem, s, P);
    else hipLaunchKernelGGL(prefill_kernel<kD>, dim3(n_wg), dim3(kThreads), smem, s, P);
  } else {
    void (*kern)(PrefillArgs) = nullptr;
#define FS_WIDE(DT) (ncb == 4 ? prefill_wide_kernel<DT, 4, 1> : prefill_wide_kernel<DT, 2, 1>)
    switch (g.kv_dtype) {
      case FS_KV_FP16: kern = FS_WIDE(FS_KV_FP16); break;
      case FS_KV_FP8_E4M3: kern = FS_WIDE(FS_KV_FP8_E4M3); break;
      case FS_KV_INT8: kern = FS_WIDE(FS_KV_INT8); break;
      default: kern = FS_WIDE(FS_KV_INT4); break;
    }
#undef FS_WIDE
    p->opt.last_prefill = ncb;
    hipLaunchKernelGGL(kern, dim3(n_wg), dim3(kThreads), smem, s, P);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return device_error(e, "prefill launch");
  return FS_OK;
}
