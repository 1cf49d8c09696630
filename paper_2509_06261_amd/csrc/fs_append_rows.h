// Device code of fs_kv_append: quantize new K/V rows and scatter them into slab blocks (shared by the append
// kernels and the decode step's front kernel, which appends and prepares the work list in one launch).
//
// FineServe Sec. 2.1: every new token appends its keys and values to the KV cache;
// Sec. 2.2 / 3.2: the cache may be FP16, FP8 or INT4 (here also INT8), with per-token
// quantization parameters stored inside the block.  The paper gives no quantizer
// arithmetic; the definitions implemented here are the ones stated in fineserve.h.
//
// A (token, KV head, K|V) row is handled by head_dim / 8 neighbouring lanes, eight elements each (a wave covers
// 4 tokens at head_dim 128): 16-byte source loads, 16 / 8 / 8 / 4-byte stores for FP16 / FP8 / INT8 / INT4.  The
// row's extrema are reduced over its lanes (max and min are exact in any order), and each lane
// stores its own bytes (INT4: a byte holds two codes of one lane, so no byte is shared between lanes or tokens).
// All arithmetic is IEEE fp32, round-to-nearest-even, correctly rounded division; every file that includes this
// header is compiled with floating-point contraction off so that the stored bytes are reproducible bit for bit.
#pragma once

#include "fs_internal.h"

namespace fs {
namespace append {


constexpr int kEpl = 8;    // elements per lane

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct AppendArgs {
  DevGeom g;
  uint8_t* pool;
  const void* k_new;
  const void* v_new;
  const int32_t* seq_idx;
  const int32_t* pos;
  const int32_t* tables;
  const float* k_scale;  // FP8: device [H] for this layer
  const float* v_scale;
  int64_t n_tokens;
  int32_t lpr_shift;     // log2 of the lanes per row (head_dim / 8)
  int64_t n_blocks;      // valid block ids are [0, n_blocks)
  int32_t layer, max_blocks;
  int32_t src_f32;       // source rows are fp32 (else fp16)
  int32_t pad;
};

// Several appends in one launch: append i is worked on by the workgroups first_block[i] .. first_block[i + 1] - 1.
constexpr int kMaxAppends = 8;
struct MultiAppendArgs {
  AppendArgs a[kMaxAppends];
  uint32_t first_block[kMaxAppends + 1];
  int32_t n;
};

// max / min over the lanes of a row (lpr neighbouring lanes, lpr a power of two, the same in every lane): DPP within
// 16 lanes -- swapped neighbours, swapped pairs, then mirrored halves, whose lanes already agree --, shuffles beyond.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), CTRL, 0xF, 0xF, true));
}
template <bool MAX>
__device__ __forceinline__ float pick(float a, float b) {
  if constexpr (MAX) return fmaxf(a, b);
  else return fminf(a, b);
}
template <bool MAX>
__device__ __forceinline__ float row_extremum(float v, int lpr) {
  if (lpr > 1) v = pick<MAX>(v, dpp<0xB1>(v));   // quad_perm 1 0 3 2
  if (lpr > 2) v = pick<MAX>(v, dpp<0x4E>(v));   // quad_perm 2 3 0 1
  if (lpr > 4) v = pick<MAX>(v, dpp<0x141>(v));  // row_half_mirror
  if (lpr > 8) v = pick<MAX>(v, dpp<0x140>(v));  // row_mirror
  if (lpr > 16) v = pick<MAX>(v, __shfl_xor(v, 16, 64));
  if (lpr > 32) v = pick<MAX>(v, __shfl_xor(v, 32, 64));
  return v;
}
__device__ __forceinline__ float row_max(float v, int lpr) { return row_extremum<true>(v, lpr); }
__device__ __forceinline__ float row_min(float v, int lpr) { return row_extremum<false>(v, lpr); }

__device__ __forceinline__ uint16_t f16_bits(float x) {
  _Float16 h = (_Float16)x;  // round-to-nearest-even
  return __builtin_bit_cast(uint16_t, h);
}
__device__ __forceinline__ float f16_value(uint16_t b) { return (float)__builtin_bit_cast(_Float16, b); }

// fp16 scale of the integer quantizers: nearest fp16, saturating, 1.0 when it rounds to zero.
__device__ __forceinline__ uint16_t scale_bits(float s32) {
  uint16_t b = f16_bits(s32);
  if ((b & 0x7FFF) >= 0x7C00) b = 0x7BFF;
  if ((b & 0x7FFF) == 0) b = 0x3C00;
  return b;
}

// Nearest OCP E4M3 code, ties to even, saturating at +-448, sign of the input kept.
__device__ __forceinline__ uint32_t e4m3_bits(float y) {
  const uint32_t fb = __float_as_uint(y);
  const uint32_t sign = (fb >> 24) & 0x80u;
  const float a = fabsf(y);
  uint32_t code;
  if (!(a < 448.0f)) {
    code = 0x7E;
  } else if (a < 0.015625f) {  // below 2^-6: subnormal codes, spacing 2^-9
    code = (uint32_t)rintf(a * 512.0f);
  } else {
    const uint32_t ab = fb & 0x7FFFFFFFu;
    const uint32_t e = ab >> 23;           // biased fp32 exponent, >= 121 here
    uint32_t m3 = (ab >> 20) & 7u;
    const uint32_t rest = ab & 0xFFFFFu;
    code = ((e - 120u) << 3) + m3;         // E4M3 bias 7: exponent field = e - 127 + 7
    if (rest > 0x80000u || (rest == 0x80000u && (code & 1u))) code += 1;  // carry runs into the exponent
  }
  return sign | code;
}

// n / d for many n and one d.  The correctly rounded fp32 division is a reciprocal estimate, one Newton step on
// it, and a quotient with two residual corrections, all in fused multiply-adds; the first half depends on d
// alone and is done once per row here.  What is left out is the operand scaling of the general sequence, which
// only matters near the ends of the exponent range: d must be a normal number of moderate size (the fp16-valued
// scales of the integer formats: 2^-24 .. 65504) and n / d must stay finite (|n| <= the row's extremum, so the
// quotient is bounded by the format's range unless the scale saturated, and then by 2^128 / 65504).  Within that
// domain the result is the division's, bit for bit; a quotient in the subnormal range may differ in its last bits,
// where every value rounds to the integer 0 anyway.
struct Divisor {
  float d, r;
  __device__ __forceinline__ explicit Divisor(float d_) : d(d_) {
    const float r0 = __builtin_amdgcn_rcpf(d);
    const float e = __builtin_fmaf(-d, r0, 1.0f);
    r = __builtin_fmaf(e, r0, r0);
  }
  __device__ __forceinline__ float operator()(float n) const {
    float q = n * r;
    const float e1 = __builtin_fmaf(-d, q, n);
    q = __builtin_fmaf(e1, r, q);
    const float e2 = __builtin_fmaf(-d, q, n);
    return __builtin_fmaf(e2, r, q);
  }
  // A quotient that rounds to the same integer (ties to even) as the correctly rounded one, for an fp16-valued d and
  // |n / d| < 2^20: one correction less.  1 / d is never within 2^-35 of a rounding midpoint for an 11-bit d, so r is
  // correctly rounded, and the quotient below is the rounding of a value within a factor 1 +- 2^-45 of n / d.  It could
  // land on the other side of a half-integer k + 1/2 than the correctly rounded quotient only if n / d were that close
  // to the midpoint between k + 1/2 and its neighbour; but n / d - (k + 1/2) is m ulp(n) / (2 d) with a small integer
  // m, which equals half an ulp exactly (impossible unless d is a power of two, and then n / d needs no rounding) or
  // differs from it by a factor of at least 1 +- 2^-11.
  __device__ __forceinline__ float near(float n) const {
    const float q = n * r;
    return __builtin_fmaf(__builtin_fmaf(-d, q, n), r, q);
  }
};

// 1.5 * 2^23: x + kRound holds the integer nearest to x (ties to even, |x| < 2^22) in its low bits, as an offset from
// the bit pattern of kRound itself.
constexpr float kRound = 12582912.0f;
constexpr uint32_t kRoundBits = 0x4B400000u;

// KV bytes are written with the non-temporal hint (FP16 -> FP16, 65 600 tokens x 8 heads of 128: 79 us with it, 107
// without); source rows are read without it: they were just produced, so part of them may still be in the memory-side
// cache (the same append: 97 us with the hint on both).
template <typename T>
__device__ __forceinline__ void kv_store(T* p, T v) {
  __builtin_nontemporal_store(v, p);
}

// the lane's eight source elements, widened exactly
template <bool kSrcF32>
__device__ __forceinline__ void load8(const void* src, int64_t idx, float (&x)[kEpl]) {
  if (kSrcF32) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const f32x4 a = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(src) + idx);
    const f32x4 b = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(src) + idx + 4);
    x[0] = a[0]; x[1] = a[1]; x[2] = a[2]; x[3] = a[3];
    x[4] = b[0]; x[5] = b[1]; x[6] = b[2]; x[7] = b[3];
  } else {
    const u32x4 v = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(src) + idx);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      x[2 * q] = f16_value((uint16_t)(v[q] & 0xFFFF));
      x[2 * q + 1] = f16_value((uint16_t)(v[q] >> 16));
    }
  }
}

// One lane's eight elements of a row, quantized and stored.  ok: the row exists and lies inside the pool (lanes of a
// row agree; a row that is skipped stores nothing, its lanes only take part in the row's extrema).
// The kernel that did the same with two residual corrections and a convert, shift and or per code, and with 64-bit
// divisions for a row's place, was bound by the vector ALU: 328 instructions per four rows, 65 600 fp32 tokens x 8
// heads -> INT4 in 157 us (3.9 TB/s).  Now about 100 instructions and 130 us (4.7 TB/s, a plain copy moves 4.3); FP16
// -> FP8 154 -> 69 us, FP16 -> FP16 117 -> 79 us.
template <int DT>
__device__ __forceinline__ void quantize_row(const float (&x)[kEpl], bool ok, uint8_t* row, uint8_t* par, float sc, int lir,
                                             int lpr) {
  const int d0 = lir * kEpl;  // this lane's first element (head_dim >= 8: always inside the row)
  if constexpr (DT == FS_KV_FP16) {
    u32x4 w;
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = (uint32_t)f16_bits(x[2 * q]) | ((uint32_t)f16_bits(x[2 * q + 1]) << 16);
    if (ok) kv_store(reinterpret_cast<u32x4*>(row + 2 * d0), w);
  } else if constexpr (DT == FS_KV_FP8_E4M3) {
    u32x2 w = {0u, 0u};
    if (sc >= 0x1p-40f && sc <= 0x1p40f) {
      // Divisor's domain; smaller quotients than it is exact for round to a zero code.  The sign is the source's own (the
      // corrections lose that of a zero), NaN and overflow become the largest magnitude, as in e4m3_bits.
      const Divisor by_scale(sc);
      float y[kEpl];
#pragma unroll
      for (int q = 0; q < kEpl; ++q) y[q] = __builtin_copysignf(fminf(fabsf(by_scale(x[q])), 448.0f), x[q]);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        int v = __builtin_amdgcn_cvt_pk_fp8_f32(y[4 * h], y[4 * h + 1], 0, false);
        w[h] = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(y[4 * h + 2], y[4 * h + 3], v, true);
      }
    } else {
#pragma unroll
      for (int q = 0; q < kEpl; ++q) w[q >> 2] |= e4m3_bits(__fdiv_rn(x[q], sc)) << (8 * (q & 3));
    }
    if (ok) kv_store(reinterpret_cast<u32x2*>(row + d0), w);
  } else if constexpr (DT == FS_KV_INT8) {
    float amax = 0.f;
#pragma unroll
    for (int q = 0; q < kEpl; ++q) amax = fmaxf(amax, fabsf(x[q]));
    amax = row_max(amax, lpr);
    const uint16_t sb = scale_bits(__fdiv_rn(amax, 127.0f));
    const Divisor by_scale(f16_value(sb));
    // codes + 128 are the digits 1 .. 255 of a base-256 number, summed with kRound's offset and taken out at once
    u32x2 w;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint32_t s = 0x80808080u - kRoundBits * 0x01010101u;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float c = __builtin_amdgcn_fmed3f(by_scale.near(x[4 * h + q]), -127.f, 127.f);  // (a NaN becomes -127)
        s += __float_as_uint(c + kRound) << (8 * q);
      }
      w[h] = s ^ 0x80808080u;
    }
    if (ok) {
      kv_store(reinterpret_cast<u32x2*>(row + d0), w);
      if (lir == 0) *reinterpret_cast<uint16_t*>(par) = sb;
    }
  } else {  // FS_KV_INT4
    float lo = 0.f, hi = 0.f;
#pragma unroll
    for (int q = 0; q < kEpl; ++q) {
      lo = fminf(lo, x[q]);
      hi = fmaxf(hi, x[q]);
    }
    lo = row_min(lo, lpr);
    hi = row_max(hi, lpr);
    const uint16_t sb = scale_bits(__fdiv_rn(hi - lo, 15.0f));
    const Divisor by_scale(f16_value(sb));
    const float z = fminf(fmaxf(rintf(by_scale(-lo)), 0.f), 15.f);
    const float top = 15.f - z;
    // rint(x / s) clamped to -z .. 15 - z, plus z: the digits 0 .. 15 of a base-16 number (element 2j in the low nibble
    // of byte j), summed with kRound's offset and taken out at once; a NaN becomes code 0
    uint32_t w = (uint32_t)z * 0x11111111u - kRoundBits * 0x11111111u;
#pragma unroll
    for (int q = 0; q < kEpl; ++q) {
      const float c = __builtin_amdgcn_fmed3f(by_scale.near(x[q]), -z, top);
      w += __float_as_uint(c + kRound) << (4 * q);
    }
    if (ok) {
      kv_store(reinterpret_cast<uint32_t*>(row + (d0 >> 1)), w);
      if (lir == 0) *reinterpret_cast<uint32_t*>(par) = (uint32_t)sb | ((uint32_t)f16_bits(z) << 16);
    }
  }
}

// The rows of one append, dealt to n_workers waves; this wave is number `worker`.  A wave's unit of work is `HP`
// neighbouring (KV head, K|V) rows of 64 / lpr consecutive tokens, a token's row per lpr lanes: the tokens' places (a
// division, a block-table entry) are looked up once per unit, the source rows of a unit are requested together and
// before that chain of look-ups, and consecutive positions of a sequence are written side by side.
template <bool kSrcF32, int DT, int HP>
__device__ __forceinline__ void append_rows(const AppendArgs& A, int64_t worker, int64_t n_workers) {
  const int lane = threadIdx.x & 63;
  const DevGeom& g = A.g;
  const int lpr = 1 << A.lpr_shift;           // lanes per row
  const int tpw = 64 >> A.lpr_shift;          // tokens per wave
  const int lir = lane & (lpr - 1);           // lane within its row
  const int kinds = 2 * g.H;                  // rows per token
  const uint32_t parts = (uint32_t)(kinds + HP - 1) / HP;  // units per group of tokens
  const int64_t n_units = (A.n_tokens + tpw - 1) / tpw * parts;
  for (int64_t unit = worker; unit < n_units; unit += n_workers) {
    int64_t grp;  // (wave-uniform: scalar arithmetic)
    uint32_t part;
    if (unit <= 0xffffffffll) {
      grp = (uint32_t)unit / parts;
      part = (uint32_t)unit % parts;
    } else {
      grp = unit / parts;
      part = (uint32_t)(unit % parts);
    }
    const int64_t tok = grp * tpw + (lane >> A.lpr_shift);
    bool ok = tok < A.n_tokens;
    const int kind0 = (int)part * HP;
    float x[HP][kEpl];
#pragma unroll
    for (int k = 0; k < HP; ++k) {
#pragma unroll
      for (int q = 0; q < kEpl; ++q) x[k][q] = 0.f;
      const int kind = kind0 + k;
      if (ok && kind < kinds) load8<kSrcF32>((kind & 1) ? A.v_new : A.k_new, (tok * g.H + (kind >> 1)) * (int64_t)g.D + lir * kEpl, x[k]);
    }
    const int p = ok ? A.pos[tok] : -1;
    const int s = ok ? A.seq_idx[tok] : -1;
    ok = ok && p >= 0 && s >= 0;
    const int bi = ok ? (int)((uint32_t)p / (uint32_t)g.T) : 0;
    ok = ok && bi < A.max_blocks;
    const int tib = ok ? p - bi * g.T : 0;
    const int32_t blk = ok ? A.tables[(int64_t)s * A.max_blocks + bi] : -1;
    ok = ok && blk >= 0 && blk < A.n_blocks;  // never write outside the pool
    uint8_t* const layer = A.pool + (uint64_t)(ok ? blk : 0) * g.block_budget + (uint64_t)A.layer * g.layer_bytes;
#pragma unroll
    for (int k = 0; k < HP; ++k) {
      const int kind = kind0 + k, head = kind >> 1, which = kind & 1;  // (wave-uniform)
      if (kind >= kinds) break;
      uint8_t* const chunk = layer + (uint64_t)head * g.head_chunk;
      uint8_t* const row = chunk + (which ? g.kv_tile : 0u) + (uint64_t)tib * g.row_bytes;
      uint8_t* const par = chunk + 2u * g.kv_tile + (which ? g.par_tile : 0u) + (uint64_t)tib * (uint32_t)g.param_bytes;
      const float sc = DT == FS_KV_FP8_E4M3 ? (which ? A.v_scale : A.k_scale)[head] : 1.0f;
      quantize_row<DT>(x[k], ok, row, par, sc, lir, lpr);
    }
  }
}

// Rows of a unit: four while that leaves every wave slot of the chip work (the look-ups are shared and four source rows
// are in flight per wave), one otherwise: a decode step's few tokens spread over as many waves as there are rows.
// Measured, 65 600 tokens x 8 heads of 128, units of 1 / 2 / 4 / 8 rows: FP16 -> FP16 89 / 80 / 79 / 82 us, FP16 -> FP8
// 84 / 79 / 73 / 82 us, FP16 -> INT8 103 / 87 / 82 / 89 us, fp32 -> INT4 124 / 120 / 122 / 123 us.
constexpr int kWideUnit = 4;

template <bool kSrcF32, int HP>
__device__ __forceinline__ void append_any(const AppendArgs& A, int64_t worker, int64_t n_workers) {
  switch (A.g.dtype) {
    case FS_KV_FP16: append_rows<kSrcF32, FS_KV_FP16, HP>(A, worker, n_workers); break;
    case FS_KV_FP8_E4M3: append_rows<kSrcF32, FS_KV_FP8_E4M3, HP>(A, worker, n_workers); break;
    case FS_KV_INT8: append_rows<kSrcF32, FS_KV_INT8, HP>(A, worker, n_workers); break;
    default: append_rows<kSrcF32, FS_KV_INT4, HP>(A, worker, n_workers); break;
  }
}

// The workgroup's share of a multi-append launch: `block` = its index among the launch's append workgroups,
// `waves` = waves per workgroup.
__device__ __forceinline__ void append_block(const MultiAppendArgs& P, uint32_t block, int waves) {
  int i = 0;
  while (i + 1 < P.n && block >= P.first_block[i + 1]) ++i;
  const AppendArgs& A = P.a[i];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t worker = (int64_t)(block - P.first_block[i]) * waves + wave;
  const int64_t n_workers = (int64_t)(P.first_block[i + 1] - P.first_block[i]) * waves;
  if (A.src_f32) append_any<true, 1>(A, worker, n_workers);
  else append_any<false, 1>(A, worker, n_workers);
}

}  // namespace append

// Host side (fs_append.hip): validates one append and fills its kernel arguments; sizes a multi-append launch for
// workgroups of `waves` waves (first_block, n; returns the number of workgroups).
int make_append_args(fs_pool* p, const fs_append_t& a, append::AppendArgs& out);
uint32_t plan_append_blocks(const fs_pool* p, append::MultiAppendArgs& P, int waves);
hipError_t launch_append_multi(const fs_pool* p, append::MultiAppendArgs& P, hipStream_t s);

}  // namespace fs
