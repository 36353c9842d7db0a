// Pieces shared by the summary-scan kernels: query loads and digits, record loads
// through a buffer resource, operand decoders, lane reductions.
#pragma once

#include "locks_internal.h"

namespace locks {
namespace {

template <typename QT>
__device__ __forceinline__ float load_q(const QT* q, size_t i);
template <>
__device__ __forceinline__ float load_q<float>(const float* q, size_t i) { return q[i]; }
template <>
__device__ __forceinline__ float load_q<uint16_t>(const uint16_t* q, size_t i) {
  return bf16_bits_to_f32(q[i]);
}

// Chunk of pages a scan block covers (blockIdx.x keeps naming its partials slot).
// Blocks go to the XCDs round-robin by linear block id, x fastest, so chunk c of
// every (sequence, KV head) would sit on XCD c mod 8: the leading chunks, which
// every sequence has, would pile onto the first XCDs when lengths vary (a batch
// with lengths uniform in [8K, 64K] scanned ~1.25x slower than the same pages in
// equal lengths).  Rotating the chunk order by the sequence index spreads them
// out, while the KV heads of one sequence keep one chunk-to-XCD map: their
// records of a page are adjacent, so the cache lines they share stay in one L2
// (rotating by head as well raised the counted fetch bytes by up to a third).
__device__ __forceinline__ int scan_chunk() {
  return (int)((blockIdx.x + blockIdx.z) % gridDim.x);
}

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ h2 as_h2(uint32_t u) { return __builtin_bit_cast(h2, u); }

// 8 excess-8 nibbles (element t in bits 4t..4t+3) -> 8 exact f16 codes in the
// order t = 0,4,1,5,2,6,3,7.
__device__ __forceinline__ h8 nib8_to_h8(uint32_t w) {
  const uint32_t M = 0x64006400u;  // f16 1024.0 in both halves
  const uint32_t w8 = w >> 8;
  const h2 y0 = as_h2((w & 0x000F000Fu) | M) - h2{(_Float16)1032.0f, (_Float16)1032.0f};
  const h2 y1 = as_h2((w & 0x00F000F0u) | M) * h2{(_Float16)0.0625f, (_Float16)0.0625f} -
                h2{(_Float16)72.0f, (_Float16)72.0f};
  const h2 y2 = as_h2((w8 & 0x000F000Fu) | M) - h2{(_Float16)1032.0f, (_Float16)1032.0f};
  const h2 y3 = as_h2((w8 & 0x00F000F0u) | M) * h2{(_Float16)0.0625f, (_Float16)0.0625f} -
                h2{(_Float16)72.0f, (_Float16)72.0f};
  return h8{y0.x, y0.y, y1.x, y1.y, y2.x, y2.y, y3.x, y3.y};
}

// 8 excess-128 bytes -> 8 exact f16 codes in natural order.
__device__ __forceinline__ h8 byte8_to_h8(uint32_t w0, uint32_t w1) {
  const uint32_t M = 0x64646464u;
  const h2 k{(_Float16)1152.0f, (_Float16)1152.0f};
  const h2 a = as_h2(__builtin_amdgcn_perm(M, w0, 0x04010400u)) - k;
  const h2 b = as_h2(__builtin_amdgcn_perm(M, w0, 0x04030402u)) - k;
  const h2 c = as_h2(__builtin_amdgcn_perm(M, w1, 0x04010400u)) - k;
  const h2 d = as_h2(__builtin_amdgcn_perm(M, w1, 0x04030402u)) - k;
  return h8{a.x, a.y, b.x, b.y, c.x, c.y, d.x, d.y};
}

__device__ __forceinline__ float lds_f16(const uint8_t* p) {
  return (float)*reinterpret_cast<const _Float16*>(p);
}

// log2(2^a + 2^b)
__device__ __forceinline__ float lse2_log2(float a, float b) {
  const float mx = fmaxf(a, b);
  return mx + __builtin_amdgcn_logf(__builtin_amdgcn_exp2f(a - mx) + __builtin_amdgcn_exp2f(b - mx));
}

// Sum over lanes l, l ^ 32 and over lanes l, l ^ 16.
__device__ __forceinline__ float swap32_sum(float v) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ float swap16_sum(float v) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// Log-sum-exp, log2 domain, over lanes {l, l ^ 16} (V = 2) or {l, l ^ 16, l ^ 32,
// l ^ 48} (V = 4); each of those lanes gets the same bits.
template <int V>
__device__ __forceinline__ float merge_sub_lse(float v) {
  if (V == 4) {
    auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = lse2_log2(__uint_as_float(p[0]), __uint_as_float(p[1]));
  }
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return lse2_log2(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Reduction over the four lanes {l, l^16, l^32, l^48} with two VALU lane swaps.
__device__ __forceinline__ float red4_max(float v) {
  auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float red4_sum(float v) {
  auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// the value of lane K of this lane's 16-lane row
template <int K>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + K, 0xF, 0xF, false));
}

// a, b, c, d hold per-lane partial sums of four columns sets; returns in row grp the
// total over the four rows of the grp-th of them: stage 1 adds rows r and r ^ 2, stage
// 2 rows r and r ^ 1 (the order of red4_sum).
__device__ __forceinline__ float reduce4(float a, float b, float c, float d) {
  const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(c), false, false);
  const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(b), __float_as_uint(d), false, false);
  const float t0 = __uint_as_float(x[0]) + __uint_as_float(x[1]);
  const float t1 = __uint_as_float(y[0]) + __uint_as_float(y[1]);
  const auto z = __builtin_amdgcn_permlane16_swap(__float_as_uint(t0), __float_as_uint(t1), false, false);
  return __uint_as_float(z[0]) + __uint_as_float(z[1]);
}

// Combines running (max, sum 2^(x - max)) pairs, log2 domain, over the lanes that
// share lane % M; every lane ends with its class's total.
template <int M>
__device__ __forceinline__ void merge_lanes_mod(float& m, float& l) {
#pragma unroll
  for (int o = M; o < 64; o <<= 1) {
    const float om = __shfl_xor(m, o, 64), ol = __shfl_xor(l, o, 64);
    const float mm = fmaxf(m, om);
    l = (mm > -INFINITY)
            ? l * __builtin_amdgcn_exp2f(m - mm) + ol * __builtin_amdgcn_exp2f(om - mm)
            : 0.0f;
    m = mm;
  }
}

// Sums of 2^z over a page's tokens are taken without their max: z are the logits minus the
// centroid logit, which sum to about 0 over the page.  Outside this range (a token 83 nats
// above that mean; every token 70 below it, where a record's coefficients are not centred)
// a sum loses bits to the ends of float32 and is taken again with a shift: the fixed
// kHighShift, for which sums of 2^116 to 2^336 are in the range, or the max.
constexpr float kSumMin = 0x1p-100f, kSumMax = 0x1p120f, kLog2SumMin = -100.0f, kHighShift = 216.0f;

// Log-sum-exp, log2 domain, of the 4 x 4 values that lanes l, l ^ 16, l ^ 32, l ^ 48 hold;
// each of those lanes gets it.
__device__ __forceinline__ float max_shifted_lse(const float (&z)[4]) {
  const float shift = red4_max(fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])));
  const float sm = (__builtin_amdgcn_exp2f(z[0] - shift) + __builtin_amdgcn_exp2f(z[1] - shift)) +
                   (__builtin_amdgcn_exp2f(z[2] - shift) + __builtin_amdgcn_exp2f(z[3] - shift));
  return shift + __builtin_amdgcn_logf(red4_sum(sm));
}

typedef int i4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// The summary store as a raw buffer resource: 32-bit byte offsets, no 64-bit
// address arithmetic per load, and loads past the store's end return zeros.
constexpr int kBufWord3 = 0x00020000;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t summ_rsrc(const uint8_t* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p), (short)0, (int)bytes, kBufWord3);
}
__device__ __forceinline__ uint4 bld16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 bld8(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
  return make_uint2(v.x, v.y);
}
// (soff: a wave-uniform part of the offset)
__device__ __forceinline__ uint32_t bld4(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff = 0) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0);
}
// Byte offset of the record of (physical block b, KV head h): b * (H_kv * stride)
// + h * stride.  32 bits hold it, as the store is below 4 GiB; a 24-bit multiply would not
// do, as a block's records pass 2^24 bytes from 20,165 KV heads on (832-byte records).  The
// full multiply runs once per lane and 16-page step.
__device__ __forceinline__ uint32_t rec_off(int b, uint32_t blk_bytes, uint32_t head_off) {
  return (uint32_t)b * blk_bytes + head_off;
}

// Query digits of a head for the int8 projection: q is scaled by a power of two to a
// fixed-point integer Q and split into ND signed 8-bit digits (most significant first):
// ND = 3, |Q| < 2^20, or ND = 4, |Q| < 2^30.  Element e of MFMA half hh <-> d =
// 32 grp + 16 hh + perm16[e], the order in which the decoders expand the packed
// codes.  bias[t] = -8 * sum(digit t) removes the excess-8 offset of the int4
// codes.
//
// The digits are the bytes of U = Q + 0x80808080 (three digits: its lower three) minus
// 128: the lower digits land in [-128, 127] (the balanced base-256 digits of Q).  Four
// elements' bytes are gathered into one digit word per digit by byte permutes, the +128
// offsets flipped back by one XOR, and each word's digit sum taken by one signed 4-way dot
// product.
template <int ND>
struct QDigits {
  i4v bd[ND][2];
  i4v bias;         // (a vector: as an array of four it was kept in LDS, 15 us a scan)
  float inv_scale;  // fixed-point unit * log2(e) / sqrt(d)
};

template <typename QT>
__device__ __forceinline__ QDigits<3> q_digits(const QT* __restrict__ qrow, int grp) {
  constexpr int kPerm16[16] = {0, 2, 4, 6, 1, 3, 5, 7, 8, 10, 12, 14, 9, 11, 13, 15};
  constexpr float c0 = 1.4426950408889634f * 0.08838834764831845f;  // log2(e) / sqrt(128)
  QDigits<3> D;
  float qf[32];
  float qmax = 0.0f;
#pragma unroll
  for (int c = 0; c < 32; ++c) {
    qf[c] = load_q(qrow + 32 * grp, c);
    qmax = fmaxf(qmax, fabsf(qf[c]));
  }
  qmax = red4_max(qmax);
  int ex = 0;
  (void)frexpf(qmax, &ex);  // qmax < 2^ex
  const float qscale = ldexpf(1.0f, 20 - ex);
  D.inv_scale = ldexpf(1.0f, ex - 20) * c0;
  int bsum[3] = {0, 0, 0};
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int dw = 0; dw < 4; ++dw) {
      uint32_t U[4];
#pragma unroll
      for (int bb = 0; bb < 4; ++bb) {
        const int e = 4 * dw + bb;
        const int Q = (qmax > 0.0f)
                          ? min(max((int)rintf(qf[16 * hh + kPerm16[e]] * qscale), -0xFFFFF), 0xFFFFF)
                          : 0;
        U[bb] = (uint32_t)(Q + 0x808080);
      }
      // bytes (U0.b0, U1.b0, U0.b1, U1.b1), (U0.b2, U1.b2, ..) and the same for U2, U3
      const uint32_t lo01 = __builtin_amdgcn_perm(U[1], U[0], 0x05010400u);
      const uint32_t lo23 = __builtin_amdgcn_perm(U[3], U[2], 0x05010400u);
      const uint32_t hi01 = __builtin_amdgcn_perm(U[1], U[0], 0x07030602u);
      const uint32_t hi23 = __builtin_amdgcn_perm(U[3], U[2], 0x07030602u);
      const uint32_t w2 = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u) ^ 0x80808080u;
      const uint32_t w1 = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u) ^ 0x80808080u;
      const uint32_t w0 = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u) ^ 0x80808080u;
      bsum[0] = __builtin_amdgcn_sdot4((int)w0, 0x01010101, bsum[0], false);
      bsum[1] = __builtin_amdgcn_sdot4((int)w1, 0x01010101, bsum[1], false);
      bsum[2] = __builtin_amdgcn_sdot4((int)w2, 0x01010101, bsum[2], false);
      D.bd[0][hh][dw] = (int)w0;
      D.bd[1][hh][dw] = (int)w1;
      D.bd[2][hh][dw] = (int)w2;
    }
#pragma unroll
  for (int t = 0; t < 3; ++t) D.bias[t] = -8 * (int)red4_sum((float)bsum[t]);
  return D;
}

// The digits of the block's HG head columns (heads past G repeat head 0), formed once per
// block of 256 threads and read back by every wave: 16 threads per head, 8 elements each
// (each wave forming all of its lanes' digits itself took about 300 VALU instructions, a
// tenth to a sixth of the wave's work).  Thread seg of a head holds elements 8 seg .. + 7:
// half of the 16 bytes that lane group seg / 4 uses in MFMA half (seg / 2) % 2.
template <int HG, int ND>
struct DigitLds {
  i4v bd[ND][2][4][HG];  // [digit][half][lane group][head]
  int bias[ND][HG];
  float inv_scale[HG];
};

// (rows of a query tensor that starts off a 16-byte boundary are read element by element)
template <typename QT>
__device__ __forceinline__ bool load8_unaligned(const QT* p, float (&x)[8]) {
  if (!(reinterpret_cast<uintptr_t>(p) & 15)) return false;
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = load_q(p, e);
  return true;
}
__device__ __forceinline__ void load8_q(const uint16_t* p, float (&x)[8]) {
  if (load8_unaligned(p, x)) return;
  const uint4 w = *reinterpret_cast<const uint4*>(p);
  const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    x[2 * e] = __uint_as_float(u[e] << 16);
    x[2 * e + 1] = __uint_as_float(u[e] & 0xffff0000u);
  }
}
__device__ __forceinline__ void load8_q(const float* p, float (&x)[8]) {
  if (load8_unaligned(p, x)) return;
  const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
  x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
  x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}
template <int C>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_mov_dpp(v, C, 0xF, 0xF, true);
}

// Called by all 256 threads (q: the group's first row); a barrier must follow before the
// digits are read.  With four digits a head whose query holds a NaN or an infinity gets a
// NaN unit, so that all its scores are NaN.
template <typename QT, int HG, int ND>
__device__ __forceinline__ void block_digits(const QT* __restrict__ q, int G, DigitLds<HG, ND>& S) {
  constexpr float c0 = 1.4426950408889634f * 0.08838834764831845f;  // log2(e) / sqrt(128)
  constexpr int kBits = ND == 4 ? 30 : 20;
  const int hd = threadIdx.x >> 4, seg = threadIdx.x & 15;
  if (hd >= HG) return;
  float x[8];
  load8_q(q + (hd < G ? hd : 0) * kDim + 8 * seg, x);
  float m = 0.0f;
  bool finite = true;
  if constexpr (ND == 4) {  // magnitudes compared as integers: infinities and NaN on top
    uint32_t u = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) u = max(u, __float_as_uint(x[e]) & 0x7fffffffu);
    u = max(u, (uint32_t)dpp_i<0xB1>((int)u));
    u = max(u, (uint32_t)dpp_i<0x4E>((int)u));
    u = max(u, (uint32_t)dpp_i<0x141>((int)u));
    u = max(u, (uint32_t)dpp_i<0x140>((int)u));
    finite = u < 0x7f800000u;
    m = finite ? __uint_as_float(u) : 1.0f;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(x[e]));
    m = fmaxf(m, __int_as_float(dpp_i<0xB1>(__float_as_int(m))));
    m = fmaxf(m, __int_as_float(dpp_i<0x4E>(__float_as_int(m))));
    m = fmaxf(m, __int_as_float(dpp_i<0x141>(__float_as_int(m))));
    m = fmaxf(m, __int_as_float(dpp_i<0x140>(__float_as_int(m))));
  }
  int ex = 0;
  (void)frexpf(m, &ex);  // m < 2^ex
  const float qscale = ldexpf(1.0f, kBits - ex);
  constexpr int kMaxQ = (1 << kBits) - 1;
  uint32_t U[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int Q = m > 0.0f ? min(max((int)rintf(x[e] * qscale), -kMaxQ), kMaxQ) : 0;
    U[e] = (uint32_t)Q + (ND == 4 ? 0x80808080u : 0x808080u);
  }
  uint32_t w[ND][2];  // [digit][even, odd elements]
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    const uint32_t lo01 = __builtin_amdgcn_perm(U[o + 2], U[o], 0x05010400u);
    const uint32_t lo23 = __builtin_amdgcn_perm(U[o + 6], U[o + 4], 0x05010400u);
    const uint32_t hi01 = __builtin_amdgcn_perm(U[o + 2], U[o], 0x07030602u);
    const uint32_t hi23 = __builtin_amdgcn_perm(U[o + 6], U[o + 4], 0x07030602u);
    w[ND - 1][o] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u) ^ 0x80808080u;
    w[ND - 2][o] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u) ^ 0x80808080u;
    w[ND - 3][o] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u) ^ 0x80808080u;
    if (ND == 4) w[0][o] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u) ^ 0x80808080u;
  }
#pragma unroll
  for (int d = 0; d < ND; ++d) {
    *reinterpret_cast<uint2*>(reinterpret_cast<uint32_t*>(&S.bd[d][(seg >> 1) & 1][seg >> 2][hd]) +
                              2 * (seg & 1)) = make_uint2(w[d][0], w[d][1]);
    int b = __builtin_amdgcn_sdot4((int)w[d][0], 0x01010101, 0, false);
    b = __builtin_amdgcn_sdot4((int)w[d][1], 0x01010101, b, false);
    b += dpp_i<0xB1>(b);
    b += dpp_i<0x4E>(b);
    b += dpp_i<0x141>(b);
    b += dpp_i<0x140>(b);
    if (seg == 0) S.bias[d][hd] = -8 * b;
  }
  if (seg == 0) S.inv_scale[hd] = finite ? ldexpf(1.0f, ex - kBits) * c0 : __int_as_float(0x7fc00000);
}

// Lane (grp, head)'s digits.
template <int HG, int ND>
__device__ __forceinline__ void lane_digits(const DigitLds<HG, ND>& S, int grp, int head, QDigits<ND>& D) {
#pragma unroll
  for (int d = 0; d < ND; ++d) {
    D.bd[d][0] = S.bd[d][0][grp][head];
    D.bd[d][1] = S.bd[d][1][grp][head];
    D.bias[d] = S.bias[d][head];
  }
  D.inv_scale = S.inv_scale[head];
}

// A 16-byte basis slice (32 excess-8 nibbles) as the int8 A operands of the two
// K halves.
__device__ __forceinline__ void nib_operands(const uint4& v, i4v (&a)[2]) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const uint32_t x0 = w[2 * hh], x1 = w[2 * hh + 1];
    a[hh] = i4v{(int)(x0 & 0x0F0F0F0Fu), (int)((x0 >> 4) & 0x0F0F0F0Fu), (int)(x1 & 0x0F0F0F0Fu),
                (int)((x1 >> 4) & 0x0F0F0F0Fu)};
  }
}

// Exact integer projection sum_d (n_d - 8) Q_d of excess-8 nibble codes n_d onto
// a 20-bit query Q = 2^16 D0 + 2^8 D1 + D2, by Horner's rule over the digits in
// one int32 accumulator: acc = 256 (256 (D0 . n') + D1 . n') + D2 . n'.  Every
// partial value is bounded by |acc| <= 128 * 8 * 2^20 = 2^30, so nothing wraps.
__device__ __forceinline__ i4v proj_horner(const i4v (&a)[2], const QDigits<3>& QD) {
  i4v acc = i4v{QD.bias[0], QD.bias[0], QD.bias[0], QD.bias[0]};
  acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[0], QD.bd[0][0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[1], QD.bd[0][1], acc, 0, 0, 0);
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = (int)(((uint32_t)acc[j] << 8) + (uint32_t)QD.bias[1]);
  acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[0], QD.bd[1][0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[1], QD.bd[1][1], acc, 0, 0, 0);
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = (int)(((uint32_t)acc[j] << 8) + (uint32_t)QD.bias[2]);
  acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[0], QD.bd[2][0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[1], QD.bd[2][1], acc, 0, 0, 0);
  return acc;
}

// Two independent projections by the same Horner steps, interleaved so that the
// matrix-core work of one covers the shifts of the other, in units of the query's scale.
__device__ __forceinline__ void project2(const i4v (&a0)[2], const i4v (&a1)[2], const QDigits<3>& QD,
                                         float (&p)[2][4]) {
  i4v x = i4v{QD.bias[0], QD.bias[0], QD.bias[0], QD.bias[0]};
  i4v y = x;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    x = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0[0], QD.bd[t][0], x, 0, 0, 0);
    y = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1[0], QD.bd[t][0], y, 0, 0, 0);
    x = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0[1], QD.bd[t][1], x, 0, 0, 0);
    y = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1[1], QD.bd[t][1], y, 0, 0, 0);
    if (t < 2) {
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = (int)(((uint32_t)x[j] << 8) + (uint32_t)QD.bias[t + 1]);
#pragma unroll
      for (int j = 0; j < 4; ++j) y[j] = (int)(((uint32_t)y[j] << 8) + (uint32_t)QD.bias[t + 1]);
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) p[0][j] = (float)x[j];
#pragma unroll
  for (int j = 0; j < 4; ++j) p[1][j] = (float)y[j];
}
// Four digits would leave int32 in one chain: two chains of two, upper and lower, joined as
// floats.  The upper one, |x| <= 128 * 8 * 2^14, converts exactly, so p carries one float32
// rounding of the sum and 2^-30 of the query's largest element per term.
__device__ __forceinline__ void project2(const i4v (&a0)[2], const i4v (&a1)[2], const QDigits<4>& QD,
                                         float (&p)[2][4]) {
  const int b0 = QD.bias[0], b1 = QD.bias[1], b2 = QD.bias[2], b3 = QD.bias[3];
  i4v x0 = {b0, b0, b0, b0}, y0 = {b2, b2, b2, b2}, x1 = x0, y1 = y0;
  auto mac = [&](int hh, const i4v& dx, const i4v& dy) {
    x0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0[hh], dx, x0, 0, 0, 0);
    x1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1[hh], dx, x1, 0, 0, 0);
    y0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0[hh], dy, y0, 0, 0, 0);
    y1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1[hh], dy, y1, 0, 0, 0);
  };
  auto shift = [](i4v& v, int bias) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = (int)(((uint32_t)v[j] << 8) + (uint32_t)bias);
  };
  mac(0, QD.bd[0][0], QD.bd[2][0]);
  mac(1, QD.bd[0][1], QD.bd[2][1]);
  shift(x0, b1);
  shift(x1, b1);
  shift(y0, b3);
  shift(y1, b3);
  mac(0, QD.bd[1][0], QD.bd[3][0]);
  mac(1, QD.bd[1][1], QD.bd[3][1]);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    p[0][j] = fmaf((float)x0[j], 65536.0f, (float)y0[j]);
    p[1][j] = fmaf((float)x1[j], 65536.0f, (float)y1[j]);
  }
}

// Integer dot product of a code row with Q from its dot products with the digits.
__device__ __forceinline__ float join_digits(const int (&d)[3]) {
  return fmaf((float)d[0], 65536.0f, (float)(d[1] * 256 + d[2]));
}
__device__ __forceinline__ float join_digits(const int (&d)[4]) {
  return fmaf((float)(d[0] * 256 + d[1]), 65536.0f, (float)(d[2] * 256 + d[3]));
}

// The two upper halves of a pair of floats, as a pair of bfloat16 (truncation).
__device__ __forceinline__ uint32_t top16(float a, float b) {
  return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
}
// Four excess-128 bytes -> four exact bfloat16 codes.
__device__ __forceinline__ uint2 byte4_to_b4(uint32_t w) {
  const uint32_t x = w ^ 0x80808080u;
  float f[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) f[e] = (float)(int)(int8_t)(x >> (8 * e));
  return make_uint2(top16(f[0], f[1]), top16(f[2], f[3]));
}
// A pair of floats as the sum of three pairs of bfloat16, exactly (8 bits of the 24 each;
// no float is too large or too small, and NaN stays NaN).
__device__ __forceinline__ void split3_b2(float a, float b, uint32_t (&t)[3]) {
  auto cut = [](float v) { return __uint_as_float(__float_as_uint(v) & 0xffff0000u); };
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    t[i] = top16(a, b);
    if (i < 2) {
      a -= cut(a);
      b -= cut(b);
    }
  }
}

template <int N>
struct IntTag {
  static constexpr int value = N;
};
// f(IntTag<0>{}), .., f(IntTag<N - 1>{}), N <= 4
template <int N, typename F>
__device__ __forceinline__ void static_for_int(F&& f) {
  f(IntTag<0>{});
  if constexpr (N > 1) f(IntTag<1>{});
  if constexpr (N > 2) f(IntTag<2>{});
  if constexpr (N > 3) f(IntTag<3>{});
}

// Block of (sub-)page min(page0 + (lane & 15), n_c - 1): always a valid page of
// the sequence.
template <int V = 1>
__device__ __forceinline__ int lane_block_clamped(const int32_t* __restrict__ pt_row, int page0,
                                                  int n_c, int lane) {
  const int pl = page0 + (lane & 15);
  return pt_row[(pl < n_c ? pl : n_c - 1) / V];
}

}  // namespace
}  // namespace locks
