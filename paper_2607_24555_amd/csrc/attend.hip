// Paged decode attention over a page list (Sec. 2 "Decode-time attention";
// App. E "sparse decode over k pages"):
//   o_g = sum_{i in S} softmax_S(q_g^T k_i / sqrt d) v_i,
// renormalised over the tokens of the listed pages.  With page_ids == nullptr the
// list is every page of the sequence (the dense baseline).
//
// Split-K: block (split, KV head, seq) walks its slice of the page list with an
// online softmax for all G query heads of the KV head (the G heads share every K/V
// page load), then writes an unnormalised partial (o, max, sum).  merge_kernel
// combines the splits exactly: m = max m_s, l = sum l_s e^{m_s - m},
// o = sum o_s e^{m_s - m} / l, lse = m + log l.
//
// bf16 Q and KV take attend_mfma_kernel: each wave owns pages_per_split / 4
// consecutive list entries and handles one page (16 tokens) per step on the
// matrix cores; the block's four waves combine in LDS before the partial is
// written.  Other dtypes take the VALU kernel attend_kernel.  In the fused
// decode step (kSelect) every block first derives its (sequence, KV head)'s
// page table from the selection chunks' survivors -- all blocks of the unit
// compute the same table -- and writes the table entries it attends together
// with their estimated page LSEs.
#include "locks_internal.h"
#include "topk.h"

namespace locks {
namespace {

constexpr int kAttnBlock = 256;

// Eight consecutive elements as floats (16-byte loads where the tensor is so aligned).
__device__ __forceinline__ void load8(const uint16_t* p, bool aligned, float (&x)[8]) {
  if (aligned) {
    const uint4 w = *reinterpret_cast<const uint4*>(p);
    const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[2 * e] = __uint_as_float(u[e] << 16);
      x[2 * e + 1] = __uint_as_float(u[e] & 0xffff0000u);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = load_elem(p, e);
  }
}
__device__ __forceinline__ void load8(const float* p, bool aligned, float (&x)[8]) {
  if (aligned) {
    const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = p[e];
  }
}
// sum over a 16-lane row
__device__ __forceinline__ float row16_sum(float v) {
  v += __int_as_float(dpp<0xB1>(__float_as_int(v)));
  v += __int_as_float(dpp<0x4E>(__float_as_int(v)));
  v += __int_as_float(dpp<0x141>(__float_as_int(v)));
  v += __int_as_float(dpp<0x140>(__float_as_int(v)));
  return v;
}

// Work is counted in 16-token sub-pages: unit t of the list is sub-page t % nsub
// of list entry t / nsub (nsub = B / 16 for pages of B tokens).
//
// Vector-ALU attention (fp32 queries or caches).  The block's 16 sixteen-lane rows take
// one token of a unit each, lane seg of a row dims 8 seg .. + 7; every row runs its own
// online softmax for the group's heads over its token slots, so the loop has no barrier
// and no LDS, and the 16 rows are combined per head at the end.
// A block holds kHeads heads (1 or 4); the further heads of a larger group are other
// blocks, n_splits apart in the grid, which read the same pages from the cache.
// Against four barriers and serial 128-term dot products per unit (sparse call and dense
// call, us): one head, 16 pages of 256: 13.9 -> 6.3 and 16.0 -> 9.8; 8 sequences x 8 KV
// heads x 4 heads, 128 pages of 1,024: 58.3 -> 30.5 and 293 -> 192 (5.6 TB/s); 16 heads
// on 2 KV heads: 29.8 -> 29.9 and 162 -> 109.
template <typename QT, typename KT, int kHeads>
__global__ __launch_bounds__(kAttnBlock) void attend_kernel(
    int H_q, int H_kv, int max_pages, int k_list, int pgsz, int lg_sub,
    const QT* __restrict__ q, const KT* __restrict__ k_cache, const KT* __restrict__ v_cache,
    const int32_t* __restrict__ page_table, const int32_t* __restrict__ seq_lens,
    const int32_t* __restrict__ page_ids, int pages_per_split, int n_splits,
    float* __restrict__ partial, float* __restrict__ out, float* __restrict__ out_lse) {
  __shared__ float sO[16][kDim + 4];
  __shared__ float sM[16], sL[16];

  const int split = blockIdx.x % n_splits, g0 = blockIdx.x / n_splits * kHeads;
  const int h = blockIdx.y, s = blockIdx.z;
  const int tid = threadIdx.x, i = tid >> 4, seg = tid & 15;
  const int G = H_q / H_kv;
  const int L = seq_lens[s];
  const int n = (L + pgsz - 1) / pgsz;
  const float zscale = 1.0f / sqrtf((float)kDim);
  const bool q_al = !(reinterpret_cast<uintptr_t>(q) & 15);
  const bool kv_al = !((reinterpret_cast<uintptr_t>(k_cache) | reinterpret_cast<uintptr_t>(v_cache)) & 15);

  const int t0 = split * pages_per_split;
  float qr[kHeads][8], o[kHeads][8], m[kHeads], l[kHeads];
#pragma unroll
  for (int g = 0; g < kHeads; ++g) {
    load8(q + ((long)s * H_q + h * G + min(g0 + g, G - 1)) * kDim + 8 * seg, q_al, qr[g]);
    m[g] = -INFINITY;
    l[g] = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[g][e] = 0.0f;
  }
  for (int t = t0; t < t0 + pages_per_split; ++t) {
    const int entry = t >> lg_sub, sub = t & ((1 << lg_sub) - 1);
    int id;
    if (page_ids) {
      id = entry < k_list ? page_ids[((long)s * H_kv + h) * k_list + entry] : -1;
    } else {
      id = entry;
    }
    if (id < 0 || id >= n) continue;  // uniform across the block
    const int tok = id * pgsz + sub * kPage + i;
    if (tok - i >= L) continue;
    const long blk = page_table[(long)s * max_pages + id];
    const long base = (((blk * H_kv + h) * pgsz + sub * kPage) + i) * kDim + 8 * seg;
    float kr[8], vr[8];
    load8(k_cache + base, kv_al, kr);
    load8(v_cache + base, kv_al, vr);
#pragma unroll
    for (int g = 0; g < kHeads; ++g) {
      float acc = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = fmaf(qr[g][e], kr[e], acc);
      acc = row16_sum(acc);
      if (tok < L) {  // uniform across the row
        const float z = acc * zscale;
        const float mx = fmaxf(m[g], z);
        const float sc = (m[g] == -INFINITY) ? 0.0f : __expf(m[g] - mx);
        const float w = (z == -INFINITY) ? 0.0f : __expf(z - mx);
        l[g] = fmaf(l[g], sc, w);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[g][e] = fmaf(o[g][e], sc, w * vr[e]);
        m[g] = mx;
      }
    }
  }
  // ---- the 16 rows of each head combined
#pragma unroll
  for (int g = 0; g < kHeads; ++g) {
    if (g0 + g >= G) break;
    if (g) __syncthreads();
    *reinterpret_cast<float4*>(&sO[i][8 * seg]) = make_float4(o[g][0], o[g][1], o[g][2], o[g][3]);
    *reinterpret_cast<float4*>(&sO[i][8 * seg + 4]) = make_float4(o[g][4], o[g][5], o[g][6], o[g][7]);
    if (seg == 0) { sM[i] = m[g]; sL[i] = l[g]; }
    __syncthreads();
    if (tid < kDim) {
      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sM[r]);
      float acc = 0.0f, ls = 0.0f;
      if (mx > -INFINITY) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float wt = sM[r] == -INFINITY ? 0.0f : __expf(sM[r] - mx);
          ls = fmaf(sL[r], wt, ls);
          acc = fmaf(sO[r][tid], wt, acc);
        }
      }
      const long row = (long)s * H_q + h * G + g0 + g;
      if (n_splits == 1) {
        out[row * kDim + tid] = ls > 0.0f ? acc / ls : 0.0f;
        if (tid == 0 && out_lse) out_lse[row] = ls > 0.0f ? mx + logf(ls) : -INFINITY;
      } else {
        float* pr = partial + (row * n_splits + split) * (kDim + 2);
        pr[tid] = acc;
        if (tid < 2) pr[kDim + tid] = tid ? ls : mx;
      }
    }
  }
}

// ---------------------------------------------------------------- MFMA path
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef short s4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ bf8v as_bf8(uint4 v) { return __builtin_bit_cast(bf8v, v); }

// Round-to-nearest-even float -> bf16 bits (finite inputs).
__device__ __forceinline__ uint32_t bf16_rne(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// Sum / max over the lanes {l, l^16, l^32, l^48} (the four 16-lane rows).
__device__ __forceinline__ float rows_max(float v) {
  auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float rows_sum(float v) {
  auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// 16-bit element e (0..7) of a uint4.
__device__ __forceinline__ uint32_t half_of(const uint4& v, int e) {
  const uint32_t w = e < 2 ? v.x : (e < 4 ? v.y : (e < 6 ? v.z : v.w));
  return (e & 1) ? (w >> 16) : (w & 0xffffu);
}

// One page of K (16 tokens x 128) and V in the operand layouts below.
struct PageRegs {
  uint4 k[4];  // lane (t = l % 16, r = l / 16): K[t][32 r + 8 kb .. + 7], kb = 0..3
  uint4 v[4];  // lane (c = l % 16, r): V[4 r + j][8 c .. 8 c + 7], j = 0..3
};

__device__ __forceinline__ void load_page(PageRegs& P, const uint16_t* kp, const uint16_t* vp,
                                          int c16, int r4) {
  const uint4* k4 = reinterpret_cast<const uint4*>(kp + c16 * kDim + 32 * r4);
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) P.k[kb] = k4[kb];
#pragma unroll
  for (int j = 0; j < 4; ++j) P.v[j] = *reinterpret_cast<const uint4*>(vp + (4 * r4 + j) * kDim + 8 * c16);
}

// Lane layout (l = 16 r + c):
//   S^T = K Q^T  (mfma 16x16x32, M = token, N = head, K = dim with dim order
//                 32 r + 8 kb + e): lane holds S^T[4 r + j][c], j = 0..3, so head
//                 c's 16 logits are the j values of lanes c, c+16, c+32, c+48;
//   O^T += V^T P (mfma 16x16x16, M = dim, N = head, K = token; tile n covers
//                 dims 8 m + n, m = 0..15): P is the B operand exactly as S^T
//                 left it, and lane holds O^T for head c, dims 32 r + 8 j + n.
// P enters as bf16 hi + lo (two MFMAs) so the weights keep ~16 bits.
// Chunk survivors and outputs of the selection merged into the attention kernel.
struct SelTable {
  SelectBufs sb;
  int n_rows, width, chunk;
  const float* s_hat;
  SHatLayout lay;
  int32_t* out_ids;
  float* out_sel_lse;
};

// kPPW > 0: every wave owns exactly kPPW list entries and keeps up to four
// pages in flight (fully unrolled, so each wait covers one page); kPPW == 0: any
// count up to 64, two units in flight, their addresses from one table read per wave
// (dense attention of 8 ragged sequences, 1.1 GB of K and V: 272 us with a lookup per
// unit and 64 stand-in loads in every block past its sequence's end, 214 us now: 5.2
// TB/s, where a plain copy runs at 5.07).
// kNK: survivors per lane of the selection merge (64 kNK per wave).
// kOne: the list is one block's, which writes the output itself (the step of 64 sequences
// x 8 KV heads, 16 entries each: 167.5 -> 161.5 us without the merge launch).  An instance
// of its own: the same branch taken at run time cost 0.8 us of 130.6 where the list is split.
template <bool kSelect, int kPPW, int kNK, bool kOne>
__global__ __launch_bounds__(256) void attend_mfma_kernel(
    int H_q, int H_kv, int max_pages, int k_list, int pgsz, int lg_sub,
    const uint16_t* __restrict__ q,
    const uint16_t* __restrict__ k_cache, const uint16_t* __restrict__ v_cache,
    const int32_t* __restrict__ page_table, const int32_t* __restrict__ seq_lens,
    const int32_t* __restrict__ page_ids, int pages_per_split, int n_splits,
    float* __restrict__ partial, float* __restrict__ out, float* __restrict__ out_lse, SelTable tb) {
  __shared__ float sO[4][kDim][kMaxGroup + 1];
  __shared__ float sM[4][kMaxGroup], sL[4][kMaxGroup];
  __shared__ int32_t s_tab[kSelect ? kFastK + 2 : 1], s_blk[kSelect ? kFastK + 2 : 1];
  __shared__ UnionLds<4> unionL;
  const int split = blockIdx.x, h = blockIdx.y, s = blockIdx.z;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int c16 = lane & 15, r4 = lane >> 4;
  const int G = H_q / H_kv;
  // the selection survivors are requested before the sequence length is known
  UnionRegs<kNK> UR;
  if constexpr (kSelect) {
    const long unit = (long)s * H_kv + h;
    const long rb = unit * tb.n_rows * tb.width;
    union_load<kNK, 4>(UR, tb.n_rows, tb.width, tb.sb.cand_key + rb, tb.sb.cand_idx + rb,
                            tb.sb.cand_blk + rb, tb.sb.sat + unit * tb.n_rows);
  }
  const int L = seq_lens[s];
  const int n = (L + pgsz - 1) / pgsz;
  const float zs = kLog2e / sqrtf((float)kDim);
  const int sub_mask = (1 << lg_sub) - 1;
  if (!kSelect && kPPW == 0 && !page_ids && split * pages_per_split * kPage >= L) {
    // no list and past the sequence's end: an empty partial
    // (not with a fixed count, whose loads the length would then hold up: four ragged
    // sequences of 2K to 16K tokens 12.36 us without, 12.56 with)
    for (int e = tid; e < G * (kDim + 2); e += 256) {
      const int g = e / (kDim + 2), c = e % (kDim + 2);
      const long row = (long)s * H_q + h * G + g;
      const float v = c == kDim ? -INFINITY : 0.0f;
      if constexpr (!kOne) partial[(row * n_splits + split) * (kDim + 2) + c] = v;
      else if (c < kDim) out[row * kDim + c] = v;
      else if (c == kDim && out_lse) out_lse[row] = v;
    }
    return;
  }

  uint4 qb[4];
  {
    const int g = c16 < G ? c16 : 0;
    const uint4* q4 = reinterpret_cast<const uint4*>(q + ((long)s * H_q + h * G + g) * kDim + 32 * r4);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) qb[kb] = c16 < G ? q4[kb] : make_uint4(0, 0, 0, 0);
  }
  const int ppw = pages_per_split / 4;
  const int t_begin = split * pages_per_split + wave * ppw, t_end = t_begin + ppw;
  const int32_t* ids = page_ids ? page_ids + ((long)s * H_kv + h) * k_list : nullptr;
  if constexpr (kSelect) {
    const long unit = (long)s * H_kv + h;
    const int used = n > k_list ? (n - 2) / tb.chunk + 1 : 0;
    union_table_from<kNK, 4>(UR, k_list, n, used, tb.width, tb.sb.keys + unit * max_pages,
                                  page_table + (long)s * max_pages, s_tab, s_blk, unionL);
    ids = s_tab;
  }
  // this block's table entries and their estimated page LSEs (NaN without a
  // summary): loaded now, written after the pages (at most 32 entries per block,
  // so at most 32 x 17 values over the 256 threads)
  constexpr int kSelPer = 3;
  const int epb = pages_per_split >> lg_sub;  // table entries per block
  float sel_v[kSelPer];
  int sel_e[kSelPer];
  if constexpr (kSelect) {
    const int t0 = split * epb, n_c = L / pgsz;
    const float* sb = tb.s_hat + tb.lay.base(s, h);
#pragma unroll
    for (int u = 0; u < kSelPer; ++u) {
      const int e = tid + 256 * u;
      const int t = t0 + e % epb, g = e / epb;
      sel_e[u] = (e < epb * (G + 1) && t < k_list) ? e : -1;
      sel_v[u] = 0.0f;
      if (sel_e[u] >= 0 && g < G) {
        const int id = s_tab[t];
        const bool ok = id >= 0 && id < n_c;
        const float v = sb[(long)(ok ? id : 0) * tb.lay.page + (long)(ok ? g : 0) * tb.lay.head];
        sel_v[u] = ok ? v : __int_as_float(0x7fc00000);
      }
    }
  }
  // unit t: sub-page t & sub_mask of list entry t >> lg_sub; returns the unit's
  // first token (-1: nothing to attend)
  auto page_at = [&](int t) -> int {
    int id = -1;
    const int entry = t >> lg_sub;
    if (t < t_end) id = ids ? (entry < k_list ? ids[entry] : -1) : entry;
    const int tok0 = (id >= 0 && id < n) ? id * pgsz + (t & sub_mask) * kPage : -1;
    return tok0 < L ? tok0 : -1;
  };
  const long kv_head = (long)h * pgsz * kDim;
  const long kv_blk = (long)H_kv * pgsz * kDim;
  // physical block of unit t starting at token tok0 (a valid block stands in for an
  // empty unit); the fused step knows the blocks from the selection
  auto blk_at = [&](int t, int tok0) -> long {
    if constexpr (kSelect) {
      const int entry = t >> lg_sub;
      const int b = entry < k_list ? s_blk[entry] : -1;
      return b >= 0 ? b : s_blk[0];
    } else {
      return page_table[(long)s * max_pages + (tok0 >= 0 ? tok0 / pgsz : 0)];
    }
  };
  auto page_ptr = [&](long blk, int t, const uint16_t* base) {
    return base + blk * kv_blk + kv_head + (long)(t & sub_mask) * kPage * kDim;
  };

  float m = -INFINITY, l = 0.0f;
  f4v o[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) o[t] = f4v{0.0f, 0.0f, 0.0f, 0.0f};

  // one 16-token unit of the list (tok0 < 0: an empty unit, nothing to add)
  auto use_page = [&](const PageRegs& cur, int tok0) {
    if (tok0 >= 0) {
      const int valid = min(kPage, L - tok0);
      f4v st = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
        st = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf8(cur.k[kb]), as_bf8(qb[kb]), st, 0, 0, 0);
      float z[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) z[j] = (4 * r4 + j < valid) ? st[j] * zs : -INFINITY;
      const float pm = rows_max(fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])));
      const float mn = fmaxf(m, pm);
      const float sc = (m == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(m - mn);
      float p[4], ps = 0.0f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        p[j] = (z[j] == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(z[j] - mn);
        ps += p[j];
      }
      l = l * sc + rows_sum(ps);
      m = mn;
      uint32_t hi[4], lo[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        hi[j] = bf16_rne(p[j]);
        lo[j] = bf16_rne(p[j] - __uint_as_float(hi[j] << 16));
      }
      const s4v bh = __builtin_bit_cast(s4v, make_uint2(hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16)));
      const s4v bl = __builtin_bit_cast(s4v, make_uint2(lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16)));
#pragma unroll
      for (int t8 = 0; t8 < 8; ++t8) {
        o[t8] *= sc;
        const uint32_t a01 = half_of(cur.v[0], t8) | (half_of(cur.v[1], t8) << 16);
        const uint32_t a23 = half_of(cur.v[2], t8) | (half_of(cur.v[3], t8) << 16);
        const s4v a = __builtin_bit_cast(s4v, make_uint2(a01, a23));
        o[t8] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, bh, o[t8], 0, 0, 0);
        o[t8] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, bl, o[t8], 0, 0, 0);
      }
    }
  };
  // loads unit t into P (a valid page stands in for an empty unit)
  auto load_entry = [&](PageRegs& P, int t) {
    const int tok0 = page_at(t);
    const long b = blk_at(t, tok0);
    load_page(P, page_ptr(b, t, k_cache), page_ptr(b, t, v_cache), c16, r4);
    return tok0;
  };

  if (n > 0) {
    if constexpr (kPPW > 0) {
      constexpr int D = kPPW < 4 ? kPPW : 4;
      PageRegs buf[D];
      int ids[D];
#pragma unroll
      for (int j = 0; j < D; ++j) ids[j] = load_entry(buf[j], t_begin + j);
#pragma unroll
      for (int i = 0; i < kPPW; ++i) {
        use_page(buf[i % D], ids[i % D]);
        if (i + D < kPPW) ids[i % D] = load_entry(buf[i % D], t_begin + i + D);
      }
    } else {
      // lane j holds the first token and the block of the wave's unit j (ppw <= 64), so
      // the loop's addresses are wave-uniform and wait for no table lookup; two units in
      // flight, loaded without a condition (past the wave's end the last unit again).
      // Without a list the wave stops at the sequence's last unit.
      const int cnt = ids ? ppw : min(ppw, (L + kPage - 1) / kPage - t_begin);
      const int mine = t_begin + min(lane, max(cnt, 1) - 1);
      const int my_tok = page_at(mine);
      const int my_blk = (int)blk_at(mine, my_tok);
      auto load_unit = [&](PageRegs& P, int j) {
        j = min(j, cnt - 1);
        const long b = __builtin_amdgcn_readlane(my_blk, j);
        const int t = t_begin + j;
        load_page(P, page_ptr(b, t, k_cache), page_ptr(b, t, v_cache), c16, r4);
      };
      if (cnt > 0) {
        PageRegs A, B;
        load_unit(A, 0);
        load_unit(B, 1);
        for (int j = 0; j < cnt; j += 2) {
          use_page(A, __builtin_amdgcn_readlane(my_tok, j));
          load_unit(A, j + 2);
          if (j + 1 < cnt) use_page(B, __builtin_amdgcn_readlane(my_tok, j + 1));
          load_unit(B, j + 3);
        }
      }
    }
  }
  if constexpr (kSelect) {
    const long unit = (long)s * H_kv + h;
    const int t0 = split * epb;
#pragma unroll
    for (int u = 0; u < kSelPer; ++u) {
      const int e = sel_e[u];
      if (e < 0) continue;
      const int t = t0 + e % epb, g = e / epb;
      if (g == G) tb.out_ids[unit * k_list + t] = s_tab[t];
      else tb.out_sel_lse[((long)s * H_q + h * G + g) * k_list + t] = sel_v[u];
    }
  }
  // combine the block's four waves; m is kept in log2 units until here.  sO is
  // [wave][d][17]: the odd row pitch keeps both the MFMA-layout writes and the
  // d-contiguous reads free of bank conflicts
  if (r4 == 0) { sM[wave][c16] = m; sL[wave][c16] = l; }
#pragma unroll
  for (int t8 = 0; t8 < 8; ++t8)
#pragma unroll
    for (int j = 0; j < 4; ++j) sO[wave][32 * r4 + 8 * j + t8][c16] = o[t8][j];
  __syncthreads();
  for (int e = tid; e < G * (kDim + 2); e += 256) {
    const int g = e / (kDim + 2), c = e % (kDim + 2);
    float mx = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) mx = fmaxf(mx, sM[w][g]);
    float acc = 0.0f, ls = 0.0f;
    if (mx > -INFINITY) {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float wt = sM[w][g] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(sM[w][g] - mx);
        ls += sL[w][g] * wt;
        if (c < kDim) acc += sO[w][c][g] * wt;
      }
    }
    const float mn = mx == -INFINITY ? mx : mx * kLn2;
    const long row = (long)s * H_q + h * G + g;
    if constexpr (kOne) {  // as merge_kernel forms it
      if (c < kDim) out[row * kDim + c] = ls > 0.0f ? acc / ls : 0.0f;
      else if (c == kDim && out_lse) out_lse[row] = ls > 0.0f ? mn + logf(ls) : -INFINITY;
    } else {
      partial[(row * n_splits + split) * (kDim + 2) + c] = c < kDim ? acc : (c == kDim ? mn : ls);
    }
  }
}

__global__ __launch_bounds__(kDim) void merge_kernel(int H_q, int n_splits,
                                                     const float* __restrict__ partial,
                                                     float* __restrict__ out,
                                                     float* __restrict__ out_lse) {
  const int hq = blockIdx.x, s = blockIdx.y, c = threadIdx.x;
  const long row = (long)s * H_q + hq;
  const float* p = partial + row * n_splits * (kDim + 2);
  constexpr int kB = 32;  // splits per round trip (every split of a sparse step)
  float m = -INFINITY, l = 0.0f, o = 0.0f;
  for (int t0 = 0; t0 < n_splits; t0 += kB) {
    float mt[kB], lt[kB], ot[kB];
#pragma unroll
    for (int u = 0; u < kB; ++u) {
      const float* pt = p + (long)min(t0 + u, n_splits - 1) * (kDim + 2);
      mt[u] = pt[kDim];
      lt[u] = pt[kDim + 1];
      ot[u] = pt[c];
    }
#pragma unroll
    for (int u = 0; u < kB; ++u) asm volatile("" : "+v"(mt[u]), "+v"(lt[u]), "+v"(ot[u]));
#pragma unroll
    for (int u = 0; u < kB; ++u) mt[u] = t0 + u < n_splits ? mt[u] : -INFINITY;
    float mm = m;
#pragma unroll
    for (int u = 0; u < kB; ++u) mm = fmaxf(mm, mt[u]);
    if (mm == -INFINITY) continue;
    const float sc = (m == -INFINITY) ? 0.0f : __expf(m - mm);
    l *= sc;
    o *= sc;
#pragma unroll
    for (int u = 0; u < kB; ++u) {
      const float w = (mt[u] == -INFINITY) ? 0.0f : __expf(mt[u] - mm);
      l += lt[u] * w;
      o += ot[u] * w;
    }
    m = mm;
  }
  out[row * kDim + c] = (l > 0.0f) ? o / l : 0.0f;
  if (out_lse && c == 0) out_lse[row] = (l > 0.0f) ? m + logf(l) : -INFINITY;
}

template <typename QT, typename KT>
void launch_typed(const locks_cfg_t& c, const void* q, const void* k_cache, const void* v_cache,
                  const int32_t* page_table, const int32_t* seq_lens, const int32_t* page_ids,
                  int pages_per_split, int n_splits, float* partial, float* out, float* out_lse,
                  hipStream_t st) {
  const int G = c.num_q_heads / c.num_kv_heads;
#define LOCKS_ATTEND(HH)                                                                       \
  hipLaunchKernelGGL((attend_kernel<QT, KT, HH>),                                              \
                     dim3(n_splits * ((G + HH - 1) / HH), c.num_kv_heads, c.num_seqs),         \
                     dim3(kAttnBlock), 0, st, c.num_q_heads, c.num_kv_heads,                   \
                     c.max_pages_per_seq, page_budget(c), c.page_size, sub_page_log2(c),       \
                     static_cast<const QT*>(q), static_cast<const KT*>(k_cache),               \
                     static_cast<const KT*>(v_cache), page_table, seq_lens, page_ids,          \
                     pages_per_split, n_splits, partial, out, out_lse)
  if (G == 1) LOCKS_ATTEND(1);
  else LOCKS_ATTEND(4);
#undef LOCKS_ATTEND
}

// bf16 MFMA kernel with the page count per wave fixed at compile time where the
// list is split into 1, 2, 4 or 8 entries per wave (a selected table always is).
template <bool kSelect>
hipError_t launch_mfma(const locks_cfg_t& c, dim3 grid, hipStream_t st, const uint16_t* q,
                 const uint16_t* k_cache, const uint16_t* v_cache, const int32_t* page_table,
                 const int32_t* seq_lens, const int32_t* page_ids, int pages_per_split,
                 int n_splits, float* partial, float* out, float* out_lse, SelTable tb) {
  const int ppw = pages_per_split % 4 == 0 ? pages_per_split / 4 : 0;
  // survivors held per lane: 2, 4 or the cap's 8 (without a selection none)
  const int held = kSelect ? tb.n_rows * tb.width : 0;
#define LOCKS_ATTEND_MFMA(P)                                               \
  if (held <= 2 * 256) LOCKS_ATTEND_MFMA_N(P, 2);                          \
  else if (held <= 4 * 256) LOCKS_ATTEND_MFMA_N(P, (kSelect ? 4 : 2));     \
  else LOCKS_ATTEND_MFMA_N(P, (kSelect ? kUnionNK : 2))
#define LOCKS_ATTEND_MFMA_N(P, NK)                                                             \
  hipLaunchKernelGGL((n_splits == 1 ? attend_mfma_kernel<kSelect, P, NK, true>                  \
                                    : attend_mfma_kernel<kSelect, P, NK, false>),               \
                     grid, dim3(256), 0, st, c.num_q_heads,                                     \
                     c.num_kv_heads, c.max_pages_per_seq, page_budget(c), c.page_size,          \
                     sub_page_log2(c), q, k_cache, v_cache, page_table, seq_lens, page_ids,     \
                     pages_per_split, n_splits, partial, out, out_lse, tb)
  switch (ppw) {
    case 1: LOCKS_ATTEND_MFMA(1); break;
    case 2: LOCKS_ATTEND_MFMA(2); break;
    case 4: LOCKS_ATTEND_MFMA(4); break;
    case 8: LOCKS_ATTEND_MFMA(8); break;
    default:
      if constexpr (kSelect) return hipErrorInvalidValue;
      else { LOCKS_ATTEND_MFMA(0); }
  }
  return hipGetLastError();
#undef LOCKS_ATTEND_MFMA_N
#undef LOCKS_ATTEND_MFMA
}

}  // namespace

hipError_t launch_attend(const locks_cfg_t& c, const void* q, const void* k_cache,
                         const void* v_cache, const int32_t* page_table, const int32_t* seq_lens,
                         const int32_t* page_ids, int pages_per_split, int n_splits,
                         float* partial, float* out, float* out_lse, hipStream_t st) {
  const bool qb = c.q_dtype == LOCKS_BF16, kb = c.kv_dtype == LOCKS_BF16;
  hipError_t e = hipSuccess;
  if (qb && kb)
    e = launch_mfma<false>(c, dim3(n_splits, c.num_kv_heads, c.num_seqs), st,
                           static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k_cache),
                           static_cast<const uint16_t*>(v_cache), page_table, seq_lens, page_ids,
                           pages_per_split, n_splits, partial, out, out_lse, SelTable{});
  else if (qb)
    launch_typed<uint16_t, float>(c, q, k_cache, v_cache, page_table, seq_lens, page_ids,
                                  pages_per_split, n_splits, partial, out, out_lse, st);
  else if (kb)
    launch_typed<float, uint16_t>(c, q, k_cache, v_cache, page_table, seq_lens, page_ids,
                                  pages_per_split, n_splits, partial, out, out_lse, st);
  else
    launch_typed<float, float>(c, q, k_cache, v_cache, page_table, seq_lens, page_ids,
                               pages_per_split, n_splits, partial, out, out_lse, st);
  if (e != hipSuccess) return e;
  if (n_splits > 1)
    hipLaunchKernelGGL(merge_kernel, dim3(c.num_q_heads, c.num_seqs), dim3(kDim), 0, st,
                       c.num_q_heads, n_splits, partial, out, out_lse);
  return hipGetLastError();
}

bool attend_select_fused(const locks_cfg_t& c) {
  return c.q_dtype == LOCKS_BF16 && c.kv_dtype == LOCKS_BF16 && select_fast_path(c);
}

hipError_t launch_attend_select(const locks_cfg_t& c, const void* q, const void* k_cache,
                                const void* v_cache, const int32_t* page_table,
                                const int32_t* seq_lens, const SelectBufs& sb, const float* s_hat,
                                SHatLayout lay, int32_t* out_ids, float* out_sel_lse,
                                int pages_per_split, int n_splits, float* partial, float* out,
                                float* out_lse, hipStream_t st) {
  const SelTable tb{sb, select_rows(c), select_width(c), select_chunk_pages(c), s_hat, lay, out_ids,
                    out_sel_lse};
  const hipError_t e = launch_mfma<true>(
      c, dim3(n_splits, c.num_kv_heads, c.num_seqs), st, static_cast<const uint16_t*>(q),
      static_cast<const uint16_t*>(k_cache), static_cast<const uint16_t*>(v_cache), page_table,
      seq_lens, nullptr, pages_per_split, n_splits, partial, out, out_lse, tb);
  if (e != hipSuccess) return e;
  if (n_splits > 1)
    hipLaunchKernelGGL(merge_kernel, dim3(c.num_q_heads, c.num_seqs), dim3(kDim), 0, st,
                       c.num_q_heads, n_splits, partial, out, out_lse);
  return hipGetLastError();
}

}  // namespace locks
