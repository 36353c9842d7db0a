// Per-page summary construction for pages of B = 32 or 64 tokens (Sec. 4
// "Build"; App. D.3 "Page size"): centre the page's B keys, form the B x B Gram of
// the deviations, find its eigenpairs, keep the r leading nonzero modes, form
// V = D^T U_r S_r^{-1} and C = U_r S_r, quantise and pack.  Everything is fp32.
//
// Mapping: one wave per block holding kI = 64 / B items (page, KV head).
//  * Centroid, Gram (upper 16 x 16 tiles) and V take their key operands straight from
//    memory in the layout their lanes need and run on all 64 lanes, item by item; the
//    Gram and V are fp32 MFMAs 16x16x4.
//  * Eigenproblem: lane (it, i) holds row i of item it's Gram in registers.  Householder
//    reduction from the last column down (step k annihilates column k above row k - 1):
//    the reflector and its update vector reach every lane as 16-lane segments copied to
//    all rows by lane swaps, whose elements are row broadcasts folded into the FMAs, so
//    a step costs three FMAs per 16-column group and lane and no LDS in its loops (with
//    the rows in LDS the loops were bound by LDS bandwidth, six 16-byte accesses per
//    four columns).  The steps are unrolled by 16 inside a loop over the groups: every
//    register index is static and the code stays well inside the instruction cache.
//  * The wanted eigenvalues of T by multisection on Sturm counts (B / n lanes per
//    eigenvalue), the r leading eigenvectors of T by inverse iteration on its LDL^T
//    factorisation (lane l solves for vector l in registers; two rounds, each followed
//    by modified Gram-Schmidt over the r vectors, so a near-degenerate pair still
//    yields an orthonormal basis of its eigenspace).
//  * Back-transformation with kCPL components of one vector per lane: a reflector is one
//    short dot product, a few lane exchanges and one update.
// Bound: VALU issue (the Householder steps are about half of it) at four waves per SIMD
// for 32 tokens and three for 64 (ranks up to 8), which the packed reflectors in LDS and the
// registers are held to: at 64 tokens by spilling 18 of them (fp32 keys 26; 76 and 108
// bytes a lane), still faster than two waves without (1,526 us against 1,604).  2 x 128K
// tokens x 8 heads at r = 8: 756 us at 32 tokens and 1,548 at 64, where Gram rows in LDS, eigenvectors solved through LDS by r
// lanes and one reduction at a time took 1,470 and 3,900.
#include "build_common.h"
#include "locks_internal.h"

namespace locks {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kInvRounds = 2;     // inverse-iteration rounds (solve + orthogonalise)

template <int C>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), C, 0xF, 0xF, true));
}
__device__ __forceinline__ float swap16_add(float v) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ float swap32_add(float v) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
// Sums over the B lanes of an item (lane groups of B consecutive lanes) of N values,
// stage by stage so that the N chains overlap: within a 16-lane row by DPP (quad xor 1,
// quad xor 2, half-row mirror, row mirror), across rows by lane swaps.
template <int B, int N>
__device__ __forceinline__ void group_sums(float (&v)[N]) {
#pragma unroll
  for (int n = 0; n < N; ++n) v[n] += dpp_f<0xB1>(v[n]);
#pragma unroll
  for (int n = 0; n < N; ++n) v[n] += dpp_f<0x4E>(v[n]);
#pragma unroll
  for (int n = 0; n < N; ++n) v[n] += dpp_f<0x141>(v[n]);
#pragma unroll
  for (int n = 0; n < N; ++n) v[n] += dpp_f<0x140>(v[n]);
  if (B >= 32)
#pragma unroll
    for (int n = 0; n < N; ++n) v[n] = swap16_add(v[n]);
  if (B >= 64)
#pragma unroll
    for (int n = 0; n < N; ++n) v[n] = swap32_add(v[n]);
}
template <int B>
__device__ __forceinline__ float group_sum(float v) {
  float a[1] = {v};
  group_sums<B, 1>(a);
  return a[0];
}
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, dpp_f<0xB1>(v));
  v = fmaxf(v, dpp_f<0x4E>(v));
  v = fmaxf(v, dpp_f<0x141>(v));
  return fmaxf(v, dpp_f<0x140>(v));
}
template <int B>
__device__ __forceinline__ float group_max(float v) {
  v = row_max(v);
  if (B >= 32) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
  }
  if (B >= 64) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
  }
  return v;
}
__device__ __forceinline__ int row_min_int(int v) {
  v = min(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false));
  return min(v, __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false));
}

// a / b and sqrt(x) of normal values, within a rounding: the hardware's value corrected by
// its residual.  (Householder steps from the hardware's own reciprocals, whose error all
// entries of a reflector share, left the eigenvalues off by 1.24e-7 in the mean at 32
// tokens and 1.22e-7 at 64, against 1.12e-7 and 1.09e-7; time of 2 x 128K builds within
// 1.5%, where IEEE divisions take 3 to 8% more for the same bits.)
__device__ __forceinline__ float quot(float a, float b) {
  const float y = __builtin_amdgcn_rcpf(b), q = a * y;
  return fmaf(fmaf(-q, b, a), y, q);
}
__device__ __forceinline__ float root(float x) {
  const float y = __builtin_amdgcn_rsqf(x), s = x * y;
  return fmaf(fmaf(-s, s, x), 0.5f * y, s);
}

// Item vector x (lane (it, i) holds x_i) as B / 16 segments: lane l of seg[g] holds
// x_{16 g + l % 16} of its item.
template <int B>
__device__ __forceinline__ void segments(float x, float (&seg)[B / 16]) {
  const uint32_t u = __float_as_uint(x);
  const auto xy = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  if constexpr (B == 32) {
    seg[0] = __uint_as_float(xy[0]);
    seg[1] = __uint_as_float(xy[1]);
  } else {
    const auto xx = __builtin_amdgcn_permlane32_swap(xy[0], xy[0], false, false);
    const auto yy = __builtin_amdgcn_permlane32_swap(xy[1], xy[1], false, false);
    seg[0] = __uint_as_float(xx[0]);
    seg[1] = __uint_as_float(yy[0]);
    seg[2] = __uint_as_float(xx[1]);
    seg[3] = __uint_as_float(yy[1]);
  }
}

// The FMAs of a Householder step whose first factor is one element of a segment, read by
// a row broadcast in the FMA itself (the compiler keeps the broadcast as a move of its own,
// twice the instructions).  Each block opens with the two wait states that a DPP read
// needs after the write of its source, whatever the compiler placed before it.
#define LOCKS_BC(J) " row_newbcast:" #J " row_mask:0xf bank_mask:0xf\n"
// p += sum_j seg_j a_j over eight columns from J0 = 0 or 8 of the segment
template <int J0>
__device__ __forceinline__ void dot8(float& p, float seg, const float (&a)[8]) {
  static_assert(J0 == 0 || J0 == 8, "half of a segment");
#define LOCKS_D(O, J) "v_fmac_f32_dpp %0, %1, %" #O LOCKS_BC(J)
  if constexpr (J0 == 0)
    asm("s_nop 1\n" LOCKS_D(2, 0) LOCKS_D(3, 1) LOCKS_D(4, 2) LOCKS_D(5, 3) LOCKS_D(6, 4)
            LOCKS_D(7, 5) LOCKS_D(8, 6) LOCKS_D(9, 7)
        : "+v"(p)
        : "v"(seg), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]),
          "v"(a[7]));
  else
    asm("s_nop 1\n" LOCKS_D(2, 8) LOCKS_D(3, 9) LOCKS_D(4, 10) LOCKS_D(5, 11) LOCKS_D(6, 12)
            LOCKS_D(7, 13) LOCKS_D(8, 14) LOCKS_D(9, 15)
        : "+v"(p)
        : "v"(seg), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]),
          "v"(a[7]));
#undef LOCKS_D
}
// a_j += vseg_j nw + wseg_j nv over eight columns from J0 of the segments
template <int J0>
__device__ __forceinline__ void rank2_8(float* a, float vseg, float wseg, float nv, float nw) {
  static_assert(J0 == 0 || J0 == 8, "half of a segment");
#define LOCKS_U(O, J) "v_fmac_f32_dpp %" #O ", %8, %11" LOCKS_BC(J) "v_fmac_f32_dpp %" #O ", %9, %10" LOCKS_BC(J)
  if constexpr (J0 == 0)
    asm("s_nop 1\n" LOCKS_U(0, 0) LOCKS_U(1, 1) LOCKS_U(2, 2) LOCKS_U(3, 3) LOCKS_U(4, 4)
            LOCKS_U(5, 5) LOCKS_U(6, 6) LOCKS_U(7, 7) "s_nop 1\n"
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]),
          "+v"(a[7])
        : "v"(vseg), "v"(wseg), "v"(nv), "v"(nw));
  else
    asm("s_nop 1\n" LOCKS_U(0, 8) LOCKS_U(1, 9) LOCKS_U(2, 10) LOCKS_U(3, 11) LOCKS_U(4, 12)
            LOCKS_U(5, 13) LOCKS_U(6, 14) LOCKS_U(7, 15) "s_nop 1\n"
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]),
          "+v"(a[7])
        : "v"(vseg), "v"(wseg), "v"(nv), "v"(nw));
#undef LOCKS_U
}
#undef LOCKS_BC

template <int N>
struct Int {
  static constexpr int value = N;
};
template <int I, int N, typename F>
__device__ __forceinline__ void static_range(F&& f) {
  if constexpr (I < N) {
    f(Int<I>{});
    static_range<I + 1, N>(f);
  }
}

// Reflector of column k >= 2 (rows 0 .. k - 1): 16 (seg + 1) floats, seg = (k - 1) / 16.
__device__ __forceinline__ int refl_off(int k) {
  const int seg = (k - 1) >> 4;
  return 128 * seg * (seg + 1) + 16 * (seg + 1) * ((k - 1) & 15) - 16;
}

// One (page, KV head) of the block; uniform over the wave.
struct PageItem {
  bool active;
  int h, e;
  long row;  // blk * H_kv + h
};

template <typename KT, int B, bool kFactors, int kMaxR>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(B == 32 && kMaxR <= 8 ? 4 : (kMaxR <= 8 ? 3 : 2)))) void build_page_kernel(
    int S, int H_kv, int max_pages, int r, const KT* __restrict__ k_cache,
    const int32_t* __restrict__ page_table, const int32_t* __restrict__ seq_lens,
    const int32_t* __restrict__ build_list, int n_items, int all_pages,
    uint8_t* __restrict__ summaries, float* __restrict__ mu_out, float* __restrict__ basis_out,
    float* __restrict__ coef_out, float* __restrict__ sigma2_out) {
  constexpr int kI = 64 / B;            // items per wave
  constexpr int kNG = B / 16;           // 16-column groups
  constexpr int kVec = 16 / (int)sizeof(KT);  // key elements per 16-byte load
  constexpr int kPad = B + 4;           // LDS row stride (floats) of Gram rows and vectors
  constexpr int kCPL = kMaxR <= 8 ? 8 : 16;   // vector components per lane (back-transform)
  constexpr int kLPV = B / kCPL;              // lanes per vector
  constexpr int kUS = kMaxR <= 8 ? 9 : 17;    // LDS stride (floats) of a row of U
  // LDS phases of sBig: 32 Gram rows at a time (layout change), the reflectors, U
  constexpr int kGramF = 32 * kPad, kReflF = kI * (128 * kNG * (kNG + 1) - 16), kUF = kI * B * kUS;
  constexpr int kBig0 = kGramF > kReflF ? kGramF : kReflF;
  __shared__ __align__(16) float sBig[kBig0 > kUF ? kBig0 : kUF];
  __shared__ __align__(16) float sX[kI][kMaxR <= 8 ? 8 : 16][kPad];  // eigenvectors of T
  __shared__ __align__(16) float sMu[kI][kDim];
  __shared__ __align__(16) float sD[kI][B];   // diagonal of T
  __shared__ __align__(16) float sE[kI][B];   // off-diagonal of T (e[k] couples k, k + 1)
  __shared__ float sLam[kI][B];               // eigenvalues, descending
  // e[k - 1]^2 (Sturm counts) before the eigenvectors take sX; the flips after sD is read
  auto& sE2 = *reinterpret_cast<float(*)[kI][B]>(&sX[0][0][0]);
  auto& sFlip = *reinterpret_cast<float(*)[kI][16]>(&sD[0][0]);

  const int lane = threadIdx.x;
  const int it = lane / B, i = lane % B;
  const int l16 = lane & 15, q4 = lane >> 4;

  // ---- which (seq, page, KV head) the block's items are
  PageItem item[kI];
  bool any = false;
#pragma unroll
  for (int t = 0; t < kI; ++t) {
    const long id = (long)blockIdx.x * kI + t;
    PageItem p{false, (int)(id % H_kv), 0, 0};
    const long rest = id / H_kv;
    int s = 0, j = 0;
    if (all_pages) {
      j = (int)(rest % max_pages);
      s = (int)(rest / max_pages);
      p.active = s < S && j < seq_lens[s < S ? s : 0] / B;
    } else if (rest < n_items) {
      p.e = (int)rest;
      s = build_list[2 * rest];
      j = build_list[2 * rest + 1];
      p.active = s >= 0 && s < S && j >= 0 && j < max_pages && j < seq_lens[s >= 0 && s < S ? s : 0] / B;
    }
    const long blk = p.active ? (long)page_table[(long)s * max_pages + j] : 0;
    p.row = blk * H_kv + p.h;
    any |= p.active;
    item[t] = p;
  }
  if (!any) return;
  auto kpage = [&](int t) { return k_cache + item[t].row * (long)B * kDim; };
  // 16 bytes of item t at token tok0 (uniform) and lane offset `off` bytes (zeros for an
  // inactive item)
  auto key16 = [&](int t, int tok0, uint32_t off) {
    const char* p = reinterpret_cast<const char*>(kpage(t) + tok0 * kDim);
    return item[t].active ? *reinterpret_cast<const uint4*>(p + off) : make_uint4(0, 0, 0, 0);
  };
  constexpr uint32_t kEl = sizeof(KT);
  const uint32_t off_row = (uint32_t)(q4 * kDim + 8 * l16) * kEl;      // token q4, dims 8 l16 ..
  const uint32_t off_op = (uint32_t)(l16 * kDim + kVec * q4) * kEl;   // row l16, columns kVec q4 ..

  // ---- centroid and mean squared norm: lane (q4, l16) sums dims 8 l16 .. + 7 over the
  //      tokens 4 s + q4, pairwise (exact for equal rows), then over q4
  float energy = 0.0f;
#pragma unroll
  for (int t = 0; t < kI; ++t) {
    float en = 0.0f, sum[8];
    // partial sums over runs of s, merged as a binary counter
    float part[5][8];
#pragma unroll
    for (int s = 0; s < B / 4; ++s) {
      if (s % 8 == 0) __builtin_amdgcn_sched_barrier(0);  // bounds the loads in flight
      float x[8];
#pragma unroll
      for (int u = 0; u < 8 / kVec; ++u)
        chunk_to_f<KT>(key16(t, 4 * s, off_row + 16u * u), &x[u * kVec]);
#pragma unroll
      for (int e = 0; e < 8; ++e) en = fmaf(x[e], x[e], en);
      int lvl = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (((s >> b) & 1) && lvl == b) {
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] = part[b][e] + x[e];
          lvl = b + 1;
        }
#pragma unroll
      for (int e = 0; e < 8; ++e) part[lvl][e] = x[e];
    }
    constexpr int kTop = B == 64 ? 4 : 3;
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[e] = swap16_add(swap32_add(part[kTop][e])) * (1.0f / B);
    if (q4 == 0) {
      *reinterpret_cast<float4*>(&sMu[t][8 * l16]) = make_float4(sum[0], sum[1], sum[2], sum[3]);
      *reinterpret_cast<float4*>(&sMu[t][8 * l16 + 4]) = make_float4(sum[4], sum[5], sum[6], sum[7]);
    }
    en = group_sum<64>(en) * (1.0f / B);
    energy = it == t ? en : energy;
  }
  __syncthreads();

  // ---- Gram of the deviations on fp32 MFMA 16x16x4, upper tiles: the lane supplies rows
  //      16 T + l16 at columns kVec (4 ch + q4) + m as both operands; register jj then
  //      holds G[16 T + 4 q4 + jj][16 U + l16].  Row i goes to lane i through LDS, 32
  //      rows of an item at a time.
  float a[B];
  int ex = 0;  // the rows are scaled by 2^-ex, so that the trace lies in [1/2, 1)
  {
    float dg = 0.0f;
    constexpr int kTiles = kNG * (kNG + 1) / 2;
    f4 acc[kI][kTiles];
#pragma unroll
    for (int t = 0; t < kI; ++t) {
#pragma unroll
      for (int n = 0; n < kTiles; ++n) acc[t][n] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int ch = 0; ch < kDim / (4 * kVec); ++ch) {
        if (B == 64) __builtin_amdgcn_sched_barrier(0);
        const int c0 = kVec * (4 * ch + q4);
        float x[kNG][kVec];
#pragma unroll
        for (int T = 0; T < kNG; ++T) chunk_to_f<KT>(key16(t, 16 * T, off_op + 64u * ch), x[T]);
#pragma unroll
        for (int m = 0; m < kVec; ++m) {
          const float mu = sMu[t][c0 + m];
#pragma unroll
          for (int T = 0; T < kNG; ++T) x[T][m] -= mu;
          int n = 0;
#pragma unroll
          for (int T = 0; T < kNG; ++T)
#pragma unroll
            for (int U = T; U < kNG; ++U) {
              acc[t][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[T][m], x[U][m], acc[t][n], 0, 0, 0);
              ++n;
            }
        }
      }
    }
    // 32 rows at a time: item st (B = 32) or rows 32 st .. of the item (B = 64)
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      const int t = B == 32 ? st : 0, hf = B == 32 ? 0 : st;
      float* A = sBig - hf * 32 * kPad;
      int n = 0;
#pragma unroll
      for (int T = 0; T < kNG; ++T)
#pragma unroll
        for (int U = T; U < kNG; ++U) {
          const f4 g = acc[t][n++];
          if (U / 2 == hf)  // G[16 U + l16][16 T + 4 q4 + jj], by symmetry
            *reinterpret_cast<float4*>(A + (16 * U + l16) * kPad + 16 * T + 4 * q4) =
                make_float4(g[0], g[1], g[2], g[3]);
          if (U != T && T / 2 == hf)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) A[(16 * T + 4 * q4 + jj) * kPad + 16 * U + l16] = g[jj];
        }
      __syncthreads();
      const bool mine = (lane >> 5) == st;
      const float* row = sBig + (lane & 31) * kPad;
      if (mine) dg = row[i];
#pragma unroll
      for (int q = 0; q < B / 4; ++q) {
        const float4 v = *reinterpret_cast<const float4*>(row + 4 * q);
        if (st == 0 || mine) {
          a[4 * q] = v.x;
          a[4 * q + 1] = v.y;
          a[4 * q + 2] = v.z;
          a[4 * q + 3] = v.w;
        }
      }
      __syncthreads();
    }
    const float tr = group_sum<B>(dg);
    ex = tr > 0.0f && tr < INFINITY ? __builtin_amdgcn_frexp_expf(tr) : 0;
#pragma unroll
    for (int j = 0; j < B; ++j) a[j] = __builtin_amdgcn_ldexpf(a[j], -ex);
  }

  // ---- Householder reduction to tridiagonal form.  Step k annihilates column k above
  //      row k - 1 with H = I - tau v v^T (v_{k-1} = 1) and updates the leading block by
  //      the rank-2 form A - v w^T - w v^T.  v and w are zero at rows >= k, so whole
  //      16-column groups run without a mask (the skipped products are exact zeros).
  //      A column whose entries above row k - 1 are below 2^-40 of the trace counts as
  //      reduced: the rounding residue of a page of few modes shrinks step by step
  //      towards the denormals, where the hardware reciprocals overflow.
  float* refl = sBig + it * (128 * kNG * (kNG + 1) - 16);
#pragma unroll 1
  for (int t = kNG - 1; t >= 0; --t) {
    static_range<0, 16>([&](auto sc) __attribute__((always_inline)) {
      constexpr int s = 15 - decltype(sc)::value;
      const int k = 16 * t + s;
      if (s < 2 && t == 0) return;  // columns 1 and 0 are done
      const int tg = s == 0 ? t - 1 : t;  // group of row k - 1
      float x = a[s];
#pragma unroll
      for (int g = 1; g < kNG; ++g) x = t == g ? a[16 * g + s] : x;
      float x0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), k - 1));
      if (kI == 2) {
        const float x1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), B + k - 1));
        x0 = it ? x1 : x0;
      }
      const float sig = group_sum<B>(i < k - 1 ? x * x : 0.0f);
      float tau = 0.0f, v0 = 1.0f, beta = x0;
      if (sig > 0x1p-80f) {
        const float mu = root(fmaf(x0, x0, sig));
        v0 = x0 <= 0.0f ? x0 - mu : -quot(sig, x0 + mu);
        tau = quot(2.0f * v0 * v0, fmaf(v0, v0, sig));
        beta = mu;
      }
      const float vi = i == k - 1 ? 1.0f : (i < k - 1 && sig > 0x1p-80f ? quot(x, v0) : 0.0f);
      if (i == k) {
        sD[it][k] = x;
        sE[it][k - 1] = beta;
      }
      // (kept as sqrt(tau) v: the back-transformation's H is then I - v v^T; the root
      // refined by one Newton step, 0 for tau = 0)
      const float ty = __builtin_amdgcn_rsqf(fmaxf(tau, 0x1p-126f)), ts = tau * ty;
      if (i < 16 * (tg + 1)) refl[refl_off(k) + i] = vi * fmaf(fmaf(-ts, ts, tau), 0.5f * ty, ts);
      float vs[kNG], ws[kNG];
      segments<B>(vi, vs);
      // p = tau A v over the leading block
      // (two partial sums: shorter chains of rounding)
      float p = 0.0f, p1 = 0.0f;
      static_range<0, kNG>([&](auto gc) __attribute__((always_inline)) {
        constexpr int g = decltype(gc)::value;
        if (g == 0 || g <= tg) {
          dot8<0>(p, vs[g], *reinterpret_cast<float(*)[8]>(&a[16 * g]));
          dot8<8>(p1, vs[g], *reinterpret_cast<float(*)[8]>(&a[16 * g + 8]));
        }
      });
      p = i < k ? tau * (p + p1) : 0.0f;
      const float kc = 0.5f * tau * group_sum<B>(p * vi);
      const float wi = fmaf(-kc, vi, p);
      segments<B>(wi, ws);
      const float nv = -vi, nw = -wi;
      static_range<0, kNG>([&](auto gc) __attribute__((always_inline)) {
        constexpr int g = decltype(gc)::value;
        if (g == 0 || g <= tg) {
          rank2_8<0>(&a[16 * g], vs[g], ws[g], nv, nw);
          rank2_8<8>(&a[16 * g + 8], vs[g], ws[g], nv, nw);
        }
      });
    });
  }
  if (i < 2) sD[it][i] = i ? a[1] : a[0];
  if (i == 1) sE[it][0] = a[0];
  if (i == B - 1) sE[it][B - 1] = 0.0f;
  __syncthreads();
  sE2[it][i] = i > 0 ? fmaf(sE[it][i - 1], sE[it][i - 1], 0x1p-126f) : 0.0f;
  __syncthreads();

  // ---- the wanted eigenvalues of T (the r largest; all B for the factor output)
  //      by multisection on Sturm counts: q = B / n lanes per eigenvalue, one
  //      point each per step, so a group cuts its interval into q + 1 parts and
  //      a wave ballot gives the part that holds the eigenvalue
  float lam, tn = 0.0f;
  {
    float lo, hi;
    {
      const float el = i > 0 ? fabsf(sE[it][i - 1]) : 0.0f, er = fabsf(sE[it][i]), dd = sD[it][i];
      lo = -group_max<B>(el + er - dd);
      hi = group_max<B>(dd + el + er);
      tn = group_max<B>(fabsf(dd) + el + er);
    }
    const int ne = kFactors ? B : r;
    const int q = B / ne;
    const int lq = i / q;
    const bool idle = lq >= ne;            // lanes past ne * q copy the last group
    const int le = idle ? ne - 1 : lq;     // the eigenvalue (0 = largest)
    const int pi = idle ? 0 : i - lq * q;  // this lane's point
    const int want = B - 1 - le;           // count(x) <= want  <=>  x <= lambda_le
    const uint64_t gmask = (q >= 64 ? ~0ull : ((1ull << q) - 1ull)) << (it * B + le * q);
    // the Sturm counts carry rounding of a few ulp of |T|: the interval is cut to
    // 2^-22 of its width (2^-24 for the factor output)
    int steps = 0;
    for (float w = 1.0f; w > (kFactors ? 0x1p-24f : 0x1p-22f); w /= (float)(q + 1)) ++steps;
#pragma unroll 1
    for (int st = 0; st < steps; ++st) {
      const float hstep = (hi - lo) / (float)(q + 1);
      const float x = fmaf((float)(pi + 1), hstep, lo);
      float qv = 1.0f;
      uint32_t cnt = 0;
#pragma unroll
      for (int qq = 0; qq < B / 4; ++qq) {
        const float4 d4 = *reinterpret_cast<const float4*>(&sD[it][4 * qq]);
        const float4 e4 = *reinterpret_cast<const float4*>(&sE2[it][4 * qq]);
        const float dd[4] = {d4.x, d4.y, d4.z, d4.w}, ee[4] = {e4.x, e4.y, e4.z, e4.w};
#pragma unroll
        for (int u2 = 0; u2 < 4; ++u2) {
          // q_t = (d_t - x) - e_{t-1}^2 / q_{t-1}, counted by sign bit: a zero
          // pivot makes the next one infinite with the opposite sign, and
          // e^2 >= FLT_MIN keeps 0 * inf out
          qv = fmaf(-ee[u2], __builtin_amdgcn_rcpf(qv), dd[u2] - x);
          cnt += __float_as_uint(qv) >> 31;
        }
      }
      const int nle = __popcll(__ballot((int)cnt <= want) & gmask);
      const float nlo = nle > 0 ? fmaf((float)nle, hstep, lo) : lo;
      const float nhi = nle < q ? fmaf((float)(nle + 1), hstep, lo) : hi;
      lo = nlo;
      hi = nhi;
    }
    const float lam_g = 0.5f * (lo + hi);
    lam = __shfl(lam_g, it * B + (i < ne ? i : ne - 1) * q, 64);
    sLam[it][i] = __builtin_amdgcn_ldexpf(lam, ex);
  }
  __syncthreads();
  const float floor_ = fmaxf(kZeroRel * fmaxf(sLam[it][0], 0.0f), kZeroAbs * energy);

  // ---- eigenvectors of T: lane l < r runs inverse iteration for eigenvalue l on
  //      T - lambda_l I = L D L^T (no pivoting; a pivot below eps |T| is replaced by
  //      eps |T|, which only scales the solution); L's entries are e_{t-1} / pivot_{t-1}
  {
    const float tiny = fmaxf(tn, 1e-30f) * 1.2e-7f;
    float Wi[B], X[B];  // reciprocal pivots, the vector
    auto e_at = [&](int t) { return sE[it][t]; };
    {
      // start vector: a fixed sequence that differs between the r vectors
      float ph = 0.37f * (float)(i + 1);
      const float stp = 0.6180339f + 0.0917f * (float)i;
#pragma unroll
      for (int t = 0; t < B; ++t) {
        ph = __builtin_amdgcn_fractf(ph + stp);
        X[t] = fmaf(ph, 1.5f, 1.0f);
      }
      float pv = sD[it][0] - lam;
      if (fabsf(pv) < tiny) pv = pv < 0.0f ? -tiny : tiny;
      Wi[0] = __builtin_amdgcn_rcpf(pv);
#pragma unroll
      for (int t = 1; t < B; ++t) {
        const float el = e_at(t - 1);
        if (t % 8 == 0) __builtin_amdgcn_sched_barrier(0);  // bounds the T entries in flight
        pv = fmaf(-el * Wi[t - 1], el, sD[it][t] - lam);
        if (fabsf(pv) < tiny) pv = pv < 0.0f ? -tiny : tiny;
        Wi[t] = __builtin_amdgcn_rcpf(pv);
      }
    }
#pragma unroll 1
    for (int round = 0; round < kInvRounds; ++round) {
      // L y = x, then D z = y, then L^T x = z; scaled to unit max to stay finite
#pragma unroll
      for (int t = 1; t < B; ++t) {
        if (t % 8 == 0) __builtin_amdgcn_sched_barrier(0);
        X[t] = fmaf(-(e_at(t - 1) * Wi[t - 1]), X[t - 1], X[t]);
      }
      X[B - 1] *= Wi[B - 1];
      float amax = fabsf(X[B - 1]);
#pragma unroll
      for (int t = B - 2; t >= 0; --t) {
        if (t % 8 == 0) __builtin_amdgcn_sched_barrier(0);
        X[t] = fmaf(-e_at(t), X[t + 1], X[t]) * Wi[t];
        amax = fmaxf(amax, fabsf(X[t]));
      }
      const float sc = amax > 0.0f ? __builtin_amdgcn_rcpf(amax) : 1.0f;
      if (i < r) {
#pragma unroll
        for (int q = 0; q < B / 4; ++q)
          *reinterpret_cast<float4*>(&sX[it][i][4 * q]) =
              make_float4(X[4 * q] * sc, X[4 * q + 1] * sc, X[4 * q + 2] * sc, X[4 * q + 3] * sc);
      }
      __syncthreads();
      // modified Gram-Schmidt over the vectors in eigenvalue order; lane i holds
      // component i (right-looking: a final vector is projected out of every later
      // one at once, their lane reductions overlapping; vectors past r are zero)
      float xr[kMaxR];
#pragma unroll
      for (int l = 0; l < kMaxR; ++l) xr[l] = l < r ? sX[it][l][i] : 0.0f;
      static_range<0, kMaxR>([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value;
        const float nn = group_sum<B>(xr[m] * xr[m]);
        xr[m] = nn > 0.0f ? xr[m] * __builtin_amdgcn_rsqf(nn) : 0.0f;
        if constexpr (m + 1 < kMaxR) {
          float d[kMaxR - 1 - m];
#pragma unroll
          for (int l = m + 1; l < kMaxR; ++l) d[l - m - 1] = xr[l] * xr[m];
          group_sums<B, kMaxR - 1 - m>(d);
#pragma unroll
          for (int l = m + 1; l < kMaxR; ++l) xr[l] = fmaf(-d[l - m - 1], xr[m], xr[l]);
        }
      });
      __syncthreads();
#pragma unroll
      for (int l = 0; l < (kMaxR <= 8 ? 8 : 16); ++l) sX[it][l][i] = l < kMaxR ? xr[l] : 0.0f;
      __syncthreads();
      if (round + 1 < kInvRounds) {
        const int iv = i < r ? i : 0;
#pragma unroll
        for (int q = 0; q < B / 4; ++q) {
          const float4 v = *reinterpret_cast<const float4*>(&sX[it][iv][4 * q]);
          X[4 * q] = v.x;
          X[4 * q + 1] = v.y;
          X[4 * q + 2] = v.z;
          X[4 * q + 3] = v.w;
        }
        __syncthreads();
      }
    }
  }

  // ---- back-transformation u_l = H_{B-1} ... H_3 H_2 x_l: lane (it, l, c) holds
  //      components kCPL c .. of vector l
  {
    const int l = i / kLPV, c = i % kLPV;
    float y[kCPL];
#pragma unroll
    for (int m = 0; m < kCPL; m += 4) {
      const float4 v = *reinterpret_cast<const float4*>(&sX[it][l][kCPL * c + m]);
      y[m] = v.x;
      y[m + 1] = v.y;
      y[m + 2] = v.z;
      y[m + 3] = v.w;
    }
#pragma unroll 4
    for (int k = 2; k < B; ++k) {
      const bool in = kCPL * c < 16 * (((k - 1) >> 4) + 1);  // inside the stored reflector
      const float* v = refl + refl_off(k) + (in ? kCPL * c : 0);
      float x[kCPL];
#pragma unroll
      for (int m = 0; m < kCPL; m += 4) {
        const float4 w = *reinterpret_cast<const float4*>(v + m);
        x[m] = w.x;
        x[m + 1] = w.y;
        x[m + 2] = w.z;
        x[m + 3] = w.w;
      }
      float d0 = 0.0f, d1 = 0.0f;
#pragma unroll
      for (int m = 0; m < kCPL; m += 2) {
        d0 = fmaf(x[m], y[m], d0);
        d1 = fmaf(x[m + 1], y[m + 1], d1);
      }
      float d = in ? d0 + d1 : 0.0f;
      d += dpp_f<0xB1>(d);
      if (kLPV >= 4) d += dpp_f<0x4E>(d);
      if (kLPV >= 8) d += dpp_f<0x141>(d);
      const float f = in ? -d : 0.0f;
#pragma unroll
      for (int m = 0; m < kCPL; ++m) y[m] = fmaf(f, x[m], y[m]);
    }
    __syncthreads();  // the reflectors are no longer read: U takes their LDS
    if (l < kMaxR) {
#pragma unroll
      for (int m = 0; m < kCPL; ++m) sBig[(it * B + kCPL * c + m) * kUS + l] = y[m];
    }
  }
  __syncthreads();
  auto U_at = [&](int t, int row, int l) { return sBig[(t * B + row) * kUS + l]; };

  // ---- basis columns V[:, l] = D^T u_l / sigma_l on fp32 MFMA 16x16x4: rows are the
  //      vectors, columns the dims 8 l16 + T of tile T, K the tokens 4 s + q4, whose keys
  //      the lane reads 16 bytes at a time (cache-resident).  Ranks up to 8 put item t's
  //      vectors in rows 8 t .. 8 t + 7, so both items of a 32-token wave share the
  //      accumulators; then sign, quantisation and packing of four vectors per lane.
  const int stride = rec_stride(r, 0, B);
  float fl[kI];
#pragma unroll
  for (int t = 0; t < kI; ++t) fl[t] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(floor_), t * B));
  constexpr int kPassItems = kMaxR <= 8 ? kI : 1;  // items per pass
#pragma unroll
  for (int t0 = 0; t0 < kI; t0 += kPassItems) {
    f4 acc[8];
#pragma unroll
    for (int T = 0; T < 8; ++T) acc[T] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int t = t0; t < t0 + kPassItems; ++t) {
      float mu8[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) mu8[e] = sMu[t][8 * l16 + e];
      const int ur = kPassItems > 1 ? l16 - 8 * t : l16;   // vector of this lane's A row
      const bool uok = ur >= 0 && ur < kMaxR;
#pragma unroll
      for (int s = 0; s < B / 4; ++s) {
        if (s % 8 == 0) __builtin_amdgcn_sched_barrier(0);
        const float uv = uok ? U_at(t, 4 * s + q4, uok ? ur : 0) : 0.0f;
        float x[8];
#pragma unroll
        for (int u = 0; u < 8 / kVec; ++u)
          chunk_to_f<KT>(key16(t, 4 * s, off_row + 16u * u), &x[u * kVec]);
#pragma unroll
        for (int T = 0; T < 8; ++T)
          acc[T] = __builtin_amdgcn_mfma_f32_16x16x4f32(uv, x[T] - mu8[T], acc[T], 0, 0, 0);
      }
    }
    const int pt = kPassItems > 1 ? q4 >> 1 : t0;              // this lane's item
    const int lb = kPassItems > 1 ? 4 * (q4 & 1) : 4 * q4;     // its first vector
    const bool act = kI > 1 && kPassItems > 1 ? (pt ? item[kI - 1].active : item[0].active) : item[t0].active;
    const long orow = kI > 1 && kPassItems > 1 ? (pt ? item[kI - 1].row : item[0].row) : item[t0].row;
    const int oe = kI > 1 && kPassItems > 1 ? (pt ? item[kI - 1].e : item[0].e) : item[t0].e;
    const int oh = kI > 1 && kPassItems > 1 ? (pt ? item[kI - 1].h : item[0].h) : item[t0].h;
    const float fle = kI > 1 && kPassItems > 1 ? (pt ? fl[kI - 1] : fl[0]) : fl[t0];
    uint8_t* rec = summaries + orow * (long)stride;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int l = lb + jj;
      if (l >= r) continue;
      const float lv = sLam[pt][l];
      const bool kl = lv > fle && lv > 0.0f;
      const float isig = kl ? 1.0f / sqrtf(lv) : 0.0f;
      float v[8], best = -1.0f, bval = 0.0f;
      int bidx = 0;
#pragma unroll
      for (int T = 0; T < 8; ++T) {
        v[T] = acc[T][jj] * isig;
        const float av = fabsf(v[T]);
        if (av > best) { best = av; bidx = 8 * l16 + T; bval = v[T]; }
      }
      // sign convention: the largest |V[c][l]| (lowest c on ties) is made positive:
      // the largest magnitude over the row, then the lowest dim holding it, its sign in
      // the low bit
      const float gbest = row_max(best);
      const int key = row_min_int(best == gbest ? 2 * bidx + (bval < 0.0f ? 1 : 0) : 0x7fffffff);
      const float flip = (key & 1) ? -1.0f : 1.0f;
      if (l16 == 0) sFlip[pt][l] = flip;
      if (kFactors) {
        if (act) {
          float* bo = basis_out + ((long)oe * H_kv + oh) * kDim * r;
#pragma unroll
          for (int T = 0; T < 8; ++T) bo[(8 * l16 + T) * r + l] = flip * v[T];
        }
      } else {
        const float vsc = f16_scale(gbest, 7.0f);
        const float ivs = inv_scale(vsc);
        uint32_t word = 0;
#pragma unroll
        for (int T = 0; T < 8; ++T) word |= (uint32_t)(quant(flip * v[T], ivs, 7) + 8) << (4 * T);
        if (act) {
          *reinterpret_cast<uint32_t*>(rec + 64 * l + 4 * l16) = word;
          if (l16 == 0) *reinterpret_cast<uint16_t*>(rec + rec_scale_off(r, 0, B) + 2 * l) = f16_bits(vsc);
        }
      }
    }
  }
  __syncthreads();

  // ---- coefficient row i: C[i][l] = flip_l u_l[i] sigma_l (0 for a dropped mode)
  const bool act = kI > 1 ? (it ? item[kI - 1].active : item[0].active) : item[0].active;
  if (!act) return;
  const long orow = kI > 1 ? (it ? item[kI - 1].row : item[0].row) : item[0].row;
  float crow[kMaxR], cabs = 0.0f;
#pragma unroll
  for (int l = 0; l < kMaxR; ++l) {
    const float lv = sLam[it][l];
    const bool kl = l < r && lv > floor_ && lv > 0.0f;
    crow[l] = kl ? sFlip[it][l] * U_at(it, i, l) * sqrtf(lv) : 0.0f;
    cabs = fmaxf(cabs, fabsf(crow[l]));
  }
  constexpr int kC = kDim / B;  // centroid elements of this lane
  if (kFactors) {
    const long oi = (long)(kI > 1 ? (it ? item[kI - 1].e : item[0].e) : item[0].e) * H_kv +
                    (kI > 1 ? (it ? item[kI - 1].h : item[0].h) : item[0].h);
#pragma unroll
    for (int cc = 0; cc < kC; ++cc) mu_out[oi * kDim + kC * i + cc] = sMu[it][kC * i + cc];
#pragma unroll
    for (int l = 0; l < kMaxR; ++l)
      if (l < r) coef_out[(oi * B + i) * r + l] = crow[l];
    sigma2_out[oi * B + i] = fmaxf(sLam[it][i], 0.0f);
    return;
  }
  uint8_t* rec = summaries + orow * (long)stride;
  const int scale_off = rec_scale_off(r, 0, B);
  {
    const float cs = f16_scale(cabs, 127.0f);
    uint8_t* dst = rec + rec_coef_off(r) + i * r;
    if (kMaxR == 8 && r == 8) {
      uint32_t w[2] = {0u, 0u};
#pragma unroll
      for (int l = 0; l < 8; ++l) w[l >> 2] |= (uint32_t)(quant_div(crow[l], cs, 127) + 128) << (8 * (l & 3));
      *reinterpret_cast<uint2*>(dst) = make_uint2(w[0], w[1]);
    } else {
#pragma unroll
      for (int l = 0; l < kMaxR; ++l)
        if (l < r) dst[l] = (uint8_t)(quant_div(crow[l], cs, 127) + 128);
    }
    *reinterpret_cast<uint16_t*>(rec + scale_off + 2 * (r + i)) = f16_bits(cs);
  }
  {
    float m = 0.0f;
#pragma unroll
    for (int cc = 0; cc < kC; ++cc) m = fmaxf(m, fabsf(sMu[it][kC * i + cc]));
    m = group_max<B>(m);
    const float ms = f16_scale(m, 127.0f);
    uint32_t w = 0;
#pragma unroll
    for (int cc = 0; cc < kC; ++cc) w |= (uint32_t)(quant_div(sMu[it][kC * i + cc], ms, 127) + 128) << (8 * cc);
    uint8_t* dst = rec + rec_mu_off(r, 0, B) + kC * i;
    if (kC == 4) *reinterpret_cast<uint32_t*>(dst) = w;
    else *reinterpret_cast<uint16_t*>(dst) = (uint16_t)w;
    if (i == 0) *reinterpret_cast<uint16_t*>(rec + scale_off + 2 * (r + B)) = f16_bits(ms);
  }
  if (rec_payload(r, 0, B) + i < stride) rec[rec_payload(r, 0, B) + i] = 0;
}

}  // namespace

hipError_t launch_build_page(const locks_cfg_t& c, const void* k_cache, const int32_t* page_table,
                             const int32_t* seq_lens, const int32_t* build_list, int32_t n_items,
                             bool all_pages, void* summaries, float* mu, float* basis,
                             float* coef, float* sigma2, hipStream_t st) {
  const long items = all_pages ? (long)c.num_seqs * c.max_pages_per_seq * c.num_kv_heads
                               : (long)n_items * c.num_kv_heads;
  if (items == 0) return hipSuccess;
  const bool factors = mu != nullptr;
  const int per = 64 / c.page_size;
  const long blocks = (items + per - 1) / per;
  if (blocks > 0x7fffffffL) return hipErrorInvalidConfiguration;
  if (c.basis != LOCKS_BASIS_INT4) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(64);
  // ranks up to 8 take the instance whose rank-sized arrays (LDS and registers)
  // hold 8 vectors: its smaller LDS fits more waves per compute unit
#define LOCKS_BUILD_PAGE_R(KT, BP, F, MR)                                                      \
  hipLaunchKernelGGL((build_page_kernel<KT, BP, F, MR>), grid, block, 0, st, c.num_seqs,        \
                     c.num_kv_heads, c.max_pages_per_seq, c.rank, static_cast<const KT*>(k_cache), \
                     page_table, seq_lens, build_list, n_items, (int)all_pages,                \
                     (uint8_t*)summaries, mu, basis, coef, sigma2)
#define LOCKS_BUILD_PAGE(KT, BP, F)                                                            \
  if (c.rank <= 8) LOCKS_BUILD_PAGE_R(KT, BP, F, 8); else LOCKS_BUILD_PAGE_R(KT, BP, F, kMaxRank)
#define LOCKS_BUILD_PAGE_B(KT)                                                                 \
  switch (c.page_size) {                                                                       \
    case 32: if (factors) LOCKS_BUILD_PAGE(KT, 32, true); else LOCKS_BUILD_PAGE(KT, 32, false); break; \
    case 64: if (factors) LOCKS_BUILD_PAGE(KT, 64, true); else LOCKS_BUILD_PAGE(KT, 64, false); break; \
    default: return hipErrorInvalidValue;                                                      \
  }
  if (c.kv_dtype == LOCKS_BF16) {
    LOCKS_BUILD_PAGE_B(uint16_t);
  } else {
    LOCKS_BUILD_PAGE_B(float);
  }
#undef LOCKS_BUILD_PAGE_B
#undef LOCKS_BUILD_PAGE
#undef LOCKS_BUILD_PAGE_R
  return hipGetLastError();
}

}  // namespace locks
