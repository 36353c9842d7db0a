// Summary scan (Sec. 4 "Score", Eq. (1)): for every complete page j of a
// (sequence, KV head) and every query head g of its group,
//   hat s_j(q_g) = log sum_i exp[(q_g^T mu_j + (V_j^T q_g)^T c_i) / sqrt(d)],
// read from the page's stored record (int4 basis, int8 coefficients and centroid,
// float16 scales).  Every block also writes, per query head, the partial
// (max, sum 2^x) of its pages' scores in the log2 domain; the select kernel
// reduces them into log Z_g = log sum_j exp(hat s_j(q_g)).
#include "locks_internal.h"
#include "scan_common.h"
#include "scan_launch.h"

namespace locks {
namespace {

// ---------------------------------------------------------------------------
// Matrix-core scan (group size G <= 16).
//
// A wave owns 64 consecutive pages (four tiles of 16) of one (sequence, KV head).
// Per tile:
//  * stage 1, the projections p = V^T q and a = mu^T q, run on 16x16x32 f16 MFMA:
//    rows are (page, basis column) pairs (16/r pages per set), columns are query
//    heads, K = d.  Each lane loads its 16-byte slice of one basis column straight
//    into its A operand; nibbles are decoded exactly to f16 through the 1024.0
//    exponent trick (OR into the mantissa, subtract the excess-8 bias in packed
//    f16).  The queries (bf16 or fp32 split hi + lo, both exact in f16 after a
//    power-of-two range scale) are the B operand, built once per wave.
//  * the rest of each record (coefficients, centroid, scales) is staged in LDS;
//    the centroid projection runs as one more MFMA set with one page per row.
//  * stage 2, the 16 logits z_i = a + c_i^T p, runs on 16x16x4 fp32 MFMA with the
//    16 tokens as rows; the 16 columns pack 16/G pages x G heads and the K axis is
//    block-diagonal over those pages, so small groups waste no lanes.
//  * log-sum-exp over the 16 rows: 4 values per lane, then two cross-lane steps.
// ---------------------------------------------------------------------------

template <int R, int BB = 0>
struct Geom {
  static constexpr int kPPS = (16 / R) > 0 ? 16 / R : 1;          // pages per stage-1 set
  static constexpr int kSets = (16 + kPPS - 1) / kPPS;
  static constexpr int kColB = rec_col_bytes(BB);                  // bytes per basis column
  static constexpr int kVW = 1 << BB;                              // 16-byte basis loads per lane and set
  static constexpr int kStride = rec_stride(R, BB);
  static constexpr int kTail = kStride - kColB * R;                // coef .. end of record
  static constexpr int kTailCh = kTail / 16;
  static constexpr int kTailLoads = (16 * kTailCh + 63) / 64;
  static constexpr int kMu = 16 * R;                               // offsets inside the tail
  static constexpr int kSc = 16 * R + kDim;
};

template <int R, int BB = 0>
struct TileRegs {
  uint4 vb[BB == 0 ? Geom<R, BB>::kSets : 1][Geom<R, BB>::kVW];  // basis slices (int4: per tile)
  uint4 tl[Geom<R, BB>::kTailLoads];  // record tails, 16-byte chunks
  int blk;                            // lanes 0..15: block of page page0 + lane (-1: none)
};

// The basis slices of stage-1 set st of a tile: lane (grp, col) takes the 32
// elements 32 grp .. 32 grp + 31 of column l = col % R of page st kPPS + col / R
// (16 << BB bytes).
template <int R, int BB>
__device__ __forceinline__ void load_set(uint4* vb, const uint8_t* __restrict__ summaries,
                                         int my_blk, int st, int H_kv, int h, int lane) {
  using Gm = Geom<R, BB>;
  const int col = lane & 15, grp = lane >> 4;
  const int pp = col / R, l = col % R;
  const int page = st * Gm::kPPS + pp;
  const int blk = __shfl(my_blk, page < 16 ? page : 0, 64);
  const bool ok = col < Gm::kPPS * R && page < 16 && blk >= 0;
#pragma unroll
  for (int w = 0; w < Gm::kVW; ++w)
    vb[w] = ok ? *reinterpret_cast<const uint4*>(summaries + ((long)blk * H_kv + h) * Gm::kStride +
                                                 Gm::kColB * l + (16 << BB) * grp + 16 * w)
               : make_uint4(0, 0, 0, 0);
}

// Issue the loads of one 16-page tile (no wait): the record tails, and for an
// int4 basis every stage-1 slice (wider bases load theirs set by set).
template <int R, int BB = 0>
__device__ __forceinline__ void issue_tile(TileRegs<R, BB>& T, const uint8_t* __restrict__ summaries,
                                           const int32_t* __restrict__ pt_row, int page0, int n_c,
                                           int H_kv, int h, int lane) {
  using Gm = Geom<R, BB>;
  const int my_blk = (lane < 16 && page0 + lane < n_c) ? pt_row[page0 + lane] : -1;
  T.blk = my_blk;
  if constexpr (BB == 0) {
#pragma unroll
    for (int st = 0; st < Gm::kSets; ++st) load_set<R, BB>(T.vb[st], summaries, my_blk, st, H_kv, h, lane);
  }
#pragma unroll
  for (int u = 0; u < Gm::kTailLoads; ++u) {
    const int c = lane + 64 * u;
    const int page = c / Gm::kTailCh, off = (c % Gm::kTailCh) * 16;
    const int blk = __shfl(my_blk, page < 16 ? page : 0, 64);
    T.tl[u] = (c < 16 * Gm::kTailCh && blk >= 0)
                  ? *reinterpret_cast<const uint4*>(summaries + ((long)blk * H_kv + h) * Gm::kStride +
                                                    Gm::kColB * R + off)
                  : make_uint4(0, 0, 0, 0);
  }
}

// BB: basis precision (0 int4, 1 int8, 2 bf16).  Wider bases decode their slice
// to f16 in natural element order (int8 codes exactly; bf16 values to the nearest
// f16) and meet the natural-order query operand.
template <typename QT, int R, int BB = 0>
__global__ __launch_bounds__(256) void scan_mfma_kernel(
    int H_q, int H_kv, int max_pages, const QT* __restrict__ q,
    const uint8_t* __restrict__ summaries, const int32_t* __restrict__ page_table,
    const int32_t* __restrict__ seq_lens, float* __restrict__ s_hat, SHatLayout lay,
    float2* __restrict__ partials) {
  using Gm = Geom<R, BB>;
  constexpr bool kSplitQ = sizeof(QT) == 4;  // fp32 queries: f16 hi + lo
  __shared__ __align__(16) uint8_t sTail[4][16][Gm::kTail];
  __shared__ float sP[4][16][R][16];
  __shared__ float sA[4][16][16];
  __shared__ float2 sRun[4][16];

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
  const int h = blockIdx.y, s = blockIdx.z;
  const int G = H_q / H_kv;
  const int n_c = seq_lens[s] / kPage;
  const int pg = scan_chunk() * 4 + wave;  // 64-page group of this wave
  const long row0 = (long)s * H_q + (long)h * G;
  const int32_t* pt_row = page_table + (long)s * max_pages;
  const int n_parts = gridDim.x;
  float run_m = -INFINITY, run_s = 0.0f;  // running normaliser, log2 domain
  const int npack = 16 / G;                // pages per stage-2 pass
  if (pg * 64 < n_c) {
  TileRegs<R, BB> buf[2];
  issue_tile<R, BB>(buf[0], summaries, pt_row, pg * 64, n_c, H_kv, h, lane);

  // ---- B operands: column = query head, K permuted to match the decoders
  constexpr int kPerm[8] = {0, 4, 1, 5, 2, 6, 3, 7};
  float qv[4][8], qm[4][8];
  float qmax = 0.0f;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int cv = 32 * grp + 8 * ks + kPerm[j], cm = 32 * grp + 8 * ks + j;
      const float a = col < G ? load_q(q, (row0 + col) * kDim + cv) : 0.0f;
      const float b = col < G ? load_q(q, (row0 + col) * kDim + cm) : 0.0f;
      qv[ks][j] = a;
      qm[ks][j] = b;
      qmax = fmaxf(qmax, fabsf(a));
    }
  qmax = warp_max(qmax);
  // power-of-two range scale so that every query element fits f16 exactly
  float qs = 1.0f;
  while (qmax * qs > 16384.0f) qs *= 0.5f;
  const float inv_qs = 1.0f / qs;
  h8 bv[4], bm[4], bvl[4], bml[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float a = qv[ks][j] * qs, b = qm[ks][j] * qs;
      const _Float16 ah = (_Float16)a, bh = (_Float16)b;
      bv[ks][j] = ah;
      bm[ks][j] = bh;
      bvl[ks][j] = (_Float16)(a - (float)ah);
      bml[ks][j] = (_Float16)(b - (float)bh);
    }

  constexpr float kLn2 = 0.69314718055994531f;
  const float c0 = 1.4426950408889634f * 0.08838834764831845f;  // log2(e) / sqrt(128)
  const int kpass = npack * R;
  const int ksteps = (kpass + 3) / 4;
  const int pcol = col / G, gcol = col % G;
  const bool colvalid = pcol < npack;

#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int page0 = (pg * 4 + t) * 16;
    if (page0 < n_c) {
      TileRegs<R, BB>& cur = buf[t & 1];
      if (t + 1 < 4 && page0 + 16 < n_c)
        issue_tile<R, BB>(buf[(t + 1) & 1], summaries, pt_row, page0 + 16, n_c, H_kv, h, lane);
      // wider bases: every set of this tile in flight at once, ahead of the LDS
      // staging of its tail
      uint4 vall[BB == 0 ? 1 : Gm::kSets][Gm::kVW];
      if constexpr (BB != 0) {
#pragma unroll
        for (int st = 0; st < Gm::kSets; ++st) load_set<R, BB>(vall[st], summaries, cur.blk, st, H_kv, h, lane);
      }
#pragma unroll
      for (int u = 0; u < Gm::kTailLoads; ++u) {
        const int c = lane + 64 * u;
        if (c < 16 * Gm::kTailCh)
          *reinterpret_cast<uint4*>(&sTail[wave][c / Gm::kTailCh][(c % Gm::kTailCh) * 16]) = cur.tl[u];
      }
      __builtin_amdgcn_wave_barrier();

      // ---- stage 1: p = V^T q (scaled by the basis column scales)
#pragma unroll
      for (int st = 0; st < Gm::kSets; ++st) {
        f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (BB == 0) {
          const uint32_t w[4] = {cur.vb[st][0].x, cur.vb[st][0].y, cur.vb[st][0].z, cur.vb[st][0].w};
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) {
            const h8 a = nib8_to_h8(w[ks]);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, bv[ks], acc, 0, 0, 0);
            if (kSplitQ) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, bvl[ks], acc, 0, 0, 0);
          }
        } else {
          const uint4* vw = vall[st];
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) {
            h8 a;
            if constexpr (BB == 1) {
              const uint4 v = vw[ks >> 1];
              a = (ks & 1) ? byte8_to_h8(v.z, v.w) : byte8_to_h8(v.x, v.y);
            } else {
              const uint4 v = vw[ks];
              const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                a[2 * e] = (_Float16)__uint_as_float(u[e] << 16);
                a[2 * e + 1] = (_Float16)__uint_as_float(u[e] & 0xffff0000u);
              }
            }
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, bm[ks], acc, 0, 0, 0);
            if (kSplitQ) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, bml[ks], acc, 0, 0, 0);
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int m = 4 * grp + j;
          const int pp = m / R, l = m % R;
          const int page = st * Gm::kPPS + pp;
          if (m < Gm::kPPS * R && page < 16 && col < G)
            sP[wave][page][l][col] = acc[j] * inv_qs * lds_f16(&sTail[wave][page][Gm::kSc + 2 * l]);
        }
      }
      // ---- centroid term a = mu^T q, one page per row
      {
        const uint4 m0 = *reinterpret_cast<const uint4*>(&sTail[wave][col][Gm::kMu + 32 * grp]);
        const uint4 m1 = *reinterpret_cast<const uint4*>(&sTail[wave][col][Gm::kMu + 32 * grp + 16]);
        const uint32_t w[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
        f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const h8 a = byte8_to_h8(w[2 * ks], w[2 * ks + 1]);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, bm[ks], acc, 0, 0, 0);
          if (kSplitQ) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, bml[ks], acc, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int page = 4 * grp + j;
          if (col < G)
            sA[wave][page][col] =
                acc[j] * inv_qs * c0 * lds_f16(&sTail[wave][page][Gm::kSc + 2 * (R + 16)]);
        }
      }
      __builtin_amdgcn_wave_barrier();

      // ---- stage 2: 16 logits per (page, head), npack pages per pass
      for (int p0 = 0; p0 < 16; p0 += npack) {
        f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int kstep = 0; kstep < ksteps; ++kstep) {
          const int k = 4 * kstep + grp;
          const int ppk = k / R, l = k % R;
          const int pk = p0 + ppk;
          const bool kv = k < kpass && pk < 16;
          const float a = kv ? (float)((int)sTail[wave][pk][col * R + l] - 128) : 0.0f;
          const float b = (kv && colvalid && ppk == pcol) ? sP[wave][pk][l][gcol] : 0.0f;
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
        }
        const int page = p0 + pcol;
        const bool live = colvalid && page < 16 && page0 + page < n_c;
        const int pl = page < 16 ? page : 15;
        const float av = sA[wave][pl][gcol];
        const uint2 csw = *reinterpret_cast<const uint2*>(&sTail[wave][pl][Gm::kSc + 2 * (R + 4 * grp)]);
        const h2 cs01 = as_h2(csw.x), cs23 = as_h2(csw.y);
        float z[4];
        z[0] = fmaf((float)cs01.x * c0, acc[0], av);
        z[1] = fmaf((float)cs01.y * c0, acc[1], av);
        z[2] = fmaf((float)cs23.x * c0, acc[2], av);
        z[3] = fmaf((float)cs23.y * c0, acc[3], av);
        float mx = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
        mx = red4_max(mx);
        float sm = __builtin_amdgcn_exp2f(z[0] - mx) + __builtin_amdgcn_exp2f(z[1] - mx) +
                   __builtin_amdgcn_exp2f(z[2] - mx) + __builtin_amdgcn_exp2f(z[3] - mx);
        sm = red4_sum(sm);
        const float s2 = mx + __builtin_amdgcn_logf(sm);  // log2-domain page score
        if (live) {
          if (grp == 0) s_hat[lay.base(s, h) + gcol * lay.head + (long)(page0 + page) * lay.page] = s2 * kLn2;
          const float e = __builtin_amdgcn_exp2f(-fabsf(s2 - run_m));
          if (s2 > run_m) { run_s = fmaf(run_s, e, 1.0f); run_m = s2; }
          else run_s += e;
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
  }  // pages of this wave
  // ---- block partial (max, sum exp) per head over its 256 pages (log2 domain)
  if (lane < 16) sRun[wave][lane] = make_float2(run_m, run_s);
  __syncthreads();
  if (threadIdx.x < G) {
    const int g = threadIdx.x;
    float m = -INFINITY, l = 0.0f;
    for (int w = 0; w < 4; ++w)
      for (int c = g; c < npack * G; c += G) m = fmaxf(m, sRun[w][c].x);
    if (m > -INFINITY)
      for (int w = 0; w < 4; ++w)
        for (int c = g; c < npack * G; c += G) {
          const float2 v = sRun[w][c];
          if (v.y > 0.0f) l += v.y * __builtin_amdgcn_exp2f(v.x - m);
        }
    partials[(row0 + g) * n_parts + blockIdx.x] = make_float2(m, l);
  }
}

// ---------------------------------------------------------------------------
// Fast path for r in {2, 4} at G = 16 (G = 16 / NPACK; the same ranks at G = 4, and r = 8,
// have kernels of their own: scan_low.hip, scan_quad.h and scan_wide.h).
//
// Differences from the generic kernel above:
//  * stage 1 runs on 16x16x64 int8 MFMA.  A basis nibble becomes an int8 with
//    three ops per eight codes; each query head is written as a 20-bit fixed-point
//    integer (power-of-two scale per head) split into three signed 8-bit digits,
//    and one int32 accumulator takes the digits most significant first, shifted
//    by 8 bits in between (Horner's rule).  The excess-8 bias of the codes is
//    removed exactly by adding -8 * sum(digit) at each stage.  Dot products of
//    codes and queries are therefore exact integers.
//  * stage-1 rows are assigned so that output register j of lane group grp holds
//    slot 4j + grp = (page, basis column); those registers are directly the B
//    operand of stage 2 (block-diagonal over the pages of a pass), so the
//    projections never go through LDS.
//  * every load is unconditional (clamped to a valid record) and 32-bit offset.
// ---------------------------------------------------------------------------

template <int R>
struct FastGeom {
  static constexpr int kPPS = 16 / R;                 // pages per stage-1 set
  static constexpr int kSets = R;                     // 16 pages x R slots / 16 rows
  static constexpr int kStride = rec_stride(R);
  static constexpr int kTail = kStride - 64 * R;
  static constexpr int kTailCh = kTail / 16;
  static constexpr int kTailLoads = (16 * kTailCh + 63) / 64;
  static constexpr int kMu = 16 * R;
  static constexpr int kSc = 16 * R + kDim;
};

template <int R>
struct FastRegs {
  uint4 vb[FastGeom<R>::kSets];
  uint4 tl[FastGeom<R>::kTailLoads];
};

template <int R>
__device__ __forceinline__ void fast_issue(FastRegs<R>& T, const uint8_t* __restrict__ summ,
                                           const int32_t* __restrict__ pt_row, int page0, int n_c,
                                           int H_kv, int h, int lane) {
  using Gm = FastGeom<R>;
  const int col = lane & 15, grp = lane >> 4;
  const int qs = 4 * (col & 3) + (col >> 2);  // stage-1 slot of A row `col`
  const int a_pp = qs / R, a_l = qs % R;
  // block of page0 + lane (lanes >= 16 and pages past the end reuse page0's block)
  const int pl = page0 + (lane & 15);
  const int my_blk = pt_row[pl < n_c ? pl : page0];
#pragma unroll
  for (int st = 0; st < Gm::kSets; ++st) {
    const int blk = __shfl(my_blk, st * Gm::kPPS + a_pp, 64);
    const uint32_t off = (uint32_t)(blk * H_kv + h) * (uint32_t)Gm::kStride + 64u * a_l + 16u * grp;
    T.vb[st] = *reinterpret_cast<const uint4*>(summ + off);
  }
#pragma unroll
  for (int u = 0; u < Gm::kTailLoads; ++u) {
    int c = lane + 64 * u;
    c = c < 16 * Gm::kTailCh ? c : 16 * Gm::kTailCh - 1;
    const int page = c / Gm::kTailCh, o = (c % Gm::kTailCh) * 16;
    const int blk = __shfl(my_blk, page, 64);
    const uint32_t off = (uint32_t)(blk * H_kv + h) * (uint32_t)Gm::kStride + 64u * R + o;
    T.tl[u] = *reinterpret_cast<const uint4*>(summ + off);
  }
}

template <typename QT, int R, int NPACK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void scan_fast_kernel(
    int H_q, int H_kv, int max_pages, const QT* __restrict__ q, const uint8_t* __restrict__ summ,
    const int32_t* __restrict__ page_table, const int32_t* __restrict__ seq_lens,
    float* __restrict__ s_hat, SHatLayout lay, float2* __restrict__ partials) {
  using Gm = FastGeom<R>;
  constexpr int G = 16 / NPACK;
  constexpr int kPasses = 16 / NPACK;
  constexpr int kKS = (NPACK * R) / 4 > 0 ? (NPACK * R) / 4 : 1;  // k-steps per pass
  __shared__ __align__(16) uint8_t sTail[4][16][Gm::kTail];
  __shared__ float sA[4][16][16];
  __shared__ float2 sRun[4][16];

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
  const int h = blockIdx.y, s = blockIdx.z;
  const int n_c = seq_lens[s] / kPage;
  const int pg = scan_chunk() * 4 + wave;
  const long row0 = (long)s * H_q + (long)h * G;
  const int32_t* pt_row = page_table + (long)s * max_pages;
  const int gcol = col % G, pcol = col / G;
  constexpr float c0 = 1.4426950408889634f * 0.08838834764831845f;  // log2(e) / sqrt(128)
  float run_m = -INFINITY, run_s = 0.0f;

  if (pg * 64 < n_c) {
    FastRegs<R> cur;
    fast_issue<R>(cur, summ, pt_row, pg * 64, n_c, H_kv, h, lane);

    const QDigits<3> QD = q_digits(q + (row0 + gcol) * kDim, grp);
    const float inv_scale = QD.inv_scale;
    const i4v(&bd)[3][2] = QD.bd;

#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int page0 = (pg * 4 + t) * 16;
      if (page0 < n_c) {
#pragma unroll
        for (int u = 0; u < Gm::kTailLoads; ++u) {
          const int c = lane + 64 * u;
          if (c < 16 * Gm::kTailCh)
            *reinterpret_cast<uint4*>(&sTail[wave][c / Gm::kTailCh][(c % Gm::kTailCh) * 16]) = cur.tl[u];
        }
        __builtin_amdgcn_wave_barrier();

        // ---- stage 1 (int8 MFMA): projections of every (page, basis column) slot
        float vals[4 * Gm::kSets];
#pragma unroll
        for (int st = 0; st < Gm::kSets; ++st) {
          if (st % 4 == 0) __builtin_amdgcn_sched_barrier(0);
          i4v a[2];
          nib_operands(cur.vb[st], a);
          const i4v acc = proj_horner(a, QD);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int slot = 4 * j + grp;
            const int page = st * Gm::kPPS + slot / R, l = slot % R;
            const float vs = lds_f16(&sTail[wave][page][Gm::kSc + 2 * l]);
            vals[4 * st + j] = (float)acc[j] * (vs * inv_scale);
          }
        }
        // the record registers are consumed: fetch the next 16 pages into them while
        // the rest of this step runs from LDS and registers
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < 4 && page0 + 16 < n_c)
          fast_issue<R>(cur, summ, pt_row, page0 + 16, n_c, H_kv, h, lane);
        __builtin_amdgcn_sched_barrier(0);
        // ---- centroid term (int8 MFMA, one page per row): sA[page][col]
        {
          const uint4 m0 = *reinterpret_cast<const uint4*>(&sTail[wave][col][Gm::kMu + 32 * grp]);
          const uint4 m1 = *reinterpret_cast<const uint4*>(&sTail[wave][col][Gm::kMu + 32 * grp + 16]);
          const uint32_t mw[8] = {m0.x ^ 0x80808080u, m0.y ^ 0x80808080u, m0.z ^ 0x80808080u,
                                  m0.w ^ 0x80808080u, m1.x ^ 0x80808080u, m1.y ^ 0x80808080u,
                                  m1.z ^ 0x80808080u, m1.w ^ 0x80808080u};
          i4v acc[3];
#pragma unroll
          for (int d = 0; d < 3; ++d) acc[d] = i4v{0, 0, 0, 0};
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            const uint32_t y0 = mw[4 * hh], y1 = mw[4 * hh + 1], y2 = mw[4 * hh + 2], y3 = mw[4 * hh + 3];
            const i4v a = {(int)__builtin_amdgcn_perm(y1, y0, 0x06040200u),
                           (int)__builtin_amdgcn_perm(y1, y0, 0x07050301u),
                           (int)__builtin_amdgcn_perm(y3, y2, 0x06040200u),
                           (int)__builtin_amdgcn_perm(y3, y2, 0x07050301u)};
#pragma unroll
            for (int d = 0; d < 3; ++d)
              acc[d] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, bd[d][hh], acc[d], 0, 0, 0);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int page = 4 * grp + j;
            const float ms = lds_f16(&sTail[wave][page][Gm::kSc + 2 * (R + 16)]);
            const float v = fmaf((float)acc[0][j], 65536.0f, fmaf((float)acc[1][j], 256.0f, (float)acc[2][j]));
            sA[wave][page][col] = v * (ms * inv_scale);
          }
        }
        __builtin_amdgcn_wave_barrier();

        // ---- stage 2 (fp32 MFMA): 16 logits per (page, head), NPACK pages per pass
#pragma unroll
        for (int ps = 0; ps < kPasses; ++ps) {
          if (ps % 4 == 0) __builtin_amdgcn_sched_barrier(0);
          const int pcpage = ps * NPACK + pcol;  // page of this lane's column
          f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int kk = 0; kk < kKS; ++kk) {
            const int rho = (NPACK * R >= 4) ? ps * kKS + kk : (ps * NPACK * R) / 4;
            const int st = rho / 4, j = rho % 4;
            const int slot = 4 * j + grp;
            const int pk = st * Gm::kPPS + slot / R, l = slot % R;
            const float a = (float)((int)sTail[wave][pk][col * R + l] - 128);
            const float b = (pk == pcpage) ? vals[rho] : 0.0f;
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
          }
          const float av = sA[wave][pcpage][col];
          const uint2 csw = *reinterpret_cast<const uint2*>(&sTail[wave][pcpage][Gm::kSc + 2 * (R + 4 * grp)]);
          const h2 cs01 = as_h2(csw.x), cs23 = as_h2(csw.y);
          float z0 = fmaf((float)cs01.x, acc[0], av), z1 = fmaf((float)cs01.y, acc[1], av);
          float z2 = fmaf((float)cs23.x, acc[2], av), z3 = fmaf((float)cs23.y, acc[3], av);
          float mx = fmaxf(fmaxf(z0, z1), fmaxf(z2, z3));
          mx = red4_max(mx);
          float sm = __builtin_amdgcn_exp2f(z0 - mx) + __builtin_amdgcn_exp2f(z1 - mx) +
                     __builtin_amdgcn_exp2f(z2 - mx) + __builtin_amdgcn_exp2f(z3 - mx);
          sm = red4_sum(sm);
          const float s2 = mx + __builtin_amdgcn_logf(sm);
          const bool live = page0 + pcpage < n_c;
          if (live && grp == 0)
            s_hat[lay.base(s, h) + gcol * lay.head + (long)(page0 + pcpage) * lay.page] = s2 * 0.69314718055994531f;
          const float e = __builtin_amdgcn_exp2f(-fabsf(s2 - run_m));
          const bool up = s2 > run_m;
          const float ns = up ? fmaf(run_s, e, 1.0f) : run_s + e;
          run_s = live ? ns : run_s;
          run_m = (live && up) ? s2 : run_m;
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  // ---- block partial (max, sum exp) per head over its 256 pages, log2 domain
  if (lane < 16) sRun[wave][lane] = make_float2(run_m, run_s);
  __syncthreads();
  if (threadIdx.x < G) {
    const int g = threadIdx.x;
    float m = -INFINITY, l = 0.0f;
    for (int w = 0; w < 4; ++w)
      for (int c = g; c < 16; c += G) m = fmaxf(m, sRun[w][c].x);
    if (m > -INFINITY)
      for (int w = 0; w < 4; ++w)
        for (int c = g; c < 16; c += G) {
          const float2 v = sRun[w][c];
          if (v.y > 0.0f) l += v.y * __builtin_amdgcn_exp2f(v.x - m);
        }
    partials[(row0 + g) * gridDim.x + blockIdx.x] = make_float2(m, l);
  }
}

template <typename QT>
hipError_t dispatch_scan(int r, int G, int basis, dim3 grid, hipStream_t st, int H_q,
                         int H_kv, int max_pages, const QT* q, const uint8_t* sum, const int32_t* pt,
                         const int32_t* sl, float* s_hat, SHatLayout lay, float2* part) {
  if (basis != LOCKS_BASIS_INT4) {  // int8 / bf16 bases: the generic kernel, r in {2, 4, 8}
#define LOCKS_SCAN_BASIS(RR, BB)                                                            \
    if (r == RR && basis == BB) {                                                           \
      hipLaunchKernelGGL((scan_mfma_kernel<QT, RR, BB>), grid, dim3(256), 0, st, H_q, H_kv, \
                         max_pages, q, sum, pt, sl, s_hat, lay, part);                      \
      return hipGetLastError();                                                             \
    }
    LOCKS_SCAN_BASIS(2, 1) LOCKS_SCAN_BASIS(4, 1) LOCKS_SCAN_BASIS(8, 1)
    LOCKS_SCAN_BASIS(2, 2) LOCKS_SCAN_BASIS(4, 2) LOCKS_SCAN_BASIS(8, 2)
#undef LOCKS_SCAN_BASIS
    return hipErrorInvalidValue;
  }
#define LOCKS_SCAN_FAST(RR, NP)                                                              \
  if (r == RR && G == 16 / NP) {                                                            \
    hipLaunchKernelGGL((scan_fast_kernel<QT, RR, NP>), grid, dim3(256), 0, st, H_q, H_kv,   \
                       max_pages, q, sum, pt, sl, s_hat, lay, part);               \
    return hipGetLastError();                                                               \
  }
  // r = 2 and 4 at G = 16 (G = 4 took the low-rank kernel of scan_low.hip)
  LOCKS_SCAN_FAST(4, 1) LOCKS_SCAN_FAST(2, 1)
#undef LOCKS_SCAN_FAST
#define LOCKS_SCAN_MFMA_CASE(RR)                                                             \
  case RR:                                                                                  \
    hipLaunchKernelGGL((scan_mfma_kernel<QT, RR>), grid, dim3(256), 0, st, H_q, H_kv,       \
                       max_pages, q, sum, pt, sl, s_hat, lay, part);               \
    break;
  switch (r) {
    LOCKS_SCAN_MFMA_CASE(1) LOCKS_SCAN_MFMA_CASE(2) LOCKS_SCAN_MFMA_CASE(3)
    LOCKS_SCAN_MFMA_CASE(4) LOCKS_SCAN_MFMA_CASE(5) LOCKS_SCAN_MFMA_CASE(6)
    LOCKS_SCAN_MFMA_CASE(7) LOCKS_SCAN_MFMA_CASE(9) LOCKS_SCAN_MFMA_CASE(10)
    LOCKS_SCAN_MFMA_CASE(11) LOCKS_SCAN_MFMA_CASE(12) LOCKS_SCAN_MFMA_CASE(13)
    LOCKS_SCAN_MFMA_CASE(14) LOCKS_SCAN_MFMA_CASE(15)
    default:
      return hipErrorInvalidValue;
  }
#undef LOCKS_SCAN_MFMA_CASE
  return hipGetLastError();
}

}  // namespace

hipError_t launch_scan_mfma(const ScanArgs& a, int rank, int basis, hipStream_t st) {
  const int G = a.H_q / a.H_kv;
  if (a.q_bf16)
    return dispatch_scan(rank, G, basis, a.grid, st, a.H_q, a.H_kv, a.max_pages,
                         static_cast<const uint16_t*>(a.q), a.summ, a.page_table, a.seq_lens,
                         a.s_hat, a.lay, a.partials);
  return dispatch_scan(rank, G, basis, a.grid, st, a.H_q, a.H_kv, a.max_pages,
                       static_cast<const float*>(a.q), a.summ, a.page_table, a.seq_lens, a.s_hat,
                       a.lay, a.partials);
}

}  // namespace locks
