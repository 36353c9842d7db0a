// Summary scan of 32- and 64-token pages at the ranks the quad scan does not cover.
#include "locks_internal.h"
#include "scan_common.h"
#include "scan_launch.h"

namespace locks {
namespace {

// ---------------------------------------------------------------------------
// Pages of B = 32 or 64 tokens (App. D.3 "Page size"), int4 basis.  The generic
// kernel's two stages with tiles of 8 pages: stage 1 (f16 MFMA, rows (page, basis
// column), columns the query heads) and the centroid projection are unchanged,
// the record tail holds B coefficient rows, and stage 2 runs one page at a time on
// fp32 MFMA 16x16x4 with the B tokens as rows (B / 16 row tiles) and the heads as
// columns; each lane then holds 4 B / 16 logits of one head and the page LSE
// takes its max and sum over them and the three other lanes of the head.
// ---------------------------------------------------------------------------
template <int R, int B>
struct PageGeom {
  static constexpr int kTP = 8;                                   // pages per tile
  static constexpr int kPPS = (16 / R) > 0 ? 16 / R : 1;          // pages per stage-1 set
  static constexpr int kSets = (kTP + kPPS - 1) / kPPS;
  static constexpr int kStride = rec_stride(R, 0, B);
  static constexpr int kTail = kStride - 64 * R;                  // coef .. end of record
  static constexpr int kTailCh = kTail / 16;
  static constexpr int kTailLoads = (kTP * kTailCh + 63) / 64;
  static constexpr int kMu = B * R;                               // offsets inside the tail
  static constexpr int kSc = B * R + kDim;
  static constexpr int kTiles = 64 / kTP;                         // tiles per wave (64 pages)
};

template <int R, int B>
struct PageRegs {
  uint4 vb[PageGeom<R, B>::kSets];
  uint4 tl[PageGeom<R, B>::kTailLoads];
};

// wave_blk: lane l holds the block of the wave's page l (-1 past the sequence's
// complete pages), read once per wave; tile t covers the wave's pages
// t kTP .. t kTP + kTP - 1.
template <int R, int B>
__device__ __forceinline__ void issue_page_tile(PageRegs<R, B>& T, const uint8_t* __restrict__ summ,
                                                int wave_blk, int t, int H_kv, int h, int lane) {
  using Gm = PageGeom<R, B>;
  const int col = lane & 15, grp = lane >> 4;
  const int pp = col / R, l = col % R;
#pragma unroll
  for (int st = 0; st < Gm::kSets; ++st) {
    const int page = st * Gm::kPPS + pp;
    const int blk = __shfl(wave_blk, (t * Gm::kTP + (page < Gm::kTP ? page : 0)) & 63, 64);
    const bool ok = col < Gm::kPPS * R && page < Gm::kTP && blk >= 0;
    T.vb[st] = ok ? *reinterpret_cast<const uint4*>(summ + ((long)blk * H_kv + h) * Gm::kStride +
                                                    64 * l + 16 * grp)
                  : make_uint4(0, 0, 0, 0);
  }
#pragma unroll
  for (int u = 0; u < Gm::kTailLoads; ++u) {
    const int c = lane + 64 * u;
    const int page = c / Gm::kTailCh, off = (c % Gm::kTailCh) * 16;
    const int blk = __shfl(wave_blk, (t * Gm::kTP + (page < Gm::kTP ? page : 0)) & 63, 64);
    T.tl[u] = (c < Gm::kTP * Gm::kTailCh && blk >= 0)
                  ? *reinterpret_cast<const uint4*>(summ + ((long)blk * H_kv + h) * Gm::kStride +
                                                    64 * R + off)
                  : make_uint4(0, 0, 0, 0);
  }
}

// NPG: pages per stage-2 pass (16 / G when the group size G divides 16 and is
// below 16: the 16 MFMA columns then hold (page, head) pairs, the K axis runs over
// (page, basis column) and each page's coefficients meet only its own
// projections; 1: the heads are the columns, any G <= 16).
template <typename QT, int R, int B, int NPG = 1>
__global__ __launch_bounds__(256) void scan_page_kernel(
    int H_q, int H_kv, int max_pages, const QT* __restrict__ q,
    const uint8_t* __restrict__ summaries, const int32_t* __restrict__ page_table,
    const int32_t* __restrict__ seq_lens, float* __restrict__ s_hat, SHatLayout lay,
    float2* __restrict__ partials, int wave_pages) {
  using Gm = PageGeom<R, B>;
  constexpr bool kSplitQ = sizeof(QT) == 4;  // fp32 queries: f16 hi + lo
  constexpr int kKS = (R + 3) / 4;           // stage-2 k-steps
  constexpr int kRT = B / 16;                // stage-2 row tiles
  __shared__ __align__(16) uint8_t sTail[4][Gm::kTP][Gm::kTail];
  __shared__ float sP[4][Gm::kTP][R][16];
  __shared__ float sA[4][Gm::kTP][16];
  __shared__ float2 sRun[4][16];

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
  const int h = blockIdx.y, s = blockIdx.z;
  const int G = H_q / H_kv;
  const int n_c = seq_lens[s] / B;
  // pages wave_pages (16, 32 or 64) from `base` are this wave's
  const int base = (scan_chunk() * 4 + wave) * wave_pages;
  const long row0 = (long)s * H_q + (long)h * G;
  const int32_t* pt_row = page_table + (long)s * max_pages;
  float run_m = -INFINITY, run_s = 0.0f;  // running normaliser of head col, log2 domain
  if (base < n_c) {
    const int wave_blk = lane < wave_pages && base + lane < n_c ? pt_row[base + lane] : -1;
    PageRegs<R, B> buf[2];
    issue_page_tile<R, B>(buf[0], summaries, wave_blk, 0, H_kv, h, lane);

    // ---- B operands: column = query head, K permuted to match the decoders
    constexpr int kPerm[8] = {0, 4, 1, 5, 2, 6, 3, 7};
    float qv[4][8], qm[4][8];
    float qmax = 0.0f;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int jj = 0; jj < 8; ++jj) {
        const int cv = 32 * grp + 8 * ks + kPerm[jj], cm = 32 * grp + 8 * ks + jj;
        const float a = col < G ? load_q(q, (row0 + col) * kDim + cv) : 0.0f;
        const float b = col < G ? load_q(q, (row0 + col) * kDim + cm) : 0.0f;
        qv[ks][jj] = a;
        qm[ks][jj] = b;
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
      for (int jj = 0; jj < 8; ++jj) {
        const float a = qv[ks][jj] * qs, b = qm[ks][jj] * qs;
        const _Float16 ah = (_Float16)a, bh = (_Float16)b;
        bv[ks][jj] = ah;
        bm[ks][jj] = bh;
        bvl[ks][jj] = (_Float16)(a - (float)ah);
        bml[ks][jj] = (_Float16)(b - (float)bh);
      }

    constexpr float kLn2 = 0.69314718055994531f;
    const float c0 = 1.4426950408889634f * 0.08838834764831845f;  // log2(e) / sqrt(128)

    // (unrolled, so the two tile buffers are named registers, not private memory)
#pragma unroll
    for (int t = 0; t < Gm::kTiles; ++t) {
      const int page0 = base + t * Gm::kTP;
      if (t * Gm::kTP >= wave_pages || page0 >= n_c) break;
      PageRegs<R, B>& cur = buf[t & 1];
      if (t + 1 < Gm::kTiles && (t + 1) * Gm::kTP < wave_pages && page0 + Gm::kTP < n_c)
        issue_page_tile<R, B>(buf[(t + 1) & 1], summaries, wave_blk, t + 1, H_kv, h, lane);
#pragma unroll
      for (int u = 0; u < Gm::kTailLoads; ++u) {
        const int c = lane + 64 * u;
        if (c < Gm::kTP * Gm::kTailCh)
          *reinterpret_cast<uint4*>(&sTail[wave][c / Gm::kTailCh][(c % Gm::kTailCh) * 16]) =
              cur.tl[u];
      }
      __builtin_amdgcn_wave_barrier();

      // ---- stage 1: p = V^T q (scaled by the basis column scales)
#pragma unroll
      for (int st = 0; st < Gm::kSets; ++st) {
        f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        const uint32_t w[4] = {cur.vb[st].x, cur.vb[st].y, cur.vb[st].z, cur.vb[st].w};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const h8 a = nib8_to_h8(w[ks]);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, bv[ks], acc, 0, 0, 0);
          if (kSplitQ) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, bvl[ks], acc, 0, 0, 0);
        }
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int m = 4 * grp + jj;
          const int pp = m / R, l = m % R;
          const int page = st * Gm::kPPS + pp;
          if (m < Gm::kPPS * R && page < Gm::kTP && col < G)
            sP[wave][page][l][col] = acc[jj] * inv_qs * lds_f16(&sTail[wave][page][Gm::kSc + 2 * l]);
        }
      }
      // ---- centroid term a = mu^T q, one page per row
      {
        const int cp = col < Gm::kTP ? col : 0;
        const uint4 m0 = *reinterpret_cast<const uint4*>(&sTail[wave][cp][Gm::kMu + 32 * grp]);
        const uint4 m1 = *reinterpret_cast<const uint4*>(&sTail[wave][cp][Gm::kMu + 32 * grp + 16]);
        const uint32_t w[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
        f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const h8 a = byte8_to_h8(w[2 * ks], w[2 * ks + 1]);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, bm[ks], acc, 0, 0, 0);
          if (kSplitQ) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, bml[ks], acc, 0, 0, 0);
        }
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int page = 4 * grp + jj;
          if (page < Gm::kTP && col < G)
            sA[wave][page][col] =
                acc[jj] * inv_qs * c0 * lds_f16(&sTail[wave][page][Gm::kSc + 2 * (R + B)]);
        }
      }
      __builtin_amdgcn_wave_barrier();

      if constexpr (NPG == 1) {
        // ---- stage 2, one page at a time: z[token][head] over B / 16 row tiles
        for (int p = 0; p < Gm::kTP; ++p) {
          if (page0 + p >= n_c) break;
          float z[kRT][4];
  #pragma unroll
          for (int rt = 0; rt < kRT; ++rt) {
            f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  #pragma unroll
            for (int kstep = 0; kstep < kKS; ++kstep) {
              const int l = 4 * kstep + grp;
              const int tok = 16 * rt + col;
              const float a = l < R ? (float)((int)sTail[wave][p][tok * R + l] - 128) : 0.0f;
              const float b = (l < R && col < G) ? sP[wave][p][l < R ? l : 0][col] : 0.0f;
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
            }
            const uint2 csw = *reinterpret_cast<const uint2*>(
                &sTail[wave][p][Gm::kSc + 2 * (R + 16 * rt + 4 * grp)]);
            const h2 cs01 = as_h2(csw.x), cs23 = as_h2(csw.y);
            const float av = sA[wave][p][col];
            z[rt][0] = fmaf((float)cs01.x * c0, acc[0], av);
            z[rt][1] = fmaf((float)cs01.y * c0, acc[1], av);
            z[rt][2] = fmaf((float)cs23.x * c0, acc[2], av);
            z[rt][3] = fmaf((float)cs23.y * c0, acc[3], av);
          }
          float mx = -INFINITY;
  #pragma unroll
          for (int rt = 0; rt < kRT; ++rt)
            mx = fmaxf(mx, fmaxf(fmaxf(z[rt][0], z[rt][1]), fmaxf(z[rt][2], z[rt][3])));
          mx = red4_max(mx);
          float sm = 0.0f;
  #pragma unroll
          for (int rt = 0; rt < kRT; ++rt)
  #pragma unroll
            for (int jj = 0; jj < 4; ++jj) sm += __builtin_amdgcn_exp2f(z[rt][jj] - mx);
          sm = red4_sum(sm);
          const float s2 = mx + __builtin_amdgcn_logf(sm);  // log2-domain page score
          if (col < G) {
            if (grp == 0)
              s_hat[lay.base(s, h) + col * lay.head + (long)(page0 + p) * lay.page] = s2 * kLn2;
            const float e = __builtin_amdgcn_exp2f(-fabsf(s2 - run_m));
            if (s2 > run_m) { run_s = fmaf(run_s, e, 1.0f); run_m = s2; }
            else run_s += e;
          }
        }
      } else {
        // ---- stage 2, NPG pages at a time: z[token][(page pc, head gc)]
        constexpr int kG = 16 / NPG;
        const int pc = col / kG, gc = col % kG;
#pragma unroll
        for (int p0 = 0; p0 < Gm::kTP; p0 += NPG) {
          if (page0 + p0 >= n_c) break;
          float z[kRT][4];
#pragma unroll
          for (int rt = 0; rt < kRT; ++rt) {
            f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
            const int tok = 16 * rt + col;
#pragma unroll
            for (int pp = 0; pp < NPG; ++pp)
#pragma unroll
              for (int kstep = 0; kstep < kKS; ++kstep) {
                const int l = 4 * kstep + grp;
                const int la = l < R ? l : 0;
                const float a = l < R ? (float)((int)sTail[wave][p0 + pp][tok * R + la] - 128) : 0.0f;
                const float b = (l < R && pc == pp) ? sP[wave][p0 + pp][la][gc] : 0.0f;
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
              }
            const uint2 csw = *reinterpret_cast<const uint2*>(
                &sTail[wave][p0 + pc][Gm::kSc + 2 * (R + 16 * rt + 4 * grp)]);
            const h2 cs01 = as_h2(csw.x), cs23 = as_h2(csw.y);
            const float av = sA[wave][p0 + pc][gc];
            z[rt][0] = fmaf((float)cs01.x * c0, acc[0], av);
            z[rt][1] = fmaf((float)cs01.y * c0, acc[1], av);
            z[rt][2] = fmaf((float)cs23.x * c0, acc[2], av);
            z[rt][3] = fmaf((float)cs23.y * c0, acc[3], av);
          }
          float mx = -INFINITY;
#pragma unroll
          for (int rt = 0; rt < kRT; ++rt)
            mx = fmaxf(mx, fmaxf(fmaxf(z[rt][0], z[rt][1]), fmaxf(z[rt][2], z[rt][3])));
          mx = red4_max(mx);
          float sm = 0.0f;
#pragma unroll
          for (int rt = 0; rt < kRT; ++rt)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) sm += __builtin_amdgcn_exp2f(z[rt][jj] - mx);
          sm = red4_sum(sm);
          const float s2 = mx + __builtin_amdgcn_logf(sm);  // log2-domain page score
          if (page0 + p0 + pc < n_c) {
            if (grp == 0)
              s_hat[lay.base(s, h) + gc * lay.head + (long)(page0 + p0 + pc) * lay.page] = s2 * kLn2;
            const float e = __builtin_amdgcn_exp2f(-fabsf(s2 - run_m));
            if (s2 > run_m) { run_s = fmaf(run_s, e, 1.0f); run_m = s2; }
            else run_s += e;
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
  // ---- block partial (max, sum exp) per head over its pages (log2 domain):
  //      head g's running pairs sit in the columns p G + g, p < NPG, of every wave
  if (lane < 16) sRun[wave][lane] = make_float2(run_m, run_s);
  __syncthreads();
  if (threadIdx.x < G) {
    const int g = threadIdx.x;
    float m = -INFINITY, l = 0.0f;
    for (int w = 0; w < 4; ++w)
      for (int p = 0; p < NPG; ++p) m = fmaxf(m, sRun[w][p * G + g].x);
    if (m > -INFINITY)
      for (int w = 0; w < 4; ++w)
        for (int p = 0; p < NPG; ++p) {
          const float2 v = sRun[w][p * G + g];
          if (v.y > 0.0f) l += v.y * __builtin_amdgcn_exp2f(v.x - m);
        }
    partials[(row0 + g) * gridDim.x + blockIdx.x] = make_float2(m, l);
  }
}

template <typename QT>
hipError_t dispatch_scan_page(int r, int B, int wp, dim3 grid, hipStream_t st, int H_q, int H_kv,
                              int max_pages, const QT* q, const uint8_t* sum, const int32_t* pt,
                              const int32_t* sl, float* s_hat, SHatLayout lay, float2* part) {
#define LOCKS_SCAN_PAGE_CASE(RR)                                                              \
  case RR:                                                                                   \
    if (B == 32)                                                                             \
      hipLaunchKernelGGL((scan_page_kernel<QT, RR, 32>), grid, dim3(256), 0, st, H_q, H_kv,  \
                         max_pages, q, sum, pt, sl, s_hat, lay, part, wp);                   \
    else                                                                                     \
      hipLaunchKernelGGL((scan_page_kernel<QT, RR, 64>), grid, dim3(256), 0, st, H_q, H_kv,  \
                         max_pages, q, sum, pt, sl, s_hat, lay, part, wp);                   \
    break;
  if (B != 32 && B != 64) return hipErrorInvalidValue;
  // four-head groups at the common ranks: four pages per stage-2 pass
  if (H_q == 4 * H_kv && (r == 2 || r == 4)) {
#define LOCKS_SCAN_PAGE4(RR)                                                                  \
    if (r == RR) {                                                                           \
      if (B == 32)                                                                           \
        hipLaunchKernelGGL((scan_page_kernel<QT, RR, 32, 4>), grid, dim3(256), 0, st, H_q,   \
                           H_kv, max_pages, q, sum, pt, sl, s_hat, lay, part, wp);           \
      else                                                                                   \
        hipLaunchKernelGGL((scan_page_kernel<QT, RR, 64, 4>), grid, dim3(256), 0, st, H_q,   \
                           H_kv, max_pages, q, sum, pt, sl, s_hat, lay, part, wp);           \
      return hipGetLastError();                                                              \
    }
    LOCKS_SCAN_PAGE4(2) LOCKS_SCAN_PAGE4(4)
#undef LOCKS_SCAN_PAGE4
  }
  switch (r) {
    LOCKS_SCAN_PAGE_CASE(1) LOCKS_SCAN_PAGE_CASE(2) LOCKS_SCAN_PAGE_CASE(3)
    LOCKS_SCAN_PAGE_CASE(4) LOCKS_SCAN_PAGE_CASE(5) LOCKS_SCAN_PAGE_CASE(6)
    LOCKS_SCAN_PAGE_CASE(7) LOCKS_SCAN_PAGE_CASE(9) LOCKS_SCAN_PAGE_CASE(10)
    LOCKS_SCAN_PAGE_CASE(11) LOCKS_SCAN_PAGE_CASE(12) LOCKS_SCAN_PAGE_CASE(13)
    LOCKS_SCAN_PAGE_CASE(14) LOCKS_SCAN_PAGE_CASE(15)
    default:
      return hipErrorInvalidValue;
  }
#undef LOCKS_SCAN_PAGE_CASE
  return hipGetLastError();
}

}  // namespace

hipError_t launch_scan_page(const ScanArgs& a, int rank, int page_size, int wave_pages,
                            hipStream_t st) {
  if (a.q_bf16)
    return dispatch_scan_page(rank, page_size, wave_pages, a.grid, st, a.H_q, a.H_kv, a.max_pages,
                              static_cast<const uint16_t*>(a.q), a.summ, a.page_table, a.seq_lens,
                              a.s_hat, a.lay, a.partials);
  return dispatch_scan_page(rank, page_size, wave_pages, a.grid, st, a.H_q, a.H_kv, a.max_pages,
                            static_cast<const float*>(a.q), a.summ, a.page_table, a.seq_lens,
                            a.s_hat, a.lay, a.partials);
}

}  // namespace locks
