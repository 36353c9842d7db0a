// Rank-8 summary scan (int4 basis) of groups of 9 to 16 heads, every page size: 16
// (sub-)pages per wave step, no LDS in the step, columns = the 16 heads (heads past G
// repeat head 0 and are never stored).
//
//  * Stage 1 (int8 MFMA, Horner over the query digits): basis set i of a pair of sets
//    has rows (page 2 i + m / 8, basis column m % 8), so lane (grp, col) receives
//    p(page 2 i + grp / 2, l = 4 (grp % 2) + j, head col) in register j.
//  * The values are split into f16 hi + lo; one 32-lane swap of hi with lo gives the
//    B operand of a 16x16x16 f16 MFMA for each of the two pages: K rows 0..7 hold hi of
//    l = 0..7, rows 8..15 lo.  Its A operand is the token's coefficient row twice, a
//    4-byte load whose record offset is wave-uniform.  So stage 2 takes one MFMA per
//    16 tokens with no zeros in it.  (With four query digits, ND of scan_digits: three
//    bfloat16 terms, the third in an MFMA of its own.)
//  * Register j of lane (grp, col) is the logit of token 4 grp + j for head col, minus
//    the centroid logit.  The sums of 2^z over a lane's 4 tokens are reduced over grp
//    four (sub-)pages at a time, the totals handed to the four lane rows (reduce4): row
//    grp finishes (sub-)page 4 u + grp.
//  * Row scales and centroid scales are loaded once per step, one (sub-)page per lane of
//    a row, and broadcast along the row as operands of their use.
// The centroid MFMA (once per step) has rows page 4 (m % 4) + m / 4, which leaves
// a(page 4 j + grp, head col) in register j.
//
// Pages of 16 V tokens (V = 2, 4) run as V sub-pages of 16 tokens: a page's B operand
// serves its V sub-pages, whose LSEs (lanes l ^ 16, l ^ 32) are merged at the end.
//
// Bound: the vector ALU and the latency of each step at two waves per SIMD (1M tokens,
// two KV heads: one round of 2,048 waves, 251 registers; with four query digits 256 and one
// spilled).  30.4 us there; with stage 2 as a
// block-diagonal 16x16x32 MFMA pair per 16 tokens (hi, lo) and per-quad row masks the
// same layout took 31.6.
#pragma once

#include "locks_internal.h"
#include "scan_common.h"
#include "scan_launch.h"

namespace locks {
namespace {

typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef short s4 __attribute__((ext_vector_type(4)));

template <typename QT, int ND, int kSteps, int V>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void scan_wide_kernel(
    int H_q, int H_kv, int G, int max_pages, const QT* __restrict__ q,
    const uint8_t* __restrict__ summ, uint32_t summ_bytes, const int32_t* __restrict__ page_table,
    const int32_t* __restrict__ seq_lens, float* __restrict__ s_hat, SHatLayout lay,
    float2* __restrict__ partials) {
  constexpr int R = 8, P = kPage * V;
  constexpr int kPages = 16 / V;   // pages per step
  constexpr int kPairs = 4 / V;    // pairs of basis sets (4 pages each) per step
  constexpr uint32_t kStride = rec_stride(R, 0, P);
  constexpr uint32_t kCoef = rec_coef_off(R), kMu = rec_mu_off(R, 0, P), kSc = rec_scale_off(R, 0, P);
  __shared__ float2 sRun[4][16];
  __shared__ DigitLds<16, ND> sDig;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
  const int h = blockIdx.y, s = blockIdx.z;
  const int n_c = seq_lens[s] / P * V;  // sub-pages of the complete pages
  const int pg = scan_chunk() * 4 + wave;
  const long row0 = (long)s * H_q + (long)h * G;
  const int32_t* pt_row = page_table + (long)s * max_pages;
  float run_m = -INFINITY, run_s = 0.0f;

  constexpr int kWavePages = 16 * kSteps;
  const int first = pg * kWavePages;
  if (scan_chunk() * 4 * kWavePages >= n_c) {  // no complete page in this block
    if (threadIdx.x < G)
      partials[(row0 + threadIdx.x) * gridDim.x + blockIdx.x] = make_float2(-INFINITY, 0.0f);
    return;
  }
  const bool has = first < n_c;  // pages for this wave
  {
    const int n_steps = has ? min(kSteps, (n_c - first + 15) / 16) : 0;
    QDigits<ND> QD;  // read from the block's once formed
    float* shat_lane = s_hat + lay.base(s, h) + (long)col * lay.head;

    // record offsets of one step: va[m][i] page 4 m + 2 i + col / 8 (stage-1 rows),
    // vsc[m][i] page 4 m + 2 i + grp / 2, own the lane's sub-page col, rm the centroid
    // row's page, ro (sub-)page 4 (col % 4) + grp; pa[p] page p (wave-uniform)
    struct Offs {
      uint32_t va[kPairs][2], vsc[kPairs][2], own, rm, ro, pa[kPages];
    };
    const __amdgpu_buffer_rsrc_t rs = summ_rsrc(summ, summ_bytes);
    const uint32_t blk_bytes = (uint32_t)H_kv * kStride, head_off = (uint32_t)h * kStride;
    auto offsets = [&](int blk) {
      Offs o;
      const int off = (int)rec_off(blk, blk_bytes, head_off);  // of sub-page lane % 16
      auto rec = [&](int sp) { return (uint32_t)__shfl(off, sp, 64); };
#pragma unroll
      for (int m = 0; m < kPairs; ++m)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          o.va[m][i] = rec((4 * m + 2 * i + (col >> 3)) * V);
          o.vsc[m][i] = rec((4 * m + 2 * i + (grp >> 1)) * V);
        }
      o.own = (uint32_t)off;
      o.rm = rec(4 * (col & 3) + (col >> 2));
      o.ro = rec(4 * (col & 3) + grp);
#pragma unroll
      for (int p = 0; p < kPages; ++p) o.pa[p] = (uint32_t)__builtin_amdgcn_readlane(off, p * V);
      return o;
    };
    uint4 vb[kPairs][2];   // basis rows of pair m, set i
    uint2 vs[kPairs][2];   // basis column scales 4 (grp % 2) .. + 3 of the lane's page of the set
    uint32_t cf[16];       // coefficients 4 (grp % 2) .. + 3 of token col of each (sub-)page
    uint2 cs;              // row scales of tokens 4 grp .. 4 grp + 3 of sub-page col
    uint32_t msw;          // centroid scale of (sub-)page 4 (col % 4) + grp (low half)
    uint4 mu[2];           // centroid bytes 32 grp .. 32 grp + 31 of the lane's centroid row
    auto ld_vb = [&](const Offs& o, int m, int i) {
      vb[m][i] = bld16(rs, o.va[m][i] + 64u * (col & 7) + 16u * grp);
    };
    auto ld_vs = [&](const Offs& o, int m, int i) { vs[m][i] = bld8(rs, o.vsc[m][i] + kSc + 8u * (grp & 1)); };
    const uint32_t cf_lane = kCoef + 8u * col + 4u * (grp & 1);
    auto ld_cf = [&](const Offs& o, int sp) { cf[sp] = bld4(rs, cf_lane, o.pa[sp / V] + 128u * (sp % V)); };
    auto ld_cs = [&](const Offs& o) { cs = bld8(rs, o.own + kSc + 2u * (R + 16u * (col % V) + 4 * grp)); };
    auto ld_ms = [&](const Offs& o) { msw = bld4(rs, o.ro + kSc + 2u * (R + P)); };
    auto ld_mu = [&](const Offs& o) {
      mu[0] = bld16(rs, o.rm + kMu + 32u * grp);
      mu[1] = bld16(rs, o.rm + kMu + 32u * grp + 16u);
    };

    // every register of the step whose (sub-)pages' blocks lanes 0..15 hold in blk
    auto load_step = [&](int blk) {
      const Offs o0 = offsets(blk);
      ld_mu(o0);
      ld_cs(o0);
      ld_ms(o0);
#pragma unroll
      for (int m = 0; m < kPairs; ++m) {
        ld_vb(o0, m, 0);
        ld_vb(o0, m, 1);
        ld_vs(o0, m, 0);
        ld_vs(o0, m, 1);
#pragma unroll
        for (int e = 0; e < 4 * V; ++e) ld_cf(o0, 4 * V * m + e);
      }
    };

    // kN consecutive 16-page steps from page `start` whose first step's registers are
    // loaded (blk_next: blocks of the second step's pages), fully unrolled so that
    // every wait for a prefetched register counts exactly the loads issued after it.
    auto run = [&](int start, auto n_tag, int blk_next) {
      constexpr int kN = decltype(n_tag)::value;
#pragma unroll
      for (int t_step = 0; t_step < kN; ++t_step) {
        const bool pf = t_step + 1 < kN;
        const int page0 = start + 16 * t_step;
        Offs on;
        int blk_after = 0;
        if (pf) {
          on = offsets(blk_next);
          if (t_step + 2 < kN) blk_after = lane_block_clamped<V>(pt_row, page0 + 32, n_c, lane);
        }

        // ---- centroid term: am[u] = a((sub-)page 4 u + grp, head col) before its scale
        float am[4];
        {
          const uint32_t mw[8] = {mu[0].x ^ 0x80808080u, mu[0].y ^ 0x80808080u,
                                  mu[0].z ^ 0x80808080u, mu[0].w ^ 0x80808080u,
                                  mu[1].x ^ 0x80808080u, mu[1].y ^ 0x80808080u,
                                  mu[1].z ^ 0x80808080u, mu[1].w ^ 0x80808080u};
          if (pf) ld_mu(on);
          i4v acc[ND];
#pragma unroll
          for (int d = 0; d < ND; ++d) acc[d] = i4v{0, 0, 0, 0};
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            const uint32_t y0 = mw[4 * hh], y1 = mw[4 * hh + 1], y2 = mw[4 * hh + 2], y3 = mw[4 * hh + 3];
            const i4v a = {(int)__builtin_amdgcn_perm(y1, y0, 0x06040200u),
                           (int)__builtin_amdgcn_perm(y1, y0, 0x07050301u),
                           (int)__builtin_amdgcn_perm(y3, y2, 0x06040200u),
                           (int)__builtin_amdgcn_perm(y3, y2, 0x07050301u)};
#pragma unroll
            for (int d = 0; d < ND; ++d)
              acc[d] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, QD.bd[d][hh], acc[d], 0, 0, 0);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            int da[ND];
#pragma unroll
            for (int d = 0; d < ND; ++d) da[d] = acc[d][j];
            am[j] = join_digits(da);
          }
        }
        // the step's row scales in fp32 and centroid scales x the query scale's unit,
        // in the lanes that loaded them
        const h2 c01 = as_h2(cs.x), c23 = as_h2(cs.y);
        const float csf[4] = {(float)c01.x, (float)c01.y, (float)c23.x, (float)c23.y};
        const float msf = (float)as_h2(msw).x;
        if (pf) {
          ld_cs(on);
          ld_ms(on);
        }

        // page LSE, store and running normaliser of (sub-)pages 4 u .. 4 u + 3 (l2: log2 of
        // the sum of (sub-)page 4 u + grp)
        auto finish = [&](auto u_tag, float l2) {
          constexpr int u = decltype(u_tag)::value;
          const int own = 4 * u + grp;
          float s2 = am[u] * (row_bcast<u>(msf) * QD.inv_scale) + l2;
          const int page = page0 + own;
          const bool live = page < n_c && own % V == 0;
          if (live && col < G) shat_lane[(long)(page / V) * lay.page] = s2 * 0.69314718055994531f;
          const float e = __builtin_amdgcn_exp2f(-fabsf(s2 - run_m));
          const bool up = s2 > run_m;
          const float ns = up ? fmaf(run_s, e, 1.0f) : run_s + e;
          run_s = live ? ns : run_s;
          run_m = (live && up) ? s2 : run_m;
        };
        static_for_int<kPairs>([&](auto m_tag) __attribute__((always_inline)) {
          constexpr int m = decltype(m_tag)::value;
          __builtin_amdgcn_sched_barrier(0);
          float p[2][4];
          {
            i4v a0[2], a1[2];
            nib_operands(vb[m][0], a0);
            nib_operands(vb[m][1], a1);
            project2(a0, a1, QD, p);
            if (pf) {
              ld_vb(on, m, 0);
              ld_vb(on, m, 1);
            }
          }
          // B operands of the pair's four pages: K rows 0..7 the first term, 8..15 the
          // second; with a third term, another operand of it and zeros
          constexpr int kOps = ND == 3 ? 1 : 2;
          uint2 bp[4][kOps];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const h2 s01 = as_h2(vs[m][i].x), s23 = as_h2(vs[m][i].y);
            const float sc[4] = {(float)s01.x, (float)s01.y, (float)s23.x, (float)s23.y};
            if (pf) ld_vs(on, m, i);
            uint32_t bt[2][2 * kOps];  // [pair of columns][term]
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const float x = p[i][2 * e] * (sc[2 * e] * QD.inv_scale);
              const float y = p[i][2 * e + 1] * (sc[2 * e + 1] * QD.inv_scale);
              if constexpr (ND == 3) {
                const auto hp = __builtin_amdgcn_cvt_pkrtz(x, y);
                const auto lp = __builtin_amdgcn_cvt_pkrtz(x - (float)hp[0], y - (float)hp[1]);
                bt[e][0] = __builtin_bit_cast(uint32_t, hp);
                bt[e][1] = __builtin_bit_cast(uint32_t, lp);
              } else {
                uint32_t t3[3];
                split3_b2(x, y, t3);
                bt[e][0] = t3[0];
                bt[e][1] = t3[1];
                bt[e][2] = t3[2];
                bt[e][3] = 0u;
              }
            }
#pragma unroll
            for (int o = 0; o < kOps; ++o) {
              const auto w0 = __builtin_amdgcn_permlane32_swap(bt[0][2 * o], bt[0][2 * o + 1], false, false);
              const auto w1 = __builtin_amdgcn_permlane32_swap(bt[1][2 * o], bt[1][2 * o + 1], false, false);
              bp[2 * i][o] = make_uint2(w0[0], w1[0]);
              bp[2 * i + 1][o] = make_uint2(w0[1], w1[1]);
            }
          }
          // V quads of (sub-)pages: quad Qv covers sub-pages 4 Qv .. of the pair
          static_for_int<V>([&](auto v_tag) __attribute__((always_inline)) {
            constexpr int Qv = decltype(v_tag)::value, u = V * m + Qv;
            float ps[4], z[4][4];
            static_for_int<4>([&](auto t_tag) __attribute__((always_inline)) {
              constexpr int t = decltype(t_tag)::value, sp = 4 * u + t;
              const uint32_t w = cf[sp];
              if (pf) ld_cf(on, sp);
              f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
              const auto& B = bp[(4 * Qv + t) / V];
              if constexpr (ND == 3) {
                const h2 k{(_Float16)1152.0f, (_Float16)1152.0f};
                const h2 a01 = as_h2(__builtin_amdgcn_perm(0x64646464u, w, 0x04010400u)) - k;
                const h2 a23 = as_h2(__builtin_amdgcn_perm(0x64646464u, w, 0x04030402u)) - k;
                const h4 A{a01.x, a01.y, a23.x, a23.y};
                acc = __builtin_amdgcn_mfma_f32_16x16x16f16(A, __builtin_bit_cast(h4, B[0]), acc, 0, 0, 0);
              } else {
                const s4 A = __builtin_bit_cast(s4, byte4_to_b4(w));
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(A, __builtin_bit_cast(s4, B[kOps - 1]), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(A, __builtin_bit_cast(s4, B[0]), acc, 0, 0, 0);
              }
#pragma unroll
              for (int j = 0; j < 4; ++j) z[t][j] = row_bcast<sp>(csf[j]) * acc[j];
              ps[t] = (__builtin_amdgcn_exp2f(z[t][0]) + __builtin_amdgcn_exp2f(z[t][1])) +
                      (__builtin_amdgcn_exp2f(z[t][2]) + __builtin_amdgcn_exp2f(z[t][3]));
            });
            const float sm = reduce4(ps[0], ps[1], ps[2], ps[3]);
            float tot = sm;  // of the page: the sums of its sub-pages added
            if constexpr (V == 4) tot = swap32_sum(tot);
            if constexpr (V > 1) tot = swap16_sum(tot);
            float l2 = __builtin_amdgcn_logf(tot);
            // tokens spread too widely: taken again from the logits in registers (1M, two KV
            // heads, every page so: 29 us, and 54 where the wave's pages were scanned a second
            // time; pages of ordinary spread 25.5)
            if (__builtin_expect(__any(!(sm >= kSumMin && sm <= kSumMax)), 0)) {
              float ph[4];
#pragma unroll
              for (int t = 0; t < 4; ++t)
                ph[t] = (__builtin_amdgcn_exp2f(z[t][0] - kHighShift) + __builtin_amdgcn_exp2f(z[t][1] - kHighShift)) +
                        (__builtin_amdgcn_exp2f(z[t][2] - kHighShift) + __builtin_amdgcn_exp2f(z[t][3] - kHighShift));
              const float sh = reduce4(ph[0], ph[1], ph[2], ph[3]);
              l2 = __builtin_amdgcn_logf(sm);
              if (sm > kSumMax) l2 = kHighShift + __builtin_amdgcn_logf(sh);
              if (__any(!(sm >= kSumMin && (sm <= kSumMax || (sh >= kSumMin && sh <= kSumMax))))) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                  const float lt = max_shifted_lse(z[t]);
                  l2 = grp == t ? lt : l2;
                }
              }
              if constexpr (V > 1) l2 = merge_sub_lse<V>(l2);
            }
            finish(IntTag<u>{}, l2);
          });
        });
        blk_next = blk_after;
      }
    };
    // with several steps a wave, the first step's records are on their way while the
    // digits are formed (1M decode steps: 53.7 us, 55.3 the other way round); with one, the
    // digits come first, as in the scan of up to 8 heads, where that was measured
    int blk0 = 0, blk1 = 0;
    if (n_steps == kSteps) {
      blk0 = lane_block_clamped<V>(pt_row, first, n_c, lane);
      blk1 = kSteps > 1 ? lane_block_clamped<V>(pt_row, first + 16, n_c, lane) : 0;
      if (kSteps > 1) load_step(blk0);
    }
    block_digits<QT, 16, ND>(q + row0 * kDim, G, sDig);
    __syncthreads();
    lane_digits(sDig, grp, col, QD);
    if (n_steps == kSteps) {
      if (kSteps == 1) load_step(blk0);
      run(first, IntTag<kSteps>{}, blk1);
    } else {
#pragma unroll 1
      for (int t = 0; t < n_steps; ++t) {
        load_step(lane_block_clamped<V>(pt_row, first + 16 * t, n_c, lane));
        run(first + 16 * t, IntTag<1>{}, 0);
      }
    }
  }
  // ---- block partial (max, sum exp) per head over its pages, log2 domain: lane
  // l holds head l % 16; the wave's lanes are merged first
  merge_lanes_mod<16>(run_m, run_s);
  if (lane < 16) sRun[wave][lane] = make_float2(run_m, run_s);
  __syncthreads();
  if (threadIdx.x < G) {
    const int g = threadIdx.x;
    float m = -INFINITY, l = 0.0f;
    for (int w = 0; w < 4; ++w) m = fmaxf(m, sRun[w][g].x);
    if (m > -INFINITY)
      for (int w = 0; w < 4; ++w) {
        const float2 v = sRun[w][g];
        if (v.y > 0.0f) l += v.y * __builtin_amdgcn_exp2f(v.x - m);
      }
    partials[(row0 + g) * gridDim.x + blockIdx.x] = make_float2(m, l);
  }
}

}  // namespace

template <typename QT>
hipError_t launch_scan_wide(const ScanArgs& a, int steps, int v, hipStream_t st) {
  const int nd = scan_digits(a.H_q / a.H_kv);
#define LOCKS_WIDE(ND, SS, VV)                                                                \
  if (nd == ND && steps == SS && v == VV) {                                                   \
    hipLaunchKernelGGL((scan_wide_kernel<QT, ND, SS, VV>), a.grid, dim3(256), 0, st, a.H_q,   \
                       a.H_kv, a.H_q / a.H_kv, a.max_pages, static_cast<const QT*>(a.q),      \
                       a.summ, a.summ_bytes, a.page_table, a.seq_lens, a.s_hat, a.lay,        \
                       a.partials);                                                           \
    return hipGetLastError();                                                                 \
  }
#define LOCKS_WIDE_V(ND, SS) LOCKS_WIDE(ND, SS, 1) LOCKS_WIDE(ND, SS, 2) LOCKS_WIDE(ND, SS, 4)
  LOCKS_WIDE_V(3, 1) LOCKS_WIDE_V(3, 4) LOCKS_WIDE_V(4, 1) LOCKS_WIDE_V(4, 4)
#undef LOCKS_WIDE_V
#undef LOCKS_WIDE
  return hipErrorInvalidValue;
}

}  // namespace locks
