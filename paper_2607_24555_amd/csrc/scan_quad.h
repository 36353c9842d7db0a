// Rank-8 summary scan (int4 basis) of groups of up to 8 heads, every page size: 16
// pages per wave step as four quads of 4 pages, no LDS in the step.
//
// The kernel is built for HG = 4 or 8 head columns; a group of G heads takes the
// smaller HG >= G (columns g >= G repeat head 0 and are never stored).  ND: query digits
// (scan_digits).  Lane l =
// (grp = l / 16, col = l % 16); col = (cb, g) = (col / HG, col % HG).
//
// For quad Q of a step:
//  * stage 1 (int8 MFMA, two basis sets i = 0, 1): A row m is (page 4 Q + m / 4, basis
//    column 4 i + m % 4); the 16 B columns are the HG heads repeated 16 / HG times.
//    Lane (grp, col) receives p(page 4 Q + grp, l = 4 i + j, head g) in register j.
//  * stage 2 (16x16x32 MFMA, B as float16 hi + lo or, with four query digits, as three
//    bfloat16 terms): rows are the 16 tokens, K index 8 a + l is (page 4 Q + a, basis column
//    l), columns are (page, head).  HG columns leave
//    room for kCP = 16 / HG pages, so a quad takes kNP = HG / 4 passes; pass t covers
//    pages kCP t + cb.  A lane's 8 stage-1 values enter where the column's page is the
//    lane's own (grp % kCP == cb, by a zero scale elsewhere), and the A rows of the
//    pages of other passes are zeroed.  Register j of lane (grp, col) is then the logit
//    of token 4 grp + j of page 4 Q + kCP t + cb for head g, minus the centroid logit.
//  * the sums of 2^z over a lane's 4 tokens are reduced over grp four passes at a time
//    by two lane-swap stages that also hand the four totals to the four lane rows
//    (reduce4): the step's 16 pages x HG heads end up one or more per lane, all 64
//    lanes busy, so the logarithm, the centroid term, the store and the running
//    normaliser run HG / 4 times per step and not once per quad on a part of the lanes.
// The centroid MFMA (once per step) leaves a(page 4 grp + j, head g) in register j,
// from which the lane takes its own pages'.
//
// Pages of 16 V tokens (V = 2, 4) run as V sub-pages of 16 tokens (coefficient rows
// and row scales 16 u .. 16 u + 15 of sub-page u, the page's basis and centroid).
// Stage 1 then runs once per four pages: at V = 4 a quad is one page, lane (grp, col)
// gets p(page grp of the step, l, head g), and three row swaps (16 and 32 lanes)
// broadcast page u's rows for quad u; at V = 2 a pass covers two quads, its rows
// ordered so that one 16-lane swap yields both quads' layouts.  The sums of a page's
// sub-pages are added over their lanes before the logarithm.
//
// Bound: at 16-token pages the scattered record gather (8 x 128K, four-head groups: 94 us,
// 4.6 TB/s, where the gather alone runs at 5.2 to 5.7); at 32 and 64 tokens the vector
// ALU's work per sub-page (58.5 and 44.5 us), so the per-step tail above is shared by the
// quads and the instances for groups of four are held to 168 registers (three waves per
// SIMD; at two, 32-token pages take 52 us for 46 with the store in the last-level cache).
// The others' four-step instances take 189 to 246 registers, two waves.
#pragma once

#include "locks_internal.h"
#include "scan_common.h"
#include "scan_launch.h"
#include "scan_wide.h"

namespace locks {
namespace {

// the value of lane l ^ X within a 16-lane row, X = 4 or 8
template <int X>
__device__ __forceinline__ float row_xor(float v) {
  int u = __float_as_int(v);
  if (X == 8) {
    u = __builtin_amdgcn_update_dpp(0, u, 0x128, 0xF, 0xF, false);  // rotate by 8
  } else {
    u = __builtin_amdgcn_update_dpp(0, u, 0x141, 0xF, 0xF, false);  // l -> 7 - l in each half row
    u = __builtin_amdgcn_update_dpp(0, u, 0x1B, 0xF, 0xF, false);   // l -> 3 - l in each quad
  }
  return __int_as_float(u);
}

template <typename QT, int HG, int ND, int kSteps, int V>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(HG == 4 && ND == 3 && V > 1 ? 3 : 2))) void scan_quad_kernel(
    int H_q, int H_kv, int G, int max_pages, const QT* __restrict__ q,
    const uint8_t* __restrict__ summ, uint32_t summ_bytes, const int32_t* __restrict__ page_table,
    const int32_t* __restrict__ seq_lens, float* __restrict__ s_hat, SHatLayout lay,
    float2* __restrict__ partials) {
  constexpr int R = 8, P = kPage * V;
  constexpr int kCP = 16 / HG, kNP = HG / 4;
  constexpr uint32_t kStride = rec_stride(R, 0, P);
  constexpr uint32_t kCoef = rec_coef_off(R), kMu = rec_mu_off(R, 0, P), kSc = rec_scale_off(R, 0, P);
  __shared__ float2 sRun[4][16];
  __shared__ DigitLds<HG, ND> sDig;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
  const int h = blockIdx.y, s = blockIdx.z;
  const int n_c = seq_lens[s] / P * V;  // sub-pages of the complete pages
  const int pg = scan_chunk() * 4 + wave;
  const long row0 = (long)s * H_q + (long)h * G;
  const int32_t* pt_row = page_table + (long)s * max_pages;
  const int cb = col / HG, g = col % HG;
  const int ra4 = col >> 2, rl4 = col & 3;       // stage-1 A row: (page of the quad, column)
  const bool mine = grp % kCP == cb;               // the column's page is this row's in some pass
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
    QDigits<ND> QD;      // read from the block's once formed
    float inv_m = 0.0f;  // scale of the stage-1 values; zero where the page is not the column's
    // own(u): the u-th page of the step (0 .. 15) whose score this lane finishes
    auto own = [&](int u) { return HG == 4 ? 4 * grp + cb : 4 * grp + 2 * u + cb; };
    float* shat_lane = s_hat + lay.base(s, h) + (long)g * lay.head;

    // record offsets of one step: ra[Q] page 4 Q + col / 4 (stage-1 rows), rb[Q] page
    // 4 Q + grp, rc[Q][t] page 4 Q + kCP t + cb (the columns' pages), rm page col (the
    // centroid row of this lane), ro[u] page own(u).  When stage 1 is shared (V > 1), pa[m] and pb[m] are the records of the
    // pages of pass m in rows col / 4 and grp: pages 4 m + x at V = 4, pages
    // 4 m + ((x & 1) << 1 | x >> 1) at V = 2.
    constexpr int kShare = V;  // quads per stage-1 pass
    constexpr int kPasses = 4 / kShare;
    struct Offs {
      uint32_t rb[4], rc[4][kNP], rm, ro[kNP];
      uint32_t pa[kPasses], pb[kPasses];
    };
    const __amdgpu_buffer_rsrc_t rs = summ_rsrc(summ, summ_bytes);
    const uint32_t blk_bytes = (uint32_t)H_kv * kStride, head_off = (uint32_t)h * kStride;
    auto offsets = [&](int blk) {
      Offs o;
      const int off = (int)rec_off(blk, blk_bytes, head_off);  // of page lane % 16
      auto rec = [&](int page) { return (uint32_t)__shfl(off, page, 64); };
#pragma unroll
      for (int Q = 0; Q < 4; ++Q) {
        o.rb[Q] = rec(4 * Q + grp);
#pragma unroll
        for (int t = 0; t < kNP; ++t) o.rc[Q][t] = rec(4 * Q + kCP * t + cb);
      }
      o.rm = (uint32_t)off;
#pragma unroll
      for (int u = 0; u < kNP; ++u) o.ro[u] = rec(own(u));
      auto row_page = [](int x) { return V == 2 ? ((x & 1) << 1 | x >> 1) : x; };
#pragma unroll
      for (int m = 0; m < kPasses; ++m) {
        o.pa[m] = HG == 4 && V == 1 ? o.rc[m][0] : rec((4 * m + row_page(ra4)) * V);
        o.pb[m] = V == 1 ? o.rb[m] : rec((4 * m + row_page(grp)) * V);
      }
      return o;
    };
    uint4 vb[kPasses][2];  // basis rows of stage-1 pass m (quad m if V = 1), set i
    uint2 cf[4];           // coefficient row `col` of page 4 Q + grp
    uint2 cs[4][kNP];      // row scales of tokens 4 grp .. 4 grp + 3 of the columns' pages
    uint4 vs[kPasses];     // basis column scales of the pass's page grp
    uint32_t msw[kNP];     // centroid scale of the lane's own pages (low half)
    uint4 mu[2];           // centroid bytes 32 grp .. 32 grp + 31 of the lane's centroid row
    // sub-page (V > 1) of the pages read through rb and rc
    const uint32_t sub_b = (uint32_t)(grp % V);
    auto sub_c = [&](int t) { return (uint32_t)((kCP * t + cb) % V); };
    // loads of one step's registers; in a run the next step's are issued right
    // after the register's last use in the current one
    auto ld_vb = [&](const Offs& o, int m, int i) { vb[m][i] = bld16(rs, o.pa[m] + 64u * (4 * i + rl4) + 16u * grp); };
    auto ld_cf = [&](const Offs& o, int Q) { cf[Q] = bld8(rs, o.rb[Q] + kCoef + 8u * (16u * sub_b + col)); };
    auto ld_cs = [&](const Offs& o, int Q, int t) {
      cs[Q][t] = bld8(rs, o.rc[Q][t] + kSc + 2u * (R + 16u * sub_c(t) + 4 * grp));
    };
    auto ld_vs = [&](const Offs& o, int m) { vs[m] = bld16(rs, o.pb[m] + kSc); };
    auto ld_ms = [&](const Offs& o, int u) { msw[u] = bld4(rs, o.ro[u] + kSc + 2u * (R + P)); };
    auto ld_mu = [&](const Offs& o) {
      mu[0] = bld16(rs, o.rm + kMu + 32u * grp);
      mu[1] = bld16(rs, o.rm + kMu + 32u * grp + 16u);
    };

    // every register of the step whose pages' blocks lanes 0..15 hold in blk
    auto load_step = [&](int blk) {
      const Offs o0 = offsets(blk);
      ld_mu(o0);
#pragma unroll
      for (int Q = 0; Q < 4; ++Q) {
        if (Q < kPasses) {
          ld_vb(o0, Q, 0);
          ld_vb(o0, Q, 1);
          ld_vs(o0, Q);
        }
        ld_cf(o0, Q);
#pragma unroll
        for (int t = 0; t < kNP; ++t) ld_cs(o0, Q, t);
      }
#pragma unroll
      for (int u = 0; u < kNP; ++u) ld_ms(o0, u);
    };

    bool low = false;    // a page's sum was too small
    uint64_t force = 0;  // ~0: every sum is taken with its max shifted out
    // kN consecutive 16-page steps from page `start` whose first step's
    // registers are loaded (blk_next: blocks of the second step's pages), fully
    // unrolled so that every wait for a prefetched register counts exactly the
    // loads issued after it.
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

        // ---- centroid term of the lane's own pages, before its scale
        float am[kNP];
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
          for (int u = 0; u < kNP; ++u) {
            int da[ND];
#pragma unroll
            for (int d = 0; d < ND; ++d) {
              if constexpr (HG == 8) {
                da[d] = cb ? acc[d][2 * u + 1] : acc[d][2 * u];
              } else {
                const int lo = (cb & 1) ? acc[d][1] : acc[d][0], hi = (cb & 1) ? acc[d][3] : acc[d][2];
                da[d] = (cb & 2) ? hi : lo;
              }
            }
            am[u] = join_digits(da);
          }
        }

        float bq[kShare][8];  // shared stage 1: the values of the step's quads
        float ps[4][kNP];     // sum of 2^z over the lane's four tokens
        float wide[kNP];      // LSE, max shifted out, of the lane's own pages (-inf: not needed)
        bool any_wide = false;
#pragma unroll
        for (int u = 0; u < kNP; ++u) wide[u] = -INFINITY;
        auto keep = [&](int u, float s2) {  // store and count the page score
          const int page = page0 + own(u);
          const bool live = page < n_c && own(u) % V == 0;
          if (live && g < G) shat_lane[(long)(page / V) * lay.page] = s2 * 0.69314718055994531f;
          const float e = __builtin_amdgcn_exp2f(-fabsf(s2 - run_m));
          const bool up = s2 > run_m;
          const float ns = up ? fmaf(run_s, e, 1.0f) : run_s + e;
          run_s = live ? ns : run_s;
          run_m = (live && up) ? s2 : run_m;
        };
        static_for_int<4>([&](auto q_tag) __attribute__((always_inline)) {
          constexpr int Q = decltype(q_tag)::value;
          __builtin_amdgcn_sched_barrier(0);
          // ---- stage 1: vals[4 i + j] = p(page 4 Q + grp, l = 4 i + j, head g)
          float vals[8];
          if (Q % kShare == 0) {
            const int m = Q / kShare;
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
            const uint32_t vsw[4] = {vs[m].x, vs[m].y, vs[m].z, vs[m].w};
            const float sc = kShare == 1 ? inv_m : QD.inv_scale;
#pragma unroll
            for (int l = 0; l < 8; ++l) {
              const int j = l & 3;
              const h2 pr = as_h2(vsw[l >> 1]);
              const float vsc = (float)((l & 1) ? pr.y : pr.x);
              vals[l] = p[l >> 2][j] * (vsc * sc);
            }
            if (pf) ld_vs(on, m);
            if constexpr (kShare > 1) {
              // the 16-lane swap of rows r0..r3 (lanes 16 u ..) gives X = (r0, r0,
              // r2, r2) and Y = (r1, r1, r3, r3).  V = 4: rows hold pages 0..3 and
              // the 32-lane swaps of X and Y put each row everywhere.  V = 2: rows
              // hold pages 4 m + 0, 2, 1, 3, so X is quad 2 m's layout (pages
              // 4 m, 4 m, 4 m + 1, 4 m + 1) and Y quad 2 m + 1's.
#pragma unroll
              for (int l = 0; l < 8; ++l) {
                const uint32_t x = __float_as_uint(vals[l]);
                const auto xy = __builtin_amdgcn_permlane16_swap(x, x, false, false);
                if constexpr (V == 4) {
                  const auto xx = __builtin_amdgcn_permlane32_swap(xy[0], xy[0], false, false);
                  const auto yy = __builtin_amdgcn_permlane32_swap(xy[1], xy[1], false, false);
                  bq[0][l] = __uint_as_float(xx[0]);
                  bq[1][l] = __uint_as_float(yy[0]);
                  bq[2][l] = __uint_as_float(xx[1]);
                  bq[3][l] = __uint_as_float(yy[1]);
                } else {
                  bq[0][l] = __uint_as_float(xy[0]);
                  bq[1][l] = __uint_as_float(xy[1]);
                }
              }
            }
          }
          if constexpr (kShare > 1) {
#pragma unroll
            for (int l = 0; l < 8; ++l) vals[l] = mine ? bq[Q % kShare][l] : 0.0f;
          }
          uint4 A;
          if constexpr (ND == 3) {
            A = __builtin_bit_cast(uint4, byte8_to_h8(cf[Q].x, cf[Q].y));
          } else {
            const uint2 a0 = byte4_to_b4(cf[Q].x), a1 = byte4_to_b4(cf[Q].y);
            A = make_uint4(a0.x, a0.y, a1.x, a1.y);
          }
          if (pf) ld_cf(on, Q);
          // ---- stage 2 for the quad
          uint32_t bt[ND - 1][4];  // the terms of B
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if constexpr (ND == 3) {
              const auto hi = __builtin_amdgcn_cvt_pkrtz(vals[2 * e], vals[2 * e + 1]);
              const auto lo = __builtin_amdgcn_cvt_pkrtz(vals[2 * e] - (float)hi[0], vals[2 * e + 1] - (float)hi[1]);
              bt[0][e] = __builtin_bit_cast(uint32_t, hi);
              bt[1][e] = __builtin_bit_cast(uint32_t, lo);
            } else {
              uint32_t t3[3];
              split3_b2(vals[2 * e], vals[2 * e + 1], t3);
#pragma unroll
              for (int i = 0; i < 3; ++i) bt[i][e] = t3[i];
            }
          }
          float z[kNP][4];
          uint64_t far = force;  // lanes whose sum is too large
          static_for_int<kNP>([&](auto t_tag) __attribute__((always_inline)) {
            constexpr int t = decltype(t_tag)::value;
            uint4 At = A;
            if (kNP > 1) {
              const bool in = grp / kCP == t;
              At = make_uint4(in ? A.x : 0u, in ? A.y : 0u, in ? A.z : 0u, in ? A.w : 0u);
            }
            f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int i = ND - 2; i >= 0; --i) {  // smallest terms first
              const uint4 Bt = make_uint4(bt[i][0], bt[i][1], bt[i][2], bt[i][3]);
              if constexpr (ND == 3)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, At),
                                                             __builtin_bit_cast(h8, Bt), acc, 0, 0, 0);
              else
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, At),
                                                              __builtin_bit_cast(b8, Bt), acc, 0, 0, 0);
            }
            const h2 c01 = as_h2(cs[Q][t].x), c23 = as_h2(cs[Q][t].y);
            z[t][0] = (float)c01.x * acc[0];
            z[t][1] = (float)c01.y * acc[1];
            z[t][2] = (float)c23.x * acc[2];
            z[t][3] = (float)c23.y * acc[3];
            if (pf) ld_cs(on, Q, t);
            ps[Q][t] = __builtin_amdgcn_exp2f(z[t][0]) + __builtin_amdgcn_exp2f(z[t][1]) +
                       __builtin_amdgcn_exp2f(z[t][2]) + __builtin_amdgcn_exp2f(z[t][3]);
            far |= __ballot(!(ps[Q][t] <= kSumMax));
          });
          // tokens spread too widely: taken again while the quad's logits are in registers
          // (8 x 128K, four-head groups, every page so: 97 us, and 150 where the wave's
          // pages were scanned a second time; pages of ordinary spread 94)
          if (__builtin_expect(far != 0, 0)) {
            any_wide = true;
#pragma unroll
            for (int t = 0; t < kNP; ++t) {
              const float l2 = max_shifted_lse(z[t]);
              wide[t] = grp == Q ? l2 : wide[t];
            }
          }
        });
        __builtin_amdgcn_sched_barrier(0);
        // ---- the LSEs of the lane's own pages: totals, four passes at a time; the sums of
        // a page's sub-pages added (every lane of the page gets the total)
        float l2[kNP];
#pragma unroll
        for (int u = 0; u < kNP; ++u) l2[u] = reduce4(ps[0][u], ps[1][u], ps[2][u], ps[3][u]);
        if (__builtin_expect(!any_wide, 1)) {
#pragma unroll
          for (int u = 0; u < kNP; ++u) {
            if (V > 1) l2[u] += row_xor<HG>(l2[u]);
            if (V == 4 && HG == 4) l2[u] += row_xor<8>(l2[u]);
          }
          if constexpr (V == 4 && HG == 8) l2[0] += l2[1];
#pragma unroll
          for (int u = 0; u < kNP; ++u) l2[u] = __builtin_amdgcn_logf(l2[u]);
        } else {
#pragma unroll
          for (int u = 0; u < kNP; ++u) {
            l2[u] = wide[u] != -INFINITY ? wide[u] : __builtin_amdgcn_logf(l2[u]);
            if (V > 1) l2[u] = lse2_log2(l2[u], row_xor<HG>(l2[u]));
            if (V == 4 && HG == 4) l2[u] = lse2_log2(l2[u], row_xor<8>(l2[u]));
          }
          if constexpr (V == 4 && HG == 8) l2[0] = lse2_log2(l2[0], l2[1]);
        }
#pragma unroll
        for (int u = 0; u < kNP; ++u) {
          low |= l2[u] < kLog2SumMin;
          const float s2 = am[u] * ((float)as_h2(msw[u]).x * QD.inv_scale) + l2[u];
          if (pf) ld_ms(on, u);
          if (!(HG == 8 && V == 4 && u == 1)) keep(u, s2);
        }
        blk_next = blk_after;
      }
    };
    // with one step a wave, in grids that leave most of the chip idle, holding the step's
    // registers across the barrier costs more than it hides (32K decode steps: 26.2 us
    // against 26.8); with several the first step's records are on their way while the
    // digits are formed, as in the scan of 9 to 16 heads, where that was measured
    int blk0 = 0, blk1 = 0;
    if (n_steps == kSteps) {
      blk0 = lane_block_clamped<V>(pt_row, first, n_c, lane);
      blk1 = kSteps > 1 ? lane_block_clamped<V>(pt_row, first + 16, n_c, lane) : 0;
      if (kSteps > 1) load_step(blk0);
    }
    block_digits<QT, HG, ND>(q + row0 * kDim, G, sDig);
    __syncthreads();
    lane_digits(sDig, grp, g, QD);
    inv_m = mine ? QD.inv_scale : 0.0f;
    if (n_steps == kSteps) {
      if (kSteps == 1) load_step(blk0);
      run(first, IntTag<kSteps>{}, blk1);
    }
    for (bool again = n_steps != kSteps;; again = true) {
      if (again)
#pragma unroll 1
        for (int t = 0; t < n_steps; ++t) {
          load_step(lane_block_clamped<V>(pt_row, first + 16 * t, n_c, lane));
          run(first + 16 * t, IntTag<1>{}, 0);
        }
      if (force || !__any(low)) break;
      force = ~0ull;
      run_m = -INFINITY;
      run_s = 0.0f;
    }
  }
  // ---- block partial (max, sum exp) per head over its pages, log2 domain: lane
  // l holds head l % HG; the wave's lanes are merged first
  merge_lanes_mod<HG>(run_m, run_s);
  if (lane < HG) sRun[wave][lane] = make_float2(run_m, run_s);
  __syncthreads();
  if (threadIdx.x < G) {
    const int gg = threadIdx.x;
    float m = -INFINITY, l = 0.0f;
    for (int w = 0; w < 4; ++w) m = fmaxf(m, sRun[w][gg].x);
    if (m > -INFINITY)
      for (int w = 0; w < 4; ++w) {
        const float2 v = sRun[w][gg];
        if (v.y > 0.0f) l += v.y * __builtin_amdgcn_exp2f(v.x - m);
      }
    partials[(row0 + gg) * gridDim.x + blockIdx.x] = make_float2(m, l);
  }
}

}  // namespace

template <typename QT>
hipError_t launch_scan_quad(const ScanArgs& a, int hg, int steps, int v, hipStream_t st) {
  const int nd = scan_digits(a.H_q / a.H_kv);
#define LOCKS_QUAD(HH, ND, SS, VV)                                                            \
  if (hg == HH && nd == ND && steps == SS && v == VV) {                                       \
    hipLaunchKernelGGL((scan_quad_kernel<QT, HH, ND, SS, VV>), a.grid, dim3(256), 0, st,      \
                       a.H_q, a.H_kv, a.H_q / a.H_kv, a.max_pages,                            \
                       static_cast<const QT*>(a.q), a.summ, a.summ_bytes, a.page_table,       \
                       a.seq_lens, a.s_hat, a.lay, a.partials);                               \
    return hipGetLastError();                                                                 \
  }
#define LOCKS_QUAD_V(HH, ND, SS) LOCKS_QUAD(HH, ND, SS, 1) LOCKS_QUAD(HH, ND, SS, 2) LOCKS_QUAD(HH, ND, SS, 4)
  LOCKS_QUAD_V(4, 3, 1) LOCKS_QUAD_V(4, 3, 4) LOCKS_QUAD_V(4, 4, 1) LOCKS_QUAD_V(4, 4, 4)
  LOCKS_QUAD_V(8, 4, 1) LOCKS_QUAD_V(8, 4, 4)
#undef LOCKS_QUAD_V
#undef LOCKS_QUAD
  return launch_scan_wide<QT>(a, steps, v, st);
}

}  // namespace locks
