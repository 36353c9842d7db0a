// Dispatch of the summary scan (Sec. 4 "Score", Eq. (1)): for every complete page j of a
// (sequence, KV head) and every query head g of its group,
//   hat s_j(q_g) = log sum_i exp[(q_g^T mu_j + (V_j^T q_g)^T c_i) / sqrt(d)].
// Every scan block also writes, per query head, the partial (max, sum 2^x) of its
// pages' scores in the log2 domain; the select kernel reduces them into log Z_g.
#include "locks_internal.h"
#include "scan_launch.h"

namespace locks {

// Rank 8 with an int4 basis takes the register-resident scans at every group and page
// size (larger pages as 16-token sub-pages): scan_quad for up to 8 heads a group,
// scan_wide above.  Against the generic matrix-core scan that groups other than 4 and 16
// heads took before: six ragged sequences of 20K to 256K tokens with eight-head groups
// 114 -> 46 us; one head over 4K tokens 43 -> 7.6 us (one step per wave where the
// generic kernel walks 64 pages per wave).
static bool use_quad_kernel(const locks_cfg_t& c) {
  return c.basis == LOCKS_BASIS_INT4 && c.rank == 8;
}

// 16-page steps per wave of those scans: 4, or 1 when a 4-step grid would have fewer
// blocks than the GPU has compute units (32K tokens x 8 heads: 7.5 us at 1 step, 12.5 at
// 4; 8 x 128K: 94 us at 4 steps, 126 at 1, 97 at 8).
static int quad_steps(const locks_cfg_t& c) {
  const long sub = (long)c.max_pages_per_seq << sub_page_log2(c);
  const long blocks4 = (sub + 255) / 256 * c.num_kv_heads * c.num_seqs;
  return blocks4 < 256 ? 1 : 4;
}

static bool use_low_kernel(const locks_cfg_t& c) {
  return c.basis == LOCKS_BASIS_INT4 && c.page_size == kPage && (c.rank == 2 || c.rank == 4) &&
         c.num_q_heads == 4 * c.num_kv_heads;
}

// Pages per wave of the 32/64-token scan: 64, or 32 / 16 when 64 would leave
// fewer than two waves per SIMD of the GPU (1,024 SIMDs).
static int page_wave_pages(const locks_cfg_t& c) {
  for (int wp = 64; wp > 16; wp /= 2)
    if ((long)((c.max_pages_per_seq + wp - 1) / wp) * c.num_kv_heads * c.num_seqs >= 2048) return wp;
  return 16;
}

int scan_pages_per_block(const locks_cfg_t& c) {
  if (use_quad_kernel(c)) return (64 * quad_steps(c)) >> sub_page_log2(c);
  if (c.page_size != kPage) return 4 * page_wave_pages(c);
  return kScanPagesPerBlock;
}

hipError_t launch_scan(const locks_cfg_t& c, const void* q, const void* summaries,
                       const int32_t* page_table, const int32_t* seq_lens, float* s_hat,
                       SHatLayout lay, float2* partials, hipStream_t st) {
  const int G = c.num_q_heads / c.num_kv_heads;
  const ScanArgs a{dim3(scan_blocks(c), c.num_kv_heads, c.num_seqs),
                   c.num_q_heads, c.num_kv_heads, c.max_pages_per_seq, q, c.q_dtype == LOCKS_BF16,
                   static_cast<const uint8_t*>(summaries), (uint32_t)summary_store_bytes(c),
                   page_table, seq_lens, s_hat, lay, partials};
  if (use_quad_kernel(c)) {
    const int hg = G <= 4 ? 4 : (G <= 8 ? 8 : 16), v = 1 << sub_page_log2(c);
    return a.q_bf16 ? launch_scan_quad<uint16_t>(a, hg, quad_steps(c), v, st)
                    : launch_scan_quad<float>(a, hg, quad_steps(c), v, st);
  }
  if (c.page_size != kPage) return launch_scan_page(a, c.rank, c.page_size, page_wave_pages(c), st);
  if (use_low_kernel(c)) return launch_scan_low(a, c.rank, st);
  return launch_scan_mfma(a, c.rank, c.basis, st);
}

}  // namespace locks
