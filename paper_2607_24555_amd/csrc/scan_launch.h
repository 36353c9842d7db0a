// Launch interface between the scan's dispatch (scan.hip) and its kernels' files.
#pragma once

#include "locks_internal.h"

namespace locks {

struct ScanArgs {
  dim3 grid;  // (scan_blocks, KV heads, sequences)
  int H_q, H_kv, max_pages;
  const void* q;
  bool q_bf16;
  const uint8_t* summ;
  uint32_t summ_bytes;
  const int32_t* page_table;
  const int32_t* seq_lens;
  float* s_hat;
  SHatLayout lay;
  float2* partials;
};

// Query digits of the rank-8 scans for groups of G heads.  Three (20 bits of the head's
// largest element) and the projections as pairs of float16 for groups of four and sixteen
// heads, whose scans have held no more since they were written; four (30 bits) and bfloat16
// triples, which hold a float32 exactly at any size, for the others, which the generic scan
// (22 bits of every element, float32 projections) would otherwise take.  Mean and largest
// error of the page scores against 64 bits, scores of up to 44 nats, 20K to 40K tokens:
// fp32 queries 1.0e-6 and 6e-6 (three digits 6.5e-6 and 3.7e-5, generic 2.0e-6 and 1.5e-5),
// bfloat16 ones 1.0e-6 and 5e-6 (1.0e-6 and 6e-6; 1.2e-6 and 8e-6).  Eight-head groups, 8 x
// 64K tokens x 4 KV heads: 25.3 us (23.4 with three, 62 generic).
inline int scan_digits(int G) { return G == 4 || G == 16 ? 3 : 4; }

// Rank 8, int4 basis: hg head columns (4, 8 or 16, at least G), `steps` 16-page steps
// per wave, v 16-token sub-pages per page.  One translation unit per query type.
template <typename QT>
hipError_t launch_scan_quad(const ScanArgs& a, int hg, int steps, int v, hipStream_t st);
// Ranks 2 and 4, four-head groups, int4 basis, 16-token pages.
hipError_t launch_scan_low(const ScanArgs& a, int rank, hipStream_t st);
// 16-token pages, any rank, group and basis.
hipError_t launch_scan_mfma(const ScanArgs& a, int rank, int basis, hipStream_t st);
// 32- and 64-token pages, any rank and group; wave_pages pages per wave.
hipError_t launch_scan_page(const ScanArgs& a, int rank, int page_size, int wave_pages,
                            hipStream_t st);

}  // namespace locks
