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
