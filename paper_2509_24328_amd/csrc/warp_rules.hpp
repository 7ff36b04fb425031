// Which way the cutoffs of a batch of rows go: plain host code, without the HIP runtime.
#pragma once

namespace sv {

constexpr int kWarpThreads = 512;                                // lanes of a row's workgroup
constexpr int kResidentMax = 16 * kWarpThreads * 8;              // bfloat16 entries of a row that a workgroup holds

// Are bfloat16 rows (`total` of n tensors) whose cutoffs alone are wanted held in registers and counted
// (warp_cutoffs_resident_kernel), not swept for lists (warp_cutoffs_kernel)?  Every size for K > 512, for which there
// are no lists (1600 x 65536, K = 2000: 88 us, 410 by radix levels).
// For top-p the counts are the better way for a nucleus of more than some ten tokens, and the lists, which end with the first sweep, for
// one of a few tokens, the usual one of a peaked row, once the chip is full.  Lists / registers, us, 2200 to 2900, 31 to 37 and 4
// tokens kept: 400 x 32000 26.5 / 17.8, 23.4 / 17.0, 15.1 / 16.9; 512 x 32768 27.7 / 18.1, 24.2 / 17.7, 16.2 / 17.6; 513 x 32768
// 30.3 / 21.4, 24.4 / 20.7, 15.5 / 20.0; 800 x 32000 39.3 / 28.2, 31.0 / 27.0, 21.4 / 27.0; 2000 x 20000 70.8 / 36.4, 48.7 / 34.1, 35.1 /
// 33.9; 1600 x 24576 65.1 / 35.9, 45.3 / 34.1, 29.7 / 33.6; 4000 x 25000 131 / 72.5, 86.4 / 68.4, 64.1 / 68.1; 200 x 49152 21.3 / 17.2, 20.5 /
// 17.0, 11.7 / 16.9.  A row of up to 64 entries is a list that one wavefront settles, and the counters are not even cleared: 4096 x 64 22.8 /
// 25.0 to 26.7, 60000 x 8 249 / 315 to 331; but 4096 x 100 41.9 to 48.5 / 25.0 to 27.4, 1500 x 520 73.4 to 77.5 / 11.8 to 13.2.
// For K up to 512 the lists are the better way throughout: 200 x 32000, K = 20 10.1 and 16.3.
// (A K of V or more keeps every entry, as one of 0 does.)
inline bool rows_in_registers(long long total, int V, int n, const int* top_k) {
  const bool few = V <= 64 ? false : V <= 24576 ? total * V <= 40000000 : V <= kResidentMax / 2 && total <= 512;
  for (int t = 0; t < n; ++t) {
    const bool use_k = top_k[t] > 0 && top_k[t] < V;
    if (!(use_k ? top_k[t] > kWarpThreads && V <= kResidentMax : few)) return false;
  }
  return true;
}

}  // namespace sv
