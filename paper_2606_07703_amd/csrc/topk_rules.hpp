// How many threads take a row of the register top-k: a rule of sizes, host code
// that needs no device (a test calls it).
#pragma once

#include "kernels.hpp"

namespace sp {

constexpr int kRun = 16;     // consecutive positions per run
constexpr int kRegSub = 4;   // runs per thread

// Most of a row's time is the passes' fixed part (clearing and scanning the
// bins, barriers), which fewer threads share out over more rows on a CU, where
// there are rows to fill the CUs with: rows with more than k positions (the
// others only list them), the more the longer they are. Few threads are slow
// at writing many positions, and 64 or 128 stage only 2048 or 4096 of them in
// LDS. Per-query rows with 64 / 128 / 256 / 512 threads, us:
//   2048 rows of 2048 keys, k = 64 17 / 15 / 21 / 33, k = 1536 21 / 15 / 14 / 16;
//   4096 rows of 4096, k = 64 22 / 25 / 38 / 62, k = 2560 39 / 27 / 28 / 40, k =
//   3072 37 / 23 / 21 / 31, k = 4080 28 / 19 / 14 / 14; 512 of them, k = 64 18 /
//   12 / 9 / 11; 8192 rows of 8192 with 128 / 256 / 512: k = 2048 68 / 81 / 117, k
//   = 5120 91 / 69 / 87; 512 of them 18 / 13 / 12; 16384 rows of 16384 with 256 /
//   512: k = 2048 211 / 296; 512 of them 18 / 16.
// ncmax: candidates of the longest row.
inline int topk_threads(const Prob &p, int ncmax) {
  const int first = p.k > p.qo ? (p.k - p.qo) / p.b : 0;   // block with more than k positions
  const int64_t rows = (int64_t)(p.R > first ? p.R - first : 0) * (p.ha ? p.Hkv : 1);
  if (ncmax <= 64 * kRun * kRegSub && p.k <= 1024 && rows >= 2500) return 64;
  if (ncmax <= 128 * kRun * kRegSub && p.k <= 4096 && rows >= 256 + ncmax / 4) return 128;
  if (ncmax <= 256 * kRun * kRegSub && rows >= 256 + ncmax / 16) return 256;
  return 512;
}

}  // namespace sp
