// Which form a prefill attention call takes: a rule on sizes (host code that
// needs no HIP, so that a test can compile it by itself).
#pragma once

#include <stdint.h>

namespace sm {

constexpr int kPfVec = 256;  // query vectors per workgroup when its waves do not split the keys
constexpr int kPfCus = 256;

struct PrefillPlan {
  int splits;  // KS: groups into which the waves of a workgroup split the keys
  bool few;    // few rows: the kernel leaves requests of few keys unsplit
};

// Where the query vectors make fewer workgroups than compute units, KS = 4 or
// 2 makes 4 or 2 times as many, each with a quarter or half of the vectors and
// its waves over different keys; with the units full it only adds LDS fills
// (16 x 2458 rows: 894, 1071 and 1663 us for KS = 1, 2, 4).  A sweep over
// rows and contexts is in profiles/prefill_attention_key-splits.md; from it,
// us for KS = 1, 2, 4 at 32/8 heads, D = 128: 512 rows after 16384: 429, 274,
// 229 (64, 128, 256 workgroups); 900 rows after 4096: 132, 94, 118 (120, ...);
// 2048 after 4096: 198, 207, 271 (256, ...); 256 rows alone: 15, 12, 10.
//  * A whole prompt's workgroups differ in length (its last rows see all of
//    it, its first almost nothing), so halving them still pays up to 3/4 of
//    the units: 1200 rows: 39, 29, 40 (152, ...); 1500: 47, 36, 51 (192, ...).
//    Not after a longer context (1200 after 4096: 141, 162, 181), which the
//    host can only rule out by the cache's capacity: it bounds the length.
//    Nor for several shorter prompts, whose workgroups differ less (4 x 400
//    rows at 28/4 heads 23, 23, 31 and at 32/8 21, 26, 33; one of 640 rows at
//    64/8 heads 26, 22, 32): hence 640 rows.
//  * Up to 128 vectors per request (half of the waves idle with KS = 1) the
//    length decides between the forms; the kernel sees it.
// The sizes are averages and bounds (the rows of each request are device
// data); a grid that a loose max_rows would blow up keeps KS = 1.
inline PrefillPlan plan_prefill(int n, int H, int G, int total_rows, int max_rows, int64_t capacity) {
  const int64_t avg = ((int64_t)total_rows + n - 1) / n;
  auto wgs = [&](int ks, int64_t rows) {
    const int bq = kPfVec / ks / G;
    return (rows + bq - 1) / bq * n * H;
  };
  for (int ks = 4; ks >= 2; ks /= 2)
    if (wgs(ks, avg) <= kPfCus && wgs(ks, max_rows) <= 8 * kPfCus)
      return PrefillPlan{ks, ks == 4 && (int64_t)max_rows * G <= 128};
  if (wgs(1, avg) <= 3 * kPfCus / 4 && wgs(2, max_rows) <= 8 * kPfCus && max_rows >= 640 &&
      capacity < 2 * (int64_t)max_rows)
    return PrefillPlan{2, false};
  return PrefillPlan{1, false};
}

}  // namespace sm
