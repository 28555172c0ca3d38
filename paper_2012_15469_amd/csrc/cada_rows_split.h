// How cada_logreg_rows.hip cuts the minibatch rows of more than 8192 columns into shares, one workgroup each: plain C++ without
// device code, so that a test can go over it on the host.
#pragma once

#include <cstdint>

namespace cada {

constexpr int64_t kWideEven = 7 * 2048;          // columns up to which a share may meet several workers
constexpr int kWideRows = 2048;                  // rows of a share at most (their offsets and labels lie in LDS)

constexpr int kSumsOfRow = 25;                   // workgroups whose sums take as long as a row

// `per` shares for every worker, or (per == 0) all M B rows, one worker's after the other's, cut evenly into `shares`.
struct WideSplit {
  int M, B;
  int shares;                                    // in all: M per, or as many as the rows are cut into
  int rows;                                      // rows per share (at most)
  int per;
};

// First row of share c, and the share that holds row f (rows of all workers in order).
constexpr int wide_first(const WideSplit &w, int c) {
  if (w.per) { const int m = c / w.per; return m * w.B + (int)((int64_t)(c - m * w.per) * w.B / w.per); }
  return (int)((int64_t)c * w.M * w.B / w.shares);
}
constexpr int wide_share(const WideSplit &w, int f) {
  if (w.per) { const int m = f / w.B; return m * w.per + (int)((((int64_t)(f - m * w.B) + 1) * w.per - 1) / w.B); }
  return (int)((((int64_t)f + 1) * w.shares - 1) / ((int64_t)w.M * w.B));
}
// Where share c leaves its sums for worker m, of wide_slots(): from one pair (share, worker) to the next one or both of the two grow.
constexpr int wide_slot(const WideSplit &w, int c, int m) { return w.per ? c : c + m; }
constexpr int wide_slots(const WideSplit &w) { return w.per ? w.shares : w.shares + w.M; }

// A workgroup fills a CU; the operands of a worker and the sums' way out cost it about as much as three
// rows, and 25 workgroups' sums cost the whole launch another.  So many shares for every worker as make the rounds of CUs
// cheapest, or, up to kWideEven columns and where it is less, all rows cut evenly over the CUs, although a share then may meet two
// workers.  Measured, us per step with a share count per worker and cut evenly: M = 37, B = 75, p = 20001: 77, 92;
// M = 100, B = 256, p = 10000: 220, 217; M = 100, B = 100, p = 8196: 113, 105.  With 1, 2, 4, 8, 16, 32 shares per worker: p = 20479,
// M = 16, B = 64: 142, 86, 58, 49, 52, 70; M = 4, B = 64: 135, 70, 47, 38, 36, 38; M = 64, B = 16: 63, 52, 55, 71, 105.
constexpr WideSplit wide_split(int M, int B, int64_t p) {
  WideSplit w{M, B, 0, 0, 0};
  const int64_t T = (int64_t)M * B;
  int64_t best = INT64_MAX;
  for (int n = (B + kWideRows - 1) / kWideRows; n <= 32 && n <= B; ++n) {
    const int r = (B + n - 1) / n;
    const int64_t cost = kSumsOfRow * (((int64_t)M * n + 255) / 256) * (r + 3) + (int64_t)M * n;
    if (cost < best) { best = cost; w.shares = M * n; w.rows = r; w.per = n; }
  }
  const int64_t cus = T < 256 ? T : 256, least = (T + kWideRows - 1) / kWideRows;
  const int64_t even = cus > least ? cus : least, most = (T + even - 1) / even;
  if (p <= kWideEven && kSumsOfRow * ((even + 255) / 256) * (most + 6) + even < best) { w.shares = (int)even; w.rows = (int)most; w.per = 0; }
  return w;
}

}  // namespace cada
