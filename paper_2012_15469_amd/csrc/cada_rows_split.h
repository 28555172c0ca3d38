// Which logistic shapes cada_logreg_rows.hip takes by itself, and how it cuts their minibatch rows into shares, one workgroup each: plain
// C++ without device code, so that a test can go over it on the host.
#pragma once

#include <cstdint>

namespace cada {

// Up to 8192 columns: rows per share and shares per worker, as many shares as give every CU a workgroup, while a share keeps the rows of one batch of its
// eight wavefronts (p <= 1024) or ten rows (each wavefront then has a part of every row) and 32 KB, at most eight.  Measured, us per step with
// 1, 2, 4, 8, 16 shares: M = 10, B = 200, p = 784: 25, 21, 19, 18, 19; M = 64, B = 128, p = 784: 23, 21.5, 21, 30, 51;
// M = 100, B = 256, p = 4000: 133, 90, 93, 111, 138; M = 10, B = 64, p = 4000: 33.5, 26.5, 22, 22 (two-pass kernels: 27, 32, 147, 25).
struct RowsSplit {
  int shares, rows;                              // per worker; per share (at most)
};
constexpr RowsSplit rows_split(int M, int B, int64_t p) {
  int64_t n = B * p / 8192 < 8 ? B * p / 8192 : 8;
  if (n > 256 / M) n = 256 / M;
  if (n > B / (p <= 1024 ? 24 : 10)) n = B / (p <= 1024 ? 24 : 10);
  if (n < 1) n = 1;
  const int rows = (int)((B + n - 1) / n);
  return {(B + rows - 1) / rows, rows};
}

// More than 8192 columns.
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

// Whether the path is taken by itself (p >= 4; vec: 4 where rows can be read 16 bytes at a time by the kernels that need that).  Not where one
// of the kernels that it stands beside is faster; measured, us per step here / two passes over the rows:
//   up to 1024 columns, many workers of few rows: a workgroup has eight wavefronts for one row each and the CUs take the workers in
//     rounds.  p = 784, B = 8: M = 256: 23.5 / 24.8; 300: 31 / 27; 1024: 66 / 50; 4096: 235 / 158; but M = 1024, B = 32: 0.94 of the time;
//   more columns: the same with some rows, p = 3000, M = 4096: B = 1: 1.24 of the time, 4: 1.09, 8: 0.91; M = 1024, B = 4: 0.99;
//   more than 4096 columns: a wavefront's part of a row takes two loads and more, and few workgroups leave CUs idle, where the two
//     passes cut the columns as well.  p = 6000, M = 4: B = 8: 0.86, 16: 1.05, 65: 1.09, 1024: 1.05; B = 65: M = 8 (48 workgroups): 1.04,
//     12 (72): 0.96.  Where the two passes read 4 bytes at a time: p = 8191, M = 4: B = 65: 0.95, 256: 0.99, 512: 1.13; M = 1, B = 256: 1.18;
//   more than 8192 columns / the single-pass kernel: p = 10240, M = 700: B = 1: 0.95, 4: 1.04, 16: 0.99; M = 4096, B = 4: 1.30; p = 20480,
//     M = 512: B = 4: 1.00, M = 700: 1.09; two passes take as long at best (p = 20479, M = 4, B = 64: 0.95 of the time, M = 16: 1.02).
//   8192 columns: the single-pass kernel takes 1.1 to 3.4 times as long.
constexpr bool rows_preferred(int M, int B, int64_t p, int vec) {
  if (p > 8192) return vec != 4 || M <= 512 || B >= 16;
  if (p <= 1024) return M <= 256 || B >= 32;
  if (M > 512 && B < 8) return false;
  if (p <= 4096 || p == 8192 || M * rows_split(M, B, p).shares >= 64) return true;
  return B <= (vec == 4 ? 10 : M > 1 ? 256 : 128);
}

}  // namespace cada
