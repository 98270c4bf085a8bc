// Rules on sizes that pick the product's layout and the way a CG step is launched.
#pragma once
#include <cstddef>
#include <cstdint>

namespace fc {

// One wave walks a slice's rows from end to end, so a matrix of few slices and long
// rows waits for single waves; the row layout deals a row to 8 to 64 lanes.  us a
// product, sliced / rows: 3-D p = 2, 381 slices 9.2 / 7.4, 1,076 11.7 / 11.8; p = 3,
// 107 13.5 / 7.7, 343 18.2 / 9.3, 791 20.5 / 16.4, 1,838 29.4 / 30.2; p = 4, 244 31.6 /
// 10.4, 1,838 54.5 / 49.5, 3,546 83.5 / 99.8; rows of up to 36 on average never.
inline bool few_long_rows(int64_t nnz, int64_t n_rows, int64_t n_slices) {
  const double mean = n_rows ? double(nnz) / double(n_rows) : 0.0;
  return mean >= 48.0 && (double)n_slices < 9.0 * mean;
}

// Stored entries, and entries of the longest row, up to which the p update of a CG step
// joins the sliced product of the next: it saves a launch and makes every gather two.
// us a step joined / apart: 2-D 40^2 p = 2 (0.1M entries) 14.0 / 15.8, 110^2 p = 3
// (2.7M) 21.3 / 22.0, 250^2 p = 2 (4.0M) 29.4 / 30.9; 3-D 16^3 p = 2 (2.1M) 23.5 / 24.9,
// 20^3 p = 2 (4.3M) 31.0 / 31.5, 60^3 p = 1 (6.1M) 47.4 / 46.9, 30^3 p = 2 (14M) 64 / 61;
// rows of up to 343, 9^3 p = 3 (2M) 45 / 34, of up to 729, 6^3 p = 4 75 / 60.
constexpr int64_t kJoinEntries = int64_t(4) << 20;
constexpr int kJoinRow = 125;
inline bool step_joins(int64_t nnz, int32_t max_row) {
  return nnz <= kJoinEntries && max_row <= kJoinRow;
}

// Layout of the product in steps whose p update may join the sliced one: few long rows
// go to the row layout only where its product wins more than the launch saved.  us a
// step sliced and joined / rows, 3-D p = 2 (slices an entry of the mean row): 5^3 cells
// (0.5) 18.2 / 20.3, 6^3 18.8 / 20.4, 7^3 19.4 / 20.5, 8^3 (1.4) 19.4 / 21.0, 9^3 (1.9)
// 19.9 .. 20.6 / 20.4, 10^3 (2.6) 21.6 / 21.5, 11^3 21.6 / 21.3, 12^3 (4.2) 22.0 / 20.6,
// 14^3 22.8 / 22.0, 15^3 (7.9) 22.5 .. 23.2 / 22.6.
inline bool rows_beat_join(int64_t nnz, int64_t n_rows, int64_t n_slices) {
  return few_long_rows(nnz, n_rows, n_slices) &&
         (double)n_slices * (double)n_rows >= 2.2 * (double)nnz;
}

// Stored rows a chunk of the block products with 64 < m <= 192, n blocks in a launch.
// A chunk costs two barriers, and the LDS it takes a workgroup less on the compute unit:
// many rows where the launch does not fill the chip, few where it does.  us a product and
// pull, FP64 (m / blocks: rows us): 81/216 24 11.9, 6 13.6; 81/1000 24 13.7, 6 14.4;
// 81/4096 24 37.5, 6 24.6; 98/16 16 13.1, 4 15.7; 125/512 16 16.3, 4 21.3; 125/1331 16 23.1,
// 4 26.3; 125/4096 16 52.5, 4 48.5; 162/256 8 19.6, 24 18.0; 162/4096 8 78.0, 24 96.5; 192
// 8 as good as any from 64 to 4,096.  FP32, the product alone: 81/216 24 12.3, 8 14.2;
// 81/2744 24 24.4, 8 18.8; 125/125 24 14.8, 8 17.2; 125/4096 24 45.2, 8 31.3; 162/256
// 24 18.5, 12 20.0, 4 27.1; 162/4096 24 71.9, 12 52.0, 4 62.2; 192/216 24 19.0, 4 20.6;
// 192/2197 24 45.9, 12 38.1, 4 34.6.
inline int staged_rows(bool f64, int m, int64_t n) {
  if (f64) return m <= 96 ? (n <= 1024 ? 24 : 6) : m <= 128 ? (n <= 1024 ? 16 : 4) : 8;
  if (m <= 128) return n <= 1024 ? 24 : 8;
  return n <= 640 ? 24 : m <= 176 ? 12 : 4;
}

// CG steps in one workgroup (k_tiny.hip).
// Bytes of matrix and local inverses a step reads, at most.  Measured, in us a step
// against separate launches: 2-D p = 3, 0.29 MB 7.3 / 15.3, 0.74 MB 13.1 / 15.3;
// p = 4, 0.45 MB 10.8 / 16.2, 1.0 MB 20.4 / 16.1; 3-D p = 1, 0.72 MB 15.2 / 16.7;
// p = 2, 0.47 MB 11.9 / 19.5, 0.9 MB 19.6 / 19.8.
constexpr size_t kTinyBytes = size_t(768) << 10;
constexpr int kTinyThreads = 1024, kTinyElems = 4;   // unknowns per thread, at most
// LDS for p, q, r, z, the block outputs and one right-hand side a wave
inline size_t tiny_lds(int64_t n, int64_t n_blocks, int m) {
  return (4 * (size_t)n + (size_t)n_blocks * m + kTinyThreads) * sizeof(double);
}
inline bool tiny_sizes(int64_t nnz, int64_t n, int64_t n_blocks, int m) {
  const size_t inverses = (size_t)n_blocks * (m / 2 + 1) * m;
  return m <= 27 && n <= (int64_t)kTinyThreads * kTinyElems &&
         tiny_lds(n, n_blocks, m) <= 150 * 1024 &&
         ((size_t)nnz + inverses) * sizeof(double) <= kTinyBytes;
}

}  // namespace fc
