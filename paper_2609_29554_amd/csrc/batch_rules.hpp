// Rules of the batched Ozaki-II LU that hold no device code (constexpr, so the
// kernel and the host share them).
#pragma once
#include <stdint.h>

namespace ozb {

constexpr int NT = 512;           // threads per workgroup
constexpr int SB = 8;             // columns of a panel's sub-block when steps are deferred
constexpr int UCH = 32, ACH = 64; // columns of U12, rows of L21 of a task

// Whether the steps of a panel of rows x width elements are worth deferring: a
// small panel's are not worth a task.  With the line at 0 / 6 / 12 / 24 NT
// elements, 71 of order 36 to 58 take 1.46 / 1.31 / 1.31 / 1.31 ms, 16 of order
// 100 to 400 12.8 / 12.6 / 12.7 / 13.4, 100 of order 150 to 300 (b = 32) 11.9 /
// 11.7 / 11.4 / 11.7
constexpr bool worth_deferring(int64_t rows, int64_t width) { return rows * width >= 12 * NT; }

// The most tasks that a system of order n offers at a time (its first block's),
// 1 where it shares nothing: as many workgroups can work on it at once.
constexpr int64_t most_tasks(int64_t n, int64_t b) {
  const int64_t w = n < b ? n : b, m2 = n - w, tiles = (m2 + 63) / 64;
  int64_t t = 1;
  if (worth_deferring(n, w) && w > SB) t = ((n - SB) * (w - SB) + NT - 1) / NT;
  if (m2 > 64) {
    const int64_t t0 = tiles * 64 / UCH + tiles * 64 / ACH, t1 = tiles * tiles;
    t = t > t0 ? t : t0;
    t = t > t1 ? t : t1;
  }
  return t;
}

// Work left of a system of nc components with rem rows to go, for the helpers'
// choice: nc^2 rem^3 / 64, at least 1 (0 stands for no job) and below 2^29 for
// the orders up to 1024 that the batch takes.
constexpr uint32_t work_left(int nc, int64_t rem) {
  return (uint32_t)(((uint64_t)(nc * nc) * (uint64_t)(rem * rem * rem)) >> 6) + 1u;
}

}  // namespace ozb
