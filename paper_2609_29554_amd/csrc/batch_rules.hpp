// Rules of the batched Ozaki-II LU that hold no device code (constexpr, so the
// kernel and the host share them).
#pragma once
#include <stdint.h>

namespace ozb {

// Work left of a system of nc components with rem rows to go, for the helpers'
// choice: nc^2 rem^3 / 64, at least 1 (0 stands for no job) and below 2^29 for
// the orders up to 1024 that the batch takes.
constexpr uint32_t work_left(int nc, int64_t rem) {
  return (uint32_t)(((uint64_t)(nc * nc) * (uint64_t)(rem * rem * rem)) >> 6) + 1u;
}

}  // namespace ozb
