// Cross-lane primitives of one 64-lane wavefront: the vocabulary of the
// lane-distributed p-bit arithmetic in limbfp.hpp.  Every call must be made
// by all 64 lanes of a converged wavefront.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define LFP_FN __device__ __forceinline__

namespace lfp {

LFP_FN int lane_id() { return (int)__lane_id(); }

// bit l set when lane l's predicate holds
LFP_FN uint64_t ballot(bool p) { return (uint64_t)__builtin_amdgcn_ballot_w64(p); }

// 1 in the lanes whose bit of a wave-uniform mask is set
LFP_FN uint64_t lane_bit(uint64_t mask) {
  return __builtin_amdgcn_inverse_ballot_w64(mask) ? 1ull : 0ull;
}

// lane l's x, for a wave-uniform l
LFP_FN uint64_t readlane64(uint64_t x, int l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), l);
  return ((uint64_t)hi << 32) | lo;
}

// lane src's x (src in 0..63, any per-lane value)
LFP_FN uint64_t shfl64(uint64_t x, int src) {
  return (uint64_t)__shfl((unsigned long long)x, src, 64);
}

// a + b + cin (cin 0 or 1) on 32-bit words, the carry out in *cout
LFP_FN uint32_t addc32(uint32_t a, uint32_t b, uint32_t cin, uint32_t *cout) {
  unsigned c;
  const uint32_t r = __builtin_addc(a, b, cin, &c);
  *cout = c;
  return r;
}

// lane l's result is lane l-1's x, lane 0's is 0 (DPP whole-wave shift)
LFP_FN uint64_t up1_64(uint64_t x) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, 0x138, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), 0x138, 0xf,
                                                            0xf, false);
  return ((uint64_t)hi << 32) | lo;
}

// lane l's result is lane l+1's x, lane 63's is 0 (DPP whole-wave shift)
LFP_FN uint64_t dn1_64(uint64_t x) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, 0x130, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), 0x130, 0xf,
                                                            0xf, false);
  return ((uint64_t)hi << 32) | lo;
}

// up1_64 on a 32-bit word
LFP_FN uint32_t up1_32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x138, 0xf, 0xf, false);
}

// the high word of {hi, lo} >> s, s in 0..31
LFP_FN uint32_t align_bits(uint32_t hi, uint32_t lo, uint32_t s) {
  return __builtin_amdgcn_alignbit(hi, lo, s);
}

typedef int v4i32 __attribute__((ext_vector_type(4)));

// acc + A B on 16 x 64 by 64 x 16 signed bytes: lane l holds bytes 16 (l / 16)
// .. + 15 of row (column) l % 16 of A (B), and rows 4 (l / 16) .. + 3 of
// column l % 16 of the result
LFP_FN v4i32 mfma_bytes(v4i32 a, v4i32 b, v4i32 acc) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, acc, 0, 0, 0);
}

// orders this wavefront's LDS accesses before and after it
LFP_FN void lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// lane l's result is lane (l-1) mod 64's x (DPP whole-wave rotation)
LFP_FN uint64_t rot1_64(uint64_t x) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, 0x13C, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), 0x13C, 0xf,
                                                            0xf, false);
  return ((uint64_t)hi << 32) | lo;
}

}  // namespace lfp
