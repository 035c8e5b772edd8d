// Ozaki-II product on arbitrary-precision limb numbers (p = 64 nlimb bits,
// the MPFR-like input of Sec. 3.3 and the p-bit results of (S6)):
//   x = (-1)^sign * (sum_q limb_q 2^(64 q)) * 2^(exp - p),  mantissa normalised,
// stored as one plane per limb (limb q of element idx at limb[q*plane + idx]).
//
//   (S1) k_limb_exponents: e = max exp over the non-zero entries of a row of
//        A / a column of B (small products: in the producer);
//   (S2)+(S3) k_producer_limbs: X = sgn(x) trunc(|x| 2^mu) is never formed;
//        every w-bit slice window is read straight from the limb planes
//        (negative values as the complement plus an incoming carry of one)
//        and reduced by the byte residue emitter shared with the expansion
//        producer, so the residue planes have the same layout;
//   (S4) the batched INT8 modular GEMM of the expansion path;
//   (S5) k_consumer_limbs: the byte CRT of every digit group, added at bit
//        w gi into the exact group sum cbar, kept as a column of 32-bit words
//        per element in workspace (word k of element e at cw[k*E + e]): the
//        groups arrive in increasing order, so each one rewrites only its own
//        window and the sign extension above it is carried as a small integer;
//   (S6) c = RN_p(cbar 2^eps), ties to even, and in mode 1 C = RN_p(C - c):
//        k_limb_finish, or k_limb_round and k_limb_sub (the exact difference
//        on a grid with a guard word and a sticky bit, rounded once).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "ozii_bytes.hpp"
#include "ozii_elem.hpp"
#include "ozii_kernels.hpp"
#include "ozii_stage.hpp"
#include "lanes.hpp"
#include "limbfp.hpp"

using namespace ozk;
using ozl::LimbOperand;

namespace {

// exponent of the entry at idx (EXP_ZERO for zero)
__device__ __forceinline__ int32_t limb_exponent(const LimbOperand &X, int nlimb, int64_t idx) {
  return X.limb[(int64_t)(nlimb - 1) * X.plane + idx] != 0 ? X.lexp[idx] : EXP_ZERO;
}

// ---------------------------------------------------------------------------
// (S1), both operands in one launch as k_exponents of the expansion product:
// the first ga workgroups take rba rows of A each, the others rbb columns of B
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_limb_exponents(LimbOperand A, LimbOperand B, int nlimb,
                                                        int64_t K, int ga, int rba, int rbb) {
  __shared__ int32_t sm[64];
  const bool isa = (int)blockIdx.x < ga;
  const LimbOperand X = isa ? A : B;
  const int rb = isa ? rba : rbb;
  const int64_t o0 = (int64_t)(isa ? blockIdx.x : blockIdx.x - ga) * rb;
  const int64_t so = isa ? 1 : X.ld, sh = isa ? X.ld : 1;
  const int32_t v = block_exponents(
      [&](int64_t o, int64_t h) { return limb_exponent(X, nlimb, o * so + h * sh); }, isa, o0,
      X.nout, K, rb, sm);
  if ((int)threadIdx.x < rb && o0 + threadIdx.x < X.nout) X.exps[o0 + threadIdx.x] = v;
}

// ---------------------------------------------------------------------------
// (S2)+(S3).  Block layout as the expansion producer: one workgroup fills
// one 1 KiB block (16 rows x 64 k) of every residue plane; thread T owns
// row (T/4)%16 and the four inner indices 16(T/64) + 4(T%4) + e.
// Element with mantissa m, exponent ex and shift s = ex - p + mu:
// |X| = trunc(m 2^s), so bit b of |X| is bit b - s of m.  The slice chain
// (carry c_t, centring flag) is that of the expansion producer; a negative
// X = ~|X| + 1 starts with c_0 = 1 and complemented windows.
// ---------------------------------------------------------------------------
// Binary64 moduli: the residues of slice t of the thread's four elements as
// doubles for the moduli l0 .. l1-1 (pp at the plane of modulus l0), in the
// binary64 GEMM's fragment order (1 KiB blocks of 16 rows x 8 k, lane l: row
// l%16, k l/16 and 4 + l/16; eight blocks per 64-k window; off: each
// element's offset in a plane).  F and sel as for the byte
// emitter: a lower slice has the value F - sel 2^w (F < 2^w), the top slice
// is the nwt-word two's complement F with sign sel; its magnitude is reduced
// and the residue negated.
template <int NWM>
__device__ __forceinline__ void emit_f64_residues(const uint32_t (&F)[4][NWM],
                                                  const uint32_t (&sel)[4], bool top, int nwt,
                                                  const DevPlan *__restrict__ pl, int l0, int l1,
                                                  double *pp, int64_t plane_elems,
                                                  const int64_t (&off)[4]) {
  constexpr int NH = 2 * NWM;
  static_assert(NH <= NHMAX, "slice digits");
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t mag[NWM];
    const bool neg = top && sel[e] != 0;
    uint32_t c = 1;
#pragma unroll
    for (int k = 0; k < NWM; ++k) {
      if (top && k >= nwt) {
        mag[k] = 0u;
      } else if (neg) {
        const uint32_t v = ~F[e][k];
        mag[k] = v + c;
        c = (c && mag[k] == 0u) ? 1u : 0u;
      } else {
        mag[k] = F[e][k];
      }
    }
    uint32_t dig[NH];
#pragma unroll
    for (int k = 0; k < NH; ++k) dig[k] = (mag[k >> 1] >> (16 * (k & 1))) & 0xffffu;
    const bool flag = !top && sel[e] != 0;
    for (int l = l0; l < l1; ++l) {
      const uint32_t m = (uint32_t)pl->m[l];
      uint32_t r = digits_mod<NH, true>(dig, pl, l);
      if (flag) {
        r += m - pl->p2w[l];  // F - 2^w (mod m)
        r = r >= m ? r - m : r;
      } else if (neg) {
        r = r == 0u ? 0u : m - r;
      }
      pp[(int64_t)(l - l0) * plane_elems + off[e]] = (double)centre(r, (int32_t)m);
    }
  }
}

template <int NWM, bool F64, bool OWN>
__global__ __launch_bounds__(256) void k_producer_limbs(LimbOperand A, LimbOperand B, int nlimb,
                                                        int64_t K, int64_t KB, int oba,
                                                        const DevPlan *__restrict__ pl) {
  constexpr int NLL = (NWM + 3) / 2;  // limbs covering NWM + 2 words
  const int T = threadIdx.x;
  const uint32_t oy = blockIdx.x / (uint32_t)KB;
  const bool isa = (int)oy < oba;
  const LimbOperand X = isa ? A : B;
  const uint64_t *__restrict__ limb = X.limb;
  const int64_t ld = X.ld, plane = X.plane, nout = X.nout, plane_elems = X.plane_elems;
  uint8_t *planes = (uint8_t *)X.planes;
  const int64_t kb = blockIdx.x - oy * (uint32_t)KB, ob = isa ? oy : oy - oba;
  const int64_t o = ob * 16 + ((T >> 2) & 15);
  const int64_t h0 = kb * 64 + 16 * (T >> 6) + 4 * (T & 3);
  const uint32_t offb = (uint32_t)((ob * KB + kb) * 1024 + 4 * T);  // < 2^31
  const int S = pl->S, w = pl->w, nmod = pl->nmod, Q = pl->Q, nwt = pl->nwt;
  const int p = 64 * nlimb;
  // blockIdx.z: a part of the moduli (small products run several parts)
  const int l0 = (int)blockIdx.z * nmod / (int)gridDim.z;
  const int l1 = ((int)blockIdx.z + 1) * nmod / (int)gridDim.z;

  int32_t ex = EXP_ZERO;
  if constexpr (OWN) {
    // the workgroup finds the exponents of its 16 outputs itself
    __shared__ int32_t sm[64], sex[16];
    const int64_t so = isa ? 1 : ld, sh_ = isa ? ld : 1;
    const int32_t v = block_exponents(
        [&](int64_t oo, int64_t h) { return limb_exponent(X, nlimb, oo * so + h * sh_); }, isa,
        ob * 16, nout, K, 16, sm);
    if (T < 16) {
      sex[T] = v;
      if (kb == 0 && blockIdx.z == 0 && ob * 16 + T < nout) X.exps[ob * 16 + T] = v;
    }
    __syncthreads();
    if (o < nout) ex = sex[(T >> 2) & 15];
  } else {
    if (o < nout) ex = X.exps[o];
  }
  int64_t idx[4];
  int32_t sh[4];
  uint32_t neg[4], live[4], cin[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    idx[e] = 0;
    sh[e] = 0;
    neg[e] = 0;
    live[e] = 0;
    const int64_t h = h0 + e;
    if (ex != EXP_ZERO && h < K) {
      const int64_t id = isa ? o + h * ld : h + o * ld;
      if (limb[(int64_t)(nlimb - 1) * plane + id] != 0) {
        const int64_t s = (int64_t)X.lexp[id] - p + (Q - 1 - (int64_t)ex);
        // below -(p + 64) every bit of the value is truncated away
        if (s > -(int64_t)(p + 64)) {
          live[e] = 1;
          sh[e] = (int32_t)s;
          idx[e] = id;
          neg[e] = X.lsign[id] & 1u;
        }
      }
    }
    cin[e] = neg[e];
  }
  for (int t = 0; t < S; ++t) {
    const bool top = t == S - 1;
    const int wq = w >> 5, wb = w & 31;
    uint32_t F[4][NWM];
    uint32_t sel[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (live[e]) {
        const int32_t pos0 = t * w - sh[e];  // mantissa bit of the window's bit 0
        const int32_t q0 = pos0 >> 6, r0 = pos0 & 63;
        uint32_t u[2 * NLL];
#pragma unroll
        for (int k = 0; k < NLL; ++k) {
          const int32_t q = q0 + k;
          const uint64_t v = (q >= 0 && q < nlimb) ? limb[(int64_t)q * plane + idx[e]] : 0ull;
          u[2 * k] = (uint32_t)v;
          u[2 * k + 1] = (uint32_t)(v >> 32);
        }
        const bool hi = (r0 >> 5) != 0;
        const uint32_t rb = (uint32_t)(r0 & 31);
#pragma unroll
        for (int j = 0; j < NWM; ++j) {
          const uint32_t a = hi ? u[j + 1] : u[j];
          const uint32_t b = hi ? u[j + 2] : u[j + 1];
          const uint32_t v = __builtin_amdgcn_alignbit(b, a, rb);
          F[e][j] = neg[e] ? ~v : v;
        }
      } else {
#pragma unroll
        for (int j = 0; j < NWM; ++j) F[e][j] = 0u;
      }
      if (!top) {
#pragma unroll
        for (int j = 0; j < NWM; ++j)
          F[e][j] = j < wq ? F[e][j] : (j == wq ? F[e][j] & ((1u << wb) - 1u) : 0u);
      }
      uint32_t c = cin[e];
#pragma unroll
      for (int j = 0; j < NWM; ++j) {
        const uint32_t sum = F[e][j] + c;
        c = sum < c ? 1u : 0u;
        F[e][j] = sum;
      }
      if (!top) {
        uint32_t co = 0, fl = 0;
        const int fq = (w - 1) >> 5, fb = (w - 1) & 31;
#pragma unroll
        for (int j = 0; j < NWM; ++j) {
          if (j == wq) {
            co = (F[e][j] >> wb) & 1u;
            F[e][j] &= ~(1u << wb);
          }
        }
#pragma unroll
        for (int j = 0; j < NWM; ++j)
          if (j == fq) fl = (F[e][j] >> fb) & 1u;
        sel[e] = fl;
        cin[e] = co + fl;
      } else {
        uint32_t sg = 0;
#pragma unroll
        for (int j = 0; j < NWM; ++j)
          if (j == nwt - 1) sg = F[e][j] >> 31;
        sel[e] = sg;
      }
    }
    if constexpr (F64) {
      int64_t off[4];
      const int r = (T >> 2) & 15;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int kk = 16 * (T >> 6) + 4 * (T & 3) + e, k8 = kk & 7;
        off[e] = ((ob * KB + kb) * 8 + (kk >> 3)) * 128 + 2 * ((k8 & 3) * 16 + r) + (k8 >> 2);
      }
      emit_f64_residues<NWM>(F, sel, top, nwt, pl, l0, l1,
                             (double *)planes + ((int64_t)t * nmod + l0) * plane_elems,
                             plane_elems, off);
    } else {
      emit_byte_residues<NWM, false>(F, sel, top ? REC_HT : REC_HW, pl, l0, l1,
                                     planes + ((int64_t)t * nmod + l0) * plane_elems, plane_elems,
                                     offb);
    }
  }
}

// ---------------------------------------------------------------------------
// (S5) on the binary64 moduli: cbar = sum_gi Sbar_(g0+gi) 2^(w gi) per
// element, words in cw.
// Invariant after each group: cbar = sum_(k < hw) cw[k] 2^(32k) + pend 2^(32 hw)
// with hw uniform.  Group gi adds V = Sbar 2^(b0) (nvw words, sign-extended
// by fill) at word q0 = floor(w gi / 32).  After the last group the final
// pend (0 or -1, the sign) is stored at word hw.
// ---------------------------------------------------------------------------
template <int ND>
__global__ __launch_bounds__(256) void k_consumer_limbs(const uint32_t *__restrict__ tpl,
                                                        int64_t Mp, int64_t Np, int64_t M,
                                                        int64_t N, const DevPlan *__restrict__ pl,
                                                        int nvw, uint32_t *__restrict__ cw,
                                                        int64_t E) {
  constexpr int NV = ND / 2 + 1;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t j = blockIdx.y;
  if (i >= M || j >= N) return;
  const int64_t e = i + j * M;
  const int nmod = pl->nmod, w = pl->w, ng = pl->ng;
  const int64_t ps = Np * Mp;
  uint32_t *col = cw + e;
  auto AT = [&](int k) -> uint32_t & { return col[(int64_t)k * E]; };
  int hw = 0;
  int32_t pend = 0;
  for (int gi = 0; gi < ng; ++gi) {
    int32_t d[ND];
    crt_digits<ND, uint32_t>(tpl + ((int64_t)gi * nmod * Np + j) * Mp + i, ps, pl, d);
    const uint32_t fill = d[ND - 1] < 0 ? 0xffffffffu : 0u;
    uint32_t st[ND / 2];
#pragma unroll
    for (int k = 0; k < ND / 2; ++k)
      st[k] = ((uint32_t)d[2 * k] & 0xffffu) | ((uint32_t)d[2 * k + 1] << 16);
    const int off = w * gi, q0 = off >> 5, b0 = off & 31;
    const uint32_t pext = pend < 0 ? 0xffffffffu : 0u;
    // a gap below the window holds the old value's extension
    for (int k = hw; k < q0; ++k) AT(k) = k == hw ? (uint32_t)pend : pext;
    if (q0 > hw) {
      hw = q0;
      pend = pend < 0 ? -1 : 0;
    }
    const uint32_t ext = pend < 0 ? 0xffffffffu : 0u;
    uint32_t carry = 0;
#pragma unroll
    for (int r = 0; r < NV; ++r) {
      if (r < nvw) {
        const int k = q0 + r;
        const uint32_t cur = r < ND / 2 ? st[r] : fill;
        const uint32_t prv = r == 0 ? 0u : (r - 1 < ND / 2 ? st[r - 1] : fill);
        const uint32_t v = b0 ? ((cur << b0) | (prv >> (32 - b0))) : cur;
        const uint32_t old = k < hw ? AT(k) : (k == hw ? (uint32_t)pend : ext);
        const uint64_t s = (uint64_t)old + v + carry;
        AT(k) = (uint32_t)s;
        carry = (uint32_t)(s >> 32);
      }
    }
    // old words above the window still take the extension of V
    for (int k = q0 + nvw; k <= hw; ++k) {
      const uint32_t old = k < hw ? AT(k) : (uint32_t)pend;
      const uint64_t s = (uint64_t)old + fill + carry;
      AT(k) = (uint32_t)s;
      carry = (uint32_t)(s >> 32);
    }
    const int kend = q0 + nvw > hw + 1 ? q0 + nvw : hw + 1;
    pend = (int32_t)carry + (pend < 0 ? -1 : 0) + (fill ? -1 : 0);
    hw = kend;
  }
  AT(hw) = (uint32_t)pend;
}

// ---------------------------------------------------------------------------
// (S5) on the byte back-ends, one wavefront per 64 consecutive elements of a
// column: the digits of each group come from the matrix-core CRT of the
// expansion consumer, and the sum slides through a window of NR registers.
// Group gi adds Sbar 2^(w gi mod 32) at the window's word 0, which stands for
// word q = floor(w gi / 32); the words below the next group's q are final and
// leave the window, each stored once.  |Sbar| < 2^(16 ND - 1), the shift is
// below 32 and the earlier groups add less than one more bit, so 32 NR >= 16
// ND + 64 bits hold the two's complement sum.  Bound by the CRT's integer
// work and the t-planes.  p = 4096, 768 x 768 outputs: dot-product CRT and
// a sum in memory, read and rewritten by every group, 883 us -> 591 us.
// ---------------------------------------------------------------------------
template <int ND>
__global__ __launch_bounds__(64) void k_consumer_limbs_mx(const uint8_t *__restrict__ tpl,
                                                          int64_t Mp, int64_t Np, int64_t M,
                                                          int64_t N,
                                                          const DevPlan *__restrict__ pl,
                                                          uint32_t *__restrict__ cw, int64_t E) {
  constexpr int NR = ND / 2 + 2;
  __shared__ __attribute__((aligned(16))) int32_t buf[32 * MX_CBS];
  const int lane = (int)threadIdx.x;
  int64_t bx, j;
  xcd_block(bx, j);
  const int64_t i0 = bx * 64, i = i0 + lane;
  const int nmod = pl->nmod, w = pl->w, ng = pl->ng;
  mxv4 tab[MX_BLK];
#pragma unroll
  for (int b = 0; b < MX_BLK; ++b) tab[b] = *(const mxv4 *)&pl->crtm[b][lane][0];
  const bool valid = i < M;
  uint32_t *col = cw + (valid ? i + j * M : 0);
  const int64_t ps = Np * Mp;
  uint32_t win[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) win[k] = 0u;
  int q0 = 0;
  for (int gi = 0; gi < ng; ++gi) {
    int32_t d[ND];
    crt_group_mx<2 * ND>(tpl + (int64_t)gi * nmod * ps + j * Mp + i0, ps, nmod, pl, tab, buf, lane, d);
    const uint32_t fill = d[ND - 1] < 0 ? 0xffffffffu : 0u;
    const uint32_t b0 = (uint32_t)(w * gi) & 31u;
    uint32_t prev = 0u, carry = 0u;
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const uint32_t cur = k < ND / 2 ? ((uint32_t)d[2 * k < ND ? 2 * k : 0] & 0xffffu) |
                                            ((uint32_t)d[2 * k < ND ? 2 * k + 1 : 0] << 16)
                                      : fill;
      const uint32_t v = b0 ? __builtin_amdgcn_alignbit(cur, prev, 32u - b0) : cur;
      unsigned co;
      win[k] = __builtin_addc(win[k], v, carry, &co);
      carry = co;
      prev = cur;
    }
    const int qn = gi + 1 < ng ? (w * (gi + 1)) >> 5 : q0 + NR;
    for (; q0 < qn; ++q0) {
      if (valid) col[(int64_t)q0 * E] = win[0];
      const uint32_t sg = (uint32_t)((int32_t)win[NR - 1] >> 31);
#pragma unroll
      for (int k = 0; k + 1 < NR; ++k) win[k] = win[k + 1];
      win[NR - 1] = sg;
    }
  }
}

// ---------------------------------------------------------------------------
// RN_p of a non-negative integer given word by word (MAG(k), zero outside
// [0, nw)) times 2^escale, with an extra sticky bit below everything; writes
// limbs, exponent and sign of the p-bit result (zero for a zero magnitude).
// ---------------------------------------------------------------------------
template <class MagF>
__device__ __forceinline__ void round_to_limbs(MagF MAG, int nw, bool sticky_in, int nlimb,
                                               int64_t escale, uint32_t sign, uint64_t *olimb,
                                               int64_t oplane, int64_t oi, int32_t *oexp,
                                               uint8_t *osign) {
  const int p = 64 * nlimb, pw = 2 * nlimb;
  int tw = -1;
  for (int k = nw - 1; k >= 0; --k) {
    if (MAG(k) != 0u) {
      tw = k;
      break;
    }
  }
  if (tw < 0) {
    for (int q = 0; q < nlimb; ++q) olimb[(int64_t)q * oplane + oi] = 0ull;
    oexp[oi] = EXP_ZERO;
    osign[oi] = 0;
    return;
  }
  const int L = 32 * tw + 32 - __builtin_clz(MAG(tw));
  const int sh = L - p;
  auto BITS = [&](int pos) -> uint32_t {  // bits [pos, pos + 32) of the magnitude
    const int q = pos >> 5, r = pos & 31;
    const uint32_t lo = MAG(q);
    return r ? (lo >> r) | (MAG(q + 1) << (32 - r)) : lo;
  };
  bool up = false;
  if (sh > 0) {
    const int rp = sh - 1;  // round bit position
    const uint32_t rb = (MAG(rp >> 5) >> (rp & 31)) & 1u;
    bool sticky = sticky_in || (MAG(rp >> 5) & ((1u << (rp & 31)) - 1u)) != 0u;
    for (int k = 0; k < (rp >> 5) && !sticky; ++k) sticky = MAG(k) != 0u;
    up = rb && (sticky || (BITS(sh) & 1u));
  }
  // an increment carries through the low mantissa words equal to all ones
  int f = 0;
  bool over = false;
  if (up) {
    f = -1;
    for (int m = 0; m < pw; ++m) {
      if (BITS(sh + 32 * m) != 0xffffffffu) {
        f = m;
        break;
      }
    }
    over = f < 0;
  }
  auto WORD = [&](int m) -> uint32_t {
    if (over) return m == pw - 1 ? 0x80000000u : 0u;
    const uint32_t raw = BITS(sh + 32 * m);
    if (!up || m > f) return raw;
    return m < f ? 0u : raw + 1u;
  };
  for (int q = 0; q < nlimb; ++q)
    olimb[(int64_t)q * oplane + oi] = ((uint64_t)WORD(2 * q + 1) << 32) | WORD(2 * q);
  oexp[oi] = (int32_t)(L + (over ? 1 : 0) + escale);
  osign[oi] = (uint8_t)sign;
}

// ---------------------------------------------------------------------------
// (S6): c = RN_p(cbar 2^eps), eps = w g0 - mu_i - nu_j, written as a limb
// matrix (ldo, planeo).  cbar is the two's complement column of nwords words
// (the top one the sign); its magnitude is read on demand: for a negative
// cbar, word k of -cbar is 0 below the lowest non-zero word z, -c_z at z and
// ~c_k above.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_limb_round(const uint32_t *__restrict__ cw, int64_t E,
                                                    int nwords, int64_t M, int64_t N,
                                                    const int32_t *__restrict__ ea,
                                                    const int32_t *__restrict__ eb, int w, int g0,
                                                    int Q, int nlimb, uint64_t *__restrict__ olimb,
                                                    int32_t *__restrict__ oexp,
                                                    uint8_t *__restrict__ osign, int64_t ldo,
                                                    int64_t planeo) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t j = blockIdx.y;
  if (i >= M || j >= N) return;
  const int64_t oi = i + j * ldo;
  const int32_t ei = ea[i], ej = eb[j];
  const uint32_t *col = cw + (i + j * M);
  auto C = [&](int k) -> uint32_t { return col[(int64_t)k * E]; };
  if (ei == EXP_ZERO || ej == EXP_ZERO) {
    round_to_limbs([](int) { return 0u; }, 0, false, nlimb, 0, 0, olimb, planeo, oi, oexp, osign);
    return;
  }
  const uint32_t neg = C(nwords - 1) >> 31;
  int z = nwords;
  if (neg) {
    for (int k = 0; k < nwords; ++k) {
      if (C(k) != 0u) {
        z = k;
        break;
      }
    }
  }
  auto MAG = [&](int k) -> uint32_t {
    if (k < 0 || k >= nwords) return 0u;
    const uint32_t v = C(k);
    if (!neg) return v;
    return k < z ? 0u : (k == z ? 0u - v : ~v);
  };
  const int64_t eps = (int64_t)w * g0 - (Q - 1 - (int64_t)ei) - (Q - 1 - (int64_t)ej);
  round_to_limbs(MAG, nwords, false, nlimb, eps, neg, olimb, planeo, oi, oexp, osign);
}

// ---------------------------------------------------------------------------
// Update: C = RN_p(C - T) for p-bit limb matrices C (ldc, planec) and T
// (M x N, ld M, plane M N).  With X the operand of larger magnitude and Y
// the other, the difference is formed on the grid of X's mantissa shifted up
// by one guard word: D_m = X_(m-1) +- (bits 32(m-1) + d .. of Y), d =
// exp(X) - exp(Y); bits of Y below the grid only set a sticky bit (for a
// subtraction they lower D by one unit first, so D + sticky brackets the
// exact value).  D (pw + 2 words per element) is written to dw, then
// rounded once.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_limb_sub(uint64_t *__restrict__ climb,
                                                  int32_t *__restrict__ cexp,
                                                  uint8_t *__restrict__ csign, int64_t ldc,
                                                  int64_t planec, const uint64_t *__restrict__ tlimb,
                                                  const int32_t *__restrict__ texp,
                                                  const uint8_t *__restrict__ tsign, int nlimb,
                                                  int64_t M, int64_t N, uint32_t *__restrict__ dw,
                                                  int64_t E) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t j = blockIdx.y;
  if (i >= M || j >= N) return;
  const int p = 64 * nlimb, pw = 2 * nlimb, nwd = pw + 2;
  const int64_t ci = i + j * ldc, ti = i + j * M, planet = M * N;
  const bool tz = tlimb[(int64_t)(nlimb - 1) * planet + ti] == 0ull;
  if (tz) return;  // C - 0 = C exactly
  const bool az = climb[(int64_t)(nlimb - 1) * planec + ci] == 0ull;
  const uint32_t sa = csign[ci] & 1u, sc = (tsign[ti] & 1u) ^ 1u;  // C + (-T)
  if (az) {
    for (int q = 0; q < nlimb; ++q)
      climb[(int64_t)q * planec + ci] = tlimb[(int64_t)q * planet + ti];
    cexp[ci] = texp[ti];
    csign[ci] = (uint8_t)sc;
    return;
  }
  auto CW = [&](int m) -> uint32_t {  // mantissa word m of C
    const uint64_t v = climb[(int64_t)(m >> 1) * planec + ci];
    return (m & 1) ? (uint32_t)(v >> 32) : (uint32_t)v;
  };
  auto TW = [&](int m) -> uint32_t {
    const uint64_t v = tlimb[(int64_t)(m >> 1) * planet + ti];
    return (m & 1) ? (uint32_t)(v >> 32) : (uint32_t)v;
  };
  const int32_t xa = cexp[ci], xt = texp[ti];
  bool cx = xa > xt;  // C is X
  if (xa == xt) {
    cx = true;
    for (int m = pw - 1; m >= 0; --m) {
      const uint32_t a = CW(m), b = TW(m);
      if (a != b) {
        cx = a > b;
        break;
      }
    }
  }
  const int64_t d = cx ? (int64_t)xa - xt : (int64_t)xt - xa;
  const uint32_t sx = cx ? sa : sc, sy = cx ? sc : sa;
  const bool sub = sx != sy;
  auto XW = [&](int m) -> uint32_t { return cx ? CW(m) : TW(m); };
  auto YW = [&](int m) -> uint32_t {
    if (m < 0 || m >= pw) return 0u;
    return cx ? TW(m) : CW(m);
  };
  auto YB = [&](int64_t pos) -> uint32_t {  // bits [pos, pos + 32) of Y's mantissa
    if (pos >= p || pos <= -32) return 0u;
    const int q = (int)(pos >> 5), r = (int)(pos & 31);
    const uint32_t lo = YW(q);
    return r ? (lo >> r) | (YW(q + 1) << (32 - r)) : lo;
  };
  // bits of Y below position d - 32 fall below the grid
  bool sticky = false;
  if (d > 32) {
    const int64_t nb = d - 32 < p ? d - 32 : p;
    const int full = (int)(nb >> 5), part = (int)(nb & 31);
    for (int k = 0; k < full && !sticky; ++k) sticky = YW(k) != 0u;
    if (!sticky && part) sticky = (YW(full) & ((1u << part) - 1u)) != 0u;
  }
  uint32_t *dcol = dw + ti;
  auto DAT = [&](int k) -> uint32_t & { return dcol[(int64_t)k * E]; };
  uint32_t cb = sub && sticky ? 1u : 0u;  // carry (add) or borrow (sub)
  for (int m = 0; m < nwd; ++m) {
    const uint32_t xg = (m >= 1 && m <= pw) ? XW(m - 1) : 0u;
    const uint32_t yg = YB((int64_t)32 * (m - 1) + d);
    if (!sub) {
      const uint64_t s = (uint64_t)xg + yg + cb;
      DAT(m) = (uint32_t)s;
      cb = (uint32_t)(s >> 32);
    } else {
      const uint64_t s = (uint64_t)xg - yg - cb;
      DAT(m) = (uint32_t)s;
      cb = (uint32_t)((s >> 63) & 1u);
    }
  }
  auto DM = [&](int k) -> uint32_t { return (k < 0 || k >= nwd) ? 0u : DAT(k); };
  const int32_t ex = cx ? xa : xt;
  round_to_limbs(DM, nwd, sticky, nlimb, (int64_t)ex - p - 32, sx, climb, planec, ci, cexp, csign);
}

// ---------------------------------------------------------------------------
// (S6) and the update in one pass, nl <= 64: c = RN_p(cbar 2^eps), then C = c
// (mode 0) or C = RN_p(C - c) (mode 1), in the lane-distributed arithmetic of
// limbfp.hpp.  A workgroup takes FE consecutive elements of a column: the
// sum's words and C's limbs come in whole lines, plane by plane, and are
// turned in LDS so that a wavefront has one element with a limb per lane; the
// results leave the same way.  Reads and writes everything once.  p = 4096,
// 768 x 768 update: rounding into a temporary, then a subtraction through a
// second one, 934 us -> 422 us.
// ---------------------------------------------------------------------------
constexpr int FE = 32;
__global__ __launch_bounds__(256) void k_limb_finish(
    const uint32_t *__restrict__ cw, int64_t E, int nwords, int64_t M, const int32_t *__restrict__ ea,
    const int32_t *__restrict__ eb, int w, int g0, int Q, int nl, int mode, uint64_t *climb,
    int32_t *cexp, uint8_t *csign, int64_t ldc, int64_t planec) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int ws = nwords | 1, ls = nl | 1;  // odd strides
  uint64_t *sc = (uint64_t *)smem_raw;     // FE * ls limbs
  int32_t *sx = (int32_t *)(sc + FE * ls);  // exponents
  int32_t *ss = sx + FE;                    // signs
  uint32_t *sw = (uint32_t *)(ss + FE);     // FE * ws words
  const int t = threadIdx.x, wv = t >> 6, l = lfp::lane_id();
  const int64_t i0 = (int64_t)blockIdx.x * FE, j = blockIdx.y;
  const int cnt = (int)(M - i0 < FE ? M - i0 : FE);
  const int e0 = t & (FE - 1), k0 = t / FE;
  const uint32_t *src = cw + i0 + e0 + j * M;
  const int64_t ci = i0 + e0 + j * ldc;
  if (e0 < cnt) {
#pragma unroll 8
    for (int k = k0; k < nwords; k += 256 / FE) sw[e0 * ws + k] = src[(int64_t)k * E];
    if (mode) {
#pragma unroll 8
      for (int q = k0; q < nl; q += 256 / FE) sc[e0 * ls + q] = climb[(int64_t)q * planec + ci];
      if (k0 == 0) {
        sx[e0] = cexp[ci];
        ss[e0] = csign[ci];
      }
    }
  }
  __syncthreads();
  const int32_t ej = eb[j];
  for (int e = wv; e < cnt; e += 4) {
    const int32_t ei = ea[i0 + e];
    const uint32_t *we = sw + e * ws;
    const uint32_t sign = __builtin_amdgcn_readfirstlane((int)we[nwords - 1]) < 0 ? 1u : 0u;
    const uint32_t ext = sign ? 0xffffffffu : 0u;
    auto limb = [&](int q) -> uint64_t {
      const int k = 2 * q;
      const uint32_t a = k < nwords ? we[k] : ext, b = k + 1 < nwords ? we[k + 1] : ext;
      return ((uint64_t)b << 32) | a;
    };
    lfp::W2 v;
    v.lo = limb(l);
    v.hi = limb(l + 64);
    if (sign) {
      lfp::W2 z;
      z.lo = 0;
      z.hi = 0;
      v.lo = ~v.lo;
      v.hi = ~v.hi;
      uint32_t co;
      v = lfp::add2(v, z, 1u, co);
    }
    lfp::WF r = lfp::wf_zero();
    if (ei != EXP_ZERO && ej != EXP_ZERO && lfp::ballot((v.lo | v.hi) != 0) != 0) {
      const int64_t eps = (int64_t)w * g0 - (Q - 1 - (int64_t)ei) - (Q - 1 - (int64_t)ej);
      int64_t bl;
      r.m = lfp::round_win(v, 0u, nl, bl);
      r.e = (int32_t)(bl + eps);
      r.s = sign;
    }
    if (mode) {
      // C - 0 leaves C as it is
      if (lfp::is_zero(r)) continue;
      lfp::WF c;
      c.m = l < nl ? sc[e * ls + l] : 0ull;
      c.e = __builtin_amdgcn_readfirstlane(sx[e]);
      c.s = (uint32_t)__builtin_amdgcn_readfirstlane(ss[e]) & 1u;
      if (!(lfp::ballot(c.m != 0) >> (nl - 1))) c = lfp::wf_zero();  // top limb 0
      r = lfp::add(c, r, 1u, nl);
    }
    if (l < nl) sc[e * ls + l] = r.m;
    if (l == 0) {
      sx[e] = r.e;
      ss[e] = (int32_t)r.s;
    }
  }
  __syncthreads();
  if (e0 < cnt) {
    for (int q = k0; q < nl; q += 256 / FE) climb[(int64_t)q * planec + ci] = sc[e0 * ls + q];
    if (k0 == 0) {
      cexp[ci] = sx[e0];
      csign[ci] = (uint8_t)ss[e0];
    }
  }
}

__global__ void k_limb_zero(uint64_t *limb, int32_t *lexp, uint8_t *lsign, int64_t ld,
                            int64_t plane, int nlimb, int64_t M, int64_t N) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t j = blockIdx.y;
  if (i >= M || j >= N) return;
  const int64_t idx = i + j * ld;
  for (int q = 0; q < nlimb; ++q) limb[(int64_t)q * plane + idx] = 0ull;
  lexp[idx] = EXP_ZERO;
  lsign[idx] = 0;
}

}  // namespace

namespace ozl {

hipError_t launch_limb_exponents(const LimbOperand &A, const LimbOperand &B, int nlimb, int64_t K,
                                 hipStream_t s) {
  if (A.nout <= 0 && B.nout <= 0) return hipSuccess;
  const int rba = exponent_rb(A.nout), rbb = exponent_rb(B.nout);
  const int64_t ga = (A.nout + rba - 1) / rba, gb = (B.nout + rbb - 1) / rbb;
  hipLaunchKernelGGL(k_limb_exponents, dim3((unsigned)(ga + gb)), dim3(256), 0, s, A, B, nlimb, K,
                     (int)ga, rba, rbb);
  return hipGetLastError();
}

// Grid of the limb producer over both operands: KB (OBA + OBB) blocks, and
// the moduli split over up to 8 parts while the blocks alone give fewer than
// 4096 wavefronts (four per SIMD).  own: small products find their exponents
// in the producer; the scans touch a limb and an exponent per element.
struct LProdGrid {
  int64_t KB, OBA;
  dim3 g;
  bool own;
};
static LProdGrid lprod_grid(const LimbOperand &A, const LimbOperand &B, int64_t K, int64_t Kp,
                            int nmod) {
  LProdGrid r{};
  r.KB = Kp / 64;
  r.OBA = A.noutp / 16;
  const int64_t nb = r.KB * (r.OBA + B.noutp / 16);
  r.g = dim3((unsigned)nb, 1, (unsigned)std::max<int64_t>(1, std::min<int64_t>({8, (int64_t)nmod,
                                                                   (4096 + 4 * nb - 1) / (4 * nb)})));
  r.own = nb * (int64_t)r.g.z * 16 * K * 12 <= OWN_EXP_BYTES;
  return r;
}

bool producer_limbs_owns_exponents(const LimbOperand &A, const LimbOperand &B, int64_t K,
                                   int64_t Kp, int nmod) {
  return lprod_grid(A, B, K, Kp, nmod).own;
}

template <bool F64, bool OWN>
static void producer_limbs_nw(int nwt, const LProdGrid &G, hipStream_t s, const LimbOperand &A,
                              const LimbOperand &B, int nlimb, int64_t K, const DevPlan *pl) {
#define OZ_PRODL(NWM_)                                                                             \
  hipLaunchKernelGGL((k_producer_limbs<NWM_, F64, OWN>), G.g, dim3(256), 0, s, A, B, nlimb, K, \
                     G.KB, (int)G.OBA, pl)
  if (nwt <= 4) OZ_PRODL(4);
  else if (nwt <= 6) OZ_PRODL(6);
  else OZ_PRODL(REC_PWMAX);
#undef OZ_PRODL
}

hipError_t launch_producer_limbs(const LimbOperand &A, const LimbOperand &B, int nlimb, int64_t K,
                                 int64_t Kp, const DevPlan *pl, int nmod, int nwt, int kind,
                                 hipStream_t s) {
  if (Kp < 64 || A.noutp + B.noutp < 16) return hipSuccess;
  if (std::max(A.plane_elems, B.plane_elems) >= ((int64_t)1 << 31) || nwt > REC_PWMAX)
    return hipErrorInvalidValue;
  if (kind != PLANES_I8 && kind != PLANES_F64) return hipErrorInvalidValue;
  const LProdGrid G = lprod_grid(A, B, K, Kp, nmod);
  if (kind == PLANES_F64) {
    if (G.own) producer_limbs_nw<true, true>(nwt, G, s, A, B, nlimb, K, pl);
    else producer_limbs_nw<true, false>(nwt, G, s, A, B, nlimb, K, pl);
  } else {
    if (G.own) producer_limbs_nw<false, true>(nwt, G, s, A, B, nlimb, K, pl);
    else producer_limbs_nw<false, false>(nwt, G, s, A, B, nlimb, K, pl);
  }
  return hipGetLastError();
}

int limb_sum_words(int nd, int tbytes, int w, int ng, int nvw_words) {
  if (tbytes != 1) return nvw_words;
  return ((w * (ng - 1)) >> 5) + (nd <= 18 ? 18 : 24) / 2 + 2;
}

hipError_t launch_consumer_limbs(const void *tpl, int tbytes, int64_t Mp, int64_t Np, int64_t M,
                                 int64_t N, const DevPlan *pl, int nd, int nvw, uint32_t *cw,
                                 hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const int ndc = nd <= 18 ? 18 : (nd <= 24 ? 24 : 32);
  if (nd > 32 || (tbytes == 1 && nd > 24) || (tbytes != 1 && tbytes != 4)) return hipErrorInvalidValue;
  if (tbytes == 1) {
    // 64-element wavefronts read whole plane rows
    if ((M + 63) / 64 * 64 > Mp) return hipErrorInvalidValue;
    const dim3 gx((unsigned)((M + 63) / 64), (unsigned)N);
    if (ndc == 18)
      hipLaunchKernelGGL(k_consumer_limbs_mx<18>, gx, dim3(64), 0, s, (const uint8_t *)tpl, Mp, Np, M,
                         N, pl, cw, M * N);
    else
      hipLaunchKernelGGL(k_consumer_limbs_mx<24>, gx, dim3(64), 0, s, (const uint8_t *)tpl, Mp, Np, M,
                         N, pl, cw, M * N);
    return hipGetLastError();
  }
  if (nvw > ndc / 2 + 1) return hipErrorInvalidValue;
  dim3 g((unsigned)((M + 255) / 256), (unsigned)N);
#define OZ_CONSL(ND_)                                                                              \
  hipLaunchKernelGGL(k_consumer_limbs<ND_>, g, dim3(256), 0, s, (const uint32_t *)tpl, Mp, Np, M, \
                     N, pl, nvw, cw, M * N)
  if (ndc == 18) OZ_CONSL(18);
  else OZ_CONSL(32);
#undef OZ_CONSL
  return hipGetLastError();
}

// One wavefront per element costs 0.2 ns an element whatever nl; a thread per
// element costs less than that for few limbs, but walks its words one by one.
// Measured (whole product, us, separate kernels / one pass), 40 x 30 x 40, 200 x
// 180 x 64, 400 x 350 x 64 and 800 x 700 x 64: mode 0  nl 4: 36 / 36, 44 / 47, 70 /
// 93, 136 / 231   nl 12: 63 / 57, 84 / 83, 136 / 150, 308 / 379   nl 24: 109 / 93,
// 146 / 129, 252 / 250, 649 / 667   nl 40: 180 / 150, 232 / 198, 436 / 409, 1137 /
// 1088; mode 1  nl 4: 47 / 41, 55 / 57, 86 / 116, 171 / 307   nl 12: 84 / 62, 112 /
// 91, 175 / 172, 415 / 462   nl 24: 148 / 99, 200 / 137, 324 / 271, 874 / 757   nl
// 40: 244 / 158, 320 / 206, 574 / 439, 1538 / 1185.  The break-even counts of
// elements grow about as nl^2; the line leaves up to 16 % to the other side (mode
// 1, nl 20 to 31, more than half a million elements).
bool limb_finish_fits(int nl, int nwords, int64_t M, int64_t N, int mode) {
  if (nl > 64 || nwords > 256) return false;
  return nl >= 32 || (double)M * (double)N <= (mode ? 768.0 : 256.0) * nl * nl;
}

hipError_t launch_limb_finish(const uint32_t *cw, int nwords, int64_t M, int64_t N,
                              const int32_t *ea, const int32_t *eb, int w, int g0, int Q, int nlimb,
                              int mode, uint64_t *climb, int32_t *cexp, uint8_t *csign, int64_t ldc,
                              int64_t planec, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  // at most 48.6 KiB (nl 64, 256 words)
  const size_t lds = (size_t)FE * ((nlimb | 1) * 8 + 8 + (nwords | 1) * 4);
  hipLaunchKernelGGL(k_limb_finish, dim3((unsigned)((M + FE - 1) / FE), (unsigned)N), dim3(256),
                     (unsigned)lds, s, cw, M * N, nwords, M, ea, eb, w, g0, Q, nlimb, mode, climb, cexp,
                     csign, ldc, planec);
  return hipGetLastError();
}

hipError_t launch_limb_round(const uint32_t *cw, int nwords, int64_t M, int64_t N,
                             const int32_t *ea, const int32_t *eb, int w, int g0, int Q, int nlimb,
                             uint64_t *olimb, int32_t *oexp, uint8_t *osign, int64_t ldo,
                             int64_t planeo, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  dim3 g((unsigned)((M + 255) / 256), (unsigned)N);
  hipLaunchKernelGGL(k_limb_round, g, dim3(256), 0, s, cw, M * N, nwords, M, N, ea, eb, w, g0, Q,
                     nlimb, olimb, oexp, osign, ldo, planeo);
  return hipGetLastError();
}

hipError_t launch_limb_sub(uint64_t *climb, int32_t *cexp, uint8_t *csign, int64_t ldc,
                           int64_t planec, const uint64_t *tlimb, const int32_t *texp,
                           const uint8_t *tsign, int nlimb, int64_t M, int64_t N, uint32_t *dw,
                           hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  dim3 g((unsigned)((M + 255) / 256), (unsigned)N);
  hipLaunchKernelGGL(k_limb_sub, g, dim3(256), 0, s, climb, cexp, csign, ldc, planec, tlimb, texp,
                     tsign, nlimb, M, N, dw, M * N);
  return hipGetLastError();
}

hipError_t launch_limb_zero(uint64_t *limb, int32_t *lexp, uint8_t *lsign, int64_t ld,
                            int64_t plane, int nlimb, int64_t M, int64_t N, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  dim3 g((unsigned)((M + 255) / 256), (unsigned)N);
  hipLaunchKernelGGL(k_limb_zero, g, dim3(256), 0, s, limb, lexp, lsign, ld, plane, nlimb, M, N);
  return hipGetLastError();
}

}  // namespace ozl
