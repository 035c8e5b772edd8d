// The LU with partial pivoting on limb matrices outside the Ozaki-II
// product (Sec. 3.4; the solve of Sec. 4.3), in the p-bit arithmetic of
// limbfp.hpp: one wavefront per element operation, lane q handling limb q.
//
//   panel, per column j of a leaf (packed by k_lpack, element by element):
//     k_lpiv (the pivot: largest exact magnitude, lowest row on ties; ipiv,
//     info, the interchange inside the leaf) -> k_ldiv (l = RN(a / pivot)) ->
//     k_lrank1 (RN(a - RN(l u)) on the leaf's remaining columns);
//   k_llaswp: the panel's interchanges on the other columns;
//   k_ltrsm:  B <- L^-1 B for a unit lower triangle (the U12 solve and the
//     leaves of its recursive form), one workgroup per column, k ascending;
//   k_lschur_naive: the native update RN(a - RN(l_ik u_kj)), k ascending, on
//     any block (the Schur update, or the inner updates of the recursion);
//   getrs: the interchanges, then blocks of LBLK rows: the diagonal block
//     by one workgroup per right-hand side, the rows below (forward) or
//     above (backward) by one wavefront each, every element taking its
//     multiply-subtracts in the order of column-oriented substitution and
//     x_k = RN(x_k / u_kk) once its updates are in, by reciprocals of the
//     diagonal found beforehand.
// A zero pivot skips its column's division and update (LAPACK's panel).
// Every kernel hands work out per wavefront, so each wavefront stays
// converged through the cross-lane arithmetic.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "lanes.hpp"
#include "limbfp.hpp"
#include "ozii_kernels.hpp"

using lfp::WF;
using ozl::LimbMat;

namespace {

constexpr int LBLK = 16;  // rows per diagonal block of the substitutions
constexpr int WPB = 4;    // wavefronts per 256-thread workgroup

__device__ __forceinline__ WF ld_el(const LimbMat &A, int64_t i, int64_t j, int nl) {
  const int l = lfp::lane_id();
  const int64_t idx = i + j * A.ld;
  uint64_t m = 0;
  if (l < nl) m = A.limb[(int64_t)l * A.plane + idx * A.es];
  const bool z = lfp::ballot(m != 0) == 0;
  WF x;
  x.m = m;
  x.e = z ? lfp::EXP_ZERO : A.exp[idx * A.xs];
  x.s = z ? 0u : (uint32_t)(A.sign[idx * A.ss] & 1u);
  return x;
}

__device__ __forceinline__ void st_el(const LimbMat &A, int64_t i, int64_t j, int nl,
                                      const WF &x) {
  const int l = lfp::lane_id();
  const int64_t idx = i + j * A.ld;
  if (l < nl) A.limb[(int64_t)l * A.plane + idx * A.es] = x.m;
  if (l == 0) {
    A.exp[idx * A.xs] = x.e;
    A.sign[idx * A.ss] = (uint8_t)x.s;
  }
}

__device__ __forceinline__ void swap_el(const LimbMat &A, int64_t i1, int64_t i2, int64_t j,
                                        int nl) {
  const int l = lfp::lane_id();
  const int64_t a = i1 + j * A.ld, b = i2 + j * A.ld;
  if (l < nl) {
    uint64_t *p = A.limb + (int64_t)l * A.plane;
    const uint64_t t = p[a * A.es], u = p[b * A.es];
    p[a * A.es] = u;
    p[b * A.es] = t;
  }
  if (l == 0) {
    const int32_t te = A.exp[a * A.xs], ue = A.exp[b * A.xs];
    const uint8_t ts = A.sign[a * A.ss], us = A.sign[b * A.ss];
    A.exp[a * A.xs] = ue;
    A.exp[b * A.xs] = te;
    A.sign[a * A.ss] = us;
    A.sign[b * A.ss] = ts;
  }
}

// a number in LDS, for the other wavefronts of the workgroup
struct SharedWF {
  uint64_t m[64];
  int32_t e;
  uint32_t s;
};
__device__ __forceinline__ void put(SharedWF &d, const WF &x) {
  const int l = lfp::lane_id();
  d.m[l] = x.m;
  if (l == 0) {
    d.e = x.e;
    d.s = x.s;
  }
}
__device__ __forceinline__ WF get(const SharedWF &d) {
  WF x;
  x.m = d.m[lfp::lane_id()];
  x.e = __builtin_amdgcn_readfirstlane(d.e);
  x.s = (uint32_t)__builtin_amdgcn_readfirstlane((int)d.s);
  return x;
}

__device__ __forceinline__ int wave_in_block() { return (int)(threadIdx.x >> 6); }
__device__ __forceinline__ int waves_in_block() { return (int)(blockDim.x >> 6); }
__device__ __forceinline__ int64_t wave_global() {
  return (int64_t)blockIdx.x * waves_in_block() + wave_in_block();
}
__device__ __forceinline__ int64_t waves_total() { return (int64_t)gridDim.x * waves_in_block(); }

// keep (r, x) when |x| is larger, or equal with a lower row
__device__ __forceinline__ void take_max(int64_t &b, WF &v, int64_t r, const WF &x) {
  const int c = b < 0 ? 1 : lfp::cmp_abs(x, v);
  if (c > 0 || (c == 0 && r < b)) {
    b = r;
    v = x;
  }
}

// The pivot of column j among rows [j, n): ipiv, info, the zero flag and the
// interchange across the panel's columns [c0, c1), by one workgroup.  Every
// thread first compares exponents and top limbs (one coalesced read of each
// per row), which decides as a rule; only rows that tie in both are compared
// whole, one wavefront per row and then a tournament through LDS (greatest
// |value|, lowest row on ties).  n = 512 rows of 49 limbs: 19 us for a
// reduction over whole numbers in two launches, 5.4 us here on a packed leaf.
constexpr int FIN_WAVES = 16;
__global__ __launch_bounds__(1024) void k_lpiv(LimbMat A, int nl, int64_t j, int64_t n, int64_t c0,
                                               int64_t c1, int64_t base, int64_t *ipiv,
                                               int32_t *info, int32_t *zflag) {
  __shared__ SharedWF sx[FIN_WAVES];
  __shared__ int32_t srow[FIN_WAVES], scnt[FIN_WAVES];
  __shared__ int32_t se[FIN_WAVES];
  __shared__ uint64_t st[FIN_WAVES];
  const int w = wave_in_block(), l = lfp::lane_id();
  const uint64_t *tops = A.limb + (int64_t)(nl - 1) * A.plane + j * A.ld * A.es;
  const int32_t *exps = A.exp + j * A.ld * A.xs;
  // greatest (exponent, top limb), the lowest row that has it, how many have it
  int32_t be = lfp::EXP_ZERO;
  uint64_t bt = 0;
  int32_t br = INT32_MAX, bc = 0;
  for (int64_t r = j + threadIdx.x; r < n; r += 1024) {
    const uint64_t t = tops[r * A.es];
    const int32_t x = exps[r * A.xs], e = t ? x : lfp::EXP_ZERO;
    const bool more = e > be || (e == be && t > bt) || bc == 0, same = e == be && t == bt;
    bc = more ? 1 : bc + (same ? 1 : 0);
    br = more ? (int32_t)r : br;
    be = more ? e : be;
    bt = more ? t : bt;
  }
  // over a wavefront, then over the wavefronts' results
  auto over = [&](int width) {
    int32_t me = bc ? be : INT32_MIN;
    for (int off = width / 2; off > 0; off >>= 1) me = max(me, __shfl_xor(me, off, 64));
    uint64_t mt = bc && be == me ? bt : 0ull;
    for (int off = width / 2; off > 0; off >>= 1) {
      const uint64_t o = (uint64_t)__shfl_xor((unsigned long long)mt, off, 64);
      mt = o > mt ? o : mt;
    }
    const bool has = bc && be == me && bt == mt;
    int32_t mr = has ? br : INT32_MAX, mc = has ? bc : 0;
    for (int off = width / 2; off > 0; off >>= 1) {
      mr = min(mr, __shfl_xor(mr, off, 64));
      mc += __shfl_xor(mc, off, 64);
    }
    be = me;
    bt = mt;
    br = mr;
    bc = mc;
  };
  over(64);
  if (l == 0) {
    se[w] = be;
    st[w] = bt;
    srow[w] = br;
    scnt[w] = bc;
  }
  __syncthreads();
  be = se[l & (FIN_WAVES - 1)];
  bt = st[l & (FIN_WAVES - 1)];
  br = srow[l & (FIN_WAVES - 1)];
  bc = scnt[l & (FIN_WAVES - 1)];
  over(FIN_WAVES);
  // (rows fit 32 bits: the limbs of a longer column would not fit the memory)
  // zeros tie only with zeros: the lowest row
  if (bt != 0 && bc > 1) {
    __syncthreads();
    int64_t b = -1;
    WF v = lfp::wf_zero();
    for (int64_t r = j + w; r < n; r += FIN_WAVES)
      if (tops[r * A.es] == bt && exps[r * A.xs] == be) take_max(b, v, r, ld_el(A, r, j, nl));
    put(sx[w], v);
    if (l == 0) srow[w] = (int32_t)b;
    __syncthreads();
    for (int step = 1; step < FIN_WAVES; step *= 2) {
      if ((w & (2 * step - 1)) == 0) {
        const int64_t r = srow[w + step];
        if (r >= 0) take_max(b, v, r, get(sx[w + step]));
      }
      __syncthreads();
      if ((w & (2 * step - 1)) == 0) {
        put(sx[w], v);
        if (l == 0) srow[w] = (int32_t)b;
      }
      __syncthreads();
    }
    br = srow[0];
  }
  if (threadIdx.x == 0) {
    ipiv[j] = base + br;
    zflag[0] = bt == 0 ? 1 : 0;
    if (bt == 0 && info[0] == 0) info[0] = (int32_t)(base + j + 1);
  }
  if (br != j)
    for (int64_t c = c0 + w; c < c1; c += FIN_WAVES) swap_el(A, j, br, c, nl);
}

// rows j <-> ipiv[j] on columns [s0, s1), one wavefront per column
__global__ __launch_bounds__(256) void k_lswap(LimbMat A, int nl, int64_t j, int64_t base,
                                               const int64_t *ipiv, int64_t s0, int64_t s1) {
  const int64_t r = ipiv[j] - base;
  if (r == j) return;
  for (int64_t c = s0 + wave_global(); c < s1; c += waves_total()) swap_el(A, j, r, c, nl);
}

__global__ __launch_bounds__(256) void k_ldiv(LimbMat A, int nl, int64_t j, int64_t n,
                                              const int32_t *zflag) {
  if (*zflag) return;
  const WF pv = ld_el(A, j, j, nl);
  for (int64_t i = j + 1 + wave_global(); i < n; i += waves_total())
    st_el(A, i, j, nl, lfp::div(ld_el(A, i, j, nl), pv, nl));
}

template <int CL>
__global__ __launch_bounds__(256) void k_lrank1(LimbMat A, int nl, int64_t j, int64_t n,
                                                int64_t c1, const int32_t *zflag) {
  __shared__ __attribute__((aligned(16))) uint8_t sbuf[WPB][lfp::PROD_LDS];
  if (*zflag) return;
  uint8_t *buf = sbuf[wave_in_block()];
  lfp::prod_init(buf);
  const int64_t rows = n - j - 1, cnt = rows * (c1 - j - 1);
  for (int64_t t = wave_global(); t < cnt; t += waves_total()) {
    const int64_t i = j + 1 + t % rows, c = j + 1 + t / rows;
    const WF a = ld_el(A, i, c, nl), lv = ld_el(A, i, j, nl), u = ld_el(A, j, c, nl);
    st_el(A, i, c, nl, lfp::fms<CL>(a, lv, u, nl, buf));
  }
}

// rows jj <-> ipiv[jj] for jj = k0 .. k0+kb-1 in order, kb <= 256, on columns
// [ca0, ca1) and [cb0, cb1).  A lane owns up to SWP of the touched rows and
// finds where each one's new contents come from by following the
// interchanges backwards; a wavefront then moves one limb plane (or the
// exponents, or the signs) of one column with all loads before its stores.
// A row outside [k0, k0+kb) that several interchanges name is moved by
// several lanes, which store the same value.  In-place swaps, one after the
// other on a wavefront per column, took 87 us per call of the n = 512,
// 49-limb LU and solve, this 34.
constexpr int SWP = 8;
__global__ __launch_bounds__(256) void k_llaswp(LimbMat A, int nl, const int64_t *ipiv, int64_t k0,
                                                int kb, int64_t ca0, int64_t ca1, int64_t cb0,
                                                int64_t cb1) {
  __shared__ int32_t sp[64 * SWP / 2];
  const int l = lfp::lane_id();
  for (int q = threadIdx.x; q < kb; q += 256) sp[q] = (int32_t)ipiv[k0 + q];
  __syncthreads();
  int32_t dst[SWP], src[SWP];
#pragma unroll
  for (int t = 0; t < SWP; ++t) {
    const int q = l + 64 * t;
    dst[t] = -1;
    src[t] = -1;
    if (q < 2 * kb) {
      const int32_t x = q < kb ? (int32_t)k0 + q : sp[q - kb];
      if (q < kb || x < k0 || x >= k0 + kb) dst[t] = x;
      src[t] = x;
    }
  }
  for (int q = kb - 1; q >= 0; --q) {
    const int32_t j = (int32_t)k0 + q, p = sp[q];
#pragma unroll
    for (int t = 0; t < SWP; ++t) {
      if (64 * t >= 2 * kb) break;
      src[t] = src[t] == j ? p : (src[t] == p ? j : src[t]);
    }
  }
  auto move = [&](auto *p) {
    typename std::remove_reference<decltype(*p)>::type v[SWP];
#pragma unroll
    for (int t = 0; t < SWP; ++t)
      if (dst[t] >= 0 && src[t] != dst[t]) v[t] = p[src[t]];
#pragma unroll
    for (int t = 0; t < SWP; ++t)
      if (dst[t] >= 0 && src[t] != dst[t]) p[dst[t]] = v[t];
  };
  const int64_t na = ca1 - ca0, cols = na + (cb1 - cb0), per = nl + 2;
  for (int64_t t = wave_global(); t < cols * per; t += waves_total()) {
    const int64_t ci = t / per, q = t - ci * per;
    const int64_t off = (ci < na ? ca0 + ci : cb0 + (ci - na)) * A.ld;
    if (q < nl) move(A.limb + q * A.plane + off);
    else if (q == nl) move(A.exp + off);
    else move(A.sign + off);
  }
}

// B = A[r0:r0+h, b0:b1] <- L^-1 B for the unit lower triangle L at (r0, r0):
// one workgroup per column, k ascending, the rows below k over its 16
// wavefronts.  RPW > 0 (h <= 16 RPW): wavefront w keeps rows w, w + 16, ..
// in registers; RPW = 0: any h, the rows in memory.  The row that is final
// after a step goes to the others through LDS.
template <int CL, int RPW>
__global__ __launch_bounds__(1024) void k_ltrsm(LimbMat A, int nl, int64_t r0, int64_t h,
                                                int64_t b0, int64_t b1) {
  constexpr int NW = 16, NR = RPW > 0 ? RPW : 1;
  __shared__ __attribute__((aligned(16))) uint8_t sbuf[NW][lfp::PROD_LDS];
  __shared__ SharedWF su[2];
  const int w = wave_in_block();
  uint8_t *buf = sbuf[w];
  lfp::prod_init(buf);
  for (int64_t c = b0 + blockIdx.x; c < b1; c += gridDim.x) {
    WF x[NR];
#pragma unroll
    for (int t = 0; t < RPW; ++t)
      if (w + NW * t < h) x[t] = ld_el(A, r0 + w + NW * t, c, nl);
    if (w == 0) put(su[0], RPW > 0 ? x[0] : ld_el(A, r0, c, nl));
    __syncthreads();
    for (int64_t k = 0; k + 1 < h; ++k) {
      const WF u = get(su[k & 1]);
      if (RPW > 0) {
#pragma unroll
        for (int t = 0; t < RPW; ++t) {
          const int64_t i = w + NW * t;
          if (i > k && i < h) {
            x[t] = lfp::fms<CL>(x[t], ld_el(A, r0 + i, r0 + k, nl), u, nl, buf);
            if (i == k + 1) put(su[(k + 1) & 1], x[t]);
          }
        }
      } else {
        // first row k + 1 of this wavefront's residue class or below
        for (int64_t i = k + 1 + (w - (k + 1) % NW + NW) % NW; i < h; i += NW) {
          const WF a = ld_el(A, r0 + i, c, nl), lv = ld_el(A, r0 + i, r0 + k, nl);
          const WF y = lfp::fms<CL>(a, lv, u, nl, buf);
          st_el(A, r0 + i, c, nl, y);
          if (i == k + 1) put(su[(k + 1) & 1], y);
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int t = 0; t < RPW; ++t)
      if (w + NW * t < h) st_el(A, r0 + w + NW * t, c, nl, x[t]);
    __syncthreads();
  }
}

// A[i0:i1, c0:c1] -= A[i0:i1, k0:k0+K] A[k0:k0+K, c0:c1] by multiply-subtracts,
// k ascending; one wavefront per element
template <int CL>
__global__ __launch_bounds__(256) void k_lschur_naive(LimbMat A, int nl, int64_t i0, int64_t i1,
                                                      int64_t c0, int64_t c1, int64_t k0,
                                                      int64_t K) {
  __shared__ __attribute__((aligned(16))) uint8_t sbuf[WPB][lfp::PROD_LDS];
  uint8_t *buf = sbuf[wave_in_block()];
  lfp::prod_init(buf);
  const int64_t m = i1 - i0, cnt = m * (c1 - c0);
  for (int64_t t = wave_global(); t < cnt; t += waves_total()) {
    const int64_t i = i0 + t % m, c = c0 + t / m;
    WF a = ld_el(A, i, c, nl);
    for (int64_t k = k0; k < k0 + K; ++k)
      a = lfp::fms<CL>(a, ld_el(A, i, k, nl), ld_el(A, k, c, nl), nl, buf);
    st_el(A, i, c, nl, a);
  }
}

// Substitution, diagonal block [k0, k1) of at most LBLK rows: one wavefront
// per row, its value in registers, the final rows broadcast through LDS;
// blockIdx.x = right-hand side.  Forward: k ascending with the unit lower
// factor; backward: k descending, x_k divided by u_kk first (RC: the
// reciprocals of the diagonal, or a null matrix).  Bound by the
// chain of LBLK dependent multiply-subtracts (and divisions): at 49 limbs
// forward 160 -> 51, backward 569 -> 106 us per block.
template <int CL, bool FWD>
__global__ __launch_bounds__(64 * LBLK) void k_ldiag(LimbMat LU, LimbMat X, LimbMat RC, int nl,
                                                     int64_t k0, int64_t k1) {
  __shared__ __attribute__((aligned(16))) uint8_t sbuf[LBLK][lfp::PROD_LDS];
  __shared__ SharedWF sx[2];
  const int64_t r = blockIdx.x;
  const int w = wave_in_block(), cnt = (int)(k1 - k0);
  uint8_t *buf = sbuf[w];
  lfp::prod_init(buf);
  auto row = [&](int q) { return FWD ? k0 + q : k1 - 1 - q; };  // in processing order
  WF x = lfp::wf_zero(), f = x, u = x, y = x;
  if (w < cnt) {
    x = ld_el(X, row(w), r, nl);
    f = w > 0 ? ld_el(LU, row(w), row(0), nl) : lfp::wf_zero();
    if (!FWD) u = ld_el(LU, row(w), row(w), nl);
    if (!FWD && RC.limb) y = ld_el(RC, row(w), 0, nl);
  }
  for (int q = 0; q < cnt; ++q) {
    if (w == q) {
      if constexpr (!FWD) {
        bool done = false;
        if constexpr (CL > 0) {
          if (RC.limb) {
            x = lfp::div_by<CL>(x, u, y, nl, buf);
            done = true;
          }
        }
        if (!done) x = lfp::div(x, u, nl);
      }
      put(sx[q & 1], x);
    }
    __syncthreads();
    if (w > q && w < cnt) {
      const WF fn = w > q + 1 ? ld_el(LU, row(w), row(q + 1), nl) : f;
      x = lfp::fms<CL>(x, f, get(sx[q & 1]), nl, buf);
      f = fn;
    }
  }
  if (w < cnt) st_el(X, row(w), r, nl, x);
}

// Substitution, the rows [i0, i1) not yet solved after the block [k0, k1),
// whose values they take in its order; one wavefront per row, blockIdx.y =
// right-hand side
template <int CL, bool FWD>
__global__ __launch_bounds__(256) void k_lrest(LimbMat LU, LimbMat X, int nl, int64_t k0,
                                               int64_t k1, int64_t i0, int64_t i1) {
  __shared__ __attribute__((aligned(16))) uint8_t sbuf[WPB][lfp::PROD_LDS];
  uint8_t *buf = sbuf[wave_in_block()];
  lfp::prod_init(buf);
  const int64_t r = blockIdx.y, cnt = k1 - k0;
  auto col = [&](int64_t q) { return FWD ? k0 + q : k1 - 1 - q; };
  for (int64_t i = i0 + wave_global(); i < i1; i += waves_total()) {
    WF x = ld_el(X, i, r, nl);
    WF f = ld_el(LU, i, col(0), nl), y = ld_el(X, col(0), r, nl);
    for (int64_t q = 0; q < cnt; ++q) {
      const int64_t kn = col(q + 1 < cnt ? q + 1 : q);
      const WF fn = ld_el(LU, i, kn, nl), yn = ld_el(X, kn, r, nl);
      x = lfp::fms<CL>(x, f, y, nl, buf);
      f = fn;
      y = yn;
    }
    st_el(X, i, r, nl, x);
  }
}

// elementwise a op b on vectors (element t at index t): CL = 0 for 0 add, 1 sub
// and 3 div; CL > 0: 2 mul on the matrix cores, from one limb on.  The products
// apart, since their registers and LDS leave the other operations fewer
// wavefronts and the division's do so to them: 200000 products of 1 / 2 / 3 / 16
// limbs in one kernel 118 / 126 / 132 / 128 us, apart 102 for all (the loop apart
// 103 / 108 / 115); sums of 33 limbs 169, 156.
template <int CL>
__global__ __launch_bounds__(256) void k_larith(int op, int nl, int64_t cnt, LimbMat A, LimbMat B,
                                                LimbMat C) {
  __shared__ __attribute__((aligned(16))) uint8_t sbuf[WPB][CL > 0 ? lfp::PROD_LDS : 16];
  uint8_t *buf = sbuf[wave_in_block()];
  if (CL > 0) lfp::prod_init(buf);
  for (int64_t t = wave_global(); t < cnt; t += waves_total()) {
    const WF a = ld_el(A, t, 0, nl), b = ld_el(B, t, 0, nl);
    WF r;
    if constexpr (CL > 0) r = lfp::mul<CL>(a, b, nl, buf);
    else if (op == 3) r = lfp::div(a, b, nl);
    else r = lfp::add(a, b, (uint32_t)op, nl);
    st_el(C, t, 0, nl, r);
  }
}

// Packing: a workgroup moves 64 rows of one column through LDS, so that both
// the limb planes and the packed numbers are read and written in order.  An
// element's limbs lie a plane apart in the caller's matrix: at orders that
// are powers of two they all fall on one memory channel, and a wavefront's
// 64-limb access took about 2 us; packed it is one run of 8 (nl + 1) bytes.
__global__ __launch_bounds__(256) void k_lpack(LimbMat A, LimbMat P, int nl, int64_t i0,
                                               int64_t rows, int64_t c0, int unpack) {
  __shared__ uint64_t sm[64 * 65];
  const int rs = nl + 1, l = lfp::lane_id(), w = wave_in_block();
  const int64_t r0 = (int64_t)blockIdx.x * 64, c = blockIdx.y;
  const int cnt = (int)(rows - r0 < 64 ? rows - r0 : 64);
  const int64_t src = i0 + r0 + l + (c0 + c) * A.ld;
  uint64_t *pk = P.limb + (r0 + c * P.ld) * rs;
  if (!unpack) {
    if (l < cnt)
      for (int q = w; q < rs; q += WPB)
        sm[l * rs + q] = q < nl ? A.limb[q * A.plane + src]
                                : (uint32_t)A.exp[src] | ((uint64_t)(A.sign[src] & 1u) << 32);
    __syncthreads();
    for (int t = threadIdx.x; t < cnt * rs; t += 256) pk[t] = sm[t];
  } else {
    for (int t = threadIdx.x; t < cnt * rs; t += 256) sm[t] = pk[t];
    __syncthreads();
    if (l < cnt)
      for (int q = w; q < rs; q += WPB) {
        const uint64_t v = sm[l * rs + q];
        if (q < nl) {
          A.limb[q * A.plane + src] = v;
        } else {
          A.exp[src] = (int32_t)(uint32_t)v;
          A.sign[src] = (uint8_t)((v >> 32) & 1u);
        }
      }
  }
}

// R = RN(1 / u_kk) of the diagonal, for the divisions of the backward solve
__global__ __launch_bounds__(256) void k_lrecip(LimbMat LU, LimbMat R, int nl, int64_t n) {
  WF one;
  one.m = lfp::lane_id() == nl - 1 ? 1ull << 63 : 0ull;
  one.e = 1;
  one.s = 0;
  for (int64_t k = wave_global(); k < n; k += waves_total())
    st_el(R, k, 0, nl, lfp::div(one, ld_el(LU, k, k, nl), nl));
}

__global__ void k_lfill_i32(int32_t *p, int32_t v, int count) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i < count) p[i] = v;
}

// The product form of nl limbs: the loop below LOOP_LIMBS, else the matrix
// cores with the tiles of up to CL limbs.  200000 products of 2 / 4 / 8 / 16
// limbs: loop 119 / 133 / 165 / 235 us, matrix cores 120 / 120 / 121 / 125 us;
// the order 192 LU + solve 6.83 / 7.47 / 8.93 / 11.8 against 7.02 / 7.35 /
// 8.15 / 9.71 ms.
constexpr int LOOP_LIMBS = 4;
#define OZ_BY_CL(nl, ...)                                      \
  do {                                                         \
    if ((nl) < LOOP_LIMBS) { constexpr int CL = 0; __VA_ARGS__; }    \
    else if ((nl) <= 16) { constexpr int CL = 16; __VA_ARGS__; }     \
    else if ((nl) <= 32) { constexpr int CL = 32; __VA_ARGS__; }     \
    else if ((nl) <= 48) { constexpr int CL = 48; __VA_ARGS__; }     \
    else { constexpr int CL = 64; __VA_ARGS__; }                     \
  } while (0)

// workgroups for `waves` independent wavefront tasks
int grid_for(int64_t waves, int64_t cap = 8192) {
  int64_t g = (waves + WPB - 1) / WPB;
  if (g < 1) g = 1;
  return (int)(g < cap ? g : cap);
}

}  // namespace

namespace ozl {

hipError_t launch_lpack(LimbMat A, LimbMat P, int nl, int64_t i0, int64_t rows, int64_t c0,
                        int64_t w, int unpack, hipStream_t s) {
  if (rows <= 0 || w <= 0) return hipSuccess;
  for (int64_t c = 0; c < w; c += 65535) {
    LimbMat Q = P;
    Q.limb += c * P.ld * P.es;
    const dim3 g((unsigned)((rows + 63) / 64), (unsigned)std::min<int64_t>(65535, w - c));
    hipLaunchKernelGGL(k_lpack, g, dim3(256), 0, s, A, Q, nl, i0, rows, c0 + c, unpack);
  }
  return hipGetLastError();
}

hipError_t launch_lpanel_column(LimbMat A, int nl, int64_t j, int64_t n, int64_t s0, int64_t s1,
                                int64_t c1, int64_t base, int64_t *ipiv, int32_t *info,
                                int32_t *zflag, hipStream_t s) {
  // a wide interchange runs on one wavefront per column after the search
  const bool wide = s1 - s0 > FIN_WAVES * 4;
  hipLaunchKernelGGL(k_lpiv, dim3(1), dim3(64 * FIN_WAVES), 0, s, A, nl, j, n, s0, wide ? s0 : s1,
                     base, ipiv, info, zflag);
  if (wide)
    hipLaunchKernelGGL(k_lswap, dim3(grid_for(s1 - s0)), dim3(256), 0, s, A, nl, j,
                       base, (const int64_t *)ipiv, s0, s1);
  if (j + 1 < n) {
    hipLaunchKernelGGL(k_ldiv, dim3(grid_for(n - j - 1)), dim3(256), 0, s, A, nl, j, n,
                       (const int32_t *)zflag);
    if (j + 1 < c1)
      OZ_BY_CL(nl, hipLaunchKernelGGL(k_lrank1<CL>, dim3(grid_for((n - j - 1) * (c1 - j - 1))),
                                      dim3(256), 0, s, A, nl, j, n, c1, (const int32_t *)zflag));
  }
  return hipGetLastError();
}

hipError_t launch_llaswp(LimbMat A, int nl, const int64_t *ipiv, int64_t k0, int64_t kb,
                         int64_t ca0, int64_t ca1, int64_t cb0, int64_t cb1, hipStream_t s) {
  const int64_t cnt = (ca1 - ca0) + (cb1 - cb0);
  if (cnt <= 0 || kb <= 0) return hipSuccess;
  constexpr int64_t CH = 64 * SWP / 2;
  for (int64_t k = k0; k < k0 + kb; k += CH)
    hipLaunchKernelGGL(k_llaswp, dim3(grid_for(cnt * (nl + 2), 2048)), dim3(256), 0, s, A, nl, ipiv,
                       k, (int)std::min<int64_t>(CH, k0 + kb - k), ca0, ca1, cb0, cb1);
  return hipGetLastError();
}

hipError_t launch_ltrsm(LimbMat A, int nl, int64_t r0, int64_t h, int64_t b0, int64_t b1,
                        hipStream_t s) {
  const int64_t cols = b1 - b0;
  if (cols <= 0 || h <= 1) return hipSuccess;
  const dim3 g((unsigned)(cols < 65535 ? cols : 65535));
  if (h <= 32)
    OZ_BY_CL(nl, hipLaunchKernelGGL((k_ltrsm<CL, 2>), g, dim3(1024), 0, s, A, nl, r0, h, b0, b1));
  else
    OZ_BY_CL(nl, hipLaunchKernelGGL((k_ltrsm<CL, 0>), g, dim3(1024), 0, s, A, nl, r0, h, b0, b1));
  return hipGetLastError();
}

hipError_t launch_lschur_naive(LimbMat A, int nl, int64_t i0, int64_t i1, int64_t c0, int64_t c1,
                               int64_t k0, int64_t K, hipStream_t s) {
  const int64_t cnt = (i1 - i0) * (c1 - c0);
  if (i1 <= i0 || c1 <= c0 || K <= 0) return hipSuccess;
  OZ_BY_CL(nl, hipLaunchKernelGGL(k_lschur_naive<CL>, dim3(grid_for(cnt)), dim3(256), 0, s, A, nl,
                                  i0, i1, c0, c1, k0, K));
  return hipGetLastError();
}

// the loop products of few limbs keep the digit chain, which is short there
bool lgetrs_wants_recip(int nl) { return nl >= LOOP_LIMBS; }

hipError_t launch_lgetrs(LimbMat LU, int nl, int64_t n, const int64_t *ipiv, LimbMat X,
                         int64_t nrhs, uint64_t *recip, hipStream_t s) {
  if (n <= 0 || nrhs <= 0) return hipSuccess;
  const LimbMat RC = packed_mat(recip, nl, n);
  if (recip)
    hipLaunchKernelGGL(k_lrecip, dim3(grid_for(n)), dim3(256), 0, s, LU, RC, nl, n);
  hipError_t e = launch_llaswp(X, nl, ipiv, 0, n, 0, nrhs, 0, 0, s);
  if (e != hipSuccess) return e;
  for (int64_t k0 = 0; k0 < n; k0 += LBLK) {
    const int64_t k1 = k0 + LBLK < n ? k0 + LBLK : n;
    OZ_BY_CL(nl, hipLaunchKernelGGL((k_ldiag<CL, true>), dim3((unsigned)nrhs), dim3(64 * LBLK), 0, s,
                                    LU, X, RC, nl, k0, k1));
    if (k1 < n)
      OZ_BY_CL(nl, hipLaunchKernelGGL((k_lrest<CL, true>),
                                      dim3(grid_for(n - k1, 2048), (unsigned)nrhs), dim3(256), 0, s,
                                      LU, X, nl, k0, k1, k1, n));
  }
  for (int64_t k1 = n; k1 > 0;) {
    const int64_t k0 = k1 - LBLK > 0 ? k1 - LBLK : 0;
    OZ_BY_CL(nl, hipLaunchKernelGGL((k_ldiag<CL, false>), dim3((unsigned)nrhs), dim3(64 * LBLK), 0, s,
                                    LU, X, RC, nl, k0, k1));
    if (k0 > 0)
      OZ_BY_CL(nl, hipLaunchKernelGGL((k_lrest<CL, false>),
                                      dim3(grid_for(k0, 2048), (unsigned)nrhs), dim3(256), 0, s, LU,
                                      X, nl, k0, k1, (int64_t)0, k0));
    k1 = k0;
  }
  return hipGetLastError();
}

hipError_t launch_larith(int op, int nl, int64_t cnt, LimbMat A, LimbMat B, LimbMat C,
                         hipStream_t s) {
  if (cnt <= 0) return hipSuccess;
  const dim3 g(grid_for(cnt));
  if (op == 2)
    OZ_BY_CL(std::max(nl, LOOP_LIMBS),
             hipLaunchKernelGGL(k_larith<CL>, g, dim3(256), 0, s, op, nl, cnt, A, B, C));
  else
    hipLaunchKernelGGL(k_larith<0>, g, dim3(256), 0, s, op, nl, cnt, A, B, C);
  return hipGetLastError();
}

hipError_t launch_lfill_i32(int32_t *p, int32_t v, int count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_lfill_i32, dim3((count + 255) / 256), dim3(256), 0, s, p, v, count);
  return hipGetLastError();
}

}  // namespace ozl
