// Batched LU + solve of many small, uneven matrices in one persistent launch
// (the batched configuration: 256 independent DD / QD systems of order 64 to
// 512).  Every workgroup takes matrices from a device work queue -- the host
// orders the batch by decreasing cost (longest-processing-time first) -- and
// factors and solves each one alone (with the Ozaki-II update: helped by the
// workgroups that have none left) with the expansion arithmetic of
// expansion.hpp: unblocked right-looking LU with partial pivoting (LAPACK's
// i?amax, whole-row interchanges), then the solve with the factors.  Per
// element the operations come in exactly the order of ozII_getrf with b = 1
// and the native update, followed by ozII_getrs, so results match those (and
// the oracle) bit for bit.  The launch allocates nothing and clears its queue
// with a kernel, so it can be captured in a hipGraph.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/ozii.h"
#include "batch_rules.hpp"
#include "expansion.hpp"
#include "ozii_elem.hpp"
#include "ozii_stage.hpp"

using namespace ozk;

typedef int v4i __attribute__((ext_vector_type(4)));

namespace {

constexpr int BT = 1024;  // threads per workgroup (4 wavefronts per SIMD)
constexpr int BTZ = ozb::NT;  // the same for the Ozaki-II update

// The elements idx = t, t + NT, t + 2 NT, ... of a rectangle with mr > 0 rows
// taken column by column, (i, c) = (idx % mr, idx / mr), with one division
// per thread instead of one per element.
template <int NT>
struct ColWalk {
  int32_t i, c, di, dc, mr;
  __device__ ColWalk(int32_t rows, int32_t t)
      : i(t % rows), c(t / rows), di(NT % rows), dc(NT / rows), mr(rows) {}
  __device__ void next() {
    i += di;
    c += dc;
    if (i >= mr) {
      i -= mr;
      ++c;
    }
  }
};

// largest |value| first, then the lower row index (a total order)
template <int NC>
__device__ __forceinline__ bool piv_better(const double (&kb_)[NC], int64_t ib,
                                           const double (&ka)[NC], int64_t ia) {
  if (ib < 0) return false;
  if (ia < 0) return true;
  if (ozx::abs_greater<NC>(kb_, ka)) return true;
  if (ozx::abs_greater<NC>(ka, kb_)) return false;
  return ib < ia;
}

// Column j of the LU: pivot search over rows j..n-1 (largest magnitude, then
// the lower row index), ipiv and info, the whole-row interchange and the
// division of the column below the pivot (nothing to divide after a zero
// pivot: the column below it is zero).  Ends with the workgroup in step and
// returns whether the pivot was exactly zero (the same in every thread).  A
// chain of the column's loads, the reduction and a division: two barriers, the
// column read once.  With seven barriers and three reads of it, and the solve
// through memory, 256 systems took 35.0 instead of 34.6 ms and 16 13.1 instead
// of 12.7.
template <int NC, int NT>
__device__ bool pivot_column(const ozII_batch_item &it, int64_t j, double (*rkey)[4],
                             int64_t *ridx, int *s_info) {
  const int tid = threadIdx.x;
  const int64_t n = it.n;
  double *A = it.A;
  auto E = [&](int64_t i, int64_t c) { return A + (i + c * n) * NC; };
  double bk[NC], x0[NC];
  int64_t bi = -1;
#pragma unroll
  for (int q = 0; q < NC; ++q) bk[q] = x0[q] = 0.0;
  for (int64_t i = j + tid; i < n; i += NT) {
    double x[NC];
    ozx::load<NC>(E(i, j), x);
    if (i == j + tid) {
#pragma unroll
      for (int q = 0; q < NC; ++q) x0[q] = x[q];
    }
    if (piv_better<NC>(x, i, bk, bi)) {
#pragma unroll
      for (int q = 0; q < NC; ++q) bk[q] = x[q];
      bi = i;
    }
  }
  // the order is total, so any reduction order gives the same winner: a
  // butterfly inside each wavefront, then every thread over the wavefront
  // winners
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    double kv[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) kv[q] = __shfl_xor(bk[q], off, 64);
    const int64_t iv = __shfl_xor(bi, off, 64);
    if (piv_better<NC>(kv, iv, bk, bi)) {
#pragma unroll
      for (int q = 0; q < NC; ++q) bk[q] = kv[q];
      bi = iv;
    }
  }
  constexpr int NW = NT / 64;  // rkey[NW]: the entry of row j
  if ((tid & 63) == 0) {
#pragma unroll
    for (int q = 0; q < NC; ++q) rkey[tid >> 6][q] = bk[q];
    ridx[tid >> 6] = bi;
  }
  if (tid == 0) {
#pragma unroll
    for (int q = 0; q < NC; ++q) rkey[NW][q] = x0[q];
  }
  __syncthreads();
  double d[NC];
  int64_t p = ridx[0];
#pragma unroll
  for (int q = 0; q < NC; ++q) d[q] = rkey[0][q];
  for (int wv = 1; wv < NW; ++wv) {
    double kv[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) kv[q] = rkey[wv][q];
    if (piv_better<NC>(kv, ridx[wv], d, p)) {
#pragma unroll
      for (int q = 0; q < NC; ++q) d[q] = kv[q];
      p = ridx[wv];
    }
  }
  bool zero = true;
#pragma unroll
  for (int q = 0; q < NC; ++q) zero = zero && (d[q] == 0.0);
  if (tid == 0) {
    it.ipiv[j] = p;
    if (zero && *s_info == 0) *s_info = (int)(j + 1);
  }
  if (!zero) {
    // whole-row interchange outside column j, its first loads under way while
    // the column is divided; column j's own is in the choice of dividends
    const bool sw = p != j && tid < n && tid != j;
    double u[NC], v[NC];
    if (sw) {
      ozx::load<NC>(E(j, tid), u);
      ozx::load<NC>(E(p, tid), v);
    }
    for (int64_t i = j + tid; i < n; i += NT) {
      double a[NC], l[NC];
      if (i == j + tid) {
#pragma unroll
        for (int q = 0; q < NC; ++q) a[q] = x0[q];
      } else {
        ozx::load<NC>(E(i, j), a);
      }
      if (i == p) {
#pragma unroll
        for (int q = 0; q < NC; ++q) a[q] = rkey[NW][q];
      }
      ozx::div<NC>(a, d, l);
      if (i == j) {
#pragma unroll
        for (int q = 0; q < NC; ++q) l[q] = d[q];
      }
      ozx::store<NC>(E(i, j), l);
    }
    if (sw) {
      ozx::store<NC>(E(j, tid), v);
      ozx::store<NC>(E(p, tid), u);
    }
    if (p != j)
      for (int64_t c = tid + NT; c < n; c += NT) {
        if (c == j) continue;
        ozx::load<NC>(E(j, c), u);
        ozx::load<NC>(E(p, c), v);
        ozx::store<NC>(E(j, c), v);
        ozx::store<NC>(E(p, c), u);
      }
  }
  __syncthreads();
  return zero;
}

template <int NC, int NT>
__device__ void solve_one(const ozII_batch_item &it, double (*xs)[4], int64_t *pv);

template <int NC>
__device__ void lu_solve_one(const ozII_batch_item &it, double (*rkey)[4], int64_t *ridx,
                             int *s_info) {
  const int tid = threadIdx.x;
  const int64_t n = it.n;
  double *A = it.A;
  auto E = [&](int64_t i, int64_t c) { return A + (i + c * n) * NC; };
  if (tid == 0) *s_info = 0;
  __syncthreads();
  for (int64_t j = 0; j < n; ++j) {
    pivot_column<NC, BT>(it, j, rkey, ridx, s_info);
    // rank-1 update of the trailing matrix (also after a zero pivot, with the
    // unscaled -- all-zero -- column, as the blocked LU with b = 1 does)
    const int64_t m = n - j - 1;
    ColWalk<BT> wk((int32_t)(m > 0 ? m : 1), tid);
    for (int64_t idx = tid; idx < m * m; idx += BT, wk.next()) {
      const int64_t i = j + 1 + wk.i, c = j + 1 + wk.c;
      double a[NC], l[NC], u[NC], o[NC];
      ozx::load<NC>(E(i, c), a);
      ozx::load<NC>(E(i, j), l);
      ozx::load<NC>(E(j, c), u);
      ozx::fms<NC>(a, l, u, o);
      ozx::store<NC>(E(i, c), o);
    }
    __syncthreads();
  }
  if (tid == 0) *it.info = *s_info;
  solve_one<NC, BT>(it, rkey, ridx);
}

// The solve with the factors: interchanges in ipiv order, forward (unit L,
// ascending), backward (descending, each x_k divided by u_kk once its
// updates are in), as ozII_getrs does for one right-hand side.  Up to SOLVE_N
// rows the right-hand side lives in registers, R rows a thread, and in LDS (xs;
// pv: the pivots), the factors' entries are requested a step ahead and a step
// takes one barrier; the division is done by all lanes of the row's wavefront
// (one lane alone was slower).  A chain of n multiply-subtracts and n
// divisions.  Larger orders (native update only) go through memory.
constexpr int SOLVE_N = 1024;
template <int NC, int NT>
__device__ void solve_one(const ozII_batch_item &it, double (*xs)[4], int64_t *pv) {
  if (!it.b) return;
  const int tid = threadIdx.x;
  const int64_t n = it.n;
  double *A = it.A;
  auto E = [&](int64_t i, int64_t c) { return A + (i + c * n) * NC; };
  double *x = it.b;
  if (n <= SOLVE_N) {
    constexpr int R = SOLVE_N / NT;
    __syncthreads();  // the pivots are written, the LDS is free
    for (int i = tid; i < n; i += NT) {
      double u[NC];
      ozx::load<NC>(x + i * NC, u);
#pragma unroll
      for (int q = 0; q < NC; ++q) xs[i][q] = u[q];
      pv[i] = it.ipiv[i];
    }
    __syncthreads();
    if (tid == 0)
      for (int j = 0; j < n; ++j) {
        const int p = (int)pv[j];
        if (p != j) {
#pragma unroll
          for (int q = 0; q < NC; ++q) {
            const double u = xs[j][q];
            xs[j][q] = xs[p][q];
            xs[p][q] = u;
          }
        }
      }
    __syncthreads();
    double xr[R][NC], cur[R][NC], nxt[R][NC], xk[NC], o[NC];
    // entry (row r of this thread, column k) of the factors; any valid entry
    // outside the matrix
    auto fetch = [&](int k, double (&f)[R][NC]) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int i = tid + r * NT;
        ozx::load<NC>(E(i < n ? i : 0, k), f[r]);
      }
    };
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < NC; ++q) xr[r][q] = tid + r * NT < n ? xs[tid + r * NT][q] : 0.0;
    fetch(0, cur);
    for (int k = 0; k + 1 < n; ++k) {
      fetch(k + 1, nxt);
#pragma unroll
      for (int q = 0; q < NC; ++q) xk[q] = xs[k][q];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int i = tid + r * NT;
        if (i > k && i < n) {
          ozx::fms<NC>(xr[r], cur[r], xk, o);
#pragma unroll
          for (int q = 0; q < NC; ++q) xr[r][q] = o[q];
          if (i == k + 1) {
#pragma unroll
            for (int q = 0; q < NC; ++q) xs[i][q] = o[q];
          }
        }
#pragma unroll
        for (int q = 0; q < NC; ++q) cur[r][q] = nxt[r][q];
      }
      __syncthreads();
    }
    fetch((int)n - 1, cur);
    for (int k = (int)n - 1; k >= 0; --k) {
      fetch(k > 0 ? k - 1 : 0, nxt);
      const int kt = k % NT, kr = k / NT;
      if (tid >> 6 == kt >> 6) {
        double u[NC];
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          double xv = xr[0][q], uv = cur[0][q];
#pragma unroll
          for (int r = 1; r < R; ++r) {
            xv = kr == r ? xr[r][q] : xv;
            uv = kr == r ? cur[r][q] : uv;
          }
          xk[q] = __shfl(xv, kt & 63, 64);
          u[q] = __shfl(uv, kt & 63, 64);
        }
        ozx::div<NC>(xk, u, o);
        if (tid == kt) {
#pragma unroll
          for (int q = 0; q < NC; ++q) xs[k][q] = o[q];
        }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < NC; ++q) xk[q] = xs[k][q];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (tid + r * NT < k) {
          ozx::fms<NC>(xr[r], cur[r], xk, o);
#pragma unroll
          for (int q = 0; q < NC; ++q) xr[r][q] = o[q];
        }
#pragma unroll
        for (int q = 0; q < NC; ++q) cur[r][q] = nxt[r][q];
      }
    }
    for (int i = tid; i < n; i += NT) {
      double u[NC];
#pragma unroll
      for (int q = 0; q < NC; ++q) u[q] = xs[i][q];
      ozx::store<NC>(x + i * NC, u);
    }
    __syncthreads();
    return;
  }
  if (tid == 0)
    for (int64_t j = 0; j < n; ++j) {
      const int64_t p = it.ipiv[j];
      if (p != j) {
        double u[NC], v[NC];
        ozx::load<NC>(x + j * NC, u);
        ozx::load<NC>(x + p * NC, v);
        ozx::store<NC>(x + j * NC, v);
        ozx::store<NC>(x + p * NC, u);
      }
    }
  __syncthreads();
  for (int64_t k = 0; k < n; ++k) {
    double xk[NC];
    ozx::load<NC>(x + k * NC, xk);
    for (int64_t i = k + 1 + tid; i < n; i += NT) {
      double a[NC], l[NC], o[NC];
      ozx::load<NC>(x + i * NC, a);
      ozx::load<NC>(E(i, k), l);
      ozx::fms<NC>(a, l, xk, o);
      ozx::store<NC>(x + i * NC, o);
    }
    __syncthreads();
  }
  for (int64_t k = n - 1; k >= 0; --k) {
    if (tid == 0) {
      double u[NC], xk[NC], o[NC];
      ozx::load<NC>(E(k, k), u);
      ozx::load<NC>(x + k * NC, xk);
      ozx::div<NC>(xk, u, o);
      ozx::store<NC>(x + k * NC, o);
    }
    __syncthreads();
    double xk[NC];
    ozx::load<NC>(x + k * NC, xk);
    for (int64_t i = tid; i < k; i += NT) {
      double a[NC], u[NC], o[NC];
      ozx::load<NC>(x + i * NC, a);
      ozx::load<NC>(E(i, k), u);
      ozx::fms<NC>(a, u, xk, o);
      ozx::store<NC>(x + i * NC, o);
    }
    __syncthreads();
  }
}

// a <- a - l u over the mr x mc elements (i, c) of one step (where(i, c) gives
// the three operands; a is updated in place), two elements per thread in
// flight: both elements' loads are issued before the first multiply-subtract,
// so one memory round trip serves two of them (the Ozaki-II workgroup has half
// the wavefronts of the native one).  Each element is updated once, so the
// order of its updates is the caller's.
template <int NC, int NT, typename W>
__device__ __forceinline__ void fms_sweep(int32_t mr, int32_t mc, W where) {
  if (mr <= 0 || mc <= 0) return;
  const int32_t total = mr * mc;
  ColWalk<NT> wk(mr, threadIdx.x);
  for (int32_t idx = threadIdx.x; idx < total; idx += 2 * NT) {
    const bool two = idx + NT < total;
    double *pa0, *pa1 = nullptr;
    const double *pl0, *pu0, *pl1 = nullptr, *pu1 = nullptr;
    where(wk.i, wk.c, pa0, pl0, pu0);
    wk.next();
    if (two) where(wk.i, wk.c, pa1, pl1, pu1);
    wk.next();
    double a0[NC], l0[NC], u0[NC], a1[NC] = {}, l1[NC] = {}, u1[NC] = {}, o[NC];
    ozx::load<NC>(pa0, a0);
    ozx::load<NC>(pl0, l0);
    ozx::load<NC>(pu0, u0);
    if (two) {
      ozx::load<NC>(pa1, a1);
      ozx::load<NC>(pl1, l1);
      ozx::load<NC>(pu1, u1);
    }
    ozx::fms<NC>(a0, l0, u0, o);
    ozx::store<NC>(pa0, o);
    if (two) {
      ozx::fms<NC>(a1, l1, u1, o);
      ozx::store<NC>(pa1, o);
    }
  }
}

// ---------------------------------------------------------------------------
// Blocked LU with the Ozaki-II Schur update, one system per workgroup
// (Sec. 3.4, Eq. (schur), with the product of Sec. 3.1-3.3 at K = b).  Per
// block of b columns: the panel (pivot_column and the rank-1 updates of the
// panel's own columns, whole-row interchanges), U12 = L11^-1 A12 (for
// k = k0 .. : a_ic -= l_ik u_kc over the rows below k of the block), then
// A22 -= L21 U12 by the stages of ozII_gemm run inside the workgroup:
//   (S1) row / column exponents into the scratch;
//   (S2)+(S3) produce_block_b, the 256-thread quarters taking the 16-row x
//        64-k blocks of L21 and U12 in turn;
//   (S4) every wavefront takes 64 x 64 tiles of the (group, modulus)
//        products: 4 x 4 MFMA 16x16x64 fragments, operands straight from
//        the scratch planes, the t-bytes stored as 4-byte column runs;
//   (S5)+(S6) every wavefront takes 64 consecutive elements of a column
//        through the matrix-core CRT (crt_group_mx), one element per lane for
//        the rounding and the expansion subtraction.
// Per element the operations are those of ozII_getrf with the same b and
// method = Ozaki-II on the INT8 back-end, so the factors agree bit for bit.
//
// Scratch of one workgroup (Mp = m2 and Kp = b rounded up to 64): ea, eb
// (Mp int32 each), S nmod planes of L21 residues and S nmod planes of U12
// residues (Mp x Kp bytes each), ng nmod t-planes (Mp x Mp bytes each).
// ---------------------------------------------------------------------------
template <int NC, int NWM, int NT>
struct OzUpdate {
  double *A;
  int64_t n, k0, k1, K, m2, Mp, Kp, KB, plane;
  const DevPlan *pl;
  int32_t *ea, *eb;
  uint8_t *pa, *pb, *tpl;
  __device__ __forceinline__ OzUpdate(double *A_, int64_t n_, int64_t k0_, int64_t k1_,
                                      const DevPlan *pl_, uint8_t *ws)
      : A(A_), n(n_), k0(k0_), k1(k1_), K(k1_ - k0_), m2(n_ - k1_), pl(pl_) {
    Mp = (m2 + 63) & ~(int64_t)63;
    Kp = (K + 63) & ~(int64_t)63;
    KB = Kp / 64;
    plane = Mp * Kp;
    ea = (int32_t *)ws;
    eb = ea + Mp;
    pa = (uint8_t *)(eb + Mp);
    pb = pa + (int64_t)pl->S * pl->nmod * plane;
    tpl = pb + (int64_t)pl->S * pl->nmod * plane;
  }

  // U12 = L11^-1 A12, forward in k, columns c0 .. c1-1 of the trailing matrix
  __device__ __forceinline__ void solve_u12(int64_t c0, int64_t c1) const {
    double *P = A;
    const int64_t ld = n, kb = k1;
    for (int64_t k = k0; k + 1 < k1; ++k) {
      fms_sweep<NC, NT>((int32_t)(k1 - k - 1), (int32_t)(c1 - c0),
                        [&](int32_t i, int32_t c, double *&pa_, const double *&pl_,
                            const double *&pu_) {
                          double *col = P + (kb + c0 + c) * ld * NC;
                          pa_ = col + (k + 1 + i) * NC;
                          pl_ = P + (k + 1 + i + k * ld) * NC;
                          pu_ = col + k * NC;
                        });
      __syncthreads();
    }
  }

  // (S1) to (S3) of rows r0 .. r1-1 of L21 (isA) or columns r0 .. r1-1 of U12;
  // multiples of 16, r1 <= Mp
  __device__ __forceinline__ void residues(bool isA, int64_t r0, int64_t r1) const {
    const double *X = isA ? A + (k1 + k0 * n) * NC : A + (k0 + k1 * n) * NC;
    const int64_t so = isA ? 1 : n, sh = isA ? n : 1;
    int32_t *ex = isA ? ea : eb;
    for (int64_t i = r0 + threadIdx.x; i < r1; i += NT) {
      int32_t be = EXP_ZERO;
      if (i < m2)
        for (int64_t h = 0; h < K; ++h) {
          const int32_t u = exponent_of<NC>(X + (i * so + h * sh) * NC);
          be = u > be ? u : be;
        }
      ex[i] = be;
    }
    __syncthreads();
    for (int64_t q = r0 / 16 * KB + (threadIdx.x >> 8); q < r1 / 16 * KB; q += NT / 256)
      produce_block_b<NC, 8, NWM, PL_I8>(X, n, isA ? 1 : 0, m2, K, KB, ex, pl, isA ? pa : pb, plane,
                                         q % KB, q / KB, threadIdx.x & 255, 0, pl->nmod);
  }

  // (S4) to (S6) and A22 -= c over the 64 x 64 tiles tm0 .. tm1-1 by tn0 .. tn1-1
  __device__ __forceinline__ void tiles(int64_t tm0, int64_t tm1, int64_t tn0, int64_t tn1,
                                        uint32_t *stage) const {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int S = pl->S, nmod = pl->nmod, ng = pl->ng, g0 = pl->g0, Q = pl->Q, w = pl->w;
    double *A22 = A + (k1 + k1 * n) * NC;

    // (S4)
    {
      const int TMc = (int)(tm1 - tm0), TNc = (int)(tn1 - tn0);
      const int items = ng * nmod * TMc * TNc;
      for (int q = wv; q < items; q += NT / 64) {
        const int64_t tn = tn0 + q % TNc, tm = tm0 + (q / TNc) % TMc;
        const int gl = q / (TMc * TNc);
        const int l = gl % nmod, g = g0 + gl / nmod;
        const int ta0 = g - (S - 1) > 0 ? g - (S - 1) : 0;
        const int ta1 = g < S - 1 ? g : S - 1;
        v4i acc[4][4];
  #pragma unroll
        for (int a = 0; a < 4; ++a)
  #pragma unroll
          for (int b = 0; b < 4; ++b) acc[a][b] = v4i{0, 0, 0, 0};
        for (int ta = ta0; ta <= ta1; ++ta) {
          const uint8_t *A0 = pa + (int64_t)(ta * nmod + l) * plane + tm * 4 * KB * 1024 + lane * 16;
          const uint8_t *B0 =
              pb + (int64_t)((g - ta) * nmod + l) * plane + tn * 4 * KB * 1024 + lane * 16;
          for (int64_t kb = 0; kb < KB; ++kb) {
            v4i af[4], bf[4];
  #pragma unroll
            for (int a = 0; a < 4; ++a) af[a] = *(const v4i *)(A0 + (a * KB + kb) * 1024);
  #pragma unroll
            for (int b = 0; b < 4; ++b) bf[b] = *(const v4i *)(B0 + (b * KB + kb) * 1024);
  #pragma unroll
            for (int a = 0; a < 4; ++a)
  #pragma unroll
              for (int b = 0; b < 4; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[a], bf[b], acc[a][b], 0, 0, 0);
          }
        }
        const uint32_t m = (uint32_t)pl->m[l];
        const double md = (double)m, yd = (double)pl->y[l], im = pl->inv_m[l];
  #pragma unroll
        for (int a = 0; a < 4; ++a)
  #pragma unroll
          for (int b = 0; b < 4; ++b) {
            uint32_t packed = 0;
  #pragma unroll
            for (int r = 0; r < 4; ++r) packed |= mod_times_y(acc[a][b][r], md, yd, im, m) << (8 * r);
            const int64_t row = tm * 64 + 16 * a + 4 * (lane >> 4);
            const int64_t col = tn * 64 + 16 * b + (lane & 15);
            *(uint32_t *)(tpl + ((int64_t)gl * Mp + col) * Mp + row) = packed;
          }
      }
    }
    __syncthreads();

    // (S5)+(S6) and A22 -= c: each wavefront takes 64 consecutive elements of
    // a column at a time through the matrix-core CRT, on its own slice of the
    // staging LDS (the route and results of k_consumer_mx)
    {
      constexpr int NB = 36, NWC = 12, ND = NB / 2, STG = stage_words<ND>();
      static_assert(64 * MX_TBS <= 32 * MX_CBS * 4 && 64 * STG <= 32 * MX_CBS, "LDS reuse");
      static_assert(NT / 64 * 32 * MX_CBS <= NT * CST, "one column-sum buffer per wavefront");
      int32_t *buf = (int32_t *)stage + wv * 32 * MX_CBS;
      uint32_t *st = (uint32_t *)buf + lane * STG;
      mxv4 tab[MX_BLK];
  #pragma unroll
      for (int b = 0; b < MX_BLK; ++b) tab[b] = *(const mxv4 *)&pl->crtm[b][lane][0];
      const int64_t ps = Mp * Mp;
      const int TMc = (int)(tm1 - tm0), chunks = (int)(tn1 - tn0) * 64 * TMc;
      for (int ch = wv; ch < chunks; ch += NT / 64) {
        const int64_t j = tn0 * 64 + ch / TMc, i0 = (tm0 + ch % TMc) * 64, i = i0 + lane;
        if (j >= m2) break;
        const bool valid = i < m2;
        const int32_t ej = eb[j], ei = valid ? ea[i] : EXP_ZERO;
        const bool zero = ei == EXP_ZERO || ej == EXP_ZERO;
        const int eps = zero ? 0 : w * g0 - (Q - 1 - ei) - (Q - 1 - ej);
        uint32_t cb[NWC];
  #pragma unroll
        for (int k = 0; k < NWC; ++k) cb[k] = 0u;
        for (int gi = 0; gi < ng; ++gi) {
          int32_t d[ND];
          crt_group_mx<NB, true>(tpl + (int64_t)gi * nmod * ps + j * Mp + i0, ps, nmod, pl, tab, buf,
                                 lane, d);
          add_shifted_digits<NWC, ND, STG>(cb, d, w * gi, st);
          mx_sync<true>();  // the buffer takes the next group's t-bytes
        }
        if (!valid) continue;
        double c[NC];
        if (zero) {
  #pragma unroll
          for (int q = 0; q < NC; ++q) c[q] = 0.0;
        } else {
          round_out_n<NWC, NC>(cb, eps, c);
        }
        double *dst = A22 + (i + j * n) * NC;
        double a[NC], nc_[NC], r[NC];
        ozx::load<NC>(dst, a);
  #pragma unroll
        for (int q = 0; q < NC; ++q) nc_[q] = -c[q];
        ozx::add<NC>(a, nc_, r);
        ozx::store<NC>(dst, r);
      }
    }
    __syncthreads();
  }
};

// ---------------------------------------------------------------------------
// Shared work.  A workgroup that finds the queue empty stays and helps those
// still factoring: once one is idle, the owner of a system offers U12 and the
// update of a step as tasks on its line of the board, takes tasks itself and
// goes on when all are done.  The tasks of phase 0 are U12 and its residues in
// chunks of 32 columns and the residues of L21 in chunks of 64 rows, those of
// phase 1 the 64 x 64 tiles of the update, those of phase 2 (inside the panel)
// the deferred steps of NT elements each; every element sees the operations it
// would see without help.  A task is taken by an atomic increment of the job
// word (priority << 32 | total << 16 | next) and runs to its end without
// waiting for anything, an owner waits only for tasks that were taken, and a
// helper leaves when every item is finished: no workgroup waits for one that
// does not run.  Both waits are bounded all the same: an owner whose tasks
// do not end raises the sticky error flag and leaves, a helper that sees
// nothing happen for as long just leaves.
// The owner's data reach the helpers, and the helpers' results the owner,
// through an agent-scope release by every wavefront before the increment (or
// the offer) and an acquire by every wavefront after it: the XCDs' L2s are not
// coherent.  The last and largest systems bound the launch, each on one CU of
// 256, so helpers take the job of the owner with the most work left (33.0 ms
// below; 34.6 in the order of the slots).  256 DD / QD systems of order 64 to
// 512, b = 64: 73.1 -> 32.9 ms, 16 of order 100 to 400 33.1 -> 12.7 ms, one of
// order 512 (QD) 66.7 -> 17.4 ms; with more work than CUs to the end (1000 of
// order 150 to 256) 33.2 -> 31.4 ms.
// ---------------------------------------------------------------------------
struct BatchSlot {  // a line of its own for each owner
  int32_t done, item, k0, phase;
  int32_t j0, j1, zeros;  // phase 2
  int32_t pad[25];
};
struct Board {
  // items taken, helpers (and CUs without a workgroup), items done, scratch
  // slots taken
  int32_t next, idle, finished, owners;
  int32_t pad[60];
  // followed by nslot job words (rounded up to 64) and nslot slots
  __device__ uint64_t *jobs() { return (uint64_t *)(this + 1); }
  __device__ BatchSlot *slots(int nslot) { return (BatchSlot *)(jobs() + ((nslot + 63) & ~63)); }
};
static_assert(sizeof(BatchSlot) == 128 && sizeof(Board) == 256, "board layout");

template <class T>
__device__ __forceinline__ T ld_agent(const T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void st_agent(T *p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ T add_agent(T *p, T v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// by all threads: what the workgroup wrote is visible to an acquirer
__device__ __forceinline__ void wg_release() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
}
// by all threads, after thread 0 saw the other side's word
__device__ __forceinline__ void wg_acquire() {
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

using ozb::ACH;
using ozb::SB;
using ozb::UCH;

template <int NC, int NWM, int NT>
__device__ __forceinline__ int tasks_of(const OzUpdate<NC, NWM, NT> &u, int phase) {
  return phase == 0 ? (int)(u.Mp / UCH + u.Mp / ACH) : (int)((u.Mp / 64) * (u.Mp / 64));
}

template <int NC, int NWM, int NT>
__device__ __forceinline__ void run_task(const OzUpdate<NC, NWM, NT> &u, int phase, int t,
                                         uint32_t *stage) {
  if (phase == 0) {
    const int nu = (int)(u.Mp / UCH);
    if (t < nu) {
      const int64_t c0 = (int64_t)t * UCH, c1 = c0 + UCH;
      if (c0 < u.m2) u.solve_u12(c0, c1 < u.m2 ? c1 : u.m2);
      u.residues(false, c0, c1);
    } else {
      u.residues(true, (int64_t)(t - nu) * ACH, (int64_t)(t - nu + 1) * ACH);
    }
  } else {
    const int tb = (int)(u.Mp / 64), tm = t % tb, tn = t / tb;
    u.tiles(tm, tm + 1, tn, tn + 1, stage);
  }
}

// Task t of the deferred steps j0 .. j1-1 on the panel's columns j1 .. k1-1,
// rows from j1 on: NT elements, one per thread, kept in registers through all
// steps; zeros: the steps with an exactly zero pivot, which update nothing.
template <int NC, int NT>
__device__ __forceinline__ void deferred_task(double *A, int64_t n, int j0, int j1, int k1,
                                              uint32_t zeros, int t) {
  const int mr = (int)n - j1, idx = t * NT + (int)threadIdx.x;
  if (idx >= mr * (k1 - j1)) return;
  const int i = j1 + idx % mr, c = j1 + idx / mr;
  const double *pl_ = A + (i + (int64_t)j0 * n) * NC, *pu = A + (j0 + (int64_t)c * n) * NC;
  double *dst = A + (i + (int64_t)c * n) * NC;
  double a[NC], l[NC], u[NC];
  ozx::load<NC>(dst, a);
  ozx::load<NC>(pl_, l);
  ozx::load<NC>(pu, u);
  for (int k = j0; k < j1; ++k) {
    double ln[NC], un[NC], o[NC];
    const bool more = k + 1 < j1;
    pl_ += more ? n * NC : 0;
    pu += more ? NC : 0;
    ozx::load<NC>(pl_, ln);
    ozx::load<NC>(pu, un);
    if (!((zeros >> (k - j0)) & 1u)) {
      ozx::fms<NC>(a, l, u, o);
#pragma unroll
      for (int q = 0; q < NC; ++q) a[q] = o[q];
    }
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      l[q] = ln[q];
      u[q] = un[q];
    }
  }
  ozx::store<NC>(dst, a);
}

// Ticks of the 100 MHz counter that an owner or helper waits: 10 s, a hundred
// times what the longest system takes alone.
constexpr uint64_t WAIT_TICKS = 1000000000ull;

// By the owner: the tasks 0 .. total-1, shared when there is a helper (share),
// else one after the other.  put() writes what the helpers need to the slot.
// False (for every thread) when a task that was taken did not end in time.
template <class P, class F>
__device__ __forceinline__ bool offer(bool share, int total, uint32_t prio, uint64_t *job,
                                      BatchSlot *sl, int *s_task, int *err, P put, F run) {
  if (!share) {
    for (int t = 0; t < total; ++t) run(t);
    __syncthreads();
    return true;
  }
  const int tid = threadIdx.x;
  if (tid == 0) {
    st_agent(&sl->done, 0);
    put();
  }
  wg_release();
  if (tid == 0) st_agent(job, (uint64_t)prio << 32 | (uint32_t)total << 16);
  int mine = 0;
  for (;; ++mine) {
    if (tid == 0) *s_task = (int)(add_agent(job, (uint64_t)1) & 0xffffu);
    __syncthreads();
    const int t = *s_task;
    __syncthreads();
    if (t >= total) break;
    run(t);
    __syncthreads();
  }
  if (tid == 0) {
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    *s_task = 0;
    while (ld_agent(&sl->done) + mine < total) {
      if (__builtin_amdgcn_s_memrealtime() - t0 > WAIT_TICKS) {
        st_agent(err, 4);
        *s_task = -1;
        break;
      }
      __builtin_amdgcn_s_sleep(4);
    }
  }
  wg_acquire();
  return *s_task == 0;
}

// False when a wait of offer() ran out; the item is then unfinished.
template <int NC, int NWM, int NT>
__device__ __forceinline__ bool lu_solve_oz(const ozII_batch_item &it, int item, int count, int cus,
                            double (*rkey)[4],
                            int64_t *ridx, int *s_info, const DevPlan *pl, uint8_t *ws, int b,
                            uint32_t *stage, double (*xs)[4], int64_t *pv, Board *bd, uint64_t *job,
                            BatchSlot *sl, int *s_task, int *err) {
  const int tid = threadIdx.x;
  const int64_t n = it.n;
  double *A = it.A;
  auto E = [&](int64_t i, int64_t c) { return A + (i + c * n) * NC; };
  // idle workgroups (the same answer for every thread)
  auto helpers = [&]() {
    __syncthreads();
    if (tid == 0) *s_task = ld_agent(&bd->idle);
    __syncthreads();
    const int h = *s_task;
    __syncthreads();
    return h;
  };
  // place among the systems that run last, by decreasing cost
  const int rank = max(0, item - max(0, count - (int)gridDim.x));
  if (tid == 0) *s_info = 0;
  __syncthreads();
  for (int64_t k0 = 0; k0 < n; k0 += b) {
    const int64_t k1 = k0 + b < n ? k0 + b : n;
    const uint32_t left = ozb::work_left(NC, n - k0);
    // deferring steps shortens the owner's work only where others take it:
    // 16 systems of order 100 to 400 17.6 -> 13.0 ms; without helpers it is 2 to
    // 3 % slower (700 of order 64 to 200, 12.25 -> 12.5 ms), and 256 systems
    // take 33.0 ms with the line at an eighth, a quarter or half of the CUs
    // idle, 33.3 at three quarters
    const bool many = ozb::worth_deferring(n - k0, k1 - k0) && helpers() * 2 > cus;
    const int64_t sb = many ? SB : b;
    for (int64_t j0 = k0; j0 < k1; j0 += sb) {
      // sub-block: its own columns see each step at once, the panel's other
      // columns all its steps together afterwards
      const int64_t j1 = j0 + sb < k1 ? j0 + sb : k1;
      uint32_t zeros = 0;
      for (int64_t j = j0; j < j1; ++j) {
        // no update after an exactly zero pivot (the column is left as it is,
        // as in LAPACK's unblocked panel)
        const bool zero = pivot_column<NC, NT>(it, j, rkey, ridx, s_info);
        zeros |= (uint32_t)zero << ((j - j0) & 31);
        fms_sweep<NC, NT>(zero ? 0 : (int32_t)(n - j - 1), (int32_t)(j1 - j - 1),
                          [&](int32_t i, int32_t c, double *&pa, const double *&pl_,
                              const double *&pu) {
                            pa = E(j + 1 + i, j + 1 + c);
                            pl_ = E(j + 1 + i, j);
                            pu = E(j, j + 1 + c);
                          });
        __syncthreads();
      }
      if (j1 == k1) break;
      // the sub-block's rows of the other columns step by step, then the rest
      for (int64_t k = j0; k + 1 < j1; ++k) {
        fms_sweep<NC, NT>((zeros >> (k - j0)) & 1u ? 0 : (int32_t)(j1 - k - 1), (int32_t)(k1 - j1),
                          [&](int32_t i, int32_t c, double *&pa, const double *&pl_,
                              const double *&pu) {
                            pa = E(k + 1 + i, j1 + c);
                            pl_ = E(k + 1 + i, k);
                            pu = E(k, j1 + c);
                          });
        __syncthreads();
      }
      const int total = (int)(((n - j1) * (k1 - j1) + NT - 1) / NT);
      const bool ok = offer(
          total > 1, total, left, job, sl, s_task, err,
          [&]() {
            st_agent(&sl->item, item);
            st_agent(&sl->k0, (int32_t)k0);
            st_agent(&sl->j0, (int32_t)j0);
            st_agent(&sl->j1, (int32_t)j1);
            st_agent(&sl->zeros, (int32_t)zeros);
            st_agent(&sl->phase, 2);
          },
          [&](int t) { deferred_task<NC, NT>(A, n, (int)j0, (int)j1, (int)k1, zeros, t); });
      if (!ok) return false;
    }
    if (k1 >= n) break;
    const OzUpdate<NC, NWM, NT> u(A, n, k0, k1, pl, ws);
    // one tile has nothing to share; and taking tiles one at a time costs an
    // owner 10 % (700 systems of order 64 to 200 12.2 -> 13.7 ms without a
    // helper), so only as many of the largest systems as there are helpers share:
    // of 256 systems half are done after 17.0 instead of 20.1 ms, all after 32.9
    // instead of 33.1
    if (u.m2 <= 64 || rank >= helpers()) {
      u.solve_u12(0, u.m2);
      u.residues(true, 0, u.Mp);
      u.residues(false, 0, u.Mp);
      __syncthreads();
      u.tiles(0, u.Mp / 64, 0, u.Mp / 64, stage);
      continue;
    }
    for (int phase = 0; phase < 2; ++phase) {
      const bool ok = offer(
          true, tasks_of(u, phase), left, job, sl, s_task, err,
          [&]() {
            st_agent(&sl->item, item);
            st_agent(&sl->k0, (int32_t)k0);
            st_agent(&sl->phase, phase);
          },
          [&](int t) { run_task(u, phase, t, stage); });
      if (!ok) return false;
    }
  }
  if (tid == 0) *it.info = *s_info;
  solve_one<NC, NT>(it, xs, pv);
  return true;
}

template <int NC, int NWM, int NT>
__device__ __forceinline__ void help(const ozII_batch_item &it, BatchSlot *sl, const DevPlan *pl,
                                     uint8_t *ws, int b, int t, uint32_t *stage) {
  const int phase = ld_agent(&sl->phase);
  const int64_t k0 = ld_agent(&sl->k0), k1 = k0 + b < it.n ? k0 + b : it.n;
  if (phase == 2)
    deferred_task<NC, NT>(it.A, it.n, ld_agent(&sl->j0), ld_agent(&sl->j1), (int)k1,
                          (uint32_t)ld_agent(&sl->zeros), t);
  else
    run_task(OzUpdate<NC, NWM, NT>(it.A, it.n, k0, k1, pl, ws), phase, t, stage);
}

// One workgroup of BTZ threads per CU (the update's stages need more than
// the 128 registers a 1024-thread workgroup leaves per thread); the
// consumer's per-thread staging shares the LDS with the pivot search (never
// live at the same time).
__global__ __launch_bounds__(BTZ) void k_batch_lu_oz(const ozII_batch_item *items, int count,
                                                    Board *bd, int nslot, int cus, uint64_t *times,
                                                    const DevPlan *pl2, const DevPlan *pl3,
                                                    const DevPlan *pl4, uint8_t *ws, int64_t slot,
                                                    int b, int *err) {
  __shared__ __attribute__((aligned(16))) uint32_t lds[BTZ * CST];
  static_assert(BTZ * CST * 4 >= BTZ * (32 + 8), "pivot search arrays fit the staging");
  double(*rkey)[4] = (double(*)[4])lds;
  int64_t *ridx = (int64_t *)(lds + BTZ * 8);
  // the solve's right-hand side and pivots too
  static_assert(BTZ * CST * 4 >= SOLVE_N * (32 + 8), "solve arrays fit the staging");
  double(*xs)[4] = (double(*)[4])lds;
  int64_t *pv = (int64_t *)(lds + SOLVE_N * 8);
  __shared__ int s_item, s_info, s_task;
  __shared__ int s_slot;
  BatchSlot *slots = bd->slots(nslot);
  if (threadIdx.x == 0) s_slot = -1;
  for (;;) {
    if (threadIdx.x == 0) {
      s_item = add_agent(&bd->next, 1);
      // at most min(count, workgroups) = nslot workgroups ever own an item
      if (s_item < count && s_slot < 0) s_slot = add_agent(&bd->owners, 1);
    }
    __syncthreads();
    const int q = s_item, ms = s_slot;
    __syncthreads();
    if (q >= count) break;
    const ozII_batch_item it = items[q];
    uint8_t *myws = ws + (int64_t)ms * slot;
    if (times && threadIdx.x == 0) times[2 * it.reserved] = __builtin_amdgcn_s_memrealtime();
    bool ok;
#define OZ_LU(NC_, NWM_, PL_)                                                                       \
  ok = lu_solve_oz<NC_, NWM_, BTZ>(it, q, count, cus, rkey, ridx, &s_info, PL_, myws, b, lds, xs, \
                                   pv, bd, bd->jobs() + ms, slots + ms, &s_task, err)
    if (it.nc == 2) OZ_LU(2, 6, pl2);
    else if (it.nc == 3) OZ_LU(3, 4, pl3);
    else OZ_LU(4, 4, pl4);
#undef OZ_LU
    if (!ok) return;
    __syncthreads();
    if (threadIdx.x == 0) {
      if (times) {
        __builtin_amdgcn_s_waitcnt(0x0F70);
        times[2 * it.reserved + 1] = __builtin_amdgcn_s_memrealtime();
      }
      add_agent(&bd->finished, 1);
    }
  }
  // the queue is empty: help until every item is finished
  if (threadIdx.x == 0) add_agent(&bd->idle, 1);
  const int lane = threadIdx.x & 63;
  for (;;) {
    if (threadIdx.x < 64) {
      int got = -1, seen = -1;
      uint64_t since = 0;
      while (got < 0) {
        const int fin = __builtin_amdgcn_readfirstlane(ld_agent(&bd->finished));
        const uint64_t now = __builtin_amdgcn_s_memrealtime();
        since = fin == seen ? since : now;
        seen = fin;
        const bool over = fin >= count || now - since > WAIT_TICKS;
        // the open job of the owner with the most work left
        uint32_t best = 0;
        int bs = -1;
        for (int s = lane; s < nslot; s += 64) {
          const uint64_t v = ld_agent(bd->jobs() + s);
          const uint32_t pr = (uint32_t)(v >> 32);
          if (((uint32_t)v & 0xffffu) < ((uint32_t)v >> 16) && pr > best) {
            best = pr;
            bs = s;
          }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
          const uint32_t ob = (uint32_t)__shfl_xor((int)best, off, 64);
          const int os = __shfl_xor(bs, off, 64);
          if (ob > best || (ob == best && os > bs)) {
            best = ob;
            bs = os;
          }
        }
        bs = __builtin_amdgcn_readfirstlane(bs);
        if (bs >= 0) {
          uint32_t v = 0;
          if (lane == 0) v = (uint32_t)add_agent(bd->jobs() + bs, (uint64_t)1);
          v = (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
          if ((v & 0xffffu) < (v >> 16)) {
            got = bs;
            if (lane == 0) s_task = (int)(v & 0xffffu);
          }
        }
        if (got < 0) {
          if (over) break;
          if (bs < 0) __builtin_amdgcn_s_sleep(32);
          else __builtin_amdgcn_s_sleep(4);
        }
      }
      if (lane == 0) s_slot = got;
    }
    wg_acquire();
    const int hs = s_slot, t = s_task;
    __syncthreads();
    if (hs < 0) break;
    const ozII_batch_item it = items[ld_agent(&slots[hs].item)];
    uint8_t *hws = ws + (int64_t)hs * slot;
    if (it.nc == 2) help<2, 6, BTZ>(it, slots + hs, pl2, hws, b, t, lds);
    else if (it.nc == 3) help<3, 4, BTZ>(it, slots + hs, pl3, hws, b, t, lds);
    else help<4, 4, BTZ>(it, slots + hs, pl4, hws, b, t, lds);
    wg_release();
    if (threadIdx.x == 0) add_agent(&slots[hs].done, 1);
  }
}

__global__ __launch_bounds__(BT) void k_batch_lu(const ozII_batch_item *items, int count,
                                                 int *queue, uint64_t *times) {
  __shared__ double rkey[BT][4];
  __shared__ int64_t ridx[BT];
  __shared__ int s_item, s_info;
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(queue, 1);
    __syncthreads();
    const int q = s_item;
    __syncthreads();
    if (q >= count) break;  // every workgroup leaves once the queue is empty
    const ozII_batch_item it = items[q];  // reserved = the item's index in the caller's order
    if (times && threadIdx.x == 0) times[2 * it.reserved] = __builtin_amdgcn_s_memrealtime();
    if (it.nc == 2) lu_solve_one<2>(it, rkey, ridx, &s_info);
    else if (it.nc == 3) lu_solve_one<3>(it, rkey, ridx, &s_info);
    else lu_solve_one<4>(it, rkey, ridx, &s_info);
    __syncthreads();
    if (times && threadIdx.x == 0) {
      // the item's global writes are complete before its end stamp
      __builtin_amdgcn_s_waitcnt(0x0F70);
      times[2 * it.reserved + 1] = __builtin_amdgcn_s_memrealtime();
    }
  }
}

__global__ void k_batch_clear(int *words, int count, int idle) {
  for (int i = threadIdx.x; i < count; i += blockDim.x) words[i] = i == 1 ? idle : 0;
}

}  // namespace

namespace ozl {
hipError_t launch_batch(const ozII_batch_item *items, int count, int *queue, uint64_t *times,
                        int grid, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_batch_clear, dim3(1), dim3(64), 0, s, queue, 1, 0);
  hipLaunchKernelGGL(k_batch_lu, dim3((unsigned)grid), dim3(BT), 0, s, items, count, queue, times);
  return hipGetLastError();
}
size_t batch_board_bytes(int nslot) {
  return sizeof(Board) + (size_t)((nslot + 63) / 64 * 64) * 8 + (size_t)nslot * sizeof(BatchSlot);
}

hipError_t launch_batch_oz(const ozII_batch_item *items, int count, void *board, int nslot,
                          uint64_t *times, int grid, int cus, const DevPlan *pl2,
                          const DevPlan *pl3, const DevPlan *pl4, uint8_t *ws, int64_t slot, int b,
                          int *err, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  if (b < 1 || b > 256 || nslot < std::min(count, grid) || grid > cus) return hipErrorInvalidValue;
  static_assert(offsetof(Board, idle) == 4, "the word that k_batch_clear sets");
  hipLaunchKernelGGL(k_batch_clear, dim3(1), dim3(256), 0, s, (int *)board,
                     (int)(sizeof(Board) / 4) + (nslot + 63) / 64 * 128, cus - grid);
  hipLaunchKernelGGL(k_batch_lu_oz, dim3((unsigned)grid), dim3(BTZ), 0, s, items, count,
                     (Board *)board, nslot, cus, times, pl2, pl3, pl4, ws, slot, b, err);
  return hipGetLastError();
}
}  // namespace ozl
