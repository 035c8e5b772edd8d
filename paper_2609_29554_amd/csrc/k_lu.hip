// LU kernels for gfx950 around the Ozaki-II update (Sec. 3.4 of the paper):
//   (P1) panel factorisation with partial pivoting,
//   (P2) row interchanges (laswp),
//   (P3) U12 = L11^{-1} A12,
//   the native expansion product C -= A B (blocked-naive comparator and the
//   triangular-solve updates), and the pieces of the solve (getrs).
// All multiple-precision arithmetic here is the expansion arithmetic of
// expansion.hpp; every element sees its multiply-subtracts in the order the
// specification fixes (ascending inner index, descending in the backward
// substitution).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "expansion.hpp"
#include "ozii_kernels.hpp"
#include "panel_tags.hpp"

namespace {

// ---------------------------------------------------------------------------
// Exchange between the workgroups of the cooperative panel kernel.
//
// Each workgroup owns two 128-byte candidate lines (one per parity of the
// pivot column) with its pivot candidate for that column -- its row position,
// its physical row and its value in the pivot column -- and two row buffers
// with the rest of that row.  Every 8-byte word carries 32 bits of payload
// and the 32-bit tag of its column, so a reader that sees the tag has the
// payload: one round trip, no arrival counter, no wait of the writer for its
// stores and no fence.  Words are written and read with device-coherent
// 8-byte accesses.  A line is overwritten two columns later, which its owner
// reaches only after every workgroup has published the column in between,
// and a workgroup publishes that after it has read all it needs of the first.
// Every panel of a handle has tags of its own (panel_tags.hpp; a device word
// that k_getrf_begin advances, so that replays of a captured factorisation
// take new ones), so nothing has to be cleared until 2^22 panels have used them
// up.  Waits are bounded: a timeout raises the sticky error flag and ends the
// kernel.
// ---------------------------------------------------------------------------
constexpr int LINE_WORDS = 16;  // 8-byte words per candidate line

__device__ __forceinline__ uint32_t ld_dev_u32(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double ld_dev_f64(const double *p) {
  const uint64_t v = __hip_atomic_load((const uint64_t *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  double d;
  __builtin_memcpy(&d, &v, 8);
  return d;
}

__device__ __forceinline__ uint64_t ld_dev_u64(const uint64_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_tagged(uint64_t *p, uint32_t v, uint32_t tag) {
  __hip_atomic_store(p, ((uint64_t)tag << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// a double as two tagged words, low half first
__device__ __forceinline__ void st_tagged_f64(uint64_t *p, double v, uint32_t tag) {
  uint64_t u;
  __builtin_memcpy(&u, &v, 8);
  st_tagged(p, (uint32_t)u, tag);
  st_tagged(p + 1, (uint32_t)(u >> 32), tag);
}
__device__ __forceinline__ double join_f64(uint64_t lo, uint64_t hi) {
  const uint64_t u = (hi << 32) | (uint32_t)lo;
  double d;
  __builtin_memcpy(&d, &u, 8);
  return d;
}

// One step of a bounded wait: true when it has to be given up, because about
// a second has passed (100 MHz real-time counter) or another wait failed.
__device__ __forceinline__ bool wait_expired(uint32_t &spins, uint64_t t0, int *err,
                                             int code = 1) {
  if ((++spins & 63u) != 0) return false;
  if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return true;
  if (__builtin_amdgcn_s_memrealtime() - t0 <= 100000000ull) return false;
  __hip_atomic_store(err, code, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// Candidate order of the pivot search: larger |value| first, then the lower
// row position.  A total order on (key, position) pairs, so any reduction
// tree picks the same winner.
template <int NC>
__device__ __forceinline__ bool cand_better(const double (&kb_)[NC], int pb, int ib,
                                            const double (&ka)[NC], int pa, int ia) {
  if (ib < 0) return false;
  if (ia < 0) return true;
  if (ozx::abs_greater<NC>(kb_, ka)) return true;
  if (ozx::abs_greater<NC>(ka, kb_)) return false;
  return pb < pa;
}

// Partner value of a 64-bit / 32-bit word under a DPP lane pattern (CTRL:
// quad_perm or row mirror, never out of range); every lane of the
// wavefront must call it.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  uint64_t u;
  __builtin_memcpy(&u, &x, 8);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, false);
  const uint64_t v = ((uint64_t)hi << 32) | lo;
  double d;
  __builtin_memcpy(&d, &v, 8);
  return d;
}
template <int CTRL>
__device__ __forceinline__ int dpp_i32(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, false);
}

// The best candidate of the wavefront in every lane (cand_better is a total
// order, so any pairing network that meets every lane gives the same one):
// lanes 32 and 16 apart through the LDS crossbar, then within each row of 16
// by DPP (mirror, half mirror, quad swaps), which needs no LDS round trip.
// All 64 lanes must call it.
template <int NC>
__device__ __forceinline__ void cand_allreduce(double (&k)[NC], int &pos, int &idx) {
  auto take = [&](const double (&ok)[NC], int op, int oi) {
    if (cand_better<NC>(ok, op, oi, k, pos, idx)) {
#pragma unroll
      for (int q = 0; q < NC; ++q) k[q] = ok[q];
      pos = op;
      idx = oi;
    }
  };
#pragma unroll
  for (int off = 32; off >= 16; off >>= 1) {
    double ok[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) ok[q] = __shfl_xor(k[q], off, 64);
    take(ok, __shfl_xor(pos, off, 64), __shfl_xor(idx, off, 64));
  }
#define OZ_DPP_STEP(CTRL)                                         \
  do {                                                            \
    double ok[NC];                                                \
    _Pragma("unroll") for (int q = 0; q < NC; ++q) ok[q] = dpp_f64<CTRL>(k[q]); \
    take(ok, dpp_i32<CTRL>(pos), dpp_i32<CTRL>(idx));              \
  } while (0)
  OZ_DPP_STEP(0x140);  // row_mirror: lane i <-> 15 - i of its row
  OZ_DPP_STEP(0x141);  // row_half_mirror: i <-> 7 - i of its half row
  OZ_DPP_STEP(0x4E);   // quad_perm [2, 3, 0, 1]
  OZ_DPP_STEP(0xB1);   // quad_perm [1, 0, 3, 2]
#undef OZ_DPP_STEP
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {
  uint64_t u;
  __builtin_memcpy(&u, &v, 8);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  const uint64_t w = ((uint64_t)hi << 32) | lo;
  double d;
  __builtin_memcpy(&d, &w, 8);
  return d;
}

__device__ __forceinline__ double wave_max_f64(double v) {
  v = fmax(v, __shfl_xor(v, 32, 64));
  v = fmax(v, __shfl_xor(v, 16, 64));
  v = fmax(v, dpp_f64<0x140>(v));
  v = fmax(v, dpp_f64<0x141>(v));
  v = fmax(v, dpp_f64<0x4E>(v));
  v = fmax(v, dpp_f64<0xB1>(v));
  return v;
}

// Leading-magnitude shortcut of the candidate order.  Each lane of a
// wavefront has reduced its own candidates to lead = the largest |k[0]|
// among them (-1 for none, NaN if one is NaN) and nlead = how many reach
// it.  The order compares |k[0]| first, so when the largest leading
// magnitude belongs to exactly one candidate, that one wins whatever its
// other components and position: returns 1 and its lane in w.  Returns 0
// when no lane has a candidate, 2 when the full order has to decide (equal
// leading magnitudes, NaN).  All 64 lanes must call it; the result is
// uniform.
__device__ __forceinline__ int lead_winner(double lead, int nlead, int &w) {
  const double M = wave_max_f64(lead);
  const uint64_t hit = __ballot(lead == M);
  const uint64_t odd = __ballot(lead != lead || (lead == M && nlead > 1));
  if (odd != 0) return 2;
  if (M < 0.0) return 0;
  if (__popcll(hit) != 1) return 2;
  w = __ffsll((unsigned long long)hit) - 1;
  return 1;
}

constexpr int PANEL_NT = 512;  // threads per panel workgroup
constexpr int PANEL_NW = PANEL_NT - 64;  // of these, the ones that apply the updates

// Before the panels of a factorisation: info, and a fresh range of tags for
// each; a workgroup, for the time when the exchange words have to be cleared.
constexpr int BEGIN_NT = 256;
__global__ __launch_bounds__(BEGIN_NT) void k_getrf_begin(uint32_t *epoch, uint32_t panels,
                                                          int32_t *info, uint64_t *lines,
                                                          int64_t line_words, uint64_t *crow,
                                                          int64_t crow_words) {
  const ozp::TagRange r = ozp::next_tags(*epoch, panels);
  __syncthreads();
  if (r.clear) {
    for (int64_t i = threadIdx.x; i < line_words; i += BEGIN_NT) lines[i] = 0;
    for (int64_t i = threadIdx.x; i < crow_words; i += BEGIN_NT) crow[i] = 0;
  }
  if (threadIdx.x == 0) {
    *epoch = r.end;
    *info = 0;
  }
}

// ---------------------------------------------------------------------------
// (P1) panel.  Panel rows [k, n), columns [k, k+kb).  Workgroup w owns the
// physical rows k + w*R .. k + w*R + R - 1 and keeps them in LDS for the
// whole panel.  Rows are never moved during the panel: the row permutation
// is tracked in LDS (position -> physical row and back, every workgroup
// keeping an identical copy) and applied once afterwards.
//
// The columns form one dependent chain, and wavefront 0 of every workgroup
// walks it alone: per column j it reads the candidates of all workgroups
// straight into registers as they arrive (largest |value|, ties to the lowest
// position: LAPACK's i?amax on the permuted column), divides its active rows
// (one per lane) by the pivot, updates column j+1, picks the local candidate
// of that column and publishes it.  The other wavefronts fetch the pivot row
// while it divides, then finish and publish the candidate's row and apply
// the rank-1 update to the rest, which may last until wavefront 0 has
// divided the next column.  Two barriers per column: after the division and
// after the choice of the candidate.  Every element still receives its
// multiply-subtracts in column order.
//
// Bound by the latency of that chain: the exchange across the XCDs (one store
// and one load), then in QD a division (3.5 us) and a multiply-subtract.
// getrf on MI355X against the same kernel with an arrival counter, separate
// payload reads and eight barriers per column: QD n = 2048, b = 128 31.0 ->
// 25.8 ms, DD n = 130, b = 32 1.07 -> 0.81 ms.
// ---------------------------------------------------------------------------
template <int NC>
__global__ __launch_bounds__(PANEL_NT) void k_panel(double *A, int64_t lda, int64_t n, int64_t k,
                                                    int kb, int R, int64_t *ipiv, int32_t *info,
                                                    uint64_t *lines, int *err, uint64_t *crow,
                                                    const uint32_t *epoch, int panel,
                                                    int *perm_out, int *moved, int *nmoved) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  // the panel is the critical path of the factorisation, and with
  // look-ahead the previous step's Schur update runs beside it on the same
  // CUs: its wavefronts take the SIMDs' issue slots first, and wavefront 0,
  // which walks the chain, before the one it shares a SIMD with
  if (threadIdx.x < 64) __builtin_amdgcn_s_setprio(3);
  else __builtin_amdgcn_s_setprio(2);
  const int nr = (int)(n - k);
  const int G = gridDim.x, wg = blockIdx.x, tid = threadIdx.x;
  double *rows = (double *)smem_raw;                 // R * kb * NC
  double *pivs = rows + (size_t)R * kb * NC;         // 2 * kb * NC, by column parity
  int *sperm = (int *)(pivs + (size_t)2 * kb * NC);  // nr
  int *sinv = sperm + nr;                            // nr
  __shared__ int s_seq, s_fail, s_info, s_best;
  __shared__ int s_wi[2], s_zero[2];
  __shared__ uint32_t s_active[2];

  const int r0 = wg * R;
  const int cnt = r0 < nr ? (nr - r0 < R ? nr - r0 : R) : 0;
  const uint32_t tag0 = ozp::panel_tag0(*epoch, (uint32_t)panel);
  auto RW = [&](int r, int c) { return rows + ((size_t)r * kb + c) * NC; };
  auto LINE = [&](int b, int w) { return lines + ((size_t)b * G + w) * LINE_WORDS; };
  auto CROW = [&](int b, int w) { return crow + ((size_t)b * G + w) * kb * NC * 2; };

  for (int idx = tid; idx < cnt * kb; idx += PANEL_NT) {
    const int r = idx % cnt, c = idx / cnt;
    const double *src = A + ((k + r0 + r) + (k + c) * lda) * NC;
#pragma unroll
    for (int q = 0; q < NC; ++q) RW(r, c)[q] = src[q];
  }
  for (int p = tid; p < nr; p += PANEL_NT) {
    sperm[p] = p;
    sinv[p] = p;
  }
  if (tid == 0) {
    s_seq = 0;
    s_fail = 0;
    s_info = 0;
    s_best = -1;
  }
  __syncthreads();
  // rows not yet chosen as pivots (wavefront 0)
  uint32_t active = cnt >= 32 ? 0xffffffffu : ((1u << cnt) - 1u);

  // wavefront 0, lane r holding row r's value x of column c (live: the row
  // is active): the local candidate, its line published
  auto choose = [&](const double (&x)[NC], bool live, int c) {
    double ck[NC];
    int cpos = 0x7fffffff, cidx = -1, w = 0;
#pragma unroll
    for (int q = 0; q < NC; ++q) ck[q] = live ? x[q] : 0.0;
    if (live) {
      cpos = sinv[r0 + tid];
      cidx = tid;
    }
    const int how = lead_winner(live ? fabs(ck[0]) : -1.0, 1, w);
    if (how == 1) cidx = w;
    else if (how == 2) cand_allreduce<NC>(ck, cpos, cidx);
    else cidx = -1;
    uint64_t *ln = LINE(c & 1, wg);
    const uint32_t tag = tag0 + (uint32_t)c;
    if (tid == (cidx < 0 ? 0 : cidx)) {
      st_tagged(ln, cidx < 0 ? 0x7fffffffu : (uint32_t)cpos, tag);
      st_tagged(ln + 1, cidx < 0 ? 0xffffffffu : (uint32_t)(r0 + cidx), tag);
#pragma unroll
      for (int q = 0; q < NC; ++q) st_tagged_f64(ln + 2 + 2 * q, x[q], tag);
      s_best = cidx;
    }
  };
  if (tid < 64) {
    double x[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) x[q] = tid < cnt ? RW(tid, 0)[q] : 0.0;
    choose(x, tid < cnt, 0);
  }
  __syncthreads();
  if (s_best >= 0) {
    uint64_t *cr = CROW(0, wg);
    for (int idx = NC + tid; idx < kb * NC; idx += PANEL_NT)
      st_tagged_f64(cr + 2 * (size_t)idx, RW(s_best, 0)[idx], tag0);
  }

  for (int j = 0; j < kb; ++j) {
    const int buf = j & 1;
    const uint32_t tag = tag0 + (uint32_t)j;
    const bool last = j + 1 >= kb;
    double *piv = pivs + (size_t)buf * kb * NC;
    double l[NC];  // wavefront 0: this lane's multiplier
#pragma unroll
    for (int q = 0; q < NC; ++q) l[q] = 0.0;
    bool live = false;
    if (tid < 64) {
      // the best of this lane's lines, two polled at a time
      double bk[NC];
      int bp = 0x7fffffff, bi = -1, bph = -1;
#pragma unroll
      for (int q = 0; q < NC; ++q) bk[q] = 0.0;
      bool expired = false;
      const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
      uint32_t spins = 0;
      for (int g0 = tid; g0 < G; g0 += 128) {
        const bool two = g0 + 64 < G;
        const uint64_t *la = LINE(buf, g0), *lb = LINE(buf, two ? g0 + 64 : g0);
        uint64_t wa[2 + 2 * NC], wb[2 + 2 * NC];
        // many lines: only the last word of each until it is there, since the
        // readers' traffic grows with the square of the workgroups (getrf QD n
        // = 2048 25.5 -> 25.0 ms; DD n = 130, 8 workgroups, 0.82 -> 0.85)
        while (G > 32) {
          const uint64_t ea = ld_dev_u64(la + 1 + 2 * NC), eb = ld_dev_u64(lb + 1 + 2 * NC);
          if ((uint32_t)(ea >> 32) == tag && (uint32_t)(eb >> 32) == tag) break;
          if (wait_expired(spins, t0, err)) {
            expired = true;
            break;
          }
        }
        if (expired) break;
        for (;;) {
#pragma unroll
          for (int q = 0; q < 2 + 2 * NC; ++q) wa[q] = ld_dev_u64(la + q);
#pragma unroll
          for (int q = 0; q < 2 + 2 * NC; ++q) wb[q] = ld_dev_u64(lb + q);
          bool ok = true;
#pragma unroll
          for (int q = 0; q < 2 + 2 * NC; ++q)
            ok = ok && (uint32_t)(wa[q] >> 32) == tag && (uint32_t)(wb[q] >> 32) == tag;
          if (ok) break;
          if (wait_expired(spins, t0, err)) {
            expired = true;
            break;
          }
        }
        if (expired) break;
        auto take = [&](const uint64_t (&w)[2 + 2 * NC], int g) {
          double kk[NC];
#pragma unroll
          for (int q = 0; q < NC; ++q) kk[q] = join_f64(w[2 + 2 * q], w[3 + 2 * q]);
          const int ph = (int)(uint32_t)w[1], pos = (int)(uint32_t)w[0];
          if (cand_better<NC>(kk, pos, ph >= 0 ? g : -1, bk, bp, bi)) {
#pragma unroll
            for (int q = 0; q < NC; ++q) bk[q] = kk[q];
            bp = pos;
            bi = g;
            bph = ph;
          }
        };
        take(wa, g0);
        if (two) take(wb, g0 + 64);
      }
      const bool fail = __ballot(expired) != 0;
      // the winner over the lanes: its entry in every lane
      int w = 0;
      const int how = lead_winner(bi >= 0 ? fabs(bk[0]) : -1.0, 1, w);
      if (how == 2) {
        int wi = bi;
        double tk[NC];
        int tp = bp;
#pragma unroll
        for (int q = 0; q < NC; ++q) tk[q] = bk[q];
        cand_allreduce<NC>(tk, tp, wi);
        w = __ffsll((unsigned long long)__ballot(bi == wi)) - 1;
      }
      const int wi = __builtin_amdgcn_readlane(bi, w), ppos = __builtin_amdgcn_readlane(bp, w);
      const int pphys = __builtin_amdgcn_readlane(bph, w);
      double d[NC];
      bool zero = true;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        d[q] = readlane_f64(bk[q], w);
        zero = zero && d[q] == 0.0;
      }
      // an empty or inconsistent table can only follow a failed wait
      const bool bad = fail || how == 0 || wi < 0 || ppos < j || ppos >= nr || pphys < 0 || pphys >= nr;
      if (!bad && pphys >= r0 && pphys < r0 + cnt) active &= ~(1u << (pphys - r0));
      if (tid == 0) {
        if (bad) {
          if (!fail) __hip_atomic_store(err, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          s_fail = 1;
        } else {
#pragma unroll
          for (int q = 0; q < NC; ++q) piv[(size_t)j * NC + q] = d[q];
          const int q = sperm[j];
          sperm[j] = pphys;
          sperm[ppos] = q;
          sinv[pphys] = j;
          sinv[q] = ppos;
          if (zero && s_info == 0) s_info = (int)(k + j + 1);
          if (wg == 0) ipiv[k + j] = k + ppos;
        }
        s_wi[buf] = bad ? -1 : wi;
        s_zero[buf] = zero ? 1 : 0;
        s_active[buf] = active;
        // the other wavefronts may fetch the pivot row now
        __hip_atomic_store(&s_seq, j + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      live = !bad && tid < cnt && ((active >> (tid & 31)) & 1u);
      if (live && !zero) {
        double a[NC];
        ozx::load<NC>(RW(tid, j), a);
        ozx::div<NC>(a, d, l);
        ozx::store<NC>(RW(tid, j), l);
      }
    } else {
      // columns j+1 .. kb-1 of the pivot row
      while (__hip_atomic_load(&s_seq, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) <= j)
        __builtin_amdgcn_s_sleep(1);
      const int wi = s_wi[buf];
      if (wi >= 0) {
        const uint64_t *cr = CROW(buf, wi) + 2 * (size_t)(j + 1) * NC;
        double *pd = piv + (size_t)(j + 1) * NC;
        const int total = (kb - j - 1) * NC;
        const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
        uint32_t spins = 0;
        constexpr int PF = 2;
        for (int b0 = tid - 64; b0 < total; b0 += PANEL_NW * PF) {
          uint64_t lo[PF], hi[PF];
          bool expired = false;
          for (;;) {
            bool ok = true;
#pragma unroll
            for (int u = 0; u < PF; ++u) {
              const int idx = b0 + u * PANEL_NW < total ? b0 + u * PANEL_NW : b0;
              lo[u] = ld_dev_u64(cr + 2 * (size_t)idx);
              hi[u] = ld_dev_u64(cr + 2 * (size_t)idx + 1);
            }
#pragma unroll
            for (int u = 0; u < PF; ++u)
              ok = ok && (uint32_t)(lo[u] >> 32) == tag && (uint32_t)(hi[u] >> 32) == tag;
            if (ok) break;
            if (wait_expired(spins, t0, err)) {
              expired = true;
              break;
            }
          }
          if (expired) {
            s_fail = 1;
            break;
          }
#pragma unroll
          for (int u = 0; u < PF; ++u) {
            const int idx = b0 + u * PANEL_NW;
            if (idx < total) pd[idx] = join_f64(lo[u], hi[u]);
          }
        }
      }
    }
    __syncthreads();
    if (s_fail) {
      if (wg == 0 && tid == 0) *nmoved = 0;  // no interchange after a failed wait
      return;
    }
    if (last) break;
    const int zero = s_zero[buf];
    if (tid < 64) {
      // column j+1 of the active rows, and this workgroup's candidate in it
      double x[NC];
#pragma unroll
      for (int q = 0; q < NC; ++q) x[q] = 0.0;
      if (live) {
        ozx::load<NC>(RW(tid, j + 1), x);
        if (!zero) {
          double u[NC], o[NC];
          ozx::load<NC>(piv + (size_t)(j + 1) * NC, u);
          ozx::fms<NC>(x, l, u, o);
          ozx::store<NC>(RW(tid, j + 1), o);
#pragma unroll
          for (int q = 0; q < NC; ++q) x[q] = o[q];
        }
      }
      choose(x, live, j + 1);
    }
    __syncthreads();
    if (tid >= 64) {
      const int best = s_best, width = kb - j - 2;
      const uint32_t act = s_active[buf];
      // the candidate's row first, published as it is finished
      if (best >= 0) {
        uint64_t *cr = CROW(buf ^ 1, wg);
        for (int c = j + 2 + tid - 64; c < kb; c += PANEL_NW) {
          double x[NC];
          ozx::load<NC>(RW(best, c), x);
          if (!zero) {
            double lv[NC], u[NC], o[NC];
            ozx::load<NC>(RW(best, j), lv);
            ozx::load<NC>(piv + (size_t)c * NC, u);
            ozx::fms<NC>(x, lv, u, o);
            ozx::store<NC>(RW(best, c), o);
#pragma unroll
            for (int q = 0; q < NC; ++q) x[q] = o[q];
          }
#pragma unroll
          for (int q = 0; q < NC; ++q)
            st_tagged_f64(cr + 2 * ((size_t)c * NC + q), x[q], tag + 1u);
        }
      }
      // the rest of the rank-1 update
      if (!zero && width > 0) {
        for (int idx = tid - 64; idx < cnt * width; idx += PANEL_NW) {
          const int r = idx % cnt, c = j + 2 + idx / cnt;
          if (((act >> r) & 1u) && r != best) {
            double a[NC], lv[NC], u[NC], o[NC];
            ozx::load<NC>(RW(r, c), a);
            ozx::load<NC>(RW(r, j), lv);
            ozx::load<NC>(piv + (size_t)c * NC, u);
            ozx::fms<NC>(a, lv, u, o);
            ozx::store<NC>(RW(r, c), o);
          }
        }
      }
    }
  }
  // write the rows back to their physical places
  for (int idx = tid; idx < cnt * kb; idx += PANEL_NT) {
    const int r = idx % cnt, c = idx / cnt;
    double *dst = A + ((k + r0 + r) + (k + c) * lda) * NC;
#pragma unroll
    for (int q = 0; q < NC; ++q) dst[q] = RW(r, c)[q];
  }
  if (wg == 0) {
    __shared__ int s_nm;
    if (tid == 0) s_nm = 0;
    __syncthreads();
    for (int p = tid; p < nr; p += PANEL_NT) {
      perm_out[p] = sperm[p];
      if (sperm[p] != p) {
        const int slot = atomicAdd(&s_nm, 1);
        moved[slot] = p;
      }
    }
    __syncthreads();
    if (tid == 0) {
      *nmoved = s_nm;
      if (s_info != 0 && *info == 0) *info = s_info;
    }
  }
}

// ---------------------------------------------------------------------------
// (P2) apply the panel's row permutation to columns [c0, c1):
// new row k+p = old row k+perm[p] for every moved position p.
// ---------------------------------------------------------------------------
template <int NC>
__global__ __launch_bounds__(256) void k_laswp(double *A, int64_t lda, int64_t k, int64_t c0,
                                               int64_t c1, const int *perm, const int *moved,
                                               const int *nmoved) {
  const int64_t c = c0 + blockIdx.x;
  if (c >= c1) return;
  const int nm = *nmoved;
  constexpr int PER = 4;  // up to 1024 moved positions per column
  double v[PER][NC];
  int pos[PER];
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int e = threadIdx.x + 256 * t;
    pos[t] = -1;
    if (e < nm) {
      const int p = moved[e];
      pos[t] = p;
      ozx::load<NC>(A + ((k + perm[p]) + c * lda) * NC, v[t]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < PER; ++t)
    if (pos[t] >= 0) ozx::store<NC>(A + ((k + pos[t]) + c * lda) * NC, v[t]);
}

// ---------------------------------------------------------------------------
// (P3) X <- L^{-1} X for a unit lower-triangular kb x kb block L (at Lp, ld
// lda) and kb x ncols right-hand sides X (at Xp, ld ldx): element i is
// updated for h = 0 .. i-1 in ascending order.  One workgroup per CPB
// columns; thread t owns rows t, t+256, ...
// ---------------------------------------------------------------------------
template <int NC, int CPB, int RPT>
__global__ __launch_bounds__(256) void k_trsm_lower_unit(const double *Lp, int64_t lda, double *Xp,
                                                         int64_t ldx, int kb, int64_t ncols) {
  __shared__ double xs[2][CPB][NC];
  const int tid = threadIdx.x;
  const int64_t cbase = (int64_t)blockIdx.x * CPB;
  double x[RPT][CPB][NC];
#pragma unroll
  for (int rr = 0; rr < RPT; ++rr) {
    const int i = tid + 256 * rr;
#pragma unroll
    for (int cc = 0; cc < CPB; ++cc) {
      const int64_t c = cbase + cc;
      if (i < kb && c < ncols) ozx::load<NC>(Xp + (i + c * ldx) * NC, x[rr][cc]);
      else
#pragma unroll
        for (int q = 0; q < NC; ++q) x[rr][cc][q] = 0.0;
    }
  }
  for (int h = 0; h < kb; ++h) {
    const int b = h & 1;
    if (tid == (h & 255)) {
#pragma unroll
      for (int rr = 0; rr < RPT; ++rr)
        if (rr == h / 256)
#pragma unroll
          for (int cc = 0; cc < CPB; ++cc)
#pragma unroll
            for (int q = 0; q < NC; ++q) xs[b][cc][q] = x[rr][cc][q];
    }
    __syncthreads();
#pragma unroll
    for (int rr = 0; rr < RPT; ++rr) {
      const int i = tid + 256 * rr;
      if (i > h && i < kb) {
        double l[NC];
        ozx::load<NC>(Lp + (i + (int64_t)h * lda) * NC, l);
#pragma unroll
        for (int cc = 0; cc < CPB; ++cc) {
          double u[NC], o[NC];
#pragma unroll
          for (int q = 0; q < NC; ++q) u[q] = xs[b][cc][q];
          ozx::fms<NC>(x[rr][cc], l, u, o);
#pragma unroll
          for (int q = 0; q < NC; ++q) x[rr][cc][q] = o[q];
        }
      }
    }
  }
#pragma unroll
  for (int rr = 0; rr < RPT; ++rr) {
    const int i = tid + 256 * rr;
#pragma unroll
    for (int cc = 0; cc < CPB; ++cc) {
      const int64_t c = cbase + cc;
      if (i < kb && c < ncols) ozx::store<NC>(Xp + (i + c * ldx) * NC, x[rr][cc]);
    }
  }
}

// Triangular solves for kb <= 64 WPC: each column is held by WPC wavefronts,
// row 64 p + l in lane l of the column's wavefront p (4 / WPC columns per
// 256-thread workgroup).  Wavefront p first applies the values of rows
// 0 .. 64 p - 1 as the wavefronts before it publish them (LDS, one counter
// per column), then solves its own 64 rows with no barrier: row h's final
// value is read from lane h - 64 p into scalar registers, published for
// the wavefronts after it, and applied to the later rows.  Every element
// receives its multiply-subtracts in ascending k, the order of
// k_trsm_lower_unit.  UPPER: the same with the rows counted from the last
// and each value divided by its diagonal entry once its updates are in
// (x_h <- x_h / u_hh, then x_i -= u_ih x_h, h descending).  Bound by the chain
// of one multiply-subtract (UPPER: and a division) per row.  A loop each for the
// rows of earlier wavefronts and the own ones, unrolled over the factor entries
// in flight, whose loads take no branch: in one loop, with the entries shifted
// from step to step, every step waited for its newest load.  That / this, us:
// unit lower 32 rows DD 18.7 / 16.1, QD 50.9 / 45.8; 100 rows DD 61 / 47, QD 140 /
// 125; UPPER 32 rows DD 42 / 37, QD 182 / 164; 100 rows DD 132 / 121, QD 549 / 527.
// 256 QD rows with a barrier and a division per row took 1490, UPPER now 1216.
template <int NC, int WPC, bool UPPER>
__global__ __launch_bounds__(256) void k_trsm_w(const double *Fp, int64_t lda, double *Xp,
                                                int64_t ldx, int kb, int64_t ncols) {
  constexpr int CPB = 4 / WPC, PF = NC == 2 ? 4 : 1;
  __shared__ double xs[CPB][WPC > 1 ? 64 * (WPC - 1) : 1][NC];
  __shared__ int done[CPB];
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  const int cc = wv / WPC, part = wv % WPC;
  const int64_t c = (int64_t)blockIdx.x * CPB + cc;
  if (tid < CPB) done[tid] = 0;
  __syncthreads();
  if (c >= ncols) return;  // whole wavefronts of a column past the end
  const int i = 64 * part + lane;  // position: row i, or UPPER row kb-1-i
  const bool mine = i < kb;
  auto row = [&](int p) { return UPPER ? kb - 1 - p : p; };
  auto F = [&](int p, int h) { return Fp + (row(p) + (int64_t)row(h) * lda) * NC; };
  double x[NC] = {}, d[NC] = {}, f[PF][NC] = {};
  if (mine) {
    ozx::load<NC>(Xp + (row(i) + c * ldx) * NC, x);
    if (UPPER) ozx::load<NC>(F(i, i), d);
  }
  const int h0 = 64 * part, h1 = kb < h0 + 64 ? kb : h0 + 64;
  if (h0 >= kb) return;
  // the factor entries of the next PF steps are in flight while one computes;
  // the load of step h has no use past the diagonal and then reads any entry
  auto fetch = [&](int h, double (&to)[NC]) { ozx::load<NC>(mine && h < i ? F(i, h) : Fp, to); };
#pragma unroll
  for (int t = 0; t < PF; ++t) fetch(t, f[t]);
  for (int hb = 0; hb < h0; hb += PF) {
#pragma unroll
    for (int t = 0; t < PF; ++t) {
      const int h = hb + t;
      double y[NC], o[NC], fh[NC];
#pragma unroll
      for (int q = 0; q < NC; ++q) fh[q] = f[t][q];
      fetch(h + PF, f[t]);
      // published by an earlier wavefront of this column (it never waits for
      // this one, so this ends)
      while (__hip_atomic_load(&done[cc], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) <= h)
        __builtin_amdgcn_s_sleep(1);
#pragma unroll
      for (int q = 0; q < NC; ++q) y[q] = xs[cc][h][q];
      if (mine) {
        ozx::fms<NC>(x, fh, y, o);
#pragma unroll
        for (int q = 0; q < NC; ++q) x[q] = o[q];
      }
    }
  }
  for (int hb = h0; hb < h1; hb += PF) {
#pragma unroll
    for (int t = 0; t < PF; ++t) {
      const int h = hb + t;
      if (PF > 1 && h >= h1) break;
      double y[NC], o[NC], fh[NC];
#pragma unroll
      for (int q = 0; q < NC; ++q) fh[q] = f[t][q];
      fetch(h + PF, f[t]);
      if (UPPER) {
        ozx::div<NC>(x, d, o);
#pragma unroll
        for (int q = 0; q < NC; ++q) x[q] = lane == h - h0 ? o[q] : x[q];
      }
      // position h is final
#pragma unroll
      for (int q = 0; q < NC; ++q) y[q] = readlane_f64(x[q], h - h0);
      if (part + 1 < WPC && lane == h - h0) {
#pragma unroll
        for (int q = 0; q < NC; ++q) xs[cc][h][q] = y[q];
        __hip_atomic_store(&done[cc], h + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      if (mine && i > h) {
        ozx::fms<NC>(x, fh, y, o);
#pragma unroll
        for (int q = 0; q < NC; ++q) x[q] = o[q];
      }
    }
  }
  if (mine) ozx::store<NC>(Xp + (row(i) + c * ldx) * NC, x);
}

// ---------------------------------------------------------------------------
// Native expansion product: C <- C - A B with one rounded multiply-subtract
// per inner index, h ascending (desc = 0) or descending (desc = 1).
// A is M x K (lda), B is K x N (ldb).  Tile TM x TN outputs per workgroup.
// ---------------------------------------------------------------------------
template <int NC, int TM, int TN>
__global__ __launch_bounds__(256) void k_naive_gemm(const double *A, int64_t lda, const double *B,
                                                    int64_t ldb, double *C, int64_t ldc, int64_t M,
                                                    int64_t N, int64_t K, int desc) {
  static_assert(TM * TN == 256, "tile");
  constexpr int KC = TM >= 128 ? 4 : 16;
  __shared__ double As[KC][TM][NC];
  __shared__ double Bs[TN][KC][NC];
  const int tid = threadIdx.x;
  const int ti = tid % TM, tj = tid / TM;
  const int64_t i = (int64_t)blockIdx.x * TM + ti, j = (int64_t)blockIdx.y * TN + tj;
  double acc[NC];
  const bool in = i < M && j < N;
  if (in) ozx::load<NC>(C + (i + j * ldc) * NC, acc);
  else
#pragma unroll
    for (int q = 0; q < NC; ++q) acc[q] = 0.0;
  const int64_t nch = (K + KC - 1) / KC;
  for (int64_t cc = 0; cc < nch; ++cc) {
    const int64_t ch = desc ? nch - 1 - cc : cc;
    const int64_t h0 = ch * KC;
    for (int e = tid; e < KC * TM; e += 256) {
      const int r = e % TM, hh = e / TM;
      const int64_t gi = (int64_t)blockIdx.x * TM + r, gh = h0 + hh;
#pragma unroll
      for (int q = 0; q < NC; ++q)
        As[hh][r][q] = (gi < M && gh < K) ? A[(gi + gh * lda) * NC + q] : 0.0;
    }
    for (int e = tid; e < KC * TN; e += 256) {
      const int hh = e % KC, cj = e / KC;
      const int64_t gj = (int64_t)blockIdx.y * TN + cj, gh = h0 + hh;
#pragma unroll
      for (int q = 0; q < NC; ++q)
        Bs[cj][hh][q] = (gj < N && gh < K) ? B[(gh + gj * ldb) * NC + q] : 0.0;
    }
    __syncthreads();
    if (in) {
      const int hmax = (int)((K - h0) < KC ? (K - h0) : KC);
      for (int t = 0; t < hmax; ++t) {
        const int hh = desc ? hmax - 1 - t : t;
        double a[NC], b[NC], o[NC];
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          a[q] = As[hh][ti][q];
          b[q] = Bs[tj][hh][q];
        }
        ozx::fms<NC>(acc, a, b, o);
#pragma unroll
        for (int q = 0; q < NC; ++q) acc[q] = o[q];
      }
    }
    __syncthreads();
  }
  if (in) ozx::store<NC>(C + (i + j * ldc) * NC, acc);
}

// getrs: apply the interchanges ipiv[0..n) in order to one column of B.
// Row interchanges of the solve, b <- P b with P the product of the
// transpositions (j, ipiv[j]), j ascending (LAPACK's i?laswp).  One
// workgroup per right-hand side.  use_lds: the pivots are staged in LDS,
// thread 0 composes the transpositions on row indices (src[j] = row that
// ends at position j), and the expansions are then gathered in parallel.
template <int NC>
__global__ __launch_bounds__(256) void k_apply_ipiv(double *B, int64_t ldb, int64_t n,
                                                    const int64_t *ipiv, int use_lds) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  double *col = B + (int64_t)blockIdx.x * ldb * NC;
  if (use_lds) {
    double *xs = (double *)smem_raw;               // n * NC
    int *pv = (int *)(xs + n * NC);                // n
    int *src = pv + n;                             // n
    for (int64_t e = threadIdx.x; e < n * NC; e += 256) xs[e] = col[e];
    for (int64_t j = threadIdx.x; j < n; j += 256) {
      pv[j] = (int)ipiv[j];
      src[j] = (int)j;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int j = 0; j < (int)n; ++j) {
        const int p = pv[j];
        const int t = src[j];
        src[j] = src[p];
        src[p] = t;
      }
    }
    __syncthreads();
    for (int64_t e = threadIdx.x; e < n * NC; e += 256) col[e] = xs[(int64_t)src[e / NC] * NC + e % NC];
  } else if (threadIdx.x == 0) {
    for (int64_t j = 0; j < n; ++j) {
      const int64_t p = ipiv[j];
      if (p != j) {
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          double t = col[j * NC + q];
          col[j * NC + q] = col[p * NC + q];
          col[p * NC + q] = t;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Triangular solves of getrs for one or a few right-hand sides, pipelined
// over the whole grid (one ordinary launch per direction).  A workgroup takes its
// block of rows from an atomic ticket when it starts, so block t belongs to
// the t-th workgroup to run: every block it waits for is owned by a
// workgroup that is already running, whatever order the hardware dispatches
// workgroups in and however few fit on the device at once.  Block t holds
// the rows at processing positions [t R, t R + R): rows 0.. in the forward
// solve with the unit lower factor, rows n-1.. in the backward solve with
// the upper factor.  Each row's value lives in one lane of wavefront 0.
//
// While earlier blocks are being finished the workgroup applies their
// published solution values to its rows: the products l_ik x_k by all
// wavefronts, then the subtractions in the order the specification fixes
// (ascending k forward, descending backward), so every element sees exactly
// fms(x_i, l_ik, x_k) = x_i (+) (-(l_ik (x) x_k)) in that order.  Its
// diagonal block, staged in LDS when the workgroup starts, is then solved by
// wavefront 0 alone, with no barrier: row q's final value (backward: its
// value divided by u_qq) is read from lane q into scalar registers and
// applied to the later rows of the block.  Wavefront 1 publishes the final
// values in groups of TRSV_PUB rows (stores, agent release, then the count
// of finished positions), so the critical chain of the solve never waits
// for a store.  Waits are bounded like the panel's.
//
// NR = 2: a workgroup takes two right-hand sides, lanes 0 .. 31 and 32 .. 63
// of wavefront 0, which share the factor entries and the division chain's
// issue slots; blockIdx.y = pair, each with its own count and ticket.
constexpr int TRSV_R = 32;    // rows per workgroup
constexpr int TRSV_PUB = 4;   // rows of the diagonal block published at a time
// solution values applied per batch; half of them where two right-hand sides
// of QD products would leave room for one workgroup per CU
template <int NC, int NR>
constexpr int trsv_b() { return NC * NR > 6 ? 16 : 32; }

template <int NC, bool FWD, int NR>
__global__ __launch_bounds__(256) void k_trsv(const double *LU, int64_t lda, double *X, int64_t ldx,
                                              int64_t nrhs, int64_t n, uint32_t *sync, int *err) {
  constexpr int TRSV_B = trsv_b<NC, NR>();
  __shared__ double dg[TRSV_R][TRSV_R][NC];      // dg[q][r]: factor entry of row r, column q
  __shared__ double pr[NR][TRSV_B][TRSV_R][NC];  // negated products of one batch
  __shared__ double ys[NR][TRSV_B][NC];          // published values of one batch
  __shared__ double xs[NR][TRSV_R][NC];          // final values of the block
  __shared__ int s_avail, s_fail, s_blk, s_done;
  uint32_t *ready = sync + 2 * blockIdx.y, *ticket = ready + 1;
  const int tid = threadIdx.x;
  if (tid == 0) s_blk = (int)atomicAdd(ticket, 1u);
  __syncthreads();
  const int64_t p0 = (int64_t)s_blk * TRSV_R;
  const int cnt = (int)(n - p0 < TRSV_R ? n - p0 : TRSV_R);
  const int64_t f0 = (int64_t)blockIdx.y * NR;  // first right-hand side
  const int nr = NR == 1 || nrhs - f0 >= NR ? NR : (int)(nrhs - f0);
  auto row = [&](int64_t p) { return FWD ? p : n - 1 - p; };
  auto L = [&](int64_t i, int64_t k) { return LU + (i + k * lda) * NC; };
  double *const x0 = X + f0 * ldx * NC, *const x1 = x0 + (NR > 1 ? ldx * NC : 0);
  auto x = [&](int f, int64_t i) { return (NR > 1 && f ? x1 : x0) + i * NC; };
  // the diagonal block (strict triangle, plus the diagonal backward); the
  // row index runs fastest, so each column is one contiguous read
  for (int e = tid; e < TRSV_R * TRSV_R * NC; e += 256) {
    const int q = e / (TRSV_R * NC), r = (e / NC) % TRSV_R, c = e % NC;
    if (q < cnt && r < cnt && (r > q || (!FWD && r == q)))
      dg[q][r][c] = L(row(p0 + r), row(p0 + q))[c];
  }
  // lane: row rr of right-hand side f of this workgroup (wavefront 0)
  const int rr = NR > 1 ? tid & (TRSV_R - 1) : tid, f = NR > 1 ? (tid >> 5) & 1 : 0;
  const bool mine = NR > 1 ? tid < TRSV_R * NR && rr < cnt && f < nr : tid < cnt;
  double v[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) v[c] = mine ? x(f, row(p0 + rr))[c] : 0.0;
  if (tid == 0) {
    s_fail = 0;
    s_done = 0;
  }
  __syncthreads();
  int64_t applied = 0;
  while (applied < p0) {
    if (tid == 0) {
      const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
      uint32_t spins = 0, w;
      while ((int64_t)(w = ld_dev_u32(ready)) <= applied) {
        if (wait_expired(spins, t0, err, 3)) {
          s_fail = 1;
          break;
        }
        // every waiting workgroup polls the same word, which holds up the one
        // that advances it: rarely while the blocks before this one are many
        if (p0 - (int64_t)w > 2 * TRSV_R) __builtin_amdgcn_s_sleep(32);
        else __builtin_amdgcn_s_sleep(2);
      }
      s_avail = (int)((int64_t)w < p0 ? (int64_t)w : p0);
    }
    __syncthreads();
    if (s_fail) return;
    const int64_t avail = s_avail;
    for (int64_t c0 = applied; c0 < avail; c0 += TRSV_B) {
      const int nb = (int)(avail - c0 < TRSV_B ? avail - c0 : TRSV_B);
      // published values: device-coherent loads, issued after the count was seen
      if (tid < nb * NC) {
#pragma unroll
        for (int g = 0; g < NR; ++g)
          if (g < nr) (&ys[g][0][0])[tid] = ld_dev_f64(x(g, row(c0 + tid / NC)) + tid % NC);
      }
      __syncthreads();
      for (int idx = tid; idx < cnt * nb; idx += 256) {
        const int q = idx % cnt, t = idx / cnt;
        double a[NC], y[NC], o[NC];
        ozx::load<NC>(L(row(p0 + q), row(c0 + t)), a);
#pragma unroll
        for (int g = 0; g < NR; ++g) {
          if (g >= nr) break;
#pragma unroll
          for (int c = 0; c < NC; ++c) y[c] = ys[g][t][c];
          ozx::mul<NC>(a, y, o);
#pragma unroll
          for (int c = 0; c < NC; ++c) pr[g][t][q][c] = -o[c];
        }
      }
      __syncthreads();
      // the subtractions, in order; the next batch's barrier waits for them
      if (mine) {
        for (int t = 0; t < nb; ++t) {
          double pv[NC], o[NC];
#pragma unroll
          for (int c = 0; c < NC; ++c) pv[c] = pr[f][t][rr][c];
          ozx::add<NC>(v, pv, o);
#pragma unroll
          for (int c = 0; c < NC; ++c) v[c] = o[c];
        }
      }
    }
    applied = avail;
  }
  __syncthreads();
  if (tid < 64) {
    // wavefront 0: the diagonal block; the factor entries of the next step
    // are read from LDS while this one computes
    double a[NC], u[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      a[c] = rr > 0 && rr < cnt ? dg[0][rr][c] : 0.0;
      u[c] = FWD ? 0.0 : dg[0][0][c];
    }
    for (int q = 0; q < cnt; ++q) {
      double an[NC], un[NC];
      const int qn = q + 1 < cnt ? q + 1 : q;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        an[c] = rr > qn && rr < cnt ? dg[qn][rr][c] : 0.0;
        un[c] = FWD ? 0.0 : dg[qn][qn][c];
      }
      if (!FWD && rr == q && (NR == 1 || f < nr)) {
        double o[NC];
        ozx::div<NC>(v, u, o);
#pragma unroll
        for (int c = 0; c < NC; ++c) v[c] = o[c];
      }
      // row q is final
      double y[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        y[c] = readlane_f64(v[c], q);
        if (NR > 1) {
          const double y1 = readlane_f64(v[c], q + TRSV_R);
          y[c] = f ? y1 : y[c];
        }
      }
      if (rr == q && (NR == 1 || f < nr)) {
#pragma unroll
        for (int c = 0; c < NC; ++c) xs[f][q][c] = v[c];
      }
      if (rr > q && rr < cnt && (NR == 1 || f < nr)) {
        double o[NC];
        ozx::fms<NC>(v, a, y, o);
#pragma unroll
        for (int c = 0; c < NC; ++c) v[c] = o[c];
      }
      if ((q + 1) % TRSV_PUB == 0 || q + 1 == cnt) {
        // the group's values are in LDS before the count is raised
        if (tid == 0)
          __hip_atomic_store(&s_done, q + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        a[c] = an[c];
        u[c] = un[c];
      }
    }
  } else if (tid < 128) {
    // wavefront 1: publication of the finished rows
    const int lane = tid - 64;
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    int done = 0;
    while (done < cnt) {
      const int d = __hip_atomic_load(&s_done, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (d <= done) {
        if (__builtin_amdgcn_s_memrealtime() - t0 > 100000000ull) {
          if (lane == 0) __hip_atomic_store(err, 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          return;
        }
        __builtin_amdgcn_s_sleep(1);
        continue;
      }
#pragma unroll
      for (int g = 0; g < NR; ++g)
        if (g < nr)
          for (int e = lane; e < (d - done) * NC; e += 64) {
            const int q = done + e / NC, c = e % NC;
            (g ? x1 : x0)[row(p0 + q) * NC + c] = xs[g][q][c];
          }
      // this wavefront's stores complete before the count is raised
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      if (lane == 0)
        __hip_atomic_store(ready, (uint32_t)(p0 + d), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      done = d;
    }
  }
}

__global__ void k_fill_int(int *p, int v, int64_t cnt) {
  int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e < cnt) p[e] = v;
}

}  // namespace

namespace ozl {

size_t panel_lds_bytes(int nc, int kb, int R, int64_t nr) {
  return (size_t)R * kb * nc * 8 + (size_t)2 * kb * nc * 8 + (size_t)nr * 8;
}

size_t panel_row_bytes(int kb) { return (size_t)kb * 4 * 16; }

const void *panel_kernel_ptr(int nc) {
  if (nc == 2) return (const void *)k_panel<2>;
  if (nc == 3) return (const void *)k_panel<3>;
  return (const void *)k_panel<4>;
}

hipError_t launch_getrf_begin(uint32_t *epoch, int64_t panels, int32_t *info, uint64_t *lines,
                              uint64_t *crow, int kb, hipStream_t s) {
  hipLaunchKernelGGL(k_getrf_begin, dim3(1), dim3(BEGIN_NT), 0, s, epoch, (uint32_t)panels, info,
                     lines, (int64_t)2 * PANEL_MAXG * LINE_WORDS, crow,
                     (int64_t)(2 * PANEL_MAXG * panel_row_bytes(kb) / 8));
  return hipGetLastError();
}

hipError_t launch_panel(int nc, double *A, int64_t lda, int64_t n, int64_t k, int kb, int R, int G,
                        int64_t *ipiv, int32_t *info, uint64_t *lines, int *err, uint64_t *crow,
                        uint32_t *epoch, int panel, int *perm, int *moved, int *nmoved,
                        hipStream_t s) {
  const size_t lds = panel_lds_bytes(nc, kb, R, n - k);
  const void *fn = panel_kernel_ptr(nc);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  void *args[] = {&A, &lda, &n, &k, &kb, &R, &ipiv, &info, &lines, &err,
                  &crow, &epoch, &panel, &perm, &moved, &nmoved};
  // one workgroup needs no others beside it: an ordinary launch, without the
  // cooperative queue's 11 us before and after it
  if (G == 1) return hipLaunchKernel(fn, dim3(1), dim3(PANEL_NT), args, (unsigned)lds, s);
  return hipLaunchCooperativeKernel(fn, dim3(G), dim3(PANEL_NT), args, (unsigned)lds, s);
}

hipError_t panel_max_blocks(int nc, int kb, int R, int64_t nr, int *maxblocks) {
  const size_t lds = panel_lds_bytes(nc, kb, R, nr);
  const void *fn = panel_kernel_ptr(nc);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int per = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, PANEL_NT, lds);
  if (e != hipSuccess) return e;
  int dev = 0, ncu = 0;
  hipGetDevice(&dev);
  hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  *maxblocks = per * ncu;
  return hipSuccess;
}

hipError_t launch_laswp(int nc, double *A, int64_t lda, int64_t k, int64_t c0, int64_t c1,
                        const int *perm, const int *moved, const int *nmoved, hipStream_t s) {
  if (c1 <= c0) return hipSuccess;
  dim3 g((unsigned)(c1 - c0));
  if (nc == 2) hipLaunchKernelGGL(k_laswp<2>, g, dim3(256), 0, s, A, lda, k, c0, c1, perm, moved, nmoved);
  else if (nc == 3) hipLaunchKernelGGL(k_laswp<3>, g, dim3(256), 0, s, A, lda, k, c0, c1, perm, moved, nmoved);
  else hipLaunchKernelGGL(k_laswp<4>, g, dim3(256), 0, s, A, lda, k, c0, c1, perm, moved, nmoved);
  return hipGetLastError();
}

template <int NC>
static void trsm_l(int kb, hipStream_t s, const double *L, int64_t lda, double *X, int64_t ldx,
                   int64_t ncols) {
  if (kb <= 64)
    hipLaunchKernelGGL((k_trsm_w<NC, 1, false>), dim3((unsigned)((ncols + 3) / 4)), dim3(256),
                       0, s, L, lda, X, ldx, kb, ncols);
  else if (kb <= 128)
    hipLaunchKernelGGL((k_trsm_w<NC, 2, false>), dim3((unsigned)((ncols + 1) / 2)),
                       dim3(256), 0, s, L, lda, X, ldx, kb, ncols);
  else if (kb <= 256)
    hipLaunchKernelGGL((k_trsm_w<NC, 4, false>), dim3((unsigned)ncols), dim3(256), 0, s, L,
                       lda, X, ldx, kb, ncols);
  else
    hipLaunchKernelGGL((k_trsm_lower_unit<NC, 1, 2>), dim3((unsigned)ncols), dim3(256), 0, s, L, lda,
                       X, ldx, kb, ncols);
}

hipError_t launch_trsm_lower_unit(int nc, const double *L, int64_t lda, double *X, int64_t ldx,
                                  int kb, int64_t ncols, hipStream_t s) {
  if (ncols <= 0 || kb <= 0) return hipSuccess;
  if (kb > 512) return hipErrorInvalidValue;
  if (nc == 2) trsm_l<2>(kb, s, L, lda, X, ldx, ncols);
  else if (nc == 3) trsm_l<3>(kb, s, L, lda, X, ldx, ncols);
  else trsm_l<4>(kb, s, L, lda, X, ldx, ncols);
  return hipGetLastError();
}

template <int NC>
static void trsm_u(int kb, hipStream_t s, const double *U, int64_t lda, double *X, int64_t ldx,
                   int64_t ncols) {
#define OZ_TRSMU(WPC_)                                                                          \
  hipLaunchKernelGGL((k_trsm_w<NC, WPC_, true>), dim3((unsigned)((ncols * WPC_ + 3) / 4)),      \
                     dim3(256), 0, s, U, lda, X, ldx, kb, ncols)
  if (kb <= 64) OZ_TRSMU(1);
  else if (kb <= 128) OZ_TRSMU(2);
  else OZ_TRSMU(4);
#undef OZ_TRSMU
}

hipError_t launch_trsm_upper(int nc, const double *U, int64_t lda, double *X, int64_t ldx, int kb,
                             int64_t ncols, hipStream_t s) {
  if (ncols <= 0 || kb <= 0) return hipSuccess;
  if (kb > 256) return hipErrorInvalidValue;
  if (nc == 2) trsm_u<2>(kb, s, U, lda, X, ldx, ncols);
  else if (nc == 3) trsm_u<3>(kb, s, U, lda, X, ldx, ncols);
  else trsm_u<4>(kb, s, U, lda, X, ldx, ncols);
  return hipGetLastError();
}

template <int NC>
static void naive_nc(int64_t M, int64_t N, hipStream_t s, const double *A, int64_t lda,
                     const double *B, int64_t ldb, double *C, int64_t ldc, int64_t K, int desc) {
  if (N >= 16) {
    dim3 g((unsigned)((M + 15) / 16), (unsigned)((N + 15) / 16));
    hipLaunchKernelGGL((k_naive_gemm<NC, 16, 16>), g, dim3(256), 0, s, A, lda, B, ldb, C, ldc, M, N, K, desc);
  } else {
    dim3 g((unsigned)((M + 255) / 256), (unsigned)N);
    hipLaunchKernelGGL((k_naive_gemm<NC, 256, 1>), g, dim3(256), 0, s, A, lda, B, ldb, C, ldc, M, N, K, desc);
  }
}

hipError_t launch_naive_gemm(int nc, const double *A, int64_t lda, const double *B, int64_t ldb,
                             double *C, int64_t ldc, int64_t M, int64_t N, int64_t K, int desc,
                             hipStream_t s) {
  if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
  if (nc == 2) naive_nc<2>(M, N, s, A, lda, B, ldb, C, ldc, K, desc);
  else if (nc == 3) naive_nc<3>(M, N, s, A, lda, B, ldb, C, ldc, K, desc);
  else naive_nc<4>(M, N, s, A, lda, B, ldb, C, ldc, K, desc);
  return hipGetLastError();
}

hipError_t launch_apply_ipiv(int nc, double *B, int64_t ldb, int64_t n, int64_t nrhs,
                             const int64_t *ipiv, hipStream_t s) {
  if (n <= 0 || nrhs <= 0) return hipSuccess;
  const size_t lds = (size_t)n * nc * 8 + (size_t)n * 8;  // expansions + pivots + sources
  const int use_lds = lds <= 160 * 1024 ? 1 : 0;
  const void *fn = nc == 2 ? (const void *)k_apply_ipiv<2>
                           : (nc == 3 ? (const void *)k_apply_ipiv<3> : (const void *)k_apply_ipiv<4>);
  if (use_lds) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  dim3 g((unsigned)nrhs);
  const unsigned shm = use_lds ? (unsigned)lds : 0u;
  if (nc == 2) hipLaunchKernelGGL(k_apply_ipiv<2>, g, dim3(256), shm, s, B, ldb, n, ipiv, use_lds);
  else if (nc == 3) hipLaunchKernelGGL(k_apply_ipiv<3>, g, dim3(256), shm, s, B, ldb, n, ipiv, use_lds);
  else hipLaunchKernelGGL(k_apply_ipiv<4>, g, dim3(256), shm, s, B, ldb, n, ipiv, use_lds);
  return hipGetLastError();
}

bool trsv_fits(int64_t n, int64_t nrhs) {
  return (n + TRSV_R - 1) / TRSV_R * ((nrhs + 1) / 2) <= TRSV_MAXGROUPS;
}

template <int NC>
static void trsv_nc(int fwd, dim3 g, int nr, hipStream_t s, const double *LU, int64_t lda,
                    double *X, int64_t ldx, int64_t nrhs, int64_t n, uint32_t *sync, int *err) {
#define OZ_TRSV(F_, NR_)                                                                         \
  hipLaunchKernelGGL((k_trsv<NC, F_, NR_>), g, dim3(256), 0, s, LU, lda, X, ldx, nrhs, n, sync, err)
  if (nr == 1) {
    if (fwd) OZ_TRSV(true, 1);
    else OZ_TRSV(false, 1);
  } else {
    if (fwd) OZ_TRSV(true, 2);
    else OZ_TRSV(false, 2);
  }
#undef OZ_TRSV
}

hipError_t launch_trsv(int nc, int fwd, const double *LU, int64_t lda, double *X, int64_t ldx,
                       int64_t nrhs, int64_t n, uint32_t *sync, int *err, hipStream_t s) {
  if (n <= 0 || nrhs <= 0) return hipSuccess;
  const int nr = nrhs > 1 ? 2 : 1;
  const dim3 g((unsigned)((n + TRSV_R - 1) / TRSV_R), (unsigned)((nrhs + nr - 1) / nr));
  // per group: finished positions and the ticket of the next row block, those
  // of the backward solve behind those of the forward one
  if (fwd)
    hipLaunchKernelGGL(k_fill_int, dim3((4 * g.y + 255) / 256), dim3(256), 0, s, (int *)sync, 0,
                       (int64_t)4 * g.y);
  else
    sync += 2 * g.y;
  if (nc == 2) trsv_nc<2>(fwd, g, nr, s, LU, lda, X, ldx, nrhs, n, sync, err);
  else if (nc == 3) trsv_nc<3>(fwd, g, nr, s, LU, lda, X, ldx, nrhs, n, sync, err);
  else trsv_nc<4>(fwd, g, nr, s, LU, lda, X, ldx, nrhs, n, sync, err);
  return hipGetLastError();
}

}  // namespace ozl
