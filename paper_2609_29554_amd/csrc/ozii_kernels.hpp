// Host-side launchers of the HIP kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/ozii.h"

namespace ozk {
struct DevPlan;
}

namespace ozl {
using ozk::DevPlan;

// (S4) GEMM workgroup tiles (values of ozII_opts.gemm_tile)
enum { GEMM_TILE_AUTO = 0, GEMM_TILE_128x128 = 1, GEMM_TILE_256x128 = 2, GEMM_TILE_256x256 = 3 };

inline bool gemm_tile_fits(int tile, int64_t Mp, int64_t Np) {
  switch (tile) {
    case GEMM_TILE_128x128: return Mp % 128 == 0 && Np % 128 == 0;
    case GEMM_TILE_256x128: return Mp % 256 == 0 && Np % 128 == 0;
    case GEMM_TILE_256x256: return Mp % 256 == 0 && Np % 256 == 0;
    default: return false;
  }
}

// The 256x128 tile (three 24 KiB stages: two workgroups per CU overlap each
// other's barriers) when it still gives every CU two workgroups (prods =
// batched (group, modulus) products), else 128x128.  Measured on MI355X it
// beats the 256x256 tile (one workgroup per CU) on both the TD 4096^3
// product and the p = 4096 limb updates; 256x256 stays selectable.
inline int gemm_tile_auto(int64_t prods, int64_t Mp, int64_t Np) {
  if (gemm_tile_fits(GEMM_TILE_256x128, Mp, Np) && prods * (Mp / 256) * (Np / 128) >= 512)
    return GEMM_TILE_256x128;
  return GEMM_TILE_128x128;
}

// C = 0 (M x N expansions of nc components, leading dimension ldc)
hipError_t launch_zero_expansions(int nc, double *C, int64_t ldc, int64_t M, int64_t N,
                                  hipStream_t s);
// Ozaki-II product stages
// One operand of a product: A (rows are the outputs) or B (columns are).
// noutp: outputs padded to the GEMM tile, the rows of its residue planes.
struct Operand {
  const double *X;
  int64_t ld, nout, noutp;
  int32_t *exps;
  void *planes;
  int64_t plane_elems;
};
// operand scans of at most this many bytes stay in the producer: they then
// cost less than the launch they save
constexpr int64_t OWN_EXP_BYTES = (int64_t)16 << 20;
// (S1) of both operands; not needed where the producer finds the exponents
hipError_t launch_exponents(int nc, const Operand &A, const Operand &B, int64_t K, hipStream_t s);
bool producer_owns_exponents(int nc, const Operand &A, const Operand &B, int64_t K, int64_t Kp,
                             int nmod, int kind);
// plane encodings of the producer (one per back-end)
enum { PLANES_I8 = 0, PLANES_F8 = 1, PLANES_F64 = 2 };
// (S2)+(S3) of both operands in one launch
hipError_t launch_producer(int nc, int nwx, int nh, int nwt, const Operand &A, const Operand &B,
                           int64_t K, int64_t Kp, const DevPlan *pl, int nmod, int kind,
                           hipStream_t s);
hipError_t launch_gemm_i8(const int8_t *pa, const int8_t *pb, uint8_t *tpl, const DevPlan *pl,
                          int ng, int nmod, int64_t Mp, int64_t Np, int64_t Kp, int64_t planeA,
                          int64_t planeB, int tile, hipStream_t s);
hipError_t launch_gemm_f8(const uint8_t *pa, const uint8_t *pb, uint8_t *tpl, const DevPlan *pl,
                          int ng, int nmod, int64_t Mp, int64_t Np, int64_t Kp, int64_t planeA,
                          int64_t planeB, hipStream_t s);
// (S4) on the FP16 engine from the INT8 residue planes (Mp, Np multiples of 128)
hipError_t launch_gemm_f16(const int8_t *pa, const int8_t *pb, uint8_t *tpl, const DevPlan *pl,
                           int ng, int nmod, int64_t Mp, int64_t Np, int64_t Kp, int64_t planeA,
                           int64_t planeB, hipStream_t s);
// fused (S4)+(S5)+(S6), INT8 planes: t-values of a 32 x 32 tile kept in LDS
// (at most fused_max_products() (group, modulus) products)
int fused_max_products();
hipError_t launch_fused_b(int nc, int nwc, int nd, const int8_t *pa, const int8_t *pb,
                          const DevPlan *pl, int ng, int nmod, int64_t Kp, int64_t planeA,
                          int64_t planeB, double *C, int64_t ldc, int64_t M, int64_t N,
                          const int32_t *ea, const int32_t *eb, int mode, hipStream_t s);
hipError_t launch_gemm_f64(const double *pa, const double *pb, uint32_t *tpl, const DevPlan *pl,
                           int ng, int nmod, int64_t Mp, int64_t Np, int64_t Kp, int64_t planeA,
                           int64_t planeB, hipStream_t s);
hipError_t launch_consumer(int nc, int nwc, int nd, const void *tpl, int tbytes, int64_t Mp,
                           int64_t Np, double *C, int64_t ldc, int64_t M, int64_t N,
                           const int32_t *ea, const int32_t *eb, const DevPlan *pl, int mode,
                           hipStream_t s);
// group sums exported by the CRT routine of the consumer that reads these
// t-planes (byte back-ends: the matrix-core route, with the consumer's
// byte-column count for nd digits; binary64 moduli: crt_digits)
hipError_t launch_crt_export(const void *tpl, int tbytes, int nd, int64_t Mp, int64_t Np,
                             int64_t M, int64_t N, const DevPlan *pl, uint64_t *out, int nlimb,
                             hipStream_t s);

// LU pieces
size_t panel_lds_bytes(int nc, int kb, int R, int64_t nr);
hipError_t panel_max_blocks(int nc, int kb, int R, int64_t nr, int *maxblocks);
// bytes of a candidate row of up to kb expansions
size_t panel_row_bytes(int kb);
// workgroups of a panel
constexpr int PANEL_MAXG = 256;
// before the panels 0 .. panels-1 of a factorisation: info = 0 and their tags;
// kb: the columns that crow was allocated for
hipError_t launch_getrf_begin(uint32_t *epoch, int64_t panels, int32_t *info, uint64_t *lines,
                              uint64_t *crow, int kb, hipStream_t s);
// lines: 2 * PANEL_MAXG candidate lines of 128 bytes; crow: 2 * PANEL_MAXG
// candidate rows; both zeroed when allocated, as is epoch, the panels' tags;
// panel: its number in the factorisation; G <= PANEL_MAXG
hipError_t launch_panel(int nc, double *A, int64_t lda, int64_t n, int64_t k, int kb, int R, int G,
                        int64_t *ipiv, int32_t *info, uint64_t *lines, int *err, uint64_t *crow,
                        uint32_t *epoch, int panel, int *perm, int *moved, int *nmoved,
                        hipStream_t s);
hipError_t launch_laswp(int nc, double *A, int64_t lda, int64_t k, int64_t c0, int64_t c1,
                        const int *perm, const int *moved, const int *nmoved, hipStream_t s);
hipError_t launch_trsm_lower_unit(int nc, const double *L, int64_t lda, double *X, int64_t ldx,
                                  int kb, int64_t ncols, hipStream_t s);
hipError_t launch_trsm_upper(int nc, const double *U, int64_t lda, double *X, int64_t ldx, int kb,
                             int64_t ncols, hipStream_t s);
hipError_t launch_naive_gemm(int nc, const double *A, int64_t lda, const double *B, int64_t ldb,
                             double *C, int64_t ldc, int64_t M, int64_t N, int64_t K, int desc,
                             hipStream_t s);
hipError_t launch_apply_ipiv(int nc, double *B, int64_t ldb, int64_t n, int64_t nrhs,
                             const int64_t *ipiv, hipStream_t s);

// limb format (k_limbs.hip): exponents, producer (INT8 or binary64 planes), consumer
// (exact group sums as nwords-word columns, word k of element i + j M at
// cw[k M N + i + j M]), the rounding of those sums into a limb matrix, the
// update C = RN_p(C - T) (T: M x N limb matrix with ld M, plane M N; dw:
// 2 nlimb + 2 words per element of scratch) and a zero fill
struct LimbOperand {
  const uint64_t *limb;
  const int32_t *lexp;
  const uint8_t *lsign;
  int64_t ld, plane, nout, noutp;
  int32_t *exps;
  void *planes;
  int64_t plane_elems;
};
hipError_t launch_limb_exponents(const LimbOperand &A, const LimbOperand &B, int nlimb, int64_t K,
                                 hipStream_t s);
bool producer_limbs_owns_exponents(const LimbOperand &A, const LimbOperand &B, int64_t K,
                                   int64_t Kp, int nmod);
hipError_t launch_producer_limbs(const LimbOperand &A, const LimbOperand &B, int nlimb, int64_t K,
                                 int64_t Kp, const DevPlan *pl, int nmod, int nwt, int kind,
                                 hipStream_t s);
// words per element of the exact sum that launch_consumer_limbs writes; words:
// the number of the binary64 back-end's walk
int limb_sum_words(int nd, int tbytes, int w, int ng, int words);
// whether launch_limb_finish takes numbers of nlimb limbs from sums of nwords
// words (else launch_limb_round and launch_limb_sub)
bool limb_finish_fits(int nlimb, int nwords, int64_t M, int64_t N, int mode);
hipError_t launch_limb_finish(const uint32_t *cw, int nwords, int64_t M, int64_t N,
                              const int32_t *ea, const int32_t *eb, int w, int g0, int Q, int nlimb,
                              int mode, uint64_t *climb, int32_t *cexp, uint8_t *csign, int64_t ldc,
                              int64_t planec, hipStream_t s);
hipError_t launch_consumer_limbs(const void *tpl, int tbytes, int64_t Mp, int64_t Np, int64_t M,
                                 int64_t N, const DevPlan *pl, int nd, int nvw, uint32_t *cw,
                                 hipStream_t s);
hipError_t launch_limb_round(const uint32_t *cw, int nwords, int64_t M, int64_t N,
                             const int32_t *ea, const int32_t *eb, int w, int g0, int Q, int nlimb,
                             uint64_t *olimb, int32_t *oexp, uint8_t *osign, int64_t ldo,
                             int64_t planeo, hipStream_t s);
hipError_t launch_limb_sub(uint64_t *climb, int32_t *cexp, uint8_t *csign, int64_t ldc,
                           int64_t planec, const uint64_t *tlimb, const int32_t *texp,
                           const uint8_t *tsign, int nlimb, int64_t M, int64_t N, uint32_t *dw,
                           hipStream_t s);
hipError_t launch_limb_zero(uint64_t *limb, int32_t *lexp, uint8_t *lsign, int64_t ld,
                            int64_t plane, int nlimb, int64_t M, int64_t N, hipStream_t s);
// pipelined triangular solve (fwd: unit lower, ascending; else upper,
// descending, dividing by the diagonal); sync: four device words owned by
// the caller per right-hand side, or per pair of them (finished-position counter
// and row-block ticket of each direction), reset by the forward solve's launch
// for the backward one after it too
hipError_t launch_trsv(int nc, int fwd, const double *LU, int64_t lda, double *X, int64_t ldx,
                       int64_t nrhs, int64_t n, uint32_t *sync, int *err, hipStream_t s);
// row blocks x pairs of right-hand sides that are on the chip at once (two
// workgroups per CU); beyond it the pipelines would run in turns
constexpr int TRSV_MAXGROUPS = 512;
bool trsv_fits(int64_t n, int64_t nrhs);

// batched LU + solve (k_batch.hip); items in processing order, each with its
// caller-order index in `reserved`
hipError_t launch_batch(const ozII_batch_item *items, int count, int *queue, uint64_t *times,
                        int grid, hipStream_t s);
// the same with the blocked LU and the in-workgroup Ozaki-II update (panel
// width b <= 256); plans at K = b for nc = 2, 3, 4 (null for absent formats),
// scratch of `slot` bytes per workgroup
// board: batch_board_bytes(nslot) bytes of device memory; ws: nslot slots of
// scratch, nslot >= min(count, grid); grid: workgroups, at most one per CU (cus);
// err: the sticky error word
size_t batch_board_bytes(int nslot);
hipError_t launch_batch_oz(const ozII_batch_item *items, int count, void *board, int nslot,
                           uint64_t *times, int grid, int cus, const ozk::DevPlan *pl2,
                           const ozk::DevPlan *pl3, const ozk::DevPlan *pl4, uint8_t *ws,
                           int64_t slot, int b, int *err, hipStream_t s);

// LU on limb matrices outside the Ozaki-II product (k_limb_lu.hip): limb q
// of element (i, j), e = i + j ld, at limb[q plane + e es], its exponent at
// exp[e xs] and sign at sign[e ss].  The caller's matrices have one plane
// per limb (es = xs = ss = 1); packed ones keep an element's limbs together
// (plane = 1), followed by a word with its exponent and sign.
struct LimbMat {
  uint64_t *limb;
  int32_t *exp;
  uint8_t *sign;
  int64_t ld, plane;
  int64_t es = 1, xs = 1, ss = 1;
};
inline int64_t packed_words(int nl) { return nl + 1; }  // per element
inline LimbMat packed_mat(uint64_t *buf, int nl, int64_t rows) {
  LimbMat m;
  m.limb = buf;
  m.exp = (int32_t *)(buf + nl);
  m.sign = (uint8_t *)(buf + nl) + 4;
  m.ld = rows;
  m.plane = 1;
  m.es = packed_words(nl);
  m.xs = 2 * m.es;
  m.ss = 8 * m.es;
  return m;
}
// P = A[i0 : i0+rows, c0 : c0+w] (unpack = 0), or the other way (unpack = 1)
hipError_t launch_lpack(LimbMat A, LimbMat P, int nl, int64_t i0, int64_t rows, int64_t c0,
                        int64_t w, int unpack, hipStream_t s);
// one panel column j: pivot search over rows [j, n), ipiv[j], info, the
// interchange on columns [s0, s1), division, rank-1 update of columns
// (j, c1); zflag: one word.  Row and column 0 of A are number base of the
// whole matrix, which ipiv and info count in (ipiv points at entry base).
hipError_t launch_lpanel_column(LimbMat A, int nl, int64_t j, int64_t n, int64_t s0, int64_t s1,
                                int64_t c1, int64_t base, int64_t *ipiv, int32_t *info,
                                int32_t *zflag, hipStream_t s);
// interchanges ipiv[k0 .. k0+kb) on columns [ca0, ca1) and [cb0, cb1)
hipError_t launch_llaswp(LimbMat A, int nl, const int64_t *ipiv, int64_t k0, int64_t kb,
                         int64_t ca0, int64_t ca1, int64_t cb0, int64_t cb1, hipStream_t s);
// A[r0:r0+h, b0:b1] <- L^-1 A[r0:r0+h, b0:b1], L unit lower at (r0, r0)
hipError_t launch_ltrsm(LimbMat A, int nl, int64_t r0, int64_t h, int64_t b0, int64_t b1,
                        hipStream_t s);
// A[i0:i1, c0:c1] -= A[i0:i1, k0:k0+K] A[k0:k0+K, c0:c1] by multiply-subtracts
hipError_t launch_lschur_naive(LimbMat A, int nl, int64_t i0, int64_t i1, int64_t c0, int64_t c1,
                               int64_t k0, int64_t K, hipStream_t s);
// recip: n packed numbers of scratch for the reciprocals of the diagonal, or
// null (each division then runs its digit chain)
bool lgetrs_wants_recip(int nl);
hipError_t launch_lgetrs(LimbMat LU, int nl, int64_t n, const int64_t *ipiv, LimbMat X,
                         int64_t nrhs, uint64_t *recip, hipStream_t s);
hipError_t launch_larith(int op, int nl, int64_t cnt, LimbMat A, LimbMat B, LimbMat C,
                         hipStream_t s);
hipError_t launch_lfill_i32(int32_t *p, int32_t v, int count, hipStream_t s);

}  // namespace ozl
