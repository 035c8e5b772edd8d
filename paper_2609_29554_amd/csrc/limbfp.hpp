// Lane-distributed p-bit binary floating point on one 64-lane wavefront.
//
// The LU on limb numbers keeps its panel, interchanges, U12 solve and
// substitutions outside the Ozaki-II product (Sec. 3.4); those steps need
// p-bit division, multiplication and subtraction of the number type of
// Sec. 2, which rounds like MPFR's RNDN.  One wavefront carries one number,
// p = 64 nl <= 4096:
//   x = (-1)^s m 2^(e - p),  2^(p-1) <= m < 2^p;   zero: m = 0, e = EXP_ZERO,
// lane q holding limb q of m (lanes nl..63 hold 0), e and s uniform.  Every
// operation returns the exact result rounded once to p bits, to nearest with
// ties to even; correct rounding makes that result unique.
//
// Carries and borrows between limbs are resolved for all lanes at once:
// lane k generates (g) or propagates (p) a carry, and the carry into every
// lane is read off the 64-bit sum (g|p) + g + cin, whose bit k is
// g_k ^ p_k ^ carry_k.  Products are byte convolutions on the matrix cores
// (few limbs: one output column per lane), their sums resolved the same way;
// division is long division on 58-bit digits with the borrows between lanes
// deferred.
//
// The includer provides LFP_FN and the cross-lane primitives lane_id,
// ballot, readlane64 (wave-uniform lane), shfl64 (any lane), up1_64 and
// up1_32 (from lane l-1, 0 into lane 0), dn1_64 (from lane l+1, 0 into lane
// 63), lane_bit (a lane's bit of a uniform mask), rot1_64 (from lane (l-1) mod
// 64), addc32 (32-bit add with carry), align_bits (funnel shift), mfma_bytes
// and lds_order.
// Every function must be called by all 64 lanes of a converged wavefront;
// branches below depend on wave-uniform values only.
#pragma once
#include <stdint.h>

namespace lfp {

constexpr int32_t EXP_ZERO = INT32_MIN;

struct WF {
  uint64_t m;  // limb lane_id() of the mantissa
  int32_t e;   // exponent; EXP_ZERO for zero
  uint32_t s;  // sign: 0 positive, 1 negative
};

// a 128-limb fixed-point window: limb k in lane k of lo, limb 64+k in hi
struct W2 {
  uint64_t lo, hi;
};

LFP_FN WF wf_zero() {
  WF z;
  z.m = 0;
  z.e = EXP_ZERO;
  z.s = 0;
  return z;
}

LFP_FN bool is_zero(const WF &x) { return x.e == EXP_ZERO; }
LFP_FN int msb64(uint64_t x) { return 63 - __builtin_clzll(x); }
LFP_FN uint64_t low_mask(int k) { return k >= 64 ? ~0ull : ((1ull << k) - 1ull); }  // k >= 0
LFP_FN uint64_t bit_of(uint64_t mask, int l) { return (mask >> l) & 1ull; }

// Carry into every lane of a 64-lane chain (bit k of the result) for
// generate mask g, propagate mask p (disjoint) and carry-in cin of lane 0;
// cout = carry out of lane 63.
LFP_FN uint64_t chain(uint64_t g, uint64_t p, uint32_t cin, uint32_t &cout) {
  const uint64_t x = g | p;
  const uint64_t s1 = x + g;
  const uint64_t s2 = s1 + cin;
  cout = (uint32_t)((s1 < x) | (s2 < s1));
  return s2 ^ x ^ g;
}

// carry out of lane nl-1 of a chain whose lanes nl..63 kill
LFP_FN uint32_t out_at(uint64_t cmask, uint32_t cout63, int nl) {
  return nl >= 64 ? cout63 : (uint32_t)bit_of(cmask, nl);
}

// x + y + cin over lanes < nl (0 above); cout = carry out of lane nl-1
LFP_FN uint64_t add1(uint64_t x, uint64_t y, int nl, uint32_t cin, uint32_t &cout) {
  const int l = lane_id();
  const bool act = l < nl;
  const uint64_t s = x + y;
  uint32_t c63;
  const uint64_t cm = chain(ballot(act && s < x), ballot(act && s == ~0ull), cin, c63);
  cout = out_at(cm, c63, nl);
  return act ? s + lane_bit(cm) : 0ull;
}

// x - y - bin over lanes < nl (0 above); bout = borrow out of lane nl-1
LFP_FN uint64_t sub1(uint64_t x, uint64_t y, int nl, uint32_t bin, uint32_t &bout) {
  const int l = lane_id();
  const bool act = l < nl;
  uint32_t b63;
  const uint64_t bm = chain(ballot(act && x < y), ballot(act && x == y), bin, b63);
  bout = out_at(bm, b63, nl);
  return act ? x - y - lane_bit(bm) : 0ull;
}

LFP_FN W2 add2(W2 x, W2 y, uint32_t cin, uint32_t &cout) {
  const uint64_t sl = x.lo + y.lo, sh = x.hi + y.hi;
  uint32_t c;
  const uint64_t cl = chain(ballot(sl < x.lo), ballot(sl == ~0ull), cin, c);
  const uint64_t ch = chain(ballot(sh < x.hi), ballot(sh == ~0ull), c, cout);
  W2 r;
  r.lo = sl + lane_bit(cl);
  r.hi = sh + lane_bit(ch);
  return r;
}

// limb j (per lane, any value) of the number held one limb per lane in v;
// 0 outside [0, 64)
LFP_FN uint64_t reg_limb(uint64_t v, int j) {
  const uint64_t t = shfl64(v, j & 63);
  return (j >= 0 && j < 64) ? t : 0ull;
}

LFP_FN uint64_t win_limb(W2 w, int j) {
  const uint64_t a = shfl64(w.lo, j & 63), b = shfl64(w.hi, j & 63);
  return (j >= 0 && j < 64) ? a : ((j >= 64 && j < 128) ? b : 0ull);
}

// bits [base, base + 64) of the window; base & 63 wave-uniform
LFP_FN uint64_t win_bits(W2 w, int64_t base) {
  const int li = (int)(base >> 6);
  const int r = (int)(base & 63);
  const uint64_t x0 = win_limb(w, li), x1 = win_limb(w, li + 1);
  return r ? ((x0 >> r) | (x1 << (64 - r))) : x0;
}

// m + 1 over lanes < nl; ovf = 1 when it carried out of p bits, m is then
// 2^(p-1) (the caller adds one to the exponent)
LFP_FN uint64_t inc_mant(uint64_t m, int nl, uint32_t &ovf) {
  const int l = lane_id();
  const bool act = l < nl;
  uint32_t c63;
  const uint64_t cm = chain(0ull, ballot(act && m == ~0ull), 1u, c63);
  ovf = out_at(cm, c63, nl);
  uint64_t r = act ? m + lane_bit(cm) : 0ull;
  if (ovf) r = (l == nl - 1) ? (1ull << 63) : 0ull;
  return r;
}

// RN_p of the non-zero window value w plus, when sticky, an inexact
// remainder below w's bit 0 (which must then lie below the rounding
// position).  Returns this lane's mantissa limb; bl = bit length of the
// rounded value in w's units (value = mantissa 2^(bl - p)).
LFP_FN uint64_t round_win(W2 w, uint32_t sticky, int nl, int64_t &bl) {
  const int l = lane_id();
  const uint64_t nzl = ballot(w.lo != 0), nzh = ballot(w.hi != 0);
  const int top = nzh ? 64 + msb64(nzh) : msb64(nzl);
  const uint64_t twh = readlane64(w.hi, nzh ? top - 64 : 0);
  const uint64_t twl = readlane64(w.lo, nzh ? 0 : top);
  const int64_t T = 64 * (int64_t)top + 64 - __builtin_clzll(nzh ? twh : twl);
  const int64_t D = T - 64 * (int64_t)nl;  // lowest kept bit
  const uint64_t mw = win_bits(w, D + 64 * (int64_t)l);
  uint64_t m = l < nl ? mw : 0ull;
  uint32_t rb = 0, st = sticky;
  if (D >= 1) {
    const int64_t rp = D - 1;
    const int rl = (int)(rp >> 6), rr = (int)(rp & 63);
    const uint64_t a = readlane64(w.lo, rl & 63), b = readlane64(w.hi, rl & 63);
    const uint64_t rlimb = rl < 64 ? a : b;
    rb = (uint32_t)((rlimb >> rr) & 1ull);
    const uint64_t ml = rl >= 64 ? ~0ull : low_mask(rl);
    const uint64_t mh = rl >= 64 ? low_mask(rl - 64) : 0ull;
    st |= (uint32_t)(((rlimb & low_mask(rr)) != 0) | ((nzl & ml) != 0) | ((nzh & mh) != 0));
  }
  const uint32_t lsb = (uint32_t)(readlane64(m, 0) & 1ull);
  uint32_t ovf = 0;
  if (rb && (st || lsb)) m = inc_mant(m, nl, ovf);
  bl = T + ovf;
  return m;
}

// mantissa comparison: sign of a - b
LFP_FN int cmp_mant(uint64_t a, uint64_t b) {
  const uint64_t diff = ballot(a != b);
  if (!diff) return 0;
  const int t = msb64(diff);
  const uint64_t x = readlane64(a, t), y = readlane64(b, t);
  return x > y ? 1 : -1;
}

// exact |a| against |b| (zero the smallest): -1, 0, 1
LFP_FN int cmp_abs(const WF &a, const WF &b) {
  const bool za = is_zero(a), zb = is_zero(b);
  if (za || zb) return (za && zb) ? 0 : (za ? -1 : 1);
  if (a.e != b.e) return a.e > b.e ? 1 : -1;
  return cmp_mant(a.m, b.m);
}

// limb j <- limb j-1 over the window (limb 0 <- 0)
LFP_FN W2 up_limb(W2 w) {
  const int l = lane_id();
  const uint64_t a = rot1_64(w.lo), b = up1_64(w.hi);
  W2 r;
  r.lo = l ? a : 0ull;
  r.hi = l ? b : a;
  return r;
}

// a b = lo + hi 2^64 from four 32 x 32 -> 64-bit multiply-adds
LFP_FN void mul128(uint64_t a, uint64_t b, uint64_t &lo, uint64_t &hi) {
  const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32);
  const uint32_t b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
  const uint64_t p00 = (uint64_t)a0 * b0;
  const uint64_t p01 = (uint64_t)a0 * b1 + (p00 >> 32);
  const uint64_t p10 = (uint64_t)a1 * b0 + (uint32_t)p01;
  hi = (uint64_t)a1 * b1 + (p01 >> 32) + (p10 >> 32);
  lo = (p10 << 32) | (uint32_t)p00;
}

// w (five 32-bit words, least significant first) += a b
LFP_FN void mac5(uint32_t (&w)[5], uint64_t a, uint64_t b) {
  uint64_t lo, hi;
  mul128(a, b, lo, hi);
  uint32_t c;
  w[0] = addc32(w[0], (uint32_t)lo, 0u, &c);
  w[1] = addc32(w[1], (uint32_t)(lo >> 32), c, &c);
  w[2] = addc32(w[2], (uint32_t)hi, c, &c);
  w[3] = addc32(w[3], (uint32_t)(hi >> 32), c, &c);
  w[4] += c;
}

// The product of two mantissas by a loop over the limbs of a: cheaper than
// the matrix-core form for few limbs.  Lane l sums column l of the schoolbook
// product (a_i b_(l-i), i <= l), then column l + 64 (a_i b_(l+64-i), i > l),
// in one 160-bit accumulator (a column sum is below 64 2^128); the running
// sum is copied aside when i passes l, and the high column is the final sum
// minus that copy.
LFP_FN W2 prod_loop(uint64_t am, uint64_t bm, int nl) {
  const int l = lane_id();
  uint32_t w[5] = {0u, 0u, 0u, 0u, 0u}, k[5] = {0u, 0u, 0u, 0u, 0u};
  uint64_t bv = bm;  // b_((l - i) mod 64) at step i: rotated by one lane per step
  for (int i = 0; i < nl; ++i) {
    const uint64_t ai = readlane64(am, i);
    const bool sw = l + 1 == i;
#pragma unroll
    for (int q = 0; q < 5; ++q) k[q] = sw ? w[q] : k[q];
    mac5(w, ai, bv);
    bv = rot1_64(bv);
  }
  const bool banked = l + 1 < nl;  // lanes >= nl-1 never reach their high column
  uint32_t lw[5], hw[5], br = 0u;
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    lw[q] = banked ? k[q] : w[q];
    const uint32_t d = addc32(w[q], ~k[q], 1u - br, &br);  // w - k, br: borrow out
    br = 1u - br;
    hw[q] = banked ? d : 0u;
  }
  W2 A, B, C;
  A.lo = ((uint64_t)lw[1] << 32) | lw[0];
  A.hi = ((uint64_t)hw[1] << 32) | hw[0];
  B.lo = ((uint64_t)lw[3] << 32) | lw[2];
  B.hi = ((uint64_t)hw[3] << 32) | hw[2];
  C.lo = lw[4];
  C.hi = hw[4];
  B = up_limb(B);
  C = up_limb(up_limb(C));  // column 2nl-2 holds one product: its c2 is 0
  uint32_t co;
  W2 S = add2(A, B, 0u, co);
  S = add2(S, C, 0u, co);
  return S;
}

// LDS of one wavefront for the matrix-core product: the signed bytes of one
// operand from PA, of the other in reverse order from PB, with the zero
// bytes around them that the fragments below reach (prod_init), and the 256
// partial sums.
constexpr int PA = 16, PB = 608 + 432, PW = 608 + 1200;
constexpr int PROD_LDS = PW + 256 * 8;  // bytes, a multiple of 16

LFP_FN void prod_init(uint8_t *buf) {
  for (int k = 16 * lane_id(); k < PW; k += 16 * 64) *(v4i32 *)(buf + k) = v4i32{0, 0, 0, 0};
  lds_order();
}

// The exact product of two nl-limb numbers on the matrix cores: limbs 0 ..
// nl-1 in lanes 0 .. nl-1 of lo, limbs nl .. 2nl-1 of hi.  CL - 16 < nl <= CL.
//
// With the operands in signed bytes (x + 0x80...80 has the bytes d_i + 128;
// its carry out c gives x = sum d_i 256^i + c 2^p) the byte products are a
// convolution.  Output byte 16 C + r, as column C and row r of a tile, is
//   sum_k d_a[r + k - 15] d_b[16 C + 15 - k],
// a contraction over k of sixteen shifted copies of a (rows) with sixteen
// 16-byte steps of b (columns): v_mfma_i32_16x16x64_i8, 26 of them at 49 to
// 64 limbs where the loop issues 4 nl multiply-adds and their carries.  Row
// fragments start at any byte (five aligned words and four funnel shifts),
// column fragments on 16-byte lines of the reversed copy; which tiles meet
// is fixed by CL, so nothing branches.  A sum has at most 512 terms, so four
// neighbouring ones make a 48-bit word of weight 2^32, and through LDS each
// lane takes the words of its limbs.  The carries c add c_a b + c_b a at
// limb nl, and the signed excess of each limb goes to the next one through
// the carry chain under a bias.  All is modulo 2^(128 nl), which the product
// is below.  With it and the sum below, the panel's rank-1 update of a column
// went from 22.5 to 10 us at 49 limbs, a U12 leaf from 499 to 179 us.
template <int CL>
LFP_FN void prod_mfma(uint64_t am, uint64_t bm, int nl, uint8_t *buf, uint64_t &lo, uint64_t &hi) {
  constexpr uint64_t B80 = 0x8080808080808080ull;
  constexpr uint64_t BIAS = 1ull << 20;
  constexpr int NT = CL / 16, NK = ((8 * CL + 14) >> 6) + 1;  // column tiles, k steps
  const int l = lane_id(), r = l & 15, kg = l >> 4;
  const bool act = l < nl;
  uint32_t ca, cb;
  const uint64_t da = add1(am, B80, nl, 0u, ca) ^ B80, db = add1(bm, B80, nl, 0u, cb) ^ B80;
  const int rev = PB + 8 * (nl & 1);  // reversed byte i at rev + i; rev + 8 nl on a 16-byte line
  if (act) {
    *(uint64_t *)(buf + PA + 8 * l) = da;
    *(uint64_t *)(buf + rev + 8 * (nl - 1 - l)) = __builtin_bswap64(db);
  }
  lds_order();
  const uint8_t *pa = buf + ((PA - 15 + r + 16 * kg) & ~3);
  const uint32_t sh = 8u * ((PA - 15 + r) & 3);
  const uint8_t *pb = buf + rev + 8 * nl - 16 * (r + 1) + 16 * kg;
  v4i32 acc[NT];
#pragma unroll
  for (int T = 0; T < NT; ++T) acc[T] = v4i32{0, 0, 0, 0};
#pragma unroll
  for (int t = 0; t < NK; ++t) {
    uint32_t w[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) w[q] = *(const uint32_t *)(pa + 64 * t + 4 * q);
    v4i32 fa;
#pragma unroll
    for (int q = 0; q < 4; ++q) fa[q] = (int)align_bits(w[q + 1], w[q], sh);
#pragma unroll
    for (int T = 0; T < NT; ++T) {
      // columns 16 T .. 16 T + 15 meet bytes of b for k in this range
      const int k0 = 256 * T + 16 - 8 * CL, k1 = 256 * T + 255;
      if (t >= (k0 > 0 ? k0 >> 6 : 0) && t <= k1 >> 6)
        acc[T] = mfma_bytes(fa, *(const v4i32 *)(pb - 256 * T + 64 * t), acc[T]);
    }
  }
  int64_t *pw = (int64_t *)(buf + PW);
#pragma unroll
  for (int T = 0; T < NT; ++T)
    pw[64 * T + 4 * r + kg] = (int64_t)acc[T][0] + ((int64_t)acc[T][1] << 8) +
                              ((int64_t)acc[T][2] << 16) + ((int64_t)acc[T][3] << 24);
  lds_order();
  // this lane's limbs as 128-bit signed sums: low word, signed excess
  auto take = [&](int limb, uint64_t &v, int64_t &x) {
    const int64_t w0 = pw[2 * limb], w1 = pw[2 * limb + 1];
    const uint64_t s = (uint64_t)w1 << 32;
    v = (uint64_t)w0 + s;
    x = (w1 >> 32) + (w0 >> 63) + (v < s ? 1 : 0);
  };
  uint64_t vl, vh;
  int64_t xl, xh;
  take(act ? l : 0, vl, xl);
  take(act ? nl + l : 0, vh, xh);
  const uint64_t ea = ca ? bm : 0ull, eb = cb ? am : 0ull;
  vh += ea;
  xh += vh < ea ? 1 : 0;
  vh += eb;
  xh += vh < eb ? 1 : 0;
  const uint64_t bl = (uint64_t)xl + BIAS, bh = (uint64_t)xh + BIAS;
  const uint64_t il = up1_64(bl), ip = up1_64(bh);  // whole-wavefront moves: every lane
  const uint64_t ih = l ? ip : readlane64(bl, nl - 1);
  uint32_t c;
  vl = add1(vl, il, nl, 0u, c);
  vh = add1(vh, ih, nl, c, c);
  lo = sub1(vl, l ? BIAS : 0ull, nl, 0u, c);
  hi = sub1(vh, BIAS, nl, c, c);
  lds_order();  // the buffer may be filled again
}

// RN_p(a b).  CL = 0: by the loop; CL = 16, 32, 48 or 64 with CL - 16 < nl <=
// CL: on the matrix cores, buf PROD_LDS bytes of LDS of this wavefront after
// prod_init.
template <int CL>
LFP_FN WF mul(const WF &a, const WF &b, int nl, uint8_t *buf) {
  if (is_zero(a) || is_zero(b)) return wf_zero();
  WF r;
  r.s = (a.s ^ b.s) & 1u;
  if constexpr (CL == 0) {
    int64_t bl;
    r.m = round_win(prod_loop(a.m, b.m, nl), 0u, nl, bl);
    r.e = (int32_t)(bl + a.e + b.e - 128 * (int64_t)nl);
  } else {
    uint64_t lo, hi;
    prod_mfma<CL>(a.m, b.m, nl, buf, lo, hi);
    // the product of two normalised mantissas has 128 nl bits or one less
    const uint64_t th = readlane64(hi, nl - 1), tl = readlane64(lo, nl - 1);
    const uint64_t low = ballot(lo != 0) & low_mask(nl - 1);
    const uint32_t sh = (uint32_t)(th >> 63) ^ 1u;
    uint64_t m = hi;
    if (sh) {
      const uint64_t up = up1_64(hi), below = lane_id() ? up : tl;
      m = lane_id() < nl ? (hi << 1) | (below >> 63) : 0ull;
    }
    const uint32_t rb = (uint32_t)((tl << sh) >> 63);
    const uint32_t st = (uint32_t)(((tl << sh) << 1) != 0) | (uint32_t)(low != 0);
    uint32_t ovf = 0;
    if (rb && (st || (readlane64(m, 0) & 1ull))) m = inc_mant(m, nl, ovf);
    r.m = m;
    r.e = a.e + b.e - (int32_t)sh + (int32_t)ovf;
  }
  return r;
}

// RN_p(a + (-1)^negb b).  The smaller operand is shifted right by the
// exponent gap onto the larger one's limbs, with 64 further bits in a
// uniform guard word and the rest as a sticky bit.  A gap of two or more
// leaves a difference at most one bit short, and a smaller one loses at most
// one bit into the guard word, so guard and sticky decide the rounding.
LFP_FN WF add(const WF &a, const WF &b, uint32_t negb, int nl) {
  const uint32_t bs = (b.s ^ negb) & 1u;
  const bool za = is_zero(a), zb = is_zero(b);
  if (za && zb) return wf_zero();
  if (zb) return a;
  if (za) {
    WF r = b;
    r.s = bs;
    return r;
  }
  // X the operand of larger magnitude
  const int c = (a.e != b.e) ? (a.e > b.e ? 1 : -1) : cmp_mant(a.m, b.m);
  const bool sw = c < 0;
  const uint64_t Xm = sw ? b.m : a.m, Ym = sw ? a.m : b.m;
  const int32_t Xe = sw ? b.e : a.e, Ye = sw ? a.e : b.e;
  const uint32_t Xs = sw ? bs : a.s, Ys = sw ? a.s : bs;
  const int64_t d = (int64_t)Xe - Ye;
  const int64_t p = 64 * (int64_t)nl;
  WF r;
  r.s = Xs;
  if (d >= p + 2) {
    // |Y| < 2^(Xe-p-2): below half the spacing on either side of X
    r.m = Xm;
    r.e = Xe;
    return r;
  }
  const int l = lane_id();
  const bool act = l < nl;
  const int q = (int)(d >> 6), rr = (int)(d & 63);
  // limbs at or past nl are 0, and so is what falls off the top
  uint64_t Y = q == 0 ? Ym : reg_limb(Ym, l + q);
  if (rr) Y = (Y >> rr) | (dn1_64(Y) << (64 - rr));
  const uint64_t yq = q < 64 ? readlane64(Ym, q & 63) : 0ull;
  const uint64_t yb = q > 0 ? readlane64(Ym, q - 1) : 0ull;
  uint64_t G = rr ? (yq << (64 - rr)) | (yb >> rr) : yb;
  uint32_t st = (uint32_t)((yb & low_mask(rr)) != 0);
  if (q > 1) st |= (uint32_t)((ballot(Ym != 0) & low_mask(q - 1)) != 0);
  uint64_t m;
  uint32_t rb, co;
  if (Xs == Ys) {
    m = add1(Xm, Y, nl, 0u, co);
    r.e = Xe + (int32_t)co;
    if (co) {
      const uint64_t dn = dn1_64(m), above = l == nl - 1 ? 1ull : dn;
      rb = (uint32_t)(readlane64(m, 0) & 1ull);
      m = act ? (m >> 1) | (above << 63) : 0ull;
      st |= (uint32_t)(G != 0);
    } else {
      rb = (uint32_t)(G >> 63);
      st |= (uint32_t)((G << 1) != 0);
    }
  } else {
    // G and the sticky part come off one unit: 2^64 - G, and when something
    // lies below G one less, the sticky bit then standing for the rest
    const uint32_t bin = (uint32_t)(G != 0) | st;
    m = sub1(Xm, Y, nl, bin, co);
    G = 0ull - G - st;
    const uint64_t nz = ballot(m != 0);
    if (nz == 0) {
      if (G == 0) return wf_zero();  // exact cancellation: +0
      const int lz = __builtin_clzll(G);
      r.m = l == nl - 1 ? G << lz : 0ull;
      r.e = (int32_t)(Xe - p - lz);
      return r;
    }
    const int top = msb64(nz), u = nl - 1 - top;
    const int lz = __builtin_clzll(readlane64(m, top));
    uint64_t g = G;
    if (u) {
      // whole limbs up: the guard word follows the lowest one
      const uint64_t t = reg_limb(m, l - u);
      m = act ? (l == u - 1 ? G : t) : 0ull;
      g = 0ull;
    }
    if (lz) {
      const uint64_t up = up1_64(m), below = l ? up : g;
      m = act ? (m << lz) | (below >> (64 - lz)) : 0ull;
      g <<= lz;
    }
    r.e = Xe - 64 * u - lz;
    rb = (uint32_t)(g >> 63);
    st |= (uint32_t)((g << 1) != 0);
  }
  if (rb && (st || (readlane64(m, 0) & 1ull))) {
    uint32_t ovf;
    m = inc_mant(m, nl, ovf);
    r.e += (int32_t)ovf;
  }
  r.m = m;
  return r;
}

// A lower bound of 2^127 / w within 4 units, for 2^63 < w < 2^64: the
// binary64 reciprocal corrected once by its exact integer residual.
LFP_FN uint64_t recip127(uint64_t w) {
  const double y = 1.0 / (double)w;
  const double ys = y * 0x1p127;  // at most 2^64
  const uint64_t y0 = (uint64_t)(ys < 0x1.fffffffffffffp63 ? ys : 0x1.fffffffffffffp63);
  uint64_t pl, ph;
  mul128(w, y0, pl, ph);
  // 2^127 - w y0, below 2^77 in magnitude
  const int64_t eh = (int64_t)((1ull << 63) - ph - (pl != 0 ? 1ull : 0ull));
  const double e = (double)eh * 0x1p64 + (double)(0ull - pl);
  return y0 + (uint64_t)(int64_t)__builtin_floor(e * y) - 2ull;
}

// RN_p(a / b); b must be non-zero (a zero b gives zero).
//
// Long division in digits of 58 bits with nothing carried between the lanes:
// R <- 2^58 R - q V, each lane keeping the borrows it owes the next lane (at
// most 3), which enter that lane's next subtraction.  The digit
// q = floor(n inv / 2^63) takes n from the top of R and the uniform inv
// from the divisor's top limb, both rounded down, so q never exceeds the
// true digit and falls short of it by less than 12: R stays in [0, 12 V), n
// below 2^62 and q below 2^63.  The digits overlap by five bits; one lane
// holds each, and at the end they are added up, R is brought below V and its
// zero test is the sticky bit.  At least two bits follow the rounding
// position.  Per digit one readlane, one uniform and one per-lane 64 x 64-bit
// product in the dependent chain; the division kernel of a panel column at 49
// limbs, one division deep, took 31 us with 64-bit digits whose remainder was
// carried through every step and takes 16 us.
LFP_FN WF div(const WF &a, const WF &b, int nl) {
  if (is_zero(a) || is_zero(b)) return wf_zero();
  constexpr int DB = 58;
  const int l = lane_id();
  const bool act = l < nl;
  const uint64_t V = b.m;
  const uint64_t v1 = readlane64(V, nl - 1);  // top divisor limb, >= 2^63
  const uint64_t inv = v1 == ~0ull ? 1ull << 63 : recip127(v1 + 1ull);
  const int K = (64 * nl + 2 + DB - 1) / DB;
  uint64_t R = a.m, top = 0, dq0 = 0, dq1 = 0;
  uint32_t owe = 0;  // borrows of this lane on the next one
  auto step = [&]() -> uint64_t {
    const uint64_t n = (top << DB) | (readlane64(R, nl - 1) >> (64 - DB));
    uint64_t ql, qh;
    mul128(n - (n > 0 ? 1ull : 0ull), inv, ql, qh);
    const uint64_t q = (qh << 1) | (ql >> 63);
    uint64_t lo, hi;
    mul128(q, V, lo, hi);
    const uint64_t x = (R << DB) | (up1_64(R) >> (64 - DB));
    const uint64_t hin = up1_64(hi);
    const uint64_t oin = (uint64_t)up1_32(owe) << DB;
    uint32_t bo = x < lo ? 1u : 0u;
    uint64_t t = x - lo;
    bo += t < hin ? 1u : 0u;
    t -= hin;
    bo += t < oin ? 1u : 0u;
    t -= oin;
    R = act ? t : 0ull;
    owe = act ? bo : 0u;
    // the part of 2^58 R - q V above limb nl-1; owe there is settled at once
    top = n - readlane64(hi, nl - 1) - (uint64_t)(uint32_t)readlane64(owe, nl - 1);
    return q;
  };
  for (int i = 0; i < (K < 64 ? K : 64); ++i) {
    const uint64_t q = step();
    dq0 = l == i ? q : dq0;
  }
  for (int i = 64; i < K; ++i) {
    const uint64_t q = step();
    dq1 = l == i - 64 ? q : dq1;
  }
  uint32_t bo, cnt = 0;
  owe = l == nl - 1 ? 0u : owe;
  R = sub1(R, (uint64_t)up1_32(owe), nl, 0u, bo);
  top -= bo;
  for (int k = 0; k < 16 && (top != 0 || cmp_mant(R, V) >= 0); ++k) {
    R = sub1(R, V, nl, 0u, bo);
    top -= bo;
    ++cnt;
  }
  const uint32_t rem = ballot(R != 0) != 0 ? 1u : 0u;
  // Q = sum_t digit_t 2^(58 t), digit t = q of step K-1-t: a limb meets three
  auto digit = [&](int t) -> uint64_t {
    const int i = K - 1 - t;
    const uint64_t x = shfl64(dq0, i & 63), y = K > 64 ? shfl64(dq1, i & 63) : 0ull;
    return t < 0 || i < 0 ? 0ull : (i < 64 ? x : y);
  };
  auto limb = [&](int k, uint64_t &v, uint64_t &cy) {
    const int th = (64 * k + 63) / DB;
    v = 0;
    cy = 0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int off = DB * (th - j) - 64 * k;
      const uint64_t g = digit(th - j);
      const uint64_t s = off >= 0 ? g << off : (off > -64 ? g >> -off : 0ull);
      v += s;
      cy += v < s ? 1ull : 0ull;
    }
  };
  W2 Q, C;
  limb(l, Q.lo, C.lo);
  Q.hi = 0;
  C.hi = 0;
  if (DB * K + 64 > 64 * 64) limb(l + 64, Q.hi, C.hi);  // uniform
  C = up_limb(C);
  C.lo = l ? C.lo : (uint64_t)cnt;
  uint32_t co;
  Q = add2(Q, C, 0u, co);
  int64_t bl;
  WF r;
  r.m = round_win(Q, rem, nl, bl);
  r.e = (int32_t)(bl - (int64_t)DB * K + a.e - b.e);
  r.s = (a.s ^ b.s) & 1u;
  return r;
}

// RN_p(a / b) with y = RN_p(1 / b) at hand (CL > 0): two products instead of
// the digit chain.  a y is the quotient's p bits to within two units; its
// exact remainder corrects it and decides the rounding.
template <int CL>
LFP_FN WF div_by(const WF &a, const WF &b, const WF &y, int nl, uint8_t *buf) {
  if (is_zero(a) || is_zero(b)) return wf_zero();
  const int l = lane_id();
  const bool act = l < nl;
  // b a power of two: 1/b has another exponent
  if (y.e + b.e != 1) return div(a, b, nl);
  const uint32_t d0 = cmp_mant(a.m, b.m) >= 0 ? 1u : 0u;
  // Q ~ floor(a 2^(p - d0) / b), taken two units low
  uint64_t lo, hi;
  prod_mfma<CL>(a.m, y.m, nl, buf, lo, hi);
  const uint64_t lt = readlane64(lo, nl - 1);
  uint64_t Q = hi;
  if (!d0) {
    const uint64_t up = up1_64(hi), below = l ? up : lt;
    // a 2p-bit product: its rounding reached 2^p
    Q = (readlane64(hi, nl - 1) >> 63) ? ~0ull : (hi << 1) | (below >> 63);
    Q = act ? Q : 0ull;
  }
  uint32_t c;
  Q = sub1(Q, l == 0 ? 2ull : 0ull, nl, 0u, c);
  // R = a 2^(p - d0) - Q b, its part above limb nl-1 in rh
  prod_mfma<CL>(Q, b.m, nl, buf, lo, hi);
  const uint64_t a0 = readlane64(a.m, 0);
  uint64_t al = 0, ah = a0;
  if (d0) {
    al = l == nl - 1 ? a0 << 63 : 0ull;
    ah = (a0 >> 1) | ((nl > 1 ? readlane64(a.m, 1) : 0ull) << 63);
  }
  uint64_t R = sub1(al, lo, nl, 0u, c);
  int64_t rh = (int64_t)(ah - readlane64(hi, 0) - c);
  uint32_t cnt = 0;
  for (int k = 0; k < 16 && (rh != 0 || cmp_mant(R, b.m) >= 0); ++k) {
    R = sub1(R, b.m, nl, 0u, c);
    rh -= c;
    ++cnt;
  }
  Q = add1(Q, l == 0 ? (uint64_t)cnt : 0ull, nl, 0u, c);
  // against half the divisor
  const uint32_t over = (uint32_t)(readlane64(R, nl - 1) >> 63);
  const uint64_t ru = up1_64(R), R2 = act ? (R << 1) | (ru >> 63) : 0ull;
  const int h = over ? 1 : cmp_mant(R2, b.m);
  uint32_t ovf = 0;
  if (h > 0 || (h == 0 && (readlane64(Q, 0) & 1ull))) Q = inc_mant(Q, nl, ovf);
  WF r;
  r.m = Q;
  r.e = a.e - b.e + (int32_t)d0 + (int32_t)ovf;
  r.s = (a.s ^ b.s) & 1u;
  return r;
}

// RN_p(c - RN_p(a b)): the multiply-subtract of the panel, the U12 solve
// and the substitutions
template <int CL>
LFP_FN WF fms(const WF &c, const WF &a, const WF &b, int nl, uint8_t *buf) {
  return add(c, mul<CL>(a, b, nl, buf), 1u, nl);
}

}  // namespace lfp
