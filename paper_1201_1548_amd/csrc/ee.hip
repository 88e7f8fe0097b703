// (b)+(c) evaluation and univariate resultant over F_p, one lane per
// (prime, point), both coefficient arrays in registers, in signed Montgomery
// arithmetic; the evaluation on the int8 matrix cores.
//
// Signed arithmetic.  A residue x is any int32 with |x| <= 1.125 p; redc_s(t) =
// t 2^{-32} mod p = (t + m p) / 2^32 with m = -t p^{-1} mod 2^32 taken as int32, so
// |redc_s(t)| <= |t| / 2^32 + p / 2.  With 3 p < 2^32 a product l x contributes at
// most |l| |x| / (3 p): a sum l2 x + l1 y + n2 z with |l2|, |l1| <= 0.584 p
// (products of two balanced residues), |n2| <= p / 2 (balanced) and |x|, |y|,
// |z| <= 1.125 p gives at most (0.584 + 0.584 + 0.5) 1.125 / 3 + 0.5 < 1.126, and
// no correction is needed after the reduction: five instructions (three
// multiply-adds, the low product, the multiply-add of the reduction) where
// the unsigned form takes seven.  Only the leading coefficients are balanced.
//
// Evaluation.  The rows of f and g at 64 points are a matrix product: 16 rows x
// 16 points x KW powers per v_mfma_i32_16x16x{32,64}_i8 and pair of balanced
// base-256 digits (the reduction writes the residues as digit words; the
// powers' digit planes go through LDS), seven classes of equal weight, and per
// value the classes join in int32 pairs and one redc_s (nine instructions
// instead of one multiply-add per coefficient and a 23-instruction fold).
// Four point tiles fill the wave; a 4 x 4 transpose over its 16-lane rows
// (v_permlane{32,16}_swap) leaves every lane with the values of its own point.
// Rows longer than KW take Horner steps in a^KW.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <type_traits>
#include <utility>

#include "device.hpp"
#include "job.hpp"
#include "kernels.hpp"

namespace bires {

namespace {

// (plain C: v_mad_i64_i32; around inline assembly the compiler puts wait states)
__device__ __forceinline__ int64_t mul_s(int32_t a, int32_t b) { return (int64_t)a * (int64_t)b; }
__device__ __forceinline__ int64_t mad_s(int32_t a, int32_t b, int64_t c) { return mul_s(a, b) + c; }
// The prime with the positive inverse p^{-1} mod 2^32 beside ModP's negative one
// (opaque, or the product with it becomes a product and a negation).
struct SModP : ModP {
  uint32_t pin;
  __device__ __forceinline__ explicit SModP(const ModP& q) : ModP(q), pin(0u - q.pinv) { asm("" : "+s"(pin)); }
};

// A copy whose p is opaque, for the code of one block: as a factor p is sign-extended,
// and an extension shared between blocks is multiplied as a 64-bit number.
__device__ __forceinline__ SModP own_mod(SModP q) {
  asm("" : "+s"(q.p));
  return q;
}

// t 2^{-32} mod p.  redc_s takes the low words' equality out of the difference:
// with m = t p^{-1} mod 2^32, t - m p has a zero low word, so its high word is
// hi(t) - mulhi(m, p), a 32-bit result of its own.  redc_p is one multiply-add,
// but leaves its result in the upper half of a register pair, which the
// register allocator then reserves for it: the two coefficient arrays take one
// form each, so that the values of one lie in the lower halves of the other's
// pairs.
__device__ __forceinline__ int32_t redc_s(int64_t t, const SModP& q) {
  const int32_t m = (int32_t)((uint32_t)t * q.pin);
  int32_t r = (int32_t)(t >> 32) - __mulhi(m, (int32_t)q.p);
  // an opaque 32-bit value: otherwise its sign extension is kept as a 64-bit
  // register pair wherever it serves as a factor
  asm("" : "+v"(r));
  return r;
}
__device__ __forceinline__ int32_t redc_p(int64_t t, const SModP& q) {
  const int32_t m = (int32_t)((uint32_t)t * q.pinv);
  int32_t r = (int32_t)(mad_s(m, (int32_t)q.p, t) >> 32);
  asm("" : "+v"(r));
  return r;
}
template <bool PAIR>
__device__ __forceinline__ int32_t redc_to(int64_t t, const SModP& q) {
  if constexpr (PAIR) return redc_p(t, q);
  return redc_s(t, q);
}
__device__ __forceinline__ int32_t smul(int32_t a, int32_t b, const SModP& q) { return redc_s(mul_s(a, b), q); }
template <bool PAIR = false>
__device__ __forceinline__ int32_t sdot2(int32_t a, int32_t b, int32_t c, int32_t d, const SModP& q) {
  return redc_to<PAIR>(mad_s(c, d, mul_s(a, b)), q);
}
template <bool PAIR>
__device__ __forceinline__ int32_t sdot3(int32_t a, int32_t b, int32_t c, int32_t d, int32_t e, int32_t f,
                                         const SModP& q) {
  return redc_to<PAIR>(mad_s(e, f, mad_s(c, d, mul_s(a, b))), q);
}
// The representative in [-(p-1)/2, (p-1)/2] of x, |x| < 1.5 p: v = x + (p-1)/2
// is brought into [0, p) by two unsigned minima (a negative v wraps above
// v + p; v - p wraps above v below p).
__device__ __forceinline__ int32_t balance(int32_t x, uint32_t p) {
  const uint32_t h = (p - 1u) >> 1;
  uint32_t v = (uint32_t)x + h;
  v = umin32(v, v + p);
  v = umin32(v, v - p);
  return (int32_t)(v - h);
}
__device__ __forceinline__ int32_t spow(int32_t a, uint32_t e, const SModP& q) {  // e >= 1
  int32_t r = 0;
  bool first = true;
  while (e) {
    if (e & 1u) {
      r = first ? a : smul(r, a, q);
      first = false;
    }
    e >>= 1;
    if (e) a = smul(a, a, q);
  }
  return r;
}

// Balanced digit word of v, |v| < 2^30 (digits4 of the symmetric representative).
__device__ __forceinline__ uint32_t sdigits(int32_t v) { return ((uint32_t)v + 0x808080u) ^ 0x808080u; }

// Operands of one matrix instruction: KW / 4 bytes per lane and digit plane.
template <int KW>
struct Oper;
template <>
struct Oper<32> {
  typedef long long T;
  static __device__ __forceinline__ T pack(const uint32_t (&w)[2]) { return (T)(((uint64_t)w[1] << 32) | w[0]); }
  static __device__ __forceinline__ im_v4i mma(T a, T b, im_v4i c) {
    return __builtin_amdgcn_mfma_i32_16x16x32_i8(a, b, c, 0, 0, 0);
  }
};
template <>
struct Oper<64> {
  typedef im_v4i T;
  static __device__ __forceinline__ T pack(const uint32_t (&w)[4]) {
    return (im_v4i){(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
  }
  static __device__ __forceinline__ im_v4i mma(T a, T b, im_v4i c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
  }
};

// What the evaluation of a block needs besides the rows.
struct EvalCtx {
  const int8_t* planes;  // LDS [4][64][KW]: digit planes of the powers of the block's points
  int32_t w32, w48;      // balanced 2^32, 2^48 mod p (uniform)
  int32_t one;           // balanced Montgomery 1
  int32_t apw;           // this lane's a^KW, balanced (rows longer than KW)
  int dmax;              // largest x-degree
};

// The rows of one operand, top-aligned: row k holds y^(deg - k).
struct Rows {
  const uint32_t* r;
  const int32_t* deg_x;
  int lp, deg;
};

// A tile of 16 rows at the block's points; out[i]: this lane's value of the
// tile's row i, zero past the degree.  Rows base .. base + 15 of x (which = 0) or
// of y (1), or (2) the 4 RJ rows from base on of x and then as many of y.  Row
// slot rho of the matrix tile holds row 4 (rho % 4) + rho / 4, so that register j
// of lane group g is row 4 j + g: the slots past the degree are whole registers
// and their epilogue is skipped.
//
// Pieces of KW coefficients: piece `part` alone, which returns false (and no
// values) if no row of the tile reaches it, or (part < 0) all of them, joined by
// Horner's rule in a^KW.
//
// Rows shorter than the tile's pieces are read past their end and masked: at most
// the longest row's coefficients and 64 more from the start of the last row on, which
// the point count (at least one more than any x-degree) keeps inside the values
// that follow the residues and their slack.
template <int KW, int RJ>
__device__ __forceinline__ bool eval_tile(const Rows& x, const Rows& y, int which, int base, int part, const EvalCtx& E,
                                          int32_t (&out)[16], const SModP& q0) {
  typedef Oper<KW> OP;
  constexpr int NQ = KW / 16;  // quads of coefficients per lane
  const int l = lane_id(), rho = l & 15, g = l >> 4;
  int jr = rho & 3;
  bool isy = which == 1, past = false;
  int live = 0;  // registers with rows up to the degree
  if (which == 2) {
    isy = jr >= RJ;
    past = jr >= 2 * RJ;
    jr = isy ? jr - RJ : jr;
#pragma unroll
    for (int j = 0; j < 2 * RJ; ++j)
      live |= base + 4 * (j % RJ) <= (j < RJ ? x.deg : y.deg) ? 1 << j : 0;
  } else {
    const int d = which ? y.deg : x.deg;
#pragma unroll
    for (int j = 0; j < 4; ++j) live |= base + 4 * j <= d ? 1 << j : 0;
  }
  const int k = base + 4 * jr + (rho >> 2), deg = isy ? y.deg : x.deg, lp = isy ? y.lp : x.lp;
  const uint32_t* rows = isy ? y.r : x.r;
  const int row = max(deg - k, 0);
  past |= k > deg;
  const bool longrows = E.dmax >= KW;
  const int rd = longrows ? (isy ? y.deg_x : x.deg_x)[row] : 0;
  bool first = true;
  for (int ch = part >= 0 ? part : longrows ? E.dmax / KW : 0; ch >= 0; --ch) {
    if (longrows && first && ch && __ballot(!past && rd >= ch * KW) == 0ull) {
      if (part >= 0) return false;
      continue;
    }
    const int c0 = ch * KW + (KW / 4) * g;
    const __attribute__((address_space(1))) u32x4* src =
        (const __attribute__((address_space(1))) u32x4*)(gmem(rows) + (size_t)row * lp + c0);
    uint32_t pl[4][NQ];
#pragma unroll
    for (int h = 0; h < NQ; ++h) {
      u32x4 v = src[h];
      if (past || c0 + 4 * h >= lp) v = (u32x4){0u, 0u, 0u, 0u};
      const u32x4 t = byte_planes(v.x, v.y, v.z, v.w);
#pragma unroll
      for (int s = 0; s < 4; ++s) pl[s][h] = t[s];
    }
    typename OP::T a[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) a[s] = OP::pack(pl[s]);
    int32_t w16 = 65536;  // (opaque: as a constant it becomes 64-bit shifts and additions)
    asm("" : "+s"(w16));
    int32_t u[4][4];  // [point tile][register]
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      typename OP::T b[4];
#pragma unroll
      for (int s = 0; s < 4; ++s)
        b[s] = *(const typename OP::T*)(E.planes + s * 64 * KW + (16 * t + rho) * KW + (KW / 4) * g);
      im_v4i G[7];
#pragma unroll
      for (int c = 0; c < 7; ++c) G[c] = (im_v4i){0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int r = 0; r < 4; ++r) G[s + r] = OP::mma(a[s], b[r], G[s + r]);
      // sum_c G_c 256^c: |G_c| <= 64 (4 * 2^14) = 2^22 and less in the outer
      // classes, so the pairs G_c + 2^8 G_{c+1} fit in int32, and the sum with the
      // balanced weights of 2^32 and 2^48 stays below 2^59
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (live >> j & 1) {
          const SModP q = own_mod(q0);
          const int32_t A = G[0][j] + (G[1][j] << 8), B = G[2][j] + (G[3][j] << 8), Cc = G[4][j] + (G[5][j] << 8);
          // (no inline assembly on the accumulators: the compiler counts the wait
          // states between a matrix product and a reader of its result only
          // for instructions it knows)
          const int64_t s = mad_s(G[6][j], E.w48, mad_s(Cc, E.w32, mad_s(B, w16, A)));
          u[t][j] = redc_s(s, q);
        } else {
          u[t][j] = 0;
        }
      }
    }
    const SModP q = own_mod(q0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      // lane row g' receives from the tile of its own points
      typedef uint32_t u2 __attribute__((ext_vector_type(2)));
      const u2 s02 = __builtin_amdgcn_permlane32_swap((uint32_t)u[0][j], (uint32_t)u[2][j], false, false);
      const u2 s13 = __builtin_amdgcn_permlane32_swap((uint32_t)u[1][j], (uint32_t)u[3][j], false, false);
      const u2 lo = __builtin_amdgcn_permlane16_swap(s02.x, s13.x, false, false);
      const u2 hi = __builtin_amdgcn_permlane16_swap(s02.y, s13.y, false, false);
      const int32_t v[4] = {(int32_t)lo.x, (int32_t)lo.y, (int32_t)hi.x, (int32_t)hi.y};
#pragma unroll
      for (int r = 0; r < 4; ++r)
        out[4 * j + r] = part >= 0 || first ? v[r] : sdot2(out[4 * j + r], E.apw, v[r], E.one, q);
    }
    if (part >= 0) break;
    first = false;
  }
  return true;
}

// f(0), ..., f(N - 1) with compile-time indices: the register arrays are only
// indexed by constants from the front end on (a loop around an unrolled loop
// over them is unrolled too late for that, and they become vectors that move
// as a whole).
#define EE_IDX(i) [&](auto i) __attribute__((always_inline))
template <class F, int... I>
__device__ __forceinline__ void sfor_seq(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void sfor(F f) {
  sfor_seq(f, std::make_integer_sequence<int, N>{});
}

// (by value: a conditional between array elements would be one between their
// addresses)
__device__ __forceinline__ int32_t sel(bool c, int32_t a, int32_t b) { return c ? a : b; }

// A copy in a register of its own (the transposes return register pairs, whose
// tuples the allocator would otherwise extend over the arrays).
__device__ __forceinline__ int32_t own_reg(int32_t x) {
  int32_t r;
  asm("v_mov_b32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

#define EE_A(k) (AX ? X[k] : Y[k])
#define EE_B(k) (AX ? Y[k] : X[k])
#define EE_SET(k, v) \
  do {               \
    if (AX)          \
      X[k] = (v);    \
    else             \
      Y[k] = (v);    \
  } while (0)

// Makes element k opaque: the sign extensions of its value as a factor are then
// local to the block that follows.  (Shared between blocks they are kept as 64-bit
// register pairs.)
#define EE_OWN(k)             \
  do {                        \
    asm("" : "+v"(X[k]));     \
    asm("" : "+v"(Y[k]));     \
  } while (0)

// The multipliers of a normal step (A of degree deg B + 1): R = l2 A + (l1 y +
// n2) B.  a0, lb: the balanced leading coefficients.
struct SStep {
  int32_t l2, l1, n2;
};
template <int C, bool AX>
__device__ __forceinline__ SStep ee_consts(const int32_t (&X)[C], const int32_t (&Y)[C], int32_t a0, int32_t lb,
                                           const SModP& q) {
  SStep c;
  const int32_t na = -a0;
  c.n2 = balance(sdot2(a0, EE_B(1), -lb, EE_A(1), q), q.p);
  c.l2 = smul(lb, lb, q);
  c.l1 = smul(lb, na, q);
  return c;
}

// The step for the degree B of the divisor known at compile time.
template <int C, int B, bool AX>
__device__ __forceinline__ int32_t ee_step(int32_t (&X)[C], int32_t (&Y)[C], int32_t a0, int32_t lb, const SModP& q0) {
  static_assert(B >= 1 && B + 1 < C, "A of degree B + 1 must fit");
  __builtin_amdgcn_sched_barrier(0);
  const SModP q = own_mod(q0);
  sfor<B + 2>(EE_IDX(k) { EE_OWN(k); });
  const SStep c = ee_consts<C, AX>(X, Y, a0, lb, q);
  sfor<B - 1>(EE_IDX(k) { EE_SET(k, sdot3<AX>(c.l2, EE_A(k + 2), c.l1, EE_B(k + 2), c.n2, EE_B(k + 1), q)); });
  EE_SET(B - 1, sdot2<AX>(c.l2, EE_A(B + 1), c.n2, EE_B(B), q));
  return c.l2;
}

// The 4-blocks below index n as a mask (opaque: comparisons with n would be seen
// to imply each other, and the guarded blocks would no longer be updates in place).
__device__ __forceinline__ uint32_t block_mask(int n, uint32_t without = 0u) {
  uint32_t m = ((1u << ((n + 3) >> 2)) - 1u) & ~without;
  asm("" : "+s"(m));
  return m;
}

// The same with the degree bs > CH at run time, in guarded blocks of four: the
// arrays hold zeros past their degrees, and the blocks up to index bs + 1 run,
// which leaves zeros past the remainder's.
template <int C, int CH, bool AX>
__device__ __forceinline__ int32_t ee_step_any(int32_t (&X)[C], int32_t (&Y)[C], int bs, int32_t a0, int32_t lb,
                                               const SModP& q0) {
  static_assert(C % 4 == 0, "blocks of four");
  const uint32_t msk = block_mask(bs + 2);
  EE_OWN(1);
  const SStep c = ee_consts<C, AX>(X, Y, a0, lb, own_mod(q0));
  sfor<C / 4>(EE_IDX(blk) {
    constexpr int k0 = 4 * blk;
    if (k0 < CH + 3 || (msk >> blk & 1u)) {
      __builtin_amdgcn_sched_barrier(0);
      const SModP q = own_mod(q0);
      sfor<6>(EE_IDX(i) {
        if constexpr (k0 + i < C) EE_OWN(k0 + i);
      });
      sfor<4>(EE_IDX(i) {
        constexpr int k = k0 + i;
        if constexpr (k + 2 < C)
          EE_SET(k, sdot3<false>(c.l2, EE_A(k + 2), c.l1, EE_B(k + 2), c.n2, EE_B(k + 1), q));
        else if constexpr (k + 1 < C)
          EE_SET(k, sdot2<false>(c.n2, EE_B(k + 1), 0, 0, q));
        else
          EE_SET(k, 0);
      });
    }
  });
  return c.l2;
}

// One elimination of A by B (degree bs): A[j] <- x A[j+1] + y B[j+1] in the
// blocks of four that reach below index bs, shifted above.  B holds zeros past
// its degree, so past bs a block gives x A[j+1]: the same residue for x = 1,
// and A's zeros when the degrees are equal.
template <int C, bool AX>
__device__ __forceinline__ void ee_elim(int32_t (&X)[C], int32_t (&Y)[C], int ap, int bs, int32_t x, int32_t y,
                                        const SModP& q0) {
  const uint32_t msk = block_mask(bs), mska = block_mask(ap + 1, msk);
  sfor<C / 4>(EE_IDX(blk) {
    constexpr int j0 = 4 * blk;
    if (msk >> blk & 1u) {
      __builtin_amdgcn_sched_barrier(0);
      const SModP q = own_mod(q0);
      sfor<5>(EE_IDX(i) {
        if constexpr (j0 + i < C) EE_OWN(j0 + i);
      });
      sfor<4>(EE_IDX(i) {
        constexpr int j = j0 + i;
        if constexpr (j + 1 < C)
          EE_SET(j, sdot2<false>(x, EE_A(j + 1), y, EE_B(j + 1), q));
        else
          EE_SET(j, 0);
      });
    }
    if (mska >> blk & 1u) {
      sfor<4>(EE_IDX(i) {
        constexpr int j = j0 + i;
        if constexpr (j + 1 < C)
          EE_SET(j, EE_A(j + 1));
        else
          EE_SET(j, 0);
      });
    }
  });
}

// Two division steps by the monic multiple of B at once: A[j] <- A[j+2] +
// y1 B[j+2] + y0 B[j+1], five instructions per coefficient instead of eight and
// one shift instead of two (the pairs of 400 curves of degrees 4 to 30: 8840 ->
// 8620 us).  |y1|, |y0| <= 0.76 p keep the values below 1.3 p, within the bounds of the
// steps that follow.  Past bs the coefficients only shift, past A's degree ap they
// are zeros.
template <int C, bool AX>
__device__ __forceinline__ void ee_elim2(int32_t (&X)[C], int32_t (&Y)[C], int ap, int bs, int32_t ninv, int32_t one,
                                         const SModP& q0) {
  const uint32_t msk = block_mask(bs), mska = block_mask(ap + 1, msk);
  EE_OWN(0);
  EE_OWN(1);
  const int32_t y1 = smul(EE_A(0), ninv, q0);
  const int32_t y0 = smul(sdot2(one, EE_A(1), y1, EE_B(1), q0), ninv, q0);
  sfor<C / 4>(EE_IDX(blk) {
    constexpr int j0 = 4 * blk;
    if (msk >> blk & 1u) {
      __builtin_amdgcn_sched_barrier(0);
      const SModP q = own_mod(q0);
      sfor<6>(EE_IDX(i) {
        if constexpr (j0 + i < C) EE_OWN(j0 + i);
      });
      sfor<4>(EE_IDX(i) {
        constexpr int j = j0 + i;
        if constexpr (j + 2 < C)
          EE_SET(j, sdot3<false>(one, EE_A(j + 2), y1, EE_B(j + 2), y0, EE_B(j + 1), q));
        else if constexpr (j + 1 < C)
          EE_SET(j, smul(y0, EE_B(j + 1), q));
        else
          EE_SET(j, 0);
      });
    }
    if (mska >> blk & 1u) {
      sfor<4>(EE_IDX(i) {
        constexpr int j = j0 + i;
        if constexpr (j + 2 < C)
          EE_SET(j, EE_A(j + 2));
        else
          EE_SET(j, 0);
      });
    }
  });
}

// The first step of a pair whose degrees do not differ by one.  Equal degrees:
// one elimination with the multipliers of eliminate(), whose factor lc(B)
// goes to the bookkeeping.  A gap: exact division steps with 1 / lc(B), which
// leave A mod B itself, in pairs; the coefficients an elimination does not touch
// are only shifted instead of scaled.
template <int C, bool AX>
__device__ __forceinline__ void ee_first(int32_t (&X)[C], int32_t (&Y)[C], int as, int bs, int32_t lb, int32_t one,
                                         const SModP& q) {
  const bool eq = as == bs;
  // equal degrees: x = lb, y = -A[0] (a product with the Montgomery one)
  const int32_t x = eq ? lb : one;
  const int32_t ninv = eq ? -one : -spow(lb, q.p - 2u, q);
  int ap = as;
#pragma unroll 1
  for (; ap > bs; ap -= 2) ee_elim2<C, AX>(X, Y, ap, bs, ninv, one, q);
  if (ap == bs) ee_elim<C, AX>(X, Y, bs, bs, x, smul(EE_A(0), ninv, q), q);
}

#undef EE_A
#undef EE_B
#undef EE_SET
#undef EE_OWN

// The normal remainder sequence from a divisor of degree bs >= 1 down to a
// constant remainder, which is left in Y[0].  A is X at even degrees of the divisor;
// a0: A's balanced leading coefficient.  post(bs, l2, lead) is called after
// every step with the divisor's degree and the remainder's leading coefficient.
// Returns false (on every lane) when a divisor's leading coefficient vanishes at
// the point of one of the lanes `live`.
#define EE_CHAIN_STEP(BV)                                                  \
  if constexpr (BV <= CH && BV + 1 < C) {                                  \
    if (bs >= BV) {                                                        \
      const int32_t lb = balance(((BV) & 1) ? X[0] : Y[0], q.p);           \
      if ((__ballot(lb == 0) & live) != 0ull) return false;                \
      const int32_t l2 = ee_step<C, BV, ((BV) & 1) == 0>(X, Y, a0, lb, q); \
      a0 = lb;                                                             \
      post(BV, l2, ((BV) & 1) ? Y[0] : X[0]);                              \
    }                                                                      \
  }
#define EE_ANY_STEP(AX)                                             \
  {                                                                 \
    const int32_t lb = balance(AX ? Y[0] : X[0], q.p);              \
    if ((__ballot(lb == 0) & live) != 0ull) return false;           \
    const int32_t l2 = ee_step_any<C, CH, AX>(X, Y, bs, a0, lb, q); \
    a0 = lb;                                                        \
    post(bs, l2, AX ? X[0] : Y[0]);                                 \
    bs -= 1;                                                        \
  }
template <int C, int CH, class F>
__device__ __forceinline__ bool ee_chain(int32_t (&X)[C], int32_t (&Y)[C], int bs, int32_t a0, uint64_t live, const SModP& q, F post) {
  if constexpr (C > CH) {
    // pairs of an even and an odd step; an odd start skips the first even one
    // (conditional updates in place, not the two arms of a branch that merge)
    int skip = bs & 1;
    while (bs > CH) {
      asm("" : "+s"(skip));
      if (!skip) EE_ANY_STEP(true)
      skip = 0;
      EE_ANY_STEP(false)
    }
  }
  EE_CHAIN_STEP(30) EE_CHAIN_STEP(29) EE_CHAIN_STEP(28) EE_CHAIN_STEP(27) EE_CHAIN_STEP(26) EE_CHAIN_STEP(25)
  EE_CHAIN_STEP(24) EE_CHAIN_STEP(23) EE_CHAIN_STEP(22) EE_CHAIN_STEP(21) EE_CHAIN_STEP(20) EE_CHAIN_STEP(19)
  EE_CHAIN_STEP(18) EE_CHAIN_STEP(17) EE_CHAIN_STEP(16) EE_CHAIN_STEP(15) EE_CHAIN_STEP(14) EE_CHAIN_STEP(13)
  EE_CHAIN_STEP(12) EE_CHAIN_STEP(11) EE_CHAIN_STEP(10) EE_CHAIN_STEP(9) EE_CHAIN_STEP(8) EE_CHAIN_STEP(7)
  EE_CHAIN_STEP(6) EE_CHAIN_STEP(5) EE_CHAIN_STEP(4) EE_CHAIN_STEP(3) EE_CHAIN_STEP(2) EE_CHAIN_STEP(1)
  return true;
}
#undef EE_CHAIN_STEP
#undef EE_ANY_STEP

// Digit planes [4][64][KW] of the powers 0..KW-1 of the lanes' points a1 (four
// chains); returns a^KW.
template <int KW>
__device__ __forceinline__ int32_t power_planes(int32_t a1, int32_t one, int8_t* planes, const SModP& q) {
  int32_t w[4];
  w[0] = one;
  w[1] = a1;
  w[2] = smul(a1, a1, q);
  w[3] = smul(w[2], a1, q);
  const int32_t a4 = smul(w[2], w[2], q);
#pragma unroll
  for (int h = 0; h < KW / 16; ++h) {
    u32x4 pl[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      uint32_t d[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        d[j] = sdigits(w[j]);
        w[j] = smul(w[j], a4, q);
      }
      const u32x4 t = byte_planes(d[0], d[1], d[2], d[3]);
#pragma unroll
      for (int s = 0; s < 4; ++s) pl[s][c] = t[s];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) *(u32x4*)(planes + s * 64 * KW + lane_id() * KW + 16 * h) = pl[s];
  }
  return w[0];
}

// The values of f and g at the block's points: of f in X if xf, else in Y.
// (The powers need no end at the rows': the rows' digits are zero past it.)
template <int C, int KW>
__device__ __forceinline__ void ee_eval(const JobDev& J, int k, int blk, TablesDev tab, int8_t* planes, bool xf,
                                        EvalCtx& E, int32_t (&X)[C], int32_t (&Y)[C], const SModP& q) {
  E.planes = planes;
  E.dmax = max(J.ldf, J.kind ? J.ldf : J.ldg) - 1;
  E.one = balance((int32_t)q.one, q.p);
  E.w32 = E.one;
  E.w48 = balance((int32_t)to_mont(65536u, q), q.p);
  E.apw = 0;
  if (KW == 32 && tab.pow_planes) {
    const int8_t* src = tab.pow_planes + ((size_t)k * tab.pow_nb + blk) * (4 * 64 * 32);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      ((u32x4*)planes)[64 * i + lane_id()] =
          ((const __attribute__((address_space(1))) u32x4*)gmem(src))[64 * i + lane_id()];
    if (E.dmax >= KW) {
      int32_t a = balance((int32_t)eval_point(tab, k, min(blk * 64 + lane_id(), J.D - 1), q), q.p);
#pragma unroll 1
      for (int i = 1; i < KW; i <<= 1) a = smul(a, a, q);
      E.apw = balance(a, q.p);
    }
  } else {
    const int32_t a1 = balance((int32_t)eval_point(tab, k, min(blk * 64 + lane_id(), J.D - 1), q), q.p);
    E.apw = balance(power_planes<KW>(a1, E.one, planes, q), q.p);
  }
  // (opaque: otherwise everything that follows is compiled once per case of the
  // branches above)
  asm("" : "+s"(E.dmax), "+v"(E.apw));
  group_sync<true>();
  Rows x, y;
  {
    const Rows f{J.res_f + (size_t)k * J.Tf, J.rowdeg_f, J.lpf, J.m};
    const Rows g{J.res_g + (size_t)k * J.Tg, J.rowdeg_g, J.lpg, J.n};
    x = xf ? f : g;
    y = xf ? g : f;
  }
  // One copy of the tile code for all tiles (unrolled it would overflow the
  // instruction cache); each tile's values are moved to their registers behind
  // a scalar branch.  The rows past the whole tiles share one.
  constexpr int T = C / 16, RJ = (C % 16) / 4;
  static_assert(C % 16 <= 8 && C % 4 == 0, "the rest of both arrays fits one tile");
  sfor<C>(EE_IDX(i) { X[i] = Y[i] = own_reg(0); });  // (opaque zeros: a fill would keep the array whole)
  // At capacity 24 the pieces of longer rows are the outer loop and join in the
  // arrays themselves: a tile's values need not be kept over its matrix products,
  // which fits the kernel into its 128 registers without scratch.  (The others have
  // registers to spare, and their code should not grow.)
  constexpr bool OUTER = C == 24;
  const int top = OUTER && E.dmax >= KW ? E.dmax / KW : 0;
  auto join = [&](int32_t& z, int32_t v, bool add) __attribute__((always_inline)) {
    if (OUTER && add)
      z = sdot2(z, E.apw, v, E.one, own_mod(q));
    else
      z = own_reg(v);
  };
#pragma unroll 1
  for (int part = top; part >= 0; --part)
#pragma unroll 1
  for (int id = 0; id < 2 * T + (RJ ? 1 : 0); ++id) {
    const int which = id == 2 * T ? 2 : id >= T ? 1 : 0, tau = which == 2 ? T : which ? id - T : id;
    if (16 * tau > (which == 0 ? x.deg : which == 1 ? y.deg : max(x.deg, y.deg))) continue;
    int32_t o[16];
    if (!eval_tile<KW, RJ ? RJ : 1>(x, y, which, 16 * tau, OUTER ? part : -1, E, o, q)) continue;
    const bool add = OUTER && part < top;
    sfor<T>(EE_IDX(t) {
      if (id == t) sfor<16>(EE_IDX(i) { join(X[16 * t + i], o[i], add); });
      if (id == T + t) sfor<16>(EE_IDX(i) { join(Y[16 * t + i], o[i], add); });
    });
    if constexpr (RJ > 0) {
      if (id == 2 * T) {
        sfor<4 * RJ>(EE_IDX(i) { join(X[16 * T + i], o[i], add); });
        sfor<4 * RJ>(EE_IDX(i) { join(Y[16 * T + i], o[4 * RJ + i], add); });
      }
    }
  }
}

// The lanes of block blk that hold one of the D points.  The others, in the last
// block, compute something of no consequence (with stored powers the powers of
// the next nodes, but a^KW of point D - 1) and must not send the block to the
// general kernel.
__device__ __forceinline__ uint64_t live_lanes(int D, int blk) { return ~0ull >> (64 - min(64, D - 64 * blk)); }

// Returns false (on every lane) when the block must be recomputed by
// dev_eval_elim: a leading coefficient vanishes at some lane's point, or a
// remainder is shorter than a normal sequence's.  Needs 1 <= m, n < C.
template <int C, int CH, int KW>
__device__ __forceinline__ bool dev_ee(const JobDev& J, int lb_, TablesDev tab, int8_t* planes) {
  const int nbpp = (J.D + 63) / 64;
  const int k = lb_ / nbpp;
  const int blk = lb_ - k * nbpp, pt = blk * 64 + lane_id();
  const int m = J.m, n = J.n;
  const SModP q(tab.primes[k]);
  // the operand of larger degree (A) and the other; which register array
  // holds A: at the start of the chain A is X when the divisor's degree is even
  const bool sw = m < n;
  const int as0 = sw ? n : m, bs0 = sw ? m : n;
  const bool normal = as0 == bs0 + 1;
  const bool ax = normal ? (bs0 & 1) == 0 : ((bs0 - 1) & 1) != 0;
  const bool xf = ax != sw;  // X holds f
  const uint64_t live = live_lanes(J.D, blk);
  EvalCtx E;
  int32_t X[C], Y[C];
  ee_eval<C, KW>(J, k, blk, tab, planes, xf, E, X, Y, q);
  int as = as0, bs = bs0;
  bool neg = sw && ((m * n) & 1);
  int32_t num = E.one, den = E.one, pfx = E.one;
  int32_t a0 = balance(sel(ax, X[0], Y[0]), q.p);
  {
    const int32_t b0 = balance(sel(ax, Y[0], X[0]), q.p);
    if ((__ballot(a0 == 0 || b0 == 0) & live) != 0ull) return false;
    if (!normal) {
      int fx = ax, fy = !ax;
      asm("" : "+s"(fx), "+s"(fy));
      if (fx) ee_first<C, true>(X, Y, as, bs, b0, E.one, q);
      if (fy) ee_first<C, false>(X, Y, as, bs, b0, E.one, q);
      neg ^= ((as * bs) & 1) != 0;
      if (as == bs) {
        // uni_resultant's bookkeeping: lc(B)^(1 - b) = lc(B)^(-2(b-1) + (b-1))
        pfx = smul(b0, b0, q);
        if (bs > 1) {
          den = pfx;
          num = spow(b0, (uint32_t)(bs - 1), q);
        }
      } else {
        num = spow(b0, (uint32_t)(as - bs + 1), q);  // res(A, B) = (-1)^(ab) lc(B)^(a - c) res(B, A mod B)
      }
      a0 = b0;
      as = bs;
      bs -= 1;
    }
  }
  if (!ee_chain<C, CH>(X, Y, bs, a0, live, q, [&](int b, int32_t l2, int32_t) __attribute__((always_inline)) {
        pfx = smul(pfx, l2, q);
        if (b > 1) den = smul(den, pfx, q);
      }))
    return false;
  // the constant remainder: degree 0 is even, so A (degree 1) is X and it is in Y
  const int32_t last = balance(Y[0], q.p);
  if ((__ballot(last == 0) & live) != 0ull) return false;
  num = smul(num, last, q);
  int32_t r = smul(num, spow(balance(den, q.p), q.p - 2u, q), q);
  if (neg) r = -r;
  r = redc_s((int64_t)r, q);  // plain residue, |r| <= p / 2 + 1
  const uint32_t v = (uint32_t)r;
  if (pt < J.D) put_value(J, k, pt, umin32(v, v + q.p), q.p);
  return true;
}

template <int C, int CH, int KW>
__device__ __forceinline__ void ee_block(const JobDev* jobs, const int* starts, int nj, TablesDev tab, int* fb_count,
                                         int* fb_queue, int8_t* lds) {
  const int b = xcd_block(blockIdx.x, gridDim.x);
  const int job = find_job(starts, nj, b, gridDim.x);
  const bool ok = dev_ee<C, CH, KW>(jobs[job], b - starts[job], tab, lds);
  if (!ok && threadIdx.x == 0) fb_queue[atomicAdd(fb_count, 1)] = b;
}

// Powers of the evaluation points in operand form, for the kernels of 32 powers
// (blocks of 64 points, primes): they depend on the nodes only, and eight loads
// replace 300 instructions of 3760 (256 pairs of degree 20, with the shared last
// tile and the shorter epilogue: 650 -> 600 us).
__global__ __launch_bounds__(64) void k_pow_planes(TablesDev tab, int nb, int8_t* out) {
  __shared__ __align__(16) int8_t planes[4 * 64 * 32];
  const int blk = blockIdx.x, k = blockIdx.y;
  const SModP q(tab.primes[k]);
  const int32_t a1 = balance((int32_t)eval_point(tab, k, blk * 64 + lane_id(), q), q.p);
  (void)power_planes<32>(a1, balance((int32_t)q.one, q.p), planes, q);
  group_sync<true>();
  u32x4* dst = (u32x4*)(out + ((size_t)k * nb + blk) * (4 * 64 * 32));
#pragma unroll
  for (int i = 0; i < 8; ++i) dst[64 * i + lane_id()] = ((const u32x4*)planes)[64 * i + lane_id()];
}

}  // namespace

size_t pow_planes_bytes(int nb, int P) { return (size_t)nb * P * (4 * 64 * 32); }

void launch_pow_planes(TablesDev tab, int nb, int P, int8_t* out, hipStream_t s) {
  hipLaunchKernelGGL(k_pow_planes, dim3(nb, P), dim3(64), 0, s, tab, nb, out);
}

#define BIRES_EE_KERNEL(C, CH, KW, WAVES)                                                                          \
  __global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WAVES, 8))) void k_eval_elim_ee##C(          \
      const JobDev* jobs, const int* starts, int nj, TablesDev tab, int* fb_count, int* fb_queue) {                \
    __shared__ __align__(16) int8_t planes[4 * 64 * KW];                                                           \
    ee_block<C, CH, KW>(jobs, starts, nj, tab, fb_count, fb_queue, planes);                                            \
  }
// Waves per SIMD and CH, the largest divisor degree of the unrolled chain
// (above it guarded blocks of four in a loop, which compute up to five
// coefficients more per step but are one copy of the code):
//   24: 128 registers, 4 waves;  32: 144, 3 waves (4 waves spill: 8.2 against
//   7.4 ms below);  48: 190 and 68: 230, 2 waves.
//   CH 30 is the whole chain of 24 and 32 (CH 14: 664 against 651 us).  68 with
//   CH 30 has 64 KB of code, the whole instruction cache, and takes 1.7 times
//   as long as with 14; 22 (46 KB) is another 2% faster than 14.
// Against the kernels with one array in LDS and unsigned arithmetic (us):
//   24  256 pairs of degree 20, 48 primes, 401 points    667 -> 600
//   32  45 pairs of degree 31 curves                   10965 -> 7370
//   48  one discriminant of degree 40                     99 -> 52
//   68  one pair of degree 64 (general kernel before)   7148 -> 1730
//   48 + 68  64 pairs of degrees 33 to 64              14432 -> 6600
// All are bound by VALU issue (4.65 cycles per multiply-add, five per
// coefficient and step); at degree 20 the evaluation is a third of the
// instructions.
BIRES_EE_KERNEL(24, 30, 32, 4)
BIRES_EE_KERNEL(32, 30, 32, 3)
BIRES_EE_KERNEL(48, 22, 64, 2)
BIRES_EE_KERNEL(68, 22, 64, 2)

// Principal subresultant coefficients sr_i(a), i < K, of degrees that differ by at
// most one: psc_lane's recurrence along the normal sequence, whose steps all
// multiply by lc(B)^2 = l2 (equal degrees: a first one by lc(B)).  nm, dn: LDS [K][64]
// numerators and denominators of the block's points, inverted together at
// the end.  Returns false when a formal or actual leading coefficient vanishes
// at some lane's point (the general kernel then does the block).
template <int C, int CH, int KW>
__device__ __forceinline__ bool dev_psc(const JobDev& J, int blk, TablesDev tab, int8_t* planes, int32_t* nm,
                                        int32_t* dn, uint32_t* out, int K) {
  const int l = lane_id(), pt = blk * 64 + l;
  const int m = J.m, n = J.n;
  const SModP q(tab.primes[0]);
  const bool sw = m < n, eq = m == n;
  const int bs0 = sw ? m : n;
  const bool ax = eq ? ((bs0 - 1) & 1) != 0 : (bs0 & 1) == 0;
  const uint64_t live = live_lanes(J.D, blk);
  EvalCtx E;
  int32_t X[C], Y[C];
  ee_eval<C, KW>(J, 0, blk, tab, planes, ax != sw, E, X, Y, q);
  int32_t a0 = balance(sel(ax, X[0], Y[0]), q.p);
  const int32_t b0 = balance(sel(ax, Y[0], X[0]), q.p);
  if ((__ballot(a0 == 0 || b0 == 0) & live) != 0ull) return false;
  int E0 = sw ? (m * n) & 1 : 0, E1 = sw ? (m + n + 1) & 1 : 0;
  int32_t Nn = E.one, Nd = E.one, sA = E.one, sB = E.one;
  auto emit = [&](int i, int32_t vn, int32_t vd) __attribute__((always_inline)) {
    if (i >= K) return;
    const int32_t x = smul(Nn, vn, q);
    nm[i * 64 + l] = ((E0 ^ (i & E1)) & 1) ? -x : x;
    dn[i * 64 + l] = smul(Nd, vd, q);
  };
  int bs = bs0;
  if (eq) {
    int fx = ax, fy = !ax;
    asm("" : "+s"(fx), "+s"(fy));
    if (fx) ee_first<C, true>(X, Y, bs, bs, b0, E.one, q);
    if (fy) ee_first<C, false>(X, Y, bs, bs, b0, E.one, q);
    E0 ^= bs & 1;
    E1 ^= 1;
    Nn = b0;
    emit(bs - 1, sel(ax, X[0], Y[0]), b0);
    sB = b0;
    a0 = b0;
    bs -= 1;
  } else if (bs0 < K) {
    nm[bs0 * 64 + l] = b0;  // lc(B)^(a - b)
    dn[bs0 * 64 + l] = E.one;
  }
  if (!ee_chain<C, CH>(X, Y, bs, a0, live, q, [&](int b, int32_t l2, int32_t lead) __attribute__((always_inline)) {
        Nn = smul(Nn, l2, q);
        Nd = smul(smul(Nd, sB, q), sB, q);
        const int32_t sR = smul(l2, sA, q);
        emit(b - 1, lead, sR);
        sA = sB;
        sB = sR;
      }))
    return false;
  int32_t pre = E.one;
#pragma unroll 4
  for (int i = 0; i < K; ++i) {
    nm[i * 64 + l] = smul(nm[i * 64 + l], pre, q);
    pre = smul(pre, dn[i * 64 + l], q);
  }
  int32_t inv = spow(balance(pre, q.p), q.p - 2u, q);
#pragma unroll 4
  for (int i = K - 1; i >= 0; --i) {
    const int32_t r = redc_s((int64_t)smul(nm[i * 64 + l], inv, q), q);
    inv = smul(inv, dn[i * 64 + l], q);
    if (pt < J.D) out[(size_t)i * J.D + pt] = umin32((uint32_t)r, (uint32_t)r + q.p);
  }
  return true;
}

// One wave per 64 points: a run has few blocks (25 at 1561 points), so latency
// counts, and registers serve it better than arrays in LDS (k_psc): 146 -> 42 us
// for the 40 indices of a degree-40 curve and its derivative.  One capacity: at a
// wave per CU the zeros of a smaller job cost less than more code would.
constexpr int PSC_CAPACITY = 68;
__global__ __launch_bounds__(64) void k_psc_ee(JobDev J, TablesDev tab, uint32_t* out, int K, int* fallback) {
  __shared__ __align__(16) int8_t planes[4 * 64 * 64];
  __shared__ int32_t nm[PSC_CAPACITY * 64], dn[PSC_CAPACITY * 64];
  const bool ok = dev_psc<PSC_CAPACITY, 22, 64>(J, blockIdx.x, tab, planes, nm, dn, out, K);
  if (threadIdx.x == 0) fallback[blockIdx.x] = !ok;
}

// Degrees that differ by at most one are the discriminant's and Q's; a larger gap
// would need the powers of psc_lane.
bool psc_registers(int m, int n) {
  return std::min(m, n) >= 1 && std::max(m, n) < PSC_CAPACITY && std::abs(m - n) <= 1;
}

void launch_psc_ee(const JobDev& J, TablesDev tab, uint32_t* out, int K, int* fallback, hipStream_t s) {
  hipLaunchKernelGGL(k_psc_ee, dim3((J.D + 63) / 64), dim3(64), 0, s, J, tab, out, K, fallback);
}

// The smallest capacity that holds both arrays: fewer registers per lane, more
// waves (degree 22 in the kernel of capacity 32: 3 waves instead of 4).  From 68
// on the arrays no longer fit beside the evaluation in the 256 registers of 2
// waves, and the general kernel takes the job.
int eval_elim_rg_capacity(int m, int n) {
  if (m < 1 || n < 1) return 0;
  const int d = std::max(m, n);
  return d < 24 ? 24 : d < 32 ? 32 : d < 48 ? 48 : d < 68 ? 68 : 0;
}

// Jobs that the general kernel does faster than capacity 24, by degree d, row length
// and the call's size: an instance costs it what d and the row (in pieces of 24
// coefficients) ask for, while ee24 evaluates 16 rows at 64 points whatever they
// are, a second time from 33 coefficients on, and has its recomputing launch
// behind it.  Below a block per SIMD the latency of the two counts, ee24's being
// the same for all d, above it the instructions.  Evaluation in us, general and
// ee24 (m = n = d, coefficients of 20 to 40 bits):
//   2000 pairs, rows of 4   d = 1 14, 28   d = 2 23, 39   d = 4 43, 60   d = 8 110, 129
//                                          d = 10 172, 163
//   300 pairs, rows of 21   d = 2 15, 18   d = 6 64, 66   d = 7 94, 89
//   300 pairs, rows of 25   d = 3 28, 30   d = 4 46, 44
//   300 pairs, rows of 33   d = 2 21, 37   d = 8 261, 279 d = 10 503, 434
//   1 pair, rows of 4       d = 1 7.7, 14.3  d = 4 13.1, 15.3  d = 7 16.2, 15.7
//   1 pair, rows of 12      d = 1 8.1, 14.3  d = 4 14.8, 15.2  d = 5 16.0, 15.5
bool eval_elim_light(int m, int n, int row, long long instances) {
  const int d = std::max(m, n);
  if (d * (row + 8) <= 80) return true;
  if (instances < 64 * 1024) return false;
  return d <= (row <= 16 ? 8 : row <= 24 ? 6 : row <= 32 ? 3 : row <= 48 ? 8 : 5);
}

void launch_eval_elim_rg(int C, const JobDev* jobs, const int* starts, int nj, int nblocks, int max_words,
                         int* fb_count, int* fb_queue, TablesDev tab, hipStream_t s) {
#define BIRES_EE_LAUNCH(N) \
  hipLaunchKernelGGL(k_eval_elim_ee##N, dim3(nblocks), dim3(64), 0, s, jobs, starts, nj, tab, fb_count, fb_queue)
  switch (C) {
    case 24: BIRES_EE_LAUNCH(24); break;
    case 32: BIRES_EE_LAUNCH(32); break;
    case 48: BIRES_EE_LAUNCH(48); break;
    default: BIRES_EE_LAUNCH(68); break;
  }
#undef BIRES_EE_LAUNCH
  // One block per CU costs an empty queue next to nothing.  At capacity 68 as many as
  // fit beside each other (34 KB of LDS each): a sequence that is not normal
  // queues every block, and the general kernel would have had them all at once
  // (20 pairs of degrees 64 and 62 in y, even: 36.6 ms with 256 blocks, 12.1
  // with 1024, 10.9 by the general kernel alone).
  const int fb_blocks = C == 68 ? 1024 : 256;
  launch_eval_elim_fb(jobs, starts, nj, nblocks, fb_blocks, max_words, fb_count, fb_queue, tab, s);
}

}  // namespace bires
