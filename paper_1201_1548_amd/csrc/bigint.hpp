// Minimal host big integers for the gcd's normalisation (contents, exact
// quotients, the gcd of leading coefficients).  Sign-magnitude, 32-bit limbs,
// little endian; the magnitude has no leading zero limbs (zero = empty).
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <vector>

namespace bires {

struct BigInt {
  bool neg = false;
  std::vector<uint32_t> mag;

  bool is_zero() const { return mag.empty(); }
  int bits() const;                                   // bit length of |x| (0 for zero)
  static BigInt from_twos(const uint32_t* limbs, int L);  // two's complement input
  void to_twos(uint32_t* limbs, int L) const;         // sign-extended; caller checks the size
  static BigInt from_u64(uint64_t v);
};

void trim(std::vector<uint32_t>& m);
int cmp_mag(const std::vector<uint32_t>& a, const std::vector<uint32_t>& b);
BigInt big_abs(const BigInt& a);
BigInt big_add(const BigInt& a, const BigInt& b);
void big_sub_from(BigInt& a, const BigInt& b);  // a -= b
BigInt big_mul(const BigInt& a, const BigInt& b);
// Quotient and remainder of |a| by |b| (b != 0), Knuth's algorithm D.
void divmod_mag(const std::vector<uint32_t>& a, const std::vector<uint32_t>& b, std::vector<uint32_t>& q,
                std::vector<uint32_t>& r);
// a / b for b dividing a exactly (signs handled); returns false if not exact.
bool big_divexact(const BigInt& a, const BigInt& b, BigInt& q);
// The same for one divisor b != 0 and many dividends, quotient limbs from the
// low end by b's inverse mod 2^64 (Hensel): a limb of the quotient costs b's
// length in 64-bit multiplications and no division.  A dividend of 2022 bits by
// 204 takes 0.15 us (algorithm D on 32-bit digits 0.76).
class ExactDiv {
 public:
  explicit ExactDiv(const BigInt& b);
  bool operator()(const BigInt& a, BigInt& q);  // false if b does not divide a (q is unspecified)
  bool one() const { return one_; }             // |b| = 1

 private:
  std::vector<uint64_t> d_, t_;  // odd part of |b|; what is left of the dividend
  uint64_t inv_ = 0;             // d_[0]^{-1} mod 2^64
  size_t zeros_ = 0;             // trailing zero limbs and bits of |b|
  int shift_ = 0;
  bool neg_, one_;
};
// gcd(|a|, |b|), Lehmer's algorithm (gcd(0, 0) = 0).
BigInt big_gcd(const BigInt& a, const BigInt& b);
uint32_t big_mod_small(const BigInt& a, uint32_t p);  // a mod p in [0, p)

}  // namespace bires
