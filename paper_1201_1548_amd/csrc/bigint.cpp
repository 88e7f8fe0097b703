// Host big-integer helpers (see bigint.hpp).  General division is Knuth's
// algorithm D (TAOCP vol. 2, 4.3.1) on 32-bit digits with 64-bit intermediates;
// exact division and the gcd run on 64-bit limbs.
#include "bigint.hpp"

#include <algorithm>

namespace bires {

void trim(std::vector<uint32_t>& m) {
  while (!m.empty() && m.back() == 0u) m.pop_back();
}

int BigInt::bits() const {
  if (mag.empty()) return 0;
  return 32 * ((int)mag.size() - 1) + (32 - __builtin_clz(mag.back()));
}

BigInt BigInt::from_twos(const uint32_t* limbs, int L) {
  BigInt r;
  const bool neg = (limbs[L - 1] >> 31) != 0u;
  r.mag.assign(limbs, limbs + L);
  if (neg) {  // magnitude = ~x + 1
    uint64_t carry = 1;
    for (auto& w : r.mag) {
      const uint64_t v = (uint64_t)(uint32_t)~w + carry;
      w = (uint32_t)v;
      carry = v >> 32;
    }
  }
  trim(r.mag);
  r.neg = neg && !r.mag.empty();
  return r;
}

void BigInt::to_twos(uint32_t* limbs, int L) const {
  for (int l = 0; l < L; ++l) limbs[l] = l < (int)mag.size() ? mag[l] : 0u;
  if (neg) {
    uint64_t carry = 1;
    for (int l = 0; l < L; ++l) {
      const uint64_t v = (uint64_t)(uint32_t)~limbs[l] + carry;
      limbs[l] = (uint32_t)v;
      carry = v >> 32;
    }
  }
}

BigInt BigInt::from_u64(uint64_t v) {
  BigInt r;
  while (v) {
    r.mag.push_back((uint32_t)v);
    v >>= 32;
  }
  return r;
}

int cmp_mag(const std::vector<uint32_t>& a, const std::vector<uint32_t>& b) {
  if (a.size() != b.size()) return a.size() < b.size() ? -1 : 1;
  for (size_t i = a.size(); i-- > 0;)
    if (a[i] != b[i]) return a[i] < b[i] ? -1 : 1;
  return 0;
}

BigInt big_abs(const BigInt& a) {
  BigInt r = a;
  r.neg = false;
  return r;
}

// |a| + |b| and |a| - |b| (|a| >= |b|) on magnitudes.
static std::vector<uint32_t> add_mag(const std::vector<uint32_t>& a, const std::vector<uint32_t>& b) {
  std::vector<uint32_t> r(std::max(a.size(), b.size()) + 1, 0u);
  uint64_t carry = 0;
  for (size_t i = 0; i + 1 < r.size(); ++i) {
    const uint64_t s = carry + (i < a.size() ? a[i] : 0u) + (i < b.size() ? b[i] : 0u);
    r[i] = (uint32_t)s;
    carry = s >> 32;
  }
  r.back() = (uint32_t)carry;
  trim(r);
  return r;
}

static std::vector<uint32_t> sub_mag(const std::vector<uint32_t>& a, const std::vector<uint32_t>& b) {
  std::vector<uint32_t> r(a.size(), 0u);
  int64_t borrow = 0;
  for (size_t i = 0; i < a.size(); ++i) {
    int64_t s = (int64_t)a[i] - (i < b.size() ? (int64_t)b[i] : 0) - borrow;
    borrow = s < 0 ? 1 : 0;
    r[i] = (uint32_t)(s + (borrow << 32));
  }
  trim(r);
  return r;
}

BigInt big_add(const BigInt& a, const BigInt& b) {
  BigInt r;
  if (a.neg == b.neg) {
    r.mag = add_mag(a.mag, b.mag);
    r.neg = a.neg;
  } else if (cmp_mag(a.mag, b.mag) >= 0) {
    r.mag = sub_mag(a.mag, b.mag);
    r.neg = a.neg;
  } else {
    r.mag = sub_mag(b.mag, a.mag);
    r.neg = b.neg;
  }
  if (r.mag.empty()) r.neg = false;
  return r;
}

void big_sub_from(BigInt& a, const BigInt& b) {
  if (b.is_zero()) return;
  if (a.is_zero() || a.neg == b.neg) {
    if (cmp_mag(a.mag, b.mag) >= 0) {
      a.mag = sub_mag(a.mag, b.mag);
      if (a.mag.empty()) a.neg = false;
    } else {
      a.mag = sub_mag(b.mag, a.mag);
      a.neg = !b.neg;
    }
  } else {
    a.mag = add_mag(a.mag, b.mag);
  }
}

BigInt big_mul(const BigInt& a, const BigInt& b) {
  BigInt r;
  if (a.is_zero() || b.is_zero()) return r;
  r.mag.assign(a.mag.size() + b.mag.size(), 0u);
  for (size_t i = 0; i < a.mag.size(); ++i) {
    uint64_t carry = 0;
    for (size_t j = 0; j < b.mag.size(); ++j) {
      const uint64_t t = (uint64_t)a.mag[i] * b.mag[j] + r.mag[i + j] + carry;
      r.mag[i + j] = (uint32_t)t;
      carry = t >> 32;
    }
    size_t k = i + b.mag.size();
    while (carry) {
      const uint64_t t = (uint64_t)r.mag[k] + carry;
      r.mag[k++] = (uint32_t)t;
      carry = t >> 32;
    }
  }
  trim(r.mag);
  r.neg = a.neg != b.neg;
  return r;
}

void divmod_mag(const std::vector<uint32_t>& a, const std::vector<uint32_t>& b, std::vector<uint32_t>& q,
                std::vector<uint32_t>& r) {
  q.clear();
  r.clear();
  if (cmp_mag(a, b) < 0) {
    r = a;
    return;
  }
  const size_t n = b.size(), m = a.size() - b.size();
  if (n == 1) {  // single-digit divisor
    q.assign(a.size(), 0u);
    uint64_t rem = 0;
    for (size_t i = a.size(); i-- > 0;) {
      const uint64_t cur = (rem << 32) | a[i];
      q[i] = (uint32_t)(cur / b[0]);
      rem = cur % b[0];
    }
    trim(q);
    if (rem) r.push_back((uint32_t)rem);
    return;
  }
  // D1: normalise so the divisor's top digit has its high bit set
  const int s = __builtin_clz(b.back());
  std::vector<uint32_t> v(n), u(a.size() + 1);
  for (size_t i = n; i-- > 0;) v[i] = (b[i] << s) | (s && i ? (uint32_t)(b[i - 1] >> (32 - s)) : 0u);
  u[a.size()] = s ? (uint32_t)(a.back() >> (32 - s)) : 0u;
  for (size_t i = a.size(); i-- > 0;) u[i] = (a[i] << s) | (s && i ? (uint32_t)(a[i - 1] >> (32 - s)) : 0u);
  q.assign(m + 1, 0u);
  const uint64_t B = 1ull << 32;
  for (size_t j = m + 1; j-- > 0;) {
    // D3: estimate qhat from the top two digits
    const uint64_t num = ((uint64_t)u[j + n] << 32) | u[j + n - 1];
    uint64_t qhat = num / v[n - 1];
    uint64_t rhat = num % v[n - 1];
    while (qhat >= B || qhat * v[n - 2] > ((rhat << 32) | u[j + n - 2])) {
      --qhat;
      rhat += v[n - 1];
      if (rhat >= B) break;
    }
    // D4: multiply and subtract
    int64_t borrow = 0;
    uint64_t carry = 0;
    for (size_t i = 0; i < n; ++i) {
      const uint64_t p = qhat * v[i] + carry;
      carry = p >> 32;
      const int64_t t = (int64_t)u[i + j] - (int64_t)(uint32_t)p + borrow;
      u[i + j] = (uint32_t)t;
      borrow = t >> 32;
    }
    const int64_t t = (int64_t)u[j + n] - (int64_t)carry + borrow;
    u[j + n] = (uint32_t)t;
    if (t < 0) {  // D6: add back
      --qhat;
      uint64_t c = 0;
      for (size_t i = 0; i < n; ++i) {
        const uint64_t s2 = (uint64_t)u[i + j] + v[i] + c;
        u[i + j] = (uint32_t)s2;
        c = s2 >> 32;
      }
      u[j + n] += (uint32_t)c;
    }
    q[j] = (uint32_t)qhat;
  }
  trim(q);
  // D8: unnormalise the remainder
  r.assign(n, 0u);
  for (size_t i = 0; i < n; ++i) r[i] = (u[i] >> s) | (s ? (uint32_t)((uint64_t)u[i + 1] << (32 - s)) : 0u);
  trim(r);
}

namespace {

typedef unsigned __int128 u128;
typedef __int128 s128;

// Magnitudes in 64-bit limbs, for the quadratic loops.
void to64(const std::vector<uint32_t>& m, std::vector<uint64_t>& w) {
  const size_t n = (m.size() + 1) / 2;
  w.resize(n);
  for (size_t i = 0; i < n; ++i)
    w[i] = m[2 * i] | (2 * i + 1 < m.size() ? (uint64_t)m[2 * i + 1] << 32 : 0);
}

void from64(const uint64_t* w, size_t n, std::vector<uint32_t>& m) {
  m.resize(2 * n);
  for (size_t i = 0; i < n; ++i) {
    m[2 * i] = (uint32_t)w[i];
    m[2 * i + 1] = (uint32_t)(w[i] >> 32);
  }
  trim(m);
}

void trim64(std::vector<uint64_t>& w) {
  while (!w.empty() && w.back() == 0) w.pop_back();
}

// w >> s, s < 64.
void shift_down(std::vector<uint64_t>& w, int s) {
  if (s)
    for (size_t i = 0; i < w.size(); ++i) w[i] = (w[i] >> s) | (i + 1 < w.size() ? w[i + 1] << (64 - s) : 0);
  trim64(w);
}

// The bits [at, at + 62) of w.
uint64_t window(const std::vector<uint64_t>& w, size_t at) {
  const size_t i = at / 64, s = at % 64;
  uint64_t v = i < w.size() ? w[i] >> s : 0;
  if (s && i + 1 < w.size()) v |= w[i + 1] << (64 - s);
  return v & (((uint64_t)1 << 62) - 1);
}

}  // namespace

ExactDiv::ExactDiv(const BigInt& b) : neg_(b.neg), one_(b.mag.size() == 1 && b.mag[0] == 1u) {
  to64(b.mag, d_);
  while (d_[zeros_] == 0) ++zeros_;
  d_.erase(d_.begin(), d_.begin() + zeros_);
  shift_ = __builtin_ctzll(d_[0]);
  shift_down(d_, shift_);
  inv_ = d_[0];  // Newton: right in 3 bits, doubled five times
  for (int i = 0; i < 5; ++i) inv_ *= 2 - d_[0] * inv_;
}

bool ExactDiv::operator()(const BigInt& a, BigInt& q) {
  const bool neg = a.neg != neg_;
  if (one_ || a.is_zero()) {
    q.mag = a.mag;
    q.neg = neg && !q.mag.empty();
    return true;
  }
  to64(a.mag, t_);
  if (t_.size() <= zeros_) return false;
  for (size_t i = 0; i < zeros_; ++i)
    if (t_[i]) return false;
  t_.erase(t_.begin(), t_.begin() + zeros_);
  if (t_[0] & (((uint64_t)1 << shift_) - 1)) return false;
  shift_down(t_, shift_);
  const size_t n = t_.size(), m = d_.size();
  if (n < m) return false;
  // quotient limbs from the low end: limb i cancels limb i of what is left
  for (size_t i = 0; i + m <= n; ++i) {
    const uint64_t x = t_[i] * inv_;
    uint64_t carry = 0;
    for (size_t j = 0; j < m; ++j) {
      const u128 p = (u128)x * d_[j] + carry;
      const uint64_t lo = (uint64_t)p;
      carry = (uint64_t)(p >> 64) + (t_[i + j] < lo);
      t_[i + j] -= lo;
    }
    for (size_t k = i + m; carry && k < n; ++k) {
      const uint64_t v = t_[k];
      t_[k] = v - carry;
      carry = v < carry;
    }
    if (carry) return false;
    t_[i] = x;
  }
  for (size_t k = n - m + 1; k < n; ++k)
    if (t_[k]) return false;
  from64(t_.data(), n - m + 1, q.mag);
  q.neg = neg && !q.mag.empty();
  return true;
}

bool big_divexact(const BigInt& a, const BigInt& b, BigInt& q) {
  ExactDiv d(b);
  return d(a, q);
}

// Lehmer's algorithm (TAOCP vol. 2, 4.5.2, Algorithm L): the quotients of the
// leading 62 bits, as long as both ends of their interval agree and the
// cofactors stay below 2^31, are applied to the numbers at once.
BigInt big_gcd(const BigInt& a, const BigInt& b) {
  std::vector<uint64_t> x, y, z;
  to64(a.mag, x);
  to64(b.mag, y);
  std::vector<uint32_t> x32, y32, q32, r32;
  if (cmp_mag(a.mag, b.mag) < 0) x.swap(y);
  while (y.size() > 1) {
    // x >= y; the window holds the leading 62 bits of x
    const size_t bits = 64 * x.size() - (size_t)__builtin_clzll(x.back());
    uint64_t u = window(x, bits - 62), v = window(y, bits - 62);
    int64_t A = 1, B = 0, C = 0, D = 1;
    while ((int64_t)v + C > 0 && (int64_t)v + D > 0) {
      const uint64_t q = (uint64_t)((int64_t)u + A) / (uint64_t)((int64_t)v + C);
      if (q != (uint64_t)((int64_t)u + B) / (uint64_t)((int64_t)v + D)) break;
      const s128 c = (s128)A - (s128)q * C, d = (s128)B - (s128)q * D;
      const s128 lim = (s128)1 << 31;
      if (c >= lim || c <= -lim || d >= lim || d <= -lim) break;
      A = C, B = D, C = (int64_t)c, D = (int64_t)d;
      const uint64_t t = u - q * v;
      u = v;
      v = t;
    }
    if (B == 0) {  // the first quotient is not certain or too long: one division
      from64(x.data(), x.size(), x32);
      from64(y.data(), y.size(), y32);
      divmod_mag(x32, y32, q32, r32);
      x.swap(y);
      to64(r32, y);
      continue;
    }
    z.assign(x.size(), 0);
    s128 cx = 0, cy = 0;
    for (size_t i = 0; i < x.size(); ++i) {
      const uint64_t xi = x[i], yi = i < y.size() ? y[i] : 0;
      cx += (s128)A * xi + (s128)B * yi;
      cy += (s128)C * xi + (s128)D * yi;
      x[i] = (uint64_t)cx;
      z[i] = (uint64_t)cy;
      cx >>= 64;
      cy >>= 64;
    }
    trim64(x);
    trim64(z);
    y.swap(z);
  }
  BigInt g;
  if (y.empty()) {
    from64(x.data(), x.size(), g.mag);
    return g;
  }
  uint64_t s = y[0], r = 0;
  for (size_t i = x.size(); i-- > 0;) r = (uint64_t)(((u128)r << 64 | x[i]) % s);
  while (r) {
    const uint64_t t = s % r;
    s = r;
    r = t;
  }
  return BigInt::from_u64(s);
}

uint32_t big_mod_small(const BigInt& a, uint32_t p) {
  // Barrett: the quotient by the reciprocal is short by at most two
  const uint64_t inv = ~(uint64_t)0 / p;
  uint64_t rem = 0;
  for (size_t i = a.mag.size(); i-- > 0;) {
    const uint64_t t = (rem << 32) | a.mag[i];
    rem = t - (uint64_t)((u128)t * inv >> 64) * p;
    if (rem >= p) rem -= p;
    if (rem >= p) rem -= p;
  }
  if (a.neg && rem) rem = p - rem;
  return (uint32_t)rem;
}

}  // namespace bires
