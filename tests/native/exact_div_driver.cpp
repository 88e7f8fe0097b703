// Test driver for ExactDiv and big_sub_from: reads "d a b c" in signed
// hexadecimal, one divisor for the dividends a and b in turn, and prints both
// quotients ("inexact") and a - c.
#include <cstdio>
#include <iostream>
#include <string>

#include "../../paper_1201_1548_amd/csrc/bigint.hpp"

using namespace bires;

static BigInt parse(const std::string& s) {
  BigInt r;
  const size_t i = s[0] == '-';
  for (size_t end = s.size(); end > i;) {
    const size_t beg = end - i >= 8 ? end - 8 : i;
    r.mag.push_back((uint32_t)std::stoul(s.substr(beg, end - beg), nullptr, 16));
    end = beg;
  }
  trim(r.mag);
  r.neg = i && !r.mag.empty();
  return r;
}

static std::string show(const BigInt& x) {
  if (x.mag.empty()) return x.neg ? "negative zero" : "0";
  std::string s = x.neg ? "-" : "";
  char buf[16];
  for (size_t i = x.mag.size(); i-- > 0;) {
    snprintf(buf, sizeof buf, "%08x", x.mag[i]);
    s += buf;
  }
  return s;
}

int main() {
  std::string d, a, b, c;
  while (std::cin >> d >> a >> b >> c) {
    ExactDiv by(parse(d));
    BigInt q, x = parse(a);
    std::cout << (by(x, q) ? show(q) : "inexact") << ",";
    std::cout << (by(parse(b), q) ? show(q) : "inexact") << ",";
    big_sub_from(x, parse(c));
    std::cout << show(x) << "\n";
  }
  return 0;
}
