// Test driver for SeqHash on TablesDev: prints the signature of the table with
// no field set, then one line per field with that field alone changed, and last
// the first table's again over other padding bytes.
#include <cstdio>
#include <cstring>

#include "../../paper_1201_1548_amd/csrc/seqhash.hpp"

using namespace bires;

static void show(const char* name, const TablesDev& t) {
  SeqHash s;
  s.add(t);
  printf("%s %016llx\n", name, (unsigned long long)s.h);
}

int main() {
  static const uint64_t mem[2] = {0, 0};
  TablesDev t{};
  show("base", t);
#define POINTER(f)                      \
  do {                                  \
    TablesDev c = t;                    \
    c.f = (decltype(c.f))(mem + 1);     \
    show(#f, c);                        \
  } while (0)
#define COUNT(f)      \
  do {                \
    TablesDev c = t;  \
    c.f = 7;          \
    show(#f, c);      \
  } while (0)
  POINTER(primes);
  POINTER(gm);
  POINTER(cm);
  POINTER(pi);
  POINTER(pm);
  POINTER(invfact);
  POINTER(inv_p);
  COUNT(K);
  COUNT(dmax);
  POINTER(qpow);
  POINTER(geo_invu);
  POINTER(geo_w);
  POINTER(geo_A);
  COUNT(geo_D);
  POINTER(pow_planes);
  COUNT(pow_nb);
  TablesDev d;
  memset((void*)&d, 0xA5, sizeof d);
  d.primes = nullptr, d.gm = d.cm = d.pi = d.pm = d.invfact = nullptr, d.inv_p = nullptr, d.K = d.dmax = 0;
  d.qpow = d.geo_invu = d.geo_w = nullptr, d.geo_A = nullptr, d.geo_D = 0, d.pow_planes = nullptr, d.pow_nb = 0;
  show("padding", d);
  return 0;
}
