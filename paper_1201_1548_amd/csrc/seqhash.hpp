// Signature of a device call sequence: a captured graph may stand for a later
// call only if every argument of every launch is the same.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "job.hpp"

namespace bires {

// FNV-1a hash of the arguments of a device call sequence.
struct SeqHash {
  uint64_t h = 1469598103934665603ull;
  void bytes(const void* p, size_t n) {
    const unsigned char* c = (const unsigned char*)p;
    for (size_t i = 0; i < n; ++i) h = (h ^ c[i]) * 1099511628211ull;
  }
  template <class T>
  void one(const T& v) {
    static_assert(std::is_arithmetic<T>::value || std::is_pointer<T>::value || std::is_enum<T>::value,
                  "hash scalars and pointers only");
    bytes(&v, sizeof v);
  }
  // Field by field (the padding is not part of it); the binding names every
  // field, so that one more does not compile until it is added here.
  void one(const TablesDev& t) {
    const auto& [primes, gm, cm, pi, pm, invfact, inv_p, K, dmax, qpow, geo_invu, geo_w, geo_A, geo_D, pow_planes,
                 pow_nb] = t;
    add(primes, gm, cm, pi, pm, invfact, inv_p, K, dmax, qpow, geo_invu, geo_w, geo_A, geo_D, pow_planes, pow_nb);
  }
  template <class... A>
  void add(const A&... a) {
    (one(a), ...);
  }
};

}  // namespace bires
