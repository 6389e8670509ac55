// binomials.h -- C(a, b) for a <= 32 as a constant table; every value fits 32 bits.
#pragma once

#include <stdint.h>

namespace gcimpl {

struct BinomTable {
  uint32_t c[33][33];  // [a][b], zero for b > a
};
constexpr BinomTable make_binom() {
  BinomTable t{};
  for (int a = 0; a <= 32; ++a)
    for (int b = 0; b <= a; ++b) t.c[a][b] = b == 0 || b == a ? 1u : t.c[a - 1][b - 1] + t.c[a - 1][b];
  return t;
}

}  // namespace gcimpl
