// Host side of the signed transforms' constants (modarith.h, pm_mul): which
// primes they take, and a factor's four words.
#pragma once
#include <stdint.h>

#include "modarith.h"

namespace heconv {

// q = 2^b - delta as the signed transforms take it (modarith.h, pm_mul):
// delta < 2^24 and d60 = 2^60 mod q = delta * 2^(60-b) < 2^31.
struct PmForm {
  bool ok;
  uint32_t b, delta;
  uint64_t d60;
};

inline PmForm pm_form(uint64_t q) {
  PmForm f{};
  f.b = 64 - (uint32_t)__builtin_clzll(q);
  if (f.b < 34 || f.b > 60) return f;
  const uint64_t delta = (1ull << f.b) - q;
  f.d60 = (unsigned __int128)delta << (60 - f.b) < (1ull << 31) ? delta << (60 - f.b) : 0;
  f.delta = (uint32_t)delta;
  f.ok = delta < (1u << 24) && f.d60 != 0;
  return f;
}

// A residue below 2^b as a factor of pm_mul: w or w - q, whichever fits two
// signed words split at bit 28, and the same for w * 2^32 mod q.
inline TwP twp_of(uint64_t w, uint64_t q, uint32_t b) {
  const auto split = [&](uint64_t r, int32_t& lo, int32_t& hi) {
    int64_t v = (int64_t)r;
    if (r + (1ull << 27) >= (1ull << (b - 1))) v -= (int64_t)q;
    hi = (int32_t)((v + (1ll << 27)) >> 28);
    lo = (int32_t)(v - ((int64_t)hi << 28));
  };
  // w * 2^32 = hi * 2^b + lo with hi < 2^32: hi * delta + lo is below 2^56 + 2^b, brought below 2q by one more fold
  const uint64_t delta = (1ull << b) - q;
  uint64_t v = (w >> (b - 32)) * delta + ((w & ((1ull << (b - 32)) - 1)) << 32);
  v = (v >> b) * delta + (v & ((1ull << b) - 1));
  if (v >= q) v -= q;
  TwP t;
  split(w, t.w0, t.w1);
  split(v, t.v0, t.v1);
  return t;
}

}  // namespace heconv
