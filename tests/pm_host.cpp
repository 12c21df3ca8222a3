// Host check of the signed transforms' arithmetic (modarith.h, pm_form.h)
// against exact 128-bit arithmetic: pm_mul (both operand forms) is x*w mod q
// and stays within T(|x|) = 0.766 * 2^60 + 0.0333 |x| for |x| up to 7.9 *
// 2^60; pm_red within 0.5 * 2^60 + 8 * d60 for |x| < 7.5 * 2^60; pm_canon the
// canonical residue; and both directions' passes, run on the stages and
// reductions that ntt_impl.h states, never leave their bounds; mac_fold over
// chunks of the MAC's products.
// Usage: pm_host <q> <trials>; prints "ok <n>" or the first failure, exit 1.
#include <cstdio>
#include <cstdlib>

#include "pm_form.h"

using namespace heconv;
typedef __int128 i128;
typedef unsigned __int128 u128;

static uint64_t sm_state = 0x1234567;
static uint64_t rnd() {
  uint64_t z = (sm_state += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

static uint64_t q;
static uint64_t mod(int64_t x) { return (uint64_t)((((i128)x % (i128)q) + q) % q); }
static uint64_t mul(uint64_t a, uint64_t b) { return (uint64_t)((u128)a * b % q); }
static const double U = 1152921504606846976.0;
static double mag(int64_t x) { return x < 0 ? -(double)x : (double)x; }

static int fail(const char* what, int64_t x, uint64_t w) {
  std::printf("%s q=%llu x=%lld w=%llu\n", what, (unsigned long long)q, (long long)x, (unsigned long long)w);
  return 1;
}

static uint64_t factor(long n) {
  switch (n % 6) {
    case 0: return q - 1 - rnd() % 8;
    case 1: return q / 2 + rnd() % (1 << 29) - (1 << 28);  // either side of the sign choice
    case 2: return rnd() % 16;
    default: return rnd() % q;
  }
}

int main(int argc, char** argv) {
  if (argc < 3) return 2;
  q = strtoull(argv[1], 0, 10);
  const long trials = strtol(argv[2], 0, 10);
  const PmForm f = pm_form(q);
  if (!f.ok) return fail("not a prime of this form", 0, 0);
  LimbConst c{};
  c.q = q, c.two28 = 1u << 28;
  c.pb32 = f.b - 32, c.pmask = (1u << c.pb32) - 1, c.pdelta = f.delta, c.d60 = (int32_t)f.d60;
  c.pk = q << (63 - f.b);
  c.c30 = 1u << 30;
  const PmRegs k = pm_regs(c);
  const int64_t top = (int64_t)(7.9 * U), redtop = (int64_t)(7.49 * U);
  for (long n = 0; n < trials; n++) {
    const uint64_t w = factor(n);
    const TwP t = twp_of(w, q, f.b);
    if (mod((int64_t)t.w0 + (int64_t)t.w1 * (1ll << 28)) != w ||
        mod((int64_t)t.v0 + (int64_t)t.v1 * (1ll << 28)) != mul(w, (1ull << 32) % q))
      return fail("twp_of", 0, w);
    int64_t x = (int64_t)(rnd() % (2 * (uint64_t)top) - (uint64_t)top);
    if (n % 5 == 1) x = top - (int64_t)(rnd() & 0xffffffff);
    if (n % 5 == 2) x = (int64_t)(rnd() & 0xffffffff) - top;
    if (n % 5 == 3) x = (int64_t)((rnd() % 15) - 7) * (1ll << 60) + (int64_t)(rnd() % 5) - 2 + (1ll << 31) * (int64_t)(rnd() % 3);
    const double T = 0.766 * U + 0.0333 * mag(x);
    const int64_t r0 = (int64_t)pm_mul_val((uint64_t)x, t, k);
    const int64_t r1 = (int64_t)pm_mul_biased((uint64_t)x + (1ull << 31), t, k);
    if (mod(r0) != mul(mod(x), w) || mag(r0) > T) return fail("pm_mul_val", x, w);
    if (r1 != r0) return fail("pm_mul_biased", x, w);
    if (pm_canon((uint64_t)x + c.pk, c) != mod(x)) return fail("pm_canon", x, 0);
    const int64_t y = mag(x) < 7.49 * U ? x : (x < 0 ? x + (1ll << 60) : x - (1ll << 60));
    const int64_t z = y > redtop ? redtop : y;
    const int64_t r = (int64_t)pm_red((uint64_t)z, k);
    if (mod(r) != mod(z) || mag(r) > 0.5 * U + 8.0 * (double)f.d60) return fail("pm_red", z, 0);
  }
  // forward: seven stages from canonical values, eight from 0.5u
  for (long n = 0; n < trials / 64; n++) {
    int64_t X = (int64_t)(n % 3 == 0 ? q - 1 : rnd() % q), Y = (int64_t)(n % 3 == 1 ? q - 1 : rnd() % q);
    uint64_t ex = mod(X), ey = mod(Y);
    X += 1ll << 31, Y += 1ll << 31;
    for (int st = 0; st < 15; st++) {
      if (st == 7) X = (int64_t)pm_red((uint64_t)X, k), Y = (int64_t)pm_red((uint64_t)Y, k);
      const uint64_t w = factor(n + st);
      const int64_t T = (int64_t)pm_mul_biased((uint64_t)Y, twp_of(w, q, f.b), k);
      const int64_t nx = X + T, ny = X - T;
      const uint64_t t = mul(ey, w), fx = (ex + t) % q, fy = (ex + q - t) % q;
      if (mod(nx - (1ll << 31)) != fx || mod(ny - (1ll << 31)) != fy || mag(nx) > 7.6 * U || mag(ny) > 7.6 * U)
        return fail("forward stage", X, w);
      const bool sw = rnd() & 1;
      X = sw ? ny : nx, Y = sw ? nx : ny, ex = sw ? fy : fx, ey = sw ? fx : fy;
    }
    if (pm_canon((uint64_t)X + (c.pk - (1ull << 31)), c) != ex) return fail("forward canonical", X, 0);
  }
  // inverse: passes of 3 or 4 stages (after a first one of 1 to 3 on canonical
  // values) on a block of registers, each pass starting at up to 1.8u with the
  // signs that add up
  for (long n = 0; n < trials / 64; n++) {
    const int loge = 3 + (int)(n & 1), E = 1 << loge, first = (int)(rnd() % loge);  // 0: no partial pass
    int64_t x[16];
    uint64_t e[16];
    double start = 1.0;
    for (int pass = 0; pass < 4; pass++) {
      const int stages = pass == 0 && first ? first : loge;
      for (int i = 0; i < E; i++) {
        // the bound that the pass may meet, reached by adding multiples of q
        const double a = pass == 0 ? 1.0 : start;
        if (pass == 0) {
          x[i] = (int64_t)(n % 3 ? rnd() % q : q - 1);
        } else {
          const int64_t m = (int64_t)(a * U) - (int64_t)(rnd() & 0xffff);
          x[i] = n % 3 == 0 ? m : (n % 3 == 1 ? ((i >> (int)(rnd() % loge)) & 1 ? -m : m) : (int64_t)(rnd() % (2 * (uint64_t)m) - (uint64_t)m));
        }
        e[i] = mod(x[i]);
      }
      for (int j = 1; j <= stages; j++) {
        const int half = 1 << (j - 1);
        for (int b = 0; b < E; b += 2 * half) {
          const uint64_t w = factor(n + b + j);
          for (int i = b; i < b + half; i++) {
            const int64_t X = x[i], Y = x[i + half];
            if (mag(X) + mag(Y) >= 8 * U && !(pass == 0 && X >= 0 && Y >= 0)) return fail("inverse sum", X, w);
            x[i] = X + Y;
            x[i + half] = (int64_t)pm_mul_val((uint64_t)(X - Y), twp_of(w, q, f.b), k);
            const uint64_t s = (e[i] + e[i + half]) % q, d = mul((e[i] + q - e[i + half]) % q, w);
            e[i] = s, e[i + half] = d;
          }
        }
        for (int i = 0; i < E; i++) {
          const bool r = (j == 1 && stages == 1 && (i & 1) == 0) || (j == 2 && (i & 3) == 0) ||
                         (j == 3 && ((i & 7) == 1 || (i & 7) == 2)) || (j == 4 && ((i & 15) == 0 || (i & 15) == 3));
          if (r) {
            if (mag(x[i]) >= 7.5 * U) return fail("inverse before pm_red", x[i], 0);
            x[i] = (int64_t)pm_red((uint64_t)x[i], k);
          }
        }
      }
      for (int i = 0; i < E; i++) {
        if (mod(x[i]) != e[i] || mag(x[i]) > 1.8 * U) return fail("inverse pass", x[i], 0);
        if (pm_canon((uint64_t)x[i] + c.pk, c) != e[i]) return fail("inverse canonical", x[i], 0);
      }
      start = 1.8;
    }
  }
  // the MAC's folds: chunks of eight products of residues (at their ends too) on a carried value
  for (long n = 0; n < trials / 16; n++) {
    uint64_t a00 = 0, am = 0, a11 = 0, want = 0;
    for (int chunk = 0; chunk < 3; chunk++) {
      for (int i = 0; i < 8; i++) {
        const uint64_t x = n % 3 == 0 ? q - 1 : factor(n + i), w = n % 2 == 0 ? q - 1 : factor(n + 2 * i + 1);
        const uint64_t xl = x & 0x3fffffff, xh = x >> 30, wl = w & 0x3fffffff, wh = w >> 30;
        if ((u128)a00 + (u128)xl * wl >> 64 || (u128)am + (u128)xl * wh + (u128)xh * wl >> 64)
          return fail("MAC accumulator", (int64_t)x, w);
        a00 += xl * wl, am += xl * wh + xh * wl, a11 += xh * wh;
        want = (want + mul(x, w)) % q;
      }
      if (mac_fold<MAC_FOLD_PM, true>(a00, am, a11, c) != want) return fail("mac_fold canonical", (int64_t)a00, am);
      a00 = mac_fold<MAC_FOLD_PM, false>(a00, am, a11, c), am = a11 = 0;
      if (a00 % q != want || a00 >= (1ull << 60) + (1ull << 52)) return fail("mac_fold carried", (int64_t)a00, 0);
    }
  }
  std::printf("ok %ld\n", trials);
  return 0;
}
