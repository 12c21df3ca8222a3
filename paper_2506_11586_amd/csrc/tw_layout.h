// Order of a twiddle table's entries, shared by the host that fills it and
// the transforms that read it.
//
// Stage s has 2^s twiddles.  A pass of LOGE stages reads, for its stage u,
// the twiddles (high << u) + g of g = 0 .. 2^u - 1, high the index of the
// thread's block: with g fastest, a load instruction (one g, consecutive
// lanes) steps 16 * 2^u bytes from block to block and touches up to four
// times the cache lines it uses.  So a stage read by lanes of different
// blocks (its pass's mapping lies below bit 6) keeps its entries with high
// fastest within 64 highs, and every load is one contiguous run.  Stages whose
// block is the same across a wave keep g fastest: their loads are scalar, and
// wider so.
// The order follows the pass structure that is used by default (16 words per
// thread at N = 2^14, else 8); other structures compute the place of each
// entry.
#pragma once

namespace heconv {

constexpr int tw_loge(int logN) { return logN == 14 ? 4 : 3; }

// The position u of stage s in its pass where high is fastest, else 0.
constexpr int tw_u(int logN, int s) {
  const int e = tw_loge(logN), full = logN / e * e;
  if (s >= full) return e - logN % e + (s - full);  // the partial pass, at bit 0
  return logN - e * (s / e + 1) >= 6 ? 0 : s % e;
}

// Place of twiddle (high << u) + g of stage s, u = tw_u: blocks of 64 highs,
// each with its 2^u runs, so that a thread's 2^u entries are 1 KiB apart
// (one address and constant offsets).
constexpr unsigned tw_place_hg(int s, int u, unsigned high, unsigned g) {
  const int lb = s - u < 6 ? s - u : 6;
  return (1u << s) + (((high >> lb) << u) << lb) + (g << lb) + (high & ((1u << lb) - 1));
}

// Place of twiddle i < 2^s of stage s.
constexpr unsigned tw_place(int logN, int s, unsigned i) {
  const int u = tw_u(logN, s);
  return u ? tw_place_hg(s, u, i >> u, i & ((1u << u) - 1)) : (1u << s) + i;
}

}  // namespace heconv
