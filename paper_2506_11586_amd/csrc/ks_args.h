// What the kernels of key switching share: the automorphism's gather and the
// operands of the inner product.
#pragma once
#include "kernels.h"
#include "modarith.h"
#include "udiv.h"

namespace heconv {

// Coefficient j of a(X^g) for the row a of N canonical residues mod q:
// with k = j * g^-1 mod 2N, a_k when k < N, else -a_{k-N}.  ginv = 1 reads
// the row as it is.
__device__ __forceinline__ uint64_t perm_load(const uint64_t* __restrict__ row, uint32_t j, uint32_t ginv, uint32_t N,
                                              uint64_t q) {
  const uint32_t k = (uint32_t)(((uint64_t)j * ginv) & (2 * N - 1));
  if (k < N) return row[k];
  const uint64_t v = row[k - N];
  return v ? q - v : 0;
}

// The inner product's operands: digits [n][L][L+1][N] and the key's rows, and
// the plaintext term.
//
// With a plaintext term (xp, wp non-null; the Z_P multiply-accumulate-rotate
// step), the sum for a ciphertext modulus m < L also takes
// xp[i][c][m] * wp[m]: the input ciphertext times a plaintext already
// multiplied by -P mod q_m.  The term is 0 mod P, so the division by P leaves
// the rotated ciphertext plus (x * plaintext) exactly.  nd digits are summed
// (L, or 0 when the rotated ciphertext is zero).  The batch may hold several
// chains of chain_cts ciphertexts that share the input x but take different
// weights: ciphertext i uses x[i % chain_cts] and the plaintext at
// wp + (i / chain_cts) * w_stride.
struct InnerArgs {
  const uint64_t *digits, *ksk, *xp, *wp;
  uint64_t w_stride;
  UDiv chain;  // by chain_cts
  uint32_t chain_cts, L, nd;
};

// (without a plaintext term, or as one chain, every ciphertext is its own)
inline InnerArgs inner_args(const uint64_t* digits, const uint64_t* ksk, const uint64_t* xp, const uint64_t* wp,
                            uint64_t chain_cts, uint64_t w_stride, uint32_t L, uint32_t nd) {
  const uint32_t cts = chain_cts && chain_cts < (1ull << 31) ? (uint32_t)chain_cts : 0x7fffffffu;
  return InnerArgs{digits, ksk, xp, wp, w_stride, udiv_make(cts), cts, L, nd};
}

}  // namespace heconv
