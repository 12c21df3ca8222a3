// NTT / inverse NTT in double precision for primes below 2^50: every
// residue is an exact double, and a modular product takes two products, two
// fused multiply-adds, a rounding and an addition, all full-rate fp64
// operations.  Same transform, order, mappings, passes, exchanges and table
// order as ntt_impl.h.
//
// mulmod(a, b), |a| <= A*q with A <= 8 (so |a| < 2^53), |b| <= q/2, q < 2^50:
//   hi = RN(a*b), lo = a*b - hi (exact, by the fused multiply-add),
//   k = rint(RN(hi * RN(1/q))): three roundings of relative size 2^-53 on a
//   quotient of at most A*q/2, plus the rounding to an integer, put it within
//   0.5 + 0.1875*A of a*b/q, and r = RN(hi - k*q) + lo = a*b - k*q exactly
//   (integers below 2^53), so |r| <= t(A)*q, t(A) = 0.5 + 0.1875*A.
// red(s), |s| < 8q: s - rint(RN(s * RN(1/q))) * q, exact, |result| <= q/2 + 8.
//
// Values are left unreduced between the stages while they stay below 8q.  A
// forward stage takes A to A + t(A): canonical words (1) reach 7.7 after six
// stages, values brought to 0.5 reach 7.9 after seven.  An inverse pass
// follows inv_pass's rule (s and p for sum and product of a stage): inputs at
// 1.92 give ss 7.7, brought to 0.5; then sps 3.9 and pss 4.9, brought to 0.5,
// and no other sum above 1.92; a fourth stage's sums are all brought to 0.5.
// Eight operations a butterfly, against fourteen with both results reduced
// each time.  Same box, before and after (with the exchanges and table order):
// N = 4096, 2048 limb polynomials, forward 39.0 -> 27.8 us, inverse 38-44 ->
// 29.5; 16384: 331 -> 253 and 312 -> 244 (4.3 TB/s); N = 8192, 24576: 991 ->
// 775 and 966 -> 772; N = 16384, 24576: 2160 -> 1583 and 2247 -> 1709.
#include "kernels.h"
#include "ntt_impl.h"

namespace heconv {

struct F64Const {
  double q, qinv, ninv, ninv_w;  // q, RN(1/q); N^-1 and N^-1 times the last inverse twiddle, balanced
};

__device__ __forceinline__ double mulmod_f64(double a, double b, double q, double qinv) {
  const double hi = a * b;
  const double lo = __fma_rn(a, b, -hi);
  const double k = rint(hi * qinv);
  return __fma_rn(-k, q, hi) + lo;
}

__device__ __forceinline__ double red_f64(double s, double q, double qinv) { return __fma_rn(-rint(s * qinv), q, s); }

// |s| < 8q brought to [0, q).
__device__ __forceinline__ double canon_f64(double s, double q, double qinv) {
  const double r = red_f64(s, q, qinv);
  return r < 0.0 ? r + q : r;
}

// A word below 2^52 as a double and back, by the bits of 2^52 + x.
__device__ __forceinline__ double to_f64(uint64_t x) {
  return __longlong_as_double((long long)(x | 0x4330000000000000ull)) - 4503599627370496.0;
}

__device__ __forceinline__ uint64_t from_f64(double x) {
  return (uint64_t)__double_as_longlong(x + 4503599627370496.0) & 0x000fffffffffffffull;
}

// As PassTw.
template <int LOGN, int LOGE, int LO, int U0>
struct PassTwF64 {
  double t[(1 << LOGE) - 1];
  __device__ __forceinline__ void load(int tid, const double* __restrict__ tw) {
    const uint32_t high = (uint32_t)block_of<LO>(tid);
#pragma unroll
    for (int u = U0; u < LOGE; u++) {
      const int s = LOGN - LOGE - LO + u;
#pragma unroll
      for (int g = 0; g < (1 << u); g++) t[(1 << u) - 1 + g] = tw[tw_at<LOGN>(s, u, high, g)];
    }
  }
};

template <bool RED, int LOGN, int LOGE, int LO, int U0>
__device__ __forceinline__ void fwd_pass_f64(double (&x)[1 << LOGE], const PassTwF64<LOGN, LOGE, LO, U0>& tw,
                                             const F64Const& c) {
  if constexpr (RED) {
#pragma unroll
    for (int k = 0; k < (1 << LOGE); k++) x[k] = red_f64(x[k], c.q, c.qinv);
  }
#pragma unroll
  for (int u = U0; u < LOGE; u++) {
    const int half = 1 << (LOGE - 1 - u);
#pragma unroll
    for (int g = 0; g < (1 << u); g++) {
      const double w = tw.t[(1 << u) - 1 + g];
#pragma unroll
      for (int e = 0; e < half; e++) {
        const int k0 = g * 2 * half + e, k1 = k0 + half;
        const double X = x[k0], T = mulmod_f64(x[k1], w, c.q, c.qinv);
        x[k0] = X + T;
        x[k1] = X - T;
      }
    }
  }
}

// Stages since the last reduction before full pass P, which reduces first
// when they and its own exceed six.
template <int LOGE>
constexpr int fwd_since_f64(int P) {
  int since = 0;
  for (int p = 0; p < P; p++) {
    if (since + LOGE > 6) since = 0;
    since += LOGE;
  }
  return since;
}

template <bool LAST, int LOGN, int LOGE, int LO, int U0>
__device__ __forceinline__ void inv_pass_f64(double (&x)[1 << LOGE], const PassTwF64<LOGN, LOGE, LO, U0>& tw,
                                             const F64Const& c) {
#pragma unroll
  for (int u = LOGE - 1; u >= U0; u--) {
    const int half = 1 << (LOGE - 1 - u);
    if (LAST && u == 0) {
#pragma unroll
      for (int e = 0; e < half; e++) {
        const double X = x[e], Y = x[e + half];
        x[e] = canon_f64(mulmod_f64(X + Y, c.ninv, c.q, c.qinv), c.q, c.qinv);
        x[e + half] = canon_f64(mulmod_f64(X - Y, c.ninv_w, c.q, c.qinv), c.q, c.qinv);
      }
      continue;
    }
#pragma unroll
    for (int g = 0; g < (1 << u); g++) {
      const double w = tw.t[(1 << u) - 1 + g];
#pragma unroll
      for (int e = 0; e < half; e++) {
        const int k0 = g * 2 * half + e, k1 = k0 + half;
        const double X = x[k0], Y = x[k1];
        x[k0] = X + Y;
        x[k1] = mulmod_f64(X - Y, w, c.q, c.qinv);
      }
    }
    const int j = LOGE - u;  // stages done
#pragma unroll
    for (int k = 0; k < (1 << LOGE); k++) {
      const bool r = (j == 1 && U0 == LOGE - 1 && (k & 1) == 0) || (j == 2 && (k & 3) == 0) ||
                     (j == 3 && ((k & 7) == 1 || (k & 7) == 2)) || (j == 4 && k < 8);
      if (r) x[k] = red_f64(x[k], c.q, c.qinv);
    }
  }
}

// As exchange.
template <int LOGE, int FROM, int TO>
__device__ __forceinline__ void exchange_f64(double* lds, double (&x)[1 << LOGE], int tid) {
  if constexpr (FROM == TO) return;
  constexpr bool WAVE = FROM <= 6 && TO <= 6;
  double* from = lds + lds_pad(elem_index<LOGE, FROM>(tid, 0));
  const double* to = lds + lds_pad(elem_index<LOGE, TO>(tid, 0));
  asm volatile("" ::: "memory");
#pragma unroll
  for (int k = 0; k < (1 << LOGE); k++) from[lds_pad(k << FROM)] = x[k];
  if constexpr (WAVE)
    asm volatile("" ::: "memory");
  else
    __syncthreads();
#pragma unroll
  for (int k = 0; k < (1 << LOGE); k++) x[k] = to[lds_pad(k << TO)];
}

template <int LOGN, int LOGE, int P>
__device__ __forceinline__ void fwd_rest_f64(double (&x)[1 << LOGE], double* lds, int tid,
                                             const double* __restrict__ tw, const F64Const& c) {
  constexpr int NFULL = LOGN / LOGE, REM = LOGN % LOGE;
  if constexpr (P < NFULL || (P == NFULL && REM > 0)) {
    constexpr int LO = P < NFULL ? LOGN - LOGE * (P + 1) : 0, U0 = P < NFULL ? 0 : LOGE - REM;
    PassTwF64<LOGN, LOGE, LO, U0> t;
    t.load(tid, tw);
    if constexpr (P > 0) exchange_f64<LOGE, LOGN - LOGE * P, LO>(lds, x, tid);
    fwd_pass_f64<(fwd_since_f64<LOGE>(P) + LOGE - U0 > 6)>(x, t, c);
    fwd_rest_f64<LOGN, LOGE, P + 1>(x, lds, tid, tw, c);
  }
}

template <int LOGN, int LOGE, int P, int PREV>
__device__ __forceinline__ void inv_rest_f64(double (&x)[1 << LOGE], double* lds, int tid,
                                             const double* __restrict__ tw, const F64Const& c) {
  constexpr int NFULL = LOGN / LOGE, REM = LOGN % LOGE;
  if constexpr (P < NFULL) {
    constexpr int LO = P < 0 ? 0 : REM + LOGE * P, U0 = P < 0 ? LOGE - REM : 0;
    PassTwF64<LOGN, LOGE, LO, U0> t;
    t.load(tid, tw);
    exchange_f64<LOGE, PREV, LO>(lds, x, tid);
    inv_pass_f64<(P == NFULL - 1)>(x, t, c);
    inv_rest_f64<LOGN, LOGE, P + 1, LO>(x, lds, tid, tw, c);
  }
}

template <int LOGN, int LOGE>
__global__ __launch_bounds__((1 << LOGN) >> LOGE, ntt_waves(LOGE)) void ntt_fwd_f64_kernel(
    uint64_t* __restrict__ polys_, uint32_t L, const double* __restrict__ tw_all, const F64Const* __restrict__ fcs) {
  constexpr int N = 1 << LOGN, E = 1 << LOGE, T = N / E;
  __shared__ double lds[N + N / 16];
  const uint32_t p = blockIdx.x, l = p % L;
  const F64Const c = fcs[l];
  gword* a = as_global(polys_) + (size_t)p * N;
  const int tid = threadIdx.x;
  double x[E];
#pragma unroll
  for (int k = 0; k < E; k++) x[k] = to_f64(a[tid + k * T]);
  fwd_rest_f64<LOGN, LOGE, 0>(x, lds, tid, tw_all + (size_t)l * N, c);
#pragma unroll
  for (int k = 0; k < E; k++) x[k] = canon_f64(x[k], c.q, c.qinv);
  exchange_f64<LOGE, 0, 6>(lds, x, tid);
  a += io_base<LOGE>(tid);
#pragma unroll
  for (int k = 0; k < E; k++) a[64 * k] = from_f64(x[k]);
}

template <int LOGN, int LOGE>
__global__ __launch_bounds__((1 << LOGN) >> LOGE, ntt_waves(LOGE)) void ntt_inv_f64_kernel(
    uint64_t* __restrict__ polys_, uint32_t L, const double* __restrict__ tw_all, const F64Const* __restrict__ fcs) {
  constexpr int N = 1 << LOGN, E = 1 << LOGE, T = N / E, REM = LOGN % LOGE;
  __shared__ double lds[N + N / 16];
  const uint32_t p = blockIdx.x, l = p % L;
  const F64Const c = fcs[l];
  gword* a = as_global(polys_) + (size_t)p * N;
  const int tid = threadIdx.x;
  double x[E];
#pragma unroll
  for (int k = 0; k < E; k++) x[k] = to_f64(a[io_base<LOGE>(tid) + 64 * k]);
  inv_rest_f64<LOGN, LOGE, (REM > 0 ? -1 : 0), 6>(x, lds, tid, tw_all + (size_t)l * N, c);
#pragma unroll
  for (int k = 0; k < E; k++) a[tid + k * T] = from_f64(x[k]);
}

template <int LOGN, int LOGE>
static hipError_t go_f64(bool inverse, uint64_t* polys, uint64_t nlp, uint32_t L, const double* tw,
                         const F64Const* fc, hipStream_t st) {
  constexpr int T = (1 << LOGN) >> LOGE;
  const uint64_t max_blocks = grid_max_blocks(T) / L * L;  // whole RNS polynomials per launch
  for (uint64_t off = 0; off < nlp; off += max_blocks) {
    const uint64_t cnt = nlp - off < max_blocks ? nlp - off : max_blocks;
    uint64_t* base = polys + off * (1ull << LOGN);
    if (inverse)
      hipLaunchKernelGGL((ntt_inv_f64_kernel<LOGN, LOGE>), dim3((uint32_t)cnt), dim3(T), 0, st, base, L, tw, fc);
    else
      hipLaunchKernelGGL((ntt_fwd_f64_kernel<LOGN, LOGE>), dim3((uint32_t)cnt), dim3(T), 0, st, base, L, tw, fc);
  }
  return hipGetLastError();
}

template <int LOGN>
static hipError_t go_f64_e(bool inverse, uint32_t loge, uint64_t* polys, uint64_t nlp, uint32_t L, const double* tw,
                           const F64Const* fc, hipStream_t st) {
  if constexpr (LOGN <= 13) {
    if (loge == 3) return go_f64<LOGN, 3>(inverse, polys, nlp, L, tw, fc, st);
  }
  return go_f64<LOGN, 4>(inverse, polys, nlp, L, tw, fc, st);
}

size_t f64_const_size() { return sizeof(F64Const); }

void f64_const_fill(void* out, double q, double qinv, double ninv, double ninv_w) {
  *static_cast<F64Const*>(out) = F64Const{q, qinv, ninv, ninv_w};
}

hipError_t ntt_f64_launch(bool inverse, uint32_t logN, uint32_t loge, uint64_t* polys, uint64_t n_rns_polys,
                          uint32_t L, const double* tw, const void* fc, hipStream_t st) {
  const uint64_t nlp = n_rns_polys * L;
  if (nlp == 0) return hipSuccess;
  const F64Const* f = static_cast<const F64Const*>(fc);
  switch (logN) {
    case 10: return go_f64_e<10>(inverse, loge, polys, nlp, L, tw, f, st);
    case 11: return go_f64_e<11>(inverse, loge, polys, nlp, L, tw, f, st);
    case 12: return go_f64_e<12>(inverse, loge, polys, nlp, L, tw, f, st);
    case 13: return go_f64_e<13>(inverse, loge, polys, nlp, L, tw, f, st);
    case 14: return go_f64_e<14>(inverse, loge, polys, nlp, L, tw, f, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace heconv
