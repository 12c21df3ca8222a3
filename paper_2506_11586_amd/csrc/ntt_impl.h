// Fused negacyclic NTT / inverse NTT for gfx950: one workgroup per limb
// polynomial, E = 2^LOGE coefficients per thread in registers, radix-E
// passes (LOGE butterfly stages each) with an LDS transpose between passes.
//
// Forward (Cooley-Tukey, natural order in, bit-reversed order out): the
// butterfly on bit b pairs j and j + 2^b with twiddle psi^brv(2^(n-1-b) +
// (j >> (b+1))), n = log2 N; stages run from bit n-1 down to bit 0.  The
// inverse (Gentleman-Sande) uses the same index with psi^-1 and runs from
// bit 0 up; its last stage also applies N^-1.  Lazy reduction after Harvey,
// with the twiddle products by mul_shoup_2q (inputs below 6q, results below
// 2.75q): forward values stay in [0, 6q) (X = x0 brought below 3q by one
// conditional subtraction, T = mul_shoup_2q(x1), outputs X + T < 5.75q and
// X - T + 3q < 6q), inverse values in [0, 3q) (the sum brought below 3q by
// one conditional subtraction, the difference X - Y + 3q, below 6q, through
// mul_shoup_2q).  Every stored word is canonical (fwd_canon, or the last
// inverse stage).
//
// With PM (every prime 2^b - delta with small delta: modarith.h, pm_mul) both
// directions work on signed values instead, with no conditional subtraction
// in a butterfly; fwd_pass and inv_pass state where pm_red is needed.  The
// words stored are the same canonical residues.  VALU cycles of a butterfly
// at full rate: 38 forward and about 45 inverse, against 84.
//
// Thread/element mapping of a pass over bits [lo, lo+LOGE): register k of
// thread t holds element j = (t mod 2^lo) | k << lo | (t >> lo) << (lo+LOGE).
// The top pass (lo = n-LOGE) is j = t + k*N/E: coefficients are loaded and
// stored in it, so every wave access is a contiguous 512-byte run.  NTT-form
// words are loaded and stored in the mapping at lo = 6, whose runs are as
// long and whose exchange with lo = 0 stays inside each wave (io_base).  When n is not a multiple of LOGE the leftover bits are
// done by a partial pass at lo = 0.
#pragma once
#include <type_traits>

#include "modarith.h"
#include "tw_layout.h"


namespace heconv {

// Waves per SIMD that the register budget must allow: two workgroups of 1024
// threads per CU with 8 words per thread (64 VGPRs; without the bound the
// signed inverse took 70 and ran one), one with 16.
constexpr int ntt_waves(int loge) { return loge == 3 ? 8 : 4; }

__device__ __forceinline__ int lds_pad(int j) { return j + (j >> 4); }

template <int LOGE, int LO>
__device__ __forceinline__ int elem_index(int tid, int k) {
  const int low = tid & ((1 << LO) - 1);
  const int high = tid >> LO;
  return low | (k << LO) | (high << (LO + LOGE));
}

// tid >> LO, the index of the thread's block of 2^LO elements.  From LO = 6
// up every lane of a wave has the same value (tid = 64w + i gives
// w >> (LO - 6)); it is then read from the first lane, so the twiddle index
// is uniform and its loads are scalar loads shared by the wave.
template <int LO>
__device__ __forceinline__ int block_of(int tid) {
  if constexpr (LO >= 6)
    return __builtin_amdgcn_readfirstlane(tid >> LO);
  else
    return tid >> LO;
}

// Place of the twiddle that a thread of block `high` reads as the g-th of a
// pass's stage u, stage s of the transform.
template <int TLOGN>
__device__ __forceinline__ uint32_t tw_at(int s, int u, uint32_t high, uint32_t g) {
  return tw_u(TLOGN, s) == u && u ? tw_place_hg(s, u, high, g) : tw_place(TLOGN, s, (high << u) + g);
}

// The twiddles of a pass's stages [U0, LOGE) in the order the stages use them
// (stage u holds 2^u of them from slot 2^u - 1 on; the inverse runs the stages
// backwards over the same slots), at their places in the table (tw_layout.h).
// They are loaded before the exchange that precedes the pass, so that their
// latency passes behind it.  24576 limb polynomials with both against loads at
// the stage and g fastest throughout: N = 16384 forward 1960 -> 1770 us,
// inverse 2200 -> 1840; N = 8192 835 -> 830 and 887 -> 845 (a bench-wide 3.8
// TB/s, where a copy in place without the arithmetic runs 5.5).  jb: index of
// the workgroup's first element when it transforms a block of a longer
// polynomial (the stages on bits below the block size only; jb a multiple of
// the block size), else 0.
// TLOGN: log2 of the length whose table tw is (of the longer polynomial's,
// whose first stages a shorter transform's coincide with).
template <int LOGN, int LOGE, int LO, int U0, bool PM, int TLOGN = LOGN>
struct PassTw {
  using T = std::conditional_t<PM, TwP, Tw>;
  T t[(1 << LOGE) - 1];
  __device__ __forceinline__ void load(int tid, const Tw* __restrict__ tw, uint32_t jb = 0) {
    const uint32_t high = (uint32_t)block_of<LO>(tid) + (jb >> (LO + LOGE));
#pragma unroll
    for (int u = U0; u < LOGE; u++) {
      const int s = LOGN - LOGE - LO + u;  // stage index
#pragma unroll
      for (int g = 0; g < (1 << u); g++)
        t[(1 << u) - 1 + g] = reinterpret_cast<const T*>(tw)[tw_at<TLOGN>(s, u, high, g)];
    }
  }
};

// Forward values of the PM form are stored with a bias of 2^31 (pm_mul_biased);
// the bias passes through X + T and X - T unchanged.  A loaded word gets it
// here, and fwd_canon takes it off.
template <bool PM>
__device__ __forceinline__ uint64_t fwd_in(uint64_t x) {
  return PM ? x + (1ull << 31) : x;
}

// A forward value (below 6q; PM: |x| < 7.9u, biased) brought to [0, q).
template <bool PM>
__device__ __forceinline__ uint64_t fwd_canon(uint64_t x, const LimbConst& c) {
  if constexpr (PM)
    return pm_canon(x + (c.pk - (1ull << 31)), c);
  else
    return canon_below6q(x, c.neg3q, c.neg2q, c.negq);
}

// Forward stages u in [U0, LOGE) of the pass at bit offset LO: butterflies on
// bit LO+LOGE-1-u.
// PM: a stage takes a bound of a to a + T(a), so canonical inputs (1u) reach
// 7.2u after seven stages, and values brought to 0.5u 7.54u after eight; RED
// brings them there before the pass (fwd_red).
template <bool RED, int LOGN, int LOGE, int LO, int U0, bool PM, int TLOGN>
__device__ __forceinline__ void fwd_pass(uint64_t (&x)[1 << LOGE], const PassTw<LOGN, LOGE, LO, U0, PM, TLOGN>& tw,
                                         const LimbConst& c, const PmRegs& pk) {
  const uint64_t q3 = c.three_q;
  if constexpr (PM && RED) {
#pragma unroll
    for (int k = 0; k < (1 << LOGE); k++) x[k] = pm_red(x[k], pk);
  }
#pragma unroll
  for (int u = U0; u < LOGE; u++) {
    const int half = 1 << (LOGE - 1 - u);
#pragma unroll
    for (int g = 0; g < (1 << u); g++) {
      const auto t = tw.t[(1 << u) - 1 + g];
#pragma unroll
      for (int e = 0; e < half; e++) {
        const int k0 = g * 2 * half + e, k1 = k0 + half;
        if constexpr (PM) {
          const uint64_t X = x[k0], T = pm_mul_biased(x[k1], t, pk);
          x[k0] = X + T;
          x[k1] = X - T;
        } else {
          const uint64_t X = csub_neg(x[k0], c.neg3q);
          const uint64_t T = mul_shoup_2q(x[k1], t.w, t.wsh, c.neg2q);
          x[k0] = X + T;
          x[k1] = X - T + q3;
        }
      }
    }
  }
}

// Whether the forward full pass P (stages LOGE*P ..) first brings its values
// to 0.5u: when the stages since the last time, with its own, exceed seven.
// fwd_since: stages since then, before pass P.
template <int LOGE>
constexpr int fwd_since(int P) {
  int since = 0;
  for (int p = 0; p < P; p++) {
    if (since + LOGE > 7) since = 0;
    since += LOGE;
  }
  return since;
}

// Inverse stages u from LOGE-1 down to U0 of the pass at LO.  With LAST, the
// stage on the top bit (u = 0 of the pass at n-LOGE) also applies N^-1 and
// leaves canonical values (RAW, PM only: signed ones below 0.9u).
//
// PM: with s and p for the sum and the product of a stage, an input bound a
// <= 1.8u gives after two stages ss 4a = 7.2u, sp T(4a) = 1.0u, ps 2T(2a) =
// 1.77u, pp 0.83u; ss is then brought to 0.5u.  After three: sss 1.0u, ssp
// 0.8u, sps 2.0u, spp 0.84u, pss 3.5u, psp 0.89u, pps 1.65u, ppp 0.83u; sps
// and pss are brought to 0.5u.  After four: ssss 2.0u, ppss 3.3u, both
// brought to 0.5u, and no other above 1.77u.  A pass of one stage on
// canonical inputs brings its sums (2u) to 0.5u.  So every pass starts below
// 1.8u again, and no value reaches 7.5u.  Register k's bit j is 0 where
// stage j of the pass left it a sum.
template <bool LAST, bool RAW = false, int LOGN, int LOGE, int LO, int U0, bool PM, int TLOGN>
__device__ __forceinline__ void inv_pass(uint64_t (&x)[1 << LOGE], const PassTw<LOGN, LOGE, LO, U0, PM, TLOGN>& tw,
                                         const LimbConst& c, const PmRegs& pk) {
  const uint64_t q3 = c.three_q;
#pragma unroll
  for (int u = LOGE - 1; u >= U0; u--) {
    const int half = 1 << (LOGE - 1 - u);
    if (LAST && u == 0) {
#pragma unroll
      for (int e = 0; e < half; e++) {
        const int k0 = e, k1 = e + half;
        uint64_t X = x[k0], Y = x[k1];
        if constexpr (PM) {
          x[k0] = pm_mul_val(X + Y, c.pninv, pk);
          x[k1] = pm_mul_val(X - Y, c.pninv_w, pk);
          if constexpr (!RAW) x[k0] = pm_canon(x[k0] + c.pk, c), x[k1] = pm_canon(x[k1] + c.pk, c);
        } else {
          x[k0] = csub_neg(mul_shoup_neg(X + Y, c.ninv, c.ninv_sh, c.negq), c.negq);
          x[k1] = csub_neg(mul_shoup_neg(X - Y + q3, c.ninv_w, c.ninv_w_sh, c.negq), c.negq);
        }
      }
      continue;
    }
#pragma unroll
    for (int g = 0; g < (1 << u); g++) {
      const auto t = tw.t[(1 << u) - 1 + g];
#pragma unroll
      for (int e = 0; e < half; e++) {
        const int k0 = g * 2 * half + e, k1 = k0 + half;
        const uint64_t X = x[k0], Y = x[k1];
        if constexpr (PM) {
          x[k0] = X + Y;
          x[k1] = pm_mul_val(X - Y, t, pk);
        } else {
          x[k0] = csub_neg(X + Y, c.neg3q);
          x[k1] = mul_shoup_2q(X - Y + q3, t.w, t.wsh, c.neg2q);
        }
      }
    }
    if constexpr (PM) {
      const int j = LOGE - u;  // stages done
#pragma unroll
      for (int k = 0; k < (1 << LOGE); k++) {
        const bool r = (j == 1 && U0 == LOGE - 1 && (k & 1) == 0) || (j == 2 && (k & 3) == 0) ||
                       (j == 3 && ((k & 7) == 1 || (k & 7) == 2)) || (j == 4 && ((k & 15) == 0 || (k & 15) == 3));
        if (r) x[k] = pm_red(x[k], pk);
      }
    }
  }
}

// Move the thread's registers from the mapping at FROM to the mapping at TO
// through LDS, element j at lds_pad(j).  A transform's exchanges form a
// chain, so each thread writes the very entries that it read in the exchange
// before (FROM is that one's TO): no other thread can still be reading them,
// and one barrier, between the writes and the reads, orders a cross-wave
// exchange.  A kernel that used LDS otherwise before its first exchange needs
// a barrier there.
//
// Wave-local form.  In a mapping with LO <= 6 the 64 threads of wave w
// (tid = 64w + i) hold exactly the elements whose index bits from 6+LOGE up
// equal w: the low LO bits come from i, and tid >> LO = w*2^(6-LO) + (i >> LO).
// When FROM and TO both satisfy this, each wave writes and reads only its
// own aligned block of 2^(6+LOGE) elements (a disjoint range of LDS after
// padding), so no other wave is involved and no workgroup barrier is needed.
// The LDS operations of one wave are performed in issue order, and the
// empty asm statements with a memory clobber keep the compiler from moving
// a read above a write (for one lane the addresses differ, so it otherwise
// could).
template <int LOGE, int FROM, int TO>
__device__ __forceinline__ void exchange(uint64_t* lds, uint64_t (&x)[1 << LOGE], int tid) {
  if constexpr (FROM == TO) return;
  constexpr bool WAVE = FROM <= 6 && TO <= 6;
  // k << LO and the thread's part share no bit, so the padded index is their
  // padded indexes' sum: one address and constant offsets
  uint64_t* from = lds + lds_pad(elem_index<LOGE, FROM>(tid, 0));
  const uint64_t* to = lds + lds_pad(elem_index<LOGE, TO>(tid, 0));
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

// The mapping in which NTT-form words are loaded and stored, at LO = 6:
// register k of lane i of wave w holds word i + 64*k of the wave's block of
// 64*2^LOGE words.  Every access is a contiguous 512-byte run, as in the top
// mapping, and the exchange with bit 0 is wave-local.
template <int LOGE>
__device__ __forceinline__ int io_base(int tid) {
  return elem_index<LOGE, 6>(tid, 0);
}

// Forward full passes at LO = LOGN-LOGE*(P+1), then the partial pass.
template <int LOGN, int LOGE, int P, bool PM>
__device__ __forceinline__ void fwd_rest(uint64_t (&x)[1 << LOGE], uint64_t* lds, int tid,
                                         const Tw* __restrict__ tw, const LimbConst& c, const PmRegs& pk) {
  constexpr int NFULL = LOGN / LOGE, REM = LOGN % LOGE;
  if constexpr (P < NFULL || (P == NFULL && REM > 0)) {
    constexpr int LO = P < NFULL ? LOGN - LOGE * (P + 1) : 0, U0 = P < NFULL ? 0 : LOGE - REM;
    PassTw<LOGN, LOGE, LO, U0, PM> t;
    t.load(tid, tw);
    if constexpr (P > 0) exchange<LOGE, LOGN - LOGE * P, LO>(lds, x, tid);
    fwd_pass<(fwd_since<LOGE>(P) + LOGE - U0 > 7)>(x, t, c, pk);
    fwd_rest<LOGN, LOGE, P + 1, PM>(x, lds, tid, tw, c, pk);
  }
}

// Inverse passes: the partial one at LO = 0 (P = -1, if any), then full ones
// at LO = REM + LOGE*P, each after the exchange from the mapping at PREV.
template <int LOGN, int LOGE, int P, int PREV, bool PM, bool RAW>
__device__ __forceinline__ void inv_rest(uint64_t (&x)[1 << LOGE], uint64_t* lds, int tid,
                                         const Tw* __restrict__ tw, const LimbConst& c, const PmRegs& pk) {
  constexpr int NFULL = LOGN / LOGE, REM = LOGN % LOGE;
  if constexpr (P < NFULL) {
    constexpr int LO = P < 0 ? 0 : REM + LOGE * P, U0 = P < 0 ? LOGE - REM : 0;
    PassTw<LOGN, LOGE, LO, U0, PM> t;
    t.load(tid, tw);
    exchange<LOGE, PREV, LO>(lds, x, tid);
    inv_pass<(P == NFULL - 1), RAW>(x, t, c, pk);
    inv_rest<LOGN, LOGE, P + 1, LO, PM, RAW>(x, lds, tid, tw, c, pk);
  }
}

// Forward transform of values in registers in the top mapping (register k of
// thread t = entry t + k*N/E; canonical, PM: any below 2^60), left canonical
// in the mapping of NTT-form words (register k = entry io_base + 64*k).
template <int LOGN, int LOGE, bool PM>
__device__ __forceinline__ void ntt_fwd_regs(uint64_t (&x)[1 << LOGE], const Tw* __restrict__ tw, const LimbConst& c,
                                             uint64_t* lds, int tid) {
  constexpr int E = 1 << LOGE;
  const PmRegs pk = pm_regs(c);
#pragma unroll
  for (int k = 0; k < E; k++) x[k] = fwd_in<PM>(x[k]);
  fwd_rest<LOGN, LOGE, 0, PM>(x, lds, tid, tw, c, pk);
#pragma unroll
  for (int k = 0; k < E; k++) x[k] = fwd_canon<PM>(x[k], c);
  exchange<LOGE, 0, 6>(lds, x, tid);
}

// Forward transform of one limb polynomial a[N] (in place) by the calling
// workgroup of N/2^LOGE threads.
template <int LOGN, int LOGE, bool PM>
__device__ __forceinline__ void ntt_fwd_poly(gword* __restrict__ a, const Tw* __restrict__ tw, const LimbConst& c,
                                             uint64_t* lds, int tid) {
  constexpr int N = 1 << LOGN, E = 1 << LOGE, T = N / E;
  uint64_t x[E];
#pragma unroll
  for (int k = 0; k < E; k++) x[k] = a[tid + k * T];
  ntt_fwd_regs<LOGN, LOGE, PM>(x, tw, c, lds, tid);
  a += io_base<LOGE>(tid);
#pragma unroll
  for (int k = 0; k < E; k++) a[64 * k] = x[k];
}

// Inverse transform of NTT values already in registers in the mapping of
// NTT-form words (register k = entry io_base + 64*k); leaves the
// coefficients canonical in the top mapping (entry t + k*N/E).  RAW (PM
// only): signed values of the coefficients times c.pninv * N, below 0.9u.
template <int LOGN, int LOGE, bool PM, bool RAW = false>
__device__ __forceinline__ void ntt_inv_regs(uint64_t (&x)[1 << LOGE], const Tw* __restrict__ tw, const LimbConst& c,
                                             uint64_t* lds, int tid) {
  constexpr int REM = LOGN % LOGE;
  const PmRegs pk = pm_regs(c);
  inv_rest<LOGN, LOGE, (REM > 0 ? -1 : 0), 6, PM, RAW>(x, lds, tid, tw, c, pk);
}

// Inverse transform of one limb polynomial a[N] (in place).  With NT the
// input is loaded and the result stored non-temporally: a layer's MAC output
// is read once here, and its result is not read again soon, so streaming
// both past the caches keeps L2 and the Infinity Cache for the weights.
template <int LOGN, int LOGE, bool PM, bool NT = false>
__device__ __forceinline__ void ntt_inv_poly(gword* __restrict__ a, const Tw* __restrict__ tw, const LimbConst& c,
                                             uint64_t* lds, int tid) {
  constexpr int N = 1 << LOGN, E = 1 << LOGE, T = N / E;
  uint64_t x[E];
#pragma unroll
  for (int k = 0; k < E; k++) {
    if constexpr (NT)
      x[k] = __builtin_nontemporal_load(&a[io_base<LOGE>(tid) + 64 * k]);
    else
      x[k] = a[io_base<LOGE>(tid) + 64 * k];
  }
  ntt_inv_regs<LOGN, LOGE, PM>(x, tw, c, lds, tid);
#pragma unroll
  for (int k = 0; k < E; k++) {
    if constexpr (NT)
      __builtin_nontemporal_store(x[k], &a[tid + k * T]);
    else
      a[tid + k * T] = x[k];
  }
}

}  // namespace heconv
