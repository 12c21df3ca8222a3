// Key switching of a few ciphertexts in three grids of small workgroups, with
// the signed transforms split at bit n-6 as in ntt_split.hip:
//   A: a workgroup takes 16 residues mod N/64 of one digit (read through the
//      automorphism) for one extended modulus: the first six forward stages;
//   B: a workgroup takes 1024 consecutive NTT indexes of one modulus: the
//      remaining stages of all L digits, one per group of 128 threads, the
//      inner product with both key components, and those sums' first inverse
//      stages, so that NTT-form words never leave the workgroup;
//   D: a workgroup takes 16 residues of one component: the last six inverse
//      stages mod P and mod one q_m side by side, the division by P, b and the
//      addend.
// One workgroup per polynomial (rotate.hip) leaves most of the chip idle with
// few ciphertexts, and each of its three kernels then takes one whole
// transform's latency; here a ciphertext at N = 8192, L = 3 is 96, 32 and 48
// workgroups, and each grid takes half a transform's: rotation of one 26.2 ->
// 16.9 us (the grids alone, as a profiler times them, 4.7, 7.8 and 5.6 us; each
// waits for the words that the last one stored, then runs at one wave per SIMD,
// bound by its own issue rate).
// With all of a block's twiddles loaded before its first pass (252 VGPRs) it
// was no faster, and 16 ciphertexts slower (34.0 against 32.6 us).
#include "ks_args.h"
#include "split_impl.h"

namespace heconv {

constexpr int KS_LDS = 1024 + 1024 / 16;  // words of one group's exchanges

// Grid A. digits[i][l][m] takes signed biased values (below 6.3 * 2^60).
template <int LOGN>
__global__ __launch_bounds__(SPLIT_T) void ks_split_a(const uint64_t* __restrict__ ct, uint64_t* __restrict__ digits,
                                                       uint32_t L, uint32_t ginv, const Tw* __restrict__ tw_all,
                                                       const LimbConst* __restrict__ ext) {
  constexpr int N = 1 << LOGN, G = N / 64, W = G / 16;
  __shared__ uint64_t lds[KS_LDS];
  const uint32_t L1 = L + 1, w = blockIdx.x % W, row = blockIdx.x / W;  // (i, l, m)
  const uint32_t il = row / L1, m = row - il * L1, i = il / L, l = il - i * L;
  const int tid = threadIdx.x;
  const LimbConst c = ext[m];
  const PmRegs pk = pm_regs(c);
  const Tw* tw = tw_all + (size_t)m * N;
  const uint64_t* src = ct + ((uint64_t)i * 2 * L + l) * N;
  const uint64_t ql = ext[l].q;
  uint64_t x[8];
  PassTw<10, 3, 7, 0, true, LOGN> t0;
  t0.load(tid, tw);
  // virtual index v = tid + 128k -> residue 16w + (v & 15), i = v >> 4
#pragma unroll
  for (int k = 0; k < 8; k++) {
    const int v = tid + 128 * k;
    x[k] = fwd_in<true>(perm_load(src, 16 * w + (v & 15) + G * (v >> 4), ginv, N, ql));
  }
  PassTw<10, 3, 4, 0, true, LOGN> t1;
  t1.load(tid, tw);
  fwd_pass<false>(x, t0, c, pk);
  exchange<3, 7, 4>(lds, x, tid);
  fwd_pass<false>(x, t1, c, pk);
  uint64_t* out = digits + (uint64_t)row * N + 16 * w;
#pragma unroll
  for (int k = 0; k < 8; k++) {
    const int v = elem_index<3, 4>(tid, k);
    out[(v & 15) + G * (v >> 4)] = x[k];
  }
}

// Grid B, max(L, 2) groups of 128 threads; group r transforms digit r, and
// groups 0 and 1 then hold the sums of the two components.  ND: the number of
// digits where it is known (0: any up to 7); the key's words are then loaded
// before the transform.
template <int LOGN, int ND>
__global__ __launch_bounds__((ND > 2 ? ND : ND ? 2 : 7) * SPLIT_T) void ks_split_b(
    InnerArgs g, uint64_t* __restrict__ acc, const Tw* __restrict__ fwd_all, const Tw* __restrict__ inv_all,
    const LimbConst* __restrict__ ext) {
  constexpr int N = 1 << LOGN, W = N / 1024, NB = LOGN - 6;
  extern __shared__ uint64_t lds_all[];
  const uint32_t L = ND ? ND : g.L, L1 = L + 1, w = blockIdx.x % W, im = blockIdx.x / W;  // (i, m)
  const uint32_t i = im / L1, m = im - i * L1, jb = w * 1024;
  const int tid = threadIdx.x % SPLIT_T;
  const uint32_t grp = __builtin_amdgcn_readfirstlane(threadIdx.x / SPLIT_T);
  const LimbConst c = ext[m];
  const PmRegs pk = pm_regs(c);
  uint64_t* lds = lds_all + grp * KS_LDS;
  // the sums are formed in the mapping at LO = 0, words jb + 8*tid + k
  const uint64_t word = (uint64_t)m * N + jb + 8 * tid;
  const bool plain = g.xp && m < L;
  uint64_t x[8], kv[ND ? ND : 1][8], xv[8], wv[8];
  if (grp < L) {
    const uint64_t* d = g.digits + ((uint64_t)i * L + grp) * L1 * N + (uint64_t)m * N + jb;
#pragma unroll
    for (int k = 0; k < 8; k++) x[k] = d[elem_index<3, NB - 3>(tid, k)];
  }
  if (ND && grp < 2) {
#pragma unroll
    for (int l = 0; l < ND; l++)
#pragma unroll
      for (int k = 0; k < 8; k++) kv[l][k] = g.ksk[((uint64_t)(l * 2) + grp) * L1 * N + word + k];
  }
  if (plain && grp < 2) {
    const uint32_t chain = udiv(i, g.chain), ic = i - chain * g.chain_cts;
    const uint64_t* xp = g.xp + ((uint64_t)ic * 2 + grp) * L * N + word;
    const uint64_t* wp = g.wp + chain * g.w_stride + word;
#pragma unroll
    for (int k = 0; k < 8; k++) xv[k] = xp[k], wv[k] = wp[k];
  }
  if (grp < L) {
    split_b_rest<LOGN, 0, true>(x, lds, tid, fwd_all + (size_t)m * N, c, pk, jb);
    // into the thread's own entries of the last exchange
#pragma unroll
    for (int k = 0; k < 8; k++) lds[lds_pad(8 * tid) + k] = fwd_canon<true>(x[k], c);
  }
  __syncthreads();
  if (grp < 2) {
    const uint64_t* own = lds_all + lds_pad(8 * tid);
#pragma unroll
    for (int h = 0; h < 8; h += 4) {  // 24 accumulator registers at a time
      uint64_t a00[4], am[4], a11[4];
      const auto add = [&](int k, uint64_t d, uint64_t kw) {
        const Half30 xs = split30(d), ws = split30(kw);
        a00[k] += (uint64_t)xs.lo * ws.lo;
        am[k] += (uint64_t)xs.lo * ws.hi;
        am[k] += (uint64_t)xs.hi * ws.lo;
        a11[k] += (uint64_t)xs.hi * ws.hi;
      };
#pragma unroll
      for (int k = 0; k < 4; k++) a00[k] = am[k] = a11[k] = 0;
      if constexpr (ND > 0) {
#pragma unroll
        for (int l = 0; l < ND; l++)
#pragma unroll
          for (int k = 0; k < 4; k++) add(k, own[l * KS_LDS + h + k], kv[l][h + k]);
      } else {
        for (uint32_t l = 0; l < L; l++) {
          const uint64_t* kp = g.ksk + ((uint64_t)(l * 2) + grp) * L1 * N + word + h;
#pragma unroll
          for (int k = 0; k < 4; k++) add(k, own[l * KS_LDS + h + k], kp[k]);
        }
      }
      if (plain) {
#pragma unroll
        for (int k = 0; k < 4; k++) add(k, xv[h + k], wv[h + k]);
      }
#pragma unroll
      for (int k = 0; k < 4; k++) x[h + k] = fold3_pm<false>(a00[k], am[k], a11[k], (uint32_t)c.d60, (uint32_t)c.c30);
    }
  }
  __syncthreads();  // both components' groups have read every digit
  if (grp < 2) {
    inv_split_c_rest<LOGN, (NB % 3 > 0 ? -1 : 0), 0, true>(x, lds, tid, inv_all + (size_t)m * N, c, pk, jb);
    uint64_t* out = acc + (((uint64_t)i * 2 + grp) * L1 + m) * N + jb;
#pragma unroll
    for (int k = 0; k < 8; k++) out[elem_index<3, NB - 3>(tid, k)] = x[k];
  }
}

// Grid D, two groups of 128 threads: group 0 the sums mod P, group 1 those mod
// q_m with P^-1 in the last stage's factors (as inner_moddown_kernel).
template <int LOGN>
__global__ __launch_bounds__(2 * SPLIT_T) void ks_split_d(const uint64_t* __restrict__ acc, uint32_t L,
                                                           const Tw* __restrict__ inv_all,
                                                           const LimbConst* __restrict__ ext, const uint64_t* ct,
                                                           uint64_t* out, uint32_t ginv, KsConst kc,
                                                           const uint64_t* addp) {
  constexpr int N = 1 << LOGN, G = N / 64, W = G / 16;
  __shared__ uint64_t lds_all[2 * KS_LDS];
  const uint32_t L1 = L + 1, w = blockIdx.x % W, row = blockIdx.x / W;  // (i, comp, m)
  const uint32_t ic = row / L, m = row - ic * L, comp = ic & 1;
  const int tid = threadIdx.x % SPLIT_T;
  const uint32_t grp = __builtin_amdgcn_readfirstlane(threadIdx.x / SPLIT_T), mod = grp ? m : L;
  LimbConst c = ext[mod];
  if (grp) c.pninv = kc.ninv[m], c.pninv_w = kc.ninv_w[m];
  const PmRegs pk = pm_regs(c);
  const Tw* tw = inv_all + (size_t)mod * N;
  const uint64_t* a = acc + ((uint64_t)ic * L1 + mod) * N + 16 * w;
  uint64_t* lds = lds_all + grp * KS_LDS;
  uint64_t x[8], e[8];
#pragma unroll
  for (int k = 0; k < 8; k++) {
    const int v = elem_index<3, 4>(tid, k);
    x[k] = a[(v & 15) + G * (v >> 4)];
  }
  PassTw<10, 3, 4, 0, true, LOGN> t0;
  t0.load(tid, tw);
  PassTw<10, 3, 7, 0, true, LOGN> t1;
  t1.load(tid, tw);
  // what the result adds: b through the automorphism, and the addend
  const uint64_t base = (uint64_t)row * N;
#pragma unroll
  for (int k = 0; k < 8; k++) {
    const int v = tid + 128 * k;
    const uint32_t j = 16 * w + (v & 15) + G * (v >> 4);
    e[k] = 0;
    if (grp && comp) e[k] = perm_load(ct + base, j, ginv, N, c.q);
    if (grp && addp) e[k] += addp[base + j];
  }
  inv_pass<false>(x, t0, c, pk);
  exchange<3, 4, 7>(lds, x, tid);
  inv_pass<true, true>(x, t1, c, pk);  // |x| < 0.9u
  if (!grp) {
    // the centred residue mod P, into the thread's own entries of the exchange
#pragma unroll
    for (int k = 0; k < 8; k++) {
      const uint64_t r = pm_canon(x[k] + c.pk, c);
      lds[lds_pad(tid) + lds_pad(128 * k)] = r > c.q / 2 ? r - c.q : r;
    }
  }
  __syncthreads();
  if (grp) {
    const TwP pinv = kc.pinv[m];
#pragma unroll
    for (int k = 0; k < 8; k++) {
      const int v = tid + 128 * k;
      const uint64_t xc = lds_all[lds_pad(tid) + lds_pad(128 * k)];
      const uint64_t y = pm_mul_val(xc, pinv, pk) - x[k] + e[k];  // |.| < 3.7u
      out[base + 16 * w + (v & 15) + G * (v >> 4)] = pm_canon(y + c.pk, c);
    }
  }
}

namespace {

template <int LOGN>
void ks_split_go(const KsSplit& s, hipStream_t st) {
  constexpr uint32_t W = (1u << LOGN) / 1024;
  const uint32_t L = s.L, n = (uint32_t)s.n;
  const InnerArgs g = inner_args(s.digits, s.ksk, s.xp, s.wp, s.chain_cts, s.w_stride, L, L);
  const dim3 tb((L > 2 ? L : 2) * SPLIT_T);
  const size_t sh = (L > 2 ? L : 2) * KS_LDS * sizeof(uint64_t);
  hipLaunchKernelGGL((ks_split_a<LOGN>), dim3(n * L * (L + 1) * W), dim3(SPLIT_T), 0, st, s.ct, s.digits, L, s.ginv,
                     s.fwd, s.ext);
#define HECONV_KS_B(ND) \
  hipLaunchKernelGGL((ks_split_b<LOGN, ND>), dim3(n * (L + 1) * W), tb, sh, st, g, s.acc, s.fwd, s.inv, s.ext)
  switch (L) {
    case 2: HECONV_KS_B(2); break;
    case 3: HECONV_KS_B(3); break;
    default: HECONV_KS_B(0); break;
  }
#undef HECONV_KS_B
  hipLaunchKernelGGL((ks_split_d<LOGN>), dim3(n * 2 * L * W), dim3(2 * SPLIT_T), 0, st, s.acc, L, s.inv, s.ext, s.ct,
                     s.out, s.ginv, s.kc, s.addp);
}

}  // namespace

bool ks_split_supported(uint32_t logN) { return logN >= 12 && logN <= 14; }

hipError_t ks_split_launch(uint32_t logN, const KsSplit& s, hipStream_t st) {
  if (!s.n) return hipSuccess;
  if (s.L < 1 || s.L > 7) return hipErrorInvalidValue;
  // the largest grid has fewer than 4*L*(L+1)*N/8 threads a ciphertext
  if (logN < 10 || s.n > grid_max_blocks(SPLIT_T) / (4ull * s.L * (s.L + 1) * ((1u << logN) / 1024)))
    return hipErrorInvalidConfiguration;
  switch (logN) {
    case 12: ks_split_go<12>(s, st); break;
    case 13: ks_split_go<13>(s, st); break;
    case 14: ks_split_go<14>(s, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace heconv
