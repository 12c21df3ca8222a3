// Ciphertext rotation for the Z_P variant (rotations need key switching
// with evaluation keys, Sec. 2; the Z_P kernels rotate once per
// multiply-accumulate iteration, Sec. 6.1): the Galois automorphism
// a(X) -> a(X^g) and hybrid key switching with one special prime P, the
// last modulus of an extended context q_0..q_{L-1}, P.  For a ciphertext
// (a, b) whose phase is b - a*s':
//   digits d_l = limb l of a, integers below q_l, reduced into every
//   modulus of the extended basis and transformed (modup_kernel + NTT);
//   A = sum_l d_l * k_a[l], B = sum_l d_l * k_b[l], point-wise in the NTT
//   domain (ks_inner_kernel), transformed back;
//   y = (x - [x]_P) / P with [x]_P the residue mod P centred into
//   (-P/2, P/2]: per modulus q_j, (x_j - ([x]_P mod q_j)) * P^-1 mod q_j
//   (moddown_kernel), giving (-A', b - B') under s.
// A rotation applies the automorphism to a while the digits are read and to
// b in the last step, so the rotated ciphertext is never stored.
// Forms, by the number of ciphertexts (ks_step in api.cpp):
//   few: three grids of small workgroups (ks_split.hip);
//   more: modup_ntt_kernel (digit extension in the forward transform's load),
//     inner_intt_kernel (the inner product in the inverse transform's load)
//     and moddown_kernel;
//   many, signed transforms: modup_ntt_kernel, inner_intt_kernel for the sums
//     mod P alone, and inner_moddown_kernel (the other sums with the division
//     by P after their transform, in registers).
// The elementwise modup_kernel and ks_inner_kernel with the library's NTT
// kernels between them are the separate-steps form, and ks_fwd_kernel the
// form with both sums kept in registers (tuning ks_fused 0 and 2).
#include "kernels.h"
#include "ks_args.h"
#include "mac_impl.h"
#include "ntt_impl.h"

namespace heconv {

constexpr uint32_t ROT_THREADS = 256;

__device__ __forceinline__ uint64_t red_word(uint64_t x, const LimbConst& c) {
  return csub(reduce64_lazy(x, c.mu64, c.q), c.q);
}

// out[r] = in[r](X^g) for every row r of N coefficients; row r is limb
// r % L and uses modulus lcs[r % L].
__global__ __launch_bounds__(ROT_THREADS) void automorph_kernel(const uint64_t* __restrict__ in,
                                                                 uint64_t* __restrict__ out, uint32_t N,
                                                                 uint32_t L, uint32_t ginv,
                                                                 const LimbConst* __restrict__ lcs) {
  const uint32_t per_row = N / ROT_THREADS;
  const uint64_t row = blockIdx.x / per_row;
  const uint32_t j = (blockIdx.x % per_row) * ROT_THREADS + threadIdx.x;
  out[row * N + j] = perm_load(in + row * N, j, ginv, N, lcs[row % L].q);
}

// work[i][l][m][k] = (a_i(X^g))[l][k] mod p_m: digit l of ciphertext i in
// extended modulus m < L+1 (ct [n][2][L][N], a is component 0).
__global__ __launch_bounds__(ROT_THREADS) void modup_kernel(const uint64_t* __restrict__ ct,
                                                             uint64_t* __restrict__ work, uint32_t N, uint32_t L,
                                                             uint32_t ginv, const LimbConst* __restrict__ ext) {
  const uint32_t per_row = N / ROT_THREADS;
  const uint64_t row = blockIdx.x / per_row;  // (i, l, m)
  const uint32_t k = (blockIdx.x % per_row) * ROT_THREADS + threadIdx.x;
  const uint32_t m = (uint32_t)(row % (L + 1));
  const uint64_t il = row / (L + 1);
  const uint32_t l = (uint32_t)(il % L);
  const uint64_t i = il / L;
  const uint64_t d = perm_load(ct + (i * 2 * L + l) * N, k, ginv, N, ext[l].q);
  work[row * N + k] = m == l ? d : red_word(d, ext[m]);
}

// acc[i][c][m][k] = sum_l work[i][l][m][k] * ksk[l][c][m][k] mod p_m: the L
// products summed in 128 bits (each below 2^120, L <= 7), reduced once.
__global__ __launch_bounds__(ROT_THREADS) void ks_inner_kernel(const uint64_t* __restrict__ work,
                                                                const uint64_t* __restrict__ ksk,
                                                                uint64_t* __restrict__ acc, uint32_t N, uint32_t L,
                                                                const LimbConst* __restrict__ ext) {
  const uint32_t per_row = N / ROT_THREADS;
  const uint64_t row = blockIdx.x / per_row;  // (i, m)
  const uint32_t k = (blockIdx.x % per_row) * ROT_THREADS + threadIdx.x;
  const uint32_t L1 = L + 1;
  const uint32_t m = (uint32_t)(row % L1);
  const uint64_t i = row / L1;
  uint64_t ah = 0, al = 0, bh = 0, bl = 0;
  for (uint32_t l = 0; l < L; l++) {
    const uint64_t d = work[((i * L + l) * L1 + m) * N + k];
    uint64_t hi, lo;
    mul_wide(d, ksk[((uint64_t)(l * 2 + 0) * L1 + m) * N + k], hi, lo);
    al += lo;
    ah += hi + (al < lo);
    mul_wide(d, ksk[((uint64_t)(l * 2 + 1) * L1 + m) * N + k], hi, lo);
    bl += lo;
    bh += hi + (bl < lo);
  }
  const LimbConst c = ext[m];
  acc[((i * 2 + 0) * L1 + m) * N + k] = reduce128(ah, al, c);
  acc[((i * 2 + 1) * L1 + m) * N + k] = reduce128(bh, bl, c);
}

// out[i] = (-A', b(X^g) - B') with y = (x_j - ([x]_P mod q_j)) * P^-1 mod q_j
// With addp non-null, the ciphertext addp[i] is added to the result.
__global__ __launch_bounds__(ROT_THREADS) void moddown_kernel(const uint64_t* __restrict__ acc,
                                                               const uint64_t* __restrict__ ct,
                                                               uint64_t* __restrict__ out, uint32_t N, uint32_t L,
                                                               uint32_t ginv, PinvConst pinv,
                                                               const uint64_t* __restrict__ addp,
                                                               const LimbConst* __restrict__ ext) {
  const uint32_t per_row = N / ROT_THREADS;
  const uint64_t row = blockIdx.x / per_row;  // (i, j), j < L
  const uint32_t k = (blockIdx.x % per_row) * ROT_THREADS + threadIdx.x;
  const uint32_t L1 = L + 1;
  const uint32_t j = (uint32_t)(row % L);
  const uint64_t i = row / L;
  const LimbConst c = ext[j];
  const uint64_t P = ext[L].q;
  uint64_t y[2];
#pragma unroll
  for (int comp = 0; comp < 2; comp++) {
    const uint64_t xj = acc[((i * 2 + comp) * L1 + j) * N + k];
    const uint64_t xp = acc[((i * 2 + comp) * L1 + L) * N + k];
    uint64_t cm;  // [x]_P mod q_j
    if (xp <= P / 2) {
      cm = red_word(xp, c);
    } else {
      const uint64_t mag = red_word(P - xp, c);
      cm = mag ? c.q - mag : 0;
    }
    const uint64_t d = csub(xj + (c.q - cm), c.q);
    y[comp] = csub(mul_shoup_lazy(d, pinv.v[j], pinv.sh[j], c.q), c.q);
  }
  const uint64_t b = ct ? perm_load(ct + ((i * 2 + 1) * L + j) * N, k, ginv, N, c.q) : 0;  // null: a zero ciphertext
  uint64_t oa = y[0] ? c.q - y[0] : 0, ob = csub(b + (c.q - y[1]), c.q);
  if (addp) {
    oa = csub(oa + addp[((i * 2 + 0) * L + j) * N + k], c.q);
    ob = csub(ob + addp[((i * 2 + 1) * L + j) * N + k], c.q);
  }
  out[((i * 2 + 0) * L + j) * N + k] = oa;
  out[((i * 2 + 1) * L + j) * N + k] = ob;
}

// Digit extension, forward transform and inner product fused: one workgroup
// per (ciphertext i, extended modulus m) runs the L digits one after the
// other.  Digit l is read from the ciphertext's a row (the automorphism
// applied through LDS: the row is staged with coalesced loads, then each
// thread gathers its permuted entries), reduced mod p_m, transformed in
// registers, and multiplied by the key's transformed rows; the two sums stay
// in registers and only they are stored.  The L+1 workgroups of one
// ciphertext run on the same XCD (block b runs on XCD b % 8), so they share
// its a rows in that XCD's L2.  Grid: ceil(n/8)*8*(L+1) workgroups.
template <int LOGN, bool PM>
__global__ __launch_bounds__((1 << LOGN) >> 3) void ks_fwd_kernel(const uint64_t* __restrict__ ct,
                                                                   const uint64_t* __restrict__ ksk,
                                                                   uint64_t* __restrict__ acc, uint64_t n, uint32_t L,
                                                                   uint32_t ginv, const Tw* __restrict__ tw_all,
                                                                   const LimbConst* __restrict__ ext) {
  constexpr int LOGE = 3, E = 1 << LOGE, N = 1 << LOGN, T = N / E;
  __shared__ uint64_t lds[N + N / 16];
  const uint32_t L1 = L + 1;
  const uint32_t xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
  const uint64_t i = (uint64_t)(slot / L1) * 8 + xcd;
  const uint32_t m = slot % L1;
  if (i >= n) return;  // the whole workgroup leaves before any barrier
  const LimbConst c = ext[m];
  uint64_t sa[E], sb[E];
#pragma unroll
  for (int k = 0; k < E; k++) sa[k] = sb[k] = 0;
  for (uint32_t l = 0; l < L; l++) {
    // The thread index and twiddle offset pass through an empty asm
    // statement each digit, so that the address arithmetic and twiddle loads
    // (the same for every digit) are redone instead of hoisted out of the
    // loop, where they would stay live across it and spill.
    int tid = threadIdx.x;
    uint32_t off = m * N;
    asm volatile("" : "+v"(tid), "+v"(off));
    const Tw* tw = tw_all + __builtin_amdgcn_readfirstlane(off);
    const uint64_t* row = ct + (i * 2 * L + l) * N;
    uint64_t x[E];
    __syncthreads();  // the previous digit's last LDS reads are done
    if (ginv == 1) {
#pragma unroll
      for (int k = 0; k < E; k++) x[k] = row[tid + k * T];
    } else {
      const uint64_t ql = ext[l].q;
#pragma unroll
      for (int k = 0; k < E; k++) lds[lds_pad(tid + k * T)] = row[tid + k * T];
      __syncthreads();
#pragma unroll
      for (int k = 0; k < E; k++) {
        const uint32_t src = (uint32_t)(((uint64_t)(tid + k * T) * ginv) & (2 * N - 1));
        const uint64_t v = lds[lds_pad(src & (N - 1))];
        x[k] = src >= (uint32_t)N && v ? ql - v : v;
      }
      __syncthreads();  // the row is read before the transform reuses its LDS
    }
    if (!PM && m != l) {  // (PM: the transform takes any word below 2^60)
#pragma unroll
      for (int k = 0; k < E; k++) x[k] = red_word(x[k], c);
    }
    ntt_fwd_regs<LOGN, LOGE, PM>(x, tw, c, lds, tid);  // entry io_base + 64*k, as the key rows are read
    // the key loads are addressed from a value defined here, so they are
    // issued after the transform rather than held in registers through it
    int tk = io_base<LOGE>(tid);
    asm volatile("" : "+v"(tk));
    const uint64_t* ka = ksk + ((uint64_t)(l * 2) * L1 + m) * N;
    const uint64_t* kb = ka + (uint64_t)L1 * N;
#pragma unroll
    for (int k = 0; k < E; k++) {
      uint64_t hi, lo;
      mul_wide(x[k], ka[tk + 64 * k], hi, lo);
      sa[k] = csub(sa[k] + reduce128(hi, lo, c), c.q);
      mul_wide(x[k], kb[tk + 64 * k], hi, lo);
      sb[k] = csub(sb[k] + reduce128(hi, lo, c), c.q);
    }
  }
  const int io = io_base<LOGE>(threadIdx.x);
  uint64_t* oa = acc + ((i * 2) * L1 + m) * N;
  uint64_t* ob = oa + (uint64_t)L1 * N;
#pragma unroll
  for (int k = 0; k < E; k++) {
    oa[io + 64 * k] = sa[k];
    ob[io + 64 * k] = sb[k];
  }
}

// Digit extension fused into the forward transform: one workgroup per
// (ciphertext i, digit l, extended modulus m) reads limb l of a (through the
// automorphism, staged in LDS as in ks_fwd_kernel), reduces it mod p_m and
// stores its transform to digits[i][l][m].  The L+1 workgroups that read one
// a row run on the same XCD.  Grid: ceil(n*L/8)*8*(L+1) workgroups.
template <int LOGN, bool PM>
__global__ __launch_bounds__((1 << LOGN) >> 3, ntt_waves(3)) void modup_ntt_kernel(const uint64_t* __restrict__ ct,
                                                                      uint64_t* __restrict__ digits, uint64_t n,
                                                                      uint32_t L, uint32_t ginv,
                                                                      const Tw* __restrict__ tw_all,
                                                                      const LimbConst* __restrict__ ext) {
  constexpr int LOGE = 3, E = 1 << LOGE, N = 1 << LOGN, T = N / E;
  __shared__ uint64_t lds[N + N / 16];
  const uint32_t L1 = L + 1;
  const uint32_t xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
  const uint64_t il = (uint64_t)(slot / L1) * 8 + xcd;  // (i, l)
  const uint32_t m = slot % L1;
  if (il >= n * L) return;  // the whole workgroup leaves before any barrier
  const uint32_t l = (uint32_t)(il % L);
  const uint64_t i = il / L;
  const int tid = threadIdx.x;
  const LimbConst c = ext[m];
  const uint64_t* row = ct + (i * 2 * L + l) * N;
  uint64_t x[E];
  if (ginv == 1) {
#pragma unroll
    for (int k = 0; k < E; k++) x[k] = row[tid + k * T];
  } else {
    const uint64_t ql = ext[l].q;
#pragma unroll
    for (int k = 0; k < E; k++) lds[lds_pad(tid + k * T)] = row[tid + k * T];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < E; k++) {
      const uint32_t src = (uint32_t)(((uint64_t)(tid + k * T) * ginv) & (2 * N - 1));
      const uint64_t v = lds[lds_pad(src & (N - 1))];
      x[k] = src >= (uint32_t)N && v ? ql - v : v;
    }
    __syncthreads();  // the row is read before the transform reuses its LDS
  }
  if (!PM && m != l) {  // (PM: the transform takes any word below 2^60)
#pragma unroll
    for (int k = 0; k < E; k++) x[k] = red_word(x[k], c);
  }
  ntt_fwd_regs<LOGN, LOGE, PM>(x, tw_all + (size_t)m * N, c, lds, tid);
  uint64_t* out = digits + (il * L1 + m) * N + io_base<LOGE>(tid);
#pragma unroll
  for (int k = 0; k < E; k++) out[64 * k] = x[k];
}

// The point-wise sums of key switching for one workgroup (ciphertext i,
// component comp, extended modulus m): x[k] = sum over l < nd of digit l times
// the key row (comp, m) at word io_base + 64*k, plus the plaintext term,
// reduced once.
//
// PM: the products of 30-bit halves in three accumulators (at most eight
// terms: am stays below 2^64) and one short fold, left below 2^60 + 2^54;
// else 128-bit sums (each product below 2^120) and a full reduction.  TERMS:
// the number of terms where it is known (0: any; with the signed transforms
// these bodies spill 7 to 11 registers a lane at the bound of two workgroups a
// CU, and wait for each term's words).
template <int LOGN, bool PM, int TERMS, int AHEAD = 2>
__device__ __forceinline__ void inner_sums(uint64_t (&x)[8], const InnerArgs& g, uint64_t i, uint32_t comp, uint32_t m,
                                           const LimbConst& c, int tid) {
  constexpr int E = 8, N = 1 << LOGN;
  const uint32_t L = g.L, L1 = L + 1;
  const bool plain = g.xp && m < L;
  const uint32_t terms = g.nd + (plain ? 1 : 0);
  // Rows are read through buffer resources (the row base in scalar
  // registers, the lane's byte offset fixed, the register's offset 64*k*8 a
  // scalar), so a load costs no per-lane address arithmetic.
  const uint32_t lane = (uint32_t)io_base<3>(tid) * 8;
  const uint64_t* d0 = g.digits + (i * L * L1 + m) * N;
  const uint64_t* k0 = g.ksk + ((uint64_t)comp * L1 + m) * N;
  const uint64_t* dp = nullptr;
  const uint64_t* kp = nullptr;
  if (plain) {
    const uint32_t chain = udiv((uint32_t)i, g.chain), ic = (uint32_t)i - chain * g.chain_cts;
    dp = g.xp + (((uint64_t)ic * 2 + comp) * L + m) * N;
    kp = g.wp + chain * g.w_stride + (uint64_t)m * N;
  }
  const auto rows = [&](uint32_t l, __amdgpu_buffer_rsrc_t& rd, __amdgpu_buffer_rsrc_t& rk) {
    const bool dig = l < g.nd;
    const uint64_t d = dig ? (uint64_t)(d0 + (uint64_t)l * L1 * N) : (uint64_t)dp;
    const uint64_t k = dig ? (uint64_t)(k0 + (uint64_t)l * 2 * L1 * N) : (uint64_t)kp;
    rd = mac_rsrc((const uint64_t*)uniform64(d), (uint64_t)N * 8);
    rk = mac_rsrc((const uint64_t*)uniform64(k), (uint64_t)N * 8);
  };
  if constexpr (PM && TERMS > 0) {
    // Two points at a time, and the operands of AHEAD steps (a step: one term of
    // two points) in flight while one is multiplied: the rows come from beyond
    // L2, and with the loads waited for step by step the waves were idle for
    // half their time (rotation of 256 ciphertexts 271 -> 248 us).  With two
    // steps ahead 12 accumulator and 24 operand registers stand beside x.
    constexpr int G = 2, STEPS = E / G * TERMS;
    uint64_t dv[AHEAD + 1][G], kv[AHEAD + 1][G];
    __amdgpu_buffer_rsrc_t rd[TERMS], rk[TERMS];
#pragma unroll
    for (int l = 0; l < TERMS; l++) rows(l, rd[l], rk[l]);
    const auto issue = [&](int st) {
#pragma unroll
      for (int k = 0; k < G; k++) {
        const uint32_t off = (uint32_t)(64 * (st / TERMS * G + k) * 8);
        dv[st % (AHEAD + 1)][k] = mac_load(rd[st % TERMS], lane, off);
        kv[st % (AHEAD + 1)][k] = mac_load(rk[st % TERMS], lane, off);
      }
    };
#pragma unroll
    for (int st = 0; st < AHEAD && st < STEPS; st++) issue(st);
    uint64_t a00[G], am[G], a11[G];
#pragma unroll
    for (int st = 0; st < STEPS; st++) {
      if (st + AHEAD < STEPS) issue(st + AHEAD);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < G; k++) {
        if (st % TERMS == 0) a00[k] = am[k] = a11[k] = 0;
        const Half30 xs = split30(dv[st % (AHEAD + 1)][k]), ws = split30(kv[st % (AHEAD + 1)][k]);
        a00[k] += (uint64_t)xs.lo * ws.lo;
        am[k] += (uint64_t)xs.lo * ws.hi;
        am[k] += (uint64_t)xs.hi * ws.lo;
        a11[k] += (uint64_t)xs.hi * ws.hi;
        if (st % TERMS == TERMS - 1)
          x[st / TERMS * G + k] = fold3_pm<false>(a00[k], am[k], a11[k], (uint32_t)c.d60, (uint32_t)c.c30);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  } else if constexpr (PM) {
    // any number of terms: four points at a time, 24 accumulator registers
#pragma unroll
    for (int h = 0; h < E; h += 4) {
      uint64_t a00[4], am[4], a11[4];
#pragma unroll
      for (int k = 0; k < 4; k++) a00[k] = am[k] = a11[k] = 0;
      for (uint32_t l = 0; l < terms; l++) {
        __amdgpu_buffer_rsrc_t rd, rk;
        rows(l, rd, rk);
        uint64_t dv[4], kv[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
          dv[k] = mac_load(rd, lane, (uint32_t)(64 * (h + k) * 8));
          kv[k] = mac_load(rk, lane, (uint32_t)(64 * (h + k) * 8));
        }
#pragma unroll
        for (int k = 0; k < 4; k++) {
          const Half30 xs = split30(dv[k]), ws = split30(kv[k]);
          a00[k] += (uint64_t)xs.lo * ws.lo;
          am[k] += (uint64_t)xs.lo * ws.hi;
          am[k] += (uint64_t)xs.hi * ws.lo;
          a11[k] += (uint64_t)xs.hi * ws.hi;
        }
      }
#pragma unroll
      for (int k = 0; k < 4; k++)
        x[h + k] = fold3_pm<false>(a00[k], am[k], a11[k], (uint32_t)c.d60, (uint32_t)c.c30);
    }
  } else {
    // Four points' words in flight: left to the compiler, the 64-register bound
    // made it wait for each pair of words before it issued the next.  Rotation,
    // us, pair by pair -> four points: one ciphertext at N = 2048, L = 2 20.3 ->
    // 17.2, L = 4 24.2 -> 19.8; 256 at N = 8192, L = 3 351 -> 336.
    constexpr int G = 4;
    uint64_t hi[E], lo[E];
#pragma unroll
    for (int k = 0; k < E; k++) hi[k] = lo[k] = 0;
    for (uint32_t l = 0; l < terms; l++) {
      __amdgpu_buffer_rsrc_t rd, rk;
      rows(l, rd, rk);
#pragma unroll
      for (int h = 0; h < E; h += G) {
        uint64_t dv[G], kv[G];
#pragma unroll
        for (int k = 0; k < G; k++) {
          dv[k] = mac_load(rd, lane, (uint32_t)(64 * (h + k) * 8));
          kv[k] = mac_load(rk, lane, (uint32_t)(64 * (h + k) * 8));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < G; k++) {
          uint64_t ph, pl;
          mul_wide(dv[k], kv[k], ph, pl);
          lo[h + k] += pl;
          hi[h + k] += ph + (lo[h + k] < pl);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int k = 0; k < E; k++) x[k] = reduce128(hi[k], lo[k], c);
  }
}

// Inner product fused into the inverse transform: one workgroup per
// (ciphertext i, component c, extended modulus m) forms the sums as it loads
// their operands, transforms back in registers and stores acc[i][c][m].  The
// two workgroups that read the same digit rows run on the same XCD.  Grid:
// ceil(n*(L+1)/8)*8*2 workgroups.
//
// PLAIN: TERMS digits, and a plaintext term where m < L.  AHEAD > 2, for calls
// of at most one workgroup per CU: more loads in flight, in the registers that
// other workgroups would need.  It gains where a workgroup has few waves: a Z_P
// call of 8 diagonals on 8 ciphertexts, L = 3, at N = 1024 105 -> 101 us (two
// steps ahead -> eight), at N = 2048 119 -> 117; at N = 4096 it lost (16
// ciphertexts 179 -> 180, L = 2 178 -> 180) and at N = 8192 it changed nothing.
// ONLY_P: the sums mod P alone (grid ceil(n/8)*8*2), stored centred into
// (-P/2, P/2] as inner_moddown_kernel takes them.
template <int LOGN, bool PM, bool ONLY_P, int TERMS, int AHEAD = 2, bool PLAIN = false>
__global__ __launch_bounds__((1 << LOGN) >> 3, AHEAD > 2 ? 4 : ntt_waves(3)) void inner_intt_kernel(
    InnerArgs g, uint64_t* __restrict__ acc, uint64_t n, const Tw* __restrict__ tw_all,
    const LimbConst* __restrict__ ext) {
  constexpr int LOGE = 3, E = 1 << LOGE, N = 1 << LOGN, T = N / E;
  __shared__ uint64_t lds[N + N / 16];
  const uint32_t L1 = g.L + 1, per = ONLY_P ? 1 : L1;
  const uint32_t xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
  const uint64_t im = (uint64_t)(slot / 2) * 8 + xcd;  // (i, m)
  const uint32_t comp = slot % 2;
  if (im >= n * per) return;  // the whole workgroup leaves before any barrier
  const uint32_t m = ONLY_P ? g.L : (uint32_t)(im % L1);
  const uint64_t i = ONLY_P ? im : im / L1;
  const int tid = threadIdx.x;
  const LimbConst c = ext[m];
  uint64_t x[E];
  if (PLAIN && m < g.L)  // (uniform)
    inner_sums<LOGN, PM, TERMS + 1, AHEAD>(x, g, i, comp, m, c, tid);
  else
    inner_sums<LOGN, PM, TERMS, AHEAD>(x, g, i, comp, m, c, tid);
  ntt_inv_regs<LOGN, LOGE, PM>(x, tw_all + (size_t)m * N, c, lds, tid);
  uint64_t* out = acc + ((i * 2 + comp) * L1 + m) * N;
#pragma unroll
  for (int k = 0; k < E; k++) out[tid + k * T] = ONLY_P && x[k] > c.q / 2 ? x[k] - c.q : x[k];
}

// The same for the ciphertext moduli m < L with the division by P after the
// transform, in registers: with xc the centred residue mod P (acc[i][c][L],
// from inner_intt_kernel<ONLY_P>), y = x*P^-1 - xc*P^-1 mod q_m, where the
// factor P^-1 of x rides on the transform's last products; the stored sums
// mod q_m and moddown_kernel's pass over them fall away.  b (component 1) is
// read through the automorphism from the transform's LDS, staged with
// coalesced loads.  Grid: ceil(n*L/8)*8*2 workgroups.  Signed transforms only.
template <int LOGN, int TERMS>
__global__ __launch_bounds__((1 << LOGN) >> 3, ntt_waves(3)) void inner_moddown_kernel(
    InnerArgs g, const uint64_t* __restrict__ acc, uint64_t n, const Tw* __restrict__ tw_all,
    const LimbConst* __restrict__ ext, const uint64_t* ct, uint64_t* out_, uint32_t ginv, KsConst kc,
    const uint64_t* addp) {
  constexpr int LOGE = 3, E = 1 << LOGE, N = 1 << LOGN, T = N / E;
  __shared__ uint64_t lds[N + N / 16];
  const uint32_t L = g.L, L1 = L + 1;
  const uint32_t xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
  const uint64_t im = (uint64_t)(slot / 2) * 8 + xcd;  // (i, m)
  const uint32_t comp = slot % 2;
  if (im >= n * L) return;  // the whole workgroup leaves before any barrier
  const uint32_t m = (uint32_t)(im % L);
  const uint64_t i = im / L;
  const int tid = threadIdx.x;
  LimbConst c = ext[m];
  c.pninv = kc.ninv[m], c.pninv_w = kc.ninv_w[m];
  uint64_t x[E];
  inner_sums<LOGN, true, TERMS>(x, g, i, comp, m, c, tid);
  ntt_inv_regs<LOGN, LOGE, true, true>(x, tw_all + (size_t)m * N, c, lds, tid);  // |x| < 0.9u
  const PmRegs pk = pm_regs(c);
  const uint64_t* xc = acc + ((i * 2 + comp) * L1 + L) * N + tid;
  const TwP pinv = kc.pinv[m];
#pragma unroll
  for (int k = 0; k < E; k++) x[k] = pm_mul_val(xc[k * T], pinv, pk) - x[k];  // -y, |.| < 1.7u
  const uint64_t row = ((i * 2 + comp) * L + m) * N;
  if (comp && ct) {  // (null: a zero ciphertext)
    const uint64_t* b = ct + row;
    if (ginv == 1) {
#pragma unroll
      for (int k = 0; k < E; k++) x[k] += b[tid + k * T];
    } else {
      // the thread's own entries of the last exchange are rewritten, so only
      // the gather needs a barrier
#pragma unroll
      for (int k = 0; k < E; k++) lds[lds_pad(tid + k * T)] = b[tid + k * T];
      __syncthreads();
#pragma unroll
      for (int k = 0; k < E; k++) {
        const uint32_t src = (uint32_t)(((uint64_t)(tid + k * T) * ginv) & (2 * N - 1));
        const uint64_t v = lds[lds_pad(src & (N - 1))];
        x[k] += src >= (uint32_t)N ? 0 - v : v;
      }
    }
  }
  if (addp) {
#pragma unroll
    for (int k = 0; k < E; k++) x[k] += addp[row + tid + k * T];
  }
  uint64_t* out = out_ + row + tid;
#pragma unroll
  for (int k = 0; k < E; k++) out[k * T] = pm_canon(x[k] + c.pk, c);  // |x| < 3.7u
}

// Galois key for digit l and extended modulus m, in NTT form:
//   ksk[l][0][m] = a[l][m],
//   ksk[l][1][m] = a[l][m]*s + e[l] + (m == l ? P mod q_l : 0) * s(X^g)  (mod p_m),
// since G_l = P * Qhat_l * (Qhat_l^-1 mod q_l) is P mod q_l in limb l and 0
// in every other limb (Qhat_l holds every other q, P is a factor).  Inputs
// are the transforms: work = [a: L][e: L][s][s(X^g)] RNS polynomials of L+1
// limbs.
__global__ __launch_bounds__(ROT_THREADS) void galois_key_kernel(const uint64_t* __restrict__ work,
                                                                  uint64_t* __restrict__ ksk, uint32_t N,
                                                                  uint32_t L, const LimbConst* __restrict__ ext) {
  const uint32_t per_row = N / ROT_THREADS;
  const uint64_t row = blockIdx.x / per_row;  // (l, m)
  const uint32_t k = (blockIdx.x % per_row) * ROT_THREADS + threadIdx.x;
  const uint32_t L1 = L + 1;
  const uint32_t m = (uint32_t)(row % L1), l = (uint32_t)(row / L1);
  const LimbConst c = ext[m];
  const uint64_t LN1 = (uint64_t)L1 * N;
  const uint64_t a = work[row * N + k];
  const uint64_t e = work[L * LN1 + row * N + k];
  const uint64_t sv = work[2 * L * LN1 + (uint64_t)m * N + k];
  uint64_t hi, lo;
  mul_wide(a, sv, hi, lo);
  uint64_t v = csub(reduce128(hi, lo, c) + e, c.q);
  if (m == l) {
    const uint64_t sg = work[(2 * L + 1) * LN1 + (uint64_t)m * N + k];
    mul_wide(red_word(ext[L].q, c), sg, hi, lo);
    v = csub(v + reduce128(hi, lo, c), c.q);
  }
  ksk[((uint64_t)(l * 2 + 0) * L1 + m) * N + k] = a;
  ksk[((uint64_t)(l * 2 + 1) * L1 + m) * N + k] = v;
}

namespace {

hipError_t rows_grid(uint64_t rows, uint32_t N, uint32_t& blocks) {
  const uint64_t b = rows * (N / ROT_THREADS);
  if (b > grid_max_blocks(ROT_THREADS)) return hipErrorInvalidConfiguration;
  blocks = (uint32_t)b;
  return hipSuccess;
}

}  // namespace

hipError_t automorph_launch(const uint64_t* in, uint64_t* out, uint64_t rows, uint32_t N, uint32_t L, uint32_t ginv,
                            const LimbConst* lc, hipStream_t st) {
  uint32_t blocks = 0;
  if (hipError_t e = rows_grid(rows, N, blocks)) return e;
  if (!blocks) return hipSuccess;
  hipLaunchKernelGGL(automorph_kernel, dim3(blocks), dim3(ROT_THREADS), 0, st, in, out, N, L, ginv, lc);
  return hipGetLastError();
}

hipError_t modup_launch(const uint64_t* ct, uint64_t* work, uint64_t n, uint32_t N, uint32_t L, uint32_t ginv,
                        const LimbConst* ext, hipStream_t st) {
  uint32_t blocks = 0;
  if (hipError_t e = rows_grid(n * L * (L + 1), N, blocks)) return e;
  if (!blocks) return hipSuccess;
  hipLaunchKernelGGL(modup_kernel, dim3(blocks), dim3(ROT_THREADS), 0, st, ct, work, N, L, ginv, ext);
  return hipGetLastError();
}

hipError_t ks_inner_launch(const uint64_t* work, const uint64_t* ksk, uint64_t* acc, uint64_t n, uint32_t N,
                           uint32_t L, const LimbConst* ext, hipStream_t st) {
  uint32_t blocks = 0;
  if (hipError_t e = rows_grid(n * (L + 1), N, blocks)) return e;
  if (!blocks) return hipSuccess;
  hipLaunchKernelGGL(ks_inner_kernel, dim3(blocks), dim3(ROT_THREADS), 0, st, work, ksk, acc, N, L, ext);
  return hipGetLastError();
}

hipError_t moddown_launch(const uint64_t* acc, const uint64_t* ct, uint64_t* out, uint64_t n, uint32_t N, uint32_t L,
                          uint32_t ginv, const PinvConst& pinv, const LimbConst* ext, hipStream_t st,
                          const uint64_t* addp) {
  uint32_t blocks = 0;
  if (hipError_t e = rows_grid(n * L, N, blocks)) return e;
  if (!blocks) return hipSuccess;
  hipLaunchKernelGGL(moddown_kernel, dim3(blocks), dim3(ROT_THREADS), 0, st, acc, ct, out, N, L, ginv, pinv, addp, ext);
  return hipGetLastError();
}

// One workgroup of N/8 threads per block of `grid`, in the transforms' form.
#define HECONV_ROT(K, LN, ...)                                                                          \
  do {                                                                                                  \
    if (pm)                                                                                             \
      hipLaunchKernelGGL((K<LN, true>), grid, dim3((1u << LN) / 8), 0, st, __VA_ARGS__);                \
    else                                                                                                \
      hipLaunchKernelGGL((K<LN, false>), grid, dim3((1u << LN) / 8), 0, st, __VA_ARGS__);               \
  } while (0)

bool ks_fwd_supported(uint32_t logN) { return logN >= 10 && logN <= 13; }

hipError_t ks_fwd_launch(uint32_t logN, const uint64_t* ct, const uint64_t* ksk, uint64_t* acc, uint64_t n, uint32_t L,
                         uint32_t ginv, const Tw* tw, const LimbConst* ext, bool pm, hipStream_t st) {
  const uint64_t blocks = (n + 7) / 8 * 8 * (L + 1);
  if (blocks > grid_max_blocks(1024)) return hipErrorInvalidConfiguration;  // up to N/8 = 1024 threads
  if (!blocks) return hipSuccess;
  const dim3 grid((uint32_t)blocks);
  switch (logN) {
    case 10: HECONV_ROT(ks_fwd_kernel, 10, ct, ksk, acc, n, L, ginv, tw, ext); break;
    case 11: HECONV_ROT(ks_fwd_kernel, 11, ct, ksk, acc, n, L, ginv, tw, ext); break;
    case 12: HECONV_ROT(ks_fwd_kernel, 12, ct, ksk, acc, n, L, ginv, tw, ext); break;
    case 13: HECONV_ROT(ks_fwd_kernel, 13, ct, ksk, acc, n, L, ginv, tw, ext); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t modup_ntt_launch(uint32_t logN, const uint64_t* ct, uint64_t* digits, uint64_t n, uint32_t L, uint32_t ginv,
                            const Tw* tw, const LimbConst* ext, bool pm, hipStream_t st) {
  const uint64_t blocks = (n * L + 7) / 8 * 8 * (L + 1);
  if (blocks > grid_max_blocks(1024)) return hipErrorInvalidConfiguration;  // up to N/8 = 1024 threads
  if (!blocks) return hipSuccess;
  const dim3 grid((uint32_t)blocks);
  switch (logN) {
    case 10: HECONV_ROT(modup_ntt_kernel, 10, ct, digits, n, L, ginv, tw, ext); break;
    case 11: HECONV_ROT(modup_ntt_kernel, 11, ct, digits, n, L, ginv, tw, ext); break;
    case 12: HECONV_ROT(modup_ntt_kernel, 12, ct, digits, n, L, ginv, tw, ext); break;
    case 13: HECONV_ROT(modup_ntt_kernel, 13, ct, digits, n, L, ginv, tw, ext); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int LOGN, bool PM, int ND, int AHEAD = 2, bool PLAIN = false>
static void inner_go(const InnerArgs& g, uint32_t blocks, uint64_t* acc, uint64_t n, const Tw* tw_inv,
                     const LimbConst* ext, hipStream_t st) {
  hipLaunchKernelGGL((inner_intt_kernel<LOGN, PM, false, ND, AHEAD, PLAIN>), dim3(blocks), dim3((1u << LOGN) / 8), 0, st,
                     g, acc, n, tw_inv, ext);
}

template <int LOGN, int ND>
static void inner_nd_go(const InnerArgs& g, uint32_t blocks, uint64_t* acc, uint64_t n, const Tw* tw_inv,
                        const LimbConst* ext, hipStream_t st) {
  if constexpr (LOGN <= 11) {
    if (blocks <= 256) {  // at most one workgroup per CU
      if (g.xp) return inner_go<LOGN, true, ND, 8, true>(g, blocks, acc, n, tw_inv, ext, st);
      return inner_go<LOGN, true, ND, 8>(g, blocks, acc, n, tw_inv, ext, st);
    }
  }
  if (g.xp) return inner_go<LOGN, true, ND, 2, true>(g, blocks, acc, n, tw_inv, ext, st);
  inner_go<LOGN, true, ND>(g, blocks, acc, n, tw_inv, ext, st);
}

template <int LOGN>
static void inner_intt_go(bool pm, const InnerArgs& g, uint32_t blocks, uint64_t* acc, uint64_t n, const Tw* tw_inv,
                          const LimbConst* ext, hipStream_t st) {
  if (!pm) return inner_go<LOGN, false, 0>(g, blocks, acc, n, tw_inv, ext, st);
  if (g.nd == 2) return inner_nd_go<LOGN, 2>(g, blocks, acc, n, tw_inv, ext, st);
  if (g.nd == 3) return inner_nd_go<LOGN, 3>(g, blocks, acc, n, tw_inv, ext, st);
  inner_go<LOGN, true, 0>(g, blocks, acc, n, tw_inv, ext, st);
}

hipError_t inner_intt_launch(uint32_t logN, const uint64_t* digits, const uint64_t* ksk, uint64_t* acc, uint64_t n,
                             uint32_t L, uint32_t nd, const uint64_t* xp, const uint64_t* wp, uint64_t chain_cts,
                             uint64_t w_stride, const Tw* tw_inv, const LimbConst* ext, bool pm, hipStream_t st) {
  const InnerArgs g = inner_args(digits, ksk, xp, wp, chain_cts, w_stride, L, nd);
  const uint64_t blocks = (n * (L + 1) + 7) / 8 * 8 * 2;
  if (blocks > grid_max_blocks(1024)) return hipErrorInvalidConfiguration;  // up to N/8 = 1024 threads
  if (!blocks) return hipSuccess;
  switch (logN) {
    case 10: inner_intt_go<10>(pm, g, (uint32_t)blocks, acc, n, tw_inv, ext, st); break;
    case 11: inner_intt_go<11>(pm, g, (uint32_t)blocks, acc, n, tw_inv, ext, st); break;
    case 12: inner_intt_go<12>(pm, g, (uint32_t)blocks, acc, n, tw_inv, ext, st); break;
    case 13: inner_intt_go<13>(pm, g, (uint32_t)blocks, acc, n, tw_inv, ext, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int LOGN, int TERMS>
static void inner_p_go(const InnerArgs& g, uint64_t* acc, uint64_t n, const Tw* tw_inv, const LimbConst* ext,
                       hipStream_t st) {
  hipLaunchKernelGGL((inner_intt_kernel<LOGN, true, true, TERMS>), dim3((uint32_t)((n + 7) / 8 * 8 * 2)),
                     dim3((1u << LOGN) / 8), 0, st, g, acc, n, tw_inv, ext);
}

template <int LOGN, int TERMS>
static void inner_q_go(const InnerArgs& g, uint64_t* acc, uint64_t n, const Tw* tw_inv, const LimbConst* ext,
                       const uint64_t* ct, uint64_t* out, uint32_t ginv, const KsConst& kc, const uint64_t* addp,
                       hipStream_t st) {
  hipLaunchKernelGGL((inner_moddown_kernel<LOGN, TERMS>), dim3((uint32_t)((n * g.L + 7) / 8 * 8 * 2)),
                     dim3((1u << LOGN) / 8), 0, st, g, acc, n, tw_inv, ext, ct, out, ginv, kc, addp);
}

// The sums mod P take the digits alone; the others the plaintext term too.
template <int LOGN>
static void inner_moddown_go(const InnerArgs& g, uint64_t* acc, uint64_t n, const Tw* tw_inv, const LimbConst* ext,
                             const uint64_t* ct, uint64_t* out, uint32_t ginv, const KsConst& kc, const uint64_t* addp,
                             hipStream_t st) {
  const uint32_t terms = g.nd + (g.xp ? 1 : 0);
  if (g.nd == 2)
    inner_p_go<LOGN, 2>(g, acc, n, tw_inv, ext, st);
  else if (g.nd == 3)
    inner_p_go<LOGN, 3>(g, acc, n, tw_inv, ext, st);
  else
    inner_p_go<LOGN, 0>(g, acc, n, tw_inv, ext, st);
  if (terms == 2)
    inner_q_go<LOGN, 2>(g, acc, n, tw_inv, ext, ct, out, ginv, kc, addp, st);
  else if (terms == 3)
    inner_q_go<LOGN, 3>(g, acc, n, tw_inv, ext, ct, out, ginv, kc, addp, st);
  else if (terms == 4)
    inner_q_go<LOGN, 4>(g, acc, n, tw_inv, ext, ct, out, ginv, kc, addp, st);
  else
    inner_q_go<LOGN, 0>(g, acc, n, tw_inv, ext, ct, out, ginv, kc, addp, st);
}

hipError_t inner_moddown_launch(uint32_t logN, const uint64_t* digits, const uint64_t* ksk, uint64_t* acc, uint64_t n,
                                uint32_t L, uint32_t nd, const uint64_t* xp, const uint64_t* wp, uint64_t chain_cts,
                                uint64_t w_stride, const Tw* tw_inv, const LimbConst* ext, const uint64_t* ct,
                                uint64_t* out, uint32_t ginv, const KsConst& kc, const uint64_t* addp,
                                hipStream_t st) {
  const InnerArgs g = inner_args(digits, ksk, xp, wp, chain_cts, w_stride, L, nd);
  if ((n * L + 7) / 8 * 8 * 2 > grid_max_blocks(1024)) return hipErrorInvalidConfiguration;
  if (!n) return hipSuccess;
  switch (logN) {
    case 10: inner_moddown_go<10>(g, acc, n, tw_inv, ext, ct, out, ginv, kc, addp, st); break;
    case 11: inner_moddown_go<11>(g, acc, n, tw_inv, ext, ct, out, ginv, kc, addp, st); break;
    case 12: inner_moddown_go<12>(g, acc, n, tw_inv, ext, ct, out, ginv, kc, addp, st); break;
    case 13: inner_moddown_go<13>(g, acc, n, tw_inv, ext, ct, out, ginv, kc, addp, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t galois_key_launch(const uint64_t* work, uint64_t* ksk, uint32_t N, uint32_t L, const LimbConst* ext,
                             hipStream_t st) {
  uint32_t blocks = 0;
  if (hipError_t e = rows_grid((uint64_t)L * (L + 1), N, blocks)) return e;
  hipLaunchKernelGGL(galois_key_kernel, dim3(blocks), dim3(ROT_THREADS), 0, st, work, ksk, N, L, ext);
  return hipGetLastError();
}

#undef HECONV_ROT

}  // namespace heconv
