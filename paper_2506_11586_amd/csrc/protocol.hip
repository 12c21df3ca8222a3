// The server's steps either side of the layer in the online protocol for a
// linear layer (Sec. 7; extraction of the sparse results, Sec. 6.2):
//   add_share:    b_l += delta_l * pack(share) mod q_l on the client's input
//                 ciphertexts (coefficient form), before the forward NTT;
//   mask_extract: after the inverse NTT, gather only the b coefficients that
//                 hold outputs, minus delta_l * mask, plus a signed smudging
//                 term, into a dense [B][M][L][Ho][Wo] array.
// One thread per coefficient (add_share) or output position (mask_extract) for
// all L limbs, consecutive threads on consecutive words.  Both move few bytes,
// so what bounds them is the index arithmetic and the reduction mod t: those
// divide by multiplications (udiv.h, and t's Shoup reduction) and run once
// for the limbs.  7 images of the 32->128 3x3 layer at 27x27: mask_extract
// 18.1 -> 11.4 us (41 MB at 3.6 TB/s), add_share 6.3 -> 5.3 us, against one thread per limb with
// integer divisions and a 64-bit remainder.
#include "kernels.h"
#include "udiv.h"

namespace heconv {

constexpr uint32_t PROTO_THREADS = 256;

// Divisors of a launch whose dividends are below 2^31 (a grid has fewer than
// 2^24 blocks, a layer's rows and columns fewer than 2^23).
struct ProtoDivs {
  UDiv per_ct, S, CB, HW, Ww, nsj;  // add_share
  UDiv bh, bw;                      // mask_extract
};

static ProtoDivs proto_divs(const ProtoGeom& g) {
  return ProtoDivs{udiv_make(g.N / PROTO_THREADS), udiv_make(g.S),   udiv_make(g.CB), udiv_make(g.Hw * g.Ww),
                   udiv_make(g.Ww),                udiv_make(g.nsj), udiv_make(g.bh), udiv_make(g.bw)};
}

// v mod t in [0, t) for a signed value (2 <= t <= 2^62), tmu = floor(2^64 / t).
__device__ __forceinline__ uint64_t mod_t(int64_t v, uint64_t t, uint64_t tmu) {
  const uint64_t mag = v < 0 ? 0ull - (uint64_t)v : (uint64_t)v;
  const uint64_t r = csub(reduce64_lazy(mag, tmu, t), t);
  return v < 0 && r ? t - r : r;
}

// v mod q in [0, q) for a signed value, via the Shoup reduction by 1.
__device__ __forceinline__ uint64_t mod_q_signed(int64_t v, const LimbConst& c) {
  const uint64_t mag = v < 0 ? 0ull - (uint64_t)v : (uint64_t)v;
  const uint64_t r = csub(reduce64_lazy(mag, c.mu64, c.q), c.q);
  return v < 0 && r ? c.q - r : r;
}

__global__ __launch_bounds__(PROTO_THREADS) void add_share_kernel(uint64_t* __restrict__ in_,
                                                                  const int64_t* __restrict__ share, ProtoGeom g,
                                                                  ProtoDivs dv, const LimbConst* __restrict__ lcs) {
  gword* in = as_global(in_);
  const uint32_t per_ct = g.N / PROTO_THREADS;
  const uint32_t ct = udiv(blockIdx.x, dv.per_ct);  // (b, cb, s)
  const uint32_t k = (blockIdx.x - ct * per_ct) * PROTO_THREADS + threadIdx.x;
  const uint32_t bcb = udiv(ct, dv.S), s = ct - bcb * g.S, b = udiv(bcb, dv.CB), cb = bcb - b * g.CB;
  // packed position -> padded (and, for a strided 1x1 conv, subsampled) input
  const uint32_t HW = g.Hw * g.Ww;
  const uint32_t cc = udiv(k, dv.HW), rem = k - cc * HW, i = udiv(rem, dv.Ww), j = rem - i * g.Ww;
  const uint32_t c = cb * g.Cw + cc;
  const uint32_t si = udiv(s, dv.nsj), sj = s - si * g.nsj;
  const uint32_t pr = si * g.bh + i, pc = sj * g.bw + j;
  uint64_t m = 0;
  if (cc < g.Cw && c < g.C && pr < g.He && pc < g.We) {
    const int64_t y = (int64_t)pr * g.step - g.pad, x = (int64_t)pc * g.step - g.pad;
    if (y >= 0 && y < g.H && x >= 0 && x < g.W)
      m = mod_t(share[(((uint64_t)b * g.C + c) * g.H + y) * g.W + x], g.t, g.tmu);
  }
  gword* bp = in + ((uint64_t)ct * 2 + 1) * g.L * g.N + k;
  for (uint32_t l = 0; l < g.L; l++) {
    const LimbConst lc = lcs[l];
    const uint64_t d = csub(mul_shoup_lazy(m, lc.delta, lc.delta_sh, lc.q), lc.q);
    bp[(uint64_t)l * g.N] = csub(bp[(uint64_t)l * g.N] + d, lc.q);
  }
}

// n output positions (b, m, oy, ox), n < 2^32.
__global__ __launch_bounds__(PROTO_THREADS) void mask_extract_kernel(const uint64_t* __restrict__ out_,
                                                                     const int64_t* __restrict__ mask,
                                                                     const int64_t* __restrict__ noise,
                                                                     uint64_t* __restrict__ y_, ProtoGeom g,
                                                                     ProtoDivs dv, uint32_t n,
                                                                     const LimbConst* __restrict__ lcs) {
  cgword* out = as_global(out_);
  gword* y = as_global(y_);
  const uint32_t HoWo = g.Ho * g.Wo;
  const uint32_t slot = blockIdx.x * PROTO_THREADS + threadIdx.x;
  if (slot >= n) return;
  const uint32_t bm = slot / HoWo, pos = slot - bm * HoWo;
  const uint32_t oy = pos / g.Wo, ox = pos - oy * g.Wo;
  const uint32_t r = oy * g.ostep, cl = ox * g.ostep;  // stride-1 output position
  const uint32_t si = udiv(r, dv.bh), i = r - si * g.bh, sj = udiv(cl, dv.bw), j = cl - sj * g.bw;
  const uint32_t s = si * g.nsj + sj, k = g.O + i * g.Ww + j;
  cgword* b = out + (((uint64_t)bm * g.S + s) * 2 + 1) * g.L * g.N + k;
  gword* yp = y + (uint64_t)bm * g.L * HoWo + pos;
  const uint64_t m = mod_t(mask[slot], g.t, g.tmu);
  for (uint32_t l = 0; l < g.L; l++) {
    const LimbConst lc = lcs[l];
    const uint64_t dm = csub(mul_shoup_lazy(m, lc.delta, lc.delta_sh, lc.q), lc.q);
    uint64_t v = csub(b[(uint64_t)l * g.N] + (lc.q - dm), lc.q);
    if (noise) v = csub(v + mod_q_signed(noise[slot], lc), lc.q);
    yp[(uint64_t)l * HoWo] = v;
  }
}

hipError_t add_share_launch(uint64_t* in, const int64_t* share, const ProtoGeom& g, const LimbConst* lc,
                            hipStream_t st) {
  const uint64_t blocks = (uint64_t)g.B * g.CB * g.S * (g.N / PROTO_THREADS);
  if (blocks == 0) return hipSuccess;
  if (blocks > grid_max_blocks(PROTO_THREADS)) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(add_share_kernel, dim3((uint32_t)blocks), dim3(PROTO_THREADS), 0, st, in, share, g,
                     proto_divs(g), lc);
  return hipGetLastError();
}

hipError_t mask_extract_launch(const uint64_t* out, const int64_t* mask, const int64_t* noise, uint64_t* y,
                               const ProtoGeom& g, const LimbConst* lc, hipStream_t st) {
  const uint64_t HoWo = (uint64_t)g.Ho * g.Wo, rows = (uint64_t)g.B * g.M;
  // what is taken: fewer than 2^32 output values, each row in whole blocks
  const uint64_t bound = rows * g.L * ((HoWo + PROTO_THREADS - 1) / PROTO_THREADS);
  if (bound == 0) return hipSuccess;
  if (bound > grid_max_blocks(PROTO_THREADS)) return hipErrorInvalidConfiguration;
  const uint32_t n = (uint32_t)(rows * HoWo);
  hipLaunchKernelGGL(mask_extract_kernel, dim3((uint32_t)((rows * HoWo + PROTO_THREADS - 1) / PROTO_THREADS)),
                     dim3(PROTO_THREADS), 0, st, out, mask, noise, y, g, proto_divs(g), n, lc);
  return hipGetLastError();
}

}  // namespace heconv
