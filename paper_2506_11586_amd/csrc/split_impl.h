// The parts of a transform split over two grids (ntt_split.hip) that other
// kernels take too: the stages within blocks of G = N/64 consecutive indexes,
// by workgroups of 128 threads on 1024 consecutive elements.  All their
// mappings lie at or below bit 6 (N <= 2^14), so every exchange stays inside
// a wave.
#pragma once
#include "ntt_impl.h"

namespace heconv {

constexpr int SPLIT_T = 128;  // threads per workgroup (8 words each)

// Forward stages on bits n-7 .. 0 of one 1024-element block, from the mapping
// at LO = n-9 to that at 0.
template <int LOGN, int P, bool PM>
__device__ __forceinline__ void split_b_rest(uint64_t (&x)[8], uint64_t* lds, int tid, const Tw* __restrict__ tw,
                                             const LimbConst& c, const PmRegs& pk, uint32_t jb) {
  constexpr int NB = LOGN - 6;  // stages in this grid
  constexpr int NFULL = NB / 3, REM = NB % 3;
  if constexpr (P < NFULL || (P == NFULL && REM > 0)) {
    constexpr int LO = P < NFULL ? NB - 3 * (P + 1) : 0, U0 = P < NFULL ? 0 : 3 - REM;
    PassTw<LOGN, 3, LO, U0, PM> t;
    t.load(tid, tw, jb);
    if constexpr (P > 0) exchange<3, NB - 3 * P, LO>(lds, x, tid);
    fwd_pass<(P == 0)>(x, t, c, pk);
    split_b_rest<LOGN, P + 1, PM>(x, lds, tid, tw, c, pk, jb);
  }
}

// Inverse stages on bits 0 .. n-7 of one 1024-element block, from the mapping at
// PREV (P = -1 first where (n-6) % 3 > 0, else 0).
template <int LOGN, int P, int PREV, bool PM>
__device__ __forceinline__ void inv_split_c_rest(uint64_t (&x)[8], uint64_t* lds, int tid,
                                                 const Tw* __restrict__ tw, const LimbConst& c,
                                                 const PmRegs& pk, uint32_t jb) {
  constexpr int NB = LOGN - 6, NFULL = NB / 3, REM = NB % 3;
  if constexpr (P < NFULL) {
    constexpr int LO = P < 0 ? 0 : REM + 3 * P, U0 = P < 0 ? 3 - REM : 0;
    PassTw<LOGN, 3, LO, U0, PM> t;
    t.load(tid, tw, jb);
    exchange<3, PREV, LO>(lds, x, tid);
    inv_pass<false>(x, t, c, pk);
    inv_split_c_rest<LOGN, P + 1, LO, PM>(x, lds, tid, tw, c, pk, jb);
  }
}

}  // namespace heconv
