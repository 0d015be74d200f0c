// rwpt_epilogue.h -- what the pair kernels share around their sums (internal
// to the HIP kernels): the block order, the fixed-order lane reductions, and
// the update, reaction and audit partials of a tile.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rwpt_device.h"
#include "rwpt_layout.h"

namespace rwpt {

// Wave-uniform block index -> logical block so that each of the 8 XCDs (which
// receive workgroups round-robin) works on one contiguous range of tiles and
// neighbouring tiles share that XCD's L2.
__device__ __forceinline__ int xcd_block(int b, int nb) {
  const int per = nb >> 3, rem = nb & 7;
  const int x = b & 7, q = b >> 3;
  return x * per + (x < rem ? x : rem) + q;
}

// Block of a pair kernel -> logical block: the XCDs take groups of
// kXcdGroup consecutive blocks in turn, so that neighbouring tiles still share an
// L2 and every XCD gets a like share of dense and sparse regions.  One
// contiguous eighth each leaves the XCDs whose realisations are sparse idle:
// a step of 64 realisations of 2 to 450 neighbours 1.58 -> 1.21 ms; one uniform one
// of 1e6 particles 0.379 -> 0.375.  Groups of 8, 16, 32, 64 and 512 blocks: the
// former 0.374, 0.375, 0.376, 0.377, 0.378 ms, the batch 1.21 up to 64, 1.32 with 512.
// The blocks after the last whole round are shared out as xcd_block does.
// One lane per particle in 1-D and 2-D, where a block's vertical neighbours are
// thousands of particles away and every cell row gathers from several: groups of
// 256 (2e6 particles of 16 neighbours, a step in groups of 16, 64, 256 blocks and
// contiguous eighths 399, 371, 349, 348 us, in binary64 545, 496, 470, 461; 8e6 in 3-D 648,
// 648, 655, 669).  The kernels of other tilings alike: 256 with 8 and 16 lanes (16, 64, 256,
// eighths: 2e6 of 12 560, 556, 532, 522; 854, 868, 840, 808), 64 with 1 and 4 (1e6 of 30 475,
// 406, 388, 374), whose clusters larger ones leave on few XCDs (2e5 of 30, a third in a
// box of 0.02, one lane 5242, 5372, 7355, 7383 us, four in binary64 4931, 5487, 8543, 13975).
// Fewer blocks take smaller groups, for the same reason and because what they read
// stays in the L2s.
constexpr int kXcdGroup = 16;
constexpr int kXcdGroupWide = 64, kXcdGroupWideBlocks = 1024;  // from so many blocks
constexpr int kXcdGroupWidest = 256, kXcdGroupWidestBlocks = 4096;
template <int DIM>
constexpr int kXcdGroupSparse = DIM < 3 ? kXcdGroupWidest : kXcdGroup;
template <int LOG2L>
constexpr int kXcdGroupLanes = LOG2L >= 3 ? kXcdGroupWidest : kXcdGroupWide;
template <int GROUP>
__device__ __forceinline__ int xcd_group_block(int b, int nb) {
  int log2g = 4;
  if (GROUP > kXcdGroup && nb >= kXcdGroupWideBlocks) log2g = 6;
  if (GROUP > kXcdGroupWide && nb >= kXcdGroupWidestBlocks) log2g = 8;
  const int R = 8 << log2g;
  const int whole = nb & -R;
  if (b >= whole) return whole + xcd_block(b - whole, nb - whole);
  const int o = b & (R - 1);
  return b - o + ((o & 7) << log2g) + (o >> 3);
}

// Exchange of a double with lane ^ M: a DPP quad permutation for M = 1, 2
// (no LDS traffic), a cross-lane permute otherwise.
template <int M>
__device__ __forceinline__ double xor_shfl(double v) {
  if constexpr (M == 1 || M == 2) {
    constexpr int ctrl = M == 1 ? 0xB1 : 0x4E;  // quad_perm [1,0,3,2] / [2,3,0,1]
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, ctrl, 0xF, 0xF, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), ctrl, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
  } else {
    return __shfl_xor(v, M);
  }
}

// Sum of NV values over each aligned group of G lanes by recursive halving (a
// reduce-scatter): at step M every lane keeps one half of its values, adds the
// partner's (lane ^ M) copy of that half, and hands over the other half, so
// the number of values exchanged halves at every step; once one value is
// left, the remaining steps add it up plainly.  On return v[0 .. NK) holds the
// group totals of values idx .. idx + NK - 1, and lanes that differ only in
// the bits above the first NB (the halving steps) hold the same totals.  An
// upper half shorter than the lower one is padded with zeros; `real` counts
// the lane's values that are not padding (only those may be written out).
constexpr int halved_count(int n, int g) {
  for (int m = 1; m < g && n > 1; m <<= 1) n = (n + 1) / 2;
  return n;
}
constexpr int halving_bits(int n, int g) {
  int b = 0;
  for (int m = 1; m < g && n > 1; m <<= 1) {
    n = (n + 1) / 2;
    ++b;
  }
  return b;
}

template <int M, int G, int N, int NV>
__device__ __forceinline__ void halve_sum(double (&v)[NV], int& idx, int& real, int lane) {
  if constexpr (M < G) {
    if constexpr (N > 1) {
      constexpr int H = (N + 1) / 2;
      const bool up = (lane & M) != 0;
#pragma unroll
      for (int k = 0; k < H; ++k) {
        double hi = 0.0;
        if (k + H < N) hi = v[k + H];
        const double keep = up ? hi : v[k];
        const double send = up ? v[k] : hi;
        v[k] = keep + xor_shfl<M>(send);
      }
      idx += up ? H : 0;
      real = up ? (real > H ? real - H : 0) : (real < H ? real : H);
      halve_sum<M * 2, G, H, NV>(v, idx, real, lane);
    } else {
      v[0] += xor_shfl<M>(v[0]);
      halve_sum<M * 2, G, 1, NV>(v, idx, real, lane);
    }
  }
}

// After the lane reductions: new masses (Eq. 6), reaction, and the tile's
// audit partials.  `writer` lanes (one per particle) hold acc / racc; lanes
// 0..G-1 are the writers' first copies, so the audit is reduced over them.
template <typename T, int SMAX, int G>
__device__ __forceinline__ void exchange_epilogue(const RealParams& P, bool sym, const double acc[SMAX],
                                                  double racc, const T Mi[SMAX], bool writer, int32_t i,
                                                  T* __restrict__ mout, int S, int react_a,
                                                  int react_b, double* __restrict__ audit_part, const OutMap& om,
                                                  int64_t t) {
  double tot[SMAX + 1];
#pragma unroll
  for (int s = 0; s <= SMAX; ++s) tot[s] = 0.0;
  if (writer) {
    double Mn[SMAX];
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
      double dm = 0.0;
      if (P.active) dm = sym ? 0.25 * acc[s] : 0.5 * acc[s] / racc;
      Mn[s] = (double)Mi[s] + dm;
    }
    // the reacting pair by its slot indices (uniform, < S <= SMAX: indexed
    // register moves, not a select over every slot)
    if (react_a >= 0) {
      const double A = Mn[react_a], B = Mn[react_b];
      double m = A < B ? A : B;
      m = m > 0.0 ? m : 0.0;
      Mn[react_a] = A - m;
      Mn[react_b] = B - m;
    }
    T out[SMAX];
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
      out[s] = s < S ? (T)Mn[s] : (T)0;  // unused species slots stay zero
      tot[s] = (double)out[s];
    }
    if (om.id) {
      const uint32_t o = om.id[i];
#pragma unroll
      for (int s = 0; s < SMAX; ++s)
        if (s < S) mout[(int64_t)s * om.n + o] = out[s];
    } else {
      store_mass<T, SMAX>(mout, i, out);
    }
    tot[SMAX] = react_a >= 0 ? tot[react_a] - tot[react_b] : 0.0;
  }
  // totals over lanes 0..G-1 (the other lanes hold zeros and are reduced
  // among themselves); value SMAX is sum(A - B)
  constexpr int NV = SMAX + 1, NK = halved_count(NV, G), NB = halving_bits(NV, G);
  const int lane = threadIdx.x & 63;
  int idx = 0, real = NV;
  halve_sum<1, G, NV, NV>(tot, idx, real, lane);
  if (lane < (1 << NB)) {
    double* part = audit_part + t * (S + 1);
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const int vi = idx + k;
      if (k < real) {
        if (vi < S) part[vi] = tot[k];
        else if (vi == SMAX) part[S] = tot[k];
      }
    }
  }
}

}  // namespace rwpt
