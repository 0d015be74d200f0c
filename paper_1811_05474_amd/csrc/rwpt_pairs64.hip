// rwpt_pairs64.hip -- binary64 pair kernels of the vector-load tiles (8 or 16
// lanes per particle), for cutoffs up to kappa^2 = kWideCutoff.
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "rwpt_cursor.h"
#include "rwpt_epilogue.h"
#include "rwpt_kernels.h"
#include "rwpt_layout.h"
#include "rwpt_pairstep.h"

namespace rwpt {

// exp(-s2 / sigma^2) for exponents down to -kWideCutoff: t = s2 esc64 counts
// 64ths of a binary octave (esc64 = -64 log2(e) / sigma^2, rounded once from
// the host's extended precision).  fma(s2, esc64, 1.5 * 2^52) leaves round(t)
// in the low word, and a second fma gives f = t - round(t) with one rounding:
// no reduction in two parts, conversion or ldexp.  Then 2^(f / 64) - 1 =
// f (c1 + f (c2 + ...)), c_n = (ln2 / 64)^n / n!, |f| <= 1/2, truncated below
// 2^-54, times the table entry.  tbl[j] is 2^(j / 64) with j << 14 taken off its
// high word, so that adding round(t) << 14 puts the octave into the exponent.
// 9 binary64 and 3 integer operations; exp_tab needs 17, of which the rounding,
// the conversion and the ldexp are not at full rate.  Larger s2 / sigma^2 give
// garbage, which the caller's predicate discards.
struct Weight64 {
  const double* tbl;
  double esc64, c5;
  static constexpr double kRound = 0x1.8p52;
  static constexpr double kC1 = 0x1.62e42fefa39efp-7;   // ln2 / 64
  static constexpr double kC2 = 0x1.ebfbdff82c58fp-15;  // its powers over n!
  static constexpr double kC3 = 0x1.c6b08d704a0c0p-23;
  static constexpr double kC4 = 0x1.3b2ab6fba4e77p-31;
  static constexpr double kC5 = 0x1.5d87fe78a6731p-40;
  __device__ __forceinline__ void init(const double* t, double esc) {
    tbl = t;
    esc64 = esc;
    c5 = kC5;
    asm("" : "+v"(c5));  // one of two constants of an fma has to be in vector registers
  }
  // fills the 64 entries, one per thread
  __device__ __forceinline__ static void fill(double* t, int k) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, kExp2Frac[k]);
    t[k] = __builtin_bit_cast(double, b - ((unsigned long long)k << 46));
  }
  // p f + c with c in scalar registers (left to itself the compiler copies the
  // constant into the accumulator of a two-operand fmac, one more instruction
  // per term)
  __device__ __forceinline__ static double fma_sc(double p, double f, double c) {
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(p), "v"(f), "s"(c));
    return d;
  }
  __device__ __forceinline__ double operator()(double s2) const {
    double z, f;
    z = __builtin_fma(s2, esc64, kRound);
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(f) : "v"(s2), "s"(esc64), "v"(kRound - z));
    const uint32_t k = (uint32_t)__builtin_bit_cast(unsigned long long, z);
    double p = fma_sc(c5, f, kC4);
    p = fma_sc(p, f, kC3);
    p = fma_sc(p, f, kC2);
    p = fma_sc(p, f, kC1);
    const uint2 b = *(const uint2*)&tbl[k & 63u];
    uint32_t hi;
    asm("v_lshl_add_u32 %0, %1, 14, %2" : "=v"(hi) : "v"(k), "v"(b.y));  // kept in 32 bits
    const double e = __builtin_bit_cast(double, ((unsigned long long)hi << 32) | b.x);
    const double pf = p * f;
    double w;
    asm("v_fma_f64 %0, %1, %2, %1" : "=v"(w) : "v"(e), "v"(pf));
    return w;
  }
};

// s^2 in the cutoff predicate's arithmetic (sep2v of the other kernels).
template <int DIM>
__device__ __forceinline__ double sep2_64(const double (&xi)[DIM], const double (&xj)[DIM]) {
#pragma clang fp contract(off)
  const double d0 = xj[0] - xi[0];
  double s = d0 * d0;
  if constexpr (DIM > 1) {
    const double d1 = xj[1] - xi[1];
    s = __builtin_fma(d1, d1, s);
  }
  if constexpr (DIM > 2) {
    const double d2 = xj[2] - xi[2];
    s = __builtin_fma(d2, d2, s);
  }
  return s;
}

// A wave takes PP consecutive tiles of G = 64 / L particles of one
// realisation, PP particles per lane and L lanes per particle.  The candidates
// of a segment (a run of its particles in one cell row) come as one virtual
// list over the stencil rows, 64 at a time: each lane loads one, a chunk ahead
// of its use, and they pass through LDS, from which lane gl of a particle
// takes every L-th.  So a short row costs no idle lanes and no latency of its
// own, and a load serves 64 / L * PP pairs.  Bound by the issue of binary64
// arithmetic: 18 (row sums) and 23 (exchange) instructions per pair.
// PP = 2 halves the LDS reads per pair for 12 % more candidates.
// 1e6 particles of 225 neighbours: row sums 339 -> 246 us, exchange 559 -> 331
// us; per-row vector loads with exp_tab before (with an early form of this
// weight and PP = 2: 340 and 474).  PP = 1: 282 and 355; PP = 4: 238 and 329, but
// 32 and 38 us at 1e5 particles against 28 and 34.
// MODE 0: row sums; 1: exchange, symmetric; 2: exchange, row normalisation.
template <int DIM, int SMAX, int LOG2L, int PP, int MODE>
__global__ __launch_bounds__(kBlock) void k_pairs64(const PairArgs a) {
  constexpr int L = 1 << LOG2L, G = 64 >> LOG2L, N = G * PP, W = kBlock / 64;
  __shared__ double tbl[64];
  __shared__ __attribute__((aligned(16))) double sh_x[W][64 * DIM];
  __shared__ double sh_q[W][MODE == 1 ? 64 : 1];
  __shared__ __attribute__((aligned(32))) double sh_m[W][MODE == 0 ? 4 : 64 * SMAX];
  if (threadIdx.x < 64) Weight64::fill(tbl, threadIdx.x);
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w = xcd_group_block<kXcdGroup>(blockIdx.x, gridDim.x) * W + wave;
  int tile = w, nt = 1;
  if constexpr (PP > 1) {
    if (w >= a.group_nitems) return;
    if (a.group_items) {
      const TileGroup it = a.group_items[w];
      tile = it.tile;
      nt = it.ntiles;
    } else {  // one realisation
      tile = w * PP;
      nt = a.ntiles - tile < PP ? a.ntiles - tile : PP;
    }
  } else if (w >= a.ntiles) {
    return;
  }
  const Tile first = a.tiles[tile];
  const int32_t begin = first.begin, n_in = a.tiles[tile + nt - 1].end - begin;
  const RealParams& R = a.rp[first.real];
  const double* __restrict__ pos = (const double*)a.pos;
  const double* __restrict__ min_ = (const double*)a.mass_in;
  const double* __restrict__ q = (const double*)a.q_in;
  const int gi = lane & (G - 1), gl = lane >> (6 - LOG2L);
  // the cell of particle lane & (N - 1), for the segments
  const int lp = lane & (N - 1);
  const uint32_t lk = a.skey[begin + (lp < n_in ? lp : n_in - 1)] - (uint32_t)R.cell_off;
  const int nc1 = R.nc[1];
  const int cx = (int)(lk % (uint32_t)R.nc[0]), row = (int)(lk / (uint32_t)R.nc[0]);
  double xi[PP][DIM], Mi[PP][SMAX], qi[PP], acc[PP][SMAX], racc[PP];
#pragma unroll
  for (int p = 0; p < PP; ++p) {
    const int o = gi + p * G;
    const int32_t ip = begin + (o < n_in ? o : n_in - 1);
    load_pos<double, DIM>(pos, ip, xi[p]);
#pragma unroll
    for (int s = 0; s < SMAX; ++s) Mi[p][s] = 0.0;
    if constexpr (MODE != 0) load_mass<double, SMAX>(min_, ip, Mi[p]);
    qi[p] = MODE == 1 ? q[ip] : 0.0;
    racc[p] = 0.0;
#pragma unroll
    for (int s = 0; s < SMAX; ++s) acc[p][s] = 0.0;
  }
  if (R.active) {
    Weight64 wfn;
    wfn.init(tbl, R.esc64_d);
    int seg = 0;
    while (seg < n_in) {
      const int seg_row = __builtin_amdgcn_readlane(row, seg);
      const unsigned long long m = __ballot(lane < N && lane > seg && (lane >= n_in || row != seg_row));
      int seg_end = m ? (__ffsll(m) - 1) : n_in;
      seg_end = seg_end > n_in ? n_in : seg_end;
      const int cxa = __builtin_amdgcn_readlane(cx, seg), cxb = __builtin_amdgcn_readlane(cx, seg_end - 1);
      // no s^2 is below the cutoff of a particle outside the segment
      double rc2[PP];
#pragma unroll
      for (int p = 0; p < PP; ++p) {
        const int o = gi + p * G;
        rc2[p] = o >= seg && o < seg_end ? R.rc2_d : -1.0;
      }
      const int cy = seg_row % nc1, cz = seg_row / nc1;
      RowTable tab;
      const bool table = PP == 1 && R.n_stencil <= RowTable::kRows;
      if (table) tab.load(R, a.st, a.cell_start, cy, cz, cxa, cxb);
      auto advance = [&](RowCursor& k) {
        if (table) tab.advance(k, R);
        else cursor_advance(k, R, a.st, a.cell_start, cy, cz, cxa, cxb);
      };
      RowCursor c;
      c.r = 0;
      c.p = 0;
      advance(c);
      double xn[DIM], qn = 0.0, mn[SMAX];
      uint32_t vbase = 0;
      int count = 0;  // candidates of the chunk in xn, qn, mn
      auto fetch = [&]() {
        int32_t j;
        bool has;
        chunk_pick(c, advance, vbase, begin, j, has);
        count = c.valid ? 64 : (int)__builtin_amdgcn_readfirstlane(c.p - vbase);
        vbase += 64;
        load_pos<double, DIM>(pos, j, xn);
        if constexpr (MODE == 1) qn = q[j];
        if constexpr (MODE != 0) load_mass<double, SMAX>(min_, j, mn);
        if (!has) xn[0] = 1e300;  // s^2 is infinite
      };
      if (c.valid) fetch();
      while (count > 0) {
        wave_lds_fence();  // the loads of the previous chunk stay before these stores
        store_pos<double, DIM>(sh_x[wave], lane, xn);
        if constexpr (MODE == 1) sh_q[wave][lane] = qn;
        if constexpr (MODE != 0) store_mass<double, SMAX>(sh_m[wave], lane, mn);
        wave_lds_fence();
        const int steps = (count + L - 1) >> LOG2L;
        count = 0;
        if (c.valid) fetch();
        // H steps' LDS reads together (row sums 28 -> 24 us at 1e5 particles with
        // two; the exchange, which has more of them, is slower with two); past
        // the chunk's end the entries are those of lanes without a candidate
        constexpr int H = MODE == 0 ? 2 : 1;
        for (int k = 0; k < steps; k += H) {
          double xj[H][DIM], mj[H][SMAX], qj[H], s2[H][PP];
#pragma unroll
          for (int h = 0; h < H; ++h) {
            const int e = ((k + h) << LOG2L) + gl;
            load_pos<double, DIM>(sh_x[wave], e, xj[h]);
            if constexpr (MODE == 1) qj[h] = sh_q[wave][e];
            if constexpr (MODE != 0) load_mass<double, SMAX>(sh_m[wave], e, mj[h]);
          }
#pragma unroll
          for (int h = 0; h < H; ++h)
#pragma unroll
            for (int p = 0; p < PP; ++p) s2[h][p] = sep2_64<DIM>(xi[p], xj[h]);
#pragma unroll
          for (int h = 0; h < H; ++h) {
#pragma unroll
            for (int p = 0; p < PP; ++p) {
              // a branch, not a select: neighbouring candidates and particles
              // agree, and a wave all of whose pairs are outside skips the rest
              if (s2[h][p] <= rc2[p]) {
                const double wt = wfn(s2[h][p]);
                if constexpr (MODE != 1) racc[p] += wt;
                if constexpr (MODE != 0) {
                  const double pw = MODE == 1 ? wt * (qi[p] + qj[h]) : wt;  // symmetric: 2 P_ij
#pragma unroll
                  for (int s = 0; s < SMAX; ++s) acc[p][s] += pw * (mj[h][s] - Mi[p][s]);
                }
              }
            }
          }
        }
      }
      seg = seg_end;
    }
  }
#pragma unroll
  for (int p = 0; p < PP; ++p) {
    if (p >= nt) break;  // uniform
    const int32_t i = begin + gi + p * G;
    const bool writer = gl == 0 && gi + p * G < n_in;
#pragma unroll
    for (int off = G; off < 64; off <<= 1) {
      if constexpr (MODE != 1) racc[p] += __shfl_xor(racc[p], off);
      if constexpr (MODE != 0) {
#pragma unroll
        for (int s = 0; s < SMAX; ++s) acc[p][s] += __shfl_xor(acc[p][s], off);
      }
    }
    if constexpr (MODE == 0) {
      if (writer) {
        if (!R.active) racc[p] = 1.0;  // only the self weight
        if (a.r_out) a.r_out[i] = racc[p];
        ((double*)a.q_out)[i] = 1.0 / racc[p];
      }
    } else {
      exchange_epilogue<double, SMAX, G>(R, MODE == 1, acc[p], racc[p], Mi[p], writer, i, (double*)a.mass_out, a.S,
                                         a.react_a, a.react_b, a.audit_part, a.out_map, tile + p);
    }
  }
}

template <int SMAX, int MODE>
static hipError_t launch64(int dim, int log2l, const PairArgs& a, hipStream_t s) {
  const bool two = a.group_nitems > 0;
  const int32_t waves = two ? a.group_nitems : a.ntiles;
  const dim3 g((unsigned)((waves + kBlock / 64 - 1) / (kBlock / 64))), b(kBlock);
  auto go = [&](auto d, auto l) {
    constexpr int D = decltype(d)::value, LG = decltype(l)::value;
    if (two) hipLaunchKernelGGL((k_pairs64<D, SMAX, LG, kGroupTiles, MODE>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_pairs64<D, SMAX, LG, 1, MODE>), g, b, 0, s, a);
  };
  auto with_l = [&](auto d) -> hipError_t {
    if (log2l == 3) go(d, std::integral_constant<int, 3>{});
    else if (log2l == 4) go(d, std::integral_constant<int, 4>{});
    else return hipErrorInvalidValue;
    return hipGetLastError();
  };
  if (dim == 1) return with_l(std::integral_constant<int, 1>{});
  if (dim == 2) return with_l(std::integral_constant<int, 2>{});
  if (dim == 3) return with_l(std::integral_constant<int, 3>{});
  return hipErrorInvalidValue;
}

hipError_t launch_rowsum64(int dim, int log2l, const PairArgs& a, hipStream_t s) {
  return launch64<2, 0>(dim, log2l, a, s);
}

hipError_t launch_exchange64(int dim, int log2l, const PairArgs& a, hipStream_t s) {
  if (a.norm == 0) {
    if (a.S <= 2) return launch64<2, 1>(dim, log2l, a, s);
    if (a.S <= 4) return launch64<4, 1>(dim, log2l, a, s);
    return launch64<8, 1>(dim, log2l, a, s);
  }
  if (a.S <= 2) return launch64<2, 2>(dim, log2l, a, s);
  if (a.S <= 4) return launch64<4, 2>(dim, log2l, a, s);
  return launch64<8, 2>(dim, log2l, a, s);
}

}  // namespace rwpt
