// rwpt_gauss1d.hip -- pair kernels of dense 1-D neighbourhoods (binary32
// state): Gauss sums by expansions over cells (the fast Gauss transform of
// Greengard & Strain, SIAM J. Sci. Stat. Comput. 12, 1991, on a uniform grid).
//
// In units of sigma, a pair of target t + u and source s + v (t, s the centres
// of their cells, d = t - s) has the weight
//   exp(-(d + u - v)^2) = sum_{a + b < P} h_{a+b}(d) v^a / a! (-u)^b / b!,
// h_n the Hermite functions (-d/dx)^n exp(-x^2), up to the truncation
//   |u - v|^P max|h_P| / P! <= 1.09 (sqrt(2) h / sigma)^P / sqrt(P!)
// for cells of width h.  So a cell's sources enter through P moments per
// column (mass, mass / r, 1 / r, 1), and every target of a cell shares one
// polynomial of P coefficients per column: the work per particle does not
// grow with the neighbours it has.  All of it is binary64; P and h / sigma are
// chosen (gauss_plan) for a truncation below 2e-9 of one weight, which is
// under the rounding of a binary32 weight; 1 / r is kept in binary64 between
// the passes.
//
// The cutoff is kept exactly: only cells all of whose points lie within the
// cutoff of all points of the target's cell (|k| <= g_in) are expanded.  The
// cells the cutoff may cut (g_in < |k| <= g_out, two on either side) are
// evaluated pair by pair with the predicate of the other pair kernels.  The
// full matrix has no such cells and expands out to weights of 2^-44.
//
// 32768 particles with 1758 neighbours: row sums 18.9 -> 13.1 us (4.0 of them
// the moments), exchange 29.7 -> 15.9 (4.6); full matrix (3080 neighbours above
// 2^-40) row sums 34 -> 12.7, exchange 119 -> 14.4 us.
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "rwpt_epilogue.h"
#include "rwpt_kernels.h"
#include "rwpt_layout.h"
#include "rwpt_pairstep.h"

namespace rwpt {

// Hermite functions h_0..h_{P-1} of the cell offsets -g_in..g_in of each
// realisation: row kk holds them at d = (g_in - kk) h / sigma, the distance
// from the source cell target + kk - g_in.
__global__ __launch_bounds__(kBlock) void k_gauss_table(const RealParams* __restrict__ rp, int32_t n_real, int32_t P,
                                                        int32_t rows, double* __restrict__ tab) {
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e >= (int64_t)n_real * rows) return;
  const RealParams& R = rp[e / rows];
  const int kk = (int)(e % rows);
  double* const o = tab + e * P;
  const double d = (double)(R.g_in - kk) * sqrt(-R.escale_d) / R.inv_h[0];
  double h0 = (R.active && kk <= 2 * R.g_in) ? exp(-d * d) : 0.0, h1 = 2.0 * d * h0;
  for (int n = 0; n < P; ++n) {
    o[n] = h0;
    const double h2 = 2.0 * d * h1 - 2.0 * (double)(n + 1) * h0;
    h0 = h1;
    h1 = h2;
  }
}

struct InvFact {
  double v[kGaussMaxTerms];
};
constexpr InvFact inv_factorials() {
  InvFact f{};
  double x = 1.0;
  for (int n = 0; n < kGaussMaxTerms; ++n) {
    f.v[n] = 1.0 / x;
    x *= (double)(n + 1);
  }
  return f;
}
__device__ constexpr InvFact kInvFact = inv_factorials();

// Columns of the sums.  MODE 0: row sums; 1: exchange, symmetric: M_s, q M_s,
// q, 1; 2: exchange, row normalisation: M_s, 1.
constexpr int gauss_columns(int smax, int mode) { return mode == 0 ? 1 : (mode == 1 ? 2 * smax + 2 : smax + 1); }

// Moments sum_j f_j v_j^n / n! of every cell and column, n < P, in planes
// [n][cell][column].  Eight lanes share the particles of one cell and column:
// with about 27 particles a cell the pass is one round of loads.
template <int P, int SMAX, int MODE>
__global__ __launch_bounds__(kBlock) void k_gauss_moments(const PairArgs a) {
  constexpr int NCOL = gauss_columns(SMAX, MODE);
  const float* __restrict__ pos = (const float*)a.pos;
  const float* __restrict__ min_ = (const float*)a.mass_in;
  const int64_t e = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 3;
  const int pt = threadIdx.x & 7;
  const int64_t n_out = a.gauss_ncell * NCOL;
  double m[P];
#pragma unroll
  for (int n = 0; n < P; ++n) m[n] = 0.0;
  if (e < n_out) {
    const int64_t cell = e / NCOL;
    const int col = (int)(e - cell * NCOL);
    const uint32_t jb = a.cell_start[cell], je = a.cell_start[cell + 1];
    // from the group's first cell, whose realisation is this cell's or, near a
    // boundary, one a few before it (searched from realisation 0: a step of 1000
    // realisations of 4000 particles 6450 us, 1710 so)
    int real = a.gauss_cell_real ? a.gauss_cell_real[cell / kGaussCellGroup] : 0;
    while (real + 1 < a.n_real && a.rp[real + 1].cell_off <= cell) ++real;
    const RealParams& R = a.rp[real];
    const double ctr = R.lo[0] + ((double)(cell - R.cell_off) + 0.5) / R.inv_h[0], gs = sqrt(-R.escale_d);
    const bool use_m = MODE == 1 ? col < 2 * SMAX : (MODE == 2 && col < SMAX);
    const bool use_q = MODE == 1 && col >= SMAX && col != 2 * SMAX + 1;
    const int sp = col % SMAX;
#pragma unroll 4
    for (uint32_t j = jb + pt; j < je; j += 8) {
      const double v = ((double)pos[j] - ctr) * gs;
      double f = use_m ? (double)min_[(int64_t)SMAX * j + sp] : 1.0;
      if (use_q) f *= a.gauss_q[j];
      m[0] += f;
#pragma unroll
      for (int n = 1; n < P; ++n) {
        f *= v;
        m[n] += f;
      }
    }
  }
#pragma unroll
  for (int n = 0; n < P; ++n) {
    m[n] += xor_shfl<1>(m[n]);
    m[n] += xor_shfl<2>(m[n]);
    m[n] += xor_shfl<4>(m[n]);
  }
  if (e < n_out && pt == 0) {
#pragma unroll
    for (int n = 0; n < P; ++n) a.gauss_mom[n * n_out + e] = m[n] * kInvFact.v[n];
  }
}

// A block takes up to 8 consecutive tiles of 16 particles of one realisation,
// so that clustered particles spread over as many blocks as elsewhere.  A
// launch has few blocks (256 at 32768 particles), one per CU, and what it
// reads was just written by another XCD, so the pass is a chain of a few long
// latencies: everything a block needs is loaded in one round.  Waves 0-7 load
// the moments and Hermite rows of the cells around CM target cells (a tile's
// particles span few: the plan asks for 18 particles per cell, the full matrix's
// for eight) and transfer them, the cell offset split over the waves; waves 8-15 load the
// particles of the cells that the cutoff may cut and evaluate those pairs,
// four lanes per particle.  Then the offsets' shares are summed and the
// polynomials evaluated at the block's particles, whose columns are shared by
// the particle's four lanes.  32768 particles, 1758 neighbours: 11.3 us; each block
// computing the moments of its own source cells, without a launch for them:
// 20 us; moments and candidates read from memory where they are used: 13.2 us
// + 5.4 for the moments.
// Columns are taken NG at a time, which bounds the LDS for eight species.
constexpr int kGaussBlock = 2 * 64 * kGaussTiles;

template <int P, int CM, int KMAX, int SMAX, int MODE>
__global__ __launch_bounds__(kGaussBlock) void k_gauss1d(const PairArgs a) {
  constexpr int NCOL = gauss_columns(SMAX, MODE);
  constexpr int NGRP = (NCOL + 5) / 6, NG = (NCOL + NGRP - 1) / NGRP;
  static_assert(CM * NG <= 64, "one lane per target cell and column");
  __shared__ double part[kGaussTiles][P][CM * NG];
  __shared__ double near_sum[SMAX + 1][kGaussTiles * 16];
  __shared__ double mom[P][(CM + 2 * KMAX) * NG];
  __shared__ double hrow[2 * KMAX + 1][P];
  // particles of the near cells; where they are more (blocks that span many
  // cells, clusters), they are read from memory
  constexpr int kNear = SMAX > 4 ? 512 : 1024;
  __shared__ float near_x[kNear], near_q[MODE == 1 ? kNear : 1];
  __shared__ __attribute__((aligned(16))) float near_m[MODE == 0 ? 4 : kNear * SMAX];
  const int blk = xcd_block(blockIdx.x, gridDim.x);
  TileGroup item;
  if (a.gauss_items) {
    item = a.gauss_items[blk];
  } else {  // one realisation
    item.tile = blk * kGaussTiles;
    item.ntiles = a.ntiles - item.tile < kGaussTiles ? a.ntiles - item.tile : kGaussTiles;
    item.real = 0;
  }
  const RealParams& R = a.rp[item.real];
  const float* __restrict__ pos = (const float*)a.pos;
  const float* __restrict__ min_ = (const float*)a.mass_in;
  const int tid = threadIdx.x, lane = tid & 63, gi = lane & 15, gl = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wt = wave % kGaussTiles;
  const bool far = wave < kGaussTiles;
  const bool has = wt < item.ntiles;
  const Tile tile = a.tiles[item.tile + (has ? wt : 0)];
  const int32_t i = tile.begin + gi;
  const bool valid = has && i < tile.end;
  const int32_t ii = i < tile.end ? i : tile.end - 1;
  const float xi = pos[ii];
  const uint32_t coff = (uint32_t)R.cell_off;
  const int ci = (int)(a.skey[ii] - coff);
  float Mi[SMAX];
  double qi = 0.0;
#pragma unroll
  for (int s = 0; s < SMAX; ++s) Mi[s] = 0.0f;
  if constexpr (MODE != 0) load_mass<float, SMAX>(min_, ii, Mi);
  if constexpr (MODE == 1) qi = a.gauss_q[ii];
  double acc[SMAX], racc = 0.0;  // MODE 0: racc alone
#pragma unroll
  for (int s = 0; s < SMAX; ++s) acc[s] = 0.0;
  const int nc = R.nc[0], K = R.g_in;
  if (R.active) {
    const double h = 1.0 / R.inv_h[0], lo = R.lo[0], gs = sqrt(-R.escale_d);
    const double* __restrict__ tab = a.gauss_tab + (int64_t)item.real * a.gauss_rows * P;
    const int64_t plane = a.gauss_ncell * NCOL;
    const int ca = (int)(a.skey[a.tiles[item.tile].begin] - coff);
    const int cb = (int)(a.skey[a.tiles[item.tile + item.ntiles - 1].end - 1] - coff);
    // near cells of all the block's particles: [L0, L1) and [R0, R1)
    auto start_of = [&](int c) { return a.cell_start[coff + (c < 0 ? 0 : (c > nc ? nc : c))]; };
    const bool near = R.g_out > K;
    const uint32_t L0 = start_of(ca - R.g_out), L1 = start_of(cb - K);
    const uint32_t R0 = start_of(ca + K + 1), R1 = start_of(cb + R.g_out + 1);
    const uint32_t nL = L1 - L0, nN = nL + (R1 - R0);
    const bool staged = nN <= (uint32_t)kNear;
    // this particle's part of them
    const uint32_t l0 = start_of(ci - R.g_out), nl = start_of(ci - K) - l0;
    const uint32_t r0 = start_of(ci + K + 1), nn = nl + (start_of(ci + R.g_out + 1) - r0);
    for (int c0 = ca;;) {
      const int ncell = cb - c0 + 1 < CM ? cb - c0 + 1 : CM;
#pragma unroll 1
      for (int grp = 0; grp < NGRP; ++grp) {
        const bool first = c0 == ca && grp == 0;
        if (far) {
          // source cells c0 - K .. c0 + ncell - 1 + K; loads of the planes together
          for (int e = tid; e < (ncell + 2 * K) * NG; e += 64 * kGaussTiles) {
            const int sc = c0 - K + e / NG, col = grp * NG + e % NG;
            const bool in = sc >= 0 && sc < nc && col < NCOL;
            const double* __restrict__ mp = a.gauss_mom + (in ? ((int64_t)coff + sc) * NCOL + col : 0);
            double mu[P];
#pragma unroll
            for (int n = 0; n < P; ++n) mu[n] = mp[n * plane];
#pragma unroll
            for (int n = 0; n < P; ++n) mom[n][e] = in ? mu[n] : 0.0;
          }
          if (first)
            for (int e = tid; e < (2 * K + 1) * P; e += 64 * kGaussTiles) (&hrow[0][0])[e] = tab[e];
        } else if (first && near && staged) {
          for (uint32_t e = tid - 64 * kGaussTiles; e < nN; e += 64 * kGaussTiles) {
            const uint32_t j = e < nL ? L0 + e : R0 + (e - nL);
            near_x[e] = pos[j];
            if constexpr (MODE == 1) near_q[e] = (float)a.gauss_q[j];
            if constexpr (MODE != 0) {
              float m[SMAX];
              load_mass<float, SMAX>(min_, j, m);
              store_mass<float, SMAX>(near_m, e, m);
            }
          }
        }
        __syncthreads();
        if (far) {
          if (lane < ncell * NG) {
            // source cell target + kk - K at the offset of Hermite row kk
            double L[P];
#pragma unroll
            for (int b = 0; b < P; ++b) L[b] = 0.0;
            for (int kk = wave; kk <= 2 * K; kk += kGaussTiles) {
              double mu[P], H[P];
#pragma unroll
              for (int n = 0; n < P; ++n) {
                mu[n] = mom[n][kk * NG + lane];
                H[n] = hrow[kk][n];
              }
#pragma unroll
              for (int b = 0; b < P; ++b)
#pragma unroll
                for (int n = 0; n < P - b; ++n) L[b] = __builtin_fma(H[n + b], mu[n], L[b]);
            }
#pragma unroll
            for (int b = 0; b < P; ++b) part[wave][b][lane] = L[b];
          }
        }
        if (first && near && valid) {
          // the left and the right cells as one list; the particle's four
          // lanes of waves 8-15 take every fourth candidate of its first two
          // thirds, those of waves 0-7, done with the transfer by then, of the
          // rest; binary32 partials of U
          constexpr int U = SMAX > 4 ? 4 : 8;
          const float rc2 = R.rc2_f, esc = R.escale_f;
          const uint32_t cut = nn - nn / 3, tb = far ? cut : 0u, te = far ? nn : cut;
          for (uint32_t t0 = tb + gl; t0 < te; t0 += 4 * U) {
            float xj[U], qj[U], mj[U][SMAX];
            bool in[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const uint32_t t = t0 + 4 * u;
              in[u] = t < te;
              const uint32_t tt = in[u] ? t : t0;
              const uint32_t j = tt < nl ? l0 + tt : r0 + (tt - nl);
              if (staged) {
                const uint32_t e = tt < nl ? j - L0 : nL + (j - R0);
                xj[u] = near_x[e];
                if constexpr (MODE == 1) qj[u] = near_q[e];
                if constexpr (MODE != 0) load_mass<float, SMAX>(near_m, e, mj[u]);
              } else {
                xj[u] = pos[j];
                if constexpr (MODE == 1) qj[u] = (float)a.gauss_q[j];
                if constexpr (MODE != 0) load_mass<float, SMAX>(min_, j, mj[u]);
              }
            }
            float accr[SMAX], rr = 0.0f;
#pragma unroll
            for (int s = 0; s < SMAX; ++s) accr[s] = 0.0f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const float d0 = xj[u] - xi;
              const float s2 = d0 * d0;
              const float w = (in[u] && s2 <= rc2) ? kweight(s2, esc) : 0.0f;
              if constexpr (MODE != 1) rr += w;
              if constexpr (MODE != 0) {
                const float p = MODE == 1 ? w * ((float)qi + qj[u]) : w;
#pragma unroll
                for (int s = 0; s < SMAX; ++s) accr[s] += p * (mj[u][s] - Mi[s]);
              }
            }
            if constexpr (MODE != 1) racc += (double)rr;
            if constexpr (MODE != 0) {
#pragma unroll
              for (int s = 0; s < SMAX; ++s) acc[s] += (double)accr[s];
            }
          }
        }
        __syncthreads();
        // the waves' shares in wave order, with (-1)^b / b!; each thread
        // rewrites only the entry it has read
        for (int e = tid; e < P * CM * NG; e += kGaussBlock) {
          const int b = e / (CM * NG), o = e % (CM * NG);
          if (o < ncell * NG) {
            double sum = 0.0;
#pragma unroll
            for (int w = 0; w < kGaussTiles; ++w) sum += part[w][b][o];
            part[0][b][o] = sum * ((b & 1) ? -kInvFact.v[b] : kInvFact.v[b]);
          }
        }
        __syncthreads();
        if (far && valid && ci >= c0 && ci < c0 + ncell) {
          const double u = ((double)xi - (lo + ((double)ci + 0.5) * h)) * gs;
#pragma unroll
          for (int g0 = 0; g0 < NG; g0 += 4) {
            const int gc = g0 + gl, col = grp * NG + gc;
            if (gc < NG && col < NCOL) {
              const int o = (ci - c0) * NG + gc;
              double val = part[0][P - 1][o];
#pragma unroll
              for (int b = P - 2; b >= 0; --b) val = __builtin_fma(val, u, part[0][b][o]);
              if constexpr (MODE == 0) {
                racc += val;
              } else if constexpr (MODE == 1) {
                // q_i sum w M_j + sum w q_j M_j - M_i (sum w q_j + q_i sum w)
                const double at = col < SMAX ? qi * val : (col < 2 * SMAX ? val : 0.0);
                const double every = col == 2 * SMAX ? val : (col == 2 * SMAX + 1 ? qi * val : 0.0);
#pragma unroll
                for (int s = 0; s < SMAX; ++s)
                  acc[s] += (col % SMAX == s ? at : 0.0) - (double)Mi[s] * every;
              } else {
                const double every = col == SMAX ? val : 0.0;
                racc += every;
#pragma unroll
                for (int s = 0; s < SMAX; ++s) acc[s] += (col == s ? val : 0.0) - (double)Mi[s] * every;
              }
            }
          }
        }
        __syncthreads();  // mom and part are written again
      }
      if (c0 + ncell > cb) break;
      c0 = (int)(a.skey[a.cell_start[coff + c0 + ncell]] - coff);  // the next cell with a particle, at most cb
    }
  }
#pragma unroll
  for (int off = 16; off < 64; off <<= 1) {
    if constexpr (MODE != 1) racc += __shfl_xor(racc, off);
    if constexpr (MODE != 0) {
#pragma unroll
      for (int s = 0; s < SMAX; ++s) acc[s] += __shfl_xor(acc[s], off);
    }
  }
  if (!far && gl == 0) {
    if constexpr (MODE != 1) near_sum[SMAX][wt * 16 + gi] = racc;
    if constexpr (MODE != 0) {
#pragma unroll
      for (int s = 0; s < SMAX; ++s) near_sum[s][wt * 16 + gi] = acc[s];
    }
  }
  __syncthreads();
  if (!has || !far) return;
  if constexpr (MODE != 1) racc += near_sum[SMAX][wt * 16 + gi];
  if constexpr (MODE != 0) {
#pragma unroll
    for (int s = 0; s < SMAX; ++s) acc[s] += near_sum[s][wt * 16 + gi];
  }
  if constexpr (MODE == 0) {
    if (gl == 0 && valid) {
      if (!R.active) racc = 1.0;  // only the self weight
      if (a.r_out) a.r_out[i] = racc;
      ((float*)a.q_out)[i] = (float)(1.0 / racc);
      if (a.gauss_q) a.gauss_q[i] = 1.0 / racc;
    }
  } else {
    exchange_epilogue<float, SMAX, 16>(R, MODE == 1, acc, racc, Mi, gl == 0 && valid, i, (float*)a.mass_out, a.S,
                                       a.react_a, a.react_b, a.audit_part, a.out_map, item.tile + wave);
  }
}

hipError_t launch_gauss_table(int plan, const RealParams* rp, int32_t n_real, double* tab, hipStream_t s) {
  if (plan < 1 || plan > kGaussPlans) return hipErrorInvalidValue;
  const int64_t n = (int64_t)n_real * gauss_rows(plan);
  hipLaunchKernelGGL(k_gauss_table, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, rp, n_real,
                     kGaussPlan[plan].terms, gauss_rows(plan), tab);
  return hipGetLastError();
}

template <int SMAX, int MODE>
static hipError_t launch_plan(int plan, const PairArgs& a, hipStream_t s) {
  const dim3 g((unsigned)a.gauss_nitems), b(kGaussBlock);
  const dim3 gm((unsigned)((a.gauss_ncell * gauss_columns(SMAX, MODE) * 8 + kBlock - 1) / kBlock));
  auto go = [&](auto pl) {
    constexpr GaussPlan p = kGaussPlan[decltype(pl)::value];
    hipLaunchKernelGGL((k_gauss_moments<p.terms, SMAX, MODE>), gm, dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL((k_gauss1d<p.terms, kGaussCells, p.reach, SMAX, MODE>), g, b, 0, s, a);
  };
  if (plan == 1) go(std::integral_constant<int, 1>{});
  else if (plan == 2) go(std::integral_constant<int, 2>{});
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_gauss_rowsum(int plan, const PairArgs& a, hipStream_t s) {
  if (a.gauss_nitems <= 0) return hipSuccess;
  return launch_plan<2, 0>(plan, a, s);
}

hipError_t launch_gauss_exchange(int plan, const PairArgs& a, hipStream_t s) {
  if (a.gauss_nitems <= 0) return hipSuccess;
  if (a.S < 1 || a.S > 8) return hipErrorInvalidValue;
  if (a.norm == 0) {
    if (a.S <= 2) return launch_plan<2, 1>(plan, a, s);
    if (a.S <= 4) return launch_plan<4, 1>(plan, a, s);
    return launch_plan<8, 1>(plan, a, s);
  }
  if (a.S <= 2) return launch_plan<2, 2>(plan, a, s);
  if (a.S <= 4) return launch_plan<4, 2>(plan, a, s);
  return launch_plan<8, 2>(plan, a, s);
}

}  // namespace rwpt
