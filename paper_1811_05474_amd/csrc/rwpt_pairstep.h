// rwpt_pairstep.h -- per-candidate steps of the row-broadcast pair kernels
// (internal to the HIP code).
//
// In the row-broadcast tiling a 16-lane row of a wave holds 16 particles i of
// a tile, and every lane of the row has loaded one candidate j.  Step K
// broadcasts lane K's candidate to the whole row (a DPP row_share, which the
// compiler folds into the consuming subtract) and every lane evaluates the
// pair (i, j_K).  A chunk is the 16 steps K = 0..15.
//
// The row-sum and exchange kernels and the instruction-rate probe all call the
// chunk functions below, so the probe times exactly the kernels' sequence.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

namespace rwpt {

// Co-location weight exp(-s2 / sigma^2) (Eq. 3 without prefactor): binary32
// uses the hardware exp2 with the scale -log2(e)/sigma^2; binary64 uses the
// library exp (the table form exp_tab below is what the binary64 kernels use).
__device__ __forceinline__ float kweight(float s2, float escale) {
  return __builtin_amdgcn_exp2f(s2 * escale);
}
__device__ __forceinline__ double kweight(double s2, double escale) { return exp(s2 * escale); }

// 2^(j/64), j = 0..63, each correctly rounded to binary64.
__device__ constexpr double kExp2Frac[64] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0, 0x1.0874518759bc8p+0,
    0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0, 0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0,
    0x1.172b83c7d517bp+0, 0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0, 0x1.2d285a6e4030bp+0,
    0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0, 0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0,
    0x1.3dea64c123422p+0, 0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0, 0x1.56f4736b527dap+0,
    0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0, 0x1.6247eb03a5585p+0, 0x1.6623882552225p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0, 0x1.868d99b4492edp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0, 0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0,
    0x1.9c49182a3f090p+0, 0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0, 0x1.bcc1e904bc1d2p+0,
    0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0, 0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0,
    0x1.d5818dcfba487p+0, 0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0, 0x1.fa7c1819e90d8p+0,
};

// Binary64 exp(x) for x <= 0 (table-driven): x = (64 n + j) ln2/64 + r with
// |r| <= ln2/128, the product t ln2/64 subtracted in two parts (a 32-bit head,
// exact for |t| < 2^21, and the tail); then exp(x) = 2^n 2^(j/64) (1 + q) with
// q = e^r - 1 = r (1 + r/2 + r^2/6 + r^3/24 + r^4/120), whose truncation is
// below 2^-54 relative.  Within 1.1 ulp of exp on [-745, 0]; arguments below
// -1000 return 0.  tbl holds kExp2Frac.
__device__ __forceinline__ double exp_tab(double x, const double* __restrict__ tbl) {
  constexpr double kInvLn2_64 = 0x1.71547652b82fep+6;   // 64 / ln 2
  constexpr double kLn2_64Hi = 0x1.62e42fee00000p-7;    // ln 2 / 64, head
  constexpr double kLn2_64Lo = 0x1.a39ef35793c76p-39;   // ln 2 / 64 - head
  x = __builtin_fmax(x, -1000.0);
  const double t = __builtin_rint(x * kInvLn2_64);
  double r = __builtin_fma(-t, kLn2_64Hi, x);
  r = __builtin_fma(-t, kLn2_64Lo, r);
  const int k = (int)t;
  double p = 1.0 / 120.0;
  p = __builtin_fma(p, r, 1.0 / 24.0);
  p = __builtin_fma(p, r, 1.0 / 6.0);
  p = __builtin_fma(p, r, 0.5);
  p = __builtin_fma(p, r, 1.0);
  const double q = p * r;
  const double f = tbl[k & 63];
  return __builtin_ldexp(__builtin_fma(f, q, f), k >> 6);
}

// Weight evaluator of the pair kernels.  setup() must be called by every
// thread of the block before any of them returns: the binary64 form fills a
// block-shared copy of kExp2Frac (one barrier); the binary32 form is the
// hardware exp2 and needs nothing.
template <typename T>
struct WeightFn {
  __device__ __forceinline__ void setup() {}
  __device__ __forceinline__ T operator()(T s2, T escale) const { return kweight(s2, escale); }
};
template <>
struct WeightFn<double> {
  const double* tbl;
  __device__ __forceinline__ void setup() {
    __shared__ double sh_tbl[64];
    if (threadIdx.x < 64) sh_tbl[threadIdx.x] = kExp2Frac[threadIdx.x];
    __syncthreads();
    tbl = sh_tbl;
  }
  __device__ __forceinline__ double operator()(double s2, double escale) const {
    return exp_tab(s2 * escale, tbl);
  }
};

// Value of lane K of this lane's 16-lane row (DPP row_share).
template <int K>
__device__ __forceinline__ float rshare(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + K, 0xf,
                                                               0xf, false));
}

// Compile-time loop K = Begin..End-1 (each step needs K as a constant).
template <int K, int N>
struct Steps {
  template <typename F>
  __device__ __forceinline__ static void run(F&& f) {
    f(std::integral_constant<int, K>{});
    Steps<K + 1, N>::run(f);
  }
};
template <int N>
struct Steps<N, N> {
  template <typename F>
  __device__ __forceinline__ static void run(F&&) {}
};

// s^2 of the pair (this lane's particle, candidate K of the row): s^2 =
// fma(d2, d2, fma(d1, d1, d0 * d0)), the cutoff predicate's arithmetic.
template <int K, int DIM>
__device__ __forceinline__ float row_s2(const float (&xj)[DIM], const float (&xi)[DIM]) {
  const float d0 = rshare<K>(xj[0]) - xi[0];
  float s2 = d0 * d0;
  if constexpr (DIM > 1) {
    const float d1 = rshare<K>(xj[1]) - xi[1];
    s2 = __builtin_fmaf(d1, d1, s2);
  }
  if constexpr (DIM > 2) {
    const float d2 = rshare<K>(xj[2]) - xi[2];
    s2 = __builtin_fmaf(d2, d2, s2);
  }
  return s2;
}

// Weight of the pair, zero unless the lane is active and s^2 <= rc2 (the cutoff
// predicate of the neighbour search).
template <int K, int DIM>
__device__ __forceinline__ float row_weight(const float (&xj)[DIM], const float (&xi)[DIM], float rc2, float esc,
                                            bool act) {
  const float s2 = row_s2<K, DIM>(xj, xi);
  const float w = kweight(s2, esc);
  return (act && s2 <= rc2) ? w : 0.0f;
}

// The sums below are taken under the predicate as execution mask instead of
// with a selected weight: one vector instruction less per pair (of 9 in the row
// sum, of 14 in the exchange), the mask's restore is a scalar one.  A group's
// pairs share one block, which restores the mask itself and ends in the five
// wait states that a DPP or lane access needs after a vector write of the mask;
// no weight is read by the block's first instruction, as an exp's result must
// not be by the next one.  lim is rc2, or -1 in a lane that takes no part.
// 1e6 particles of 225 neighbours: row sums 134 -> 120 us, exchange 206 -> 197.
// (The same as a branch in the source: the compiler selects again, and the
// shorter blocks schedule worse, 0.409 ms a step against 0.375 before.)

// a += w[u] where s2[u] <= lim, u in order.
__device__ __forceinline__ void add_within(float& a, const float (&s2)[8], const float (&w)[8], float lim) {
  unsigned long long save;
  asm("s_mov_b64 %[save], exec\n\t"
      "v_cmpx_le_f32 vcc, %[s0], %[lim]\n\tv_add_f32 %[a], %[a], %[w0]\n\ts_mov_b64 exec, %[save]\n\t"
      "v_cmpx_le_f32 vcc, %[s1], %[lim]\n\tv_add_f32 %[a], %[a], %[w1]\n\ts_mov_b64 exec, %[save]\n\t"
      "v_cmpx_le_f32 vcc, %[s2], %[lim]\n\tv_add_f32 %[a], %[a], %[w2]\n\ts_mov_b64 exec, %[save]\n\t"
      "v_cmpx_le_f32 vcc, %[s3], %[lim]\n\tv_add_f32 %[a], %[a], %[w3]\n\ts_mov_b64 exec, %[save]\n\t"
      "v_cmpx_le_f32 vcc, %[s4], %[lim]\n\tv_add_f32 %[a], %[a], %[w4]\n\ts_mov_b64 exec, %[save]\n\t"
      "v_cmpx_le_f32 vcc, %[s5], %[lim]\n\tv_add_f32 %[a], %[a], %[w5]\n\ts_mov_b64 exec, %[save]\n\t"
      "v_cmpx_le_f32 vcc, %[s6], %[lim]\n\tv_add_f32 %[a], %[a], %[w6]\n\ts_mov_b64 exec, %[save]\n\t"
      "v_cmpx_le_f32 vcc, %[s7], %[lim]\n\tv_add_f32 %[a], %[a], %[w7]\n\ts_mov_b64 exec, %[save]\n\t"
      "s_nop 4"
      : [a] "+&v"(a), [save] "=&s"(save)
      : [lim] "v"(lim), [s0] "v"(s2[0]), [s1] "v"(s2[1]), [s2] "v"(s2[2]), [s3] "v"(s2[3]), [s4] "v"(s2[4]),
        [s5] "v"(s2[5]), [s6] "v"(s2[6]), [s7] "v"(s2[7]), [w0] "v"(w[0]), [w1] "v"(w[1]), [w2] "v"(w[2]),
        [w3] "v"(w[3]), [w4] "v"(w[4]), [w5] "v"(w[5]), [w6] "v"(w[6]), [w7] "v"(w[7])
      : "vcc");
}

// acc0 += (w qs) d0 and acc1 += (w qs) d1 where s2 <= lim, for four pairs.
__device__ __forceinline__ void exchange_within(float& acc0, float& acc1, const float (&s2)[4], const float (&w)[4],
                                                const float (&qs)[4], const float (&d0)[4], const float (&d1)[4],
                                                float lim) {
  unsigned long long save;
  float p;
#define RWPT_PAIR(u)                                                                               \
  "v_cmpx_le_f32 vcc, %[s" #u "], %[lim]\n\tv_mul_f32 %[p], %[w" #u "], %[q" #u "]\n\t"           \
  "v_fmac_f32 %[a0], %[p], %[x" #u "]\n\tv_fmac_f32 %[a1], %[p], %[y" #u "]\n\ts_mov_b64 exec, %[save]\n\t"
  asm("s_mov_b64 %[save], exec\n\t" RWPT_PAIR(0) RWPT_PAIR(1) RWPT_PAIR(2) RWPT_PAIR(3) "s_nop 4"
      : [a0] "+&v"(acc0), [a1] "+&v"(acc1), [p] "=&v"(p), [save] "=&s"(save)
      : [lim] "v"(lim), [s0] "v"(s2[0]), [s1] "v"(s2[1]), [s2] "v"(s2[2]), [s3] "v"(s2[3]), [w0] "v"(w[0]),
        [w1] "v"(w[1]), [w2] "v"(w[2]), [w3] "v"(w[3]), [q0] "v"(qs[0]), [q1] "v"(qs[1]), [q2] "v"(qs[2]),
        [q3] "v"(qs[3]), [x0] "v"(d0[0]), [x1] "v"(d0[1]), [x2] "v"(d0[2]), [x3] "v"(d0[3]), [y0] "v"(d1[0]),
        [y1] "v"(d1[1]), [y2] "v"(d1[2]), [y3] "v"(d1[3])
      : "vcc");
#undef RWPT_PAIR
}

// Row sum over one chunk: sum over K of w(i, j_K).  NK < 16: only the
// first NK lanes of each row hold candidates (a segment's short last chunk).
template <int DIM, int NK = 16>
__device__ __forceinline__ float rowsum_chunk(const float (&xj)[DIM], const float (&xi)[DIM], float rc2, float esc,
                                              bool act) {
  float a = 0.0f;
  if constexpr (NK >= 8) {
    const float lim = act ? rc2 : -1.0f;
    Steps<0, NK / 8>::run([&](auto bc) {
      constexpr int B = 8 * decltype(bc)::value;
      float s2[8], w[8];
      Steps<0, 8>::run([&](auto uc) {
        constexpr int U = decltype(uc)::value;
        s2[U] = row_s2<B + U, DIM>(xj, xi);
        w[U] = kweight(s2[U], esc);
      });
      add_within(a, s2, w, lim);
    });
  } else {
    Steps<0, NK>::run([&](auto kc) {
      constexpr int K = decltype(kc)::value;
      a += row_weight<K, DIM>(xj, xi, rc2, esc, act);
    });
  }
  return a;
}

// Exchange over one chunk, symmetric normalisation: accr[s] += w (q_j + q_i)
// (m_j[s] - M_i[s]) with q = 1 / r, i.e. twice the symmetric P_ij times the
// mass difference.
template <int DIM, int SMAX, int NK = 16>
__device__ __forceinline__ void exchange_chunk_sym(const float (&xj)[DIM], const float (&xi)[DIM], float qj, float qi,
                                                   const float (&mj)[SMAX], const float (&Mi)[SMAX], float rc2,
                                                   float esc, bool act, float (&accr)[SMAX]) {
  if constexpr (SMAX == 2) {
    const float lim = act ? rc2 : -1.0f;
    Steps<0, NK / 4>::run([&](auto bc) {
      constexpr int B = 4 * decltype(bc)::value;
      float s2[4], w[4], qs[4], d0[4], d1[4];
      Steps<0, 4>::run([&](auto uc) {
        constexpr int U = decltype(uc)::value;
        s2[U] = row_s2<B + U, DIM>(xj, xi);
        w[U] = kweight(s2[U], esc);
        qs[U] = rshare<B + U>(qj) + qi;  // w qs = 2 * symmetric P_ij
        d0[U] = rshare<B + U>(mj[0]) - Mi[0];
        d1[U] = rshare<B + U>(mj[1]) - Mi[1];
      });
      exchange_within(accr[0], accr[1], s2, w, qs, d0, d1, lim);
    });
  } else {
    Steps<0, NK>::run([&](auto kc) {
      constexpr int K = decltype(kc)::value;
      const float w = row_weight<K, DIM>(xj, xi, rc2, esc, act);
      const float p = w * (rshare<K>(qj) + qi);  // 2 * symmetric P_ij
#pragma unroll
      for (int s = 0; s < SMAX; ++s) accr[s] += p * (rshare<K>(mj[s]) - Mi[s]);
    });
  }
}

// Exchange over one chunk, row normalisation: rr += w and accr[s] += w
// (m_j[s] - M_i[s]); the caller divides by r_i = rr summed over all chunks.
template <int DIM, int SMAX, int NK = 16>
__device__ __forceinline__ void exchange_chunk_row(const float (&xj)[DIM], const float (&xi)[DIM],
                                                   const float (&mj)[SMAX], const float (&Mi)[SMAX], float rc2,
                                                   float esc, bool act, float& rr, float (&accr)[SMAX]) {
  Steps<0, NK>::run([&](auto kc) {
    constexpr int K = decltype(kc)::value;
    const float w = row_weight<K, DIM>(xj, xi, rc2, esc, act);
    rr += w;
#pragma unroll
    for (int s = 0; s < SMAX; ++s) accr[s] += w * (rshare<K>(mj[s]) - Mi[s]);
  });
}

}  // namespace rwpt
