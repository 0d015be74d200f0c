// rwpt_walk.h -- the random walk of one particle and its cell (internal to the
// HIP kernels).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "rwpt_device.h"

namespace rwpt {

// Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11): 10 rounds of the
// multiply/xor S-box with the key bumped by the golden-ratio and sqrt(3)-1
// Weyl constants between rounds.
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint32_t a0 = c[0], a2 = c[2];
    const uint32_t hi0 = __umulhi(0xD2511F53u, a0), lo0 = 0xD2511F53u * a0;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, a2), lo1 = 0xCD9E8D57u * a2;
    c[0] = hi1 ^ c[1] ^ k0;
    c[1] = lo1;
    c[2] = hi0 ^ c[3] ^ k1;
    c[3] = lo0;
  }
}

// Box-Muller pair from the uniforms (u, v): sqrt(-2 ln u) (cos 2 pi v, sin 2 pi v).
// Binary32 uses the hardware log2 / sqrt / sin / cos (sin and cos take the
// angle in revolutions), accurate to ~1e-6 relative -- far below what a
// random displacement needs; binary64 uses the library functions.
__device__ __forceinline__ void box_muller(float u, float v, float* z0, float* z1) {
  const float r = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u));  // -2 ln 2 log2 u
  *z0 = r * __builtin_amdgcn_cosf(v);
  *z1 = r * __builtin_amdgcn_sinf(v);
}
__device__ __forceinline__ void box_muller(double u, double v, double* z0, double* z1) {
  const double r = sqrt(-2.0 * log(u));
  double sn, cs;
  sincospi(2.0 * v, &sn, &cs);
  *z0 = r * cs;
  *z1 = r * sn;
}

// Three standard normals for (particle id, step) under the 64-bit seed:
// counter (id, step lo, step hi, 0); uniforms u = w * 2^-32 + 2^-33;
// Box-Muller on (u0, u1) and (u2, u3).
template <typename T, int DIM>
__device__ __forceinline__ void walk_normals(uint32_t pid, uint64_t seed, uint64_t step, T z[3]) {
  uint32_t c[4] = {pid, (uint32_t)step, (uint32_t)(step >> 32), 0u};
  philox4x32_10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
  const T s32 = (T)2.3283064365386962890625e-10;   // 2^-32
  const T half = (T)1.16415321826934814453125e-10; // 2^-33
  const T u0 = (T)c[0] * s32 + half;
  const T u1 = (T)c[1] * s32 + half;
  box_muller(u0, u1, &z[0], &z[1]);
  z[2] = (T)0;
  if constexpr (DIM > 2) {
    const T u2 = (T)c[2] * s32 + half;
    const T u3 = (T)c[3] * s32 + half;
    T unused;
    box_muller(u2, u3, &z[2], &unused);
  }
}

// Mirror at zero-flux walls until inside the closed box.
template <typename T>
__device__ __forceinline__ T reflect(T x, T lo, T hi) {
  for (int it = 0; it < 64 && (x < lo || x > hi); ++it) x = (x < lo) ? (T)2 * lo - x : (T)2 * hi - x;
  x = x < lo ? lo : x;
  x = x > hi ? hi : x;
  return x;
}

// One walk step of particle pid: drift v dt, isotropic amplitude, extra
// amplitude along v (Eq. 1), mirrored at the walls.
template <typename T, int DIM>
__device__ __forceinline__ void walk_particle(const RealParams& P, uint32_t pid, uint64_t seed, uint64_t step,
                                              T (&x)[DIM]) {
  T z[3];
  walk_normals<T, DIM>(pid, seed, step, z);
  const T amp = (T)P.amp, ampx = (T)P.amp_x;
  T uz = (T)0;
#pragma unroll
  for (int k = 0; k < DIM; ++k) uz += (T)P.udir[k] * z[k];
#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    const T move = (T)P.drift[k] + amp * z[k] + ampx * uz * (T)P.udir[k];
    x[k] = reflect<T>(x[k] + move, (T)P.lo[k], (T)P.hi[k]);
  }
}

// Cell of a position within its realisation's grid.
template <typename T, int DIM>
__device__ __forceinline__ int64_t cell_index(const RealParams& P, const T (&x)[DIM]) {
  int64_t c = 0;
#pragma unroll
  for (int k = DIM - 1; k >= 0; --k) {
    const double u = ((double)x[k] - P.lo[k]) * P.inv_h[k];
    int ck = (int)floor(u);
    ck = ck < 0 ? 0 : ck;
    ck = ck > P.nc[k] - 1 ? P.nc[k] - 1 : ck;
    c = c * P.nc[k] + ck;
  }
  return c;
}

}  // namespace rwpt
