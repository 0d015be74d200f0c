// rwpt_cursor.h -- a tile segment's candidates as one virtual list (internal to
// the HIP kernels).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rwpt_device.h"

namespace rwpt {

// Between a wave's LDS stores and its loads of what other lanes of the same
// wave stored: the LDS executes one wave's operations in order, so only the
// compiler has to be kept from moving the loads above the stores.
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Wave-uniform cursor over the non-empty stencil rows of one segment.
struct RowCursor {
  int r;            // next stencil entry to examine
  uint32_t jb, je;  // current row's sorted candidate range
  uint32_t p;       // virtual index of jb
  bool valid;
};

__device__ __forceinline__ void cursor_advance(RowCursor& c, const RealParams& P, const StencilRow* __restrict__ st,
                                               const uint32_t* __restrict__ cell_start, int cy, int cz, int cxa,
                                               int cxb) {
  const int nc0 = P.nc[0], nc1 = P.nc[1], nc2 = P.nc[2];
  c.valid = false;
  while (c.r < P.n_stencil) {
    const StencilRow sr = st[P.stencil_off + c.r];
    ++c.r;
    const int ny = cy + sr.dy, nz = cz + sr.dz;
    if (ny < 0 || ny >= nc1 || nz < 0 || nz >= nc2) continue;
    const int xa = cxa - sr.rx < 0 ? 0 : cxa - sr.rx;
    const int xb = cxb + sr.rx > nc0 - 1 ? nc0 - 1 : cxb + sr.rx;
    const int64_t cb = P.cell_off + ((int64_t)nz * nc1 + ny) * nc0;
    const uint32_t jb = cell_start[cb + xa], je = cell_start[cb + xb + 1];
    if (je > jb) {
      c.jb = jb;
      c.je = je;
      c.valid = true;
      return;
    }
  }
}

// A segment's row ranges looked up together: row r's in lane r, one round of
// loads instead of one per row.  For launches too small to hide those rounds
// behind other waves (a call of 2000 particles of 25
// neighbours in 2-D 26.0 -> 22.9 us, 60000 of 60 neighbours 64 -> 56); with
// enough waves the lane accesses cost more than the scalar lookups they replace
// (1e6 particles: row sums 136.6 -> 139.2 us, exchange 208.1 -> 216.3).
struct RowTable {
  static constexpr int kRows = 64;  // of a stencil: one per lane
  uint32_t jb, je;
  __device__ __forceinline__ void load(const RealParams& P, const StencilRow* __restrict__ st,
                                       const uint32_t* __restrict__ cell_start, int cy, int cz, int cxa, int cxb) {
    const int lane = threadIdx.x & 63;
    const int nc0 = P.nc[0], nc1 = P.nc[1], nc2 = P.nc[2];
    jb = je = 0u;
    if (lane < P.n_stencil) {
      const StencilRow sr = st[P.stencil_off + lane];
      const int ny = cy + sr.dy, nz = cz + sr.dz;
      if (ny >= 0 && ny < nc1 && nz >= 0 && nz < nc2) {
        const int xa = cxa - sr.rx < 0 ? 0 : cxa - sr.rx;
        const int xb = cxb + sr.rx > nc0 - 1 ? nc0 - 1 : cxb + sr.rx;
        const int64_t cb = P.cell_off + ((int64_t)nz * nc1 + ny) * nc0;
        jb = cell_start[cb + xa];
        je = cell_start[cb + xb + 1];
      }
    }
  }
  __device__ __forceinline__ void advance(RowCursor& c, const RealParams& P) const {
    c.valid = false;
    while (c.r < P.n_stencil) {
      const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)jb, c.r);
      const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)je, c.r);
      ++c.r;
      if (e > b) {
        c.jb = b;
        c.je = e;
        c.valid = true;
        return;
      }
    }
  }
};

// Lane `lane` of the chunk starting at virtual index vbase: its candidate j
// (or jdummy when the chunk runs past the segment's last row), advancing the
// cursor with advance(c) over every row that ends inside the chunk.
template <typename AdvanceFn>
__device__ __forceinline__ void chunk_pick(RowCursor& c, AdvanceFn&& advance, uint32_t vbase, int32_t jdummy,
                                           int32_t& j, bool& has) {
  const uint32_t v = vbase + (uint32_t)(threadIdx.x & 63);
  j = jdummy;
  has = false;
  while (c.valid) {
    const uint32_t len = c.je - c.jb;
    if (v >= c.p && v < c.p + len) {
      j = (int32_t)(c.jb + (v - c.p));
      has = true;
    }
    if (c.p + len <= vbase + 64) {
      c.p += len;
      advance(c);
    } else {
      break;
    }
  }
}

}  // namespace rwpt
