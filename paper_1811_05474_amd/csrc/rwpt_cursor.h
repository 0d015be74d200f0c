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

// Lane `lane` of the chunk starting at virtual index vbase: its candidate j
// (or jdummy when the chunk runs past the segment's last row), advancing the
// cursor over every row that ends inside the chunk.
__device__ __forceinline__ void chunk_pick(RowCursor& c, const RealParams& P, const StencilRow* __restrict__ st,
                                           const uint32_t* __restrict__ cell_start, int cy, int cz, int cxa,
                                           int cxb, uint32_t vbase, int32_t jdummy, int32_t& j, bool& has) {
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
      cursor_advance(c, P, st, cell_start, cy, cz, cxa, cxb);
    } else {
      break;
    }
  }
}

}  // namespace rwpt
