// rwpt_smallsort.hip -- the sort of small realisations in one launch: walk, cell
// keys, counts, cell starts, canonical order and gather, one block per
// realisation.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "rwpt_kernels.h"
#include "rwpt_layout.h"
#include "rwpt_walk.h"

namespace rwpt {

constexpr int kSmallBlock = 1024;
constexpr int kSmallItems = (int)(kSmallParticles / kSmallBlock);

// LDS word of cell k: one pad word per 16, so that threads scanning consecutive
// runs of counts meet in few banks (2000 particles: 10.7 -> 9.7 us).
__device__ __forceinline__ int cell_word(int k) { return k + (k >> 4); }

// The launches of the general sort (walk + key, scan, scatter, canonical
// gather) take 3 to 5 us each and a gap, whatever they sort; here their steps
// are separated by block barriers.  Bound by that chain's latency: 2000
// particles of 8000 cells, 9.7 us, before that 24 and five gaps between seven
// launches (the whole call 37.9 -> 28.4 us); 75 realisations of 2000 in 1-D 8.8
// us, before 24 and three gaps (a step 55 -> 41 us).  Limit: what fits the LDS of
// one block and stays shorter than the launches.
// Inside a cell the order is by id.  In a cell of up to kBigCell particles each
// counts the smaller ids; in a larger one, where that grows with the square and
// runs on one CU, the cell's ids are marked in a bitmap over the realisation's and
// a particle counts the bits below its own (a step of 4096 particles in one cell
// 820 -> 46 us, 650 with the general sort; half of 4096 in one cell 184 -> 42).
// The search for large cells costs the others 0.16 us.
// A realisation's particles, counts and cell starts never leave the block: its
// positions are all read (into registers) before any is written, so pos_out may
// be pos_in.
// NA (the allocation-free call): one realisation whose parameters come as
// arguments and are written out for the kernels that follow, masses in the
// caller's order (S x n species-major), ids = indices, no walk.
constexpr uint32_t kBigCell = 128;
constexpr int kBigCells = (int)(kSmallParticles / (kBigCell + 1));
constexpr int kIdWords = (int)(kSmallParticles / 32);
static_assert(kIdWords == 128, "two words per lane of the wave that sums a cell's bitmap");
static_assert(kSmallParticles < (1 << 16) && kBigCells < (1 << 16), "a cell's word holds its start and its bitmap");

template <typename T, int DIM, int SMAX, bool NA>
__global__ __launch_bounds__(kSmallBlock) void k_small_sort(const SmallSortArgs a, const NoAllocParams na) {
  __shared__ uint32_t cnt[kSmallCells + kSmallCells / 16 + 1];
  __shared__ uint32_t sid[kSmallParticles];
  __shared__ uint32_t sh[kSmallBlock / 64];
  __shared__ uint32_t bits[kBigCells][kIdWords];   // the ids of a large cell
  __shared__ uint16_t below[kBigCells][kIdWords];  // how many lie in earlier words
  __shared__ uint32_t any_big, n_big;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = NA ? 0 : (int)blockIdx.x;
  const RealParams& P = NA ? na.P : a.rp[r];
  const int n = (int)(P.p_end - P.p_begin), ncell = P.nc[0] * P.nc[1] * P.nc[2];
  const int64_t p0 = P.p_begin;
  const T* __restrict__ mass_in = (const T*)a.mass_in;
  uint32_t* __restrict__ start = a.cell_start + P.cell_off;
  if (n <= 0) {  // an empty realisation keeps its cells and its counter
    for (int k = tid; k <= ncell; k += kSmallBlock) start[k] = (uint32_t)p0;
    if (!NA && tid == 0) a.step_ctr[r] += (uint64_t)a.bump;
    return;
  }
  for (int k = tid; k < ncell; k += kSmallBlock) cnt[cell_word(k)] = 0u;
  if (tid == 0) any_big = n_big = 0u;
  if constexpr (NA) {
    if (tid == 0) a.rp_out[0] = na.P;
    if (tid < na.n_st) a.st_out[tid] = na.st[tid];
    for (int t = tid; t < a.ntiles; t += kSmallBlock) {
      const int32_t b = t * a.G;
      a.tiles[t] = Tile{b, b + a.G < n ? b + a.G : n, 0, 0};
    }
  }
  T x[kSmallItems][DIM], m[kSmallItems][SMAX];
  uint32_t id[kSmallItems], key[kSmallItems], slot[kSmallItems];
#pragma unroll
  for (int u = 0; u < kSmallItems; ++u) {
    const int o = tid + u * kSmallBlock;
    const int64_t p = p0 + (o < n ? o : n - 1);
    if constexpr (NA) load_pos_unaligned<T, DIM>((const T*)a.pos_in, p, x[u]);
    else load_pos<T, DIM>((const T*)a.pos_in, p, x[u]);
    id[u] = NA ? (uint32_t)p : a.id[p];
    if (a.src_out == nullptr) {
      if constexpr (NA) {
#pragma unroll
        for (int s = 0; s < SMAX; ++s) m[u][s] = s < a.S ? mass_in[(int64_t)s * n + p] : (T)0;
      } else {
        load_mass<T, SMAX>(mass_in, p, m[u]);
      }
    }
  }
  const uint64_t step = !NA && a.do_walk ? a.step_ctr[r] : 0u;
  __syncthreads();  // cnt is clear
#pragma unroll
  for (int u = 0; u < kSmallItems; ++u) {
    const int o = tid + u * kSmallBlock;
    if (o < n) {
      if (!NA && a.do_walk && P.moves) walk_particle<T, DIM>(P, id[u], a.seed, step, x[u]);
      key[u] = (uint32_t)cell_index<T, DIM>(P, x[u]);
      slot[u] = atomicAdd(&cnt[cell_word(key[u])], 1u);
      if (slot[u] >= kBigCell) any_big = 1u;
    }
  }
  __syncthreads();
  if (!NA && tid == 0) a.step_ctr[r] += (uint64_t)a.bump;  // every thread has read it
  // exclusive scan in place, consecutive counts per thread
  constexpr int kPer = kSmallCells / kSmallBlock;
  const int per = (ncell + kSmallBlock - 1) / kSmallBlock, c0 = tid * per;
  uint32_t sum = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k)
    if (k < per && c0 + k < ncell) sum += cnt[cell_word(c0 + k)];
  uint32_t v = sum;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t t = __shfl_up(v, off);
    if (lane >= off) v += t;
  }
  if (lane == 63) sh[wave] = v;
  __syncthreads();
  const uint32_t large = any_big;  // some cell is
  uint32_t run = v - sum;
  for (int w = 0; w < wave; ++w) run += sh[w];
#pragma unroll
  for (int k = 0; k < kPer; ++k)
    if (k < per && c0 + k < ncell) {
      const uint32_t c = cnt[cell_word(c0 + k)];
      cnt[cell_word(c0 + k)] = run;
      run += c;
    }
  __syncthreads();
  // kRanked + its rank in slot for a particle of a large cell
  constexpr uint32_t kRanked = 1u << 31;
  // (unlikely, but laid out of line it makes binary64 with eight species spill)
  bool ranked = __builtin_amdgcn_readfirstlane(large) != 0u;
  if constexpr (sizeof(T) * SMAX <= 32) ranked = __builtin_expect(ranked, false);
  if (ranked) {
    // a large cell's bitmap, plus one, above its start
    for (int k = tid; k < ncell; k += kSmallBlock) {
      const uint32_t c = cnt[cell_word(k)] & 0xffffu;
      const uint32_t e = k + 1 < ncell ? cnt[cell_word(k + 1)] & 0xffffu : (uint32_t)n;
      if (e - c > kBigCell) cnt[cell_word(k)] = c | (atomicAdd(&n_big, 1u) + 1u) << 16;
    }
    __syncthreads();
    for (int k = tid; k < (int)n_big * kIdWords; k += kSmallBlock) (&bits[0][0])[k] = 0u;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSmallItems; ++u)
      if (tid + u * kSmallBlock < n) {
        const uint32_t b = cnt[cell_word(key[u])] >> 16, l = id[u] - (uint32_t)p0;
        if (b) atomicOr(&bits[b - 1u][l >> 5], 1u << (l & 31u));
      }
    __syncthreads();
    for (int b = wave; b < (int)n_big; b += kSmallBlock / 64) {
      const uint32_t first = (uint32_t)__popc(bits[b][2 * lane]);
      const uint32_t both = first + (uint32_t)__popc(bits[b][2 * lane + 1]);
      uint32_t t = both;
      // (unrolled, it shares its lanes' addresses with the scan above, and they take ten
      // registers from there to here)
#pragma unroll 1
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t s = __shfl_up(t, off);
        if (lane >= off) t += s;
      }
      below[b][2 * lane] = (uint16_t)(t - both);
      below[b][2 * lane + 1] = (uint16_t)(t - both + first);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSmallItems; ++u)
      if (tid + u * kSmallBlock < n) {
        const uint32_t b = cnt[cell_word(key[u])] >> 16, l = id[u] - (uint32_t)p0;
        if (b)
          slot[u] = kRanked + below[b - 1u][l >> 5] + (uint32_t)__popc(bits[b - 1u][l >> 5] & ((1u << (l & 31u)) - 1u));
      }
    __syncthreads();
    for (int k = tid; k < ncell; k += kSmallBlock) cnt[cell_word(k)] &= 0xffffu;
    __syncthreads();
  }
  for (int k = tid; k < ncell; k += kSmallBlock) start[k] = (uint32_t)p0 + cnt[cell_word(k)];
  if (tid == 0) start[ncell] = (uint32_t)P.p_end;  // the next realisation writes the same
#pragma unroll
  for (int u = 0; u < kSmallItems; ++u) {
    const int o = tid + u * kSmallBlock;
    if (o < n && slot[u] < kRanked) sid[cnt[cell_word(key[u])] + slot[u]] = id[u];
  }
  __syncthreads();
  // canonical order inside a cell: by id
#pragma unroll
  for (int u = 0; u < kSmallItems; ++u) {
    const int o = tid + u * kSmallBlock;
    if (o < n) {
      const uint32_t cs = cnt[cell_word(key[u])];
      uint32_t rank = slot[u] & ~kRanked;
      if (slot[u] < kRanked) {
        const uint32_t ce = (int)key[u] + 1 < ncell ? cnt[cell_word(key[u] + 1)] : (uint32_t)n;
        rank = 0;
        for (uint32_t f = cs; f < ce; ++f) rank += sid[f] < id[u] ? 1u : 0u;
      }
      const int64_t dst = p0 + cs + rank;
      store_pos<T, DIM>((T*)a.pos_out, dst, x[u]);
      if (a.src_out) a.src_out[dst] = (uint32_t)(p0 + o);
      else store_mass<T, SMAX>((T*)a.mass_out, dst, m[u]);
      a.id_out[dst] = id[u];
      a.skey[dst] = (uint32_t)P.cell_off + key[u];
    }
  }
}

hipError_t launch_small_sort(int fp64, int dim, int32_t n_real, const SmallSortArgs& a, const NoAllocParams* na,
                             hipStream_t s) {
  static const NoAllocParams none{};
  const dim3 g((unsigned)(na ? 1 : n_real)), b(kSmallBlock);
  auto go = [&](auto t, auto d, auto sm) {
    using T = decltype(t);
    constexpr int D = decltype(d)::value, SM = decltype(sm)::value;
    if (na) hipLaunchKernelGGL((k_small_sort<T, D, SM, true>), g, b, 0, s, a, *na);
    else hipLaunchKernelGGL((k_small_sort<T, D, SM, false>), g, b, 0, s, a, none);
  };
  auto with_s = [&](auto t, auto d) {
    if (a.S <= 2) go(t, d, std::integral_constant<int, 2>{});
    else if (a.S <= 4) go(t, d, std::integral_constant<int, 4>{});
    else go(t, d, std::integral_constant<int, 8>{});
  };
  auto with_d = [&](auto t) -> hipError_t {
    if (dim == 1) with_s(t, std::integral_constant<int, 1>{});
    else if (dim == 2) with_s(t, std::integral_constant<int, 2>{});
    else if (dim == 3) with_s(t, std::integral_constant<int, 3>{});
    else return hipErrorInvalidValue;
    return hipGetLastError();
  };
  return fp64 ? with_d(double{}) : with_d(float{});
}

}  // namespace rwpt
