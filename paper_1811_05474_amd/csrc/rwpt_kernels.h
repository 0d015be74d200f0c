// rwpt_kernels.h -- host-callable launchers of the HIP kernels (internal).
#pragma once
#include "rwpt_device.h"

namespace rwpt {

// Phase identifiers used for per-phase timing.
enum Phase {
  PH_WALK_KEY = 0,
  PH_SCAN,
  PH_SCATTER,
  PH_CANON,
  PH_ROWSUM,
  PH_EXCHANGE,
  PH_AUDIT,
  PH_DENSE,
  PH_COUNT,
  PH_N
};

constexpr int kBlock = 256;        // threads per block of every kernel
constexpr int kScanItems = 16;     // counts per thread in the cell-count scan
constexpr int kScanChunk = kBlock * kScanItems;
// Up to this many scan blocks the cell scan is one launch (one block total per
// thread; beyond, every block would read all the totals before it).
constexpr int64_t kScanDirectMax = 256;
// Words of 64 bits the cell scan keeps for ncell cells: kBlock chunk totals
// and a ticket, or the 32-bit totals of the three-launch form.
inline size_t scan_state_words(int64_t ncell) {
  const int64_t nb = (ncell + kScanChunk - 1) / kScanChunk;
  return (size_t)(nb / 2 + 1 > kBlock + 1 ? nb / 2 + 1 : kBlock + 1);
}

// Random walk + reflection (optional) and cell key / in-cell slot of every particle.
// pos_in/pos_out may not alias.  blk_real[b] is the realisation of particle
// b * kBlock (one entry per block of the launch).  Clears scan_state for the
// cell scan that follows.
hipError_t launch_walk_key(int fp64, int dim, const void* pos_in, void* pos_out,
                           const uint32_t* id, int32_t n, const RealParams* rp,
                           const int64_t* real_start, const int32_t* blk_real, int32_t n_real,
                           const uint64_t* step_ctr,
                           uint64_t seed, int32_t do_walk, uint32_t* cell_count, uint32_t* key,
                           uint32_t* slot, uint64_t* scan_state, hipStream_t s);

// Looks at another block's total before the one-launch cell scan sums that
// chunk itself (about 1 us each: a block that has started answers in a few).
constexpr int32_t kScanPolls = 4096;
// Exclusive scan of cell_count[0..ncell) into cell_start[0..ncell].
// scan_state holds scan_state_words(ncell) words, cleared by launch_walk_key.
// Advances the n_real step counters by bump.
hipError_t launch_cell_scan(const uint32_t* cell_count, uint32_t* cell_start, int64_t ncell, uint64_t* scan_state,
                            uint64_t* step_ctr, int32_t n_real, int32_t bump, int32_t polls, hipStream_t s);

// Place every particle at cell_start[key] + slot (arrival order inside a cell);
// id null: the identity.  Zeroes cell_count[0..ncell) unless it is null.
hipError_t launch_scatter(int32_t n, const uint32_t* key, const uint32_t* slot,
                          const uint32_t* cell_start, const uint32_t* id, uint32_t* tmp_src,
                          uint32_t* tmp_id, uint32_t* tmp_key, uint32_t* cell_count, int64_t ncell, hipStream_t s);

// Reorder inside every cell by particle id (canonical order), gathering
// positions, ids and keys into the sorted arrays, and the masses too when
// src_out is NULL; otherwise the masses stay in the previous order and
// src_out[i] receives the previous slot of sorted particle i.  caller_S > 0:
// mass_in holds the caller's masses, caller_S x n species-major.  inv_out (or
// null) receives the sorted slot of each id.
hipError_t launch_canon(int fp64, int dim, int32_t n, const uint32_t* tmp_src,
                        const uint32_t* tmp_id, const uint32_t* tmp_key,
                        const uint32_t* cell_start, const void* pos_in, void* pos_out,
                        const void* mass_in, void* mass_out, int32_t S,
                        uint32_t* id_out, uint32_t* skey, uint32_t* src_out, int32_t caller_S, uint32_t* inv_out,
                        hipStream_t s);

// Species slots per particle the mass arrays hold for S species: the kernels
// are instantiated for 2, 4 or 8 species and read every slot of their
// instantiation, so slots S..padded_species(S)-1 are allocated and kept zero.
inline int padded_species(int S) { return S <= 2 ? 2 : (S <= 4 ? 4 : 8); }

// Pair kernels (one wave per tile).  log2l: lanes per particle = 1 << log2l,
// or kPrivateLists: one lane per particle with its own candidate rows (tiles
// of 64 particles).
constexpr int kPrivateLists = -1;
// Neighbour cache of the one-lane-per-particle kernels: the row-sum pass keeps
// every in-cutoff neighbour j != i of a lane (sorted index and weight) for the
// exchange pass, in a region of kCacheWave entries owned by the lane's wave.
// A lane with more than kCacheLane neighbours, or whose entries would not fit
// its wave's region, is marked kCacheMiss and searches its stencil again.
constexpr int kCacheLane = 8;
constexpr int kCacheWave = 256;
constexpr uint32_t kCacheMiss = 15;
// From this many expected neighbours the cache keeps them in slots instead
// (PairArgs::nb_slots), read and written in place without LDS: the compacted
// region overflows and its rounds of 64 entries leave most lanes idle.
// 1.5e5 particles in 3-D, eight species, cells of 2 x 1 x 1 per cutoff, whole
// call, compacted / slots: 2 neighbours 91 / 80 us, 4: 103 / 84, 8: 126 / 92,
// 12: 142 / 100; at 0.7 both take 77 (sparse cells: 73 compacted).
// A large ensemble's slots, one line of the memory per lane and entry, leave the
// caches, and the masses have to follow every sort; few neighbours are then
// fewer bytes compacted (a step, us: 3-D in cells of two cutoffs compacted, slots: 8e5
// particles of 1.6 neighbours 116, 112, 1.6e6 171, 188, eight species 195, 242; 1.6e6 of 3
// 263, 238, eight species 298, 296; 2-D: 8e5 of 2 106, 102, 1.6e6 162, 166, eight species
// 188, 224; 1.6e6 of 4 234, 212, 274, 269; binary64 with eight species 8e5 of 1.6 in 3-D
// 181, 190, in 2-D 142, 162).
inline double slots_from(int dim, int64_t n, bool fp64, int S) {
  return n <= (fp64 && S > 4 ? 600000 : 1000000) ? 1.5 : (dim == 3 ? 3.0 : 4.0);
}
constexpr uint16_t kSlotMiss = 0xffff;
// Slots per particle, 0 for the compacted cache.  16 hold nearly all of Poisson
// counts up to a mean of 6, 32 up to 16; beyond, more and more particles fill
// their slots in vain and search again, in large ensembles at more bytes.  Without
// a walk a call fills them once and its steps read them, so they pay for longer
// (`fixed`; the allocation-free call too, for the bits of such a step).  A step,
// compacted / slots in us, fixed and with the walk: 2-D 1e5 particles of 20 neighbours
// 32 / 25, 67 / 63, of 32 38 / 35, 78 / 77; 4e5 of 14 39 / 40, 104 / 105, of 18 47 / 46, 112 /
// 124; 1e6 of 12 88 / 55, 187 / 188, of 18 96 / 84, 204 / 258, of 25 115 / 159; 2e6 of 12
// 163 / 124, 327 / 398, of 16 170 / 167; binary64 1e6 of 10 112 / 76, 244 / 257, of 16
// 121 / 121, 2e6 of 12 216 / 185, 439 / 573.  3-D 1e5 of 40 111 / 90, 192 / 162; 4e5 of 24
// 134 / 110, 236 / 260; 2e6 of 20 471 / 299, 804 / 892, of 24 504 / 516; with eight species
// 4e5 of 24 181 / 174, 288 / 321, binary64 of 20 172 / 111, 320 / 297.  1-D 4e5 of 12 32 / 29
// (binary64), of 16 25 / 31, 69 / 76; 1e6 of 12 49 / 40, 114 / 118; 2e6 of 12 199 / 257 with
// the walk.  3-D realisations of at most 200 particles, most of them one another's
// neighbours from 20 on, then have the cells of two cutoffs that suit them (sparse_cells).
constexpr int64_t kSlotsSizes[3] = {150000, 600000, 1500000};  // particles: up to each, beyond
constexpr double kSlotsUpTo[3][2][2][4] = {  // expected neighbours: dimension, fixed, binary64, size
    {{{16, 12, 10, 10}, {12, 12, 8, 8}}, {{20, 14, 14, 12}, {16, 12, 12, 10}}},
    {{{24, 14, 12, 10}, {20, 14, 8, 8}}, {{32, 18, 20, 16}, {20, 18, 16, 12}}},
    {{{40, 20, 20, 18}, {40, 20, 20, 20}}, {{40, 24, 24, 22}, {40, 24, 22, 22}}}};
inline int slots_for(double nb, int dim, int64_t n, int64_t n_real, bool fp64, int S, bool fixed) {
  int size = 0;
  while (size < 3 && n > kSlotsSizes[size]) ++size;
  double up_to = kSlotsUpTo[dim - 1][fixed][fp64][size];
  if (dim == 3 && n <= 200 * n_real && up_to > 20.0) up_to = 20.0;
  return !(nb > slots_from(dim, n, fp64, S) && nb <= up_to) ? 0 : (nb <= 6.0 ? 16 : 32);
}
// Half-stencil tiling (binary32): every unordered pair evaluated once, its
// far-end share accumulated into slot planes and summed by a finalizer.
constexpr int kHalfPairs = -4;
// Slot planes per direction of the half-stencil tiling: segments of
// ceil(2 * reach / (kHalfParities - 1)) cells, so that a cell row of a
// realisation gives enough work items to fill the device.
constexpr int kHalfParities = 2;
// Candidate evaluations per work item of the half-stencil tiling aimed at on
// average (segments are widened up to this where neighbourhoods are sparse).
constexpr int64_t kHalfTarget = 32768;
// Consecutive blocks of the half-stencil launch that one XCD takes in turn.
constexpr int64_t kHalfGroup = 16;
// Up to this many tiles, the row-broadcast kernels give each tile a whole block
// (its four waves take every fourth chunk of the candidates), so that a small
// ensemble still puts enough waves on the 1024 SIMDs to hide latency.  Whole
// calls in 2-D, split / whole, us: 24000 particles (1500 tiles) of 60 neighbours
// 38.3 / 38.1, of 225 40.6 / 43.8; 40000 of 60 45.9 / 42.0, of 225 50.1 / 49.2; 64000
// of 60 57.2 / 46.3.  Many more candidates per tile keep four waves busy for
// longer (1-D, 32768 particles of 1758 neighbours, a step: 59 / 63 us).
inline int32_t split_tiles_for(double nb) { return nb > 400.0 ? 4096 : 1536; }
hipError_t launch_rowsum(int fp64, int dim, int log2l, const PairArgs& a, hipStream_t s);
hipError_t launch_exchange(int fp64, int dim, int log2l, const PairArgs& a, hipStream_t s);
hipError_t launch_count(int fp64, int dim, int log2l, const PairArgs& a, hipStream_t s);
hipError_t launch_nbr_count(int fp64, int dim, int log2l, const PairArgs& a, hipStream_t s);
hipError_t launch_nbr_fill(int fp64, int dim, int log2l, const PairArgs& a, hipStream_t s);

// Per-realisation FP64 reduction of the per-tile audit partials in two fixed-
// order levels (chunks of at most kAuditChunk tiles inside one realisation,
// then the chunks of each realisation) in one launch; `done` holds n_real
// zeroed completion counters that the kernel returns to zero.  Advances the
// n_real step counters by bump.
// Few, large chunks: every chunk block of a realisation with more than one
// chunk ends in a device-scope fence and a completion atomic on a shared
// counter, which serialise across blocks; a realisation of one chunk needs
// neither.
constexpr int kAuditChunk = 2048;
struct AuditChunk {
  int32_t begin, end;  // tiles [begin, end) of one realisation
  int32_t real;        // that realisation
  int32_t n_in_real;   // chunks of that realisation
};
hipError_t launch_audit_reduce(const double* part, int32_t S1, const AuditChunk* chunks, int32_t nchunks,
                               double* chunk_part, const int32_t* chunk_start, int32_t n_real,
                               double* out, uint32_t* done, uint64_t* step_ctr, int32_t bump,
                               hipStream_t s);

// Allocation-free transfer of one realisation in caller arrays.  Its grid
// parameters and stencil rows travel as kernel arguments (at most
// kNoAllocStencil rows) and are written to device memory for the kernels that
// follow.
constexpr int kNoAllocStencil = 64;
struct NoAllocParams {
  RealParams P;
  StencilRow st[kNoAllocStencil];
  int32_t n_st;
};
// Parameters, stencil, tiles of G particles, cleared counts and scan words;
// then the cell key and place of every particle of the caller's positions (n x
// dim row-major).  mass_out not null: the caller's masses (S x n species-major)
// to the particle-major layout.
hipError_t launch_noalloc_key(int fp64, int dim, int S, const NoAllocParams& a, int32_t n, const void* pos,
                              const void* mass, void* mass_out, Tile* tiles, int32_t G, int32_t ntiles, RealParams* rp,
                              StencilRow* st, uint32_t* cell_count, int64_t ncell, uint64_t* scan_state, uint32_t* key,
                              uint32_t* slot, hipStream_t s);
// The whole sort of realisations of at most kSmallParticles particles and
// kSmallCells cells each, one block per realisation (where small_sort_fits each and
// small_sort_pays).  na: the allocation-free
// call (one realisation, parameters from `na`, written to rp_out, st_out and
// tiles; pos_in and mass_in in the caller's layouts); else null.
constexpr int64_t kSmallParticles = 4096;
constexpr int64_t kSmallCells = 16384;
// 3-D in binary64 with eight species slots: the particles a thread holds spill (one
// realisation, a step, one launch / general, us: 1500 particles 40 / 35, 2500 49 / 36, 4096
// 62 / 36; 75 realisations of 2500 70 / 69), and from 3000 on the step was slower than before
// there was this sort.
inline bool small_sort_fits(int64_t n, int64_t ncell, int dim, bool fp64, int S) {
  return n <= (dim == 3 && fp64 && S > 4 ? kSmallParticles / 2 : kSmallParticles) && ncell <= kSmallCells;
}
// One block per CU: beyond three rounds of them realisations of few particles leave
// most of their threads idle, where the general sort fills the chip (a step, one launch
// / general, us: 512 of 300 2-D 61 / 68, 600 of 50 53 / 54, 1024 of 100 64 / 60, 2048 of 100
// 107 / 89, 10000 of 100 456 / 320, 2048 of 500 264 / 264, 3000 of 700 464 / 474, 10000 of 1000
// 2129 / 2240; of single particles, each of whose realisation the general sort looks
// up, 1200 36 / 53, 2000 50 / 53, 4000 90 / 58).
inline bool small_sort_pays(int64_t n_real, int64_t n) {
  return n_real <= (n < 2 * n_real ? 2048 : 768) || n >= 700 * n_real;
}
struct SmallSortArgs {
  const void* pos_in;
  void* pos_out;           // may be pos_in
  const void* mass_in;
  void* mass_out;          // written in the new order when src_out is null
  uint32_t* src_out;       // else the previous slot of each sorted particle
  const uint32_t* id;
  uint32_t* id_out;        // may be id
  uint32_t* skey;
  uint32_t* cell_start;
  const RealParams* rp;
  uint64_t* step_ctr;      // one per realisation, advanced by bump
  uint64_t seed;
  int32_t do_walk, bump, S;
  RealParams* rp_out;
  StencilRow* st_out;
  Tile* tiles;
  int32_t G, ntiles;
};
hipError_t launch_small_sort(int fp64, int dim, int32_t n_real, const SmallSortArgs& a, const NoAllocParams* na,
                             hipStream_t s);
// Sorted masses (particle-major) back to the caller's order (S x n
// species-major); inv: the sorted slot of each of the caller's particles.
hipError_t launch_noalloc_store(int fp64, int S, int32_t n, const void* mass_sorted, const uint32_t* inv,
                                void* mass, hipStream_t s);

// comps values per particle (stride slots per particle in `in`, cell-sorted) to
// the caller's order in `out`: out[k n + i] (species_major) or out[comps i + k]
// for the caller's particle i = id[p].  inv (n entries) is overwritten with the
// inverse of the id map; *bad (device or page-locked host memory, cleared by the
// caller, or null) is set if an id is not below n.
hipError_t launch_unsort(int fp64, int32_t n, const uint32_t* id, uint32_t* inv, const void* in, void* out, int comps,
                         int stride, int species_major, uint32_t* bad, hipStream_t s);

// Binary64 tiles of 8 or 16 lanes (log2l 3, 4): exponents -s^2 / sigma^2 at the
// cutoff down to -kWideCutoff (results stay normal numbers); wider cutoffs and
// kappa = inf keep the exp of the other binary64 kernels, which ends in zero.
constexpr double kWideCutoff = 700.0;
// Tiles per wave, and the number of tiles from which there are enough waves
// for it.
constexpr int kGroupTiles = 2;
constexpr int32_t kGroupMinTiles = 8192;
hipError_t launch_rowsum64(int dim, int log2l, const PairArgs& a, hipStream_t s);
hipError_t launch_exchange64(int dim, int log2l, const PairArgs& a, hipStream_t s);

// Dense 1-D neighbourhoods by expansions over cells (binary32, tiles of 16
// particles).  Each plan: `refine` cells per cutoff length, terms of the
// expansions, the widest cell in units of sigma (whose truncation is below
// 2e-9 of a weight), the largest g_in, and the mean particles per cell from
// which it is taken.  Plan 2 is the full matrix's, whose "cutoff" is the distance
// of weights 2^-40.
constexpr int kGaussTiles = 8;
constexpr int kGaussPlans = 2;
constexpr int kGaussFull = 2;
constexpr int kGaussMaxTerms = 10;
constexpr int kGaussCells = 8;  // target cells a block takes at a time
constexpr int kGaussCellGroup = 32;  // cells per entry of PairArgs::gauss_cell_real
struct GaussPlan {
  int refine, terms;
  double width;
  int reach;
  int per_cell;
};
constexpr GaussPlan kGaussPlan[kGaussPlans + 1] = {{0, 0, 0.0, 0, 0}, {32, 8, 0.1, 31, 18}, {32, 10, 0.2, 40, 8}};
// Pairs of a step, all realisations, from which a cutoff's expansions pay: up to
// 32768 particles a launch of them is one round of blocks and takes 18 to 22 us
// whatever it holds; the pair tiles' time grows with the pairs (a step with fixed
// positions / with the walk, expansions, tiles, us: 16000 particles of 1200 neighbours 21 /
// 54, 15 / 46, of 1800 19 / 51, 20 / 57; 8000 of 1800 19 / 50, 14 / 49, of 3000 22 / 61, 19 / 67).
constexpr double kGaussPairs = 2.4e7;
// values of the moment buffer for ncell cells of S species
inline size_t gauss_moment_words(int plan, int64_t ncell, int S) {
  return (size_t)kGaussPlan[plan].terms * (size_t)ncell * (2 * padded_species(S) + 2);
}
inline int gauss_rows(int plan) { return 2 * kGaussPlan[plan].reach + 1; }
// tab: n_real * gauss_rows(plan) * terms values
hipError_t launch_gauss_table(int plan, const RealParams* rp, int32_t n_real, double* tab, hipStream_t s);
hipError_t launch_gauss_rowsum(int plan, const PairArgs& a, hipStream_t s);
hipError_t launch_gauss_exchange(int plan, const PairArgs& a, hipStream_t s);

// Full-matrix path of one realisation (binary32 state, bf16-split MFMA).
struct DenseArgs {
  const float* pos;        // [cap][PS] particle-major, sorted
  int64_t cap;
  int32_t n;               // particles (one realisation)
  const float* mass_in;    // [cap][SP] particle-major
  float* mass_out;
  float* q;                // written by the row-sum pass, read by the exchange
  double* r;
  float* bbox;             // [ceil(n / 32)][2 dim]
  float escale;            // -log2(e) / sigma^2
  float skip_s2;           // column tiles at squared distance > skip_s2 hold weights < 2^-40
  __bf16* bparts;          // [3][16 ncb][cap]
  int32_t ncb;             // column blocks of 16 (1 or 2)
  int32_t S, react_a, react_b, norm;
  double* audit_part;      // [ceil(n / 16)][S + 1]
};
constexpr int kDenseRowTile = 16;
constexpr int kDenseColTile = 32;
constexpr int64_t kDenseMaxN = (int64_t)1 << 17;
// column blocks of 16 the contraction needs: [M_s, q M_s, q, 1] (symmetric) or [M_s, 1] (row)
inline int dense_ncb(int S, int norm) { return ((norm == 0 ? 2 * S + 2 : S + 1) + 15) / 16; }
// Tile boxes and row sums (functions of the positions alone), then the exchange.
hipError_t launch_dense_rowsum(int dim, const DenseArgs& a, hipStream_t s);
hipError_t launch_dense_exchange(int dim, const DenseArgs& a, hipStream_t s);

// Instruction-rate probes (register-only kernels of rwpt_probe.hip): binary32
// FMA, binary32 exp2, and the per-candidate code of the row-broadcast row-sum
// and symmetric exchange kernels.  `reps` is iterations (FMA, exp) or chunks
// of 16 candidates (row sum, exchange) per lane; out holds one float per
// thread of the grid (blocks * probe_block()).
enum ProbeKind { PROBE_FMA = 0, PROBE_EXP = 1, PROBE_ROWSUM = 2, PROBE_EXCHANGE = 3 };
int probe_block();
int64_t probe_ops_per_lane(int kind, int reps);
hipError_t launch_probe(int kind, int dim, int slots, int blocks, int reps, float rc2, float esc, float h, float* out,
                        hipStream_t s);

}  // namespace rwpt
