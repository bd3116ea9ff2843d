// Internal declarations shared by the host runtime (qw_host.cpp) and the
// HIP kernels (qw_kernels.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace qwk {

// Layout of the coined general path: contiguous vertex ranges whose arcs fit
// one workgroup's LDS tile are processed together.
constexpr int kTileArcs = 2048;
constexpr int kTileThreads = 256;
constexpr int kCoinedTileThreads = 512;  // single coined walks: four gathers in flight per thread
// The LDS-staged batch stage, per state type: workgroup size, the LDS block of
// the input vector it stages (whole rounds of 1 KiB direct loads by every
// wavefront) and rows per thread for walks of degree d (1..8).  A row takes d
// index and four sum registers, so sparser walks fit more rows.  Chosen on the
// kernel as it was before its last loads were cut, where one row more than here
// spilled (96 walks of one degree, complex64, ms a pass: degree 3 with 12, 13, 14
// rows 7.7, 8.6, 9.2; degree 4 with 11, 12 8.4, 8.7; degree 5 with 10, 11, 12
// 10.0, 9.4, 9.7).
constexpr int kLdsTileThreads64 = 768;
constexpr int kLdsBlockBytes64 = 156 * 1024;
constexpr int kLdsTileThreads128 = 1024;
constexpr int kLdsBlockBytes128 = 144 * 1024;
constexpr int lds_rows_per_thread(bool c128, int d) {
  constexpr int r64[9] = {12, 12, 12, 12, 11, 11, 10, 9, 9}, r128[9] = {8, 8, 8, 8, 8, 7, 7, 6, 6};
  return c128 ? r128[d] : r64[d];
}
constexpr int lds_tile_rows(bool c128, int d) {
  return lds_rows_per_thread(c128, d) * (c128 ? kLdsTileThreads128 : kLdsTileThreads64);
}
// single-walk ELL stage: vectors above kEllSliceFrom bytes are gathered in
// slices of kEllSliceEntries entries (measured best on 2^20 vertices for both
// types, against 64Ki and 256Ki: 1 MiB complex64, 2 MiB complex128).  The
// slicing pays from about 8 MiB on (random 6-regular graphs: 9.6 MiB and up
// faster, 4.8 MiB complex64 even, 7.2 MiB complex128 and below slower).
#ifndef QW_ELL_SLICE_FROM
#define QW_ELL_SLICE_FROM (int64_t{15} << 19)
#endif
constexpr int64_t kEllSliceFrom = QW_ELL_SLICE_FROM;
constexpr int kEllSliceEntries = 131072;
#ifndef QW_ELL_SLICE_ROWS
#define QW_ELL_SLICE_ROWS 2
#endif
constexpr int kEllSliceRows = QW_ELL_SLICE_ROWS;  // rows per thread of the sliced stage
constexpr int kDirRows = 256;   // rows per workgroup tile of the direct out-of-core stage (one per thread)
constexpr int kDirArcs = 8192;  // neighbour indices such a tile stages in LDS (32 KiB)
constexpr int kLinkCopyGroups = 16;  // workgroups of the device-to-pinned-host copy (enough for the link)
constexpr int kTileMaxVerts = 1024;
// Threads per workgroup of the elementwise/stencil kernels.
constexpr int kBlock = 256;
// LDS budget of the one-workgroup whole-walk kernels.
constexpr size_t kSmallLdsBytes = 156 * 1024;  // dynamic LDS of the one-workgroup path (of 160 KiB)
// The one-workgroup CTQW keeps the neighbours of a thread's vertices in
// registers.  Of `per_thread` vertices (1, 2 or 4, the i-th of rank
// i * 1024 + thread in falling degree) the i-th may have this many: 128
// registers a thread hold no more.
constexpr int small_row(bool c128, int per_thread, int i) {
  if (per_thread == 1) return c128 ? 24 : 32;
  if (per_thread == 2) return c128 ? (i == 0 ? 16 : 8) : (i == 0 ? 24 : 16);
  return c128 ? 8 : (i == 0 ? 16 : 8);
}
// CSR stages with 16 lanes a row and more (rows of 3 to 6 arcs a lane) have eight of
// a lane's arcs in flight up to this many threads.  Few wavefronts wait for
// memory, and the loads in flight serve them; many hide it, and the tests for
// arcs that are not there cost more.  us for two steps, in flight and one by one:
// 3000 vertices of mean degree 80 (48000 threads) 106 and 135, of 250 (192000)
// 125 and 145; 20000 of 80 (320000) 236 and 217, of 150 (640000) 376 and 331.
constexpr int kCsrBatchedThreads = 1 << 18;

// Arcs lane, lane + G, ... of the row [lo, hi), M at a time.  Plans have up to
// 2^31 - 1 arcs, so an index past hi is never formed.
template <int G, int M> struct LaneArcs {
  int hi, left;
  constexpr LaneArcs(int lo, int hi_, int lane) : hi(hi_), left(hi_ - lo - lane) {}
  constexpr bool more() const { return left > 0; }
  constexpr bool has(int m) const { return m * G < left; }
  constexpr int at(int m) const { return hi - left + m * G; }
  constexpr void next() { left -= M * G; }
};
// The lane's arcs of a row, counted as the kernels walk them (an overflow in a
// constant expression does not compile).
template <int G, int M> constexpr int lane_arcs(int lo, int hi, int lane) {
  int n = 0;
  for (LaneArcs<G, M> a(lo, hi, lane); a.more(); a.next())
    for (int m = 0; m < M; ++m)
      if (a.has(m) && a.at(m) == lo + lane + n * G) ++n;
  return n;
}
static_assert(lane_arcs<2, 8>(0, 35, 1) == 17 && lane_arcs<64, 8>(7, 8, 1) == 0 && lane_arcs<4, 8>(9, 9, 0) == 0);
static_assert(lane_arcs<2, 8>(0x7fffffff - 21, 0x7fffffff, 0) == 11 && lane_arcs<64, 8>(0x7fffffff - 600, 0x7fffffff, 63) == 9 &&
              lane_arcs<64, 8>(0x7fffffff - 1, 0x7fffffff, 63) == 0);

// Largest hypercube dimension the structured kernels handle.
constexpr int kMaxHypercubeDim = 30;

enum Structure : int32_t {
  kGeneral = 0, kCycle = 1, kTorus = 2, kHypercube = 3, kSmall = 4, kEll = 5, kDense = 6, kStagLattice = 7
};
// Dense-H GEMM tiles: rows of H per workgroup, k per LDS chunk.
constexpr int kDenseRows = 64;
constexpr int kDenseK = 32;  // H's leading dimension and split-k ranges are multiples of it
constexpr int kMaxDenseColumns = 128;
constexpr int kMaxDenseSplits = 8;
// Largest degree of the ELL (regular-graph) CTQW layout.
constexpr int kMaxEllDegree = 64;

// Grid CTQW strips (streaming temporal blocking): one wavefront sweeps a strip
// of 64 columns; strips are sized so each SIMD gets two of them (complex64,
// strips of at least 2S core rows), else one (at least kSweepMinRowsPerStage
// * S rows).
constexpr int kStripWaves = 4;  // wavefronts (strips) per workgroup
constexpr int kSimds = 256 * 4;  // MI355X: 256 compute units of 4 SIMDs
constexpr int kSweepMinRowsPerStage = 4;

// Coined grid sweep: steps per launch by type and coin, and rows read ahead.
// Measured over 2 to 6 steps, 3 to 6 rows ahead and one to two wavefronts per
// SIMD (us for 50 steps of 1024^2 Fourier complex64, 150 of 707 x 709 Grover
// complex128, 150 of 700^2 Grover complex64, 50 of 700^2 Fourier complex128):
//   steps         2      3      4      5      6
//   Fourier c64   464    442    432    417    430
//   Grover c128   1006   738    623    536    515
//   Grover c64    674    522    460    448    469
//   Fourier c128  479    333    299    346    332
// More steps move fewer bytes per step but compute more halo: the matrix coin
// (96 FP64 operations per vertex) pays for that first.  Three rows ahead are
// best throughout, and one wavefront per SIMD (two: 5-30% slower).
constexpr int kCoinedSteps64 = 5, kCoinedSteps128 = 6, kCoinedMatrixSteps128 = 4;
constexpr int kCoinedAhead = 3;
// Grids below these cells take the matrix coin one step per launch: a strip has
// twice its halo's rows at least, and on a small grid the chain of that many rows
// of FP64 products in each of few wavefronts takes longer than the launches it
// saves.  us for 50 steps one by one and swept:
//   cells              22500  65536  90000  122500  160000  202500  250000  302500
//   Fourier c64, one     157    165    178     188     211     235     245     271
//                swept   217    220    223     225     229     233     237     240
//   Fourier c128, one    170    191    208     231     256
//                 swept  198    204    211     216     219
// and on narrow ones, 64 x 4000 complex64 245 and 254, 64 x 2000 complex128 234
// and 239, 64 x 2400 220 and 208.
constexpr int64_t kCoinedMatrixFrom64 = 300000, kCoinedMatrixFrom128 = 150000;

// Square-lattice sweep: steps per launch by type, and row pairs read ahead.
// Measured, one wavefront per SIMD (us for 60 steps of 768 x 1100 complex128 and
// of 760 x 1000 complex64, 24 of 2048^2; two steps per launch through LDS tiles
// 405, 308, 493 and 377):
//   steps, pairs ahead       3, 1   4, 1   6, 1   3, 2   4, 2   6, 2   4, 4
//   768 x 1100 complex128    179    169    160    186    174    179    195
//   2048^2 complex128        237    193    168    238    198    178    209
//   760 x 1000 complex64     181    180    178    167    168    182    184
//   2048^2 complex64         212    192    187    179    177    188    194
// Reading further ahead unrolls the loop further, and the longer code costs more
// in instruction fetches than the loads it hides; two wavefronts per SIMD are
// 5-40% slower (more halo).
constexpr int kStagSteps64 = 4, kStagSteps128 = 6;
constexpr int kStagAhead64 = 2, kStagAhead128 = 1;

// Two-column complex64 grid sweep: stages per launch, K split into launches of
// nearly equal depth.  Measured against the one-column sweep (S = 5, or the
// largest of 5, 4, 3, 2 that divides K; us per step; waves per SIMD in brackets):
//                           one col.  6 (1)  6 (2)  7 (1)  10 (1)  10 (2)
//   128^2        K 20          31.6    16.8   16.8   19.2   22.4   22.4
//   300 x 301    K 12 marked   24.1    17.3   17.2   17.3   17.2   17.4
//   700 x 300    K 20          31.8    21.6   24.4   21.6   25.8   28.8
//   601 x 777    K 15          24.1    19.7   20.9   19.2   20.3   22.0
//   601 x 777    K 20 marked   41.4    35.5   35.1   36.9   37.7   37.5
//   601 x 777    K 14 marked   33.0    24.9   24.4   26.3   26.4   25.2
//   1024^2       K 20          33.7    35.1   33.9   34.7   38.4   37.9
//   1024^2       K 20 marked   38.2    50.3   41.8   49.4   49.5   44.7
//   2048^2       K 20          78.8    82.1   81.1   76.2   76.5   66.8
//   2048^2       K 20 marked   89.4     116   97.3    108   98.1   78.9
//   3000^2       K 20           153     173    154    145    136    104
// and on either side of the lines below, the marks again costing most:
//                                   one col.  6 (1)  10 (2)
//   700^2         K 9 marked          18.1    16.7   15.7
//   800^2         K 9 marked          15.8    17.1   16.5
//   5400 x 128    K 24 marked         43.2    56.7   45.7
//   830^2         K 24 marked         49.8    48.0   41.0
//   900^2         K 24 marked         43.1    50.4   43.5
//   1200^2        K 20                39.2    41.7   42.5
//   1448^2        K 14 marked         67.9    53.1   36.1
//   700 x 3010    K 20 marked         51.1           54.0
//   16500 x 128   K 20                55.0           57.9
//   1800 x 1801   K 20 marked         69.6    99.6   66.8
// Small grids are bound by launches and by the chain of one wavefront's stages,
// large ones by memory, which deep launches pass less often.  Small is measured
// in the cells that the strips cover (of 128 columns two strips cover 232); the
// lines with Few are for K that only divides by 2 or 3, whose other choice is
// shallower launches.  Between the lines those K take 6 (2), and the others one
// column, as they do on large grids of which the strips cover an eighth twice.
constexpr int kDeepStages = 10, kDeepStagesSmall = 6, kDeepUnroll = 3;
constexpr int64_t kDeepSmall = 780000, kDeepSmallFew = 600000;
constexpr int64_t kDeepLarge = 3000000, kDeepLargeFew = int64_t{1} << 21;

// Strip decomposition of an l1 x l2 grid for S stages per launch.
struct StripGrid {
  int rows = 0;     // core rows per strip
  int width = 0;    // columns a wavefront holds
  int core = 0;     // core columns = width - 2S
  int halo = 0;     // S
  int tiles_r = 0;  // strips along the rows (last one clamped to the grid edge)
  int tiles_c = 0;
  int64_t count() const { return static_cast<int64_t>(tiles_r) * tiles_c; }
};

// Staggered walk: polygons of at most kStagThreadMax vertices are handled one
// per thread; larger ones are cut into chunks of at most kStagChunk positions,
// one workgroup per chunk (partial inner products, then the update).
constexpr int kStagThreadMax = 16;
constexpr int kStagChunk = 2048;
constexpr int kStagMaxTess = 64;
constexpr int kStagRegSize = 4;  // one-workgroup walks: polygons up to this size fit a thread's registers

// One tessellation of a staggered walk as the kernels see it.  Offsets are
// bytes from the start of the plan's device buffer (-1: absent).
struct StagTess {
  int32_t n_small = 0;     // polygons on the thread path
  int32_t small_size = 0;  // > 0: all of size small_size, column-major table vert[j*n_small + p]; 0: CSR
  int32_t max_small = 0;   // largest thread-path polygon
  int32_t n_big = 0;       // polygons above kStagThreadMax vertices
  int32_t n_chunks = 0;    // chunks of the big polygons
  int32_t pad = 0;
  int64_t off_ptr = -1;    // thread path, CSR: int32[n_small + 1]
  int64_t off_vert = -1;   // thread path: int32 vertices
  int64_t off_amp = -1;    // thread path: double amplitudes (same layout as vert), -1 = uniform
  int64_t off_bptr = -1;   // big polygons: int32[n_big + 1] into bvert
  int64_t off_bvert = -1;
  int64_t off_bamp = -1;   // -1 = uniform
  int64_t off_chunk = -1;  // StagChunk[n_chunks]
  double c0[2] = {0.0, 0.0};  // U = c0 I + c1 (2P - I): reflection (0, 1), Hamiltonian (cos t, i sin t)
  double c1[2] = {1.0, 0.0};
};

// A chunk of a big polygon: positions [begin, end) of bvert; the polygon's
// chunks are first .. first + count - 1.
struct StagChunk {
  int32_t begin;
  int32_t end;
  int32_t first;
  int32_t count;
  int32_t size;  // vertices of the polygon
  int32_t pad[3];
};

// Device view of a plan's graph tables (pointers into the caller's buffer).
struct GraphView {
  int32_t n = 0;
  int32_t n_arcs = 0;
  int32_t structure = kGeneral;
  int32_t dims[2] = {0, 0};
  int32_t n_marked = 0;
  int32_t n_tiles = 0;
  int32_t group = 1;           // CTQW CSR: lanes per row
  int32_t sorted_rows = 0;     // CTQW CSR: every row's neighbours in increasing order
  const int32_t *rp = nullptr;      // n+1
  const int32_t *col = nullptr;     // n_arcs (CTQW general/small: CSR order; ELL: col[j*n + v])
  int32_t ell_d = 0;                // ELL degree
  int32_t columns = 1;              // dense: walks sharing H
  int32_t ld = 0;                   // dense: leading dimension of H (multiple of kDenseK)
  void *dense = nullptr;            // dense: H, rows padded to kDenseRows, FP64 or FP32
  double *dense_partial = nullptr;  // dense: split-k partial products (workspace)
  const int32_t *rev = nullptr;     // n_arcs (coined general/small)
  const int32_t *tiles = nullptr;   // n_tiles+1 (coined general)
  const int32_t *perm = nullptr;    // n_arcs (coined structured: slot-major -> CSR position)
  const uint32_t *markbits = nullptr;  // ceil(n/32)
  const int32_t *marklist = nullptr;   // n_marked
  const uint8_t *tmark = nullptr;      // grid CTQW strips: 1 if a marked vertex lies in the strip's window
  int32_t strip_rows = 0;              // grid CTQW strips: core rows per strip
  int32_t two_reg = 0;                 // coined, one workgroup: 1 if every vertex has degree 2 and n <= 64
                                       // (amplitudes in one wavefront's registers), 2 if moreover a cycle in
                                       // direction order (rev[2v] = 2(v+1)+1, rev[2v+1] = 2(v-1), mod n)
  int32_t persistent = 0;              // coined on a lattice: persistent shift
  const double *coin = nullptr;        // coined on a lattice: d x d complex coin (row-major), else null
  const double *sqrtp = nullptr;       // Szegedy coin: sqrt(P) per arc, else null
  const unsigned char *base = nullptr; // start of the plan's device buffer
  // Every launch carries a GraphView, so the two share their place: with 8 bytes
  // more, 40 steps on a 6-regular graph of 10^6 vertices took 25.08 ms, not 24.99.
  union {
    const StagTess *stag = nullptr;    // staggered: device array of n_tess descriptors
    const int32_t *order;              // CTQW, one workgroup, tables in registers: vertices by falling degree
  };
  int32_t n_tess = 0;
  int32_t stag_regs = 0;               // staggered, one workgroup: polygons kept in registers (small_stag_regs)
};

;

// One walk of a many-small-walks launch (the whole walk in one workgroup's LDS).
struct SmallWalk {
  GraphView g;
  void *psi = nullptr;
  int32_t coined = 0;
  int32_t hadamard = 0;
  int32_t K = 0;
  int32_t staggered = 0;
  int64_t steps = 0;
  double alpha[64] = {};  // CTQW stage coefficients gamma dt / k, dt / k
  double beta[64] = {};
};

// Readout request: any pointer may be null.  `pscratch` (n doubles) and
// `partials` (enough for the launch) come from the workspace.
struct Readout {
  double *p = nullptr;
  double *norm = nullptr;
  double *pmarked = nullptr;
  double *pscratch = nullptr;
  double *partials = nullptr;
  bool any() const { return p || norm || pmarked; }
  double *p_out() const { return p ? p : pscratch; }
};

// Coefficients of one Horner stage y_out = psi + i*(alpha*sum_nbr y + beta*[marked] y_v),
// alpha = gamma*dt/k, beta = dt/k (FP64; rounded once for complex64).
struct StageCoef {
  double alpha;
  double beta;
};

// ---- launchers (qw_kernels.hip) -------------------------------------------
// All return the hipError_t of the launch (hipGetLastError after it).
hipError_t coined_small(bool c128, const GraphView &g, void *psi, int hadamard, int64_t steps,
                        const Readout &ro, hipStream_t s);
size_t coined_small_lds(bool c128, int n, int n_arcs);

// One step in CSR arc order.  gather: `in` holds the previous step's coin output,
// still to be shifted; scatter: shift on the way out (else `out` needs the next
// step's gather, or coined_shift).  complex128 steps scatter.
hipError_t coined_tile_step(bool c128, const GraphView &g, const void *in, void *out, int hadamard, bool gather,
                            bool scatter, hipStream_t s);
hipError_t coined_shift(const GraphView &g, const void *phi, void *out, hipStream_t s);
hipError_t coined_struct_step(bool c128, const GraphView &g, const void *in, void *out,
                              int hadamard, hipStream_t s);
// Grid walks: how many of `left` steps the next launch takes (1: one step by
// coined_struct_step), and a launch of S >= 2 steps.
int coined_sweep_steps(bool c128, const GraphView &g, int64_t left);
hipError_t coined_sweep(bool c128, const GraphView &g, int S, const void *in, void *out, hipStream_t s);
hipError_t coined_perm_in(bool c128, const GraphView &g, const void *psi, void *internal,
                          hipStream_t s);
hipError_t coined_perm_out(bool c128, const GraphView &g, const void *internal, void *psi,
                           const Readout &ro, hipStream_t s);
hipError_t copy_state(bool c128, int64_t len, const void *in, void *out, hipStream_t s);
hipError_t coined_prob_csr(bool c128, const GraphView &g, const void *psi, const Readout &ro,
                           hipStream_t s);

hipError_t small_many(bool c128, const SmallWalk *d_walks, int count, size_t lds, int threads, hipStream_t s);
hipError_t ctqw_small(bool c128, const GraphView &g, void *psi, const double *alpha,
                      const double *beta, int K, int64_t steps, const Readout &ro, hipStream_t s);
size_t ctqw_small_lds(bool c128, int n, int n_arcs);
hipError_t ctqw_stage(bool c128, const GraphView &g, const void *y, const void *psi, void *out,
                      StageCoef c, const Readout *fused, hipStream_t s);
hipError_t vertex_prob(bool c128, const GraphView &g, const void *psi, const Readout &ro,
                       hipStream_t s);

// Dense H: expand the CSR into H (zero fill then scatter of -gamma and the
// marked diagonal), and one Horner stage y_out = psi + (-i c) H y_in on MFMA.
hipError_t dense_fill(bool c128, const GraphView &g, double gamma, size_t rows_pad, hipStream_t s);
// Number of k ranges the dense stage splits into (1 = no split; partials then unused).
int dense_splits(bool c128, const GraphView &g);
hipError_t dense_stage(bool c128, const GraphView &g, const void *y, const void *psi, void *out, double c,
                       hipStream_t s);

// Grid CTQW with temporal blocking: depth S (stages per launch, dividing K;
// 1 = not applicable), and S stages k = kfirst..kfirst-S+1 of one time step
// from (P, Yin) to Out (Yin may equal P at the first stage of a step).
// alpha/beta hold 64 entries (stage k at [k-1]).
int torus_block_depth(bool c128, const GraphView &g, int K);
// The two-column complex64 sweep for order K: its strips (count 0: the grid is
// not for it) and the stages of its deepest launch; and a launch of S stages,
// kfirst down, on the strips of g, `core` columns each.
StripGrid deep_strips(int l1, int l2, int K, int block_depth, int *depth);
hipError_t torus_deep(const GraphView &g, int core, int S, const void *P, const void *Yin, void *Out, int kfirst,
                      const double *alpha, const double *beta, hipStream_t s);
StripGrid torus_strips(bool c128, int l1, int l2, int S);
hipError_t torus_block_stages(bool c128, const GraphView &g, int S, const void *P, const void *Yin, void *Out,
                              int kfirst, const double *alpha, const double *beta, hipStream_t s);

// Staggered walk.  stag_small: every step in one workgroup's LDS (descriptors
// read from g.stag).  stag_tess: one tessellation in place on psi; `mark`
// applies the marked phase flip to what it reads (first tessellation of a
// step); `partials` holds t.n_chunks complex partial sums (workspace).
size_t stag_small_lds(bool c128, int n);
hipError_t stag_small(bool c128, const GraphView &g, void *psi, int64_t steps, const Readout &ro, hipStream_t s);
hipError_t stag_tess(bool c128, const GraphView &g, const StagTess &t, void *psi, bool mark, double *partials,
                     hipStream_t s);
// Staggered walk on the square lattice (structure kStagLattice, dims {l1, l2}):
// `steps` steps (at most what stag_lattice_steps gives), both tessellations
// each, in one launch, from `in` to `out` (distinct buffers); `ta`, `tb` give
// the tessellations' (c0, c1).
int stag_lattice_steps(bool c128, int64_t left);
hipError_t stag_lattice_step(bool c128, const GraphView &g, const StagTess &ta, const StagTess &tb, int steps,
                             const void *in, void *out, hipStream_t s);

// Sum of `count` partials -> *norm; sum over the marked list of p -> *pmarked.
hipError_t finish_readout(const GraphView &g, int count, const Readout &ro, hipStream_t s);

// ---- batched execution ------------------------------------------------------
// Launch counter shared by all workgroups of a batched launch: every
// workgroup reads L at its start; the last one to finish advances it.
struct BatchCtl {
  unsigned long long L;      // launches completed
  unsigned int done;         // workgroups finished in the current launch
  unsigned int probe;        // 1: timing probe (every walk runs its first stage, L frozen)
};

// One walk of a batch (device copy).  kind < 0 marks an empty slot.
struct WalkSlot {
  int32_t kind;      // QW_COINED / QW_CTQW, -1 = empty
  int32_t n;
  int32_t K;         // CTQW Taylor order (>= 2); 1 for coined
  int32_t hadamard;
  int64_t L0;        // global launch index at which the walk starts
  int64_t units;     // launches it needs: steps * K (CTQW) or steps (coined)
  const int32_t *rp;
  const int32_t *col;     // CTQW (CSR order, or column-major when ell_d > 0)
  int32_t ell_d;          // CTQW: regular degree of the ELL layout, 0 = CSR
  int32_t pad0;
  const int32_t *rev;     // coined
  const uint32_t *markbits;
  void *psi;
  void *w0;
  void *w1;
  const double *alpha;    // K entries, stage k at [k-1]
  const double *beta;
  double *hist;           // CTQW: p_marked after each step (caller-zeroed), may be null
  int32_t structure;      // coined: kGeneral (CSR tiles, state in psi/w0) or kCycle/kTorus/
                          // kHypercube (slot-major state in w0/w1, see k_batch_struct)
  int32_t sdims[2];       // structured coined: {n, 0} / {l1, l2} / {dim, 0}
  int32_t pad1;
};

// A unit of work of a batched launch: rows (CTQW) or vertices (coined) [begin, end) of a slot.
struct TileEntry {
  int32_t slot;      // -1 = padding
  int32_t begin;
  int32_t end;
  int32_t pad;
};

// The gather-path stage of a batched launch (CSR and ELL CTQW tiles, general
// coined tiles); the last workgroup advances the launch counter when
// `advance` is nonzero.
hipError_t batch_stage(bool c128, BatchCtl *ctl, const WalkSlot *slots, const TileEntry *tiles,
                       const int32_t *n_tiles, int grid, int advance, hipStream_t s);
// Out-of-core CTQW stage on rows [r0, r1) whose neighbour indices (CSR arcs
// [arc0, ...)) sit in a device slot: slot[a - arc0] = col[a].
hipError_t ctqw_slot_stage(bool c128, const GraphView &g, const int32_t *slot, int64_t arc0, int r0, int r1,
                           const void *y, const void *psi, void *out, double alpha, double beta, hipStream_t s);
// Copy `bytes` bytes of device memory src to dst, the device view of pinned
// host memory, by a kernel on stream s (both 16-byte aligned).
hipError_t copy_link(void *dst, const void *src, size_t bytes, hipStream_t s);
// Direct out-of-core CTQW stage: workgroup tile w holds rows [wg_row[w],
// wg_row[w+1]) (at most kDirRows rows and kDirArcs arcs, or one longer row);
// neighbour indices of arcs below `split` (a multiple of 4) come from the
// device prefix dcol, the others straight from pinned host memory hcol (both
// 16-byte aligned, hcol padded to a multiple of 4 entries).
hipError_t ctqw_direct_stage(bool c128, const GraphView &g, const int32_t *wg_row, int64_t n_wg, const int32_t *dcol,
                             const int32_t *hcol, int64_t split, const void *y, const void *psi, void *out,
                             double alpha, double beta, hipStream_t s);
// The LDS-staged stage of the batch's CTQW walks on the ELL layout (degree
// <= 8): tiles of lds_tile_rows rows, one workgroup of kLdsTileThreads64/128
// each, the input vector staged in blocks of kLdsBlockBytes64/128.  The last workgroup
// advances the launch counter when `advance` is nonzero.
hipError_t batch_ell_lds(bool c128, BatchCtl *ctl, const WalkSlot *slots, const TileEntry *tiles,
                         const int32_t *n_tiles, int grid, int advance, hipStream_t s);
// The structured coined tiles of a batched launch (run before batch_stage in
// each launch unit; reads the launch counter, does not advance it).
hipError_t batch_struct(bool c128, const BatchCtl *ctl, const WalkSlot *slots, const TileEntry *tiles,
                        const int32_t *n_tiles, int grid, hipStream_t s);

// Number of partial sums the readout kernels (one thread per vertex) write.
int readout_partials(const GraphView &g);
// Number of partial sums a CTQW stage with the readout fused writes.
int ctqw_stage_partials(const GraphView &g);

}  // namespace qwk
