// Kernels of the coefficient form (d2q37_coeff.h) and their launchers: the
// fused step, the transposed step, the way in from and out to the 37
// populations, and the readers of the state.
//
// The sweep (fused step and transposed step).  One wave64 takes 56 rows of TX
// consecutive columns: its lanes hold the rows y0 - 4 .. y0 + 59, four of
// them halo on each side, so that a population hopping up to three rows finds
// its target inside the wave, and stores start 128-byte aligned (56 rows of
// 16-byte pairs).  The wave walks over the TX + 6 source columns.  For each
// it loads the site's 15 coefficients, rebuilds the populations of every
// e_x group that reaches one of its TX columns, shifts them to their target
// row across its lanes (DPP) and adds them to the target's 15 sums; a column
// is complete six source columns after its first and is collided and stored
// at once.
//
// What bounds it and why this split.  The step moves 240 bytes per site
// (15 FP64 in, 15 out) instead of the 592 of the 37 populations, at 5.3 TB/s
// (1920 x 2048: 176 us against 405; 4096 x 4096: 735 us against 1646; a copy
// reaches 5.2 to 5.7 TB/s).  Rebuilding populations is done once per (source
// site, e_x group) whatever TX is; TX trades registers (30 VGPRs per column:
// 4, 3, 2, 2 waves per SIMD at TX = 1, 2, 3, 4) against re-reading source
// columns ((TX + 6) / TX times, nearly all from the XCD's L2: 1.05 x and
// 1.11 x of the state fetched past it at TX = 3 and 4).  16-byte accesses
// matter: with 8-byte ones the L1 handles half the bytes per cycle (230
// against 200 us).  Source columns are loaded ahead of their use (191 -> 181
// us at TX = 4).  On small lattices the instructions of a wave's walk count:
// powers of the hops instead of Hermite values as factors took 1305 to 1106
// instructions per column, and DPP instead of LDS took the waits (256 x 128:
// 5.7 -> 5.2 -> 5.1 us, 331 x 205: 7.8 -> 7.2 -> 6.7).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "d2q37_coeff.h"
#include "d2q37_launch.h"
#include "d2q37_tiles.h"

#pragma clang fp contract(off)  // as in d2q37_coeff.h

namespace d2q37 {

namespace {

typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kHalo = 4;             // halo rows on each side of a wave
constexpr int kRows = 64 - 2 * kHalo;  // target rows of a wave
constexpr int kWaves = 4;            // waves per workgroup (independent)
// States from these sizes to kCachedTo are stored into the caches (us per step,
// streamed and cached).  Steps: 331 x 331 7.1 and 8.3, 512 x 512 15.8 and 16.8,
// 560 x 560 19.4 and 18.9, 700 x 700 26.9 and 24.3, 1000 x 1000 43.4 and 39.6
// (with tape 61.0 and 47.6), 1200 x 1200 60.0 and 61.5.  Transposed steps:
// 331 x 331 11.4 and 11.1, 400 x 400 18.7 and 16.4, 512 x 512 25.3 and 22.4,
// 1000 x 1000 69.8 and 67.2, 1100 x 1100 86.4 and 89.0.
constexpr long long kCachedTo = 135LL * 1000 * 1000;
constexpr long long kStepCachedFrom = 36LL * 1000 * 1000;
constexpr long long kAdjointCachedFrom = 12LL * 1000 * 1000;
// Up to this state size the transposed step reads its tape through the caches
// as well, which hold what a run of steps just recorded (400 x 400 16.4 us
// past them and 14.7 through them, 512 x 512 22.4 and 22.1, 1000 x 1000 67.4
// and 70.3).
constexpr long long kTapeCachedTo = 32LL * 1000 * 1000;
// Lane offset of rows that do not exist: it, its half, and either of them plus
// any plane's offset lie beyond every column (NC * pitch * 8 < 2^31 bytes), so
// loads give 0 and stores do nothing.
constexpr unsigned kOutside = 0x80000000u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t column_rsrc(const double* buf, const CGeom& g,
                                                              int x) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)(buf + x * g.cs), (short)0,
                                           NC * g.pitch * 8u, kBufferWord3);
}

// coefficients of row `row_bytes / 16` of a column (zero where row_bytes is kOutside)
__device__ __forceinline__ void load_column(__amdgpu_buffer_rsrc_t r, const CGeom& g,
                                            unsigned row_bytes, double (&b)[NC]) {
#pragma unroll
  for (int m = 0; m < NC / 2; ++m) {
    const v2d d = __builtin_bit_cast(
        v2d, __builtin_amdgcn_raw_buffer_load_b128(r, row_bytes, m * g.pitch * 16u, 0));
    b[2 * m] = d.x;
    b[2 * m + 1] = d.y;
  }
  b[NC - 1] = __builtin_bit_cast(
      double, __builtin_amdgcn_raw_buffer_load_b64(r, row_bytes >> 1, (NC - 1) * g.pitch * 8u, 0));
}

// Row `row_bytes` of a column (kOutside: not stored), streamed past the caches
// where they do not hold the lattice until the next step.  The plane is added
// to the lane's offset, not given as the scalar offset of the instruction:
// with a scalar offset the compiler lets the next vector instruction overwrite
// the data of a 16-byte store, which here changed the low word of a few stored
// values in a million.
template <int kPolicy>
__device__ __forceinline__ void store_planes(__amdgpu_buffer_rsrc_t r, const CGeom& g,
                                             unsigned row_bytes, const double (&b)[NC]) {
#pragma unroll
  for (int m = 0; m < NC / 2; ++m)
    __builtin_amdgcn_raw_buffer_store_b128(
        __builtin_bit_cast(v4u, (v2d{b[2 * m], b[2 * m + 1]})), r, row_bytes + m * g.pitch * 16u,
        0, kPolicy);
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, b[NC - 1]), r,
                                        (row_bytes >> 1) + (NC - 1) * g.pitch * 8u, 0, kPolicy);
}
__device__ __forceinline__ void store_column(__amdgpu_buffer_rsrc_t r, const CGeom& g,
                                             unsigned row_bytes, const double (&b)[NC]) {
  if (g.stream)
    store_planes<kNonTemporal>(r, g, row_bytes, b);
  else
    store_planes<0>(r, g, row_bytes, b);
}

// Lane i gets the value of lane i - n (up) or i + n (down); zero beyond the
// wave.  A shift of the whole wave by one lane is a DPP move, two for 64 bits.
constexpr int kUp = 0x138, kDown = 0x130;  // wave_shr:1, wave_shl:1
template <int ctrl, int n>
__device__ __forceinline__ double shift_lanes(double v) {
  if constexpr (n == 0) {
    return v;
  } else {
    const v2u u = __builtin_bit_cast(v2u, v);
    const v2u w = {unsigned(__builtin_amdgcn_update_dpp(0, int(u.x), ctrl, 0xf, 0xf, true)),
                   unsigned(__builtin_amdgcn_update_dpp(0, int(u.y), ctrl, 0xf, 0xf, true))};
    return shift_lanes<ctrl, n - 1>(__builtin_bit_cast(double, w));
  }
}

// (ex, +k) arrives from the row k below its target; the transposed hop from
// the row above.  104 moves per site for the 30 populations that change rows;
// passing them through LDS (60 accesses) makes every group wait for its round
// trip: 331 x 205 step 7.2 us against 6.7, 777 x 1501 63.5 against 63.2.
template <class K>
constexpr bool kForward = true;
template <>
constexpr bool kForward<Adjoint> = false;
template <class K, int ex, int k = 1>
__device__ __forceinline__ void shift_group(Group& f) {
  f.plus[k - 1] = shift_lanes<kForward<K> ? kUp : kDown, k>(f.plus[k - 1]);
  f.minus[k - 1] = shift_lanes<kForward<K> ? kDown : kUp, k>(f.minus[k - 1]);
  if constexpr (k < reach(ex)) shift_group<K, ex, k + 1>(f);
}

// Row of this lane: its index, whether it exists, its byte offset in a pair
// plane for loads, and for stores (only the wave's own rows).
struct Row {
  int y, from;  // from: the row that is read (inside the lattice)
  bool in;
  unsigned load, store;
};
__device__ __forceinline__ Row wave_row(const CGeom& g, int w, int rows = kRows,
                                        int halo = kHalo) {
  const int lane = threadIdx.x & 63;
  Row r;
  r.y = w * rows - halo + lane;
  r.in = r.y >= 0 && r.y < g.ly;
  int y = r.y;
  if (g.periodic) {  // rows beyond the three that are read may fold anywhere
    if (y < 0) y += g.ly;
    if (y >= g.ly) y -= g.ly;
    if (y < 0 || y >= g.ly) y = 0;
  }
  r.from = r.in || g.periodic ? y : 0;
  r.load = r.in || g.periodic ? unsigned(y) * 16u : kOutside;
  r.store = r.in && lane >= halo && lane < halo + rows ? unsigned(r.y) * 16u : kOutside;
  return r;
}

// Wave of this workgroup: rows w, first column x0; false beyond the lattice.
// Consecutive waves go up a strip of TX columns, then to the next strip; the
// strips are taken in the order in which a wave walks over its columns.  A
// column that two strips share is then read by the later one sooner than its
// walk alone would have it, and more often still in the XCD's L2: with the
// adjoint's descending walk over ascending strips its step fetched 1.23 GB
// instead of 0.6 at 1920 x 2048 (241 us against 212).
template <class K, int TX>
__device__ __forceinline__ bool wave_tile(const CGeom& g, unsigned nb, int& w, int& x0) {
  const unsigned wave = unsigned(__builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)));
  const unsigned t = tile_index(nb) * kWaves + wave;
  const int strips = (g.lx + TX - 1) / TX;
  w = int(t % unsigned(g.nw));
  const int s = int(t / unsigned(g.nw));
  x0 = (kForward<K> ? s : strips - 1 - s) * TX;
  return s < strips;
}

// The sweep of one wave.  Target t of the TX columns (in the order of the
// walk) takes the e_x group t + 3 - j of source column j, so every target
// receives its groups in the order 3, 2, .., -3.  Site: what is done with a
// finished target (walls, local operator, store).
template <class K, int TX, int kAhead, class Site>
struct Sweep {
  const double* src;
  const CGeom& g;
  const Site& site;
  int x0;
  Row row;
  double c[kAhead][NC];  // source columns in flight
  double m[TX][NC];      // sums of the targets

  __device__ __forceinline__ int source(int j) const {
    int x = kForward<K> ? x0 - 3 + j : x0 + TX + 2 - j;
    x = x < 0 ? x + g.lx : (x >= g.lx ? x - g.lx : x);
    return x;  // (lx >= 6: one wrap reaches every column of a ragged last tile too)
  }
  __device__ __forceinline__ int target(int t) const {
    return kForward<K> ? x0 + t : x0 + TX - 1 - t;
  }
  __device__ __forceinline__ void load(int j, double (&v)[NC]) {
    load_column(column_rsrc(src, g, source(j)), g, row.load, v);
  }
  template <int j, int t>
  __device__ __forceinline__ void add() {
    if constexpr (t < TX) {
      constexpr int ex = t + 3 - j;
      if constexpr (ex >= -3 && ex <= 3) {
        Group f;
        expand_group<K, ex>(c[j % kAhead], f);
        shift_group<K, ex>(f);
        project_group<K, ex>(f, m[t]);
        // keeps the sums here: left to itself the compiler defers them to
        // the end and holds every group of the target in registers (127
        // instead of 87 VGPRs at TX = 1, spills from TX = 3)
#pragma unroll
        for (int k = 0; k < NC; ++k) asm volatile("" : "+v"(m[t][k]));
      }
      add<j, t + 1>();
    }
  }
  template <int j>
  __device__ __forceinline__ void walk() {
    if constexpr (j < TX + 6) {
      typename Site::Input in;
      if constexpr (j >= 6) site.load(in, target(j - 6), row);
      add<j, 0>();
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (j + kAhead < TX + 6) load(j + kAhead, c[j % kAhead]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (j >= 6) site.finish(in, m[j - 6], target(j - 6), row);
      walk<j + 1>();
    }
  }
  template <int j = 0>
  __device__ __forceinline__ void prefetch() {
    if constexpr (j < kAhead) {
      load(j, c[j]);
      prefetch<j + 1>();
    }
  }
};

__device__ __forceinline__ void store_tape(double* tape, long long S2, long long s,
                                           const double (&a)[NC]) {
  __builtin_nontemporal_store(a[slot(0, 0)], &tape[s]);
  __builtin_nontemporal_store(R * a[slot(1, 0)], &tape[S2 + s]);
  __builtin_nontemporal_store(R * a[slot(0, 1)], &tape[2 * S2 + s]);
  __builtin_nontemporal_store(R2 * (a[slot(2, 0)] + a[slot(0, 2)]), &tape[3 * S2 + s]);
}

// The way in from 37 stored populations: the moments of those that arrive at a
// site (0 for the ones a wall will supply).  The columns wrap here, so halo
// columns are not read.
__device__ __forceinline__ double arriving(const double* __restrict__ src, const Geom& gf,
                                           const CGeom& g, int x, int y, int l) {
  int xs = x - EX[l], ys = y - EY[l];
  xs = xs < 0 ? xs + g.lx : (xs >= g.lx ? xs - g.lx : xs);
  const bool outside = ys < 0 || ys >= g.ly;
  if (g.periodic)
    ys = ys < 0 ? ys + g.ly : (ys >= g.ly ? ys - g.ly : ys);
  else if (outside)
    ys = y;
  const double v = src[l * gf.ps + (long long)(xs + HX) * gf.cs + ys + gf.hy];
  return !g.periodic && outside ? 0.0 : v;
}
template <int ex = 3>
__device__ __forceinline__ void project_arriving(const double* src, const Geom& gf,
                                                 const CGeom& g, int x, int y, double (&m)[NC]) {
  // one group after the other, and no strides kept from one column to the
  // next: the sweep has no registers for more
  Geom h = gf;
  asm volatile("" : "+s"(src), "+s"(h.ps), "+s"(h.cs));
  Group f;
  f.zero = arriving(src, h, g, x, y, label(ex, 0));
#pragma unroll
  for (int k = 1; k <= reach(ex); ++k) {
    f.plus[k - 1] = arriving(src, h, g, x, y, label(ex, k));
    f.minus[k - 1] = arriving(src, h, g, x, y, label(ex, -k));
  }
  project_group<Forward, ex>(f, m);
#pragma unroll
  for (int k = 0; k < NC; ++k) asm volatile("" : "+v"(m[k]));
  if constexpr (ex > -3) project_arriving<ex - 1>(src, gf, g, x, y, m);
}

// Forward: walls on the six wall rows, optional tape of the pre-collision
// moments (rho, j_x, j_y, sum |c|^2 f), collide, store.
template <bool kTape>
struct StepSite {
  double* dst;
  const CGeom& g;
  const CPhys& P;
  const WallTable& wt;
  double* tape;
  struct Input {};
  __device__ __forceinline__ void load(Input&, int, const Row&) const {}
  __device__ __forceinline__ void finish(const Input&, double (&a)[NC], int x,
                                         const Row& r) const {
    if (x >= g.lx) return;  // ragged last tile
    int i;
    if (r.in && wall_row(g, r.y, i)) wall_moments(a, wt, i);
    if (kTape) {
      if (r.store != kOutside) {
        const long long S2 = (long long)g.lx * g.ly, s = (long long)x * g.ly + r.y;
        store_tape(tape, S2, s, a);
      }
    }
    collide_moments(a, P);
    store_column(column_rsrc(dst, g, x), g, r.store, a);
  }
};

// Adjoint: the step's moments from the tape, C^T and B^T, store.
template <int kTapePolicy>
struct AdjointSite {
  double* dst;
  const CGeom& g;
  const CPhys& P;
  const WallTable& wt;
  const double* tape;
  struct Input {
    double m[4];
  };
  // Issued before the column's exchange and sums, without a branch: in a
  // masked load the compiler puts the first use, and so the wait, right there.
  __device__ __forceinline__ void load(Input& in, int x, const Row& r) const {
    if (x >= g.lx) return;  // ragged last tile (the whole wave)
    const long long S2 = (long long)g.lx * g.ly;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      in.m[k] = __builtin_bit_cast(
          double, __builtin_amdgcn_raw_buffer_load_b64(
                      __builtin_amdgcn_make_buffer_rsrc(
                          (void*)(tape + k * S2 + (long long)x * g.ly), (short)0, g.ly * 8,
                          kBufferWord3),
                      r.load >> 1, 0, kTapePolicy));
  }
  __device__ __forceinline__ void finish(const Input& in, double (&a)[NC], int x,
                                         const Row& r) const {
    if (x >= g.lx) return;
    adjoint_moments(a, in.m[0], in.m[1], in.m[2], in.m[3], P);
    int i;
    if (r.in && wall_row(g, r.y, i)) wall_adjoint(a, wt, i);
    store_column(column_rsrc(dst, g, x), g, r.store, a);
  }
};

// waves per SIMD that a sweep's registers leave room for
template <int TX, int kAhead>
constexpr int kOccupancy = TX == 1 ? 4 : (TX == 2 || (TX == 3 && kAhead == 1)) ? 3 : 2;

// word: of a source whose form is not known (null: coefficients).  Populations
// are taken through the same tiles; k_coeff_first, which is made for them, is
// launched where they are expected.
template <int TX, int kAhead, bool kTape, bool kEither>
__global__ __launch_bounds__(64 * kWaves, (kOccupancy<TX, kAhead>)) void k_coeff_step(
    const double* __restrict__ src, double* __restrict__ dst, Geom gf, CGeom g, CPhys P,
    WallTable wt, double* __restrict__ tape, unsigned nb, const unsigned* word) {
  set_form(dst, kFormCoeff);
  int w, x0;
  if (!wave_tile<Forward, TX>(g, nb, w, x0)) return;
  const StepSite<kTape> site{coeffs(dst), g, P, wt, tape};
  const Row row = wave_row(g, w);
  if (kEither && holds_populations(word)) {
#pragma unroll 1
    for (int x = x0; x < x0 + TX && x < g.lx; ++x) {
      double m[NC];
      project_arriving(src, gf, g, x, row.from, m);
      site.finish({}, m, x, row);
    }
    return;
  }
  Sweep<Forward, TX, kAhead, StepSite<kTape>> s{coeffs(src), g, site, x0, row};
  s.prefetch();
  s.template walk<0>();
}

// ---------------------------------------------------------------------------
// Two steps in one launch.  A workgroup takes 52 rows (64 lanes, six halo rows
// on each side) of `chunk` columns and marches along x, four columns at a
// time.  Two producer waves make the first step's coefficients of four
// columns and put them into a ring of ten columns in LDS; two consumer waves
// make the second step of the four columns three behind from that ring and
// store it.  While the consumers read iteration i - 1's columns the producers
// work on iteration i's in registers; a barrier, the ring's four oldest
// columns are replaced, a barrier.  The producers load four source columns
// ahead, across iterations.
//
// What bounds it.  The state is read and written once for two steps (272 of
// the 480 bytes per site, with the re-read halo rows), so the vector unit
// takes over from HBM: 550 instructions per column and wave, on 64 of 52 rows
// and (chunk + 6) of chunk columns, 55 % of the issue slots; the rest is
// waiting at the two barriers.  Two workgroups share a CU (77 KB of LDS
// each), eight waves in all.  Per step, against k_coeff_step: 1920 x 2048 140 us
// (176), 4096 x 4096 577 us (735), 777 x 1501 48 us (63).  Tried: every wave
// making first its column of step one, then of step two (216 us: the two
// phases load the L1 and the LDS in turn instead of together), one workgroup
// of eight waves (161), rows exchanged through LDS (161), source columns
// loaded two ahead (162), three and four waves per SIMD with one column each
// (157, 175).
// ---------------------------------------------------------------------------
constexpr int kPairRows = 52, kPairHalo = 6;
constexpr int kPairWave = 2;                  // columns of a wave
constexpr int kPairMakers = 2;                // producer waves, and consumer waves
constexpr int kPairCols = kPairWave * kPairMakers;  // columns of an iteration
constexpr int kRing = kPairCols + 6, kRingCol = NC * 64;
constexpr int kPairAhead = 4;  // divides kPairWave + 6: the loads run on across iterations

// One wave's walk over TX + 6 source columns; load(j, v) fetches source column
// j, beyond the walk's end the next walk's first ones.
template <int TX, int kAhead>
struct PairWalk {
  const CGeom& g;
  const CPhys& P;
  const WallTable& wt;
  const Row& row;
  double m[TX][NC];

  template <int j, int t>
  __device__ __forceinline__ void add(const double (&c)[NC]) {
    if constexpr (t < TX) {
      constexpr int ex = t + 3 - j;
      if constexpr (ex >= -3 && ex <= 3) {
        Group f;
        expand_group<Forward, ex>(c, f);
        shift_group<Forward, ex>(f);
        project_group<Forward, ex>(f, m[t]);
#pragma unroll
        for (int k = 0; k < NC; ++k) asm volatile("" : "+v"(m[t][k]));  // as in Sweep
      }
      add<j, t + 1>(c);
    }
  }
  __device__ __forceinline__ void finish(double (&a)[NC]) const {
    int i;
    if (row.in && wall_row(g, row.y, i)) wall_moments(a, wt, i);
    collide_moments(a, P);
  }
  template <int j = 0, class Load>
  __device__ __forceinline__ void walk(double (&c)[kAhead][NC], const Load& load) {
    if constexpr (j < TX + 6) {
      add<j, 0>(c[j % kAhead]);
      __builtin_amdgcn_sched_barrier(0);
      load(j + kAhead, c[j % kAhead]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (j >= 6) finish(m[j - 6]);
      walk<j + 1>(c, load);
    }
  }
  // the TX columns from x on, from stored populations
  __device__ __forceinline__ void from_populations(const double* src, const Geom& gf, int x) {
#pragma unroll
    for (int t = 0; t < TX; ++t) {
      project_arriving(src, gf, g, x + t >= g.lx ? x + t - g.lx : x + t, row.from, m[t]);
      finish(m[t]);
    }
  }
};

__device__ __forceinline__ int ring_slot(int s) { return s >= kRing ? s - kRing : s; }

__device__ __forceinline__ void ring_store(double* col, int lane, const double* m) {
#pragma unroll
  for (int k = 0; k < NC / 2; ++k)
    *reinterpret_cast<v2d*>(col + k * 128 + 2 * lane) = v2d{m[2 * k], m[2 * k + 1]};
  col[(NC - 1) * 64 + lane] = m[NC - 1];
}
__device__ __forceinline__ void ring_load(const double* col, int lane, double (&v)[NC]) {
#pragma unroll
  for (int k = 0; k < NC / 2; ++k) {
    const v2d d = *reinterpret_cast<const v2d*>(col + k * 128 + 2 * lane);
    v[2 * k] = d.x;
    v[2 * k + 1] = d.y;
  }
  v[NC - 1] = col[(NC - 1) * 64 + lane];
}

// kEither: the source may hold populations (word, as k_coeff_step).
template <bool kEither>
__global__ __launch_bounds__(64 * 2 * kPairMakers, 2) void k_coeff_pair(
    const double* __restrict__ src, double* __restrict__ dst, Geom gf, CGeom g, CPhys P,
    WallTable wt, int windows, int chunk, unsigned nb, const unsigned* word) {
  __shared__ __align__(16) double ring[kRing * kRingCol];
  set_form(dst, kFormCoeff);
  const unsigned t = tile_index(nb);
  const int xa = int(t / unsigned(windows)) * chunk, xb = min(xa + chunk, g.lx);
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const Row row = wave_row(g, int(t % unsigned(windows)), kPairRows, kPairHalo);
  // iteration i: step one of columns xa - 3 + 4 i .., step two of the targets
  // whose sources iteration i - 1 completed; both barriers every time
  const int iters = (xb - xa + 6 + kPairCols - 1) / kPairCols;
  if (wave < kPairMakers) {
    int slot = wave * kPairWave;
    int x = xa - 3 + wave * kPairWave;
    if (x < 0) x += g.lx;
    auto load = [&](int j, double (&v)[NC]) {
      int xs = x - 3 + (j < kPairWave + 6 ? j : j - (kPairWave + 6) + kPairCols);
      xs = xs < 0 ? xs + g.lx : (xs >= g.lx ? xs - g.lx : xs);
      load_column(column_rsrc(coeffs(src), g, xs), g, row.load, v);
    };
    const auto march = [&](const auto& make) {
      for (int i = 0; i <= iters; ++i) {
        PairWalk<kPairWave, kPairAhead> s{g, P, wt, row};
        if (i < iters) {
          make(s);
          if (!g.periodic && !row.in) {  // nothing comes from beyond the walls
#pragma unroll
            for (int k = 0; k < kPairWave * NC; ++k) s.m[k / NC][k % NC] = 0.0;
          }
        }
        __syncthreads();
        if (i < iters) {
#pragma unroll
          for (int n = 0; n < kPairWave; ++n) {
            double* col = ring + ring_slot(slot + n) * kRingCol;
            ring_store(col, lane, s.m[n]);
          }
        }
        __syncthreads();
        slot = ring_slot(slot + kPairCols);
        x += kPairCols;
        if (x >= g.lx) x -= g.lx;
      }
    };
    if (kEither && holds_populations(word)) {
      march([&](auto& s) { s.from_populations(src, gf, x); });
    } else {
      double c[kPairAhead][NC];
#pragma unroll
      for (int j = 0; j < kPairAhead; ++j) load(j, c[j]);
      march([&](auto& s) { s.walk(c, load); });
    }
  } else {
    const int first = (wave - kPairMakers) * kPairWave;
    int base = ring_slot(first + kPairCols);  // the slot of column x - 3
    for (int i = 0; i <= iters; ++i) {
      const int x = xa - 6 + (i - 1) * kPairCols + first;
      if (i > 0) {
        if (x + kPairWave > xa && x < xb) {
          auto load = [&](int j, double (&v)[NC]) {
            if (j >= kPairWave + 6) return;
            const double* col = ring + ring_slot(base + j) * kRingCol;
            ring_load(col, lane, v);
          };
          double c[1][NC];
          load(0, c[0]);
          PairWalk<kPairWave, 1> s{g, P, wt, row};
          s.walk(c, load);
#pragma unroll
          for (int n = 0; n < kPairWave; ++n)
            if (x + n >= xa && x + n < xb)
              store_column(column_rsrc(coeffs(dst), g, x + n), g, row.store, s.m[n]);
        }
        base = ring_slot(base + kPairCols);
      }
      __syncthreads();
      __syncthreads();
    }
  }
}

// Two steps in one launch for lattices that leave most of the GPU idle, where
// a launch costs as much as its work: one column of a window of rows by seven
// waves.  Each makes one column of the first step, from three before to three
// after, into LDS; the first of them then makes the second step.  The column's
// chain of instructions (about 600, 1 us) runs three times as often as in two
// launches of k_coeff_step, on SIMDs that have nothing else to do: per step
// 16 x 16 4.7 us and 3.7, 64 x 48 4.8 and 3.8, 128 x 48 4.6 and 4.1, but
// 100 x 100 (200 columns of windows) 4.7 and 4.5, 128 x 128 4.8 and 6.3.  Two
// columns by eight waves 4.1 at 64 x 48; three steps in a loop over stages 4.7.
constexpr int kSmallWaves = 7;
template <bool kEither>
__global__ __launch_bounds__(64 * kSmallWaves) void k_coeff_two(
    const double* __restrict__ src, double* __restrict__ dst, Geom gf, CGeom g, CPhys P,
    WallTable wt, int windows, int rows, int halo, const unsigned* word) {
  __shared__ __align__(16) double ring[kSmallWaves * kRingCol];
  set_form(dst, kFormCoeff);
  const int x = int(blockIdx.x / unsigned(windows));
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const Row row = wave_row(g, int(blockIdx.x % unsigned(windows)), rows, halo);
  {
    auto load = [&](int j, double (&v)[NC]) {
      if (j >= 7) return;
      int xs = x - 6 + wave + j;
      xs = xs < 0 ? xs + g.lx : (xs >= g.lx ? xs - g.lx : xs);
      load_column(column_rsrc(coeffs(src), g, xs), g, row.load, v);
    };
    double c[2][NC];
    load(0, c[0]);
    load(1, c[1]);
    PairWalk<1, 2> s{g, P, wt, row};
    if (kEither && holds_populations(word)) {
      const int xw = x - 3 + wave;
      s.from_populations(src, gf, xw < 0 ? xw + g.lx : (xw >= g.lx ? xw - g.lx : xw));
    } else {
      s.walk(c, load);
    }
    if (!g.periodic && !row.in) {  // nothing comes from beyond the walls
#pragma unroll
      for (int k = 0; k < NC; ++k) s.m[0][k] = 0.0;
    }
    ring_store(ring + wave * kRingCol, lane, s.m[0]);
  }
  __syncthreads();
  if (wave == 0) {
    auto load = [&](int j, double (&v)[NC]) {
      if (j < 7) ring_load(ring + j * kRingCol, lane, v);
    };
    double c[1][NC];
    load(0, c[0]);
    PairWalk<1, 1> s{g, P, wt, row};
    s.walk(c, load);
    store_column(column_rsrc(coeffs(dst), g, x), g, row.store, s.m[0]);
  }
}

template <int TX, int kAhead, int kTapePolicy>
__global__ __launch_bounds__(64 * kWaves, (kOccupancy<TX, kAhead>)) void k_coeff_adjoint(
    const double* __restrict__ tape, const double* __restrict__ src, double* __restrict__ dst,
    CGeom g, CPhys P, WallTable wt, unsigned nb) {
  int w, x0;
  if (!wave_tile<Adjoint, TX>(g, nb, w, x0)) return;
  const AdjointSite<kTapePolicy> site{dst, g, P, wt, tape};
  Sweep<Adjoint, TX, kAhead, AdjointSite<kTapePolicy>> s{src, g, site, x0, wave_row(g, w)};
  s.prefetch();
  s.template walk<0>();
}

// ---------------------------------------------------------------------------
// Site kernels: one thread per site.
// ---------------------------------------------------------------------------

__device__ __forceinline__ void store_coeffs(double* __restrict__ dst, const CGeom& g, int x,
                                             int y, const double (&b)[NC]) {
  double* col = dst + x * g.cs;
#pragma unroll
  for (int m = 0; m < NC / 2; ++m)
    __builtin_nontemporal_store(
        (v2d{b[2 * m], b[2 * m + 1]}),
        reinterpret_cast<v2d*>(col + 2 * m * (long long)g.pitch + 2 * y));
  __builtin_nontemporal_store(b[NC - 1], &col[(NC - 1) * (long long)g.pitch + y]);
}

// adjoint arrays are compact, in the lattice's layout
struct LamAt {
  long long ps, cs;
};
__device__ __forceinline__ LamAt lam_at(const Geom& g) {
  const long long s2 = (long long)g.lx * g.ly;
  return g.ps < g.cs ? LamAt{g.ly, (long long)Q * g.ly} : LamAt{s2, g.ly};
}

// The step from the 37 stored populations of a padded buffer: gather, walls,
// collide, coefficients out (296 bytes in, 120 out per site; runs once after
// the state was replaced).  It is launched on the host's guess: if the word
// names coefficients, it gathers from those.
template <bool kTape>
__global__ __launch_bounds__(kThreads) void k_coeff_first(
    const double* __restrict__ src, double* __restrict__ dst, Geom gf, CGeom g, CPhys P, WallTable wt,
    double* __restrict__ tape, int by, int bx, int nty, unsigned nb, const unsigned* word) {
  set_form(dst, kFormCoeff);
  int x, y;
  if (!site_of(g.lx, g.ly, by, bx, nty, nb, x, y)) return;
  double v[Q];
  if (holds_coeffs(word)) {
    gather_coeffs(coeffs(src), g, x, y, [&](int l, double f) { v[l] = f; });
  } else {
#pragma unroll
    for (int l = 0; l < Q; ++l) v[l] = arriving(src, gf, g, x, y, l);
  }
  double a[NC];
  project_site<Forward>(v, a);
  int i;
  if (wall_row(g, y, i)) wall_moments(a, wt, i);
  if (kTape) {
    const long long S2 = (long long)g.lx * g.ly, s = (long long)x * g.ly + y;
    store_tape(tape, S2, s, a);
  }
  collide_moments(a, P);
  store_coeffs(coeffs(dst), g, x, y, a);
}

// f^eq(rho0, u0, T0) as coefficients.
__global__ __launch_bounds__(kThreads) void k_coeff_init(
    double* __restrict__ dst, const double* __restrict__ rho, const double* __restrict__ ux,
    const double* __restrict__ uy, const double* __restrict__ T, CGeom g, int by, int bx, int nty,
    unsigned nb) {
  set_form(dst, kFormCoeff);
  int x, y;
  if (!site_of(g.lx, g.ly, by, bx, nty, nb, x, y)) return;
  const long long s = (long long)x * g.ly + y;
  double aeq[5][5], b[NC];
  equilibrium_coeffs(rho[s], ux[s], uy[s], T[s] - 1.0, aeq);
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const int p = kCI[k], q = kCJ[k];
    constexpr double power[5] = {1.0, R, R2, R * R2, R4};
    b[k] = power[p + q] * INVFAC[p] * INVFAC[q] * aeq[p][q];  // r^(p+q) / (p! q!) a_pq
  }
  add_tails(b);
  store_coeffs(coeffs(dst), g, x, y, b);
}

// ---------------------------------------------------------------------------
// Adjoint: way in, way out, and the single step on compact arrays.
// ---------------------------------------------------------------------------

// C_ij of one site whose arriving lambda are given
__device__ __forceinline__ void adjoint_local(const double (&lam)[Q], const double* tape,
                                              long long S2, long long s, const CGeom& g,
                                              const CPhys& P, const WallTable& wt, int y,
                                              double (&C)[NC]) {
  project_site<Adjoint>(lam, C);
  adjoint_moments(C, tape[s], tape[S2 + s], tape[2 * S2 + s], tape[3 * S2 + s], P);
  int i;
  if (wall_row(g, y, i)) wall_adjoint(C, wt, i);
}

// First kernel of a run: compact lambda in, coefficients of mu out.
__global__ __launch_bounds__(kThreads) void k_coeff_adjoint_first(
    const double* __restrict__ tape, const double* __restrict__ lam, double* __restrict__ dst,
    Geom gf, CGeom g, CPhys P, WallTable wt, int by, int bx, int nty, unsigned nb) {
  int x, y;
  if (!site_of(g.lx, g.ly, by, bx, nty, nb, x, y)) return;
  const LamAt la = lam_at(gf);
  const long long sl = x * la.cs + y;
  double v[Q], B[NC];
#pragma unroll
  for (int l = 0; l < Q; ++l) v[l] = lam[l * la.ps + sl];
  adjoint_local(v, tape, (long long)g.lx * g.ly, (long long)x * g.ly + y, g, P, wt, y, B);
  store_coeffs(dst, g, x, y, B);
}

// Last kernel of a run: lambda_l(z) = mu_l(z + e_l), rebuilt from the source
// site's coefficients and passed to its row as in the sweep.
struct ExportWalk {
  const double* src;
  double* lam;
  const CGeom& g;
  const LamAt& la;
  Row row;

  template <int ex>
  __device__ __forceinline__ void group(const double (&b)[NC], int x) const {
    Group f;
    expand_group<Adjoint, ex>(b, f);
    shift_group<Adjoint, ex>(f);
    if (row.store == kOutside || x >= g.lx) return;
    double* out = lam + x * la.cs + row.y;
    store<ex, 0>(out, f.zero);
    pair<ex, 1>(out, f);
  }
  template <int ex, int ey>
  __device__ __forceinline__ void store(double* out, double v) const {
    constexpr int l = label(ex, ey);
    __builtin_nontemporal_store(v, &out[l * la.ps]);
  }
  template <int ex, int k>
  __device__ __forceinline__ void pair(double* out, const Group& f) const {
    store<ex, k>(out, f.plus[k - 1]);
    store<ex, -k>(out, f.minus[k - 1]);
    if constexpr (k < reach(ex)) pair<ex, k + 1>(out, f);
  }
  // source column x0 - 3 + j of a strip of TX columns
  template <int TX, int j, int t>
  __device__ __forceinline__ void targets(const double (&b)[NC], int x0) const {
    if constexpr (t < TX) {
      constexpr int ex = j - 3 - t;
      if constexpr (ex >= -3 && ex <= 3) group<ex>(b, x0 + t);
      targets<TX, j, t + 1>(b, x0);
    }
  }
  template <int TX, int j>
  __device__ __forceinline__ void walk(int x0, double (&b)[NC]) const {
    if constexpr (j < TX + 6) {
      double next[NC];
      if constexpr (j + 1 < TX + 6) load(x0 - 2 + j, next);
      targets<TX, j, 0>(b, x0);
      walk<TX, j + 1>(x0, next);
    }
  }
  __device__ __forceinline__ void load(int x, double (&b)[NC]) const {
    x = x < 0 ? x + g.lx : (x >= g.lx ? x - g.lx : x);
    load_column(column_rsrc(src, g, x), g, row.load, b);
  }
};

template <int TX>
__global__ __launch_bounds__(64 * kWaves) void k_coeff_adjoint_last(
    const double* __restrict__ src, double* __restrict__ lam, CGeom g, Geom gf, unsigned nb) {
  int w, x0;
  if (!wave_tile<Forward, TX>(g, nb, w, x0)) return;
  const LamAt la = lam_at(gf);
  const ExportWalk e{src, lam, g, la, wave_row(g, w)};
  double b[NC];
  e.load(x0 - 3, b);
  e.template walk<TX, 0>(x0, b);
}

// One transposed step on compact arrays: aligned reads, every component
// written to the site it was propagated from; populations that leave through
// a wall are written as zero by their own site.
__global__ __launch_bounds__(kThreads) void k_coeff_adjoint_step(
    const double* __restrict__ tape, const double* __restrict__ lam_in,
    double* __restrict__ lam_out, Geom gf, CGeom g, CPhys P, WallTable wt, int by, int bx, int nty,
    unsigned nb) {
  int x, y;
  if (!site_of(g.lx, g.ly, by, bx, nty, nb, x, y)) return;
  const LamAt la = lam_at(gf);
  const long long sl = x * la.cs + y;
  double v[Q], B[NC];
#pragma unroll
  for (int l = 0; l < Q; ++l) v[l] = lam_in[l * la.ps + sl];
  adjoint_local(v, tape, (long long)g.lx * g.ly, (long long)x * g.ly + y, g, P, wt, y, B);
  expand_site<Adjoint>(B, v);
#pragma unroll
  for (int l = 0; l < Q; ++l) {
    int ys = y - EY[l];
    if (!g.periodic && (ys < 0 || ys >= g.ly)) continue;
    if (g.periodic) ys += ys < 0 ? g.ly : (ys >= g.ly ? -g.ly : 0);
    int xs = x - EX[l];
    xs += xs < 0 ? g.lx : (xs >= g.lx ? -g.lx : 0);
    lam_out[l * la.ps + xs * la.cs + ys] = v[l];
  }
  int i;
  if (wall_row(g, y, i)) {
#pragma unroll
    for (int l = 0; l < Q; ++l) {
      const int yd = y + EY[l];
      if (yd < 0 || yd >= g.ly) lam_out[l * la.ps + sl] = 0.0;
    }
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers.  Buffers are whole state buffers: a word that names the form,
// then (256 bytes in) the coefficients.
// ---------------------------------------------------------------------------

namespace {

long long state_bytes(const CGeom& g) { return g.lx * g.cs * (long long)sizeof(double); }
CGeom make_cgeom(const Geom& g, long long cached_from = kStepCachedFrom) {
  CGeom c = coeff_geom(g);
  c.nw = (g.ly + kRows - 1) / kRows;
  c.stream = streams_output(state_bytes(c), cached_from, kCachedTo);
  return c;
}

// workgroups of a sweep with TX columns per wave
unsigned sweep_grid(const CGeom& g, int tx) {
  const long long waves = (long long)g.nw * ((g.lx + tx - 1) / tx);
  return unsigned((waves + kWaves - 1) / kWaves);
}

// Columns per wave, by the wave-columns (56 rows of one column) of the
// lattice.  Few: the length of a wave's walk is what counts; many: the
// re-read columns.  Step times in us for 1 / 2 / 3 / 4 columns per wave:
// 256 x 128 (768): 5.1 / 6.4 / 8.0 / 9.7; 331 x 205 (1324): 7.4 / 6.7 / 8.3 /
// 9.9; 512 x 512 (5120): 22.3 / 20.3 / 15.8 / 20.7; 777 x 1501 (20979): 86 /
// 68.5 / 63.2 / 64.7; 1920 x 2048 (71040): 266 / 203 / 183 / 178.  The adjoint's
// order is the same (512 x 512: 25.2 / 24.2 / 22.6 / 25.4).
int sweep_columns(const CGeom& g) {
  const long long cols = (long long)g.nw * g.lx;
  return cols >= 40960 ? 4 : cols >= 3584 ? 3 : cols >= 1280 ? 2 : 1;
}
// Three columns: with one source column ahead (three waves per SIMD) the
// forward step is faster while all its waves run at once (512 x 512: 15.8 us
// against 19.8 with two ahead; 777 x 1501: 72.8 against 63.2).
bool shallow_sweep(const CGeom& g) { return (long long)g.nw * g.lx < 9216; }

}  // namespace

hipError_t launch_coeff_step(const void* src, void* dst, const Geom& gf, const Phys& p,
                             double* tape, hipStream_t s) {
  const CGeom g = make_cgeom(gf);
  const WallTable wt = make_walls(p);
  const CPhys cp = make_cphys(p);
  const double* from = static_cast<const double*>(src);
  double* to = static_cast<double*>(dst);
  const unsigned* word = word_if_unsure(src, gf);
  if (gf.steps == 2 && two_steps_small(gf)) {
    // between walls 64 rows need no halo rows
    const bool one = !g.periodic && g.ly <= 64;
    const int rows = one ? 64 : kPairRows, halo = one ? 0 : kPairHalo;
    const int windows = (g.ly + rows - 1) / rows;
    hipLaunchKernelGGL(word ? k_coeff_two<true> : k_coeff_two<false>, dim3(windows * g.lx),
                       dim3(64 * kSmallWaves), 0, s, from, to, gf, g, cp, wt, windows, rows, halo,
                       word);
    return hipGetLastError();
  }
  if (gf.steps == 2) {
    const int windows = (g.ly + kPairRows - 1) / kPairRows;
    const int chunk = march_chunk(g.lx, windows, 512, kPairCols);
    const unsigned nb = unsigned(windows) * unsigned((g.lx + chunk - 1) / chunk);
    hipLaunchKernelGGL(word ? k_coeff_pair<true> : k_coeff_pair<false>, dim3(nb),
                       dim3(64 * 2 * kPairMakers), 0, s, from, to, gf, g, cp, wt, windows, chunk, nb,
                       word);
    return hipGetLastError();
  }
  if (gf.form == kFormFull || gf.form == kFormUnknown) {  // probably the populations
    const Tiling t = make_tiling(g.lx, g.ly);
    hipLaunchKernelGGL(tape ? k_coeff_first<true> : k_coeff_first<false>, dim3(t.nb),
                       dim3(kThreads), 0, s, from, to, gf, g, cp, wt, tape, t.by, t.bx, t.nty, t.nb,
                       word);
    return hipGetLastError();
  }
  const int tx = sweep_columns(g);
  const unsigned nb = sweep_grid(g, tx);
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(nb), dim3(64 * kWaves), 0, s, from, to, gf, g, cp, wt, tape, nb,
                       word);
  };
  const auto by_word = [&](auto either) {
    constexpr bool e = decltype(either)::value;
    if (tx == 4)
      tape ? run(k_coeff_step<4, 2, true, e>) : run(k_coeff_step<4, 2, false, e>);
    else if (tx == 3 && shallow_sweep(g))
      tape ? run(k_coeff_step<3, 1, true, e>) : run(k_coeff_step<3, 1, false, e>);
    else if (tx == 3)
      tape ? run(k_coeff_step<3, 2, true, e>) : run(k_coeff_step<3, 2, false, e>);
    else if (tx == 2)
      tape ? run(k_coeff_step<2, 2, true, e>) : run(k_coeff_step<2, 2, false, e>);
    else
      tape ? run(k_coeff_step<1, 2, true, e>) : run(k_coeff_step<1, 2, false, e>);
  };
  word ? by_word(std::true_type{}) : by_word(std::false_type{});
  return hipGetLastError();
}

hipError_t launch_coeff_init(void* dst, const double* rho, const double* ux, const double* uy,
                             const double* T, const Geom& gf, hipStream_t s) {
  const Tiling t = make_tiling(gf.lx, gf.ly);
  hipLaunchKernelGGL(k_coeff_init, dim3(t.nb), dim3(kThreads), 0, s, static_cast<double*>(dst),
                     rho, ux, uy, T, make_cgeom(gf), t.by, t.bx, t.nty, t.nb);
  return hipGetLastError();
}

hipError_t launch_coeff_adjoint_mu(const double* tape, const double* in, bool from_compact,
                                   double* mu_out, const Geom& gf, const Phys& p, hipStream_t s) {
  const CGeom g = make_cgeom(gf, kAdjointCachedFrom);
  const WallTable wt = make_walls(p);
  const CPhys cp = make_cphys(p);
  if (from_compact) {
    const Tiling t = make_tiling(g.lx, g.ly);
    hipLaunchKernelGGL(k_coeff_adjoint_first, dim3(t.nb), dim3(kThreads), 0, s, tape, in,
                       coeffs(static_cast<void*>(mu_out)), gf, g, cp, wt, t.by, t.bx, t.nty, t.nb);
    return hipGetLastError();
  }
  const int tx = sweep_columns(g);
  const unsigned nb = sweep_grid(g, tx);
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(nb), dim3(64 * kWaves), 0, s, tape, coeffs(static_cast<const void*>(in)),
                       coeffs(static_cast<void*>(mu_out)), g, cp, wt, nb);
  };
  if (tx == 4)
    run(k_coeff_adjoint<4, 2, kNonTemporal>);
  else if (tx == 3)
    state_bytes(g) > kTapeCachedTo ? run(k_coeff_adjoint<3, 2, kNonTemporal>)
                                   : run(k_coeff_adjoint<3, 2, 0>);
  else if (tx == 2)
    run(k_coeff_adjoint<2, 2, 0>);
  else
    run(k_coeff_adjoint<1, 2, 0>);
  return hipGetLastError();
}

hipError_t launch_coeff_adjoint_gather(const double* mu, double* lam, const Geom& gf,
                                       hipStream_t s) {
  const CGeom g = make_cgeom(gf);
  const int tx = sweep_columns(g) > 2 ? 4 : 1;
  const unsigned nb = sweep_grid(g, tx);
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(nb), dim3(64 * kWaves), 0, s,
                       coeffs(static_cast<const void*>(mu)), lam, g, gf, nb);
  };
  tx == 4 ? run(k_coeff_adjoint_last<4>) : run(k_coeff_adjoint_last<1>);
  return hipGetLastError();
}

hipError_t launch_coeff_adjoint_step(const double* tape, const double* lam_in, double* lam_out,
                                     const Geom& gf, const Phys& p, hipStream_t s) {
  const Tiling t = make_tiling(gf.lx, gf.ly);
  hipLaunchKernelGGL(k_coeff_adjoint_step, dim3(t.nb), dim3(kThreads), 0, s, tape, lam_in, lam_out,
                     gf, make_cgeom(gf), make_cphys(p), make_walls(p), t.by, t.bx, t.nty, t.nb);
  return hipGetLastError();
}

}  // namespace d2q37
