// Tiles of the site kernels (one thread per lattice site) and the
// workgroup-to-XCD map, shared by the kernel files.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <type_traits>

#include "d2q37_device.h"

namespace d2q37 {

constexpr int kThreads = 256;
constexpr int kXcds = 8;

// buffer instructions
constexpr int kBufferWord3 = 0x00020000;  // raw 32-bit buffer, gfx9 family
constexpr int kNonTemporal = 2;           // cache policy bits of a streaming access
typedef unsigned v2u __attribute__((ext_vector_type(2)));

struct Tiling {
  int by, bx;    // tile shape (rows, columns)
  int nty, ntx;  // tiles along y and x
  unsigned nb;   // total tiles
};

inline Tiling make_tiling(int lx, int ly) {
  Tiling t;
  t.by = ly > 128 ? 256 : (ly > 64 ? 128 : 64);
  t.bx = kThreads / t.by;
  t.nty = (ly + t.by - 1) / t.by;
  t.ntx = (lx + t.bx - 1) / t.bx;
  t.nb = unsigned(t.nty) * unsigned(t.ntx);
  return t;
}

// Whether a step streams its output past the caches.  The two buffers of a
// state of up to about 150 MB stay in the 256 MB of Infinity Cache from one
// step to the next if the stores are ordinary ones; above, they only push out
// what the step still has to read.  Small states are in the L2s either way,
// and a streamed store saves the write-back at the kernel's end.  The kernels
// name their lines and what they measured there.
inline bool streams_output(long long buffer_bytes, long long cached_from, long long cached_to) {
  return buffer_bytes < cached_from || buffer_bytes > cached_to;
}

// Populations: us per step, streamed and cached, of FP32 with the FP32 collision
// 360 x 360 13.4 and 14.2, 400 x 400 18.7 and 16.7, 512 x 512 21.5 and 18.4,
// 700 x 700 37.2 and 31.0, 1000 x 1000 65 and 64, 1200 x 1200 88 and 94; plain
// FP64 BGK 280 x 280 15.6 and 13.0, 512 x 512 31.5 and 25.2, 700 x 700 56.0 and
// 50.7, 850 x 850 80.5 and 88.3.
inline bool streams_populations(const Geom& g, size_t elem_bytes) {
  return streams_output((long long)g.np * g.nx * g.ny * (long long)elem_bytes,
                        21LL * 1000 * 1000, 156LL * 1000 * 1000);
}

// Columns of a workgroup that makes two steps of a window of rows, `cols`
// columns at a time: its time is the iterations of a chunk, (chunk + 6) / cols
// and one to fill the pipeline, times the rounds in which the workgroups pass
// through the GPU, `slots` at once; the chunk with the least of that product.
// Chunks of cols n - 6 columns use every iteration fully.
inline int march_chunk(int lx, int windows, int slots, int cols) {
  const int first = (6 / cols + 1) * cols - 6;
  int best = first;
  double best_cost = 0.0;
  for (int chunk = first; chunk < lx + cols && chunk <= 2048; chunk += cols) {
    const long long groups = (long long)windows * ((lx + chunk - 1) / chunk);
    // beyond a few rounds the workgroups even out
    const double rounds =
        groups <= 4 * slots ? double((groups + slots - 1) / slots) : double(groups) / slots + 0.5;
    const double cost = rounds * ((std::min(chunk, lx) + 6) / cols + 1);
    if (best_cost == 0.0 || cost < best_cost) {
      best = chunk;
      best_cost = cost;
    }
  }
  return best;
}

inline unsigned grid_1d(long long n) { return unsigned((n + kThreads - 1) / kThreads); }

// Tile of this workgroup after the XCD-aware remap (a bijection of [0, nb)).
__device__ __forceinline__ unsigned tile_index(unsigned nb) {
  const unsigned b = blockIdx.x;
  const unsigned q = nb / kXcds, rem = nb % kXcds;
  const unsigned xcd = b % kXcds, j = b / kXcds;
  return xcd * q + (xcd < rem ? xcd : rem) + j;
}

// Physical (x, y) of this thread; false if it falls outside the lattice.
__device__ __forceinline__ bool site_of(int lx, int ly, int by, int bx, int nty, unsigned nb,
                                        int& x, int& y) {
  const unsigned t = tile_index(nb);
  const int ty = int(t % unsigned(nty)), tx = int(t / unsigned(nty));
  const int lin = threadIdx.x;
  y = ty * by + (lin % by);
  x = tx * bx + (lin / by);
  return x < lx && y < ly;
}
__device__ __forceinline__ bool site_of(const Geom& g, int by, int bx, int nty, unsigned nb,
                                        int& x, int& y) {
  return site_of(g.lx, g.ly, by, bx, nty, nb, x, y);
}

// Block-wide sum of one double per thread; result valid in thread 0.
__device__ __forceinline__ double block_sum(double v) {
  __shared__ double red[kThreads];
  red[threadIdx.x] = v;
  __syncthreads();
#pragma unroll
  for (int s = kThreads / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  return red[0];
}

// Loads before this are issued before the word is read, whose latency then
// passes beside theirs; they are of what the buffer probably holds, and within
// it in either form.
__device__ __forceinline__ void loads_before_word() { asm volatile("" ::: "memory"); }

// What a buffer holds, by its first word (null: as the kernel expects).
__device__ __forceinline__ bool holds_populations(const unsigned* word) {
  return word && *word == unsigned(kFormFull);
}
__device__ __forceinline__ bool holds_coeffs(const unsigned* word) {
  return word && (*word == unsigned(kFormCoeff) || *word == unsigned(kFormCoeffWalls));
}
__device__ __forceinline__ void set_form(void* buf, Form f) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
    *static_cast<unsigned*>(buf) = unsigned(f);
}

// Names the form of an FP64 buffer that a kernel fills with populations.
template <class S>
__device__ __forceinline__ void set_full(S* buf) {
  if constexpr (std::is_same<S, double>::value) set_form(buf, kFormFull);
}

__device__ __forceinline__ bool on_wall_rows(const Geom& g, int y) {
  return g.walls && (y < 3 || y >= g.ly - 3);
}

// The word by which a kernel tells what a buffer holds: null if populations are
// certain ...
inline const unsigned* word_of(const void* buf, const Geom& g) {
  return g.form == kFormFull ? nullptr : static_cast<const unsigned*>(buf);
}
// ... or if either form is.
inline const unsigned* word_if_unsure(const void* buf, const Geom& g) {
  return g.form == kFormCoeff ? nullptr : word_of(buf, g);
}

}  // namespace d2q37
