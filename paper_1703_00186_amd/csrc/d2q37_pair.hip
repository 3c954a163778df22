// Two steps in one launch from and to stored populations: plain FP64 BGK and the
// shifted FP32 forms (for the FP64 coefficients see d2q37_coeff.hip).
#include <hip/hip_runtime.h>

#include "d2q37_coeff.h"
#include "d2q37_launch.h"
#include "d2q37_tiles.h"

namespace d2q37 {

namespace {

// ---------------------------------------------------------------------------
// Two fused steps in one launch, for the column layout.  A workgroup takes a
// window of 58 rows (64 lanes, three halo rows on each side) of `chunk`
// columns and marches along x, N = 4 columns at a time.  Four producer waves
// gather a column each from memory and collide it; four consumer waves gather
// their columns of the second step from a ring in LDS, collide and store them.
// While the consumers work on the columns that iteration i - 1 completed, the
// producers make iteration i's in registers; a barrier, the oldest slots of
// the ring are overwritten, a barrier.  Every site is computed as by k_fused:
// the same bits.
//
// What bounds it.  The state crosses HBM once for two steps, in both
// directions, plus the halo rows (64 of 58).  Plain FP64 BGK stays bound by
// that: 2048 x 2048 305 us a step against 420, 1024 x 1000 80 against 109.
// The shifted FP32 forms come to the vector unit's rate (two waves on a SIMD):
// 4096 x 4096 852 and 812 us, 1024 x 1000 60 and 49.  The local-reference forms,
// with 1400 and 1750 vector instructions a site, were there before: 4096 x
// 4096 913 and 958, so they have no such kernel.
// Tried: the next columns loaded an iteration ahead (no gain, 81 us at
// 1024 x 1000), two and three columns at a time (89, 82), six with three
// waves per SIMD (spills).
// ---------------------------------------------------------------------------
constexpr int kPairRows = 58, kPairCols = 4;

__device__ __forceinline__ void load_elem(float& v, __amdgpu_buffer_rsrc_t r, unsigned vo,
                                          unsigned so) {
  v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
}
__device__ __forceinline__ void load_elem(double& v, __amdgpu_buffer_rsrc_t r, unsigned vo,
                                          unsigned so) {
  v = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0));
}
template <int kPolicy>
__device__ __forceinline__ void store_elem(float v, __amdgpu_buffer_rsrc_t r, unsigned vo,
                                           unsigned so) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, vo, so, kPolicy);
}
template <int kPolicy>
__device__ __forceinline__ void store_elem(double v, __amdgpu_buffer_rsrc_t r, unsigned vo,
                                           unsigned so) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, v), r, vo, so, kPolicy);
}
// A stride whose multiples are computed where they are used: 37 of them kept
// over a loop would be spilled.
__device__ __forceinline__ unsigned recompute(long long stride) {
  unsigned v = unsigned(stride);
  asm volatile("" : "+s"(v));
  return v;
}

// The ring.  A population is read once, by the target e_x columns on, so those
// of one e_x are kept for e_x + 3 + N columns ([slot][hop][64 rows], one e_x
// after the other), 4 + 3 columns on average instead of N + 6: 133 KB in FP64,
// which a whole ring of ten columns (189 KB) would not fit.
constexpr int hops_of(int ex) {
  int n = 0;
  for (int l = 0; l < Q; ++l) n += EX[l] == ex;
  return n;
}
constexpr int hop_index(int l) {  // among the hops of its e_x
  int n = 0;
  for (int k = 0; k < l; ++k) n += EX[k] == EX[l];
  return n;
}
constexpr int ring_depth(int ex) { return ex + 3 + kPairCols; }
constexpr int ring_start(int ex) {
  int n = 0;
  for (int e = -3; e < ex; ++e) n += ring_depth(e) * hops_of(e) * 64;
  return n;
}

// slots of a column in the rings of e_x = -3 .. 3
struct RingSlots {
  int s[7];
  __device__ __forceinline__ explicit RingSlots(int column) {  // < 2 N
#pragma unroll
    for (int e = 0; e < 7; ++e) s[e] = column >= depth(e) ? column - depth(e) : column;
  }
  static constexpr int depth(int e) { return ring_depth(e - 3); }
  __device__ __forceinline__ void advance() {
#pragma unroll
    for (int e = 0; e < 7; ++e) {
      s[e] += kPairCols;
      if (s[e] >= depth(e)) s[e] -= depth(e);
    }
  }
  __device__ __forceinline__ int at(int l) const {
    return ring_start(EX[l]) + (s[EX[l] + 3] * hops_of(EX[l]) + hop_index(l)) * 64;
  }
};

template <class S, class A, bool kReg, bool kStream, bool kEither>
__global__ __launch_bounds__(128 * kPairCols, 2) void k_fused_pair(const S* __restrict__ src,
                                                                  S* __restrict__ dst, Geom g,
                                                                  Phys P, int windows, int chunk,
                                                                  unsigned nb,
                                                                  const unsigned* word) {
  __shared__ __align__(16) S ring[ring_start(4)];
  set_full(dst);
  const unsigned t = tile_index(nb);
  const int xa = int(t / unsigned(windows)) * chunk, xb = min(xa + chunk, g.lx);
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int y = int(t % unsigned(windows)) * kPairRows - 3 + lane;
  // iteration i: columns xa - 3 + 4 i .. of step one, and the targets whose
  // sources iteration i - 1 completed; both barriers every time
  const int iters = (xb - xa + 6 + kPairCols - 1) / kPairCols;
  if (wave < kPairCols) {
    // rows beyond the walls and beyond the window's halo: any row, not used
    int ys = y;
    if (!g.walls) ys = ys < 0 ? ys + g.ly : (ys >= g.ly ? ys - g.ly : ys);
    ys = min(max(ys, 0), g.ly - 1);
    const bool wall = on_wall_rows(g, ys);
    const unsigned lane_in = unsigned(ys + g.hy - 3) * unsigned(sizeof(S));
    const bool from_coeffs = kEither && holds_coeffs(word);
    RingSlots slot(wave);
    int x = xa - 3 + wave;
    if (x < 0) x += g.lx;
    for (int i = 0; i <= iters; ++i) {
      A f[Q];
      if (i < iters) {
        if (x >= g.lx) x -= g.lx;
        if (from_coeffs) {
          if constexpr (kEither)
            gather_coeffs(coeffs(src), coeff_geom(g), x, ys, [&](int l, double v) { f[l] = v; });
        } else {
          const unsigned cs = recompute(g.cs), ps = recompute(g.ps);
          // padded columns x .. x + 6, the sources of column x
          const __amdgpu_buffer_rsrc_t in = __builtin_amdgcn_make_buffer_rsrc(
              (void*)(src + x * g.cs), (short)0, (2 * HX + 1) * cs * unsigned(sizeof(S)),
              kBufferWord3);
          S raw[Q];
#pragma unroll
          for (int l = 0; l < Q; ++l)
            load_elem(raw[l], in, lane_in + unsigned(3 - EY[l]) * unsigned(sizeof(S)),
                      (unsigned(HX - EX[l]) * cs + unsigned(l) * ps) * unsigned(sizeof(S)));
          __builtin_amdgcn_sched_barrier(0);  // all loads first
#pragma unroll
          for (int l = 0; l < Q; ++l) f[l] = A(raw[l]);
        }
        if (wall) wall_site<A>(f, ys, g.ly, P.th_bottom, P.th_top, P.rho_ref);
        collide<A, kReg>(f, P);
        x += kPairCols;
      }
      __syncthreads();
      if (i < iters) {
#pragma unroll
        for (int l = 0; l < Q; ++l) ring[slot.at(l) + lane] = S(f[l]);
      }
      __syncthreads();
      slot.advance();
    }
  } else {
    const int k = wave - kPairCols;
    const bool store = y >= 0 && y < g.ly && lane >= 3 && lane < 3 + kPairRows;
    const bool wall = store && on_wall_rows(g, y);
    const int from = min(max(lane, 3), 60);  // lanes without a row of their own repeat one
    const unsigned lane_out = store ? unsigned(y + g.hy) * unsigned(sizeof(S)) : 0x80000000u;
    RingSlots slot(k + kPairCols);  // of column x - e_x
    for (int i = 0; i <= iters; ++i) {
      const int x = xa - 6 + (i - 1) * kPairCols + k;
      if (i > 0) {
        if (x >= xa && x < xb) {
          A f[Q];
#pragma unroll
          for (int l = 0; l < Q; ++l) f[l] = A(ring[slot.at(l) + from - EY[l]]);
          if (wall) wall_site<A>(f, y, g.ly, P.th_bottom, P.th_top, P.rho_ref);
          collide<A, kReg>(f, P);
          constexpr int kPolicy = kStream ? kNonTemporal : 0;
          auto put = [&](int X) {  // padded column X
            const unsigned ps = recompute(g.ps);
            const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(
                (void*)(dst + X * g.cs), (short)0, unsigned(g.cs) * unsigned(sizeof(S)),
                kBufferWord3);
#pragma unroll
            for (int l = 0; l < Q; ++l)
              store_elem<kPolicy>(S(f[l]), out, lane_out, unsigned(l) * ps * unsigned(sizeof(S)));
          };
          put(x + HX);
          if (x < HX) put(x + HX + g.lx);
          if (x >= g.lx - HX) put(x + HX - g.lx);
        }
        slot.advance();
      }
      __syncthreads();
      __syncthreads();
    }
  }
}

}  // namespace

hipError_t launch_fused_pair(const void* src, void* dst, const Geom& g, const Phys& p, int prec,
                             int regularize, hipStream_t s) {
  const int windows = (g.ly + kPairRows - 1) / kPairRows;
  const int chunk = march_chunk(g.lx, windows, 256, kPairCols);
  const unsigned n = unsigned(windows) * unsigned((g.lx + chunk - 1) / chunk);
  const auto run = [&](auto kernel, auto elem) {
    using S = decltype(elem);
    hipLaunchKernelGGL(kernel, dim3(n), dim3(128 * kPairCols), 0, s, static_cast<const S*>(src),
                       static_cast<S*>(dst), g, p, windows, chunk, n, word_of(src, g));
  };
  const auto launch = [&](auto streamed) {
    constexpr bool kStream = decltype(streamed)::value;
    if (prec == kF64)
      run(word_of(src, g) ? k_fused_pair<double, double, false, kStream, true>
                          : k_fused_pair<double, double, false, kStream, false>,
          double{});
    else if (prec == kF32Shifted)
      run(regularize ? k_fused_pair<float, double, true, kStream, false>
                     : k_fused_pair<float, double, false, kStream, false>,
          float{});
    else
      run(regularize ? k_fused_pair<float, float, true, kStream, false>
                     : k_fused_pair<float, float, false, kStream, false>,
          float{});
  };
  if (streams_populations(g, prec == kF64 ? sizeof(double) : sizeof(float)))
    launch(std::true_type{});
  else
    launch(std::false_type{});
  return hipGetLastError();
}

}  // namespace d2q37
