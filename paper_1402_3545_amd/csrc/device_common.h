// Device helpers shared by the kernel files: tile order, addressing, lane
// exchange, reductions and the elimination step of the line kernels.
#pragma once

#include <type_traits>

#include "gmg_internal.h"

namespace gmg {

namespace {

constexpr int NTHREADS = 256;

__device__ __forceinline__ int xcd_remap(int b, int n) {
  const int x = b & 7, q = n >> 3, r = n & 7;
  return x * q + min(x, r) + (b >> 3);
}

// A gated launch (a solver's iteration enqueued past its convergence)
// returns at once; the flag is uniform, so whole workgroups leave together.
template <typename T>
__device__ __forceinline__ bool gated(const Lvl<T>& L) {
  return L.gate && *L.gate;
}

// Sum NC per-thread values over the workgroup; thread 0 stores them to
// partials[blockIdx.x*NC + c].  Fixed order, so results are reproducible.
template <int NC, int NW = NTHREADS / 64>
__device__ __forceinline__ void block_partials(double (&v)[NC], double* __restrict__ partials) {
  __shared__ double sm[NC][NW];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v[c] += __shfl_xor(v[c], off);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int c = 0; c < NC; ++c) sm[c][w] = v[c];
  __syncthreads();
  if (threadIdx.x == 0) {
    const int nw = blockDim.x >> 6;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      double s = 0.0;
      for (int q = 0; q < nw; ++q) s += sm[c][q];
      partials[(int64_t)blockIdx.x * NC + c] = s;
    }
  }
}

// Tile coordinates of logical workgroup b (all wave-uniform).  Tiles are
// walked in groups of `group` tile columns: inside a group the tiles of one
// tile row are adjacent and tile rows follow each other, so a tile's
// east/west and north/south neighbours run within a few workgroups of it and
// its halo rows are still in the XCD's L2.  group <= 0 or >= nti: row-major.
// Segments of layers (kb) vary slowest.
__device__ __forceinline__ void tile_coords(int b, int nti, int ntj, int group, int& ti, int& tj,
                                            int& kb) {
  const int per = nti * ntj;
  kb = b / per;
  int r = b - kb * per;
  if (group <= 0 || group >= nti) {
    tj = r / nti;
    ti = r - tj * nti;
    return;
  }
  const int gsize = group * ntj;
  const int gi = r / gsize;
  const int g0 = gi * group;
  const int w = min(group, nti - g0);
  r -= gi * gsize;
  tj = r / w;
  ti = g0 + (r - tj * w);
}

// The item of a grouped launch that workgroup B belongs to (sorted by their
// first workgroups).
template <typename I>
__device__ __forceinline__ int find_item(const I* __restrict__ items, int nitems, int B) {
  int lo = 0, hi = nitems - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (items[mid].blk0 <= B) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Byte base of grid row j of a field (layer 0, column 0).
template <typename T>
__device__ __forceinline__ const char* rowc(const T* f, int j, int64_t jstride) {
  return reinterpret_cast<const char*>(f + (int64_t)j * jstride);
}
template <typename T>
__device__ __forceinline__ char* roww(T* f, int j, int64_t jstride) {
  return reinterpret_cast<char*>(f + (int64_t)j * jstride);
}

// Load/store through a wave-uniform base and a 32-bit per-lane byte offset
// (the saddr form of the global memory instructions).  Stores are
// non-temporal: every output is written once and read by a later kernel, so
// it should not displace the halo rows the L2 is holding for neighbouring
// tiles.  ldn is the non-temporal load for fields a kernel reads exactly once
// (no halo); fields read with horizontal neighbours use ldo.
template <typename T>
__device__ __forceinline__ T ldo(const char* base, uint32_t off) {
  return *reinterpret_cast<const T*>(base + off);
}
template <typename T>
__device__ __forceinline__ T ldn(const char* base, uint32_t off) {
  return __builtin_nontemporal_load(reinterpret_cast<const T*>(base + off));
}
// non-temporal load of a pair (double2 / float2) as one 16- or 8-byte access
template <typename V>
__device__ __forceinline__ V ldn2(const char* base, uint32_t off) {
  using E = decltype(V{}.x);
  typedef E N2 __attribute__((ext_vector_type(2)));
  const N2 t = __builtin_nontemporal_load(reinterpret_cast<const N2*>(base + off));
  return V{t.x, t.y};
}
template <typename T>
__device__ __forceinline__ void sto(char* base, uint32_t off, T v) {
  if constexpr (std::is_arithmetic_v<T>)
    __builtin_nontemporal_store(v, reinterpret_cast<T*>(base + off));
  else
    *reinterpret_cast<T*>(base + off) = v;
}

// A value from another lane of the wavefront by a DPP wave shift: CTRL
// kWaveShl1 gives lane l the value of lane l+1, kWaveShr1 that of lane l-1
// (the lane at the end receives 0).  Every lane of the wavefront must be
// active.
constexpr int kWaveShl1 = 0x130;
constexpr int kWaveShr1 = 0x138;
template <int CTRL, typename T>
__device__ __forceinline__ T wave_shift(T v) {
  if constexpr (sizeof(T) == 8) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf,
                                                              0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL,
                                                              0xf, 0xf, false);
    return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
  } else {
    return __builtin_bit_cast(
        T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
  }
}

// u + (9 a + wb b + wc c + wd d) / 16: the cell-centred bilinear correction of
// one fine cell from its coarse parent a, x and y neighbours b, c and diagonal
// d, with the fused multiply-adds spelled out so that every kernel that forms
// it (the prolongation, and the smoother that folds it in) rounds the same way.
template <typename T>
__device__ __forceinline__ T prolong_add(T u, T a, T b, T c, T d, T wb, T wc, T wd) {
  T p = T(9) * a;
  p = fma(wb, b, p);
  p = fma(wc, c, p);
  p = fma(wd, d, p);
  return fma(p, T(0.0625), u);
}

template <typename T>
struct Vec2;
template <>
struct Vec2<double> { using type = double2; };
template <>
struct Vec2<float> { using type = float2; };

// Reciprocal: hardware estimate refined by Newton-Raphson steps
// r <- r (2 - p r), written as e = 1 - p r, r <- r + r e (two steps in FP64,
// one in FP32 bring the estimate to the last bit or so).  Pivots here are
// positive and well scaled, so no special cases arise.
__device__ __forceinline__ double rcp_nr(double p) {
  double r = __builtin_amdgcn_rcp(p);
  double e = fma(-p, r, 1.0);
  r = fma(r, e, r);
  e = fma(-p, r, 1.0);
  return fma(r, e, r);
}
__device__ __forceinline__ float rcp_nr(float p) {
  const float r = __builtin_amdgcn_rcpf(p);
  const float e = fmaf(-p, r, 1.0f);
  return fmaf(r, e, r);
}

// One elimination step: pivot, its reciprocal and the new c' of this row.
// The line kernels spell out every fused multiply-add, so that each kernel
// (and the back sweep's recomputation of the forward sweep) rounds the same
// way whatever the compiler would contract.
template <typename T>
__device__ __forceinline__ void elim_step(T diag, T cpv, T cnx, T cprev, T& piv, T& inv, T& c) {
  piv = fma(-cpv, cprev, diag);
  inv = rcp_nr(piv);
  c = cnx * inv;
}

}  // namespace

}  // namespace gmg
