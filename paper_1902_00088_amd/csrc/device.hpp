// Device helpers shared by the kernel files: the prediction and difference stencils, stage
// value sources, XCD-aware work lists, exact index splits and wave reductions.
#pragma once
#include "internal.hpp"

#include <hip/hip_runtime.h>

namespace mrb {

template <int DIM, int N>
struct Pow { static constexpr int v = N * Pow<DIM - 1, N>::v; };
template <int N>
struct Pow<0, N> { static constexpr int v = 1; };

// midpoint prediction from four equidistant points (cubic through a, b, c, d)
__device__ __forceinline__ double P4(double a, double b, double c, double d) {
  return (9.0 * (b + c) - (a + d)) * 0.0625;
}
__device__ __forceinline__ float P4(float a, float b, float c, float d) {
  return (9.0f * (b + c) - (a + d)) * 0.0625f;
}
// 4th-order central first derivative, r = 1/(12 h)
__device__ __forceinline__ double D4(double um2, double um1, double up1, double up2, double r) {
  return (8.0 * (up1 - um1) - (up2 - um2)) * r;
}
__device__ __forceinline__ float D4(float um2, float um1, float up1, float up2, float r) {
  return (8.0f * (up1 - um1) - (up2 - um2)) * r;
}

// Tensor-product prediction: per axis either one point (n = 1) or four points
// base + q*stride (n = 4) combined by P4; x first, then y, then z.  The number of
// points per axis is fixed at compile time (fully unrolled).
template <int NX, int NY, int NZ, typename T, typename AT>
__device__ __forceinline__ T tensor_fixed(const AT& at, const int* base, const int* stride) {
  T vz[4];
#pragma unroll
  for (int iz = 0; iz < NZ; ++iz) {
    T vy[4];
#pragma unroll
    for (int iy = 0; iy < NY; ++iy) {
      T vx[4];
#pragma unroll
      for (int ix = 0; ix < NX; ++ix)
        vx[ix] = at(base[0] + ix * stride[0], base[1] + iy * stride[1], base[2] + iz * stride[2]);
      vy[iy] = NX == 4 ? P4(vx[0], vx[1], vx[2], vx[3]) : vx[0];
    }
    vz[iz] = NY == 4 ? P4(vy[0], vy[1], vy[2], vy[3]) : vy[0];
  }
  return NZ == 4 ? P4(vz[0], vz[1], vz[2], vz[3]) : vz[0];
}

// p / d for 0 <= p < 2^21 and d >= 1, through the float reciprocal rd = fl(1/d):
// (p + 1/2)/d lies at least 1/(2d) from an integer, and the two roundings (of 1/d and
// of the product) move it by at most (p + 1/2)/d * 2^-23, less than that.  Index splits
// by sizes known only at run time use it: an integer division costs tens of
// instructions per point.
__device__ __forceinline__ int fdiv(int p, float rd) { return (int)(((float)p + 0.5f) * rd); }

// maximum that propagates NaN (a NaN detail must block coarsening)
__device__ __forceinline__ double nanmax(double a, double b) {
  if (a != a) return a;
  if (b != b) return b;
  return a > b ? a : b;
}

// Stage value source: y = u (+ alpha * k), minus a per-field offset in FP32 tiles.
template <typename TT, typename KT, bool HASK>
struct YSrc {
  const double* u;
  const KT* k;
  double alpha;
  const double* off;
  __device__ __forceinline__ TT operator()(size_t i, int f) const {
    double y = u[i];
    if (HASK) y = y + alpha * (double)k[i];
    if constexpr (sizeof(TT) == 4) return (TT)(y - off[f]);
    else return y;
  }
};

// Work items of a launch, XCD-aware: workgroups are dealt round-robin to the 8 XCDs
// (each with its own L2), so XCD x takes the contiguous chunk x of the work list
// (neighbouring blocks in forest order share halo lines in one L2) and its
// workgroups stride through it.  The grid is a multiple of 8.
struct XcdWork {
  int w, end, step;
  __device__ __forceinline__ explicit XcdWork(int total) {
    const int x = blockIdx.x & 7, per = gridDim.x >> 3;
    const int chunk = (total + 7) >> 3;
    w = x * chunk + (blockIdx.x >> 3);
    end = min(total, (x + 1) * chunk);
    step = per;
  }
  __device__ __forceinline__ bool ok() const { return w < end; }
  __device__ __forceinline__ void next() { w += step; }
};

// Source address of a held point as base + sum_a f(t_a) BS^a, with f(t) = 2t for a
// finer holder, t for a same-level one and t/2 (floor) for a coarser one (its points are
// even); f(t) = (2t) >> sh with sh = 1 - dl.  The holder's origin is folded into base.
struct SEnt {
  int base;
  int sh;   // 2 coarser, 1 same level, 0 finer
};

// A 64-bit value moved between lanes of a row by a DPP pattern (both halves; every lane
// active).
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_u64(unsigned long long x) {
  const unsigned lo = __builtin_amdgcn_update_dpp(0u, (unsigned)x, CTRL, 0xF, 0xF, false);
  const unsigned hi = __builtin_amdgcn_update_dpp(0u, (unsigned)(x >> 32), CTRL, 0xF, 0xF, false);
  return ((unsigned long long)hi << 32) | lo;
}

__device__ __forceinline__ unsigned long long lane_u64(unsigned long long x, int lane) {
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)x, lane);
  const unsigned hi = __builtin_amdgcn_readlane((unsigned)(x >> 32), lane);
  return ((unsigned long long)hi << 32) | lo;
}

__device__ __forceinline__ unsigned long long umax64(unsigned long long a, unsigned long long b) {
  return a > b ? a : b;
}

// Maximum over the 64 lanes of a wave (every lane active) of values that are +0, positive
// or NaN with the sign bit clear (|detail| maxima): as unsigned integers such bit patterns
// order as the values do and every NaN lies above +inf, so the integer maximum is the
// NaN-propagating maximum, without branches.  Within rows of 16 lanes by DPP moves (swap
// neighbours, swap pairs, mirror the half rows, mirror the rows), then the four rows'
// results read out; every lane returns it.
__device__ __forceinline__ double wave_nanmax(double v) {
  unsigned long long u = (unsigned long long)__double_as_longlong(v);
  u = umax64(u, dpp_u64<0xB1>(u));    // quad_perm [1, 0, 3, 2]
  u = umax64(u, dpp_u64<0x4E>(u));    // quad_perm [2, 3, 0, 1]
  u = umax64(u, dpp_u64<0x141>(u));   // row_half_mirror
  u = umax64(u, dpp_u64<0x140>(u));   // row_mirror
  u = umax64(umax64(lane_u64(u, 0), lane_u64(u, 16)), umax64(lane_u64(u, 32), lane_u64(u, 48)));
  return __longlong_as_double((long long)u);
}

}  // namespace mrb
