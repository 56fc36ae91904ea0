// near.hpp -- pieces shared by the near-field kernels (p2p.hip, near_f16.hip).
#pragma once
#include "plan.hpp"

namespace ccfmm {

template <typename T>
__device__ __forceinline__ T rsqrt_t(T x);
template <>
__device__ __forceinline__ float rsqrt_t<float>(float x) {
  return __builtin_amdgcn_rsqf(x);
}
template <>
__device__ __forceinline__ double rsqrt_t<double>(double x) {
  // hardware estimate y (relative error e/2 below 2^-22, e = 1 - x y^2)
  // refined by one third-order step y (1 + e/2 + 3 e^2/8), the binomial series
  // of (1 - e)^(-1/2): five operations where two Newton steps take eight, and the
  // cubed error is far below 2^-53.  (x beyond FP64's range gives inf 0, not zero.)
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * y), y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kP2PWaves = 4;

struct P2PArgs {
  const P2PChunk* chunks;
  const int32_t* nchunks;    // device: the number of chunks (the launch covers the capacity)
  const int32_t* near_ptr;   // level L, compact leaves
  const int32_t* near_idx;
  const int32_t* coord;      // level L, compact leaves
  const int32_t* lstart;
  const int32_t* lcount;
  const int32_t* perm;
  int64_t n;
  int nb;
  int cfg0;                  // first configuration of the launch (k_p2p_multi)
  int split;                 // wavefronts that share a chunk's near list (kSplit kernels): 2 or 4
  double g[3];               // leaf sides / smallest leaf side
  double inv_s3;             // 1 / s_L^3
  int64_t voff;              // offset of level L in V
  const int32_t* leaf_p;     // per-cell local order (compact leaves), or null
  const float* yhi;          // FP32 positions (SoA [3][n])
  const float* ylo;          // FP32 residuals of the positions (SoA [3][n]); null in FP64
  const uint32_t* range;     // null, or (k_p2p_multi) the moments' ranges: only configurations
                             // that the FP16 form leaves (moments_wide) are computed
};

// readlane of a float or double held as bits
__device__ __forceinline__ uint32_t readlane_t(float v, int k) {
  return (uint32_t)__builtin_amdgcn_readlane((int)__builtin_bit_cast(uint32_t, v), k);
}
__device__ __forceinline__ uint64_t readlane_t(double v, int k) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, k);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), k);
  return ((uint64_t)hi << 32) | lo;
}

// Blocks of a launch go to the 8 XCDs in turn, each XCD with its own L2.
// Chunks in key order that are close in the list are close in space and share
// source cells, so each XCD is given runs of kXcdRun consecutive block slots:
// XCD x runs block slots x, x + 8, ... of the remapped order, i.e. runs x,
// x + 8, x + 16, ... of kXcdRun chunks-blocks each.  Within a run the sources
// stay in one L2; every XCD still draws runs from the whole domain, which
// keeps uneven work (clustered dipoles) balanced across the XCDs.  Blocks
// past the last whole group of 8 runs keep their order.
constexpr int kXcdRun = 32;
__device__ __forceinline__ int64_t xcd_run_block(int nblk, int bid) {
  const int full = nblk / (8 * kXcdRun) * (8 * kXcdRun);
  if (bid >= full) return bid;
  const int x = bid & 7, s = bid >> 3;
  return ((int64_t)(s / kXcdRun) * 8 + x) * kXcdRun + s % kXcdRun;
}

// Whether configuration b's moments are too far apart for the FP16 near field, or
// not finite.  range: FP32 bits of the largest one, and of the smallest less one,
// of nb configurations each.
__device__ __forceinline__ bool moments_wide(const uint32_t* range, int nb, int b) {
  const uint32_t top = range[b], low = range[nb + b];  // (low: all ones without any moment)
  return top >= 0x7f800000u || (low != 0xffffffffu && (int)(top >> 23) - (int)((low + 1) >> 23) > 27);
}

P2PArgs p2p_args(Plan& P, int nb, bool fp64);
// near field of a mixed plan for several configurations on the FP16 matrix cores
void run_near_f16(Plan& P, int nb, double* d_H, hipStream_t st);

}  // namespace ccfmm
