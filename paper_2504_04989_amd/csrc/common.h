// Shared device/host definitions for the gfx950 T-SVD kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tsvd {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// Interleaved complex value, 8 B (float) or 16 B (double) aligned so a
// complex element moves with one vector load/store.
template <typename T>
struct alignas(2 * sizeof(T)) cx {
  T re, im;
};

// 16x16x4 MFMA: D(16x16) += A(16x4) B(4x16).  Lane l supplies A[l%16][l/16]
// and B[l/16][l%16].  Accumulator r of lane l holds D[row(l/16, r)][l%16]:
// row = 4*(l/16) + r for f32 and (l/16) + 4*r for f64 (measured on gfx950).
template <typename T>
struct Mfma;
template <>
struct Mfma<float> {
  typedef f32x4 acc_t;
  static __device__ __forceinline__ acc_t run(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int q4, int r) { return 4 * q4 + r; }
};
template <>
struct Mfma<double> {
  typedef f64x4 acc_t;
  static __device__ __forceinline__ acc_t run(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int q4, int r) { return q4 + 4 * r; }
};

// Lane exchanges without LDS: a DPP move (the control codes are the wave64 row
// operations quad_perm [1,0,3,2] = 0xB1 and [2,3,0,1] = 0x4E, row_half_mirror
// = 0x141, row_mirror = 0x140, row_ror:8 = 0x128) and the value of one lane.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_value(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_value(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

// Sum over the 64 lanes (all active), the same bits in every lane.  Register
// latency: four DPP steps inside the rows of 16, then the four row sums
// through the scalar unit; six LDS shuffles took about four times as long.
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v += dpp_mov<0x141>(v);
  v += dpp_mov<0x140>(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Sum over the 32 lanes of each half (all 64 active), in every lane of the half.
__device__ __forceinline__ double half_sum(double v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v += dpp_mov<0x141>(v);
  v += dpp_mov<0x140>(v);
  const double lo = lane_value(v, 0) + lane_value(v, 16), hi = lane_value(v, 32) + lane_value(v, 48);
  return (threadIdx.x & 32) ? hi : lo;
}

// Workgroup barrier for data exchanged through LDS alone: unlike
// __syncthreads() it does not wait for the wave's global stores to complete
// (about a microsecond in a step that has just stored a result).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Block-wide sum for blockDim.x == NT (multiple of 64); `red` holds NT/64
// entries of shared memory.  All threads receive the result.
template <int NT, typename T>
__device__ __forceinline__ T block_sum(T v, T* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  T s = 0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) s += red[i];
  return s;
}

// Diagnostic counters kept at the start of the workspace.
enum { INFO_CHOL_SHIFTED = 0, INFO_CHOL_BREAKDOWN = 1, INFO_EIG_NOCONV = 2, INFO_NONFINITE = 3, INFO_TIE = 4,
       INFO_COUNT = 8 };

}  // namespace tsvd
