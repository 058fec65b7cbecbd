// Device helpers shared by the exact and the inverted-file kNN kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ivhd {

// orders the LDS accesses of a wavefront's lanes on both sides of it
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ bool pair_less(float a, int32_t ia, float b, int32_t ib) {
  return a < b || (a == b && ia < ib);
}

// rows of both arrays start on 16-byte boundaries
__device__ __forceinline__ bool rows_are_vec4(const float *X, const float *Q, int N) {
  return N % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0 && (reinterpret_cast<uintptr_t>(Q) & 15) == 0;
}

// FP32 squared distance of two rows, the features taken in order (16-byte
// loads where the rows allow; the additions are the same)
__device__ __forceinline__ float exact_distance(const float *__restrict__ qr, const float *__restrict__ xr, int N,
                                                bool vec4) {
  float d = 0.f;
  if (vec4) {
    int kk = 0;
    // a 128-byte line of each row at a time, so that a line is fetched once
    // however many rows the wavefronts of a CU are walking
    for (; kk + 32 <= N; kk += 32) {
      float4 u[8], v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        u[j] = *reinterpret_cast<const float4 *>(qr + kk + 4 * j);
        v[j] = *reinterpret_cast<const float4 *>(xr + kk + 4 * j);
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float e = u[j].x - v[j].x;
        d = fmaf(e, e, d);
        e = u[j].y - v[j].y;
        d = fmaf(e, e, d);
        e = u[j].z - v[j].z;
        d = fmaf(e, e, d);
        e = u[j].w - v[j].w;
        d = fmaf(e, e, d);
      }
    }
    for (; kk < N; kk += 4) {
      const float4 u = *reinterpret_cast<const float4 *>(qr + kk);
      const float4 v = *reinterpret_cast<const float4 *>(xr + kk);
      float e = u.x - v.x;
      d = fmaf(e, e, d);
      e = u.y - v.y;
      d = fmaf(e, e, d);
      e = u.z - v.z;
      d = fmaf(e, e, d);
      e = u.w - v.w;
      d = fmaf(e, e, d);
    }
  } else {
    for (int kk = 0; kk < N; ++kk) {
      const float e = qr[kk] - xr[kk];
      d = fmaf(e, e, d);
    }
  }
  return d;
}

}  // namespace ivhd
