// What the real-to-real kernels share beside the FFTs: the pass descriptor, the
// boundary terms of the inhomogeneous FD2 solves (Section 2.4.2), the weighted
// face values added to the source at the unknowns next to a face, and the
// coefficients of the series derivatives.
#pragma once

#include "hp_device.hpp"
#include "hp_internal.hpp"

namespace hp {

// The pass descriptor where the launch put it (the kernels' only argument).
// Read as a parameter it is copied to scratch memory once its uses are many.
// One word of every 64-byte line of it is read at once first: the fields are
// read where they are needed, and each line's first read would be a miss of
// the scalar cache of its own in the chain of a workgroup.
__device__ __forceinline__ const PassArgs& kernel_args() {
  typedef const volatile __attribute__((address_space(4))) int* cptr;
  const cptr w = (cptr)__builtin_amdgcn_kernarg_segment_ptr();
  int x[(sizeof(PassArgs) + 63) / 64];
#pragma unroll
  for (unsigned i = 0; i < sizeof(x) / sizeof(x[0]); ++i) x[i] = w[16 * i];
#pragma unroll
  for (unsigned i = 0; i < sizeof(x) / sizeof(x[0]); ++i) asm volatile("" ::"s"(x[i]));
  return *(const PassArgs*)(const __attribute__((address_space(4))) PassArgs*)__builtin_amdgcn_kernarg_segment_ptr();
}

// Boundary terms of inhomogeneous FD2 problems (added to the source value of
// an unknown next to a face).
template <typename T>
__device__ __forceinline__ double face_terms(const PassArgs& a, int j, int p, int o) {
  int c[3] = {0, 0, 0};
  if (a.ax_j >= 0) c[a.ax_j] = j;
  if (a.ax_p >= 0) c[a.ax_p] = p;
  if (a.ax_o >= 0) c[a.ax_o] = o;
  double add = 0.0;
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      const T* g = (const T*)a.face[ax][side];
      if (!g) continue;
      const int edge = side == 0 ? 0 : a.nunk[ax] - 1;
      if (c[ax] != edge) continue;
      long long off = 0;
      int r = 0;
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        if (b == ax || a.nunk[b] <= 0) continue;
        if (r < 2) off += (long long)(c[b] + ((a.face_off >> b) & 1)) * a.face_s[ax][r];
        ++r;
      }
      add += a.face_w[ax][side] * (double)g[off];
    }
  }
  return add;
}

// Series derivatives (FanJob): the factor of coefficient k of the input for its
// place in the derivative series, and that place (a Laplacian's coefficients
// stay in theirs, its factors are the caller's).  HARTLEY: a Hartley series.
template <bool HARTLEY>
__device__ __forceinline__ double fan_factor(const FanJob& q, int k) {
  if constexpr (HARTLEY) {
    const int s = k == 0 ? 0 : q.n - k;
    return -q.scale * (double)(2 * s < q.n ? s : (2 * s == q.n ? 0 : s - q.n));
  }
  return q.scale * (double)(q.basis == FB_SINE ? k + 1 : k);
}
template <bool HARTLEY>
__device__ __forceinline__ int fan_place(const FanJob& q, int k) {
  if constexpr (HARTLEY) return k == 0 ? 0 : q.n - k;
  return k - q.shift;
}

}  // namespace hp
