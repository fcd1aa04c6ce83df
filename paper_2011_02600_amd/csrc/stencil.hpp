// Device code shared by the stage kernels: the interior stencils, field
// access, the pointwise part of the right-hand side and the point sources.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.hpp"
#include "kernels.hpp"

namespace sbp {

template <int ORDER>
struct Stencil;
// Table tab:upwind: interior forward stencils alpha_{-r} .. alpha_{q}.
template <>
struct Stencil<2> {
  static constexpr int R = 0, Q = 2, M = 2;
  static constexpr double a[3] = {-3.0 / 2, 2.0, -1.0 / 2};
};
template <>
struct Stencil<3> {
  static constexpr int R = 1, Q = 2, M = 3;
  static constexpr double a[4] = {-1.0 / 3, -1.0 / 2, 1.0, -1.0 / 6};
};
template <>
struct Stencil<4> {
  static constexpr int R = 1, Q = 3, M = 4;
  static constexpr double a[5] = {-1.0 / 4, -5.0 / 6, 3.0 / 2, -1.0 / 2, 1.0 / 12};
};
template <>
struct Stencil<5> {
  static constexpr int R = 2, Q = 3, M = 5;
  static constexpr double a[6] = {1.0 / 20, -1.0 / 2, -1.0 / 3, 1.0, -1.0 / 4, 1.0 / 30};
};
template <>
struct Stencil<6> {
  static constexpr int R = 2, Q = 4, M = 6;
  static constexpr double a[7] = {1.0 / 30, -2.0 / 5, -7.0 / 12, 4.0 / 3, -1.0 / 2, 2.0 / 15, -1.0 / 60};
};
template <>
struct Stencil<7> {
  static constexpr int R = 3, Q = 4, M = 7;
  static constexpr double a[8] = {-1.0 / 105, 1.0 / 10, -3.0 / 5, -1.0 / 4, 1.0, -3.0 / 10, 1.0 / 15, -1.0 / 140};
};
// (alpha_4 printed +1/28; -1/28 sums the coefficients to zero)
template <>
struct Stencil<8> {
  static constexpr int R = 3, Q = 5, M = 8;
  static constexpr double a[9] = {-1.0 / 168, 1.0 / 14, -1.0 / 2,  -9.0 / 20,  5.0 / 4,
                                  -1.0 / 2,   1.0 / 6,  -1.0 / 28, 1.0 / 280};
};

// ---------------------------------------------------------------------------
// element `off` of the field starting at the uniform address `base`: the byte
// offset is formed in 32 bits so that the load uses a scalar base address plus
// a 32-bit vector offset (fields are smaller than 4 GiB)
template <typename T>
__device__ __forceinline__ T ldf(const T* base, unsigned off) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + (unsigned)(off * sizeof(T)));
}
template <typename T>
__device__ __forceinline__ void stf(T* base, unsigned off, T v) {
  *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + (unsigned)(off * sizeof(T))) = v;
}

// Field array accessor: BUF = true uses a buffer resource (one descriptor per
// array, the field offset in a scalar register, the element offset as a
// 32-bit vector offset; the array must be smaller than 4 GiB); BUF = false
// uses plain pointers.  ldn / st mark the access non-temporal (cache policy
// bit NT): data that no other block reads during the launch (the Runge-Kutta
// register, the material, every store) then does not push the halo lines
// that neighbouring tiles are about to read out of L2.
template <typename T, bool BUF>
struct Arr;

template <typename T>
struct Arr<T, true> {
  __amdgpu_buffer_rsrc_t r;
  unsigned fbytes;
  __device__ Arr(const T* p, std::size_t field)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), (short)0, -1, 0x00020000)),
        fbytes((unsigned)(field * sizeof(T))) {}
  static constexpr int kNT = 2;  // cache policy: non-temporal
  template <int POL = 0>
  __device__ __forceinline__ T ldp(int c, unsigned off) const {
    if constexpr (sizeof(T) == 4) {
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)(off * 4u), (int)(c * fbytes), POL));
    } else {
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)(off * 8u), (int)(c * fbytes), POL));
    }
  }
  __device__ __forceinline__ T ld(int c, unsigned off) const { return ldp<0>(c, off); }
  __device__ __forceinline__ T ldn(int c, unsigned off) const { return ldp<kNT>(c, off); }
  template <int POL>
  __device__ __forceinline__ void stp(int c, unsigned off, T v) const {
    if constexpr (sizeof(T) == 4) {
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)(off * 4u), (int)(c * fbytes), POL);
    } else {
      using u2 = unsigned __attribute__((ext_vector_type(2)));
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, (int)(off * 8u), (int)(c * fbytes), POL);
    }
  }
  __device__ __forceinline__ void st(int c, unsigned off, T v) const { stp<kNT>(c, off, v); }
};

template <typename T>
struct Arr<T, false> {
  T* p;
  std::size_t field;
  __device__ Arr(const T* p_, std::size_t f) : p(const_cast<T*>(p_)), field(f) {}
  __device__ __forceinline__ T ld(int c, unsigned off) const { return ldf(p + c * field, off); }
  __device__ __forceinline__ T ldn(int c, unsigned off) const { return ldf(p + c * field, off); }
  __device__ __forceinline__ void st(int c, unsigned off, T v) const { stf(p + c * field, off, v); }
};

// Flux e . sigma_i for the three components i, with e = (m0, m1, m2) a metric
// row: explicit fused multiply-adds in a fixed order, so that every site that
// forms the flux of a node (own point, halo point, s-queue) rounds identically
// and results do not depend on the tiling.
template <typename T>
__device__ __forceinline__ void flux3(T m0, T m1, T m2, T sxx, T syy, T szz, T sxy, T sxz, T syz, T f[3]) {
  f[0] = fma(m2, sxz, fma(m1, sxy, m0 * sxx));
  f[1] = fma(m2, syz, fma(m1, syy, m0 * sxy));
  f[2] = fma(m2, szz, fma(m1, syz, m0 * sxz));
}

// In double precision the scheduler's hoisting of every stencil load of a
// derivative (three components, value and flux) ahead of its arithmetic
// takes more registers than a thread has: a fence between components keeps
// one component's loads in flight at a time.
template <typename T>
__device__ __forceinline__ void sched_fence() {
  if constexpr (sizeof(T) == 8) __builtin_amdgcn_sched_barrier(0);
}

// ---------------------------------------------------------------------------
// pointwise part of the right-hand side at one node: stress rates from the
// velocity derivatives u[xi][i] = D+_xi v_i (non-conservative metric form
// and Hooke's law) and momentum rates from dv[i] = sum_xi D-_xi F_xi,i
template <typename T>
__device__ __forceinline__ void node_rates(const T u[3][3], const T dv[3], const T mq[3], const T mr[3],
                                           const T ms[3], T lamJ, T muJ, T rJ, T rate[9]) {
  T G[3][3];  // G[c][ii] = sum_xi M[xi][c] u[xi][ii]  (= J dv_ii/dx_c)
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int ii = 0; ii < 3; ++ii) G[c][ii] = mq[c] * u[0][ii] + mr[c] * u[1][ii] + ms[c] * u[2][ii];
  const T div = G[0][0] + G[1][1] + G[2][2];
  rate[0] = rJ * dv[0];
  rate[1] = rJ * dv[1];
  rate[2] = rJ * dv[2];
  rate[3] = lamJ * div + T(2) * muJ * G[0][0];
  rate[4] = lamJ * div + T(2) * muJ * G[1][1];
  rate[5] = lamJ * div + T(2) * muJ * G[2][2];
  rate[6] = muJ * (G[1][0] + G[0][1]);
  rate[7] = muJ * (G[2][0] + G[0][2]);
  rate[8] = muJ * (G[2][1] + G[1][2]);
}

// ---------------------------------------------------------------------------
// the point-source increments dt g(t) w M of node (i, j, k) (stress
// components), summed over the sources whose stencil holds it; stride, off: rows
// of the source-time table and the grid's first entry in one
template <typename T>
__device__ __forceinline__ void source_add(const StageArgs<T>& A, int i, int j, int k, T add[6],
                                           int stride = kMaxSources, int off = 0) {
  const int w = A.src_w;
  for (int s = 0; s < A.nsrc; ++s) {
    const int dk = k - A.src_k0[s], dj = j - A.src_j0[s], di = i - A.src_i0[s];
    if ((unsigned)dk < (unsigned)w && (unsigned)dj < (unsigned)w && (unsigned)di < (unsigned)w) {
      const T gdt = A.src_clock
                        ? static_cast<const T*>(A.src_clock->gtab)[((std::size_t)A.src_clock->step * 5 + A.src_stage) *
                                                                       stride + off + s]
                        : A.src_gdt[s];
      const T* wm =
          A.src_wm + ((std::size_t)s * kMaxSrcWidth * kMaxSrcWidth * kMaxSrcWidth + (dk * w + dj) * w + di) * 6;
#pragma unroll
      for (int f = 0; f < 6; ++f) add[f] += gdt * wm[f];
    }
  }
}

// several grids in one launch: last entry of first[0 .. n-1] (non-decreasing, first[0] = 0) that is <= item
__device__ __forceinline__ int batch_find(const int* __restrict__ first, int n, int item) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first[mid] <= item) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

constexpr std::size_t kLdsBytes = 160 * 1024;

}  // namespace sbp
