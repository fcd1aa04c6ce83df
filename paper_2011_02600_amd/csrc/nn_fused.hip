// Fused layers of the surrogate network (spectral operator with n <= 64 points
// per axis, n a multiple of 4, m <= 16 modes, C <= 64 channels): each pass
// over the activations does everything a layer needs of them.  The operator
// has about 5 flop per byte of activations, far below the matrix cores'
// ridge, so a layer is bound by the activations' traffic; as separate GEMM
// and elementwise calls a layer moved them 9 times forward and 11 backward,
// here 3 and 4.
//
// The unit of work is a line: the C x n values of one (s, z, y), one wave.
// Products are 16 x 16 x 32 bf16 MFMA with the operands rounded to bf16
// where sbp_nn_gemm rounds them and summed in its order (k ascending in
// steps of 32), so every value equals that of the separate calls bit for bit
// (weight and bias gradients, sums over the grid, to rounding).  In a product
// with the line's x as columns, column c16 of tile j is x = 4 c16 + j, so that
// a lane's four tiles are four consecutive x: 16-byte loads and stores.
//
// 8 media of 64^3, 32 channels, 8 modes, 4 layers (forward, loss, backward):
// 6.67 -> 1.91 ms; one medium forward 386 -> 159 us (line_forward 24 us a layer:
// 101 MB, h read, z and h written, at 4.1 TB/s).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "../../include/sbp_nn.h"
#include "nn_math.hpp"

namespace {

using sbp_nn::bf16x8;
using sbp_nn::bf16x4;
using sbp_nn::f32x4;
using sbp_nn::gelu;
using sbp_nn::gelu_grad;

constexpr int kWaves = 4;      // waves per block
constexpr int kLinePitch = 72; // LDS row of a line's bf16 values (64 x + padding)

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ bf16x8 zero8() {
  bf16x8 z;
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.f;
  return z;
}
// LDS values written by this wave are read by its other lanes
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// p[i], or 0 without a branch around the load (p[0] is always readable): one
// branch per load puts their latencies in a row (a medium's forward pass 221
// us with the branches, 159 without)
__device__ __forceinline__ float pick(const float* p, int i, bool ok) {
  const float v = p[ok ? i : 0];
  return ok ? v : 0.f;
}

// operand of the x transform: lane column kx = l % 16, k = x = 32 s + 8 (l / 16) + e
__device__ __forceinline__ bf16x8 basis_x(const float* B, int n, int m, int s, int lane) {
  bf16x8 v;
  const int kx = lane & 15, x0 = 32 * s + 8 * (lane >> 4);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (__bf16)pick(B, (x0 + e) * m + kx, kx < m && x0 + e < n);
  return v;
}
// operand of the inverse x transform: lane column x = 4 (l % 16) + j, k = kx = 8 (l / 16) + e
__device__ __forceinline__ bf16x8 basis_inv(const float* B, int n, int m, int j, int lane) {
  bf16x8 v;
  const int x = 4 * (lane & 15) + j, k0 = 8 * (lane >> 4);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (__bf16)pick(B, x * m + k0 + e, x < n && k0 + e < m);
  return v;
}

struct LineArgs {
  int S, C, n, m;
  const float* basis;    // n x m
  const float* x;        // (S, n^3) input field
  const float* wl;       // lift weights and biases
  const float* bl;
  const float* i1;       // (S, C, n, n, m): the spectral path before the inverse x transform
  const float* src;      // (S, C, n^3) operand of the pointwise product: h_l, or dz_{l+1}; NULL: h_0 from x
                         // (forward) or the values at the receivers (backward)
  const float* W;        // C x C
  const float* bias;
  const float* z_in;     // backward: z_l
  const float* h_in;     // backward: h_l (NULL: h_0 from x)
  const float* wdz;      // backward, last layer: (S, U, C) W^T dz at the U receiver positions
  const int* line_u0;    // first receiver position of a line (n^2 + 1 entries), positions sorted
  const int* upos;       // U flat positions
  int U;
  float* z;              // forward: z_l; backward: dz_l
  float* h;              // forward: h_{l+1}
  float* t1;             // (S, C, n, n, m): x transform of h_{l+1} or dz_l
  float* gw;             // backward: partial sums of dz h^T, C x C per block
  double* gb;            // backward: partial sums of dz, C per block; last pass: of dh and dh x, 2 C
};

// values at a uniform address plus a lane's 32-bit element offset
__device__ __forceinline__ f32x4 ld4(const float* base, unsigned o) {
  return *reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(base) + 4u * o);
}
__device__ __forceinline__ void st4(float* base, unsigned o, f32x4 v) {
  *reinterpret_cast<f32x4*>(reinterpret_cast<char*>(base) + 4u * o) = v;
}
__device__ __forceinline__ void st1(float* base, unsigned o, float v) {
  *reinterpret_cast<float*>(reinterpret_cast<char*>(base) + 4u * o) = v;
}

// operand k = channel, columns x: rows ch = 32 ks + 8 (l / 16) + e of src, tile
// j of lane column c16 = x 4 c16 + j
template <int KS, bool FULL>
__device__ __forceinline__ void load_src(const LineArgs& A, long long off, int lane, f32x4 xin, bool lift,
                                         bf16x8 (&b)[KS][4]) {
  const long long P = (long long)A.n * A.n * A.n;
  const int x = 4 * (lane & 15);
  const bool full = FULL && (KS == 1 ? A.C == 32 : A.C == 64);
  const unsigned lrow = 8u * (lane >> 4) * (unsigned)P + x;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    f32x4 v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int ch = 32 * ks + 8 * (lane >> 4) + e;
      v[e] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (lift) {
        if (full || (ch < A.C && x < A.n)) {
          const float w = A.wl[ch], c = A.bl[ch];
#pragma unroll
          for (int j = 0; j < 4; ++j) v[e][j] = w * xin[j] + c;
        }
      } else if (full || (ch < A.C && x < A.n)) {
        v[e] = ld4(A.src + off + (32 * ks + e) * P, lrow);
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int j = 0; j < 4; ++j) b[ks][j][e] = (__bf16)v[e][j];
  }
}

// W (TR: its transpose) as bf16 in LDS, rows r of 64 + 8 values k, zero past C
constexpr int kWPitch = 72;
template <int CT, bool TR>
__device__ __forceinline__ void stage_w(const float* W, int C, __bf16* lw) {
  for (int e = threadIdx.x; e < 16 * CT * 64; e += 64 * kWaves) {
    const int r = e >> 6, k = e & 63;
    lw[r * kWPitch + k] = (__bf16)pick(W, TR ? k * C + r : r * C + k, r < C && k < C);
  }
}

// inverse x transform of rows 16 i .. 16 i + 15 of the line: acc[j] rows c =
// 16 i + 4 (l / 16) + t, column x = 4 (l % 16) + j.  a: the operand's values
// (inverse_load), loaded ahead
__device__ __forceinline__ bf16x8 inverse_load(const LineArgs& A, const float* i1, int i, int lane) {
  const long long cs = (long long)A.n * A.n * A.m;  // channel stride
  const int c = 16 * i + (lane & 15), k0 = 8 * (lane >> 4);
  bf16x8 a = zero8();
  if (c < A.C && k0 < A.m) {
    const float* const p = i1 + 16 * i * cs;
    const unsigned lo = (lane & 15) * (unsigned)cs + k0;
    // (rows of a multiple of 4 values start on 16 bytes; loads per value instead:
    // forward pass of 4 media of 64^3, 32 channels, m = 12 458 -> 483 us, m = 16
    // 525 -> 564)
    if (A.m % 4 == 0) {
      f32x4 v0 = ld4(p, lo), v1 = {0.f, 0.f, 0.f, 0.f};
      if (k0 + 4 < A.m) v1 = ld4(p + 4, lo);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        a[e] = (__bf16)v0[e];
        a[4 + e] = (__bf16)v1[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        a[e] = (__bf16)pick(p, lo + e, k0 + e < A.m);
    }
  }
  return a;
}
__device__ __forceinline__ void inverse_x(bf16x8 a, const bf16x8 (&bi)[4], f32x4 (&acc)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = mfma(a, bi[j], f32x4{0.f, 0.f, 0.f, 0.f});
}

// rows 16 i .. of the pointwise product
template <int KS>
__device__ __forceinline__ void pointwise(const __bf16* lw, int i, int lane, const bf16x8 (&b)[KS][4],
                                          f32x4 (&acc)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const bf16x8 w =
        *reinterpret_cast<const bf16x8*>(lw + (16 * i + (lane & 15)) * kWPitch + 32 * ks + 8 * (lane >> 4));
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = mfma(w, b[ks][j], acc[j]);
  }
}

// line [c][x] in LDS -> operand rows c = 16 i + l % 16, k = x = 32 s + 8 (l / 16) + e
__device__ __forceinline__ bf16x8 line_operand(const __bf16* lds, int i, int s, int lane) {
  return *reinterpret_cast<const bf16x8*>(lds + (16 * i + (lane & 15)) * kLinePitch + 32 * s + 8 * (lane >> 4));
}

// t1[c][kx] of the line in LDS
template <int CT, int KX>
__device__ __forceinline__ void transform_x(const LineArgs& A, const __bf16* lds, const bf16x8 (&bx)[KX], float* t1,
                                            int lane) {
  const long long cs = (long long)A.n * A.n * A.m;
  const int kx = lane & 15;
  const unsigned lo = 4u * (lane >> 4) * (unsigned)cs + kx;
#pragma unroll
  for (int i = 0; i < CT; ++i) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KX; ++s) v = mfma(line_operand(lds, i, s, lane), bx[s], v);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int c = 16 * i + 4 * (lane >> 4) + t;
      if (c < A.C && kx < A.m) st1(t1 + (16 * i + t) * cs, lo, v[t]);
    }
  }
}

// ---- forward: z_l = T^T(..) + W h_l + b, h_{l+1} = gelu(z_l), t1 = its x
// transform; LIFT_ONLY: t1 of h_0 = w x + b alone
// FULL: lines and channels fill the tiles (n = 64 and C = 16 CT), no masks.
// Forward and backward of 4 media of 64^3, 8 modes, with and without: 16 channels
// 738 and 764 us, 32 1124 and 1208, 48 1642 and 1715, 64 2230 and 2305, though
// the backward pass spills more at 64 (at 48 the forward pass alone is 692 and
// 663, for one medium 234 and 251)
template <int CT, int KS, int KX, bool LIFT_ONLY, bool FULL>
__global__ __launch_bounds__(64 * kWaves, CT <= 2 ? 4 : 2) void line_forward_kernel(const LineArgs A) {
  __shared__ __align__(16) __bf16 lds_all[kWaves][16 * CT * kLinePitch];
  __shared__ __align__(16) __bf16 lw[LIFT_ONLY ? 8 : 16 * CT * kWPitch];
  // (scalar, so that the line's base addresses are)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4;
  __bf16* const lds = lds_all[wave];
  const int n = A.n, C = A.C, nn = n * n;
  const long long P = (long long)nn * n, lines = (long long)A.S * nn;
  const int x = 4 * (lane & 15);
  const bool xok = FULL || x < n;
  const unsigned lrow = 4u * g * (unsigned)P + x;
  const bool lift = A.src == nullptr;
  bf16x8 bi[4], bx[KX];
#pragma unroll
  for (int s = 0; s < KX; ++s) bx[s] = basis_x(A.basis, n, A.m, s, lane);
  if constexpr (!LIFT_ONLY) {
    stage_w<CT, false>(A.W, C, lw);
#pragma unroll
    for (int j = 0; j < 4; ++j) bi[j] = basis_inv(A.basis, n, A.m, j, lane);
  }
  // (columns past the line's end are read with zero basis values: keep them finite)
  if constexpr (!FULL)
    for (int e = lane; e < 16 * CT * kLinePitch; e += 64) lds[e] = (__bf16)0.f;
  __syncthreads();
  for (long long ln = (long long)blockIdx.x * kWaves + wave; ln < lines; ln += (long long)gridDim.x * kWaves) {
    const long long s = ln / nn, zy = ln - s * nn;
    const long long off = s * C * P + zy * n;  // channel 0 of the line
    f32x4 xin = {0.f, 0.f, 0.f, 0.f};
    if (lift && xok) xin = *reinterpret_cast<const f32x4*>(A.x + s * P + zy * n + x);
    if constexpr (LIFT_ONLY) {
#pragma unroll
      for (int i = 0; i < CT; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int c = 16 * i + 4 * g + t;
          if (FULL || (c < C && xok)) {
            const float w = A.wl[c], b = A.bl[c];
#pragma unroll
            for (int j = 0; j < 4; ++j) lds[c * kLinePitch + x + j] = (__bf16)(w * xin[j] + b);
          }
        }
    } else {
      bf16x8 b[KS][4], a[CT];
      load_src<KS, FULL>(A, off, lane, xin, lift, b);
      const float* const i1 = A.i1 + (s * C * nn + zy) * A.m;
#pragma unroll
      for (int i = 0; i < CT; ++i) a[i] = inverse_load(A, i1, i, lane);
#pragma unroll
      for (int i = 0; i < CT; ++i) {
        f32x4 ak[4], au[4];
        inverse_x(a[i], bi, ak);
        pointwise<KS>(lw, i, lane, b, au);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int c = 16 * i + 4 * g + t;
          if (FULL || (c < C && xok)) {
            const float bc = A.bias[c];
            f32x4 zv, hv;
            bf16x4 hb;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              zv[j] = ak[j][t] + au[j][t] + bc;
              hv[j] = gelu(zv[j]);
              hb[j] = (__bf16)hv[j];
            }
            *reinterpret_cast<bf16x4*>(lds + c * kLinePitch + x) = hb;
            st4(A.z + off + (16 * i + t) * P, lrow, zv);
            st4(A.h + off + (16 * i + t) * P, lrow, hv);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    wave_lds_sync();
    transform_x<CT, KX>(A, lds, bx, A.t1 + (s * C * nn + zy) * A.m, lane);
    wave_lds_sync();
  }
}

// ---- backward: dh = T^T(..) + W^T dz_{l+1} (the second term at the receivers
// alone below the last layer), dz_l = dh gelu'(z_l), t1 = its x transform,
// partial sums of dz_l h_l^T and dz_l; LAST: partial sums of dh_0 x and dh_0
template <int CT, int KS, int KX, bool LAST, bool FULL>
__global__ __launch_bounds__(64 * kWaves, 2) void line_backward_kernel(const LineArgs A) {
  __shared__ __align__(16) __bf16 lds_all[kWaves][16 * CT * kLinePitch];
  __shared__ __align__(16) __bf16 lw[16 * CT * kWPitch];
  __shared__ float red[LAST ? 1 : 16 * CT * 16 * CT];
  __shared__ double redb[2 * 16 * CT];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  __bf16* const lds = lds_all[wave];
  const int n = A.n, C = A.C, nn = n * n;
  const long long P = (long long)nn * n, lines = (long long)A.S * nn;
  const int x = 4 * (lane & 15), g = lane >> 4;
  const bool xok = FULL || x < n;
  const unsigned lrow = 4u * g * (unsigned)P + x;
  const bool sparse = A.src == nullptr, lift = A.h_in == nullptr;
  bf16x8 bi[4], bx[KX];
  if (!sparse) stage_w<CT, true>(A.W, C, lw);
#pragma unroll
  for (int j = 0; j < 4; ++j) bi[j] = basis_inv(A.basis, n, A.m, j, lane);
  if constexpr (!LAST) {
#pragma unroll
    for (int s = 0; s < KX; ++s) bx[s] = basis_x(A.basis, n, A.m, s, lane);
    if constexpr (!FULL)
      for (int e = lane; e < 16 * CT * kLinePitch; e += 64) lds[e] = (__bf16)0.f;
  }
  __syncthreads();
  f32x4 aw[CT][CT];
  double sb[CT][4], sx[LAST ? CT : 1][4];
#pragma unroll
  for (int i = 0; i < CT; ++i)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      sb[i][t] = 0.0;
      if constexpr (LAST) sx[i][t] = 0.0;
    }
#pragma unroll
  for (int i = 0; i < CT; ++i)
#pragma unroll
    for (int k = 0; k < CT; ++k) aw[i][k] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (long long ln = (long long)blockIdx.x * kWaves + wave; ln < lines; ln += (long long)gridDim.x * kWaves) {
    const long long s = ln / nn, zy = ln - s * nn;
    const long long off = s * C * P + zy * n;
    bf16x8 b[KS][4], a[CT];
    if (!sparse) load_src<KS, FULL>(A, off, lane, f32x4{0.f, 0.f, 0.f, 0.f}, false, b);
    const float* const i1 = A.i1 + (s * C * nn + zy) * A.m;
#pragma unroll
    for (int i = 0; i < CT; ++i) a[i] = inverse_load(A, i1, i, lane);
    f32x4 xv = {0.f, 0.f, 0.f, 0.f};
    if (LAST && xok) xv = *reinterpret_cast<const f32x4*>(A.x + s * P + zy * n + x);
    const int u0 = sparse ? A.line_u0[zy] : 0, u1 = sparse ? A.line_u0[zy + 1] : 0;
#pragma unroll
    for (int i = 0; i < CT; ++i) {
      f32x4 zv[4];  // [t]: z of the lane's four x
      if constexpr (!LAST) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int c = 16 * i + 4 * g + t;
          zv[t] = f32x4{0.f, 0.f, 0.f, 0.f};
          if (FULL || (c < C && xok)) zv[t] = ld4(A.z_in + off + (16 * i + t) * P, lrow);
        }
      }
      f32x4 dh[4];
      inverse_x(a[i], bi, dh);
      if (!sparse) {
        f32x4 au[4];
        pointwise<KS>(lw, i, lane, b, au);
#pragma unroll
        for (int j = 0; j < 4; ++j) dh[j] += au[j];
      } else {
        for (int u = u0; u < u1; ++u) {
          const int xu = A.upos[u] - (int)zy * n;
          if (xu >= x && xu < x + 4) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const int c = 16 * i + 4 * g + t;
              const float v = c < C ? A.wdz[(s * A.U + u) * C + c] : 0.f;
#pragma unroll
              for (int j = 0; j < 4; ++j)
                if (xu == x + j) dh[j][t] += v;
            }
          }
        }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int c = 16 * i + 4 * g + t;
        if (FULL || (c < C && xok)) {
          if constexpr (LAST) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              sb[i][t] += (double)dh[j][t];
              sx[i][t] += (double)dh[j][t] * (double)xv[j];
            }
          } else {
            f32x4 dz;
            bf16x4 db;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              dz[j] = dh[j][t] * gelu_grad(zv[t][j]);
              sb[i][t] += (double)dz[j];
              db[j] = (__bf16)dz[j];
            }
            *reinterpret_cast<bf16x4*>(lds + c * kLinePitch + x) = db;
            st4(A.z + off + (16 * i + t) * P, lrow, dz);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (!LAST) {
      wave_lds_sync();
      transform_x<CT, KX>(A, lds, bx, A.t1 + (s * C * nn + zy) * A.m, lane);
      // weight gradient: rows co of dz, columns ci = 16 k + l % 16 of h, k index
      // x = 32 q + 8 g + e
#pragma unroll
      for (int k = 0; k < CT; ++k) {
        const int c = 16 * k + (lane & 15);
        const float wc = lift && c < C ? A.wl[c] : 0.f, bc = lift && c < C ? A.bl[c] : 0.f;
#pragma unroll
        for (int q = 0; q < KX; ++q) {
          bf16x8 hb;
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            const int xx = 32 * q + 8 * g + 4 * p;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (FULL || (c < C && xx < n)) {
              if (lift) {
                v = ld4(A.x + s * P + zy * n + 32 * q + 4 * p, 8 * g);
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = wc * v[j] + bc;
              } else {
                v = ld4(A.h_in + off + 16 * k * P + 32 * q + 4 * p, (lane & 15) * (unsigned)P + 8 * g);
              }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) hb[4 * p + j] = (__bf16)v[j];
          }
#pragma unroll
          for (int i = 0; i < CT; ++i) aw[i][k] = mfma(line_operand(lds, i, q, lane), hb, aw[i][k]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      wave_lds_sync();
    }
  }
  // ---- the block's partial sums: wave after wave, in order
  if constexpr (!LAST) {
    for (int wv = 0; wv < kWaves; ++wv) {
      if (wave == wv) {
#pragma unroll
        for (int i = 0; i < CT; ++i)
#pragma unroll
          for (int k = 0; k < CT; ++k)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              float* r = red + (16 * i + 4 * g + t) * 16 * CT + 16 * k + (lane & 15);
              *r = wv == 0 ? aw[i][k][t] : *r + aw[i][k][t];
            }
      }
      __syncthreads();
    }
    for (int e = threadIdx.x; e < C * C; e += 64 * kWaves)
      A.gw[(long long)blockIdx.x * C * C + e] = red[(e / C) * 16 * CT + e % C];
  }
  // sums over the 16 lanes that hold a row's columns
#pragma unroll
  for (int i = 0; i < CT; ++i)
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int d = 1; d < 16; d <<= 1) {
        sb[i][t] += __shfl_xor(sb[i][t], d, 16);
        if constexpr (LAST) sx[i][t] += __shfl_xor(sx[i][t], d, 16);
      }
  for (int wv = 0; wv < kWaves; ++wv) {
    if (wave == wv && (lane & 15) == 0) {
#pragma unroll
      for (int i = 0; i < CT; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int c = 16 * i + 4 * g + t;
          redb[c] = wv == 0 ? sb[i][t] : redb[c] + sb[i][t];
          if constexpr (LAST) redb[16 * CT + c] = wv == 0 ? sx[i][t] : redb[16 * CT + c] + sx[i][t];
        }
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < (LAST ? 2 * C : C); e += 64 * kWaves)
    A.gb[(long long)blockIdx.x * (LAST ? 2 * C : C) + e] = redb[e < C ? e : 16 * CT + e - C];
}

// out[c] = sum over the nb blocks' partial sums part[b * stride + c], a block
// per entry, in a fixed order; the entries past C go to out2
__global__ __launch_bounds__(256) void sum_blocks_kernel(int nb, int stride, int C, const double* part, float* out,
                                                         float* out2) {
  __shared__ double red[256];
  const int c = blockIdx.x;
  double v = 0.0;
  for (int b = threadIdx.x; b < nb; b += 256) v += part[(long long)b * stride + c];
  red[threadIdx.x] = v;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) (c < C ? out[c] : out2[c - C]) = (float)red[0];
}

// ---- y and z transforms of t1 in two launches, a wave per planes and per
// column tile: with one block per (s, c) doing both, one medium of 32 channels
// filled 32 of 256 CUs (32 us; now 4 + 3)
// t1 (SC, n, n, m) -> the y transform of each plane z, in place: [z][ky][kx] over
// the plane's first m m values.  A wave takes two planes and reads both before
// it writes.
__global__ __launch_bounds__(256) void modes_y_kernel(int n, int m, const float* B, float* t1) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c16 = lane & 15, g = lane >> 4;
  const int ks = (n + 31) / 32, z0 = 8 * blockIdx.y + 2 * wave;
  float* const src = t1 + (long long)blockIdx.x * n * n * m;
  float v[2][2][8];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int z = z0 + u, y = 32 * s + 8 * g + e;
        v[u][s][e] = pick(src, (z * n + y) * m + c16, z < n && y < n && c16 < m);
      }
  bf16x8 bt[2];  // rows k = l % 16 of B^T, k index 32 s + 8 g + e
#pragma unroll
  for (int s = 0; s < 2; ++s) bt[s] = s < ks ? basis_x(B, n, m, s, lane) : zero8();
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (s < ks) {
        bf16x8 b;
#pragma unroll
        for (int e = 0; e < 8; ++e) b[e] = (__bf16)v[u][s][e];
        acc = mfma(bt[s], b, acc);
      }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int ky = 4 * g + t;
      if (z0 + u < n && ky < m && c16 < m) src[(z0 + u) * n * m + ky * m + c16] = acc[t];
    }
  }
}

// out (SC, m, m m) = z transform of what modes_y_kernel left in t1; a wave per
// 16 columns (ky, kx)
__global__ __launch_bounds__(64) void modes_z_kernel(int n, int m, const float* B, const float* t1, float* out) {
  const int lane = threadIdx.x, c16 = lane & 15, g = lane >> 4, col = 16 * blockIdx.y + c16, mm = m * m;
  const float* const src = t1 + (long long)blockIdx.x * n * n * m;
  float v[2][8];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int z = 32 * s + 8 * g + e;
      v[s][e] = pick(src, z * n * m + col, z < n && col < mm);
    }
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 2; ++s)
    if (s < (n + 31) / 32) {
      bf16x8 b;
#pragma unroll
      for (int e = 0; e < 8; ++e) b[e] = (__bf16)v[s][e];
      acc = mfma(basis_x(B, n, m, s, lane), b, acc);
    }
  float* const dst = out + (long long)blockIdx.x * m * mm;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int kz = 4 * g + t;
    if (kz < m && col < mm) dst[kz * mm + col] = acc[t];
  }
}

// operand rows p = 16 i + l % 16 of B (points), k = mode 8 (l / 16) + e
__device__ __forceinline__ bf16x8 basis_rows(const float* B, int n, int m, int p, int lane) {
  bf16x8 v;
  const int k0 = 8 * (lane >> 4);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (__bf16)pick(B, p * m + k0 + e, p < n && k0 + e < m);
  return v;
}

// ---- inverse z and y transforms of one (s, c): (m, m, m) -> i1 (n, n, m).
// After the z transform of 16 planes their values wait in LDS with ky
// innermost for the y transform
constexpr int kInvThreads = 512;
__global__ __launch_bounds__(kInvThreads) void modes_inverse_kernel(int n, int m, const float* B, const float* y,
                                                            float* i1) {
  __shared__ __align__(16) __bf16 t2[16][16][24];  // [z][kx][ky]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c16 = lane & 15, g = lane >> 4;
  const int mm = m * m, nt = (n + 15) / 16;
  const float* src = y + (long long)blockIdx.x * m * mm;
  float* dst = i1 + (long long)blockIdx.x * n * n * m;
  for (int e = threadIdx.x; e < 16 * 16 * 24; e += kInvThreads) (&t2[0][0][0])[e] = (__bf16)0.f;
  bf16x8 ay[4];  // basis rows of the y tiles
#pragma unroll
  for (int q = 0; q < 4; ++q) ay[q] = basis_rows(B, n, m, 16 * q + c16, lane);
  __syncthreads();
  const int zt = blockIdx.y;
  const bf16x8 az = basis_rows(B, n, m, 16 * zt + c16, lane);
  for (int j = wave; j < (mm + 15) / 16; j += kInvThreads / 64) {
    const int col = 16 * j + c16;
    bf16x8 b;
#pragma unroll
    for (int e = 0; e < 8; ++e) b[e] = (__bf16)pick(src, (8 * g + e) * mm + col, 8 * g + e < m && col < mm);
    const f32x4 v = mfma(az, b, f32x4{0.f, 0.f, 0.f, 0.f});
    if (col < mm) {
#pragma unroll
      for (int t = 0; t < 4; ++t) t2[4 * g + t][col % m][col / m] = (__bf16)v[t];
    }
  }
  __syncthreads();
  for (int zl = wave; zl < 16; zl += kInvThreads / 64) {
    const int z = 16 * zt + zl;
    if (z >= n) break;
    bf16x8 b = zero8();
    if (g < 2) b = *reinterpret_cast<const bf16x8*>(&t2[zl][c16][8 * g]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q >= nt) break;
      const f32x4 v = mfma(ay[q], b, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int yy = 16 * q + 4 * g + t;
        if (yy < n && c16 < m) dst[(z * n + yy) * m + c16] = v[t];
      }
    }
  }
}

// ---- the last layer at one receiver: f[s][r][c] = (T^T y)[c] + (W h)[c] + b[c]
// at its point; one block per (r, s, 16 channels), one wave per channel
constexpr int kRecWaves = 16;
__global__ __launch_bounds__(64 * kRecWaves) void receiver_forward_kernel(int C, int n, int m, int R, const float* B,
                                                                          const float* y, const float* h,
                                                                          const float* W, const float* bias,
                                                                          const int* pos, float* f) {
  __shared__ __align__(16) __bf16 t2[kRecWaves][16][24];  // [kx][ky] of the wave's channel
  __shared__ __align__(16) __bf16 li[16][24];             // [c][kx]
  __shared__ __align__(16) __bf16 hp[64];                 // h at the point
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c16 = lane & 15, g = lane >> 4;
  const int r = blockIdx.x, s = blockIdx.y, i = blockIdx.z, c = 16 * i + wave, mm = m * m;
  const long long P = (long long)n * n * n;
  const int p = pos[r], zr = p / (n * n), yr = p / n % n, xr = p % n;
  for (int e = threadIdx.x; e < kRecWaves * 16 * 24; e += 64 * kRecWaves) (&t2[0][0][0])[e] = (__bf16)0.f;
  for (int e = threadIdx.x; e < 16 * 24; e += 64 * kRecWaves) (&li[0][0])[e] = (__bf16)0.f;
  if (threadIdx.x < 64) hp[threadIdx.x] = (__bf16)((int)threadIdx.x < C ? h[((long long)s * C + threadIdx.x) * P + p] : 0.f);
  __syncthreads();
  // the point is row 0 of the basis operands, column 0 of the last one
  const bf16x8 az = c16 == 0 ? basis_rows(B, n, m, zr, lane) : zero8();
  const bf16x8 ay = c16 == 0 ? basis_rows(B, n, m, yr, lane) : zero8();
  const bf16x8 ax = c16 == 0 ? basis_rows(B, n, m, xr, lane) : zero8();
  if (c < C) {
    const float* src = y + ((long long)s * C + c) * m * mm;
    const int nj = (mm + 15) / 16;
    for (int j0 = 0; j0 < nj; j0 += 4) {  // (four tiles' loads in flight)
      float l[4][8];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int k = 8 * g + e, col = 16 * (j0 + j) + c16;
          l[j][e] = pick(src, k * mm + col, k < m && col < mm);
        }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (j0 + j >= nj) break;
        const int col = 16 * (j0 + j) + c16;
        bf16x8 b;
#pragma unroll
        for (int e = 0; e < 8; ++e) b[e] = (__bf16)l[j][e];
        const f32x4 v = mfma(az, b, f32x4{0.f, 0.f, 0.f, 0.f});
        if (g == 0 && col < mm) t2[wave][col % m][col / m] = (__bf16)v[0];
      }
    }
    wave_lds_sync();
    bf16x8 b = zero8();
    if (g < 2) b = *reinterpret_cast<const bf16x8*>(&t2[wave][c16][8 * g]);
    const f32x4 v = mfma(ay, b, f32x4{0.f, 0.f, 0.f, 0.f});
    if (g == 0 && c16 < m) li[wave][c16] = (__bf16)v[0];
  }
  __syncthreads();
  if (wave == 0) {
    bf16x8 a = zero8();
    if (g < 2) a = *reinterpret_cast<const bf16x8*>(&li[c16][8 * g]);
    const f32x4 k = mfma(a, ax, f32x4{0.f, 0.f, 0.f, 0.f});
    f32x4 u = {0.f, 0.f, 0.f, 0.f};
    for (int ks = 0; ks < (C + 31) / 32; ++ks) {
      bf16x8 w;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int row = 16 * i + c16, ci = 32 * ks + 8 * g + e;
        w[e] = (__bf16)pick(W, row * C + ci, row < C && ci < C);
      }
      const bf16x8 b = c16 == 0 ? *reinterpret_cast<const bf16x8*>(hp + 32 * ks + 8 * g) : zero8();
      u = mfma(w, b, u);
    }
    if (c16 == 0) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int c = 16 * i + 4 * g + t;
        if (c < C) f[((long long)s * R + r) * C + c] = k[t] + u[t] + bias[c];
      }
    }
  }
}

// ---- last layer backward at the receivers: dz at the U distinct positions
// (the receivers of a position in their order), its x transform (t1, cleared
// by the caller), h there; block (line with receivers, s)
__global__ __launch_bounds__(64) void receiver_backward_kernel(int C, int n, int m, int R, int U, const float* B,
                                                               const float* df, const float* h, const int* lines,
                                                               const int* line_u0, const int* upos, const int* u_r0,
                                                               const int* u_r, float* dzu, float* hu, float* t1) {
  __shared__ __align__(16) __bf16 lds[64 * kLinePitch];
  const int lane = threadIdx.x, s = blockIdx.y, zy = lines[blockIdx.x];
  const long long P = (long long)n * n * n, nn = (long long)n * n;
  for (int e = lane; e < 64 * kLinePitch; e += 64) lds[e] = (__bf16)0.f;
  wave_lds_sync();
  for (int u = line_u0[zy]; u < line_u0[zy + 1]; ++u) {
    const int c = lane;
    if (c < C) {
      float v = 0.f;
      for (int q = u_r0[u]; q < u_r0[u + 1]; ++q) v += df[((long long)s * R + u_r[q]) * C + c];
      dzu[((long long)s * U + u) * C + c] = v;
      hu[((long long)s * U + u) * C + c] = h[((long long)s * C + c) * P + upos[u]];
      lds[c * kLinePitch + upos[u] - zy * n] = (__bf16)v;
    }
  }
  wave_lds_sync();
  const int kx = lane & 15;
  for (int i = 0; i < (C + 15) / 16; ++i) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    for (int q = 0; q < (n + 31) / 32; ++q) v = mfma(line_operand(lds, i, q, lane), basis_x(B, n, m, q, lane), v);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int c = 16 * i + 4 * (lane >> 4) + t;
      if (c < C && kx < m) t1[(((long long)s * C + c) * nn + zy) * m + kx] = v[t];
    }
  }
}

__global__ void clear_kernel(long long n4, f32x4* p) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n4; e += (long long)gridDim.x * blockDim.x)
    p[e] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// out[c] = sum over the rows of x (rows, C), in double, in a fixed order; a
// block per column
__global__ __launch_bounds__(256) void column_sum_kernel(long long rows, int C, const float* x, float* out) {
  __shared__ double red[256];
  const int c = blockIdx.x;
  double v = 0.0;
  for (long long r = threadIdx.x; r < rows; r += 256) v += (double)x[r * C + c];
  red[threadIdx.x] = v;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[c] = (float)red[0];
}

int fail(const char* msg) { return sbp_nn::set_error(msg); }

bool shape_ok(int S, int C, int n, int m) {
  return S >= 0 && C >= 1 && C <= 64 && n >= 4 && n <= 64 && n % 4 == 0 && m >= 1 && m <= 16 && m <= n;
}

int line_blocks(int S, int n) {
  const long long lines = (long long)S * n * n, b = (lines + kWaves - 1) / kWaves;
  return (int)std::min<long long>(b, SBP_NN_LINE_BLOCKS);
}

template <int CT, int KS, bool ONLY>
void forward_kx(const LineArgs& a, hipStream_t st) {
  const dim3 grid(line_blocks(a.S, a.n)), block(64 * kWaves);
  if (a.n == 64 && a.C == 16 * CT)
    hipLaunchKernelGGL((line_forward_kernel<CT, KS, 2, ONLY, true>), grid, block, 0, st, a);
  else if (a.n > 32)
    hipLaunchKernelGGL((line_forward_kernel<CT, KS, 2, ONLY, false>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((line_forward_kernel<CT, KS, 1, ONLY, false>), grid, block, 0, st, a);
}
template <bool ONLY>
void forward_c(const LineArgs& a, hipStream_t st) {
  if (a.C <= 16) forward_kx<1, 1, ONLY>(a, st);
  else if (a.C <= 32) forward_kx<2, 1, ONLY>(a, st);
  else if (a.C <= 48) forward_kx<3, 2, ONLY>(a, st);
  else forward_kx<4, 2, ONLY>(a, st);
}
template <int CT, int KS, bool LAST>
void backward_kx(const LineArgs& a, hipStream_t st) {
  const dim3 grid(line_blocks(a.S, a.n)), block(64 * kWaves);
  if (a.n == 64 && a.C == 16 * CT)
    hipLaunchKernelGGL((line_backward_kernel<CT, KS, 2, LAST, true>), grid, block, 0, st, a);
  else if (a.n > 32)
    hipLaunchKernelGGL((line_backward_kernel<CT, KS, 2, LAST, false>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((line_backward_kernel<CT, KS, 1, LAST, false>), grid, block, 0, st, a);
}
template <bool LAST>
void backward_c(const LineArgs& a, hipStream_t st) {
  if (a.C <= 16) backward_kx<1, 1, LAST>(a, st);
  else if (a.C <= 32) backward_kx<2, 1, LAST>(a, st);
  else if (a.C <= 48) backward_kx<3, 2, LAST>(a, st);
  else backward_kx<4, 2, LAST>(a, st);
}

}  // namespace

extern "C" {

int sbp_nn_lift_modes(int S, int C, int n, int m, const float* basis, const float* x, const float* wl,
                      const float* bl, float* t1, void* stream) {
  if (!shape_ok(S, C, n, m) || !basis || !x || !wl || !bl || !t1) return fail("invalid lift_modes arguments");
  if (S == 0) return SBP_NN_OK;
  LineArgs a{};
  a.S = S, a.C = C, a.n = n, a.m = m, a.basis = basis, a.x = x, a.wl = wl, a.bl = bl, a.t1 = t1;
  forward_c<true>(a, (hipStream_t)stream);
  return sbp_nn::status();
}

int sbp_nn_line_forward(int S, int C, int n, int m, const float* basis, const float* i1, const float* h,
                        const float* x, const float* wl, const float* bl, const float* W, const float* bias, float* z,
                        float* hn, float* t1, void* stream) {
  if (!shape_ok(S, C, n, m) || !basis || !i1 || !x || !wl || !bl || !W || !bias || !z || !hn || !t1)
    return fail("invalid line_forward arguments");
  if (S == 0) return SBP_NN_OK;
  LineArgs a{};
  a.S = S, a.C = C, a.n = n, a.m = m, a.basis = basis, a.x = x, a.wl = wl, a.bl = bl, a.i1 = i1, a.src = h, a.W = W,
  a.bias = bias, a.z = z, a.h = hn, a.t1 = t1;
  forward_c<false>(a, (hipStream_t)stream);
  return sbp_nn::status();
}

int sbp_nn_line_backward(int S, int C, int n, int m, const float* basis, const float* i1, const float* dz_next,
                         const float* W, int U, const int* line_u0, const int* upos, const float* wdz, const float* z,
                         const float* h, const float* x, const float* wl, const float* bl, float* dz, float* t1,
                         float* gw_part, double* gb_part, void* stream) {
  if (!shape_ok(S, C, n, m) || !basis || !i1 || !z || !x || !wl || !bl || !dz || !t1 || !gw_part || !gb_part ||
      (dz_next ? !W : (U <= 0 || !line_u0 || !upos || !wdz)))
    return fail("invalid line_backward arguments");
  if (S == 0) return SBP_NN_OK;
  LineArgs a{};
  a.S = S, a.C = C, a.n = n, a.m = m, a.basis = basis, a.x = x, a.wl = wl, a.bl = bl, a.i1 = i1, a.src = dz_next,
  a.W = W, a.U = U, a.line_u0 = line_u0, a.upos = upos, a.wdz = wdz, a.z_in = z, a.h_in = h, a.z = dz, a.t1 = t1,
  a.gw = gw_part, a.gb = gb_part;
  backward_c<false>(a, (hipStream_t)stream);
  return sbp_nn::status();
}

int sbp_nn_lift_backward(int S, int C, int n, int m, const float* basis, const float* i1, const float* dz0,
                         const float* W, const float* x, const float* wl, const float* bl, double* part, float* gw,
                         float* gb, void* stream) {
  if (!shape_ok(S, C, n, m) || S == 0 || !basis || !i1 || !dz0 || !W || !x || !wl || !bl || !part || !gw || !gb)
    return fail("invalid lift_backward arguments");
  LineArgs a{};
  a.S = S, a.C = C, a.n = n, a.m = m, a.basis = basis, a.x = x, a.wl = wl, a.bl = bl, a.i1 = i1, a.src = dz0, a.W = W,
  a.gb = part;
  const hipStream_t st = (hipStream_t)stream;
  backward_c<true>(a, st);
  hipLaunchKernelGGL(sum_blocks_kernel, dim3(2 * C), dim3(256), 0, st, line_blocks(S, n), 2 * C, C, part, gb, gw);
  return sbp_nn::status();
}

int sbp_nn_line_sums(int S, int C, int n, const float* gw_part, const double* gb_part, float* gw, float* gb,
                     void* stream) {
  if (S <= 0 || C < 1 || C > 64 || n < 4 || n > 64 || !gw_part || !gb_part || !gw || !gb)
    return fail("invalid line_sums arguments");
  const hipStream_t st = (hipStream_t)stream;
  const int nb = line_blocks(S, n);
  const int rc = sbp_nn_sum_rows(nb, C * C, gw_part, gw, 0, stream);
  if (rc) return rc;
  hipLaunchKernelGGL(sum_blocks_kernel, dim3(C), dim3(256), 0, st, nb, C, C, gb_part, gb, (float*)nullptr);
  return sbp_nn::status();
}

int sbp_nn_modes_forward(int SC, int n, int m, const float* basis, float* t1, float* out, void* stream) {
  if (!shape_ok(1, 1, n, m) || SC < 0 || !basis || !t1 || !out) return fail("invalid modes_forward arguments");
  if (SC == 0) return SBP_NN_OK;
  hipLaunchKernelGGL(modes_y_kernel, dim3(SC, (n + 7) / 8), dim3(256), 0, (hipStream_t)stream, n, m, basis, t1);
  hipLaunchKernelGGL(modes_z_kernel, dim3(SC, (m * m + 15) / 16), dim3(64), 0, (hipStream_t)stream, n, m, basis, t1, out);
  return sbp_nn::status();
}

int sbp_nn_modes_inverse(int SC, int n, int m, const float* basis, const float* y, float* i1, void* stream) {
  if (!shape_ok(1, 1, n, m) || SC < 0 || !basis || !y || !i1) return fail("invalid modes_inverse arguments");
  if (SC == 0) return SBP_NN_OK;
  hipLaunchKernelGGL(modes_inverse_kernel, dim3(SC, (n + 15) / 16), dim3(kInvThreads), 0, (hipStream_t)stream, n, m, basis, y,
                     i1);
  return sbp_nn::status();
}

int sbp_nn_receiver_forward(int S, int C, int n, int m, int R, const float* basis, const float* y, const float* h,
                            const float* W, const float* bias, const int* pos, float* f, void* stream) {
  if (!shape_ok(S, C, n, m) || R <= 0 || S > 65535 || !basis || !y || !h || !W || !bias || !pos || !f)
    return fail("invalid receiver_forward arguments");
  if (S == 0) return SBP_NN_OK;
  hipLaunchKernelGGL(receiver_forward_kernel, dim3(R, S, (C + 15) / 16), dim3(64 * kRecWaves), 0, (hipStream_t)stream, C, n, m, R, basis, y,
                     h, W, bias, pos, f);
  return sbp_nn::status();
}

int sbp_nn_receiver_backward(int S, int C, int n, int m, int R, int U, int nlines, const float* basis,
                             const float* df, const float* h, const int* lines, const int* line_u0, const int* upos,
                             const int* u_r0, const int* u_r, float* dzu, float* hu, float* gb, float* t1,
                             void* stream) {
  if (!shape_ok(S, C, n, m) || S == 0 || S > 65535 || R <= 0 || U <= 0 || nlines <= 0 || !basis || !df || !h ||
      !lines || !line_u0 || !upos || !u_r0 || !u_r || !dzu || !hu || !gb || !t1)
    return fail("invalid receiver_backward arguments");
  const hipStream_t st = (hipStream_t)stream;
  const long long n4 = (long long)S * C * n * n * m / 4;  // (n is a multiple of 4)
  hipLaunchKernelGGL(clear_kernel, dim3((unsigned)std::min<long long>((n4 + 255) / 256, 8192)), dim3(256), 0, st, n4,
                     (f32x4*)t1);
  hipLaunchKernelGGL(receiver_backward_kernel, dim3(nlines, S), dim3(64), 0, st, C, n, m, R, U, basis, df, h, lines,
                     line_u0, upos, u_r0, u_r, dzu, hu, t1);
  hipLaunchKernelGGL(column_sum_kernel, dim3(C), dim3(256), 0, st, (long long)S * U, C, dzu, gb);
  return sbp_nn::status();
}

}  // extern "C"
