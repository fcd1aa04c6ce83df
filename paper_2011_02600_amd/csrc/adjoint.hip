// HIP kernels (gfx950) of the discrete adjoint: the transposed operator and
// the misfit gradient with respect to the nodal material.
//
// The transposed semi-discrete operator is built from the forward one.  With
// W the energy weights H J diag(rho I_3, C^{-1}) (per node; H the tensor
// norm), the volume operator L_v satisfies the energy identity of the scheme
// (summation by parts along each axis, H D+ + (H D-)^T = B):
//   W L_v + L_v^T W = Bd,
//   Q^T Bd Q' = sum_xi sum_i [v_i^T B_xi F_xi,i(sigma') + v'_i^T B_xi F_xi,i(sigma)],
// B_xi = +-(norm weights of the two other axes) on the faces xi = 0, 1 and F
// the stress flux with the metric row M_xi.  Hence
//   L^T l = -W L_v(W^{-1} l) + Bd W^{-1} l + P^T l,
// P the face-local penalty blocks.  L_v(W^{-1} l) is one forward
// right-hand-side evaluation with the penalties off (the stage kernel); the
// kernels here apply W^{-1} (pre_node), -W (stage_node) and Bd and P^T
// (face_node, face nodes only).
//
// The material enters the right-hand side pointwise: 1/(rho J) times the
// flux divergence dv, lambda/J and mu/J times the velocity gradient terms,
// and the penalty coefficients of the node's faces.  stage_node takes dv and
// the gradient terms from a forward evaluation with unit material
// (lambda/J = 0, mu/J = 1, 1/(rho J) = 1, penalties off); face_node
// differentiates the penalties.
//
// Everything between two right-hand sides is local to a node: one launch
// (adj_stage_kernel).  It reads and writes 73 words per node and is bound by
// them: 138 us a stage for 129^3 in single precision (the nine passes it replaces
// took 256), 26 for 33^3 in double (was 110), where the chain of the face
// nodes counts.
#include <hip/hip_runtime.h>

#include "adjoint.hpp"

namespace sbp {
namespace {

// (the weight is loaded by every node, also where it is 1: a branch around each
// of the three loads puts their latencies in a row)
template <typename T>
__device__ __forceinline__ T norm_w(const AdjArgs<T>& A, int i, int n) {
  const int e = min(i, n - 1 - i);
  const T w = A.w[min(e, kMaxM - 1)];
  return e < A.m ? w : T(1);
}

struct Node {
  int i, j, k;
  long long o;
};

// (a grid of 2^32 nodes does not fit the memory)
template <typename T>
__device__ __forceinline__ Node node_of(const AdjArgs<T>& A, unsigned n) {
  Node d;
  d.i = (int)(n % A.nq);
  const unsigned t = n / A.nq;
  d.j = (int)(t % A.nr);
  d.k = (int)(t / A.nr);
  d.o = A.nm(d.i, d.j, d.k);
  return d;
}

template <typename T>
__host__ __device__ __forceinline__ unsigned surface_nodes(const AdjArgs<T>& A) {
  return 2u * (unsigned)A.nq * A.nr + 2u * (unsigned)A.nq * (A.ns - 2) + 2u * (unsigned)(A.nr - 2) * (A.ns - 2);
}

// d = a dqb + b qb (dqb: its 9 values), y = W^{-1} d; both stored
template <typename T>
__device__ __forceinline__ void pre_node(const AdjArgs<T>& A, const Node& nd, const T dqb[9], const T qb[9], T lamJ,
                                         T muJ, T rJ) {
  const std::size_t F = A.field;
  const long long o = nd.o;
  T d[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) {
    const T prev = A.a != T(0) ? A.a * dqb[c] : T(0);
    d[c] = prev + A.b * qb[c];
    A.dqb[c * F + o] = d[c];
  }
  const T iH = T(1) / (A.h[0] * norm_w(A, nd.i, A.nq) * A.h[1] * norm_w(A, nd.j, A.nr) * A.h[2] *
                       norm_w(A, nd.k, A.ns));
  // W^{-1}: v / (H rho J), and C / (H J) on the stress (engineering shear)
  const T tr = d[3] + d[4] + d[5];
  T y[9];
  y[0] = rJ * d[0] * iH;
  y[1] = rJ * d[1] * iH;
  y[2] = rJ * d[2] * iH;
  y[3] = (lamJ * tr + T(2) * muJ * d[3]) * iH;
  y[4] = (lamJ * tr + T(2) * muJ * d[4]) * iH;
  y[5] = (lamJ * tr + T(2) * muJ * d[5]) * iH;
  y[6] = muJ * d[6] * iH;
  y[7] = muJ * d[7] * iH;
  y[8] = muJ * d[8] * iH;
#pragma unroll
  for (int c = 0; c < 9; ++c) A.y[c * F + o] = y[c];
}

template <typename T>
__global__ void adj_pre_kernel(const AdjArgs<T> A) {
  const unsigned N = (unsigned)A.nq * A.nr * A.ns;
  const std::size_t F = A.field;
  for (unsigned n = blockIdx.x * blockDim.x + threadIdx.x; n < N; n += gridDim.x * blockDim.x) {
    const Node nd = node_of(A, n);
    const long long o = nd.o;
    T l[9], qb[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) {
      l[c] = A.a != T(0) ? A.dqb[c * F + o] : T(0);
      qb[c] = A.qb[c * F + o];
    }
    pre_node(A, nd, l, qb, A.coef[9 * F + o], A.coef[10 * F + o], A.coef[11 * F + o]);
  }
}

// Face terms of one of the two faces xi at one of its nodes.  With the penalty
// split as in face_penalty,
//   Gn = cv Z_p v_n + ct T_n,   g = cv Z_s (v - v_n n) + ct (T - T_n n),
// and b the vector the stress rows give to l . rate = -kr (Gn n + g) . l_v +
// (Gn / Z_p n + g / Z_s) . b, the transpose P^T l comes from hn = -kr l_v . n +
// b . n / Z_p (against Gn) and h = -kr l_v + b / Z_s (against g), and the
// derivative with respect to each face coefficient is a product of the same
// terms.  qb += dt (Bd y + P^T l); GRAD: grad += dt times the derivative with
// respect to the node's rho, lambda, mu.
template <typename T, bool GRAD>
__device__ __forceinline__ void face_node(const AdjArgs<T>& A, const Node& nd, int xi, bool side, const T l[9],
                                          const T y[9], const T qs[9], T rho, T qb[9], T grad[3]) {
  const std::size_t F = A.field;
  const std::size_t idx = xi == 0 ? (std::size_t)nd.k * A.nr + nd.j
                                  : (xi == 1 ? (std::size_t)nd.k * A.nq + nd.i : (std::size_t)nd.j * A.nq + nd.i);
  const std::size_t off = side ? A.face_off[2 * xi + 1] : A.face_off[2 * xi];
  const T gamma = side ? A.gamma[2 * xi + 1] : A.gamma[2 * xi];
  const bool traction = (side ? A.traction[2 * xi + 1] : A.traction[2 * xi]) != 0;
  const long long o = nd.o;
  T fc[kNumFaceCoef];
#pragma unroll
  for (int kk = 0; kk < kNumFaceCoef; ++kk) fc[kk] = A.face[off + idx + (std::size_t)kk * A.face_n[2 * xi]];
  const T m0 = A.coef[(3 * xi) * F + o], m1 = A.coef[(3 * xi + 1) * F + o], m2 = A.coef[(3 * xi + 2) * F + o];
  const T sgn = side ? T(1) : T(-1);
  const T wq = norm_w(A, nd.i, A.nq), wr = norm_w(A, nd.j, A.nr), ws = norm_w(A, nd.k, A.ns);
  // B_xi: sign times the norm weights of the two other axes
  const T b = sgn * (xi == 0 ? A.h[1] * wr * A.h[2] * ws : (xi == 1 ? A.h[0] * wq * A.h[2] * ws : A.h[0] * wq * A.h[1] * wr));
  T out[9];
  // Bd y: velocity rows take the flux of y_sigma, stress rows the
  // transposed flux map of y_v
  out[0] = b * (m0 * y[3] + m1 * y[6] + m2 * y[7]);
  out[1] = b * (m0 * y[6] + m1 * y[4] + m2 * y[8]);
  out[2] = b * (m0 * y[7] + m1 * y[8] + m2 * y[5]);
  const T z0 = b * y[0], z1 = b * y[1], z2 = b * y[2];
  out[3] = m0 * z0;
  out[4] = m1 * z1;
  out[5] = m2 * z2;
  out[6] = m1 * z0 + m0 * z1;
  out[7] = m2 * z0 + m0 * z2;
  out[8] = m2 * z1 + m1 * z2;

  const T nx = fc[FN_X], ny = fc[FN_Y], nz = fc[FN_Z];
  const T zp = fc[F_ZP], zs = fc[F_ZS], izp = fc[F_IZP], izs = fc[F_IZS], kr = fc[F_KR], kl = fc[F_KL], km = fc[F_KM];
  const T ln = l[0] * nx + l[1] * ny + l[2] * nz;
  // b = -sgn (kl tr(l_sigma) n + km s)
  const T trl = l[3] + l[4] + l[5];
  const T sx = T(2) * l[3] * nx + l[6] * ny + l[7] * nz, sy = l[6] * nx + T(2) * l[4] * ny + l[8] * nz,
          sz = l[7] * nx + l[8] * ny + T(2) * l[5] * nz;
  const T e = -sgn;
  const T bx = e * (kl * trl * nx + km * sx), by = e * (kl * trl * ny + km * sy), bz = e * (kl * trl * nz + km * sz);
  const T bn = bx * nx + by * ny + bz * nz;
  const T cv = traction ? T(0) : T(0.5) * (T(1) - gamma);
  const T ct = T(0.5) * sgn * (T(1) + gamma);
  const T hn = izp * bn - kr * ln;
  const T hx = izs * bx - kr * l[0], hy = izs * by - kr * l[1], hz = izs * bz - kr * l[2];
  const T hhn = hx * nx + hy * ny + hz * nz;
  const T gx = hx - hhn * nx, gy = hy - hhn * ny, gz = hz - hhn * nz;
  // against the traction T = sigma n
  const T tx = traction ? e * kr * l[0] : ct * (hn * nx + gx), ty = traction ? e * kr * l[1] : ct * (hn * ny + gy),
          tz = traction ? e * kr * l[2] : ct * (hn * nz + gz);
  out[0] += cv * (zp * hn * nx + zs * gx);
  out[1] += cv * (zp * hn * ny + zs * gy);
  out[2] += cv * (zp * hn * nz + zs * gz);
  out[3] += tx * nx;
  out[4] += ty * ny;
  out[5] += tz * nz;
  out[6] += tx * ny + ty * nx;
  out[7] += tx * nz + tz * nx;
  out[8] += ty * nz + tz * ny;
#pragma unroll
  for (int c = 0; c < 9; ++c) qb[c] += A.dt * out[c];

  if constexpr (GRAD) {
    const T Tx = qs[3] * nx + qs[6] * ny + qs[7] * nz, Ty = qs[6] * nx + qs[4] * ny + qs[8] * nz,
            Tz = qs[7] * nx + qs[8] * ny + qs[5] * nz;
    const T vn = qs[0] * nx + qs[1] * ny + qs[2] * nz;
    const T Tn = Tx * nx + Ty * ny + Tz * nz;
    const T ux = qs[0] - vn * nx, uy = qs[1] - vn * ny, uz = qs[2] - vn * nz;
    const T Gn = cv * zp * vn + ct * Tn;
    const T gtx = cv * zs * ux + ct * (Tx - Tn * nx), gty = cv * zs * uy + ct * (Ty - Tn * ny),
            gtz = cv * zs * uz + ct * (Tz - Tn * nz);
    const T gn = Gn * izp;
    const T Gx = gn * nx + gtx * izs, Gy = gn * ny + gty * izs, Gz = gn * nz + gtz * izs;
    // derivatives of l . rate with respect to the face coefficients
    const T d_kr = traction ? e * (Tx * l[0] + Ty * l[1] + Tz * l[2])
                            : -(Gn * ln + gtx * l[0] + gty * l[1] + gtz * l[2]);
    T d_zp = cv * vn * hn;
    T d_zs = cv * (ux * hx + uy * hy + uz * hz);
    T d_izp = Gn * bn;
    T d_izs = gtx * bx + gty * by + gtz * bz;
    T d_kl = e * trl * (nx * Gx + ny * Gy + nz * Gz);
    T d_km = e * (sx * Gx + sy * Gy + sz * Gz);
    if (traction) d_zp = d_zs = d_izp = d_izs = d_kl = d_km = T(0);
    // and theirs (Z_p = sqrt(rho (lambda + 2 mu)), Z_s = sqrt(rho mu), the
    // inverses, kappa/rho, kappa lambda, kappa mu) with respect to rho, lambda, mu
    const T kap = kr * rho, hr = T(0.5) / rho;
    const T zp1 = T(0.5) * rho * izp, zs2 = T(0.5) * rho * izs;
    const T p = zp1 * (d_zp - izp * izp * d_izp);
    grad[0] += A.dt * (hr * (zp * d_zp + zs * d_zs - izp * d_izp - izs * d_izs) - kr / rho * d_kr);
    grad[1] += A.dt * (p + kap * d_kl);
    grad[2] += A.dt * (T(2) * p + zs2 * (d_zs - izs * izs * d_izs) + kap * d_km);
  }
}

// One node between two right-hand sides of the reverse sweep: -W r and the
// face terms into qb, GRAD: the gradient terms into grad, PRE: d and y of the
// next stage.
template <typename T, bool GRAD, bool PRE, bool FACE>
__device__ __forceinline__ void stage_node(const AdjArgs<T>& A, const Node& nd) {
  const std::size_t F = A.field;
  const long long o = nd.o;
  T r[9], l[9], ru[9], qb[9], grad[3];
#pragma unroll
  for (int c = 0; c < 9; ++c) {
    r[c] = A.r[c * F + o];
    qb[c] = A.qb[c * F + o];
    if constexpr (GRAD || PRE || FACE) l[c] = A.dqb[c * F + o];
    if constexpr (GRAD) ru[c] = A.ru[c * F + o];
  }
  const T lamJ = A.coef[9 * F + o], muJ = A.coef[10 * F + o], rJ = A.coef[11 * F + o];
  T J;
  if constexpr (GRAD) {
    J = A.jac[o];
#pragma unroll
    for (int p = 0; p < 3; ++p) grad[p] = A.grad[p * F + o];
  }
  {
    const T wq = norm_w(A, nd.i, A.nq), wr = norm_w(A, nd.j, A.nr), ws = norm_w(A, nd.k, A.ns);
    const T Hn = A.h[0] * wq * A.h[1] * wr * A.h[2] * ws;
    T out[9];
    // -W r: -H rho J r_v and -H J C^{-1} r_sigma
    const T hv = -Hn / rJ, im = T(1) / muJ, hs = -Hn * im;
    out[0] = hv * r[0];
    out[1] = hv * r[1];
    out[2] = hv * r[2];
    const T trr = r[3] + r[4] + r[5];
    const T cl = lamJ / (T(3) * lamJ + T(2) * muJ);
    const T h2 = T(0.5) * hs;
    out[3] = h2 * (r[3] - cl * trr);
    out[4] = h2 * (r[4] - cl * trr);
    out[5] = h2 * (r[5] - cl * trr);
    out[6] = hs * r[6];
    out[7] = hs * r[7];
    out[8] = hs * r[8];
#pragma unroll
    for (int c = 0; c < 9; ++c) qb[c] += A.dt * out[c];
  }
  if constexpr (GRAD) {
    const T iJ = T(1) / J;
    // volume terms: d(1/(rho J))/d rho = -rJ^2 J, d(lambda/J)/d lambda = d(mu/J)/d mu = 1/J
    const T g0 = -rJ * rJ * J * (l[0] * ru[0] + l[1] * ru[1] + l[2] * ru[2]);
    const T div = T(0.5) * (ru[3] + ru[4] + ru[5]);
    const T g1 = iJ * div * (l[3] + l[4] + l[5]);
    const T g2 = iJ * (l[3] * ru[3] + l[4] * ru[4] + l[5] * ru[5] + l[6] * ru[6] + l[7] * ru[7] + l[8] * ru[8]);
    grad[0] += A.dt * g0;
    grad[1] += A.dt * g1;
    grad[2] += A.dt * g2;
  }
  if constexpr (FACE) {
    T y[9], qs[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) {
      y[c] = A.y[c * F + o];
      if constexpr (GRAD) qs[c] = A.qs[c * F + o];
    }
    T rho = T(0);
    if constexpr (GRAD) rho = T(1) / (rJ * J);
    if (nd.i == 0 || nd.i == A.nq - 1) face_node<T, GRAD>(A, nd, 0, nd.i != 0, l, y, qs, rho, qb, grad);
    if (nd.j == 0 || nd.j == A.nr - 1) face_node<T, GRAD>(A, nd, 1, nd.j != 0, l, y, qs, rho, qb, grad);
    if (nd.k == 0 || nd.k == A.ns - 1) face_node<T, GRAD>(A, nd, 2, nd.k != 0, l, y, qs, rho, qb, grad);
  }
#pragma unroll
  for (int c = 0; c < 9; ++c) A.qb[c * F + o] = qb[c];
  if constexpr (GRAD) {
#pragma unroll
    for (int p = 0; p < 3; ++p) A.grad[p * F + o] = grad[p];
  }
  if constexpr (PRE) pre_node(A, nd, l, qb, lamJ, muJ, rJ);
}

// Node t of the block's surface: s faces, then the rest of the r faces, then
// the rest of the q faces
template <typename T>
__device__ __forceinline__ Node face_node_of(const AdjArgs<T>& A, unsigned t) {
  const unsigned nq = A.nq, nr = A.nr, ns = A.ns;
  Node d;
  if (t < 2 * nq * nr) {
    d.i = t % nq;
    const unsigned u = t / nq;
    d.j = u % nr;
    d.k = u >= nr ? ns - 1 : 0;
  } else if ((t -= 2 * nq * nr) < 2 * nq * (ns - 2)) {
    d.i = t % nq;
    const unsigned u = t / nq;
    d.k = 1 + u % (ns - 2);
    d.j = u >= ns - 2 ? nr - 1 : 0;
  } else {
    t -= 2 * nq * (ns - 2);
    d.j = 1 + t % (nr - 2);
    const unsigned u = t / (nr - 2);
    d.k = 1 + u % (ns - 2);
    d.i = u >= ns - 2 ? nq - 1 : 0;
  }
  d.o = A.nm(d.i, d.j, d.k);
  return d;
}

// stage_node of every node: the first fb blocks take the surface (its
// penalties are long chains on few nodes, so they start first), the rest the
// interior.
template <typename T, bool GRAD, bool PRE>
__global__ __launch_bounds__(256) void adj_stage_kernel(const AdjArgs<T> A, int fb) {
  if ((int)blockIdx.x < fb) {
    const unsigned t = blockIdx.x * 256 + threadIdx.x;
    if (t < surface_nodes(A)) stage_node<T, GRAD, PRE, true>(A, face_node_of(A, t));
    return;
  }
  const unsigned N = (unsigned)A.nq * A.nr * A.ns;
  for (unsigned n = (blockIdx.x - fb) * 256 + threadIdx.x; n < N; n += (gridDim.x - fb) * 256) {
    const Node nd = node_of(A, n);
    if (nd.i > 0 && nd.i < A.nq - 1 && nd.j > 0 && nd.j < A.nr - 1 && nd.k > 0 && nd.k < A.ns - 1)
      stage_node<T, GRAD, PRE, false>(A, nd);
  }
}

template <typename T>
__global__ void adj_inject_kernel(T* qb, std::size_t field, const long long* off, int nrec, const T* res) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nrec) return;
  const long long o = off[r];
#pragma unroll
  for (int c = 0; c < 3; ++c) atomicAdd(qb + c * field + o, res[3 * r + c]);
}

template <typename T>
__global__ void fill_kernel(T* dst, std::size_t n, T v) {
  for (std::size_t e = blockIdx.x * (std::size_t)blockDim.x + threadIdx.x; e < n; e += (std::size_t)gridDim.x * blockDim.x)
    dst[e] = v;
}

template <typename T>
int node_blocks(const AdjArgs<T>& a) {
  const long long N = (long long)a.nq * a.nr * a.ns;
  return (int)std::min<long long>((N + 255) / 256, 1 << 16);
}

}  // namespace

template <typename T>
hipError_t launch_adj_pre(const AdjArgs<T>& a, hipStream_t st) {
  hipLaunchKernelGGL(adj_pre_kernel<T>, dim3(node_blocks(a)), dim3(256), 0, st, a);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_adj_stage(const AdjArgs<T>& a, bool grad, bool pre, hipStream_t st) {
  const int fb = (int)((surface_nodes(a) + 255) / 256);
  const dim3 nb(fb + node_blocks(a)), tb(256);
  if (!grad)
    hipLaunchKernelGGL((adj_stage_kernel<T, false, false>), nb, tb, 0, st, a, fb);
  else if (pre)
    hipLaunchKernelGGL((adj_stage_kernel<T, true, true>), nb, tb, 0, st, a, fb);
  else
    hipLaunchKernelGGL((adj_stage_kernel<T, true, false>), nb, tb, 0, st, a, fb);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_adj_inject(T* qb, std::size_t field, const long long* off, int nrec, const T* res,
                             hipStream_t st) {
  if (nrec <= 0) return hipSuccess;
  hipLaunchKernelGGL(adj_inject_kernel<T>, dim3((nrec + 255) / 256), dim3(256), 0, st, qb, field, off, nrec, res);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_fill(T* dst, std::size_t n, T v, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const int nb = (int)std::min<std::size_t>((n + 255) / 256, 1 << 16);
  hipLaunchKernelGGL(fill_kernel<T>, dim3(nb), dim3(256), 0, st, dst, n, v);
  return hipGetLastError();
}

template hipError_t launch_adj_pre<float>(const AdjArgs<float>&, hipStream_t);
template hipError_t launch_adj_pre<double>(const AdjArgs<double>&, hipStream_t);
template hipError_t launch_adj_stage<float>(const AdjArgs<float>&, bool, bool, hipStream_t);
template hipError_t launch_adj_stage<double>(const AdjArgs<double>&, bool, bool, hipStream_t);
template hipError_t launch_adj_inject<float>(float*, std::size_t, const long long*, int, const float*, hipStream_t);
template hipError_t launch_adj_inject<double>(double*, std::size_t, const long long*, int, const double*,
                                              hipStream_t);
template hipError_t launch_fill<float>(float*, std::size_t, float, hipStream_t);
template hipError_t launch_fill<double>(double*, std::size_t, double, hipStream_t);

}  // namespace sbp
