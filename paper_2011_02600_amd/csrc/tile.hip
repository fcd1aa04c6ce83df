// The tile stage kernel (gfx950): one launch per Runge-Kutta stage that
// computes every node of a grid -- derivatives, rates, boundary penalties,
// point sources and the stage update.  It serves the grids whose fields the
// 256 MB memory-side cache holds (use_tile in api.cpp), where the stage
// kernel's march along s is bound by its chain of planes: there the time of a
// stage is the time of a block, and a block here has one chain of loads,
// one barrier and one chain of derivatives.
//
// A block of 256 threads owns 32 (q) x 8 (r) nodes of one plane (33 x 7 in the
// last tile of axes of 32 k + 1 points), a thread one node.  The block issues
// all loads of the tile before it uses the first: its nodes' v, sigma and
// metric rows, the r and q halos (spread over the threads), and the planes
// below and above, each thread its own node's.  v, F_q and F_r go to LDS; the
// s derivatives are summed in registers.  After the barrier the q and r
// derivatives come from LDS.  Reading the planes around a node once per node
// costs 7 reads of v, sigma and M_s where tiles of 4 planes would take 2.5;
// they come from L1 and L2, and tiles of 2 and 4 planes measured no faster up
// to 10^6 nodes (more registers, fewer blocks in flight).
//
// Order 6, us per stage with its edge, penalty and source launches before
// (march) and now: single precision 65^3 82 -> 24, 97^3 95 -> 55; order 4 in
// double precision 21^3 124 -> 12.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.hpp"
#include "kernels.hpp"
#include "penalty.hpp"
#include "stencil.hpp"
#include "tile.hpp"

namespace sbp {

namespace {

template <typename T, int ORDER>
struct TileLds {
  using S = Stencil<ORDER>;
  static constexpr int R = S::R, Q = S::Q, M = S::M, NC = M + Q, H = Q;
  static constexpr int PX = kTileW + 2 * H;  // pitch of the v and F_q rows
  static constexpr int RX = kTileW;          // pitch of the F_r rows
  static constexpr int ROWS = kTileH + Q + R;
  // weight rows (interior, left closure rows, right closure rows) over
  // ascending columns, each after M zeros; D+ rows, then D- rows
  static constexpr int WR = 2 * M + 1, WL = M + NC;
  static constexpr int n_w = 2 * WR * WL;
  // the three components of a row lie one after the other
  static constexpr int o_v = n_w, o_q = o_v + ROWS * 3 * PX, o_r = o_q + kTileH * 3 * PX,
                       total = o_r + ROWS * 3 * RX;
  static constexpr std::size_t bytes = total * sizeof(T);
};

// a point's v, sigma and one metric row
template <typename T>
struct TilePoint {
  T v[3], s[6], m[3];
};

// MODE 0: Runge-Kutta stage; 1: the right-hand side into dq
template <typename T, int ORDER, int MODE>
__device__ __forceinline__ void tile_body(const TileArgs<T>& A, const int tile, char* lds) {
  using S = Stencil<ORDER>;
  using L = TileLds<T, ORDER>;
  using P = TilePoint<T>;
  constexpr int R = S::R, Q = S::Q, M = S::M, QD = R + Q + 1, NC = L::NC, H = Q;
  constexpr int PX = L::PX, RX = L::RX, WL = L::WL, WR = L::WR, NT = kTileNT;
  static_assert(kTileH * 2 * H <= NT && NT / 32 == kTileH && 2 * Q <= 2 * kTileH, "halo points per thread");
  const TileShape& G = A.tile;
  if (tile >= G.ntiles) return;
  const int nq = A.nq, nr = A.nr, ns = A.ns;
  // (read here, before the barrier, where arguments in memory are scalar loads)
  const T ihq = A.inv_h[0], ihr = A.inv_h[1], ihs = A.inv_h[2], dt = A.dt, Ak = A.Ak, Bk = A.Bk;
  const int sat = A.sat, nsrc = A.nsrc, read_dq = A.read_dq, ey = A.ey;
  // tile order: q fastest, then s, then r
  const int xt = tile % G.q.T, ks = tile / G.q.T;
  const int k = ks % ns, yt = ks / ns;
  const int x0 = G.q.start(xt), x1 = G.q.start(xt + 1);
  const int y0 = G.r.start(yt), y1 = G.r.start(yt + 1);
  if (G.part == 2 && x1 < nq && y1 <= nr - ey) return;
  const int w = x1 - x0, h = y1 - y0;
  const bool yfirst = y0 == 0, ylast = y1 == nr;

  // thread -> row tid / 32, column tid % 32: a quarter wave reads one aligned
  // 64-byte piece of a row (33 lanes per row took three times the L1
  // accesses).  In a tile of 33 columns the rows end at thread 224 and the
  // next ones take column 32
  const int tid = threadIdx.x;
  const bool wide = w > 32;
  const int hx = tid & 31, hy = tid >> 5;
  const bool xtra = wide && tid >= 224;
  const int ty = xtra ? hx : hy, tx = xtra ? 32 : hx;
  const bool own = tx < w && ty < h;
  const unsigned px = A.px, plane = A.plane;
  const unsigned nqm = A.nm.nqm, cbase = (unsigned)A.nm.cbase;
  const std::size_t field = A.field;
  const Arr<T, true> gq(A.qin, field), gc(A.coef, field), gd(A.dq, field), go(A.qout, field);
  auto at = [&](int i, int j) -> unsigned {  // a node of plane k
    return (unsigned)i < nqm ? (unsigned)k * plane + (unsigned)j * px + (unsigned)i
                             : cbase + (unsigned)k * (unsigned)nr + (unsigned)j;
  };
  auto load = [&](unsigned ov, unsigned of, int row, P& p) {  // v at ov, sigma and metric row `row` at of
#pragma unroll
    for (int c = 0; c < 3; ++c) p.v[c] = gq.ld(c, ov);
#pragma unroll
    for (int c = 0; c < 6; ++c) p.s[c] = gq.ld(3 + c, of);
#pragma unroll
    for (int c = 0; c < 3; ++c) p.m[c] = gc.ld(3 * row + c, of);
  };
  auto flux = [](const P& p, T f[3]) {
    flux3(p.m[0], p.m[1], p.m[2], p.s[0], p.s[1], p.s[2], p.s[3], p.s[4], p.s[5], f);
  };
  T* const lw = reinterpret_cast<T*>(lds);
  T* const lv0 = lw + L::o_v;
  T* const lq0 = lw + L::o_q;
  T* const lr0 = lw + L::o_r;

  // ---- loads: the own node (lanes without one read the tile's first), the
  // weight rows, the halos
  const int i = x0 + (own ? tx : 0), j = y0 + (own ? ty : 0);
  const unsigned os = (unsigned)i < nqm ? plane : (unsigned)nr;  // s step of the column
  const unsigned o = at(i, j);
  P me;  // (with M_s)
  T mq[3], mr[3];
  load(o, o, 2, me);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    mq[c] = gc.ld(c, o);
    mr[c] = gc.ld(3 + c, o);
  }
  constexpr int NWP = (L::n_w + NT - 1) / NT;
  T wv[NWP];
#pragma unroll
  for (int p = 0; p < NWP; ++p) wv[p] = A.tw[min(tid + p * NT, L::n_w - 1)];

  // r halo: rows y0-Q .. y0-1 and y1 .. y1+Q-1, row y0-Q+u or y1+u-Q for
  // u = tid / 32 + 8 p.  v is read R rows below and Q above, the flux Q below
  // and R above (both Q in the tiles that hold closure rows)
  const int vlo = yfirst ? 0 : (ylast ? y0 - Q : y0 - R), vhi = ylast ? nr : y1 + Q;
  const int flo = yfirst ? 0 : y0 - Q, fhi = ylast ? nr : (yfirst ? y1 + Q : y1 + R);
  struct RHalo {
    P p;
    int x, y;
    bool nv, nf;
  };
  auto rload = [&](int u, int x, RHalo& r) {
    r.y = u < Q ? y0 - Q + u : y1 + u - Q;
    r.x = x;
    const bool in = u < 2 * Q && x < w;
    r.nv = in && r.y >= vlo && r.y < vhi;
    r.nf = in && r.y >= flo && r.y < fhi;
    const unsigned oh = at(x0 + min(x, w - 1), min(max(r.y, 0), nr - 1));
    load(r.nv ? oh : o, r.nf ? oh : o, 1, r.p);
  };
  auto rstore = [&](const RHalo& r) {
    if (r.nv) {
#pragma unroll
      for (int c = 0; c < 3; ++c) lv0[((r.y - vlo) * 3 + c) * PX + r.x + H] = r.p.v[c];
    }
    if (r.nf) {
      T f[3];
      flux(r.p, f);
#pragma unroll
      for (int c = 0; c < 3; ++c) lr0[((r.y - flo) * 3 + c) * RX + r.x] = f[c];
    }
  };
  constexpr int NP = (2 * Q + kTileH - 1) / kTileH;
  RHalo rh[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) rload(hy + kTileH * p, hx, rh[p]);

  // q halo: H columns on either side of the tile's rows, a point per thread
  const int qrow_ = tid / (2 * H), qc = tid - qrow_ * (2 * H);
  const int qx = qc < H ? x0 - H + qc : x1 + qc - H;
  const bool qin = qrow_ < h && qx >= 0 && qx < nq;
  const unsigned oqh = qin ? at(qx, y0 + qrow_) : o;
  P qh;
  load(oqh, oqh, 0, qh);

  if (wide) {  // column 32 of the r halo
    RHalo r;
    rload(tid, 32, r);
    rstore(r);
  }

  // planes below and above (nodes with an interior s row)
  const bool sint = k >= M && k < ns - M;
  T us[3] = {T(0), T(0), T(0)}, fs[3] = {T(0), T(0), T(0)};
  // plane t of them: v at k + dv, the flux at k + df
  constexpr int NS = Q + R;
  auto off_v = [](int t) { return t < R ? t - R : t - R + 1; };
  auto off_f = [](int t) { return t < Q ? t - Q : t - Q + 1; };
  auto ssum = [&](int t, const P& p) {
    T f[3];
    flux(p, f);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      us[c] += T(S::a[R + off_v(t)]) * p.v[c];
      fs[c] -= T(S::a[R - off_f(t)]) * f[c];
    }
  };
  auto stage_lds = [&]() {
    if (own) {
      T f[3];
      P t = me;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        lv0[((j - vlo) * 3 + c) * PX + tx + H] = me.v[c];
        t.m[c] = mq[c];
      }
      flux(t, f);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        lq0[(ty * 3 + c) * PX + tx + H] = f[c];
        t.m[c] = mr[c];
      }
      flux(t, f);
#pragma unroll
      for (int c = 0; c < 3; ++c) lr0[((j - flo) * 3 + c) * RX + tx] = f[c];
    }
#pragma unroll
    for (int p = 0; p < NWP; ++p)
      if (tid + p * NT < L::n_w) lw[tid + p * NT] = wv[p];
#pragma unroll
    for (int p = 0; p < NP; ++p) rstore(rh[p]);
    if (qin) {
      T f[3];
      flux(qh, f);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        lv0[((y0 + qrow_ - vlo) * 3 + c) * PX + qx - x0 + H] = qh.v[c];
        lq0[(qrow_ * 3 + c) * PX + qx - x0 + H] = f[c];
      }
    }
  };
  if (sint) {
    // single precision: the planes' loads go out with the halos'; in double
    // precision their values do not fit beside the halos' and come in groups
    constexpr int G0 = sizeof(T) == 4 || NS < 3 ? NS : (ORDER < 6 ? 3 : 2);
    P sp[G0];
    auto sload = [&](int t0) {
#pragma unroll
      for (int t = 0; t < G0; ++t)
        if (t0 + t < NS)
          load(o + (unsigned)off_v(t0 + t) * os, o + (unsigned)off_f(t0 + t) * os, 2, sp[t]);
    };
    if constexpr (G0 == NS) sload(0);
    __builtin_amdgcn_sched_barrier(0);
    stage_lds();
    T f[3];
    flux(me, f);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      us[c] = T(S::a[R]) * me.v[c];
      fs[c] = -T(S::a[R]) * f[c];
    }
#pragma unroll
    for (int t0 = 0; t0 < NS; t0 += G0) {
      if constexpr (G0 < NS) {
        __builtin_amdgcn_sched_barrier(0);
        sload(t0);
      }
#pragma unroll
      for (int t = 0; t < G0; ++t)
        if (t0 + t < NS) ssum(t0 + t, sp[t]);
    }
    __syncthreads();
  } else {
    stage_lds();
    __syncthreads();
    // closure row: its NC planes, weights from the table
    const int row = k < M ? 1 + k : 1 + M + (ns - 1 - k);
    const unsigned op = o + (unsigned)((k < M ? 0 : ns - NC) - k) * os;
    constexpr int KU = sizeof(T) == 4 ? (NC + 1) / 2 : (ORDER < 6 ? 3 : 2);  // planes loaded together
#pragma unroll 1
    for (int t0 = 0; t0 < NC; t0 += KU) {
      P p[KU];
#pragma unroll
      for (int u = 0; u < KU; ++u) {
        const unsigned oo = op + (unsigned)min(t0 + u, NC - 1) * os;
        load(oo, oo, 2, p[u]);
      }
#pragma unroll
      for (int u = 0; u < KU; ++u) {
        const int t = t0 + u;
        // (past the row's end: the zero before its first weight)
        const T cv = lw[row * WL + (t < NC ? M + t : 0)], cf = lw[(WR + row) * WL + (t < NC ? M + t : 0)];
        T f[3];
        flux(p[u], f);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          us[c] += cv * p[u].v[c];
          fs[c] += cf * f[c];
        }
      }
    }
  }
  const bool act = G.part == 0 || (((unsigned)i < nqm && j < nr - ey) == (G.part == 1));
  if (!own || !act) return;

  // ---- what the update needs (double precision, orders 6 to 8: loaded where
  // it is used, the registers are not there)
  constexpr bool LATE = sizeof(T) == 8 && ORDER >= 6;
  T mat[3], dqo[9];
  auto uload = [&]() {
#pragma unroll
    for (int c = 0; c < 3; ++c) mat[c] = gc.ld(9 + c, o);
    if constexpr (MODE == 0) {
      const unsigned od = read_dq ? o : 0u;
#pragma unroll
      for (int c = 0; c < 9; ++c) dqo[c] = gd.ld(c, od);
    }
  };
  if constexpr (!LATE) uload();

  // ---- q derivatives: NC taps with the lane's own weight row (interior rows
  // padded with zeros), from its first column, or from further down, behind
  // zero weights, where the taps would leave the window
  const T* const lv = lv0 + (j - vlo) * 3 * PX + tx + H;
  T u[3][3], dv[3];
  constexpr bool WREG = sizeof(T) == 4;  // weights in registers, else read from LDS per tap
  {
    const int row = i < M ? 1 + i : (i >= nq - M ? 1 + M + (nq - 1 - i) : 0);
    const int whi = min(nq, x1 + H);
    const int sv = row == 0 ? i - R : (i < M ? 0 : nq - NC), sf = row == 0 ? i - Q : sv;
    const int ev = max(0, sv + NC - whi), ef = max(0, sf + NC - whi);
    const T* const wp = lw + row * WL + M - ev;
    const T* const wm = lw + (WR + row) * WL + M - ef;
    const T* const tv = lv + (sv - ev - i);
    const T* const tf = lq0 + ty * 3 * PX + tx + H + (sf - ef - i);
    T cp[WREG ? NC : 1], cm[WREG ? NC : 1];
    if constexpr (WREG) {
#pragma unroll
      for (int t = 0; t < NC; ++t) {
        cp[t] = wp[t];
        cm[t] = wm[t];
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      T sp = T(0), sm = T(0);
#pragma unroll
      for (int t = 0; t < NC; ++t) {
        sp += (WREG ? cp[WREG ? t : 0] : wp[t]) * tv[c * PX + t];
        sm += (WREG ? cm[WREG ? t : 0] : wm[t]) * tf[c * PX + t];
      }
      u[0][c] = sp * ihq;
      dv[c] = sm * ihq;
      sched_fence<T>();
    }
  }
  // ---- r derivatives: the interior stencil, or in tiles that hold closure
  // rows the lane's weight row as along q
  {
    const T* const lr = lr0 + (j - flo) * 3 * RX + tx;
    if (!yfirst && !ylast) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        T sp = T(0), sm = T(0);
#pragma unroll
        for (int s = 0; s < QD; ++s) {
          sp += T(S::a[s]) * lv[((s - R) * 3 + c) * PX];
          sm += T(S::a[s]) * lr[((R - s) * 3 + c) * RX];
        }
        u[1][c] = sp * ihr;
        dv[c] -= sm * ihr;
        sched_fence<T>();
      }
    } else {
      const int row = j < M ? 1 + j : (j >= nr - M ? 1 + M + (nr - 1 - j) : 0);
      const int sv = row == 0 ? j - R : (j < M ? 0 : nr - NC), sf = row == 0 ? j - Q : sv;
      const int ev = max(0, sv + NC - vhi), ef = max(0, sf + NC - fhi);
      const T* const wp = lw + row * WL + M - ev;
      const T* const wm = lw + (WR + row) * WL + M - ef;
      const T* const tv = lv + (sv - ev - j) * 3 * PX;
      const T* const tf = lr + (sf - ef - j) * 3 * RX;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        T sp = T(0), sm = T(0);
#pragma unroll
        for (int t = 0; t < NC; ++t) {
          sp += wp[t] * tv[(t * 3 + c) * PX];
          sm += wm[t] * tf[(t * 3 + c) * RX];
        }
        u[1][c] = sp * ihr;
        dv[c] += sm * ihr;
        sched_fence<T>();
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      u[2][c] = us[c] * ihs;
      dv[c] += fs[c] * ihs;
    }
  }

  if constexpr (LATE) uload();
  T rate[9];
  node_rates(u, dv, mq, mr, me.m, mat[0], mat[1], mat[2], rate);
  // the penalties of the node's faces (one per axis at most)
  auto face = [&](int ax, bool hi, std::size_t idx) {
    const std::size_t f0 = A.face_off[2 * ax], f1 = A.face_off[2 * ax + 1];
    const T* p = A.face + (hi ? f1 : f0) + idx;
    const std::size_t n = A.face_n[2 * ax];
    T fc[kNumFaceCoef];
#pragma unroll
    for (int c = 0; c < kNumFaceCoef; ++c) fc[c] = p[c * n];
    const T g0 = A.gamma[2 * ax], g1 = A.gamma[2 * ax + 1], g = hi ? g1 : g0;
    const int t0 = A.traction[2 * ax], t1 = A.traction[2 * ax + 1];
    const bool tr = (hi ? t1 : t0) != 0;
    face_penalty(fc, g, hi ? T(1) : T(-1), tr, me.v, me.s, rate);
  };
  if (sat) {
    if (i == 0 || i == nq - 1) face(0, i != 0, (std::size_t)k * nr + j);
    if (j == 0 || j == nr - 1) face(1, j != 0, (std::size_t)k * nq + i);
    if (k == 0 || k == ns - 1) face(2, k != 0, (std::size_t)j * nq + i);
  }
  T sadd[6] = {T(0), T(0), T(0), T(0), T(0), T(0)};
  if (nsrc > 0) source_add(A, i, j, k, sadd, A.src_stride, A.src_off);
#pragma unroll
  for (int c = 0; c < 9; ++c) {
    T d = dt * rate[c];
    if constexpr (MODE == 0) d += Ak * (read_dq ? dqo[c] : T(0));
    if (c >= 3) d += sadd[c >= 3 ? c - 3 : 0];
    // (kept in the caches: the next stage reads them)
    gd.template stp<0>(c, o, d);
    if constexpr (MODE == 0) go.template stp<0>(c, o, (c < 3 ? me.v[c < 3 ? c : 0] : me.s[c < 3 ? 0 : c - 3]) + Bk * d);
  }
}

template <typename T, int ORDER, int MODE>
__global__ __launch_bounds__(kTileNT, sizeof(T) == 4 && ORDER <= 6 ? 3 : 2) void tile_kernel(const TileArgs<T> A) {
  __shared__ __align__(16) char lds[TileLds<T, ORDER>::bytes];
  // consecutive tiles on the same XCD
  const int per = gridDim.x >> 3;
  tile_body<T, ORDER, MODE>(A, (blockIdx.x & 7) * per + (blockIdx.x >> 3), lds);
}

// the tiles of several grids (a Runge-Kutta stage)
template <typename T, int ORDER>
__global__ __launch_bounds__(kTileNT, sizeof(T) == 4 && ORDER <= 6 ? 3 : 2) void tile_kernel_batch(
    const BatchArgs<T, TileArgs<T>> B) {
  __shared__ __align__(16) char lds[TileLds<T, ORDER>::bytes];
  const int per = gridDim.x >> 3;
  const int item = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (item >= B.total) return;
  const int g = batch_find(B.first, B.n, item);
  const TileArgs<T>& A = B.args[g];
  tile_body<T, ORDER, 0>(A, item - B.first[g], lds);
}

template <typename T, int ORDER>
hipError_t launch_bt(const BatchArgs<T, TileArgs<T>>& b, hipStream_t st) {
  hipLaunchKernelGGL((tile_kernel_batch<T, ORDER>), dim3((b.total + 7) / 8 * 8), dim3(kTileNT), 0, st, b);
  return hipGetLastError();
}

template <typename T, int ORDER>
hipError_t launch_t(int mode, const TileArgs<T>& a, hipStream_t st) {
  const int nb = (a.tile.ntiles + 7) / 8 * 8;
  if (mode == 0)
    hipLaunchKernelGGL((tile_kernel<T, ORDER, 0>), dim3(nb), dim3(kTileNT), 0, st, a);
  else
    hipLaunchKernelGGL((tile_kernel<T, ORDER, 1>), dim3(nb), dim3(kTileNT), 0, st, a);
  return hipGetLastError();
}

template <typename T, int ORDER>
std::size_t scratch_t() {
  std::size_t m = 0;
  const void* fns[] = {reinterpret_cast<const void*>(&tile_kernel<T, ORDER, 0>),
                       reinterpret_cast<const void*>(&tile_kernel<T, ORDER, 1>),
                       reinterpret_cast<const void*>(&tile_kernel_batch<T, ORDER>)};
  for (const void* f : fns) {
    hipFuncAttributes at{};
    if (hipFuncGetAttributes(&at, f) != hipSuccess) return (std::size_t)-1;
    m = at.localSizeBytes > m ? at.localSizeBytes : m;
  }
  return m;
}

}  // namespace

template <typename T>
hipError_t launch_tile(int order, int mode, const TileArgs<T>& a, hipStream_t st) {
  switch (order) {
    case 2: return launch_t<T, 2>(mode, a, st);
    case 3: return launch_t<T, 3>(mode, a, st);
    case 4: return launch_t<T, 4>(mode, a, st);
    case 5: return launch_t<T, 5>(mode, a, st);
    case 6: return launch_t<T, 6>(mode, a, st);
    case 7: return launch_t<T, 7>(mode, a, st);
    case 8: return launch_t<T, 8>(mode, a, st);
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_tile_batch(int order, const BatchArgs<T, TileArgs<T>>& b, hipStream_t st) {
  switch (order) {
    case 2: return launch_bt<T, 2>(b, st);
    case 3: return launch_bt<T, 3>(b, st);
    case 4: return launch_bt<T, 4>(b, st);
    case 5: return launch_bt<T, 5>(b, st);
    case 6: return launch_bt<T, 6>(b, st);
    case 7: return launch_bt<T, 7>(b, st);
    case 8: return launch_bt<T, 8>(b, st);
  }
  return hipErrorInvalidValue;
}

template <typename T>
std::size_t tile_scratch(int order) {
  switch (order) {
    case 2: return scratch_t<T, 2>();
    case 3: return scratch_t<T, 3>();
    case 4: return scratch_t<T, 4>();
    case 5: return scratch_t<T, 5>();
    case 6: return scratch_t<T, 6>();
    case 7: return scratch_t<T, 7>();
    case 8: return scratch_t<T, 8>();
  }
  return (std::size_t)-1;
}

#ifdef SBP_TILE_F64
template hipError_t launch_tile<double>(int, int, const TileArgs<double>&, hipStream_t);
template hipError_t launch_tile_batch<double>(int, const BatchArgs<double, TileArgs<double>>&, hipStream_t);
template std::size_t tile_scratch<double>(int);
#else
template hipError_t launch_tile<float>(int, int, const TileArgs<float>&, hipStream_t);
template hipError_t launch_tile_batch<float>(int, const BatchArgs<float, TileArgs<float>>&, hipStream_t);
template std::size_t tile_scratch<float>(int);
#endif

}  // namespace sbp
