// sgn_vjp.hpp -- vector-Jacobian product of the split-form right-hand side
// (discrete adjoint of eq. (sd_periodic_2D_SGN) / eq. (semi_2D)) and of the
// classical RK4 stages.
//
// The rates at a node c are sums over the neighbours m that its difference
// operators name,
//   a(c) . k(c) = sum_m w(c, m) G(c; m) + (terms of c alone),
// with w = +-1/(2d) on interior and periodic rows and +-1/d on a reflecting closure
// row, where c itself is one of the two (AxisStencil).  The cotangent of node d
// gathers, for each neighbour m, the derivative of G(d; m) by d's values as the
// centre and the derivative of G(m; d) by d's values as the neighbour, the latter
// with the transposed weight (AxisTranspose); on a closure row m may be d.  G is
// the printed split form term by term (n the velocity along the axis, t the one
// across, r = eta/h - 1, an = a_n/h and so on for t and w):
//   G(c; m) = -ah (n h_m + h n_m) - ae n (eta_m + 3/2 b_m)
//     - an/2 [2g h_m (h_m + b_m - h - b) + h n_m^2 - n^2 h_m + n h_m n_m - h n n_m
//             + lam/3 ((1 + r)^2 h_m - eta_m^2/h_m) - 2 lam/3 r eta_m - lam r b_m]
//     - at/2 [h_m n_m t_m - n t h_m + h n t_m - h t n_m] - aw/2 [the same with w]
// so that its derivatives share their factors: with Q = h n + h_m n_m and the
// differences of the two neighbours' values, a node takes about 330 operations;
// forming the cotangents of the 24 derivative values of every neighbour first and
// chaining them back took 700.  The pair kernels were bound by that arithmetic,
// then by waiting on the sums they wrote between their two evaluations: 1500 x 900
// FP32 with walls 81 and 78 us, with this form 63 and 62, with the sums in
// registers 54 and 52 (28 and 33 values a node: 2.8 and 3.4 TB/s).  Differences of
// seeds and of r are formed before they are scaled by lambda: in FP32 the reverse
// step's error against 64 bits fell from 7e-6 to 5e-7.
// No value crosses threads except through LDS.
#pragma once

#include "sgn_fused.hpp"
#include "sgn_stage.hpp"

namespace sgn {

// Reverse-mode stage roles.  Cotangent of the step output: Qb.
//   PLAIN: kb = Kin;           out = Ybar (5 planes), bout = bbar      (rhs VJP)
//   S4:    kb = a * Qb;        Kout = cq Qb + cy Ybar, Acc  = Ybar
//   S3/S2: kb = Kin;           Kout = cq Qb + cy Ybar, Acc += Ybar
//   S1:    kb = Kin;           Qb  = Qb + Acc + Ybar
// and every role but PLAIN adds the bathymetry cotangent into Bb.
enum : int { VJP_PLAIN = 0, VJP_S4 = 4, VJP_S3 = 3, VJP_S2 = 2, VJP_S1 = 1 };

// A node as the reverse reads it: its state, the bottom, r = eta/h - 1 and the seed
// of its rates, those of u, v and w times 1/(2h).
template <typename T>
struct VNode {
  T h, u, v, w, eta, r, b, ah, au, av, aw, ae;
};

template <typename T>
struct Cot {
  T h, u, v, w, eta, b;
};

// Column d of the 1D operator: weights of the lower and the upper neighbour that
// row d names (itself on a closure row) in (D^T Dbar)(d).  Interior/periodic
// rows are (-1, 0, 1)/(2 delta); the reflecting first and last rows are (-2, 2)/(2
// delta) (n >= 4 assumed).
template <typename T, int BC>
struct AxisTranspose {
  T wm, wp;
  __device__ __forceinline__ AxisTranspose(int i, int n, double inv2d, double invd) {
    wm = T(inv2d);
    wp = T(-inv2d);
    if (BC == BC_REFLECTING) {
      if (i == 0) wm = T(-invd);
      if (i == 1) wm = T(invd);
      if (i == n - 1) wp = T(invd);
      if (i == n - 2) wp = T(-invd);
    }
  }
};

// Planes of 16-byte vectors (128-bit LDS reads move twice the bytes per clock).
// Parts of a vector are stored through pointers of their own type: an element
// assignment would store the whole vector, and other threads write the rest.
typedef float sgn_f2 __attribute__((ext_vector_type(2)));
template <typename T, int H, int W>
struct VjpSmem;

template <int H, int W>
struct VjpSmem<double, H, W> {
  sgn_d2 hu[H][W], vw[H][W], er[H][W], bs[H][W], uv[H][W], we[H][W];
  __device__ __forceinline__ VNode<double> load(int r, int c) const {
    const sgn_d2 p = hu[r][c], q = vw[r][c], e = er[r][c], b = bs[r][c], x = uv[r][c], y = we[r][c];
    return VNode<double>{p.x, p.y, q.x, q.y, e.x, e.y, b.x, b.y, x.x, x.y, y.x, y.y};
  }
  __device__ __forceinline__ void store_state(int r, int c, const double (&y)[5], double rr) {
    hu[r][c] = sgn_d2{y[0], y[1]};
    vw[r][c] = sgn_d2{y[2], y[3]};
    er[r][c] = sgn_d2{y[4], rr};
  }
  __device__ __forceinline__ void store_b(int r, int c, double b) { ((double*)&bs[r][c])[0] = b; }
  __device__ __forceinline__ void store_seed(int r, int c, const double (&a)[5]) {
    ((double*)&bs[r][c])[1] = a[0];
    uv[r][c] = sgn_d2{a[1], a[2]};
    we[r][c] = sgn_d2{a[3], a[4]};
  }
};

template <int H, int W>
struct VjpSmem<float, H, W> {
  sgn_f4 y4[H][W], eb[H][W], a4[H][W];
  __device__ __forceinline__ VNode<float> load(int r, int c) const {
    const sgn_f4 p = y4[r][c], q = eb[r][c], a = a4[r][c];
    return VNode<float>{p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w, a.x, a.y, a.z, a.w};
  }
  __device__ __forceinline__ void store_state(int r, int c, const float (&y)[5], float rr) {
    y4[r][c] = sgn_f4{y[0], y[1], y[2], y[3]};
    ((sgn_f2*)&eb[r][c])[0] = sgn_f2{y[4], rr};
  }
  __device__ __forceinline__ void store_b(int r, int c, float b) { ((float*)&eb[r][c])[2] = b; }
  __device__ __forceinline__ void store_seed(int r, int c, const float (&a)[5]) {
    ((float*)&eb[r][c])[3] = a[0];
    a4[r][c] = sgn_f4{a[1], a[2], a[3], a[4]};
  }
};

// Seeds as they are staged, from the cotangent k of the five rates; ih = 1/h.
template <typename T>
__device__ __forceinline__ void staged_seed(const T (&k)[5], T ih, T (&a)[5]) {
#pragma clang fp contract(off)
  const T hih = T(0.5) * ih;
  a[0] = k[0];
  a[1] = k[1] * hih;
  a[2] = k[2] * hih;
  a[3] = k[3] * hih;
  a[4] = k[4];
}

// The values of a node by axis (n along, t across) and the products its own
// derivatives share.
template <typename T>
struct VAxisNode {
  T n, t, an, at;
};
template <typename T>
__device__ __forceinline__ VAxisNode<T> along_x(const VNode<T>& c) {
  return VAxisNode<T>{c.u, c.v, c.au, c.av};
}
template <typename T>
__device__ __forceinline__ VAxisNode<T> along_y(const VNode<T>& c) {
  return VAxisNode<T>{c.v, c.u, c.av, c.au};
}

// What one axis gives: the cotangents of the node's values (r: through r, the
// centre's only) and the sums A, Tt, Tw of the rates h n_t, h t_t and h w_t along it
// (twice the negative of their part, times the scale s).
template <typename T>
struct VAxis {
  T h, n, t, w, eta, b, r, A, Tt, Tw;
};

template <typename T>
__device__ __forceinline__ VAxis<T> axis_reverse(const VNode<T>& c, const VAxisNode<T>& ca, const VNode<T>& m,
                                                 const VAxisNode<T>& ma, const VNode<T>& p, const VAxisNode<T>& pa,
                                                 T s, T wm, T wp, T g2, T lam) {
#pragma clang fp contract(off)
  const T lam3 = lam * T(1.0 / 3.0);
  const T h = c.h, n = ca.n, t = ca.t, w = c.w;
  const T H = h + c.b, hn = h * n, r2 = c.r * c.r, rho = T(1) + c.r;
  VAxis<T> o;
  // the centre's part: differences of the two neighbours
  const T dh = p.h - m.h, dn = pa.n - ma.n, dt = pa.t - ma.t, dw = p.w - m.w, deta = p.eta - m.eta, db = p.b - m.b;
  const T sn = pa.n + ma.n;
  const T hdn = h * dn, ndh = n * dh;
  const T dR = ndh + hdn;
  const T Qp = fused(p.h, pa.n, hn), Qm = fused(m.h, ma.n, hn);
  const T X = (Qp - Qm) - dR;
  const T zp = (p.h + p.b) - H, zm = (m.h + m.b) - H;
  o.Tt = fused(Qp, pa.t, fused(-Qm, ma.t, -(t * dR)));
  o.Tw = fused(Qp, p.w, fused(-Qm, m.w, -(w * dR)));
  const T P = fused(zp, p.h, -(zm * m.h));
  const T ddh = deta - dh;
  const T R = fused(T(-2) * rho, ddh, fused(r2, dh, fused(m.r * m.r, m.h, -((p.r * p.r) * p.h))));
  o.A = fused(-(lam * c.r), db, fused(lam3, R, fused(g2, P, fused(hdn, sn, n * X))));
  const T gdh = (g2 * ca.an) * dh;
  const T cn = -fused(c.ah, dh,
                      fused(ca.an, X - ndh,
                            fused(ca.at, fused(h, dt, -(t * dh)),
                                  fused(c.aw, fused(h, dw, -(w * dh)), c.ae * fused(T(1.5), db, deta)))));
  const T ch = gdh - fused(c.ah, dn,
                           fused(ca.an * dn, sn - n,
                                 fused(ca.at, fused(n, dt, -(t * dn)), c.aw * fused(n, dw, -(w * dn)))));
  o.r = (s * (lam * ca.an)) * fused(T(2.0 / 3.0), fused(-c.r, dh, ddh), db);
  o.n = s * cn;
  o.h = s * ch;
  o.t = s * (ca.at * dR);
  o.w = s * (c.aw * dR);
  o.b = s * gdh;
  // the neighbours' rates, in which this node is the neighbour
  const T ht = h * t, hw = h * w, nt = n * t, nw = n * w, n2 = n + n;
  const auto side = [&](const VNode<T>& q, const VAxisNode<T>& qa, T Q, T z, T wt, T x2) {
#pragma clang fp contract(off)
    const T x1 = wt * q.ah, x3 = wt * qa.at, x4 = wt * q.aw;
    o.t = fused(-x3, Q, o.t);
    o.w = fused(-x4, Q, o.w);
    const T fn = fused(q.h, n2, qa.n * (h - q.h));  // 2 h_m n + n_m (h - h_m)
    o.n = fused(-x1, q.h, fused(-x2, fn, fused(-x3, fused(-q.h, qa.t, ht), fused(-x4, fused(-q.h, q.w, hw), o.n))));
    const T fh = fused(-g2, z, qa.n * (n - qa.n));  // and 2g h of the sum below
    o.h = fused(-x1, qa.n, fused(-x2, fh, fused(-x3, fused(-qa.n, qa.t, nt), fused(-x4, fused(-qa.n, q.w, nw), o.h))));
  };
  // The terms that carry g or lambda and this node's values take the difference
  // of the neighbours' seeds first:
  //   h: 2g h + lam/3 ((1 + r)^2 + 1 + 2 r_m + r_m^2),  eta: -2 lam/3 (1 + r + r_m),
  //   b: 2g h - lam r_m,  times -x2 each
  const T x2m = wm * ma.an, x2p = wp * pa.an;
  side(m, ma, Qm, zm, wm, x2m);
  side(p, pa, Qp, zp, wp, x2p);
  const T x2 = x2m + x2p, tm = x2m * m.r, tp = x2p * p.r;
  const T xr = tm + tp, xrr = fused(tm, m.r, tp * p.r);
  const T x5 = fused(wm * m.ae, ma.n, (wp * p.ae) * pa.n);
  const T g2h = g2 * h;
  o.h = fused(-lam3, fused(T(2), xr, xrr), fused(-fused(lam3, fused(rho, rho, T(1)), g2h), x2, o.h));
  o.eta = fused(T(2) * lam3, fused(rho, x2, xr), -x5);
  o.b = fused(lam, xr, fused(-g2h, x2, fused(T(-1.5), x5, o.b)));
  return o;
}

// Cotangent of the raw values of node (i, j), in the domain, from a staging s
// around the node's position (r, c).  All multiply-adds are written out and no
// others are formed, so every kernel rounds it alike.
template <typename T, int BCX, int BCY, class Smem>
__device__ __forceinline__ Cot<T> vjp_node(const Smem& s, int r, int c, int i, int j, const GridConst& gc) {
#pragma clang fp contract(off)
  const int nx = gc.nx, ny = gc.ny;
  const T g2 = T(2) * T(gc.g), lam = T(gc.lam);
  const AxisStencil<BCX> ax(i, nx, gc.inv2dx, gc.invdx);
  const AxisTranspose<T, BCX> tx(i, nx, gc.inv2dx, gc.invdx);
  const AxisStencil<BCY> ay(j, ny, gc.inv2dy, gc.invdy);
  const AxisTranspose<T, BCY> ty(j, ny, gc.inv2dy, gc.invdy);
  const VNode<T> cn = s.load(r, c);
  const VNode<T> xm = s.load(r, c + ax.om), xp = s.load(r, c + ax.op);
  const T ih = recip_staged(cn.h);
  const T sx = T(ax.scale), sy = T(ay.scale);
  const VAxis<T> x = axis_reverse<T>(cn, along_x(cn), xm, along_x(xm), xp, along_x(xp), sx, tx.wm, tx.wp, g2, lam);
  const VNode<T> ym = s.load(r + ay.om, c), yp = s.load(r + ay.op, c);
  const VAxis<T> y = axis_reverse<T>(cn, along_y(cn), ym, along_y(ym), yp, along_y(yp), sy, ty.wm, ty.wp, g2, lam);
  // through r = eta/h - 1 and the 1/h of the rates
  const T xr = (x.r + y.r) - (T(2) * lam) * cn.aw;
  const T kh = fused(cn.au, fused(sx, x.A, sy * y.Tt),
                     fused(cn.av, fused(sy, y.A, sx * x.Tt),
                           cn.aw * fused(sx, x.Tw, fused(sy, y.Tw, (T(2) * lam) * cn.r))));
  Cot<T> o;
  o.h = fused(ih, fused(-xr, T(1) + cn.r, kh), x.h + y.h);
  o.u = x.n + y.t;
  o.v = x.t + y.n;
  o.w = (x.w + y.w) + cn.ae;
  o.eta = fused(xr, ih, x.eta + y.eta);
  o.b = x.b + y.b;
  if (BCX == BC_REFLECTING && (i == 0 || i == nx - 1)) {  // the wall SAT ah satx h u
    const T a = cn.ah * T(i == 0 ? -2.0 * gc.invdx : 2.0 * gc.invdx);
    o.h = fused(a, cn.u, o.h);
    o.u = fused(a, cn.h, o.u);
  }
  if (BCY == BC_REFLECTING && (j == 0 || j == ny - 1)) {
    const T a = cn.ah * T(j == 0 ? -2.0 * gc.invdy : 2.0 * gc.invdy);
    o.h = fused(a, cn.v, o.h);
    o.v = fused(a, cn.h, o.v);
  }
  return o;
}

// Stages a node: v = its state, b and the seed before its factor a.
template <typename T, class Smem>
__device__ __forceinline__ void stage_node(Smem& s, int r, int c, const T (&v)[11], T a) {
  const T ih = recip_staged(v[0]);
  const T y[5] = {v[0], v[1], v[2], v[3], v[4]};
  const T k[5] = {a * v[6], a * v[7], a * v[8], a * v[9], a * v[10]};
  T sd[5];
  staged_seed(k, ih, sd);
  s.store_state(r, c, y, (y[4] - y[0]) * ih);
  s.store_b(r, c, v[5]);
  s.store_seed(r, c, sd);
}

// One reverse-mode stage (role ROLE) on a 64 x TY tile per workgroup.
template <typename T, int BCX, int BCY, int ROLE, int TY>
__global__ __launch_bounds__(STAGE_THREADS) void vjp_kernel(const GridConst gc, const T* __restrict__ Y,
                                                            const T* __restrict__ bplane, const T* Kin, T* Qb,
                                                            T* __restrict__ Kout, T* __restrict__ Acc,
                                                            T* __restrict__ Bb, T a_in, T cq, T cy) {
  static_assert(TY % THREAD_ROWS == 0, "tile height must be a multiple of 4");
  constexpr int RPT = TY / THREAD_ROWS;
  constexpr int W = TILE_X + 2;
  constexpr int REGION = (TY + 2) * W;
  __shared__ VjpSmem<T, TY + 2, W> s;
  const int nx = gc.nx, ny = gc.ny;
  const size_t N = (size_t)nx * (size_t)ny;
  const int ntx = (nx + TILE_X - 1) / TILE_X;
  const int nty = (ny + TY - 1) / TY;
  const int tile = xcd_tile(blockIdx.x, ntx * nty);
  const int i0 = (tile % ntx) * TILE_X;
  const int j0 = (tile / ntx) * TY;
  const int tid = threadIdx.x;
  const int tx = tid & (TILE_X - 1);
  const int ty = tid >> 6;

  // Stage Y, b and the scaled seeds with a one-node halo.  Every load of the
  // region is issued before the first LDS write waits for one, so each
  // workgroup keeps the whole region in flight.
  {
    constexpr int ITER = (REGION + STAGE_THREADS - 1) / STAGE_THREADS;
    T v[ITER][11];
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      const int idx = tid + it * STAGE_THREADS;
      if (idx < REGION) {
        const int rr = idx / W;
        const int cc = idx - rr * W;
        int gi = i0 - 1 + cc;
        int gj = j0 - 1 + rr;
        if (BCX == BC_PERIODIC) {
          if (gi < 0) gi += nx;
          while (gi >= nx) gi -= nx;
        } else {
          gi = gi < 0 ? 0 : (gi >= nx ? nx - 1 : gi);
        }
        if (BCY == BC_PERIODIC) {
          if (gj < 0) gj += ny;
          while (gj >= ny) gj -= ny;
        } else {
          gj = gj < 0 ? 0 : (gj >= ny ? ny - 1 : gj);
        }
        const size_t o = (size_t)gj * nx + gi;
#pragma unroll
        for (int f = 0; f < 5; ++f) v[it][f] = Y[f * N + o];
        v[it][5] = bplane[o];
#pragma unroll
        for (int f = 0; f < 5; ++f) v[it][6 + f] = Kin[f * N + o];
      }
    }
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      const int idx = tid + it * STAGE_THREADS;
      if (idx < REGION) {
        const int rr = idx / W;
        const int cc = idx - rr * W;
        stage_node<T>(s, rr, cc, v[it], a_in);
      }
    }
  }
  __syncthreads();

  const int i = i0 + tx;
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int lr = ty + k * THREAD_ROWS;
    const int j = j0 + lr;
    if (i >= nx || j >= ny) continue;
    // this node's qbar and bbar, loaded before the evaluation so that their
    // latency overlaps it (the sum Acc is read at the end: loaded here too it
    // takes the reflecting instances past 256 registers)
    const size_t od = (size_t)j * nx + i;
    T qv[5], bv = T(0);
    if (ROLE != VJP_PLAIN) {
#pragma unroll
      for (int f = 0; f < 5; ++f) qv[f] = Qb[f * N + od];
      bv = Bb[od];
    }
    const Cot<T> out = vjp_node<T, BCX, BCY>(s, lr + 1, tx + 1, i, j, gc);
    const T yb[5] = {out.h, out.u, out.v, out.w, out.eta};
    if (ROLE == VJP_PLAIN) {
#pragma unroll
      for (int f = 0; f < 5; ++f) Kout[f * N + od] = yb[f];
      Bb[od] = out.b;
    } else {
      if (ROLE == VJP_S4) {
#pragma unroll
        for (int f = 0; f < 5; ++f) {
          Kout[f * N + od] = fused(cq, qv[f], cy * yb[f]);
          Acc[f * N + od] = yb[f];
        }
      } else if (ROLE == VJP_S3 || ROLE == VJP_S2) {
#pragma unroll
        for (int f = 0; f < 5; ++f) {
          Kout[f * N + od] = fused(cq, qv[f], cy * yb[f]);
          Acc[f * N + od] = Acc[f * N + od] + yb[f];
        }
      } else {
#pragma unroll
        for (int f = 0; f < 5; ++f) Qb[f * N + od] = qv[f] + Acc[f * N + od] + yb[f];
      }
      Bb[od] = bv + out.b;
    }
  }
}

// Two consecutive reverse stages in one launch, the reverse counterpart of the
// step kernel's temporal blocking: PAIR = 2 runs roles S4 and S3, PAIR = 1
// roles S2 and S1, over the step kernel's TX x (512 / TX) tiles.  The first
// evaluation (state YA and seed aA * KinA, staged with a two-node halo) runs
// on the tile and on the ring of nodes around it; there its stage cotangent
// YbarA gives the second evaluation's seed kbB = cqA qbar + cyA YbarA, which
// replaces the first seed in LDS beside the second state YB (one-node halo),
// and the second evaluation runs on the tile:
//   PAIR 2: KinA = qbar, aA = dt/6, YA = Y4, YB = Y3, (cqA, cyA) = (dt/3, dt),
//           Kout = cqB qbar + cyB YbarB with (cqB, cyB) = (dt/3, dt/2),
//           Acc = YbarA + YbarB
//   PAIR 1: KinA = the seed of S2, aA = 1, YA = Y2, YB = Y1 = q_n,
//           (cqA, cyA) = (dt/6, dt/2), QbOut = qbar + (Acc + YbarA) + YbarB
//           (a buffer other than Qb: neighbouring tiles still read qbar on
//           their rings while this one writes)
//   both:   bbar = (bbar + bbarA) + bbarB.
// YbarA and bbarA of the owned nodes stay in registers.  Node by node this is the
// arithmetic of the two role kernels, and the results do not depend on the tile
// shape.  Algorithmic traffic per node: 28 values for S4 + S3
// (role kernels: 56) and 33 for S2 + S1 (61); the price is the ring of first
// evaluations (1 + 2 (TX + 2 + TY) / 512 of them per owned node).
// The reverse kernels use the 512-node step tiles: 32 x 16 or 64 x 8.
template <int TX>
using VjpGeom = StepGeom<TX == 64 ? 8 : 16>;

template <typename T, int BCX, int BCY, int PAIR, int TX>
__global__ __launch_bounds__(STAGE_THREADS, 2) void vjp_pair_kernel(const GridConst gc, const T* __restrict__ YA,
                                                                 const T* __restrict__ YB,
                                                                 const T* __restrict__ bplane, const T* KinA,
                                                                 const T* Qb, T* __restrict__ QbOut,
                                                                 T* __restrict__ Kout, T* __restrict__ Acc,
                                                                 T* __restrict__ Bb, T aA, T cqA, T cyA, T cqB,
                                                                 T cyB) {
  static_assert(PAIR == 1 || PAIR == 2, "PAIR is 2 (S4 + S3) or 1 (S2 + S1)");
  using G = VjpGeom<TX>;
  static_assert(G::TX == TX, "32 x 16 or 64 x 8 tiles");
  constexpr int TY = G::TY;
  constexpr int H = 2;  // LDS position of tile node (0, 0)
  constexpr int RXA = TX + 2 * H, REGA = RXA * (TY + 2 * H);
  constexpr int RXB = TX + 2, REGB = RXB * (TY + 2);
  __shared__ VjpSmem<T, TY + 2 * H, RXA> s;
  const int nx = gc.nx, ny = gc.ny;
  const size_t N = (size_t)nx * (size_t)ny;
  const int ntx = (nx + TX - 1) / TX;
  const int nty = (ny + TY - 1) / TY;
  const int tile = xcd_tile(blockIdx.x, ntx * nty);
  const int i0 = (tile % ntx) * TX;
  const int j0 = (tile / ntx) * TY;
  const int tid = threadIdx.x;

  // 1. YA, b and aA * KinA with a two-node halo; all loads issued first
  {
    constexpr int ITER = (REGA + STAGE_THREADS - 1) / STAGE_THREADS;
    T v[ITER][11];
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      const int idx = tid + it * STAGE_THREADS;
      if (idx < REGA) {
        const int rr = idx / RXA;
        const int cc = idx - rr * RXA;
        const size_t o = (size_t)wrap_or_clamp<BCY>(j0 - H + rr, ny) * nx + wrap_or_clamp<BCX>(i0 - H + cc, nx);
#pragma unroll
        for (int f = 0; f < 5; ++f) v[it][f] = YA[f * N + o];
        v[it][5] = bplane[o];
#pragma unroll
        for (int f = 0; f < 5; ++f) v[it][6 + f] = KinA[f * N + o];
      }
    }
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      const int idx = tid + it * STAGE_THREADS;
      if (idx < REGA) {
        const int rr = idx / RXA;
        const int cc = idx - rr * RXA;
        stage_node<T>(s, rr, cc, v[it], aA);
      }
    }
  }

  // Slots of this thread: slot 0 the ring node tid (if any), slots 1 and 2 the
  // tile nodes (lx, ly0) and (lx, ly0 + 1); positions relative to the tile.
  const int lx = tid % TX;
  const int ly0 = 2 * (tid / TX);
  int pr[3], pc[3];
  bool slot[3], ev[3];
  slot[0] = tid < G::RING1;
  pr[0] = 0;
  pc[0] = 0;
  if (slot[0]) ring_node<TY>(tid, pr[0], pc[0]);
  pr[1] = ly0;
  pc[1] = lx;
  pr[2] = ly0 + 1;
  pc[2] = lx;
  slot[1] = slot[2] = true;
#pragma unroll
  for (int q = 0; q < 3; ++q)
    ev[q] = slot[q] && on_axis<BCX>(i0 + pc[q], nx) && on_axis<BCY>(j0 + pr[q], ny);
  __syncthreads();

  // 2. First evaluation on the ring and the tile (periodic images of nodes past
  //    a ragged edge included).
  T ybA[3][5], bbA[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    __builtin_amdgcn_sched_barrier(0);
    if (!ev[q]) continue;
    const int iw = wrap_or_clamp<BCX>(i0 + pc[q], nx), jw = wrap_or_clamp<BCY>(j0 + pr[q], ny);
    const Cot<T> out = vjp_node<T, BCX, BCY>(s, pr[q] + H, pc[q] + H, iw, jw, gc);
    ybA[q][0] = out.h, ybA[q][1] = out.u, ybA[q][2] = out.v, ybA[q][3] = out.w, ybA[q][4] = out.eta;
    bbA[q] = out.b;
  }
  __builtin_amdgcn_sched_barrier(0);
  // the second state, loaded while the other waves finish their evaluations,
  // and the seeds of the second evaluation
  constexpr int ITB = (REGB + STAGE_THREADS - 1) / STAGE_THREADS;
  T w[ITB][5];
#pragma unroll
  for (int it = 0; it < ITB; ++it) {
    const int idx = tid + it * STAGE_THREADS;
    if (idx < REGB) {
      const int rr = idx / RXB;
      const int cc = idx - rr * RXB;
      const size_t o = (size_t)wrap_or_clamp<BCY>(j0 - 1 + rr, ny) * nx + wrap_or_clamp<BCX>(i0 - 1 + cc, nx);
#pragma unroll
      for (int f = 0; f < 5; ++f) w[it][f] = YB[f * N + o];
    }
  }
  T kbB[3][5];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if (!ev[q]) continue;
    const size_t o = (size_t)wrap_or_clamp<BCY>(j0 + pr[q], ny) * nx + wrap_or_clamp<BCX>(i0 + pc[q], nx);
    T kb[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) kb[f] = fused(cqA, Qb[f * N + o], cyA * ybA[q][f]);
    staged_seed(kb, recip_staged(YB[o]), kbB[q]);
  }
  __syncthreads();

  // 3. YB and its r over the one-node halo (b stays), the new seeds on the tile and
  //    ring.  Positions outside a reflecting wall keep old seeds: a node's neighbours
  //    are taken where its stencil names them, never beyond a wall.
#pragma unroll
  for (int it = 0; it < ITB; ++it) {
    const int idx = tid + it * STAGE_THREADS;
    if (idx < REGB) {
      const int rr = idx / RXB + H - 1;
      const int cc = idx - (idx / RXB) * RXB + H - 1;
      s.store_state(rr, cc, w[it], (w[it][4] - w[it][0]) * recip_staged(w[it][0]));
    }
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if (!ev[q]) continue;
    s.store_seed(pr[q] + H, pc[q] + H, kbB[q]);
  }
  __syncthreads();

  // 4. Second evaluation on the owned nodes in the domain, and the outputs.
  const int i = i0 + lx;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    __builtin_amdgcn_sched_barrier(0);
    const int j = j0 + ly0 + k;
    if (i >= nx || j >= ny) continue;
    const size_t od = (size_t)j * nx + i;
    T qv[5], av[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) qv[f] = Qb[f * N + od];
    if (PAIR == 1) {
#pragma unroll
      for (int f = 0; f < 5; ++f) av[f] = Acc[f * N + od];
    }
    const T bv = Bb[od];
    const Cot<T> out = vjp_node<T, BCX, BCY>(s, ly0 + k + H, lx + H, i, j, gc);
    const T yb[5] = {out.h, out.u, out.v, out.w, out.eta};
    if (PAIR == 2) {
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        Kout[f * N + od] = fused(cqB, qv[f], cyB * yb[f]);
        Acc[f * N + od] = ybA[1 + k][f] + yb[f];
      }
    } else {
#pragma unroll
      for (int f = 0; f < 5; ++f) QbOut[f * N + od] = qv[f] + (av[f] + ybA[1 + k][f]) + yb[f];
    }
    Bb[od] = bv + bbA[1 + k] + out.b;
  }
}

}  // namespace sgn
