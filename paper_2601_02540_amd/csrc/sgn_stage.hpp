// sgn_stage.hpp -- the fused right-hand-side + Runge-Kutta stage kernel.
//
// One workgroup of 256 threads (four wave64s) owns a tile of 64 x TY nodes.
// It stages the tile plus a one-node halo of the six input planes
// (h, u, v, w, eta, b) and of (eta - h)^2/h in LDS, with the periodic wrap or
// the reflecting clamp applied while loading.  Each thread then evaluates the
// split-form rates of eq. (sd_periodic_2D_SGN) / eq. (semi_2D) for TY/4 nodes
// of one column, with the one-sided closure rows and the wall SATs of Remark
// "Concrete SBP operators and SATs" resolved per node, and applies the stage
// update in registers.
#pragma once

#include "sgn_common.hpp"
#include "sgn_mms.hpp"

namespace sgn {

constexpr int TILE_X = 64;
constexpr int STAGE_THREADS = 256;
constexpr int THREAD_ROWS = STAGE_THREADS / TILE_X;  // 4

// Neighbour selection along one axis for node index i of n: the left/right
// LDS offsets (relative to the node) and the derivative scale.  Interior and
// periodic rows use (f[i+1] - f[i-1]) / (2 d); reflecting first/last rows use
// (f[1] - f[0]) / d and (f[n-1] - f[n-2]) / d.
template <int BC>
struct AxisStencil {
  int om, op;
  double scale;
  __device__ __forceinline__ AxisStencil(int i, int n, double inv2d, double invd) {
    om = -1;
    op = 1;
    scale = inv2d;
    if (BC == BC_REFLECTING) {
      if (i == 0) {
        om = 0;
        scale = invd;
      }
      if (i == n - 1) {
        op = 0;
        scale = invd;
      }
    }
  }
};

// A node as the right-hand side reads it: the state, the bottom and
// e = (eta - h)^2 / h, the only quantity of a neighbour that needs a division
// (formed once per node and stage, where the node is staged).
template <typename T>
struct Node {
  T h, u, v, w, eta, b, e;
};

// e of a staged node; ih = recip_staged(h).
template <typename T>
__device__ __forceinline__ T node_e(T h, T eta, T ih) {
#pragma clang fp contract(off)
  const T d = eta - h;
  return (d * d) * ih;
}

// The two forms in which the rates are evaluated, equal to rounding.  FORM_SHARED
// (everything but the FP64 gauge rollouts): the split form gathered over the two
// neighbours of an axis, products shared between the rates (axis_terms).
// FORM_TERMS: the printed sums term by term (term_rates), Node::e holding 1/h.  The
// FP64 rollouts and gradients of the gauge loss keep the second: the bottom's
// gradient is the difference of two sums of the misfits' size (grad_b = bbar -
// grad_zeta0) that cancel where the water rests, down to 1e-10 of them and less, so
// its digits there are the rounding of every evaluation that went into the sums.
// With this form they stay those of the gradients on record; the other moved
// grad_b by 4e-10 of its norm and single nodes by 6e-8 (146 x 261, 24 steps), no
// nearer to the exact value.  Its price: 48 steps of 640 x 512 take 6660 us with
// their gradient (6930 on the tiles of the time before), 5330 in FORM_SHARED.
enum : int { FORM_SHARED = 0, FORM_TERMS = 1 };

// The seventh value of a staged node.
template <int FORM, typename T>
__device__ __forceinline__ T node_extra(T h, T eta, T ih) {
  return FORM == FORM_TERMS ? ih : node_e(h, eta, ih);
}

template <typename T, int TY>
struct StageSmem {
  T f[7][TY + 2][TILE_X + 2];  // h u v w eta b e
};

template <typename T, int TY>
__device__ __forceinline__ Node<T> lds_node(const StageSmem<T, TY>& s, int r, int c) {
  Node<T> n;
  n.h = s.f[0][r][c];
  n.u = s.f[1][r][c];
  n.v = s.f[2][r][c];
  n.w = s.f[3][r][c];
  n.eta = s.f[4][r][c];
  n.b = s.f[5][r][c];
  n.e = s.f[6][r][c];
  return n;
}

__device__ __forceinline__ double fused(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fused(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// Rates of the five evolved variables at one node given its value, its four
// neighbours (already resolved for closures) and the derivative scales.
template <typename T>
struct Rates {
  T h, u, v, w, eta;
};

// The terms of one axis at a node: n is the velocity along the axis, t the one
// across.  With the sums over the two neighbours m = +, - written S(f_m) =
// f_+ - f_- (one-sided rows name the node itself as a neighbour; S(1) = 0), the
// split form of the axis is
//   dR = S(n h_m + h n_m)                               D-part of h_t
//   A2 = h S(n_m^2) - n^2 S(h_m) + n S(h_m n_m) - h n S(n_m)
//      = h S(n_m) (n_+ + n_-) + n (S(Q_m) - dR)         Q_m = h_m n_m + h n
//   Tf = S(h_m n_m f_m) - n f S(h_m) + h n S(f_m) - h f S(n_m)
//      = S(Q_m f_m) - f dR                              f = t, w
//   P  = S(h_m (h_m + b_m)) - (h + b) S(h_m) = S(h_m (zeta_m - zeta))
//   relaxation, r = eta/h - 1: lambda/3 R - lambda r S(b_m) is twice
//      lambda/6 (eta^2/h^2 S(h_m) - S(eta_m^2/h_m)) - lambda/3 r S(eta_m)
//      - lambda/2 r S(b_m), with R = r^2 S(h_m) - (2 + 2 r) S(eta_m - h_m) - S(e_m)
// A = 2 g P + A2 + lambda/3 R - lambda r S(b), so that h n_t = -s/2 A + (cross
// axis); E = S(eta) + 3/2 S(b).  Each line is exact algebra on the printed
// sums, with products shared between the rates and none formed twice per
// neighbour; the small differences (S(h), S(n), zeta_m - zeta, eta - h) are
// formed first, so a state at rest gives exact zeros.
template <typename T>
struct AxisTerms {
  T dR, A, Tt, Tw, E;
};

template <typename T>
__device__ __forceinline__ AxisTerms<T> axis_terms(T h, T n, T hn, T t, T w, T H, T r2, T c2, T lamr, T g2, T lam3,
                                                   T mh, T mn, T mt, T mw, T meta, T mb, T me, T ph, T pn, T pt, T pw,
                                                   T peta, T pb, T pe) {
#pragma clang fp contract(off)
  AxisTerms<T> o;
  const T dh = ph - mh;
  const T dn = pn - mn;
  const T hdn = h * dn;
  o.dR = fused(n, dh, hdn);
  const T Qp = fused(ph, pn, hn);
  const T Qm = fused(mh, mn, hn);
  const T A2 = fused(hdn, pn + mn, n * ((Qp - Qm) - o.dR));
  o.Tt = fused(Qp, pt, fused(-Qm, mt, -(t * o.dR)));
  o.Tw = fused(Qp, pw, fused(-Qm, mw, -(w * o.dR)));
  const T P = fused((ph + pb) - H, ph, -(((mh + mb) - H) * mh));
  const T deta = peta - meta;
  const T db = pb - mb;
  const T R = fused(-c2, deta - dh, fused(r2, dh, me - pe));
  o.A = fused(-lamr, db, fused(lam3, R, fused(g2, P, A2)));
  o.E = fused(T(1.5), db, deta);
  return o;
}

// What the axis terms and the rates share of a node's own values.
template <typename T>
struct CenterTerms {
  T hu, hv, H, r2, c2, lamr;
  __device__ __forceinline__ CenterTerms(const Node<T>& c, T ih, T lam) {
#pragma clang fp contract(off)
    hu = c.h * c.u;
    hv = c.h * c.v;
    H = c.h + c.b;
    const T r = (c.eta - c.h) * ih;
    r2 = r * r;
    c2 = fused(T(2), r, T(2));
    lamr = lam * r;
  }
};

template <typename T>
__device__ __forceinline__ AxisTerms<T> x_terms(const Node<T>& c, const CenterTerms<T>& t, const Node<T>& m,
                                                const Node<T>& p, T g, T lam) {
  return axis_terms<T>(c.h, c.u, t.hu, c.v, c.w, t.H, t.r2, t.c2, t.lamr, T(2) * g, lam * T(1.0 / 3.0), m.h, m.u, m.v,
                       m.w, m.eta, m.b, m.e, p.h, p.u, p.v, p.w, p.eta, p.b, p.e);
}

template <typename T>
__device__ __forceinline__ AxisTerms<T> y_terms(const Node<T>& c, const CenterTerms<T>& t, const Node<T>& m,
                                                const Node<T>& p, T g, T lam) {
  return axis_terms<T>(c.h, c.v, t.hv, c.u, c.w, t.H, t.r2, t.c2, t.lamr, T(2) * g, lam * T(1.0 / 3.0), m.h, m.v, m.u,
                       m.w, m.eta, m.b, m.e, p.h, p.v, p.u, p.w, p.eta, p.b, p.e);
}

// The rates from the terms of the two axes.  Every derivative along one axis
// at a node carries the same scale (1/(2d) on interior and periodic rows, 1/d on
// a closure row), applied once per axis sum.  The wall SAT enters only on
// reflecting axes.
template <typename T, int BCX, int BCY>
__device__ __forceinline__ Rates<T> join_rates(const Node<T>& c, T ih, const CenterTerms<T>& t, const AxisTerms<T>& x,
                                               const AxisTerms<T>& y, T sx, T sy, T satx_coef, T saty_coef) {
#pragma clang fp contract(off)
  const T hsx = T(0.5) * sx, hsy = T(0.5) * sy;
  Rates<T> k;
  k.h = fused(-sx, x.dR, -(sy * y.dR));
  if (BCX == BC_REFLECTING) k.h = fused(satx_coef, t.hu, k.h);
  if (BCY == BC_REFLECTING) k.h = fused(saty_coef, t.hv, k.h);
  k.u = fused(-hsx, x.A, -(hsy * y.Tt)) * ih;
  k.v = fused(-hsy, y.A, -(hsx * x.Tt)) * ih;
  k.w = (fused(-hsx, x.Tw, -(hsy * y.Tw)) - t.lamr) * ih;
  k.eta = fused(-(c.u * sx), x.E, fused(-(c.v * sy), y.E, c.w));
  return k;
}

// Rates at node c; ih = recip_staged(c.h).  All multiply-adds are written out
// and the compiler forms no others, so every kernel rounds an evaluation alike,
// whatever surrounds it.
template <typename T, int BCX, int BCY>
__device__ __forceinline__ Rates<T> split_form_rates(const Node<T>& c, T ih, const Node<T>& xm, const Node<T>& xp,
                                                     const Node<T>& ym, const Node<T>& yp, T sx, T sy, T g, T lam,
                                                     T satx_coef, T saty_coef) {
  const CenterTerms<T> t(c, ih, lam);
  const AxisTerms<T> x = x_terms(c, t, xm, xp, g, lam);
  const AxisTerms<T> y = y_terms(c, t, ym, yp, g, lam);
  return join_rates<T, BCX, BCY>(c, ih, t, x, y, sx, sy, satx_coef, saty_coef);
}

// a b - x y, the first product unrounded.
template <typename T>
__device__ __forceinline__ T diff_of_products(T a, T b, T x, T y) {
#pragma clang fp contract(off)
  return fused(a, b, -(x * y));
}

// FORM_TERMS, one axis (n the velocity along it, t the one across): the differences
// of the printed products, unscaled, and the sums of the rates' terms.  With
// D(eta^2/h) = D(h) + D((eta - h)(eta + h)/h), whose second part is small (eta stays
// close to h), lambda/6 (r^2 D h - D(eta^2/h)) is formed without cancellation.
//   A1 = g (D(h(h+b)) - (h+b) D h) + lambda/6 ((r^2 - 1) D h - D((eta-h)(eta+h)/h))
//        + lambda/3 (1 - r) D eta + lambda/2 (1 - r) D b
//   A2 = h D(n^2) - n^2 D h + n D(h n) - h n D n,  T = D(h n t) - n t D h + h n D t - h t D n
//   C  = the same with w for t,  R = n D h + h D n,  E = n D eta + 3/2 n D b
template <typename T>
struct AxisSums {
  T A1, A2, Tt, C, R, E;
};

template <typename T>
__device__ __forceinline__ AxisSums<T> axis_sums(T h, T n, T t, T w, T H, T hn, T ht, T hw, T uv, T r2m1, T omr, T g,
                                                 T lam, const Node<T>& m, T mn, T mt, const Node<T>& p, T pn, T pt) {
#pragma clang fp contract(off)
  const T dh = p.h - m.h, dn = pn - mn, dt = pt - mt, dw = p.w - m.w, deta = p.eta - m.eta, db = p.b - m.b;
  const T phn = p.h * pn, mhn = m.h * mn;
  const T dhH = diff_of_products(p.h, p.h + p.b, m.h, m.h + m.b);
  const T dn2 = diff_of_products(pn, pn, mn, mn);
  const T dhn = diff_of_products(p.h, pn, m.h, mn);
  const T dhnt = diff_of_products(phn, pt, mhn, mt);
  const T de2 = diff_of_products((p.eta - p.h) * (p.eta + p.h), p.e, (m.eta - m.h) * (m.eta + m.h), m.e);
  const T dhnw = diff_of_products(phn, p.w, mhn, m.w);
  const T lam6 = lam * T(1.0 / 6.0), lam3 = lam * T(1.0 / 3.0), lam2 = lam * T(0.5);
  AxisSums<T> o;
  o.A1 = fused(lam2 * omr, db,
               fused(lam3 * omr, deta, fused(g, fused(-H, dh, dhH), lam6 * fused(r2m1, dh, -de2))));
  o.A2 = fused(-hn, dn, fused(n, dhn, diff_of_products(h, dn2, n * n, dh)));
  o.Tt = fused(-ht, dn, fused(hn, dt, fused(-uv, dh, dhnt)));
  o.C = fused(-hw, dn, fused(hn, dw, fused(-(n * w), dh, dhnw)));
  o.R = fused(n, dh, h * dn);
  o.E = fused(n, deta, (T(1.5) * n) * db);
  return o;
}

// FORM_TERMS: rates at node c.  Every derivative along one axis at a node carries the
// same scale, applied once per sum.  All multiply-adds are written out, as the
// gradients on record were rounded.
template <typename T, int BCX, int BCY>
__device__ __forceinline__ Rates<T> term_rates(const Node<T>& c, const Node<T>& xm, const Node<T>& xp,
                                               const Node<T>& ym, const Node<T>& yp, T sx, T sy, T g, T lam,
                                               T satx_coef, T saty_coef) {
#pragma clang fp contract(off)
  const T h = c.h, u = c.u, v = c.v, w = c.w, ih = c.e;
  // r - 1 = (eta - h)/h and r^2 - 1 = (r - 1)(r + 1), formed from eta - h, so
  // that a state at rest (eta = h) gives exactly zero relaxation terms
  const T rm1 = (c.eta - h) * ih;
  const T omr = -rm1;
  const T r2m1 = rm1 * (rm1 + T(2));
  const T H = h + c.b, hu = h * u, hv = h * v, uv = u * v, hw = h * w;
  const AxisSums<T> x = axis_sums<T>(h, u, v, w, H, hu, hv, hw, uv, r2m1, omr, g, lam, xm, xm.u, xm.v, xp, xp.u, xp.v);
  const AxisSums<T> y = axis_sums<T>(h, v, u, w, H, hv, hu, hw, uv, r2m1, omr, g, lam, ym, ym.v, ym.u, yp, yp.v, yp.u);
  const T hsx = T(0.5) * sx, hsy = T(0.5) * sy;
  Rates<T> k;
  k.h = -fused(sx, x.R, sy * y.R);
  if (BCX == BC_REFLECTING) k.h = fused(satx_coef, hu, k.h);
  if (BCY == BC_REFLECTING) k.h = fused(saty_coef, hv, k.h);
  k.u = -fused(hsy, y.Tt, fused(hsx, x.A2, sx * x.A1)) * ih;
  k.v = -fused(hsx, x.Tt, fused(hsy, y.A2, sy * y.A1)) * ih;
  k.w = fused(lam, omr, -fused(hsx, x.C, hsy * y.C)) * ih;
  k.eta = w - fused(sx, x.E, sy * y.E);
  return k;
}

template <typename T, int BCX, int BCY, int MODE, bool SRC, int TY>
__global__ __launch_bounds__(STAGE_THREADS) void stage_kernel(const GridConst gc, const T* __restrict__ Y,
                                                              const T* __restrict__ bplane,
                                                              const T* __restrict__ qn, T* __restrict__ acc,
                                                              T* __restrict__ out, T c_acc, T c_y, double t,
                                                              int* __restrict__ flag) {
  static_assert(TY % THREAD_ROWS == 0, "tile height must be a multiple of 4");
  constexpr int RPT = TY / THREAD_ROWS;
  constexpr int W = TILE_X + 2;
  constexpr int REGION = (TY + 2) * W;
  __shared__ StageSmem<T, TY> s;

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

  // Stage the tile and its halo.  Periodic axes wrap, reflecting axes clamp
  // (clamped halo values are never used: the closure rows are one-sided).
  for (int idx = tid; idx < REGION; idx += STAGE_THREADS) {
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
    const T h = Y[o];
    const T eta = Y[4 * N + o];
    s.f[0][rr][cc] = h;
    s.f[1][rr][cc] = Y[N + o];
    s.f[2][rr][cc] = Y[2 * N + o];
    s.f[3][rr][cc] = Y[3 * N + o];
    s.f[4][rr][cc] = eta;
    s.f[5][rr][cc] = bplane[o];
    s.f[6][rr][cc] = node_e(h, eta, recip_staged(h));
  }

  // Own-node operands of the stage update, fetched before the barrier so the
  // loads overlap the LDS staging.
  const int i = i0 + tx;
  T pre[RPT][5];
  T pacc[RPT][5];
  if (MODE == MODE_MID || MODE == MODE_LAST) {
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int j = j0 + ty + k * THREAD_ROWS;
      if (i < nx && j < ny) {
        const size_t o = (size_t)j * nx + i;
#pragma unroll
        for (int f = 0; f < 5; ++f) {
          pacc[k][f] = acc[f * N + o];
          if (MODE == MODE_MID) pre[k][f] = qn[f * N + o];
        }
      }
    }
  }
  __syncthreads();

  const T g = T(gc.g), lam = T(gc.lam);
  const AxisStencil<BCX> ax(i, nx, gc.inv2dx, gc.invdx);
  T satx = T(0);
  if (BCX == BC_REFLECTING) {
    if (i == 0) satx = T(-2.0 * gc.invdx);
    if (i == nx - 1) satx = T(2.0 * gc.invdx);
  }
  int health = 0;

#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int lr = ty + k * THREAD_ROWS;
    const int j = j0 + lr;
    if (i >= nx || j >= ny) continue;
    const AxisStencil<BCY> ay(j, ny, gc.inv2dy, gc.invdy);
    T saty = T(0);
    if (BCY == BC_REFLECTING) {
      if (j == 0) saty = T(-2.0 * gc.invdy);
      if (j == ny - 1) saty = T(2.0 * gc.invdy);
    }
    const int r = lr + 1, cidx = tx + 1;
    const Node<T> c = lds_node(s, r, cidx);
    const Node<T> xm = lds_node(s, r, cidx + ax.om);
    const Node<T> xp = lds_node(s, r, cidx + ax.op);
    const Node<T> ym = lds_node(s, r + ay.om, cidx);
    const Node<T> yp = lds_node(s, r + ay.op, cidx);
    Rates<T> kk = split_form_rates<T, BCX, BCY>(c, recip_staged(c.h), xm, xp, ym, yp, T(ax.scale), T(ay.scale), g, lam,
                                                satx, saty);
    if (SRC) {
      double S[5];
      mms_source(gc.xmin + i * gc.dx, gc.ymin + j * gc.dy, t, gc.g, S);
      kk.h += T(S[0]);
      kk.u += T(S[1]);
      kk.v += T(S[2]);
      kk.w += T(S[3]);
      kk.eta += T(S[4]);
    }
    const T kv[5] = {kk.h, kk.u, kk.v, kk.w, kk.eta};
    const T yv[5] = {c.h, c.u, c.v, c.w, c.eta};
    const size_t o = (size_t)j * nx + i;
    if (MODE == MODE_RHS) {
#pragma unroll
      for (int f = 0; f < 5; ++f) out[f * N + o] = kv[f];
    } else if (MODE == MODE_FIRST) {
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        acc[f * N + o] = fused(c_acc, kv[f], yv[f]);
        out[f * N + o] = fused(c_y, kv[f], yv[f]);
      }
    } else if (MODE == MODE_MID) {
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        acc[f * N + o] = fused(c_acc, kv[f], pacc[k][f]);
        out[f * N + o] = fused(c_y, kv[f], pre[k][f]);
      }
    } else {
      T nv[5];
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        nv[f] = fused(c_acc, kv[f], pacc[k][f]);
        out[f * N + o] = nv[f];
      }
      if (!(nv[0] > T(0))) health |= FLAG_NONPOS;
      const T sum = nv[0] + nv[1] + nv[2] + nv[3] + nv[4];
      if (!isfinite(sum)) health |= FLAG_NONFINITE;
    }
  }
  if (MODE == MODE_LAST && health) atomicOr(flag, health);
}

}  // namespace sgn
