// sgn_small.hpp -- one or two classical RK4 steps in one kernel, small grids.
//
// On a small grid a step lasts as long as one workgroup's chain of work: the
// launch, the staging and four stages with their barriers, while most of the chip
// idles.  This kernel makes the chain short.  A workgroup owns 8 x 8 nodes and
// takes two steps: it stages the nodes with a halo of eight and evaluates the
// eight stages on squares of 22^2, 20^2, ..., 8^2 nodes, one node per thread.  The
// redundant evaluations (31 per owned node and two steps, against 10.5 on 32 x 16
// tiles) run on compute units that had nothing else to do.  Threads are numbered
// from the owned square outwards, so that the nodes of a stage are the first ones
// and whole waves fall idle as the squares shrink.  Two LDS buffers alternate
// between the stages: one barrier each.
//
// FP64 64^2: 9.4 us a step on tiles, 5.1 us in this kernel (10.2 us a launch, of
// which about 4 are the launch and the staging).
#pragma once

#include "sgn_fused.hpp"

namespace sgn {

constexpr int SMALL_SIDE = 8;  // owned nodes per axis

template <int STEPS>
struct SmallGeom {
  static constexpr int HALO = 4 * STEPS;
  static constexpr int R = SMALL_SIDE + 2 * HALO;                        // staged nodes per axis
  static constexpr int EVAL = (R - 2) * (R - 2);                         // nodes of the first stage
  static constexpr int THREADS = (EVAL + 63) / 64 * 64;
};

// One stage's state around the workgroup's nodes, in 16-byte vectors.
template <typename T, int R>
struct SmallLds;

template <int R>
struct SmallLds<double, R> {
  sgn_d2 a[3][R * R];  // (h, u), (v, w), (eta, e)
  __device__ __forceinline__ Node<double> load(int k, double b) const {
    const sgn_d2 x = a[0][k], y = a[1][k], z = a[2][k];
    return Node<double>{x.x, x.y, y.x, y.y, z.x, b, z.y};
  }
  __device__ __forceinline__ void store(int k, const Node<double>& n) {
    a[0][k] = sgn_d2{n.h, n.u};
    a[1][k] = sgn_d2{n.v, n.w};
    a[2][k] = sgn_d2{n.eta, n.e};
  }
};

template <int R>
struct SmallLds<float, R> {
  sgn_f4 a[R * R];
  sgn_d2 z[R * R / 2];  // (eta, e) of two nodes
  __device__ __forceinline__ Node<float> load(int k, float b) const {
    const sgn_f4 x = a[k];
    const float* y = (const float*)z + 2 * k;
    return Node<float>{x.x, x.y, x.z, x.w, y[0], b, y[1]};
  }
  __device__ __forceinline__ void store(int k, const Node<float>& n) {
    a[k] = sgn_f4{n.h, n.u, n.v, n.w};
    float* y = (float*)z + 2 * k;
    y[0] = n.eta;
    y[1] = n.e;
  }
};

// Index of a node or of its periodic image, clamped at reflecting walls; the halo
// may be wider than the axis.
template <int BC>
__device__ __forceinline__ int small_index(int g, int n) {
  if (BC == BC_PERIODIC) {
    while (g < 0) g += n;
    while (g >= n) g -= n;
    return g;
  }
  return g < 0 ? 0 : (g >= n ? n - 1 : g);
}

// Position of thread t relative to the owned square: the square row by row,
// then the rings around it, each clockwise from its upper left corner.
__device__ __forceinline__ void small_node(int t, int& r, int& c) {
  if (t < SMALL_SIDE * SMALL_SIDE) {
    r = t / SMALL_SIDE;
    c = t % SMALL_SIDE;
    return;
  }
  int k = 1;  // ring
  while (t >= (SMALL_SIDE + 2 * k) * (SMALL_SIDE + 2 * k)) ++k;
  const int inner = SMALL_SIDE + 2 * (k - 1), len = inner + 1;
  const int p = t - inner * inner, side = p / len, off = p % len;
  const int lo = -k, hi = SMALL_SIDE - 1 + k;
  r = side == 0 ? lo : side == 1 ? lo + off : side == 2 ? hi : hi - off;
  c = side == 0 ? lo + off : side == 1 ? hi : side == 2 ? hi - off : lo;
}

// STEPS RK4 steps from q into qout (distinct).
template <typename T, int BCX, int BCY, int STEPS>
__global__ __launch_bounds__(SmallGeom<STEPS>::THREADS) void small_step_kernel(const GridConst gc,
                                                                               const T* __restrict__ q,
                                                                               const T* __restrict__ bplane,
                                                                               T* __restrict__ qout, T c6, T c3, T c2,
                                                                               T c1, int* __restrict__ flag) {
  using G = SmallGeom<STEPS>;
  constexpr int R = G::R, H = G::HALO;
  __shared__ SmallLds<T, R> s[2];
  __shared__ T sb[R * R];
  const int nx = gc.nx, ny = gc.ny;
  const size_t N = (size_t)nx * (size_t)ny;
  const int ntx = (nx + SMALL_SIDE - 1) / SMALL_SIDE;
  const int i0 = (int)(blockIdx.x % ntx) * SMALL_SIDE, j0 = (int)(blockIdx.x / ntx) * SMALL_SIDE;
  const int t = threadIdx.x;

  // own node
  int r, c;
  small_node(t, r, c);
  const int i = i0 + c, j = j0 + r, k = (r + H) * R + c + H;
  const bool dom = t < G::EVAL && on_axis<BCX>(i, nx) && on_axis<BCY>(j, ny);
  // staging: each thread its own node, then the outermost ring
  constexpr int EDGE = R * R - G::EVAL;
  static_assert(EDGE <= G::THREADS, "one edge node per thread");
  T v[2][6];
  int ke = 0;
  if (t < G::EVAL) {
    const size_t o = (size_t)small_index<BCY>(j, ny) * nx + small_index<BCX>(i, nx);
#pragma unroll
    for (int f = 0; f < 5; ++f) v[0][f] = q[f * N + o];
    v[0][5] = bplane[o];
  }
  if (t < EDGE) {
    int re, ce;
    small_node(G::EVAL + t, re, ce);
    ke = (re + H) * R + ce + H;
    const size_t o = (size_t)small_index<BCY>(j0 + re, ny) * nx + small_index<BCX>(i0 + ce, nx);
#pragma unroll
    for (int f = 0; f < 5; ++f) v[1][f] = q[f * N + o];
    v[1][5] = bplane[o];
  }
  Node<T> n{T(1), T(0), T(0), T(0), T(1), T(0), T(0)};
  T ih = T(1), qn[5] = {}, acc[5] = {};
  if (t < G::EVAL) {
    n = Node<T>{v[0][0], v[0][1], v[0][2], v[0][3], v[0][4], v[0][5], T(0)};
    ih = recip_staged(n.h);
    n.e = node_e(n.h, n.eta, ih);
    s[0].store(k, n);
    sb[k] = n.b;
#pragma unroll
    for (int f = 0; f < 5; ++f) qn[f] = v[0][f];
  }
  if (t < EDGE) {
    Node<T> m{v[1][0], v[1][1], v[1][2], v[1][3], v[1][4], v[1][5], T(0)};
    m.e = node_e(m.h, m.eta, recip_staged(m.h));
    s[0].store(ke, m);
    sb[ke] = m.b;
  }
  __syncthreads();

  const AxisStencil<BCX> ax(i, nx, gc.inv2dx, gc.invdx);
  const AxisStencil<BCY> ay(j, ny, gc.inv2dy, gc.invdy);
  const bool own = t < SMALL_SIDE * SMALL_SIDE && i < nx && j < ny;
  const size_t o = (size_t)j * nx + i;
  const int kxm = k + ax.om, kxp = k + ax.op, kym = k + R * ay.om, kyp = k + R * ay.op;
  int health = 0;
#pragma unroll 1
  for (int p = 0; p < STEPS; ++p) {
#pragma unroll
    for (int st = 1; st <= 4; ++st) {
      const int g = 4 * p + st;  // stage of the launch
      const SmallLds<T, R>& in = s[(st - 1) & 1];
      const int side = R - 2 * g;
      if (dom && t < side * side) {
        const Node<T> xm = in.load(kxm, sb[kxm]), xp = in.load(kxp, sb[kxp]);
        const Node<T> ym = in.load(kym, sb[kym]), yp = in.load(kyp, sb[kyp]);
        const Rates<T> kk = node_rates<T, BCX, BCY, false>(n, ih, xm, xp, ym, yp, ax, ay, i, j, gc, 0.0);
        const T kv[5] = {kk.h, kk.u, kk.v, kk.w, kk.eta};
        const T cy = st == 3 ? c1 : c2;
        const T ca = st == 1 || st == 4 ? c6 : c3;
        T y[5];
#pragma unroll
        for (int f = 0; f < 5; ++f) {
          acc[f] = fused(ca, kv[f], st == 1 ? qn[f] : acc[f]);
          y[f] = st < 4 ? fused(cy, kv[f], qn[f]) : acc[f];
          if (st == 4) qn[f] = acc[f];
        }
        if (st == 4 && own) {
          if (!(y[0] > T(0))) health |= FLAG_NONPOS;
          const T sum = y[0] + y[1] + y[2] + y[3] + y[4];
          if (!isfinite(sum)) health |= FLAG_NONFINITE;
        }
        if (STEPS == 1 && st == 4) break;
        n.h = y[0], n.u = y[1], n.v = y[2], n.w = y[3], n.eta = y[4];
        ih = recip_staged(n.h);
        n.e = node_e(n.h, n.eta, ih);
        s[st & 1].store(k, n);
      }
      if (p < STEPS - 1 || st < 4) __syncthreads();
    }
  }
  if (own) {
#pragma unroll
    for (int f = 0; f < 5; ++f) qout[f * N + o] = qn[f];
  }
  if (health) atomicOr(flag, health);
}

}  // namespace sgn
