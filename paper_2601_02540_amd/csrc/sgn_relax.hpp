// sgn_relax.hpp -- relaxation Runge-Kutta (fully discrete energy conservation).
//
// The semi-discretization conserves the total energy E = 1^T M E (Theorem 2);
// classical RK4 does not quite.  Relaxation in the incremental direction form
// takes the RK4 update d = q_RK4 - q_n, advances q_{n+1} = q_n + gam d and
// t_{n+1} = t_n + gam dt, with gam the root near 1 of E(q_n + gam d) = E(q_n);
// the method keeps its fourth order and conserves E to rounding.
//
// E(q_n + gam d) and E(q_n) agree in their leading digits (the potential
// energy dominates both), so their difference is not formed by subtraction.
// Per node, the change of each part of the energy density divided by gam is
// written out as a polynomial (a rational function for the lambda term) in gam
// whose coefficients are products of the node's values and increments:
//   kinetic   (h (u^2 + v^2)/2):  [dh (u^2 + v^2) + H (2u du + 2v dv + gam (du^2 + dv^2))] / 2
//   w term    (h w^2 / 6):        [dh w^2 + H (2w dw + gam dw^2)] / 6
//   potential (g h (h + 2b)/2):   g/2 dh (2h + 2b + gam dh)
//   lambda    (lam/6 (eta - h)^2 / h), A = eta - h, B = deta - dh:
//                                  lam/6 [h (2AB + gam B^2) - dh A^2] / (h H)
// with H = h + gam dh.  Their M-weighted sum s(gam) = (E(q_n + gam d) - E(q_n))/gam
// has no root at gam = 0; two Newton iterations from gam = 1 find the relaxation
// root.  All of it in FP64 whatever the storage type, with deterministic
// reductions (s and s' compensated).
//
// The second iteration would take a pass over 11 values a node.  It takes s and s'
// at its start gam_1 = 1 + delta from the series of s about 1 instead, whose
// coefficients are summed along with s(1) and s'(1): the polynomial parts end with
// delta^2, and the lambda term's coefficients fall by rho delta, rho = dh / (h + dh).
// Where the terms from delta^5 on could move gam by more than 2^-56 (sum M |t_5|
// bounds them), the pass runs.  2048^2 FP64 with walls: 71 + 5 us a step saved of 345.
#pragma once

#include "sgn_fused.hpp"
#include "sgn_reduce.hpp"

namespace sgn {

// Device scalars of a relaxation run.
struct RelaxScalars {
  double gam, t;
  double done;      // 1 when the second iteration has been made from the series
  int ticket, pad;  // of last_block; zero between kernels
};

// One Newton update of gam from s and s' at gam.  A step without a usable root
// (s' zero or not finite, or gam leaving [1/2, 3/2]) takes gam = 1.
__device__ __forceinline__ double relax_next(double gam, double s, double ds) {
  double next = gam;
  if (ds != 0.0 && isfinite(s) && isfinite(ds)) next = gam - s / ds;
  if (!(next >= 0.5 && next <= 1.5)) next = 1.0;
  return next;
}

// Both iterations from the sums at gam = 1, the second one where its series is exact
// enough (rs->done).
static __device__ void relax_root(const RelaxSums& a, RelaxScalars* __restrict__ rs, double dt) {
  const double s0 = a.s.s + a.s.c, s1 = a.ds.s + a.ds.c;
  const bool root = s1 != 0.0 && isfinite(s0) && isfinite(s1);
  const double gam1 = root ? 1.0 - s0 / s1 : 1.0;
  double gam = relax_next(1.0, s0, s1);
  double done = 1.0;  // without a usable root a second iteration repeats the first
  if (root && gam1 >= 0.5 && gam1 <= 1.5) {
    const double d = gam1 - 1.0;  // exact
    // s(1 + d) = s0 + s1 d + ..., the first two of which cancel but for the rounding of gam_1
    const double d2 = d * d;
    const double s = __builtin_fma(s1, d, s0) + d2 * (a.c2 + d * (a.c3 + d * a.c4));
    const double ds = s1 + d * (2.0 * a.c2 + d * (3.0 * a.c3 + 4.0 * d * a.c4));
    // sum_{k>=5} |t_k d^k| <= rem |d|^5 / (1 - |rho d|), and 5 rem |d|^4 / (1 - |rho d|)^2 for the derivative
    const double x = 1.0 - a.rho * fabs(d);
    const double es = a.rem * fabs(d) * d2 * d2 / x, eds = 5.0 * a.rem * d2 * d2 / (x * x);
    const double lim = 0x1p-56 * fabs(ds);
    if (x > 0.5 && es <= lim && eds * fabs(s) <= lim * fabs(ds) && isfinite(s) && isfinite(ds) && ds != 0.0) {
      gam = gam1 - s / ds;
      if (!(gam >= 0.5 && gam <= 1.5)) gam = 1.0;
    } else {
      done = 0.0;
    }
  }
  rs->gam = gam;
  rs->done = done;
  if (done != 0.0) rs->t += gam * dt;
}

// The sums at gam = 1 of an RK4 update q -> qrk, per block (the pair path; the step
// tile reduces them itself).
template <typename T>
__global__ __launch_bounds__(RED_THREADS) void relax_sums(const GridConst gc, const T* __restrict__ q,
                                                          const T* __restrict__ qrk, const T* __restrict__ bplane,
                                                          double* __restrict__ partials) {
  const int nx = gc.nx, ny = gc.ny;
  const size_t N = (size_t)nx * (size_t)ny;
  __shared__ double sh[RELAX_LDS];
  RelaxSums a;
  a.init();
  for (int j = blockIdx.x; j < ny; j += gridDim.x) {
    const double wy = axis_weight(j, ny, gc.bc_y, gc.dy);
    for (int i = threadIdx.x; i < nx; i += RED_THREADS) {
      const double M = axis_weight(i, nx, gc.bc_x, gc.dx) * wy;
      const size_t o = (size_t)j * nx + i;
      double x[5], dx[5];
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        x[f] = (double)q[f * N + o];
        dx[f] = (double)qrk[f * N + o] - x[f];
      }
      a.add(M, relax_node_terms(x, dx, (double)bplane[o], gc.g, gc.lam, 1.0));
    }
  }
  block_merge(a, sh);
  if (threadIdx.x == 0) a.put(partials + RELAX_PART * blockIdx.x);
}

// gam from the partial sums at gam = 1: block b merges partials [b per, (b + 1) per),
// the last block the blocks' results in order.
static __global__ __launch_bounds__(RED_THREADS) void relax_newton(const double* __restrict__ in, int n, int per,
                                                            double* __restrict__ out, RelaxScalars* __restrict__ rs,
                                                            double dt) {
  __shared__ double sh[RELAX_LDS];
  RelaxSums a;
  a.init();
  const int lo = blockIdx.x * per, hi = lo + per < n ? lo + per : n;
  for (int p = lo + threadIdx.x; p < hi; p += RED_THREADS) {
    RelaxSums o;
    o.get(in + (size_t)RELAX_PART * p);
    a.merge(o);
  }
  block_merge(a, sh);
  if (threadIdx.x == 0) a.put(out + RELAX_PART * blockIdx.x);
  if (!last_block(&rs->ticket)) return;
  a.init();
  for (int p = threadIdx.x; p < (int)gridDim.x; p += RED_THREADS) {
    RelaxSums o;
    o.get(out + RELAX_PART * p);
    a.merge(o);
  }
  __syncthreads();  // block_merge's LDS is used again
  block_merge(a, sh);
  if (threadIdx.x == 0) relax_root(a, rs, dt);
}

// The second iteration by a pass over the states, where the series was not enough:
// per-block compensated sums of s and s' at rs->gam, the last block makes the
// Newton update and advances the time by gam dt.
template <typename T>
__global__ __launch_bounds__(RED_THREADS) void relax_second(const GridConst gc, const T* __restrict__ q,
                                                            const T* __restrict__ qrk, const T* __restrict__ bplane,
                                                            RelaxScalars* __restrict__ rs,
                                                            double* __restrict__ partials, double dt) {
  if (rs->done != 0.0) return;
  const int nx = gc.nx, ny = gc.ny;
  const size_t N = (size_t)nx * (size_t)ny;
  const double gam = rs->gam;
  CSum a[2];
  a[0].init();
  a[1].init();
  for (int j = blockIdx.x; j < ny; j += gridDim.x) {
    const double wy = axis_weight(j, ny, gc.bc_y, gc.dy);
    for (int i = threadIdx.x; i < nx; i += RED_THREADS) {
      const double M = axis_weight(i, nx, gc.bc_x, gc.dx) * wy;
      const size_t o = (size_t)j * nx + i;
      double x[5], dx[5];
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        x[f] = (double)q[f * N + o];
        dx[f] = (double)qrk[f * N + o] - x[f];
      }
      const RelaxTerms t = relax_node_terms(x, dx, (double)bplane[o], gc.g, gc.lam, gam);
      a[0].add(M * t.s);
      a[1].add(M * t.ds);
    }
  }
  block_merge<2>(a);
  if (threadIdx.x == 0) {
    partials[4 * blockIdx.x + 0] = a[0].s;
    partials[4 * blockIdx.x + 1] = a[0].c;
    partials[4 * blockIdx.x + 2] = a[1].s;
    partials[4 * blockIdx.x + 3] = a[1].c;
  }
  if (!last_block(&rs->ticket)) return;
  a[0].init();
  a[1].init();
  for (int p = threadIdx.x; p < (int)gridDim.x; p += RED_THREADS) {
    a[0].merge(partials[4 * p + 0], partials[4 * p + 1]);
    a[1].merge(partials[4 * p + 2], partials[4 * p + 3]);
  }
  __syncthreads();
  block_merge<2>(a);
  if (threadIdx.x == 0) {
    const double next = relax_next(gam, a[0].s + a[0].c, a[1].s + a[1].c);
    rs->gam = next;
    rs->t += next * dt;
  }
}

// The scalars at the start of a relaxation run from time t0.
static __global__ void relax_start(RelaxScalars* __restrict__ rs, double t0) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *rs = RelaxScalars{1.0, t0, 0.0, 0, 0};
}

// out <- q + gam (q_RK4 - q), elementwise over the five planes (out may be q).
template <typename T>
__global__ __launch_bounds__(256) void relax_update(size_t n5, T* out, const T* q, const T* __restrict__ qrk,
                                                    const RelaxScalars* __restrict__ rs) {
  const size_t k = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (k >= n5) return;
  const T gam = T(rs->gam);
  const T x = q[k];
  out[k] = fused(gam, qrk[k] - x, x);
}

// One RK4 step of a relaxation run after its first: the step tile stages the
// relaxed state of the previous step, qa + gam (ra - qa), writes it out for
// its owned nodes (qbase) beside the RK4 result (qout), and reduces the sums at
// gam = 1 per tile (EPI_RELAX), so no update pass runs between the steps.
template <typename T, int BCX, int BCY, int TY>
__global__ __launch_bounds__(STAGE_THREADS) void relax_step_kernel(const GridConst gc, const T* __restrict__ qa,
                                                                   const T* __restrict__ bplane,
                                                                   T* __restrict__ qout, const RelaxIn<T> rx, T c6,
                                                                   T c3, T c2, T c1, double dt,
                                                                   int* __restrict__ flag,
                                                                   double* __restrict__ rpart) {
  constexpr int TX = StepGeom<TY>::TX;
  __shared__ StepSmem<T, TY, 1> s;
  const int ntx = (gc.nx + TX - 1) / TX;
  const int nty = (gc.ny + TY - 1) / TY;
  const int tile = xcd_tile(blockIdx.x, ntx * nty);
  step_tile<T, BCX, BCY, false, TY, false, 1, EPI_RELAX, RK_RELAXED>(
      s, gc, (tile % ntx) * TX, (tile / ntx) * TY, qa, bplane, qout, c6, c3, c2, c1, 0.0, dt, flag, nullptr,
      rpart + RELAX_PART * tile, nullptr, &rx);
}

}  // namespace sgn
