// sgn_fused.hpp -- one classical RK4 step in one kernel.
//
// Each workgroup owns a tile of TX x TY nodes (32 x 24 by default, or 32 x 16
// or 64 x 8) and stages the state q with a four-node halo of
// (h, u, v, w, eta, b, e) in LDS, e = (eta - h)^2/h.  The four right-hand
// sides of the step are evaluated on shrinking regions, since each evaluation
// reaches one node further than the stage it reads:
//   k1 = f(q)   on the tile and the rings at distance 1..3,  Y2 = q + dt/2 k1
//   k2 = f(Y2)  on the tile and the rings at distance 1..2,  Y3 = q + dt/2 k2
//   k3 = f(Y3)  on the tile and the ring at distance 1,      Y4 = q + dt k3
//   k4 = f(Y4)  on the tile:  q_new = acc + dt/6 k4,
// with acc = q + dt/6 k1 + dt/3 k2 + dt/3 k3 kept in registers for the owned
// nodes.  Each intermediate stage overwrites the previous one in LDS (b is
// kept).  Only q and b are read and q_new written: 11 values per node and
// step from HBM, against 37 for the two pair kernels and 84 for four stage
// kernels.  The price is the ring evaluations: 1.24 right-hand sides per owned
// node and stage for a 32 x 24 tile, 1.31 for 32 x 16 and 1.42 for 64 x 8.
//
// Thread map: thread t owns the NO = TX TY / 256 tile nodes
// (t mod TX, NO floor(t / TX) + k), k < NO (three for 32 x 24, two for the
// others), in every stage, so their q and acc stay in registers (and, see KEEP,
// their current stage); each node
// shares y-neighbours with the one below it.  Ring nodes are numbered by distance (all of
// ring 1 first, then ring 2, then ring 3); thread t evaluates ring nodes t and
// t + 256 in every stage whose region contains them, so the q of a ring node is
// read from LDS once, in the first stage.
//
// The output buffer must not alias the input (neighbouring tiles read the
// halo of q); sgn_step alternates between the caller's buffer and the
// context's accumulator buffer.
//
// What bounds it: the FP64 (FP32) vector pipe with two workgroups per CU, then
// what those two leave uncovered of staging and barriers.  4096^2 periodic, 32 x 24:
// FP64 701 us with a plane per value and 126 operations a node, 615 us with the
// rates in two-point form, 602 us with 16-byte LDS vectors (a stage's reads took
// half the LDS cycles); FP32 357 and 324 us.
#pragma once

#include "sgn_pair.hpp"
#include "sgn_reduce.hpp"

namespace sgn {

constexpr int STEP_HALO = 4;  // one node per right-hand side of the step

// Tile shapes of the step kernel: TX x TY with TY = 24 (32 wide, three owned
// nodes per thread), 16 (32 wide) or 8 (64 wide; both two per thread).
template <int TY_>
struct StepGeom {
  static constexpr int TY = TY_;
  static constexpr int TX = TY == 8 ? 64 : 32;
  static constexpr int NO = TX * TY / STAGE_THREADS;  // owned nodes per thread
  static constexpr int RX = TX + 2 * STEP_HALO;
  static constexpr int RY = TY + 2 * STEP_HALO;
  // nodes of the ring at distance d around the tile
  static constexpr int ring(int d) { return 2 * (TX + 2 * d) + 2 * (TY + 2 * d - 2); }
  static constexpr int RING1 = ring(1);
  static constexpr int RING2 = RING1 + ring(2);
  static constexpr int RING3 = RING2 + ring(3);
  static_assert(TY == 8 || TY == 16 || TY == 24, "tile shapes 64 x 8, 32 x 16, 32 x 24");
  static_assert(NO * STAGE_THREADS == TX * TY && (NO == 2 || NO == 3), "two or three owned nodes per thread");
  static_assert(RING3 <= 2 * STAGE_THREADS, "two ring slots per thread");
};

// Rows are padded to an odd number of elements (PAD = 1) so that the ring
// columns, which lanes read down a column, spread over the LDS banks.  The
// manufactured-source instantiations (the heaviest, with the source evaluated
// inline) keep unpadded rows (PAD = 0): their reflecting variant returned wrong
// values near the x-walls with padded rows, a failure not explained by the
// source; unpadded they agree bit for bit with the four-stage path.
template <typename T, int TY, int PAD>
struct StepSmem;

typedef double sgn_d2 __attribute__((ext_vector_type(2)));
typedef float sgn_f4 __attribute__((ext_vector_type(4)));

template <int TY, int PAD>
struct StepSmem<double, TY, PAD> {
  static constexpr int RY = StepGeom<TY>::RY, P = StepGeom<TY>::RX + PAD;
  sgn_d2 a[3][RY][P];  // (h, u), (v, w), (eta, e) of the current stage
  double b[RY][P];
  __device__ __forceinline__ Node<double> load(int r, int c) const {
    const sgn_d2 x = a[0][r][c], y = a[1][r][c], z = a[2][r][c];
    return Node<double>{x.x, x.y, y.x, y.y, z.x, b[r][c], z.y};
  }
  // everything but b (`bb`: the node's b, unused here)
  __device__ __forceinline__ void store(int r, int c, const double (&y)[5], double e, double) {
    a[0][r][c] = sgn_d2{y[0], y[1]};
    a[1][r][c] = sgn_d2{y[2], y[3]};
    a[2][r][c] = sgn_d2{y[4], e};
  }
  __device__ __forceinline__ void store_b(int r, int c, double bb) { b[r][c] = bb; }
};

template <int TY, int PAD>
struct StepSmem<float, TY, PAD> {
  static constexpr int RY = StepGeom<TY>::RY, P = StepGeom<TY>::RX + PAD;
  sgn_f4 a[2][RY][P];  // (h, u, v, w), (eta, e, b, unused) of the current stage
  __device__ __forceinline__ Node<float> load(int r, int c) const {
    const sgn_f4 x = a[0][r][c], y = a[1][r][c];
    return Node<float>{x.x, x.y, x.z, x.w, y.x, y.z, y.y};
  }
  __device__ __forceinline__ void store(int r, int c, const float (&y)[5], float e, float bb) {
    a[0][r][c] = sgn_f4{y[0], y[1], y[2], y[3]};
    a[1][r][c] = sgn_f4{y[4], e, bb, 0.0f};
  }
  __device__ __forceinline__ void store_b(int, int, float) {}
};

// Which Runge-Kutta method a step tile runs.  RK_CLASSIC: one classical RK4
// step from q.  RK_FSAL: evaluations 2 to 5 of one attempt of the adaptive
// five-stage pair (sgn_fsal.hpp): the tile stages Y_2 = y + h c_2 k_1 (from
// the input y and the attempt's k_1), evaluates k_2 .. k_5 on the shrinking
// regions, and writes y_{n+1} = y + h (b_1 k_1 + ... + b_5 k_5) and the partial
// error estimate e' = h b_5 (k_5 - (1 - c_5) k_1) of the owned nodes.  The
// tile first stages y, from which the owned and ring nodes keep their y in
// registers (as the classical step keeps q), then overwrites it with Y_2; k_1
// of the owned nodes is read again from global memory (L2).
// RK_RELAXED: one classical RK4 step from the relaxed state of the previous
// relaxation step, q = qa + gam (ra - qa), formed while staging (the arithmetic
// of relax_update, so the same bits), which the tile also writes out for its
// owned nodes (RelaxIn).
enum : int { RK_CLASSIC = 0, RK_FSAL = 1, RK_RELAXED = 2 };

// Operands of an RK_RELAXED tile: q (the step's input pointer) is qa.
template <typename T>
struct RelaxIn {
  const T* ra;             // the previous step's RK4 result
  const double* rs;        // gam of the previous step
  T* qbase;                // out: the relaxed state of the owned nodes
};

// Coefficients and extra operands of an RK_FSAL tile (h already applied).
template <typename T>
struct FsalStage {
  const T* k1;  // k_1 of the attempt
  T* e;         // out: e' of the owned nodes
  T cin;        // h c_2
  T c1a;        // h b_1
  T cy[3];      // evaluation s = k_{s+1}: Y_{s+2} = y + cy[s-1] k_{s+1}  (s = 1, 2, 3)
  T ca[4];      // acc += ca[s-1] k_{s+1}                                  (s = 1 .. 4)
  T ce1;        // h b_5 (1 - c_5)
};

// Position (r, c), relative to the tile origin, of ring node m (0 <= m < RING3).
template <int TY>
__device__ __forceinline__ void ring_node(int m, int& r, int& c) {
  using G = StepGeom<TY>;
  constexpr int TX = G::TX;
  int d;
  if (m < G::RING1) {
    d = 1;
  } else if (m < G::RING2) {
    d = 2;
    m -= G::RING1;
  } else {
    d = 3;
    m -= G::RING2;
  }
  const int w = TX + 2 * d;          // top and bottom rows
  const int hs = G::TY + 2 * d - 2;  // left and right columns without the corners
  if (m < w) {
    r = -d;
    c = m - d;
  } else if (m < 2 * w) {
    r = G::TY - 1 + d;
    c = m - w - d;
  } else if (m < 2 * w + hs) {
    r = m - 2 * w - d + 1;
    c = -d;
  } else {
    r = m - 2 * w - hs - d + 1;
    c = TX - 1 + d;
  }
}

// KEEP: the owned nodes' current stage Y and its 1/h stay in registers from stage
// to stage, so that LDS gives them only the nodes around the column of NO (one
// above, one below, two beside each), two thirds of the reads.  Without KEEP they
// read their centres back: where the registers would pass 256 (the adaptive attempt;
// and, by their callers' choice, the FP64 ensemble kernels, which hold all four
// boundary variants, and gauge rollouts on 32 x 24 tiles with a wall; a 4096^2 step
// on 32 x 24 tiles with walls took 900 us with KEEP and 640 without).
template <typename T, int RK>
constexpr bool step_keeps() {
  return sizeof(T) == 4 || RK != RK_FSAL;
}

// One tile (origin i0, j0) of one RK4 step, executed by a whole workgroup.
// SAVE (the adjoint's recomputation): also write the intermediate stages
// Y2, Y3, Y4 of the owned nodes to ysave, three consecutive states.
// EPI (EPI_RELAX or EPI_TOTALS): also reduce the tile's sums (see the enum;
// from the step's input and output values held in registers) into rpart.
// The caller synchronizes the workgroup before reusing `s` for another tile.
// RK = RK_FSAL (no source, no stage saving, no epilogue): q is the attempt's
// y_n, qout receives y_{n+1}, *fx supplies k_1, the coefficients and the e'
// output; c6 .. c1, t0, dt and flag are unused (the health of y_{n+1} is
// checked by the attempt's FSAL evaluation).
template <typename T, int BCX, int BCY, bool SRC, int TY, bool SAVE, int PAD, int EPI = EPI_NONE,
          int RK = RK_CLASSIC, bool KEEP = step_keeps<T, RK>(), int FORM = FORM_SHARED>
__device__ __forceinline__ void step_tile(StepSmem<T, TY, PAD>& s, const GridConst& gc, int i0, int j0,
                                          const T* __restrict__ q, const T* __restrict__ bplane,
                                          T* __restrict__ qout, T c6, T c3, T c2, T c1, double t0, double dt,
                                          int* __restrict__ flag, T* __restrict__ ysave,
                                          double* __restrict__ rpart = nullptr,
                                          const FsalStage<T>* __restrict__ fx = nullptr,
                                          const RelaxIn<T>* __restrict__ rx = nullptr) {
  static_assert(RK != RK_FSAL || (!SRC && !SAVE && EPI == EPI_NONE), "the FSAL tile has no extras");
  static_assert(RK != RK_RELAXED || (!SRC && !SAVE), "the relaxed tile has no source or stage saving");
  using G = StepGeom<TY>;
  constexpr int TX = G::TX, NO = G::NO, NR = 2;
  constexpr int RX = G::RX;
  constexpr int REGION = G::RX * G::RY;

  const int nx = gc.nx, ny = gc.ny;
  const size_t N = (size_t)nx * (size_t)ny;
  const int tid = threadIdx.x;

  // 1. Stage q and b with the four-node halo (periodic wrap or wall clamp).
  //    Every load of the region is issued before the first one is waited
  //    for: the step kernel reads little per unit of work, so its bandwidth
  //    is set by how many bytes each workgroup keeps in flight.
  constexpr int NF = RK == RK_FSAL ? 1 : 0;
  T yown[NF ? NO : 1][5], yring[NF ? NR : 1][5];  // RK_FSAL: y of the owned and ring nodes
  {
    constexpr int ITER = (REGION + STAGE_THREADS - 1) / STAGE_THREADS;
    T v[ITER][6];
    T kst[RK != RK_CLASSIC ? ITER : 1][5];
    // The staging waves take the issue priority until the barrier: their loads
    // and LDS writes go out ahead of the other workgroup's evaluation on the
    // same SIMDs (measured: FP32 2% and FP64 0.3-0.5% faster, same bits).
    __builtin_amdgcn_s_setprio(3);
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      const int idx = tid + it * STAGE_THREADS;
      if (idx < REGION) {
        const int rr = idx / RX;
        const int cc = idx - rr * RX;
        const int gi = wrap_or_clamp<BCX>(i0 - STEP_HALO + cc, nx);
        const int gj = wrap_or_clamp<BCY>(j0 - STEP_HALO + rr, ny);
        const size_t o = (size_t)gj * nx + gi;
#pragma unroll
        for (int f = 0; f < 5; ++f) v[it][f] = q[f * N + o];
        v[it][5] = bplane[o];
        if constexpr (RK == RK_FSAL) {
#pragma unroll
          for (int f = 0; f < 5; ++f) kst[it][f] = fx->k1[f * N + o];
        }
        if constexpr (RK == RK_RELAXED) {
#pragma unroll
          for (int f = 0; f < 5; ++f) kst[it][f] = rx->ra[f * N + o];
        }
      }
    }
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      const int idx = tid + it * STAGE_THREADS;
      if (idx < REGION) {
        const int rr = idx / RX;
        const int cc = idx - rr * RX;
        if constexpr (RK == RK_RELAXED) {
          const T gam = T(rx->rs[0]);
#pragma unroll
          for (int f = 0; f < 5; ++f) v[it][f] = fused(gam, kst[it][f] - v[it][f], v[it][f]);
        }
        s.store_b(rr, cc, v[it][5]);
        const T y[5] = {v[it][0], v[it][1], v[it][2], v[it][3], v[it][4]};
        s.store(rr, cc, y, RK == RK_FSAL ? T(0) : node_extra<FORM>(y[0], y[4], recip_staged(y[0])), v[it][5]);
      }
    }
    if constexpr (RK == RK_FSAL) {
      __syncthreads();
      // LDS holds y: the owned and ring nodes take their y from it (the ring's
      // periodic images and clamped wall copies included), then Y_2 =
      // y + h c_2 k_1 and its e replace it
      const int lx_ = tid % TX, ly_ = NO * (tid / TX);
#pragma unroll
      for (int k = 0; k < NO; ++k) {
        {
          const Node<T> n = s.load(ly_ + k + STEP_HALO, lx_ + STEP_HALO);
          yown[k][0] = n.h, yown[k][1] = n.u, yown[k][2] = n.v, yown[k][3] = n.w, yown[k][4] = n.eta;
        }
      }
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        const int m = tid + k * STAGE_THREADS;
        if (m < G::RING3) {
          int r_, c_;
          ring_node<TY>(m, r_, c_);
          const Node<T> n = s.load(r_ + STEP_HALO, c_ + STEP_HALO);
          yring[k][0] = n.h, yring[k][1] = n.u, yring[k][2] = n.v, yring[k][3] = n.w, yring[k][4] = n.eta;
        }
      }
      __syncthreads();
#pragma unroll
      for (int it = 0; it < ITER; ++it) {
        const int idx = tid + it * STAGE_THREADS;
        if (idx < REGION) {
          const int rr = idx / RX;
          const int cc = idx - rr * RX;
          T y2[5];
#pragma unroll
          for (int f = 0; f < 5; ++f) {
            y2[f] = fused(fx->cin, kst[it][f], v[it][f]);
          }
          s.store(rr, cc, y2, node_e(y2[0], y2[4], recip_staged(y2[0])), v[it][5]);
        }
      }
    }
  }

  __builtin_amdgcn_s_setprio(0);
  // Owned nodes (lx, ly0 + k), k < NO, and ring slots of this thread.
  const int lx = tid % TX;
  const int ly0 = NO * (tid / TX);
  const int i = i0 + lx;
  bool own_dom[NO];
#pragma unroll
  for (int k = 0; k < NO; ++k) {
    const int j = j0 + ly0 + k;
    own_dom[k] = on_axis<BCX>(i, nx) && on_axis<BCY>(j, ny);
  }
  int ring_r[NR], ring_c[NR];
  bool ring_ok[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    const int m = tid + k * STAGE_THREADS;
    ring_r[k] = 0;
    ring_c[k] = 0;
    ring_ok[k] = false;
    if (m < G::RING3) {
      ring_node<TY>(m, ring_r[k], ring_c[k]);
      ring_ok[k] = on_axis<BCX>(i0 + ring_c[k], nx) && on_axis<BCY>(j0 + ring_r[k], ny);
    }
  }
  __syncthreads();

  // ihr: 1/h of the ring nodes' current stage
  Node<T> Y[NO];
  T ih[NO], ihr[NR];
  T qo[NO][5], acc[NO][5], qr[NR][5];
#pragma unroll
  for (int k = 0; k < NO; ++k) {
    if (KEEP) {
      Y[k] = s.load(ly0 + k + STEP_HALO, lx + STEP_HALO);
      ih[k] = recip_staged(Y[k].h);
    }
    if constexpr (RK == RK_FSAL) {
#pragma unroll
      for (int f = 0; f < 5; ++f) qo[k][f] = yown[k][f];
    }
  }
  if constexpr (RK == RK_FSAL) {
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      if (tid + k * STAGE_THREADS < G::RING3) {
#pragma unroll
        for (int f = 0; f < 5; ++f) qr[k][f] = yring[k][f];
      }
    }
  }
  int health = 0;
  CSum rsum[2];
  RelaxSums xsum;
  if (EPI == EPI_TOTALS) {
    rsum[0].init();
    rsum[1].init();
  }
  if (EPI == EPI_RELAX) xsum.init();
#pragma unroll
  for (int st = 1; st <= 4; ++st) {
    T cy = st == 3 ? c1 : c2;             // Y_{st+1} = q + cy k_st
    T ca = st == 1 || st == 4 ? c6 : c3;  // acc += ca k_st
    if constexpr (RK == RK_FSAL) {
      cy = st < 4 ? fx->cy[st - 1] : T(0);
      ca = fx->ca[st - 1];
    }
    const double ts = t0 + (st == 1 ? 0.0 : (st == 4 ? dt : 0.5 * dt));
    const int ring_lim = st == 1 ? G::RING3 : (st == 2 ? G::RING2 : G::RING1);
    // Owned nodes, upwards: node k's lower neighbour is node k - 1 (its stage
    // before this evaluation replaced it), its upper neighbour node k + 1.
    const AxisStencil<BCX> ax(i, nx, gc.inv2dx, gc.invdx);
    Node<T> below, above;
#pragma unroll
    for (int k = 0; k < NO; ++k) {
      __builtin_amdgcn_sched_barrier(0);
      const int j = j0 + ly0 + k;
      const bool run = st < 4 ? own_dom[k] : (i < nx && j < ny);
      if (!run) continue;
      int r = ly0 + k + STEP_HALO;
      const int c = lx + STEP_HALO;
      // the printed terms take more registers than sharing the column's nodes leaves
      // them: each is read anew, at a row that the compiler cannot tell
      constexpr bool ANEW = FORM == FORM_TERMS && !KEEP;
      if (ANEW) asm volatile("" : "+v"(r));
      const AxisStencil<BCY> ay(j, ny, gc.inv2dy, gc.invdy);
      const Node<T> cn = KEEP ? Y[k] : (k == 0 || ANEW ? s.load(r, c) : above);
      const Node<T> xm = s.load(r, c + ax.om);
      const Node<T> xp = s.load(r, c + ax.op);
      Node<T> dn, up;
      if (k == 0 || ANEW) {
        dn = s.load(r + ay.om, c);
      } else {
        dn = below;  // j > 0 here
      }
      if (k == NO - 1 || !KEEP) {
        up = s.load(r + ay.op, c);
        above = up;
      } else {
        up = Y[k + 1];
        if (BCY == BC_REFLECTING && j == ny - 1) up = cn;
      }
      below = cn;
      const size_t o = (size_t)j * nx + i;
      if constexpr (RK != RK_FSAL) {
        if (st == 1) {
          qo[k][0] = cn.h;
          qo[k][1] = cn.u;
          qo[k][2] = cn.v;
          qo[k][3] = cn.w;
          qo[k][4] = cn.eta;
          if constexpr (RK == RK_RELAXED) {
            if (i < nx && j < ny) {
#pragma unroll
              for (int f = 0; f < 5; ++f) rx->qbase[f * N + o] = qo[k][f];
            }
          }
        }
      }
      T k1o[5];  // RK_FSAL: k_1 of the node, read (from L2) where it is used
      if constexpr (RK == RK_FSAL) {
        if (st == 1 || st == 4) {
          const size_t ow = (size_t)wrap_or_clamp<BCY>(j, ny) * nx + wrap_or_clamp<BCX>(i, nx);
#pragma unroll
          for (int f = 0; f < 5; ++f) k1o[f] = fx->k1[f * N + ow];
        }
      }
      const Rates<T> kk = node_rates<T, BCX, BCY, SRC, FORM>(cn, KEEP ? ih[k] : recip_staged(cn.h), xm, xp, dn, up, ax,
                                                             ay, i, j, gc, ts);
      const T kv[5] = {kk.h, kk.u, kk.v, kk.w, kk.eta};
      if (st < 4) {
#pragma unroll
        for (int f = 0; f < 5; ++f) {
          T a = qo[k][f];
          if constexpr (RK == RK_FSAL) {
            if (st == 1) a = fused(fx->c1a, k1o[f], a);
          }
          acc[k][f] = fused(ca, kv[f], st == 1 ? a : acc[k][f]);
        }
        Y[k].h = fused(cy, kv[0], qo[k][0]);
        Y[k].u = fused(cy, kv[1], qo[k][1]);
        Y[k].v = fused(cy, kv[2], qo[k][2]);
        Y[k].w = fused(cy, kv[3], qo[k][3]);
        Y[k].eta = fused(cy, kv[4], qo[k][4]);
        Y[k].b = cn.b;
        if (KEEP) {
          ih[k] = recip_staged(Y[k].h);
          Y[k].e = node_extra<FORM>(Y[k].h, Y[k].eta, ih[k]);
        }
        if (SAVE && i < nx && j < ny) {
          T* ys = ysave + (size_t)(st - 1) * 5 * N + o;
          ys[0] = Y[k].h;
          ys[N] = Y[k].u;
          ys[2 * N] = Y[k].v;
          ys[3 * N] = Y[k].w;
          ys[4 * N] = Y[k].eta;
        }
      } else {
        T nv[5];
#pragma unroll
        for (int f = 0; f < 5; ++f) {
          nv[f] = fused(ca, kv[f], acc[k][f]);
          qout[f * N + o] = nv[f];
        }
        if constexpr (RK == RK_FSAL) {
#pragma unroll
          for (int f = 0; f < 5; ++f) fx->e[f * N + o] = fused(-fx->ce1, k1o[f], ca * kv[f]);
        } else {
          if (!(nv[0] > T(0))) health |= FLAG_NONPOS;
          const T sum = nv[0] + nv[1] + nv[2] + nv[3] + nv[4];
          if (!isfinite(sum)) health |= FLAG_NONFINITE;
        }
        if (EPI == EPI_TOTALS) {
          const double M = axis_weight(i, nx, gc.bc_x, gc.dx) * axis_weight(j, ny, gc.bc_y, gc.dy);
          rsum[0].add(M * (double)nv[0]);
          rsum[1].add(M * energy_density((double)nv[0], (double)nv[1], (double)nv[2], (double)nv[3], (double)nv[4],
                                         (double)cn.b, gc.g, gc.lam));
        }
        if (EPI == EPI_RELAX) {
          double x[5], d[5];
#pragma unroll
          for (int f = 0; f < 5; ++f) {
            x[f] = (double)qo[k][f];
            d[f] = (double)nv[f] - x[f];
          }
          const double M = axis_weight(i, nx, gc.bc_x, gc.dx) * axis_weight(j, ny, gc.bc_y, gc.dy);
          xsum.add(M, relax_node_terms(x, d, (double)cn.b, gc.g, gc.lam, 1.0));
        }
      }
    }
    if (st == 4) break;
    // ring nodes inside this stage's region
    T rr[NR][5], re[NR], rb[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      __builtin_amdgcn_sched_barrier(0);
      const int m = tid + k * STAGE_THREADS;
      if (m >= ring_lim || !ring_ok[k]) continue;
      const int r = ring_r[k] + STEP_HALO, c = ring_c[k] + STEP_HALO;
      const AxisStencil<BCX> axr(i0 + ring_c[k], nx, gc.inv2dx, gc.invdx);
      const AxisStencil<BCY> ayr(j0 + ring_r[k], ny, gc.inv2dy, gc.invdy);
      const Node<T> cn = s.load(r, c);
      if (st == 1) {
        if (KEEP) ihr[k] = recip_staged(cn.h);
        if constexpr (RK != RK_FSAL) {
          qr[k][0] = cn.h;
          qr[k][1] = cn.u;
          qr[k][2] = cn.v;
          qr[k][3] = cn.w;
          qr[k][4] = cn.eta;
        }
      }
      const Node<T> xm = s.load(r, c + axr.om);
      const Node<T> xp = s.load(r, c + axr.op);
      const Node<T> dn = s.load(r + ayr.om, c);
      const Node<T> up = s.load(r + ayr.op, c);
      const Rates<T> kk =
          node_rates<T, BCX, BCY, SRC, FORM>(cn, KEEP ? ihr[k] : recip_staged(cn.h), xm, xp, dn, up, axr, ayr,
                                             i0 + ring_c[k], j0 + ring_r[k], gc, ts);
      const T kv[5] = {kk.h, kk.u, kk.v, kk.w, kk.eta};
#pragma unroll
      for (int f = 0; f < 5; ++f) rr[k][f] = fused(cy, kv[f], qr[k][f]);
      if (KEEP) {
        ihr[k] = recip_staged(rr[k][0]);
        re[k] = node_extra<FORM>(rr[k][0], rr[k][4], ihr[k]);
      }
      rb[k] = cn.b;
    }
    __syncthreads();
    // the stage just formed replaces the one read
#pragma unroll
    for (int k = 0; k < NO; ++k) {
      if (!own_dom[k]) continue;
      const int r = ly0 + k + STEP_HALO, c = lx + STEP_HALO;
      const T y[5] = {Y[k].h, Y[k].u, Y[k].v, Y[k].w, Y[k].eta};
      s.store(r, c, y, KEEP ? Y[k].e : node_extra<FORM>(y[0], y[4], recip_staged(y[0])), Y[k].b);
    }
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      const int m = tid + k * STAGE_THREADS;
      if (m >= ring_lim || !ring_ok[k]) continue;
      const int r = ring_r[k] + STEP_HALO, c = ring_c[k] + STEP_HALO;
      s.store(r, c, rr[k], KEEP ? re[k] : node_extra<FORM>(rr[k][0], rr[k][4], recip_staged(rr[k][0])), rb[k]);
    }
    __syncthreads();
  }
  if constexpr (RK != RK_FSAL) {
    if (health) atomicOr(flag, health);
  }
  if (EPI == EPI_RELAX) {
    static_assert(sizeof(s) >= RELAX_LDS * sizeof(double), "the staging serves the reduction");
    __syncthreads();  // of the staging, no longer read
    block_merge(xsum, (double*)&s);
    if (tid == 0) xsum.put(rpart);
  }
  if (EPI == EPI_TOTALS) {
    block_merge<2>(rsum);
    if (tid == 0) {
      rpart[0] = rsum[0].s;
      rpart[1] = rsum[0].c;
      rpart[2] = rsum[1].s;
      rpart[3] = rsum[1].c;
    }
  }
}

// EPI != EPI_NONE: rpart holds epi_part(EPI) doubles per tile, in tile order.
template <typename T, int BCX, int BCY, bool SRC, int TY, bool SAVE = false, int EPI = EPI_NONE>
__global__ __launch_bounds__(STAGE_THREADS) void step_kernel(const GridConst gc, const T* __restrict__ q,
                                                             const T* __restrict__ bplane, T* __restrict__ qout,
                                                             T c6, T c3, T c2, T c1, double t0, double dt,
                                                             int* __restrict__ flag, T* __restrict__ ysave,
                                                             double* __restrict__ rpart) {
  constexpr int TX = StepGeom<TY>::TX;
  __shared__ StepSmem<T, TY, SRC ? 0 : 1> s;
  const int ntx = (gc.nx + TX - 1) / TX;
  const int nty = (gc.ny + TY - 1) / TY;
  const int tile = xcd_tile(blockIdx.x, ntx * nty);
  step_tile<T, BCX, BCY, SRC, TY, SAVE, SRC ? 0 : 1, EPI>(s, gc, (tile % ntx) * TX, (tile / ntx) * TY, q, bplane,
                                                          qout, c6, c3, c2, c1, t0, dt, flag, ysave,
                                                          EPI != EPI_NONE ? rpart + epi_part(EPI) * tile : nullptr);
}

}  // namespace sgn
