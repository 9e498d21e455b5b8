// sgn_march.hpp -- one classical RK4 step in one kernel, one wave per strip.
//
// A wave owns a strip of MARCH_COLS columns and marches over its rows.  Lane l
// holds column i0 - 4 + l (64 lanes: the strip and its four-node halo), and the
// four stages of the step follow each other one row apart: with row R just
// loaded, stage 1 evaluates row R - 1, stage 2 row R - 2, stage 3 row R - 3 and
// stage 4 row R - 4, whose q_new is stored.  An evaluation needs three rows of
// its stage: the one above is the previous stage's result of this very step (in
// registers), the one below was the middle one a step ago (in registers), and
// the middle one lies in an LDS row of the wave's own, where the lanes find
// their x-neighbours.  Nothing is shared between waves, so there is no barrier,
// and the loads of row R + 1 are in flight during the whole step of row R.
//
// What bounds it: the FP64 (FP32) vector pipe, and the power budget behind it.
// Each row costs 4 evaluations in 64 lanes for 56 owned columns (1.14) and a
// strip of H rows 12 / (4 H) more for the rows below and above it; the tile
// kernel (step_kernel) evaluates 1.24 .. 1.31 right-hand sides per node, waits
// at seven barriers and for its staging.  The tile kernel stays the better one
// where a grid gives too few strips of useful height (march_plan).  Step of
// 4096^2, tile kernel and this one: FP64 periodic 602 and 463 us, FP32 324 and
// 257 us; FP64 with walls 687 (the tile kernel of the time) and 579 us; 2048^2
// FP64 155 and 136 us, 1024^2 42.5 and 41 us.  The chip lowers its clock to 1.8 ..
// 1.95 GHz under it.
//
// Registers decide the layout (FP64, two waves per SIMD: 256).  Rows below the
// middle (4 x 6 values), the accumulators q + dt (...) of the rows in flight (15),
// q of row R - 3 (5), 1/h of the middle rows (4) and the row being loaded (6) stay
// in registers; the middle rows are read back from LDS, which costs three 16-byte
// reads and saves 24 values.  Where more is needed (walls beside the strip, the
// totals epilogue) the last accumulator and q of row R - 3 move to LDS too (HOLD).
#pragma once

#include <type_traits>

#include "sgn_fused.hpp"

namespace sgn {

constexpr int MARCH_LANES = 64;
constexpr int MARCH_COLS = MARCH_LANES - 2 * STEP_HALO;  // columns a strip owns

// One row of a stage in LDS, one pad column at each end (read by the outermost
// lanes, whose values are never used).
template <typename T>
struct MarchLds;

template <>
struct MarchLds<double> {
  sgn_d2 a[3][MARCH_LANES + 2];
  double b[MARCH_LANES + 2];
  __device__ __forceinline__ Node<double> load(int c) const {
    const sgn_d2 x = a[0][c], y = a[1][c], z = a[2][c];
    return Node<double>{x.x, x.y, y.x, y.y, z.x, b[c], z.y};
  }
  __device__ __forceinline__ double load_b(int c) const { return b[c]; }
  __device__ __forceinline__ void store(int c, const Node<double>& n) {
    a[0][c] = sgn_d2{n.h, n.u};
    a[1][c] = sgn_d2{n.v, n.w};
    a[2][c] = sgn_d2{n.eta, n.e};
    b[c] = n.b;
  }
};

template <>
struct MarchLds<float> {
  sgn_f4 a[2][MARCH_LANES + 2];
  __device__ __forceinline__ Node<float> load(int c) const {
    const sgn_f4 x = a[0][c], y = a[1][c];
    return Node<float>{x.x, x.y, x.z, x.w, y.x, y.z, y.y};
  }
  __device__ __forceinline__ float load_b(int c) const { return a[1][c].z; }
  __device__ __forceinline__ void store(int c, const Node<float>& n) {
    a[0][c] = sgn_f4{n.h, n.u, n.v, n.w};
    a[1][c] = sgn_f4{n.eta, n.e, n.b, 0.0f};
  }
};

// Five values of each lane, kept in LDS from one step to the next.
template <typename T>
struct MarchHold;

template <>
struct MarchHold<double> {
  sgn_d2 a[2][MARCH_LANES];
  double b[MARCH_LANES];
  __device__ __forceinline__ void put(int l, const double (&y)[5]) {
    a[0][l] = sgn_d2{y[0], y[1]};
    a[1][l] = sgn_d2{y[2], y[3]};
    b[l] = y[4];
  }
  __device__ __forceinline__ void get(int l, double (&y)[5]) const {
    const sgn_d2 p = a[0][l], q = a[1][l];
    y[0] = p.x, y[1] = p.y, y[2] = q.x, y[3] = q.y, y[4] = b[l];
  }
};

template <>
struct MarchHold<float> {
  sgn_f4 a[MARCH_LANES];
  float b[MARCH_LANES];
  __device__ __forceinline__ void put(int l, const float (&y)[5]) {
    a[l] = sgn_f4{y[0], y[1], y[2], y[3]};
    b[l] = y[4];
  }
  __device__ __forceinline__ void get(int l, float (&y)[5]) const {
    const sgn_f4 p = a[l];
    y[0] = p.x, y[1] = p.y, y[2] = p.z, y[3] = p.w, y[4] = b[l];
  }
};

template <typename T>
struct MarchSmem {
  MarchLds<T>* row[4];  // the middle row of each stage
  T* b5;                // b of the row below stage 4's middle row
  MarchHold<T>* hold;   // two
};

// Access to a row at a scalar address: lanes add a 32-bit byte offset to it,
// where the compiler would otherwise keep a 64-bit address per plane in every
// lane.
#define SGN_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ T row_load(const T* p, unsigned off) {
  const SGN_GLOBAL char* g = (const SGN_GLOBAL char*)p;
  asm volatile("" : "+s"(g));
  return *(const SGN_GLOBAL T*)(g + off);
}
template <typename T>
__device__ __forceinline__ void row_store(T* p, unsigned off, T v) {
  SGN_GLOBAL char* g = (SGN_GLOBAL char*)p;
  asm volatile("" : "+s"(g));
  *(SGN_GLOBAL T*)(g + off) = v;
}

// A copy that the compiler takes for a new value: the offset has to be a 32-bit
// value of the block that uses it to be taken as one.
__device__ __forceinline__ unsigned local_copy(unsigned x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Orders the wave's own LDS accesses: the rows pass values between the lanes of
// one wave, whose LDS operations complete in order, so no instruction is needed,
// but the compiler must not move a lane's store above other lanes' loads of that
// slot (within one thread the addresses differ).
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T>
struct MarchRow {
  T h, u, v, w, eta, e;
};

template <typename T>
__device__ __forceinline__ Node<T> row_node(const MarchRow<T>& r, T b) {
  return Node<T>{r.h, r.u, r.v, r.w, r.eta, b, r.e};
}

template <typename T>
__device__ __forceinline__ MarchRow<T> node_row(const Node<T>& n) {
  return MarchRow<T>{n.h, n.u, n.v, n.w, n.eta, n.e};
}

// A wave's strip: columns [i0, i0 + MARCH_COLS) and rows [j0, j0 + nrows) of one
// RK4 step.  XW: a reflecting wall lies among the 64 columns; YW: the rows
// its stages evaluate reach a reflecting wall.  SAVE: also the stages Y2, Y3, Y4 to three
// consecutive states at ysave.  EPI_TOTALS: the strip's sums M h and M E of the
// state it writes (compensated) to rpart[0..3].
// Every load is wrapped or clamped into the grid; stores carry their own guard.
template <typename T, int BCX, int BCY, bool XW, bool YW, bool SAVE, int EPI>
__device__ __forceinline__ void march_strip(const MarchSmem<T>& s, const GridConst& gc, int i0, int j0, int nrows,
                                            const T* __restrict__ q, const T* __restrict__ bplane,
                                            T* __restrict__ qout, T c6, T c3, T c2, T c1, int* __restrict__ flag,
                                            T* __restrict__ ysave, double* __restrict__ rpart) {
  static_assert(EPI == EPI_NONE || EPI == EPI_TOTALS, "no other epilogue");
  constexpr bool HOLD_A = sizeof(T) == 8, HOLD_Q = HOLD_A && EPI == EPI_NONE && XW;
  constexpr int RX = XW ? BC_REFLECTING : BC_PERIODIC;
  const int nx = gc.nx, ny = gc.ny;
  const size_t N = (size_t)nx * (size_t)ny;
  const int lane = threadIdx.x;
  const int i = i0 - STEP_HALO + lane;
  const unsigned col = (unsigned)wrap_or_clamp<BCX>(i, nx) * (unsigned)sizeof(T);
  const bool own = lane >= STEP_HALO && lane < MARCH_LANES - STEP_HALO && i < nx;
  const int c = lane + 1;
  const T g = T(gc.g), lam = T(gc.lam);

  MarchRow<T> W[4] = {};  // the row below each stage's middle row
  T IH[4] = {};           // 1/h of each stage's middle row
  T q3[5] = {};           // q of row R - 3
  T acc[3][5] = {};       // accumulators of rows R - 2, R - 3, R - 4
  T pf[6];                // the row being loaded
  int health = 0;
  // the lane's sums, kept in LDS where q of row R - 3 might have gone (FP32: both holds)
  static_assert(EPI == EPI_NONE || sizeof(MarchHold<double>) <= (HOLD_A ? 1 : 2) * sizeof(MarchHold<T>),
                "the sums fit the LDS they take over");
  static_assert(alignof(MarchHold<T>) >= alignof(MarchHold<double>), "and its alignment");
  MarchHold<double>* const sums = (MarchHold<double>*)s.hold;
  if (EPI != EPI_NONE) sums->put(lane, {0.0, 0.0, 0.0, 0.0, 0.0});
  const auto fetch = [&](int row) {
    const size_t o = (size_t)wrap_or_clamp<BCY>(row, ny) * nx;
    const unsigned cl = local_copy(col);
#pragma unroll
    for (int f = 0; f < 5; ++f) pf[f] = row_load(q + f * N + o, cl);
    pf[5] = row_load(bplane + o, cl);
  };

  // The step of row R with the first NS stages at work (the others only pass b
  // on), a reflecting wall's rows recognized when W_ is set.
  const auto step = [&](auto ns, auto wall, int R) {
    constexpr int NS = decltype(ns)::value;
    constexpr bool WALL = decltype(wall)::value;
    constexpr int RY = WALL ? BC_REFLECTING : BC_PERIODIC;
    MarchRow<T> hi{pf[0], pf[1], pf[2], pf[3], pf[4], T(0)};
    T hib = pf[5];
    fetch(R + 1);
    T ihh = recip_staged(hi.h);
    hi.e = node_e(hi.h, hi.eta, ihh);
    T qlo[5] = {W[0].h, W[0].u, W[0].v, W[0].w, W[0].eta};  // q of row R - 2
    T accn[5];
#pragma unroll
    for (int st = 1; st <= 4; ++st) {
      if (st > NS) {  // pass on: this stage's newest row, if it has one, and b
        const Node<T> m = s.row[st - 1]->load(c);
        Node<T> n = st == NS + 1 ? row_node(hi, hib) : m;
        n.b = hib;
        W[st - 1] = node_row(m);
        if (st == NS + 1) {
          IH[st - 1] = ihh;
          if (st > 1) {
#pragma unroll
            for (int f = 0; f < 5; ++f) acc[st >= 2 ? st - 2 : 0][f] = accn[f];
          }
        }
        wave_order();
        s.row[st - 1]->store(c, n);
        if (st == 4) s.b5[c] = m.b;
        wave_order();
        hib = m.b;
        continue;
      }
      const int row = R - st;
      // formed anew for each evaluation: scale and wall term would take six registers
      const int iw = XW ? (int)local_copy((unsigned)i) : i;
      const AxisStencil<RX> ax(iw, nx, gc.inv2dx, gc.invdx);
      T satx = T(0);
      if (XW) {
        if (iw == 0) satx = T(-2.0 * gc.invdx);
        if (iw == nx - 1) satx = T(2.0 * gc.invdx);
      }
      T lob = st < 4 ? s.row[st & 3]->load_b(c) : s.b5[c];
      const Node<T> cn = s.row[st - 1]->load(c);
      const Node<T> xm = s.row[st - 1]->load(c + ax.om), xp = s.row[st - 1]->load(c + ax.op);
      if (HOLD_Q && st == 3) s.hold[0].get(lane, q3);
      if (HOLD_A && st == 3) s.hold[1].get(lane, acc[2]);
      const AxisStencil<RY> ay(row, ny, gc.inv2dy, gc.invdy);
      T saty = T(0);
      if (WALL) {  // the closure rows name the node itself beyond the wall
        if (row == 0) {
          W[st - 1] = node_row(cn);
          lob = cn.b;
          saty = T(-2.0 * gc.invdy);
        }
        if (row == ny - 1) {
          hi = node_row(cn);
          hib = cn.b;
          saty = T(2.0 * gc.invdy);
        }
      }
      const Node<T> dn = row_node(W[st - 1], lob), up = row_node(hi, hib);
      __builtin_amdgcn_sched_barrier(0);  // or the arithmetic is spread over more registers than there are
      const Rates<T> kk = split_form_rates<T, RX, RY>(cn, IH[st - 1], xm, xp, dn, up, T(ax.scale), T(ay.scale), g, lam,
                                                      satx, saty);
      const T kv[5] = {kk.h, kk.u, kk.v, kk.w, kk.eta};
      const T cy = st == 3 ? c1 : c2;             // Y_{st+1} = q + cy k_st
      const T ca = st == 1 || st == 4 ? c6 : c3;  // acc += ca k_st
      const bool mine = own && row >= j0 && row < j0 + nrows;
      const size_t o = (size_t)row * nx;
      MarchRow<T> yn;
      T ihn;
      if (st == 4) {
        T nv[5];
#pragma unroll
        for (int f = 0; f < 5; ++f) nv[f] = fused(ca, kv[f], acc[2][f]);
        if (mine) {
          const unsigned cl = local_copy(col);
#pragma unroll
          for (int f = 0; f < 5; ++f) row_store(qout + f * N + o, cl, nv[f]);
          if (!(nv[0] > T(0))) health |= FLAG_NONPOS;
          const T sum = nv[0] + nv[1] + nv[2] + nv[3] + nv[4];
          if (!isfinite(sum)) health |= FLAG_NONFINITE;
          if (EPI == EPI_TOTALS) {
            const double M = axis_weight(i, nx, gc.bc_x, gc.dx) * axis_weight(row, ny, gc.bc_y, gc.dy);
            double a[5];
            sums->get(lane, a);
            CSum m{a[0], a[1]}, e{a[2], a[3]};
            m.add(M * (double)nv[0]);
            e.add(M * energy_density((double)nv[0], (double)nv[1], (double)nv[2], (double)nv[3], (double)nv[4],
                                     (double)cn.b, gc.g, gc.lam));
            sums->put(lane, {m.s, m.c, e.s, e.c, 0.0});
          }
        }
        if (!HOLD_A) {
#pragma unroll
          for (int f = 0; f < 5; ++f) acc[2][f] = accn[f];
        }
      } else {
        const T qm[5] = {cn.h, cn.u, cn.v, cn.w, cn.eta};
        T y[5];
#pragma unroll
        for (int f = 0; f < 5; ++f) {
          const T qv = st == 1 ? qm[f] : st == 2 ? qlo[f] : q3[f];
          y[f] = fused(cy, kv[f], qv);
          const T a = fused(ca, kv[f], st == 1 ? qv : acc[st >= 2 ? st - 2 : 0][f]);
          if (st > 1) acc[st >= 2 ? st - 2 : 0][f] = accn[f];
          accn[f] = a;
        }
        if (HOLD_A && st == 3) s.hold[1].put(lane, accn);
        if (SAVE && mine) {
          const unsigned cl = local_copy(col);
#pragma unroll
          for (int f = 0; f < 5; ++f) row_store(ysave + ((size_t)(st - 1) * 5 + f) * N + o, cl, y[f]);
        }
        yn = MarchRow<T>{y[0], y[1], y[2], y[3], y[4], T(0)};
        ihn = recip_staged(yn.h);
        yn.e = node_e(yn.h, yn.eta, ihn);
      }
      W[st - 1] = node_row(cn);
      IH[st - 1] = ihh;
      wave_order();
      s.row[st - 1]->store(c, row_node(hi, hib));
      if (st == 4) s.b5[c] = cn.b;
      wave_order();
      hib = cn.b;
      if (st < 4) {
        hi = yn;
        ihh = ihn;
      }
    }
    // q of row R - 2 is the next step's q of row R - 3
    if (HOLD_Q) {
      s.hold[0].put(lane, qlo);
    } else {
#pragma unroll
      for (int f = 0; f < 5; ++f) q3[f] = qlo[f];
    }
  };

  const std::integral_constant<bool, YW> wall{};
  int R = j0 - STEP_HALO;
  fetch(R);
  step(std::integral_constant<int, 0>{}, wall, R);
  step(std::integral_constant<int, 0>{}, wall, R + 1);
  step(std::integral_constant<int, 1>{}, wall, R + 2);
  step(std::integral_constant<int, 1>{}, wall, R + 3);
  step(std::integral_constant<int, 2>{}, wall, R + 4);
  step(std::integral_constant<int, 2>{}, wall, R + 5);
  step(std::integral_constant<int, 3>{}, wall, R + 6);
  step(std::integral_constant<int, 3>{}, wall, R + 7);
  R += 8;
  const int rend = j0 + nrows + STEP_HALO;
  // The waves of a SIMD are served oldest first, so of two with the same work
  // the older one would end well before the younger and leave it the SIMD to
  // itself.  The priority falls as the work left does (at a half, a quarter, an
  // eighth), which lets the one behind catch up.
  __builtin_amdgcn_s_setprio(3);
  int level = 3, left = nrows / 2;
  const std::integral_constant<int, 4> all{};
  if (YW && j0 == 0) {  // rows 0 of stages 1 .. 4 fall into steps 1 .. 4
    step(all, wall, R);
    step(all, wall, R + 1);
    R += 2;
  }
  const int rwall = YW && rend > ny ? ny : rend;  // rows ny - 1 into steps ny .. ny + 3
  for (; YW ? R + 1 < rwall : R < rend; R += 2) {
    if (rend - R <= left && level > 0) {
      --level;
      left /= 2;
      if (level == 2) __builtin_amdgcn_s_setprio(2);
      if (level == 1) __builtin_amdgcn_s_setprio(1);
      if (level == 0) __builtin_amdgcn_s_setprio(0);
    }
    step(all, std::false_type{}, R);
    step(all, std::false_type{}, R + 1);
  }
  if (YW) {
#pragma unroll 1
    for (; R < rend; ++R) step(all, wall, R);
  }
  if (health) atomicOr(flag, health);
  if (EPI != EPI_NONE) {
    double a[5];
    sums->get(lane, a);
    CSum m{a[0], a[1]}, e{a[2], a[3]};
    wave_merge(m);
    wave_merge(e);
    if (lane == 0) {
      rpart[0] = m.s;
      rpart[1] = m.c;
      rpart[2] = e.s;
      rpart[3] = e.c;
    }
  }
}

// The strip's variant by the walls it touches (the same for the whole wave).
template <typename T, int BCX, int BCY, bool SAVE, int EPI>
__device__ __forceinline__ void march_any(const MarchSmem<T>& s, const GridConst& gc, int i0, int j0, int nrows,
                                          const T* __restrict__ q, const T* __restrict__ bplane, T* __restrict__ qout,
                                          T c6, T c3, T c2, T c1, int* __restrict__ flag, T* __restrict__ ysave,
                                          double* __restrict__ rpart) {
  const bool xw = BCX == BC_REFLECTING && (i0 - STEP_HALO <= 0 || i0 - STEP_HALO + MARCH_LANES >= gc.nx);
  const bool yw = BCY == BC_REFLECTING && (j0 < STEP_HALO || j0 + nrows > gc.ny - STEP_HALO);
#define SGN_STRIP(XW, YW) \
  march_strip<T, BCX, BCY, XW, YW, SAVE, EPI>(s, gc, i0, j0, nrows, q, bplane, qout, c6, c3, c2, c1, flag, ysave, rpart)
  if constexpr (BCX == BC_REFLECTING) {
    if (xw) {
      if constexpr (BCY == BC_REFLECTING) {
        if (yw) return SGN_STRIP(true, true);
      }
      return SGN_STRIP(true, false);
    }
  }
  if constexpr (BCY == BC_REFLECTING) {
    if (yw) return SGN_STRIP(false, true);
  }
  SGN_STRIP(false, false);
#undef SGN_STRIP
}

// Declares a wave's LDS and its MarchSmem `s`.
#define SGN_MARCH_LDS(T)                                    \
  __shared__ MarchLds<T> march_r1, march_r2, march_r3, march_r4; \
  __shared__ T march_b5[MARCH_LANES + 2];                   \
  __shared__ MarchHold<T> march_hold[2];                    \
  const MarchSmem<T> s{{&march_r1, &march_r2, &march_r3, &march_r4}, march_b5, march_hold}

// Waves per SIMD of the march kernels (their registers: 256 in FP64, 168 in FP32).
template <typename T>
constexpr int march_waves() {
  return sizeof(T) == 8 ? 2 : 3;
}

// First row of run `chunk` of `nchunks` over ny rows.  Runs that end at a
// reflecting wall are a fifth shorter: the steps at the wall take longer, and the
// kernel ends with its slowest wave.
__device__ __forceinline__ int march_row(int chunk, int nchunks, int ny, bool walls) {
  if (chunk <= 0) return 0;
  if (chunk >= nchunks) return ny;
  return walls ? (int)((long long)ny * (5 * chunk - 1) / (5 * nchunks - 2)) : (int)((long long)ny * chunk / nchunks);
}

// Rows of the shortest run of march_row's division: with walls the first one.
inline long long march_least_rows(int nchunks, int ny, bool walls) {
  if (nchunks <= 1) return ny;
  return walls ? 4LL * ny / (5LL * nchunks - 2) : ny / nchunks;
}
// What a run holds at least: a run whose halo of four rows reaches a wall takes the
// wall's variant (march_any), whose prelude and last steps are laid out for runs that
// hold as many rows themselves.  Plans are checked for it.
constexpr int MARCH_LEAST_ROWS = 4;

// One wave per workgroup.  Tasks: with reflecting walls in x first those of the
// first and the last strip, cut into wchunks runs of rows each (more than the
// others, as their evaluations take longer), then those of the other strips, cut
// into nchunks, strips fastest.  EPI: 4 doubles per task, in task order.
template <typename T, int BCX, int BCY, bool SAVE, int EPI>
__global__ __launch_bounds__(MARCH_LANES, march_waves<T>()) void march_kernel(
    const GridConst gc, int nstrips, int nchunks, int wchunks, const T* __restrict__ q, const T* __restrict__ bplane,
    T* __restrict__ qout, T c6, T c3, T c2, T c1, int* __restrict__ flag, T* __restrict__ ysave,
    double* __restrict__ rpart) {
  SGN_MARCH_LDS(T);
  const int task = xcd_tile(blockIdx.x, (int)gridDim.x);
  int strip, chunk, n = nchunks;
  if (BCX == BC_REFLECTING) {
    if (task < 2 * wchunks) {
      n = wchunks;
      strip = task < wchunks ? 0 : nstrips - 1;
      chunk = task < wchunks ? task : task - wchunks;
    } else {
      strip = 1 + (task - 2 * wchunks) % (nstrips - 2);
      chunk = (task - 2 * wchunks) / (nstrips - 2);
    }
  } else {
    strip = task % nstrips;
    chunk = task / nstrips;
  }
  const int j0 = march_row(chunk, n, gc.ny, BCY == BC_REFLECTING);
  const int j1 = march_row(chunk + 1, n, gc.ny, BCY == BC_REFLECTING);
  march_any<T, BCX, BCY, SAVE, EPI>(s, gc, strip * MARCH_COLS, j0, j1 - j0, q, bplane, qout, c6, c3, c2, c1, flag,
                                    ysave, EPI != EPI_NONE ? rpart + 4 * task : nullptr);
}

}  // namespace sgn
