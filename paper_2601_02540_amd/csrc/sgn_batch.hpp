// sgn_batch.hpp -- an ensemble of independent problems in one launch per RK4
// step (step tiles, or the march kernel's strips) or per stage pair (pair tiles).
//
// Every instance has its own grid size, boundary types, spacing, g, lambda and
// time step.  The tiles of all instances form one work list (instance-major,
// row-major tiles within an instance), cut into eight contiguous ranges, one per
// XCD, so tiles of the same instance (and their shared halo rows) stay in one
// L2.  Each work item runs the same tile or strip code as the single-problem kernels,
// with the boundary variant chosen per instance at run time (uniform per
// workgroup).  A launch has either one workgroup per work item or a persistent
// grid of workgroups that walks the list.
#pragma once

#include "sgn_fused.hpp"
#include "sgn_march.hpp"
#include "sgn_pair.hpp"

namespace sgn {

struct InstDesc {
  GridConst gc;
  double dt;
  int tile_base;  // first work item of this instance
  int ntx, nty;   // tiles per axis (march kernel: strips, and runs of rows per strip)
  int pad;
  void* q;        // caller's state
  void* acc;      // scratch state (second buffer of the ping-pong)
  void* yb;       // scratch stage plane set (pair path), third buffer of an odd count of steps (fused)
  const void* b;  // bathymetry copy
};

template <typename T, int PAIR, int TY, int BCX, int BCY>
__device__ __forceinline__ void batch_tile(PairSmem<T, TY>& s, const InstDesc& d, int i0, int j0, int parity,
                                           int* flag) {
  T* q = (T*)d.q;
  T* acc = (T*)d.acc;
  T* cur = parity ? acc : q;
  T* oth = parity ? q : acc;
  const T* b = (const T*)d.b;
  T* yb = (T*)d.yb;
  const double dt = d.dt;
  if (PAIR == 1)
    pair_tile<T, BCX, BCY, 1, false, TY>(s, d.gc, i0, j0, cur, b, nullptr, oth, yb, T(dt / 6.0), T(dt / 2.0),
                                         T(dt / 3.0), T(dt / 2.0), 0.0, 0.0, flag);
  else
    pair_tile<T, BCX, BCY, 2, false, TY>(s, d.gc, i0, j0, yb, b, cur, oth, nullptr, T(dt / 3.0), T(dt),
                                         T(dt / 6.0), T(0.0), 0.0, 0.0, flag);
}

// Work item w of a stage pair.
template <typename T, int PAIR, int TY>
__device__ __forceinline__ void batch_pair_item(PairSmem<T, TY>& s, const InstDesc* __restrict__ desc,
                                                const int* __restrict__ work_inst, int w, int parity,
                                                int* __restrict__ flags) {
  const int inst = work_inst[w];
  const InstDesc d = desc[inst];
  const int t = w - d.tile_base;
  const int i0 = (t % d.ntx) * TILE_X;
  const int j0 = (t / d.ntx) * TY;
  switch (d.gc.bc_x * 2 + d.gc.bc_y) {
    case 0: batch_tile<T, PAIR, TY, 0, 0>(s, d, i0, j0, parity, flags + inst); break;
    case 1: batch_tile<T, PAIR, TY, 0, 1>(s, d, i0, j0, parity, flags + inst); break;
    case 2: batch_tile<T, PAIR, TY, 1, 0>(s, d, i0, j0, parity, flags + inst); break;
    default: batch_tile<T, PAIR, TY, 1, 1>(s, d, i0, j0, parity, flags + inst); break;
  }
}

// parity 0: state in q, written to acc; parity 1: state in acc, written to q.
// PERSIST: a persistent grid (a multiple of 8 workgroups) walks the list, one
// contiguous range per XCD.  Otherwise one workgroup per work item (a grid of
// nwork), dealt to the XCDs in the same contiguous ranges; such a kernel holds
// no loop-invariant state across tiles, so it needs fewer registers and runs
// at a higher occupancy.
template <typename T, int PAIR, int TY, bool PERSIST>
__global__ __launch_bounds__(STAGE_THREADS) void batch_pair_kernel(const InstDesc* __restrict__ desc,
                                                                   const int* __restrict__ work_inst, int nwork,
                                                                   int parity, int* __restrict__ flags) {
  __shared__ PairSmem<T, TY> s;
  if (!PERSIST) {
    batch_pair_item<T, PAIR, TY>(s, desc, work_inst, xcd_tile(blockIdx.x, nwork), parity, flags);
    return;
  }
  const int xcd = blockIdx.x & 7;
  const int k = blockIdx.x >> 3;
  const int blocks_per_xcd = gridDim.x >> 3;
  const int start = (int)((long long)nwork * xcd / 8);
  const int end = (int)((long long)nwork * (xcd + 1) / 8);
  for (int w = start + k; w < end; w += blocks_per_xcd) {
    batch_pair_item<T, PAIR, TY>(s, desc, work_inst, w, parity, flags);
    __syncthreads();
  }
}

// Input and output state of a step of the fused path.  Steps go in twos by way
// of acc; an odd count begins with three by way of acc and yb.
enum : int { BATCH_Q_ACC = 0, BATCH_ACC_Q = 1, BATCH_ACC_YB = 2, BATCH_YB_Q = 3 };
template <typename T>
__device__ __forceinline__ const T* batch_in(void* q, void* acc, void* yb, int route) {
  return (const T*)(route == BATCH_Q_ACC ? q : route == BATCH_YB_Q ? yb : acc);
}
template <typename T>
__device__ __forceinline__ T* batch_out(void* q, void* acc, void* yb, int route) {
  return (T*)(route == BATCH_Q_ACC ? acc : route == BATCH_ACC_YB ? yb : q);
}

// Work item w of one RK4 step by the step tile (tiles of TX x TY, StepGeom).
template <typename T, int TY>
__device__ __forceinline__ void batch_step_item(StepSmem<T, TY, 1>& s, const InstDesc* __restrict__ desc,
                                                const int* __restrict__ work_inst, int w, int route,
                                                int* __restrict__ flags) {
  constexpr int TX = StepGeom<TY>::TX;
  const int inst = work_inst[w];
  const InstDesc d = desc[inst];
  const int t = w - d.tile_base;
  const int i0 = (t % d.ntx) * TX;
  const int j0 = (t / d.ntx) * TY;
  const T* cur = batch_in<T>(d.q, d.acc, d.yb, route);
  T* oth = batch_out<T>(d.q, d.acc, d.yb, route);
  const T* b = (const T*)d.b;
  const double dt = d.dt;
  const T c6 = T(dt / 6.0), c3 = T(dt / 3.0), c2 = T(dt / 2.0), c1 = T(dt);
  switch (d.gc.bc_x * 2 + d.gc.bc_y) {
    case 0: step_tile<T, 0, 0, false, TY, false, 1, EPI_NONE, RK_CLASSIC, sizeof(T) == 4>(s, d.gc, i0, j0, cur, b, oth, c6, c3, c2, c1, 0.0, dt, flags + inst, nullptr); break;
    case 1: step_tile<T, 0, 1, false, TY, false, 1, EPI_NONE, RK_CLASSIC, sizeof(T) == 4>(s, d.gc, i0, j0, cur, b, oth, c6, c3, c2, c1, 0.0, dt, flags + inst, nullptr); break;
    case 2: step_tile<T, 1, 0, false, TY, false, 1, EPI_NONE, RK_CLASSIC, sizeof(T) == 4>(s, d.gc, i0, j0, cur, b, oth, c6, c3, c2, c1, 0.0, dt, flags + inst, nullptr); break;
    default: step_tile<T, 1, 1, false, TY, false, 1, EPI_NONE, RK_CLASSIC, sizeof(T) == 4>(s, d.gc, i0, j0, cur, b, oth, c6, c3, c2, c1, 0.0, dt, flags + inst, nullptr); break;
  }
}

// One RK4 step of every instance.  route: BATCH_*; PERSIST as for batch_pair_kernel.
template <typename T, int TY, bool PERSIST>
__global__ __launch_bounds__(STAGE_THREADS) void batch_step_kernel(const InstDesc* __restrict__ desc,
                                                                   const int* __restrict__ work_inst, int nwork,
                                                                   int route, int* __restrict__ flags) {
  __shared__ StepSmem<T, TY, 1> s;
  if (!PERSIST) {
    batch_step_item<T, TY>(s, desc, work_inst, xcd_tile(blockIdx.x, nwork), route, flags);
    return;
  }
  const int xcd = blockIdx.x & 7;
  const int k = blockIdx.x >> 3;
  const int blocks_per_xcd = gridDim.x >> 3;  // the grid is a multiple of 8
  const int start = (int)((long long)nwork * xcd / 8);
  const int end = (int)((long long)nwork * (xcd + 1) / 8);
  for (int w = start + k; w < end; w += blocks_per_xcd) {
    batch_step_item<T, TY>(s, desc, work_inst, w, route, flags);
    __syncthreads();
  }
}

// One RK4 step of every instance by the march kernel: work item = one run of
// rows of one strip of one instance, one wave each.
template <typename T>
__global__ __launch_bounds__(MARCH_LANES, march_waves<T>()) void batch_march_kernel(const InstDesc* __restrict__ desc,
                                                                                 const int* __restrict__ work_inst,
                                                                                 int nwork, int route,
                                                                                 int* __restrict__ flags) {
  SGN_MARCH_LDS(T);
  const int w = xcd_tile(blockIdx.x, nwork);
  const int inst = work_inst[w];
  const InstDesc& d = desc[inst];
  const GridConst gc = d.gc;
  const int t = w - d.tile_base;
  const int strip = t % d.ntx, chunk = t / d.ntx, nchunks = d.nty;
  const int j0 = march_row(chunk, nchunks, gc.ny, gc.bc_y == BC_REFLECTING);
  const int j1 = march_row(chunk + 1, nchunks, gc.ny, gc.bc_y == BC_REFLECTING);
  const T* cur = batch_in<T>(d.q, d.acc, d.yb, route);
  T* oth = batch_out<T>(d.q, d.acc, d.yb, route);
  const T* b = (const T*)d.b;
  const double dt = d.dt;
  const T c6 = T(dt / 6.0), c3 = T(dt / 3.0), c2 = T(dt / 2.0), c1 = T(dt);
  const int i0 = strip * MARCH_COLS;
  switch (gc.bc_x * 2 + gc.bc_y) {
    case 0: march_any<T, 0, 0, false, EPI_NONE>(s, gc, i0, j0, j1 - j0, cur, b, oth, c6, c3, c2, c1, flags + inst, nullptr, nullptr); break;
    case 1: march_any<T, 0, 1, false, EPI_NONE>(s, gc, i0, j0, j1 - j0, cur, b, oth, c6, c3, c2, c1, flags + inst, nullptr, nullptr); break;
    case 2: march_any<T, 1, 0, false, EPI_NONE>(s, gc, i0, j0, j1 - j0, cur, b, oth, c6, c3, c2, c1, flags + inst, nullptr, nullptr); break;
    default: march_any<T, 1, 1, false, EPI_NONE>(s, gc, i0, j0, j1 - j0, cur, b, oth, c6, c3, c2, c1, flags + inst, nullptr, nullptr); break;
  }
}

// q <- acc of the ninst instances (after a single step of the fused path); block row
// blockIdx.y takes instances blockIdx.y, blockIdx.y + gridDim.y, ... (a launch has at
// most 65536 rows, an ensemble may have more instances).
constexpr int BATCH_COPY_ROWS = 16384;
template <typename T>
__global__ __launch_bounds__(256) void batch_copy_kernel(const InstDesc* __restrict__ desc, int ninst) {
  for (int i = blockIdx.y; i < ninst; i += gridDim.y) {
    const InstDesc& d = desc[i];
    const size_t n = 5 * (size_t)d.gc.nx * (size_t)d.gc.ny;
    const T* src = (const T*)d.acc;
    T* dst = (T*)d.q;
    for (size_t k = (size_t)blockIdx.x * 256 + threadIdx.x; k < n; k += (size_t)gridDim.x * 256) dst[k] = src[k];
  }
}

}  // namespace sgn
