// sgn_march.hip -- launches of the march kernel (sgn_march.hpp) for one problem.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sgn.h"
#include "sgn_internal.hpp"
#include "sgn_march.hpp"

namespace {

using sgn_host::MarchPlan;

template <typename T, int BCX, int BCY, bool SAVE, int EPI>
hipError_t launch(const sgn_ctx* c, hipStream_t s, const MarchPlan& m, const void* qin, void* qout, double dt,
                  void* ysave, double* rpart) {
  const dim3 grid((unsigned)m.tasks), block(sgn::MARCH_LANES);
  const T c6 = (T)(dt / 6.0), c3 = (T)(dt / 3.0), c2 = (T)(dt / 2.0), c1 = (T)dt;
  if (c->prof_start)
    hipExtLaunchKernelGGL((sgn::march_kernel<T, BCX, BCY, SAVE, EPI>), grid, block, 0, s, c->prof_start, c->prof_stop, 0,
                          c->gc, m.strips, m.chunks, m.wall_chunks, (const T*)qin, (const T*)c->b, (T*)qout, c6, c3, c2, c1, c->flag,
                          (T*)ysave, rpart);
  else
    hipLaunchKernelGGL((sgn::march_kernel<T, BCX, BCY, SAVE, EPI>), grid, block, 0, s, c->gc, m.strips, m.chunks,
                       m.wall_chunks, (const T*)qin, (const T*)c->b, (T*)qout, c6, c3, c2, c1, c->flag, (T*)ysave, rpart);
  return hipGetLastError();
}

template <typename T, bool SAVE, int EPI>
hipError_t launch_bc(const sgn_ctx* c, hipStream_t s, const MarchPlan& m, const void* qin, void* qout, double dt,
                     void* ysave, double* rpart) {
  const int bx = c->p.bc_x, by = c->p.bc_y;
  if (bx == 0 && by == 0) return launch<T, 0, 0, SAVE, EPI>(c, s, m, qin, qout, dt, ysave, rpart);
  if (bx == 0) return launch<T, 0, 1, SAVE, EPI>(c, s, m, qin, qout, dt, ysave, rpart);
  if (by == 0) return launch<T, 1, 0, SAVE, EPI>(c, s, m, qin, qout, dt, ysave, rpart);
  return launch<T, 1, 1, SAVE, EPI>(c, s, m, qin, qout, dt, ysave, rpart);
}

template <typename T>
hipError_t launch_t(const sgn_ctx* c, hipStream_t s, const MarchPlan& m, const void* qin, void* qout, double dt,
                    void* ysave, double* rpart) {
  if (ysave) return launch_bc<T, true, sgn::EPI_NONE>(c, s, m, qin, qout, dt, ysave, nullptr);
  if (rpart) return launch_bc<T, false, sgn::EPI_TOTALS>(c, s, m, qin, qout, dt, nullptr, rpart);
  return launch_bc<T, false, sgn::EPI_NONE>(c, s, m, qin, qout, dt, nullptr, nullptr);
}

}  // namespace

namespace sgn_host {

MarchPlan march_plan(const sgn_ctx* c) {
  MarchPlan m;
  if (c->step_tile != 24 || c->p.source != SGN_SRC_NONE || (int64_t)c->N < MARCH_MIN_NODES) return m;
  const int strips = (c->p.nx + sgn::MARCH_COLS - 1) / sgn::MARCH_COLS;
  const int slots = c->num_cus * 4 * (c->p.dtype == SGN_F64 ? sgn::march_waves<double>() : sgn::march_waves<float>());
  const int most = std::max(1, c->p.ny / MARCH_MIN_HEIGHT);
  // the two strips at reflecting walls in x are cut into a quarter more runs
  const bool xw = c->p.bc_x == SGN_REFLECTING;
  if (xw && strips < 3) return m;
  const int chunks = std::max(1, std::min(xw ? 2 * slots / (2 * strips + 1) : slots / strips, most));
  const bool f64_walls = xw && c->p.bc_y == SGN_REFLECTING && c->p.dtype == SGN_F64;
  if (!march_pays(march_evals(strips, c->p.ny, chunks), tile_evals(c->p.nx, c->p.ny), f64_walls)) return m;
  const int wall_chunks = xw ? std::min(chunks + chunks / 4, most) : 0;
  const bool yw = c->p.bc_y == SGN_REFLECTING;
  if (sgn::march_least_rows(std::max(chunks, wall_chunks), c->p.ny, yw) < sgn::MARCH_LEAST_ROWS) return m;
  m.strips = strips;
  m.chunks = chunks;
  m.wall_chunks = wall_chunks;
  m.tasks = xw ? 2 * m.wall_chunks + (strips - 2) * chunks : strips * chunks;
  return m;
}

hipError_t launch_march(const sgn_ctx* c, hipStream_t s, const MarchPlan& m, const void* qin, void* qout, double dt,
                        void* ysave, double* rpart) {
  return c->p.dtype == SGN_F64 ? launch_t<double>(c, s, m, qin, qout, dt, ysave, rpart)
                               : launch_t<float>(c, s, m, qin, qout, dt, ysave, rpart);
}

}  // namespace sgn_host
