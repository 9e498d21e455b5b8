// sgn_totals.hip -- C ABI of RK4 stepping with the total mass and energy of
// every step recorded on the device (sgn_step_totals).
//
// Each step runs the step kernel with its totals epilogue: every tile reduces
// M h and M E of the state it writes, from the values it holds in registers,
// so the series costs no pass over the state.  One small kernel per group of up to
// eight steps reduces their partials (in a fixed order: deterministic) into the next
// slots of the caller's series, whose index lives in device memory, so that the
// steps replay from one captured graph.
#include <hip/hip_runtime.h>

#include <cmath>

#include "sgn.h"
#include "sgn_internal.hpp"
#include "sgn_reduce.hpp"

namespace {

using sgn_host::fail;
using sgn_host::hip_fail;

#define HIPCHK(c, expr) SGN_HIPCHK(c, expr)

// Steps captured per graph replay (even: the state returns to the caller's buffer).
constexpr int TOTALS_GRAPH_STEPS = 8;

// Most blocks per step of the merge (c->partials holds the results of a group of steps).
constexpr int TOTALS_MERGE_BLOCKS = sgn::RED_MAX_BLOCKS / sgn_host::TOTALS_GROUP;

// The totals of the `rows` steps whose partials lie in c->tile_partials.
hipError_t enqueue_totals(const sgn_ctx* c, hipStream_t s, int rows, double* series) {
  const int parts = sgn_host::step_parts(c, sgn::EPI_TOTALS);
  int nb = (parts + sgn::RED_THREADS - 1) / sgn::RED_THREADS;
  if (nb > TOTALS_MERGE_BLOCKS) nb = TOTALS_MERGE_BLOCKS;
  const int per = (parts + nb - 1) / nb;
  hipLaunchKernelGGL(sgn::series_merge, dim3(nb, rows), dim3(sgn::RED_THREADS), 0, s, (const double*)c->tile_partials,
                     parts, per, c->partials, series, c->series_counter);
  return hipGetLastError();
}

// `steps` steps of the state in q, which ends in q: in twos by way of acc, an
// odd count >= 3 beginning with three by way of acc and ya, a single one copied
// back.  The partials of up to totals_group(c) steps are kept and merged in one
// launch: two launches a step took 10 us of the 60 us of a 1024^2 FP64 step.
hipError_t enqueue_steps_with_totals(const sgn_ctx* c, hipStream_t s, void* q, double dt, int steps, double* series) {
  const int group = sgn_host::totals_group(c);
  const size_t row = (size_t)4 * sgn_host::step_parts(c, sgn::EPI_TOTALS);
  const bool odd = steps & 1;
  void* cur = q;
  hipError_t e = hipSuccess;
  for (int k = 0; k < steps && !e; ++k) {
    void* oth = odd && k < 3 ? (k == 0 ? c->acc : k == 1 ? c->ya : q) : cur == q ? c->acc : q;
    e = sgn_host::enqueue_step_into(c, s, cur, oth, dt, 0.0, nullptr, c->tile_partials + row * (k % group),
                                    sgn::EPI_TOTALS);
    cur = oth;
    if (!e && (k % group == group - 1 || k == steps - 1)) e = enqueue_totals(c, s, k % group + 1, series);
  }
  if (!e && cur != q) e = hipMemcpyAsync(q, cur, 5 * c->N * c->esize, hipMemcpyDeviceToDevice, s);
  return e;
}

}  // namespace

extern "C" {

sgn_status sgn_step_totals(sgn_ctx* c, void* q, double dt, int64_t nsteps, double* series) {
  sgn_status st = sgn_host::check_ctx(c, true);
  if (st) return st;
  if (!q) return fail(c, SGN_E_ARG, "q is NULL");
  if (!(std::isfinite(dt) && dt > 0.0)) return fail(c, SGN_E_ARG, "dt must be finite and > 0");
  if (nsteps < 0) return fail(c, SGN_E_ARG, "nsteps must be >= 0");
  if (nsteps > (int64_t)0x3fffffff) return fail(c, SGN_E_ARG, "nsteps too large for one series");
  if (c->p.source != SGN_SRC_NONE)
    return fail(c, SGN_E_UNSUPPORTED, "recorded totals need the semi-discretization without source terms");
  if (nsteps == 0) return SGN_OK;
  if (!series) return fail(c, SGN_E_ARG, "series is NULL");
  if ((st = sgn_host::ensure_tile_partials(c))) return st;
  if (!c->series_counter && hipMalloc((void**)&c->series_counter, 2 * sizeof(int)) != hipSuccess) {
    c->series_counter = nullptr;
    return fail(c, SGN_E_ALLOC, "series counter");
  }
  hipLaunchKernelGGL(sgn::counter_reset, dim3(1), dim3(64), 0, c->stream, c->series_counter);
  HIPCHK(c, hipGetLastError());
  int64_t left = nsteps;
  if (left >= TOTALS_GRAPH_STEPS) {
    auto& g = c->totals_graph;
    if (!(g.exec && g.q == q && g.dt == dt && g.step_tile == c->step_tile && c->totals_series == series)) {
      if (g.exec) (void)hipGraphExecDestroy(g.exec);
      g = sgn_host::GraphCache{};
      c->totals_series = nullptr;
      HIPCHK(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal));
      hipError_t le = enqueue_steps_with_totals(c, c->cap_stream, q, dt, TOTALS_GRAPH_STEPS, series);
      hipGraph_t graph = nullptr;
      hipError_t ce = hipStreamEndCapture(c->cap_stream, &graph);
      if (le != hipSuccess) {
        if (graph) (void)hipGraphDestroy(graph);
        return hip_fail(c, le, "step launch during capture");
      }
      if (ce != hipSuccess) return hip_fail(c, ce, "hipStreamEndCapture");
      hipGraphExec_t exec = nullptr;
      hipError_t ie = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
      (void)hipGraphDestroy(graph);
      if (ie != hipSuccess) return hip_fail(c, ie, "hipGraphInstantiate");
      g.exec = exec;
      g.q = q;
      g.dt = dt;
      g.steps = TOTALS_GRAPH_STEPS;
      g.path = c->step_path;
      g.tile_y = c->tile_y;
      g.step_tile = c->step_tile;
      c->totals_series = series;
    }
    for (; left >= TOTALS_GRAPH_STEPS; left -= TOTALS_GRAPH_STEPS) HIPCHK(c, hipGraphLaunch(g.exec, c->stream));
  }
  if (left > 0) HIPCHK(c, enqueue_steps_with_totals(c, c->stream, q, dt, (int)left, series));
  return SGN_OK;
}

}  // extern "C"
