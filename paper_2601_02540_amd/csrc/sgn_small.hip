// sgn_small.hip -- launches of the small-grid step kernel (sgn_small.hpp).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <vector>

#include "sgn.h"
#include "sgn_internal.hpp"
#include "sgn_small.hpp"

namespace {

template <typename T, int STEPS>
hipError_t launch_t(const sgn_ctx* c, hipStream_t s, const void* qin, void* qout, double dt) {
  const int side = sgn::SMALL_SIDE;
  const dim3 grid((unsigned)(((c->p.nx + side - 1) / side) * ((c->p.ny + side - 1) / side)));
  const dim3 block(sgn::SmallGeom<STEPS>::THREADS);
#define SGN_SMALL(BX, BY)                                                                                            \
  do {                                                                                                               \
    if (c->prof_start)                                                                                               \
      hipExtLaunchKernelGGL((sgn::small_step_kernel<T, BX, BY, STEPS>), grid, block, 0, s, c->prof_start,            \
                            c->prof_stop, 0, c->gc, (const T*)qin, (const T*)c->b, (T*)qout, (T)(dt / 6.0),          \
                            (T)(dt / 3.0), (T)(dt / 2.0), (T)dt, c->flag);                                           \
    else                                                                                                             \
      hipLaunchKernelGGL((sgn::small_step_kernel<T, BX, BY, STEPS>), grid, block, 0, s, c->gc, (const T*)qin,        \
                         (const T*)c->b, (T*)qout, (T)(dt / 6.0), (T)(dt / 3.0), (T)(dt / 2.0), (T)dt, c->flag);     \
  } while (0)
  const int bx = c->p.bc_x, by = c->p.bc_y;
  if (bx == 0 && by == 0) SGN_SMALL(0, 0);
  else if (bx == 0) SGN_SMALL(0, 1);
  else if (by == 0) SGN_SMALL(1, 0);
  else SGN_SMALL(1, 1);
#undef SGN_SMALL
  return hipGetLastError();
}

}  // namespace

namespace sgn_host {

bool small_pays(const sgn_ctx* c) {
  return c->step_path == SGN_PATH_FUSED && c->step_auto && c->p.source == SGN_SRC_NONE &&
         (int64_t)((c->p.nx + 7) / 8) * ((c->p.ny + 7) / 8) <=
             (int64_t)(c->p.dtype == SGN_F64 ? 1 : 2) * c->num_cus;
}

hipError_t launch_small(const sgn_ctx* c, hipStream_t s, const void* qin, void* qout, double dt, int steps) {
  if (c->p.dtype == SGN_F64)
    return steps == 2 ? launch_t<double, 2>(c, s, qin, qout, dt) : launch_t<double, 1>(c, s, qin, qout, dt);
  return steps == 2 ? launch_t<float, 2>(c, s, qin, qout, dt) : launch_t<float, 1>(c, s, qin, qout, dt);
}

namespace {

// The launches of `steps` >= 1 steps of the state in q: f(in, out, steps of the launch)
// for each; a single one leaves the state in acc.
template <typename F>
void small_launches(const sgn_ctx* c, void* q, int steps, F&& f) {
  // as many double steps as there are; the state has to end in q: two launches
  // alternate with acc, an odd count of launches begins with three by way of acc and ya
  int twos = steps / 2, ones = steps & 1;
  if (steps == 2) twos = 0, ones = 2;
  int left = twos + ones;
  const auto take = [&](void* in, void* out) {
    const int n = twos > 0 ? 2 : 1;
    --(n == 2 ? twos : ones);
    --left;
    f(in, out, n);
  };
  if (left == 1) return take(q, c->acc);
  if (left & 1) {
    take(q, c->acc);
    take(c->acc, c->ya);
    take(c->ya, q);
  }
  while (left > 0) {
    take(q, c->acc);
    take(c->acc, q);
  }
}

}  // namespace

hipError_t enqueue_small_steps(const sgn_ctx* c, hipStream_t s, void* q, double dt, int steps) {
  hipError_t e = hipSuccess;
  void* end = q;
  small_launches(c, q, steps, [&](void* in, void* out, int n) {
    if (!e) e = launch_small(c, s, in, out, dt, n);
    end = out;
  });
  if (!e && end != q) e = hipMemcpyAsync(q, end, 5 * c->N * c->esize, hipMemcpyDeviceToDevice, s);
  return e;
}

hipError_t profile_small_steps(sgn_ctx* c, void* q, double dt, int steps, double* ms_per_step) {
  std::vector<hipEvent_t> ev;
  std::vector<int> taken;
  hipError_t e = hipSuccess;
  small_launches(c, q, steps, [&](void* in, void* out, int n) {
    hipEvent_t pair[2] = {nullptr, nullptr};
    for (hipEvent_t& x : pair) {
      if (!e) e = hipEventCreate(&x);
      ev.push_back(x);
    }
    taken.push_back(n);
    c->prof_start = pair[0];
    c->prof_stop = pair[1];
    if (!e) e = launch_small(c, c->stream, in, out, dt, n);
    c->prof_start = c->prof_stop = nullptr;
  });
  if (!e) e = hipEventSynchronize(ev.back());
  double sum = 0.0;
  int used = 0;
  for (size_t k = taken.size() > 1 ? 1 : 0; k < taken.size() && !e; ++k) {
    float m = 0.f;
    e = hipEventElapsedTime(&m, ev[2 * k], ev[2 * k + 1]);
    sum += m;
    used += taken[k];
  }
  for (hipEvent_t x : ev)
    if (x) (void)hipEventDestroy(x);
  *ms_per_step = used ? sum / used : 0.0;
  return e;
}

}  // namespace sgn_host
