// sgn_internal.hpp -- host-side context shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <string>

#include "sgn.h"
#include "sgn_common.hpp"

namespace sgn_host {

struct GraphCache {
  hipGraphExec_t exec = nullptr;
  const void* q = nullptr;
  double dt = 0.0;
  int steps = 0;
  int path = -1;
  int tile_y = 0;
  int step_tile = 0;
};

// Buffers of the discrete adjoint, allocated on first use and kept by the context.
struct AdjointBuffers {
  void* kb_a = nullptr;   // stage cotangents (ping-pong)
  void* kb_b = nullptr;
  void* accb = nullptr;   // running sum of the stage cotangents of one step
  void* qbar = nullptr;   // cotangent of the state
  void* state = nullptr;  // state of a rollout
  void* stages = nullptr; // per-step stored states of a segment: (steps+1) states and 3 stage states per step
  size_t stage_slots = 0; // number of state-sized slots in `stages`
  void* ckpt = nullptr;   // checkpoints
  size_t ckpt_slots = 0;
  double* misfit = nullptr;  // nsteps * ngauges misfits of the forward rollout
  size_t misfit_len = 0;
  double* loss = nullptr;    // device accumulator
};

// Buffers of the adaptive pair (sgn_step_adaptive), allocated on first use.
struct FsalBuffers {
  void* k[2] = {nullptr, nullptr};  // k_1 of the current step / of the next one (FSAL)
  void* e = nullptr;                // partial error estimate
  double* part = nullptr;           // per-tile sums of the scaled squares
  size_t part_cap = 0;              // doubles in part
  void* ctl = nullptr;              // run state (sgn::AdaptCtl) in device memory
  void* host_ctl = nullptr;         // pinned copy read by the host
  GraphCache graph;                 // attempts captured for replay
  double* graph_rec = nullptr;      // record pointer and capacity captured in the graph
  long long graph_rec_cap = 0;
};

}  // namespace sgn_host

struct sgn_ctx {
  sgn_params p{};
  sgn::GridConst gc{};
  hipStream_t stream = nullptr;
  hipStream_t cap_stream = nullptr;
  int device = 0;
  int num_cus = 256;
  size_t N = 0;
  size_t esize = 0;
  void* b = nullptr;
  void* acc = nullptr;
  void* ya = nullptr;
  void* yb = nullptr;
  double* partials = nullptr;
  double* tile_partials = nullptr;  // the epilogue sums of each step tile or run
  size_t tile_partials_cap = 0;     // doubles allocated there
  int* series_counter = nullptr;    // next slot of a recorded totals series (sgn_step_totals)
  double* result = nullptr;
  double* host_result = nullptr;
  int* flag = nullptr;
  int* host_flag = nullptr;
  bool b_set = false;
  int step_path = SGN_PATH_FUSED;
  int tile_y = 8;     // stage and pair kernels
  bool step_auto = true;  // the step kernel's shape is the size rule's (no height was set)
  int step_tile = 16;  // step kernel: 24 the march kernel's strips or 32 x 24 tiles, 16 32 x 16, 8 64 x 8
  sgn_host::GraphCache graphs[2];
  sgn_host::GraphCache relax_graph;   // relaxation steps (sgn_step_relaxation)
  sgn_host::GraphCache totals_graph;  // steps with recorded totals (sgn_step_totals)
  double* totals_series = nullptr;    // the series pointer captured in totals_graph
  sgn_host::AdjointBuffers adj;
  int64_t adj_store_bytes = 0;  // SGN_OPT_ADJOINT_STORE
  sgn_host::FsalBuffers fs;
  // Set only inside sgn_profile_stages: the step kernel is then launched with
  // these events bound to its own start and end.
  hipEvent_t prof_start = nullptr, prof_stop = nullptr;
  std::string err;
};

namespace sgn_host {

// How the march kernel cuts a grid: strips of MARCH_COLS columns, each cut into
// `chunks` runs of rows (wall_chunks: the strips at reflecting walls in x);
// tasks = 0: the grid runs the tile kernel instead.
struct MarchPlan {
  int strips = 0, chunks = 0, wall_chunks = 0, tasks = 0;
};
// One round of waves (as many as the GPU holds at once) covers the grid, in runs of
// MARCH_MIN_HEIGHT rows on average or more (12 evaluations of the rows around a
// run against 4 per row of it; runs at walls in y are a fifth shorter, and the runs of
// an ensemble's instance of a few rows have four or more).  Below MARCH_MIN_NODES the strips are too few or
// too short: FP64 512^2 takes 31 us in runs of 8 rows and 14.5 us on tiles, 1024^2
// 41 us against 43, 2048^2 136 against 155.
constexpr int64_t MARCH_MIN_NODES = (int64_t)1 << 20;
constexpr int MARCH_MIN_HEIGHT = 8;
// Evaluations per step in waves of 64: a strip's rows and those around its runs
// against a 32 x 24 tile's owned and ring nodes (60 waves in four stages).  The march
// kernel runs one in 0.78 of the tile kernel's time on large grids (4096^2: FP64 466
// against 602 us, FP32 257 against 324, about 1.31e6 of them either way) and loses
// some of that where its runs are short.  It is taken where it does not need 1.25
// times as many: not where a last strip of a few columns leaves most of its lanes
// idle.  In FP64 with walls on both axes the line is 1.2, as the runs in the corners
// hold all others up and a last strip of up to four columns leaves its
// neighbour at the wall too.  Strips and tiles in us, at the ratio given (five runs on
// three GPUs; the tiles are 32 x 24 ones periodic and in FP32, 32 x 16 ones else):
//   FP64 periodic  1.04 (1448^2) 71 and 80, 1.13 (1500 x 900) 51 and 51, 1.15 (1063 x
//     1009) 46 and 46, 1.24 (1024^2) 46.7 and 47.3
//   FP64, one axis with walls  1.15 (1063 x 1009) 45 .. 47 and 49 .. 50, 1.21 (1065 x
//     1000) 46 and 49 .. 51, 1.24 (1024^2) 44 .. 47 and 45 .. 46
//   FP64, both  1.04 (1448^2) 80 and 94, 1.19 (1200 x 900) 49 and 52, 1.21 (1065 x 1000)
//     55 .. 58 and 52, 1.21 (300 x 3600) 53 and 52, 1.23 (1024^2) 50 and 47
//   FP32  1.11 (1448^2) 42 .. 44 and 45 .. 48, 1.20 (1063 x 1009) 27 .. 28 and 26 .. 28, 1.25
//     (1500 x 900) 30 .. 31 and 30 .. 32
inline bool march_pays(int64_t march_evals, int64_t tile_evals, bool f64_walls = false) {
  return f64_walls ? 5 * march_evals < 6 * tile_evals : 4 * march_evals < 5 * tile_evals;
}
inline int64_t march_evals(int64_t strips, int64_t ny, int64_t chunks) { return strips * (4 * ny + 12 * chunks); }
inline int64_t tile_evals(int64_t nx, int64_t ny) { return 60 * ((nx + 31) / 32) * ((ny + 23) / 24); }
MarchPlan march_plan(const sgn_ctx* c);
// One step by the march kernel; ysave and rpart as for enqueue_step_into (rpart:
// mass and energy of the new state per task).
hipError_t launch_march(const sgn_ctx* c, hipStream_t s, const MarchPlan& m, const void* qin, void* qout, double dt,
                        void* ysave, double* rpart);
// Whether the small-grid kernel takes the steps (no stage saving, no totals): where
// its 8 x 8 tiles are at most one per compute unit, in FP32 at most two.  A step
// takes, tile kernel and this one, in us: FP64 64^2 9.4 and 5.1, 128^2 (one tile per
// unit) 9.4 and 5.3, 192^2 (2.25) 9.6 and 10.3; FP32 7.9 and 4.0, 7.8 and 4.2, 8.0 and
// 6.8, 256^2 (four) 8.0 and 9.0.
bool small_pays(const sgn_ctx* c);
// One or two steps by the small-grid kernel, qin into qout.
hipError_t launch_small(const sgn_ctx* c, hipStream_t s, const void* qin, void* qout, double dt, int steps);
// `steps` >= 1 steps by it of the state in q, which ends in q.
hipError_t enqueue_small_steps(const sgn_ctx* c, hipStream_t s, void* q, double dt, int steps);
// The same launches (an even count of steps), each timed by events of its own;
// *ms_per_step: mean over all launches but the first.  Waits for the last.
hipError_t profile_small_steps(sgn_ctx* c, void* q, double dt, int steps, double* ms_per_step);
// The tile shape a step kernel of this context runs (24: 32 x 24, ...).
int tile_of(const sgn_ctx* c, int epi = 0);

sgn_status fail(sgn_ctx* c, sgn_status st, const std::string& msg);
sgn_status hip_fail(sgn_ctx* c, hipError_t e, const char* what);
sgn_status sync_results(sgn_ctx* c, int nres);
sgn_status check_ctx(sgn_ctx* c, bool need_b);
void free_adjoint(sgn_ctx* c);
void free_fsal(sgn_ctx* c);
// stage kernel of the four-stage path in mode `mode` (sgn::MODE_*)
hipError_t launch_stage_mode(const sgn_ctx* c, hipStream_t s, int mode, const void* Y, const void* qn, void* acc,
                             void* out, double c_acc, double c_y, double t);
// one RK4 step on the pair path from `cur` into `oth`
hipError_t enqueue_pair_step(const sgn_ctx* c, hipStream_t s, void* cur, void* oth, double dt, double t);
// One RK4 step by the step kernel from `cur` into `oth` (distinct buffers);
// with `ysave` non-null the stage states Y2, Y3, Y4 go to three consecutive
// state slots there; with `rpart` non-null each tile's epilogue sums `epi`
// (sgn::EPI_RELAX: relaxation sums at gam = 1; sgn::EPI_TOTALS: mass and
// energy of the new state) go to rpart[epi_part(epi) tile ..] (step_parts(c, epi) of them).
// Neither with source terms, and not both.
hipError_t enqueue_step_into(const sgn_ctx* c, hipStream_t s, const void* cur, void* oth, double dt, double t,
                             void* ysave, double* rpart = nullptr, int epi = 0);
// Number of partial sums a step with epilogue `epi` leaves.
int step_parts(const sgn_ctx* c, int epi);
// Steps whose totals are merged in one launch: their partials are all kept, up to
// 32 MB of them.
constexpr int TOTALS_GROUP = 8;
int totals_group(const sgn_ctx* c);
// Makes c->tile_partials hold the epilogue sums of every shape
// (synchronizes and drops the graphs that captured an older buffer).
sgn_status ensure_tile_partials(sgn_ctx* c);
// Validation of sgn_params (the rules of sgn_create; failures leave their
// message for sgn_last_error(NULL)) and the grid constants the kernels take.
sgn_status check_params(const sgn_params* p);
sgn::GridConst grid_const(const sgn_params& p);

}  // namespace sgn_host

#define SGN_HIPCHK(c, expr)                                                \
  do {                                                                     \
    hipError_t e_ = (expr);                                                \
    if (e_ != hipSuccess) return sgn_host::hip_fail((c), e_, #expr);       \
  } while (0)
