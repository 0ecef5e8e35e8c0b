// Host-side interface between the library's C entry points (dpf_lib.hip) and
// the per-model translation units (dpf_eng_*.hip), each of which instantiates
// the step kernels of one model for every tile class and exposes them through
// an Engine table.  Splitting the models over translation units lets them
// compile in parallel.
#pragma once
#include <hip/hip_runtime.h>

#include <vector>

#include "../../include/dpf.h"
#include "dpf_kernels.hpp"

namespace dpf {

// Record a failure message for dpf_last_error and return s.
dpf_status fail(dpf_status s, const char* fmt, ...);

#define HIP_TRY(expr)                                                                      \
  do {                                                                                     \
    hipError_t e_ = (expr);                                                                \
    if (e_ != hipSuccess) return fail(DPF_EDEVICE, "%s failed: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

#define LAUNCH_CHECK(what)                                                                 \
  do {                                                                                     \
    hipError_t e_ = hipGetLastError();                                                     \
    if (e_ != hipSuccess) return fail(DPF_EDEVICE, "launch of %s failed: %s", what, hipGetErrorString(e_)); \
  } while (0)

// ------------------------------------------------------------ tile classes
struct ClassShape {
  int seg, jpt;
};
// The first six are the defaults (the first that holds M); the others are
// chosen only by dpf_set_tiling (an autotuner).  For 129..256 inner particles
// the default is one wave per outer particle with four inner particles per
// lane, which measured faster than a 256-lane workgroup per particle.
static constexpr ClassShape kClasses[] = {{32, 1}, {64, 1}, {128, 1}, {64, 4},  {256, 4}, {256, 16},
                                          {32, 2}, {32, 4}, {64, 2},  {256, 1}, {128, 2},
                                          {16, 2}, {16, 4}, {16, 8}};
constexpr int kNumClasses = 14;
constexpr int kNumDefaultClasses = 6;
// Narrow classes, which stand in for the default ones of up to 128 lanes and
// one inner particle per lane (M <= ord): several outer particles per wave, so
// what a segment costs whatever its size (searches, scans, reductions, the
// offsets' Philox block) is shared by more inner particles, and fewer idle
// lanes where M does not fill the default class.  Their log-sum-exps add in
// the default class's order, so a filter's particles and weights are the same
// bits in either.  Built for the models of one or two inner components
// (narrow_from); indices from kNumClasses on, not public.  256 filters of
// 200 x 20: 51.8 us per step in 32 lanes, 34.3 in 8 x 3; 32 of 1000 x 100: 105 us
// in 128 lanes, 62 in 16 x 7.
// The last three (wave classes: also for the nonlinear model) take one wave per
// particle instead of the two of 128 lanes, or the four of 256 x 4 where at most
// half of its places would be used, of which all but the first await its outer
// draws.  One filter of 3805 particles of the nonlinear model: M = 303 70 us per
// step in 256 x 4, 44 in 64 x 6; M = 90 35 us in 128, 31 in 64 x 2.
struct NarrowShape {
  int seg, jpt;
  int ord, items;  // of the class stood in for
};
static constexpr NarrowShape kNarrow[] = {{8, 1, 32, 1},   {8, 2, 32, 1},   {8, 3, 32, 1},   {8, 4, 32, 1},
                                          {16, 3, 64, 1},  {16, 4, 64, 1},  {16, 5, 128, 1}, {16, 6, 128, 1},
                                          {16, 7, 128, 1}, {16, 8, 128, 1}, {64, 2, 128, 1}, {64, 6, 256, 4},
                                          {64, 8, 256, 4}};
constexpr int kNumNarrow = 13;
constexpr int kNarrowWave = 10;  // from here on: a wave per particle

struct TileClass {
  int cls;  // kClasses, then kNarrow
  int n_tiles;
  int4* d_tiles;
};

enum Op {
  OP_INIT_LA,
  OP_INIT_PLAIN,
  OP_LA_WEIGHTS,
  OP_DPF_WEIGHTS,
  OP_NEWCLOUD_LA,
  OP_NEWCLOUD_PLAIN,
  OP_LEARNED_INNER,
  OP_MOMENTS,
  OP_LA_WEIGHTS_FALLBACK,
  OP_NEWCLOUD_FALLBACK,
  OP_LA_WEIGHTS_NESTED
};

// Kernels between two look-ahead new-cloud launches.
enum EndOp { END_POST, END_FINISH, END_RUN_STATS, END_RESOLVE };
struct StepEnd {
  int took;   // bit of act that says a filter took the step (END_POST, END_FINISH)
  int next;   // END_POST: also the next step's statistics; END_RESOLVE: also the finished step's estimates
  int split;  // END_POST: END_FINISH or END_RESOLVE finishes the filters
};

// Extra arguments of OP_MOMENTS (feature rows for dpf_features).
struct MomArgs {
  const float* y;
  float* feat;
};
extern thread_local MomArgs g_mom_args;

// ------------------------------------------------------------ model engines
struct Engine {
  int dx, dz, dy;
  size_t n_raw;
  size_t n_total;
  void (*derive)(const double* raw, std::vector<float>& out);
  dpf_status (*launch)(int op, const StepArgs& a, const TileClass& tc, hipStream_t s);
  dpf_status (*mlp_state)(const StepArgs& a, hipStream_t s);  // null: no learned proposal
  dpf_status (*mdn_draw)(const StepArgs& a, hipStream_t s);
  bool moments;
  dpf_status (*rb)(const StepArgs& a, double* tmp, float* out, hipStream_t s);
  // plain DPF estimates (one workgroup per filter)
  dpf_status (*finalize)(const StepArgs& a, int F, hipStream_t s);
  // the kernels between look-ahead new clouds (EndOp)
  dpf_status (*post)(int op, const StepArgs& a, const int2* rgroups, int n_rgroups, int F, const StepEnd& e,
                     hipStream_t s);
  bool yhat;  // the look-ahead pass can form the predicted observation
  int narrow_from;  // the narrow classes from this one on are built
  bool plain_fused;  // a plain run's new-cloud kernel computes the next step's weights
};

extern const Engine kEngLinGauss, kEngNonLin, kEngHighDim, kEngTwoDim, kEngFourDim, kEngTwoDimZ;

}  // namespace dpf
