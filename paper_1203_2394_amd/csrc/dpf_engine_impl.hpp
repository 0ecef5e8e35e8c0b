// Per-model launchers of the step kernels, instantiated by each model's
// translation unit (dpf_eng_*.hip) through DPF_DEFINE_ENGINE.
#pragma once
#include <hip/hip_runtime.h>

#include "dpf_aux.hpp"
#include "dpf_engine.hpp"
#include "dpf_kernels.hpp"
#include "dpf_learned.hpp"
#include "dpf_mlp.hpp"
#include "dpf_rb.hpp"

namespace dpf {

// Models served by the learned proposal (the network's mixture is over a
// two-dimensional x; the features must fit its input).
template <class Mdl>
constexpr bool learned_model() { return Mdl::DX == 2 && has_moments<Mdl>(); }


template <class Mdl, int SEG, int JPT>
static void launch_op(int op, const StepArgs& a, int n, hipStream_t s) {
  switch (op) {
    case OP_INIT_LA:
      hipLaunchKernelGGL((k_init<Mdl, SEG, JPT, false>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_INIT_PLAIN:
      hipLaunchKernelGGL((k_init<Mdl, SEG, JPT, true>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_LA_WEIGHTS:
      hipLaunchKernelGGL((k_la_weights<Mdl, SEG, JPT>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_LA_WEIGHTS_NESTED:
      hipLaunchKernelGGL((k_la_weights_nested<Mdl, SEG, JPT>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_DPF_WEIGHTS:
      hipLaunchKernelGGL((k_dpf_weights<Mdl, SEG, JPT>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_NEWCLOUD_LA:
      hipLaunchKernelGGL((k_newcloud<Mdl, SEG, JPT, false>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_NEWCLOUD_PLAIN:
      hipLaunchKernelGGL((k_newcloud<Mdl, SEG, JPT, true>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_LEARNED_INNER:
      if constexpr (learned_model<Mdl>())
        hipLaunchKernelGGL((k_learned_inner<Mdl, SEG, JPT>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_LA_WEIGHTS_FALLBACK:
      if constexpr (learned_model<Mdl>())
        hipLaunchKernelGGL((k_la_weights_fallback<Mdl, SEG, JPT>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_NEWCLOUD_FALLBACK:
      if constexpr (learned_model<Mdl>())
        hipLaunchKernelGGL((k_newcloud_fallback<Mdl, SEG, JPT>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_MOMENTS:
      if constexpr (has_moments<Mdl>())
        hipLaunchKernelGGL((k_moments<Mdl, SEG, JPT>), dim3(n), dim3(kBlock), 0, s, a, g_mom_args.y,
                           g_mom_args.feat);
      break;
  }
}

// Narrow classes: the small models (a segment's fixed work outweighs its inner
// particles' there; NONLIN's eight-component clouds gain nothing in 8 or 16
// lanes, and the wide z in none).
template <class Mdl>
constexpr int narrow_from() { return Mdl::DZ <= 2 ? 0 : Mdl::DZ <= 8 ? kNarrowWave : kNumNarrow; }

template <class Mdl, int K>
static void launch_narrow(int op, const StepArgs& a, int n, hipStream_t s) {
  constexpr int SEG = kNarrow[K].seg, JPT = kNarrow[K].jpt, ORD = kNarrow[K].ord;
  static_assert(ORD <= 128 ? kNarrow[K].items == 1 : SEG == kWave, "SegLse");
  switch (op) {
    case OP_INIT_LA:
      hipLaunchKernelGGL((k_init<Mdl, SEG, JPT, false>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_INIT_PLAIN:
      hipLaunchKernelGGL((k_init<Mdl, SEG, JPT, true>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_LA_WEIGHTS:
      hipLaunchKernelGGL((k_la_weights<Mdl, SEG, JPT, ORD>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_LA_WEIGHTS_NESTED:
      hipLaunchKernelGGL((k_la_weights_nested<Mdl, SEG, JPT, ORD>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_DPF_WEIGHTS:
      hipLaunchKernelGGL((k_dpf_weights<Mdl, SEG, JPT, ORD>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_NEWCLOUD_LA:
      hipLaunchKernelGGL((k_newcloud<Mdl, SEG, JPT, false, ORD>), dim3(n), dim3(kBlock), 0, s, a);
      break;
    case OP_NEWCLOUD_PLAIN:
      hipLaunchKernelGGL((k_newcloud<Mdl, SEG, JPT, true, ORD>), dim3(n), dim3(kBlock), 0, s, a);
      break;
  }
}

// Narrow class k, of the classes K and on.
template <class Mdl, int K>
static bool launch_narrow_class(int k, int op, const StepArgs& a, int n, hipStream_t s) {
  if constexpr (K < kNumNarrow) {
    if (k != K) return launch_narrow_class<Mdl, K + 1>(k, op, a, n, s);
    // (the small models take 16 lanes where the first wave class would do)
    if constexpr (K != kNarrowWave || narrow_from<Mdl>() == kNarrowWave) launch_narrow<Mdl, K>(op, a, n, s);
    return true;
  } else {
    return false;
  }
}

// Row tiles per workgroup of k_mlp_fwd_state.  Two workgroups fit a CU, and
// each fetches the whole network (156 KB): past 512 of them the next round
// starts over, so larger batches take more rows per workgroup.  One, two and
// four tiles: 11.0, 11.2, 16.0 us at 8192 rows; 15.5, 14.8, 16.4 at 12288;
// 19.2, 15.7, 16.6 at 16384; 34.1, 26.0, 23.5 at 32768.
constexpr int mlp_row_tiles(int rows) { return rows <= 8192 ? 1 : rows <= 16384 ? 2 : 4; }

template <class Mdl>
static dpf_status engine_mlp_state(const StepArgs& a, hipStream_t s) {
  if constexpr (learned_model<Mdl>()) {
    const int rt = mlp_row_tiles(a.NT), rows = kMlpRows * rt;
    const dim3 n((a.NT + rows - 1) / rows);
    if (rt == 4) hipLaunchKernelGGL((k_mlp_fwd_state<Mdl, 4>), n, dim3(kBlock), 0, s, a);
    else if (rt == 2) hipLaunchKernelGGL((k_mlp_fwd_state<Mdl, 2>), n, dim3(kBlock), 0, s, a);
    else hipLaunchKernelGGL((k_mlp_fwd_state<Mdl, 1>), n, dim3(kBlock), 0, s, a);
    LAUNCH_CHECK("k_mlp_fwd_state");
    return DPF_OK;
  } else {
    return fail(DPF_EUNSUPPORTED, "no learned proposal for this model");
  }
}

template <class Mdl>
static dpf_status engine_mdn_draw(const StepArgs& a, hipStream_t s) {
  if constexpr (learned_model<Mdl>()) {
    hipLaunchKernelGGL(k_mdn_draw<Mdl>, dim3((a.NT + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a);
    LAUNCH_CHECK("k_mdn_draw");
    return DPF_OK;
  } else {
    return fail(DPF_EUNSUPPORTED, "no learned proposal for this model");
  }
}

template <class Mdl>
static dpf_status engine_launch(int op, const StepArgs& a, const TileClass& tc, hipStream_t s) {
  const int n = tc.n_tiles;
  if constexpr (narrow_from<Mdl>() < kNumNarrow) {
    if (tc.cls >= kNumClasses) {
      // (the learned passes and the moments run in the public classes)
      if (op == OP_LEARNED_INNER || op == OP_MOMENTS || op == OP_LA_WEIGHTS_FALLBACK || op == OP_NEWCLOUD_FALLBACK)
        return fail(DPF_EUNSUPPORTED, "operation %d has no narrow class", op);
      if (!launch_narrow_class<Mdl, narrow_from<Mdl>()>(tc.cls - kNumClasses, op, a, n, s))
        return fail(DPF_EUNSUPPORTED, "no kernel class %d", tc.cls);
      LAUNCH_CHECK("step kernel");
      return DPF_OK;
    }
  }
  switch (tc.cls) {
    case 0: launch_op<Mdl, 32, 1>(op, a, n, s); break;
    case 1: launch_op<Mdl, 64, 1>(op, a, n, s); break;
    case 2: launch_op<Mdl, 128, 1>(op, a, n, s); break;
    case 3: launch_op<Mdl, 64, 4>(op, a, n, s); break;
    case 4: launch_op<Mdl, 256, 4>(op, a, n, s); break;
    case 5: launch_op<Mdl, 256, 16>(op, a, n, s); break;
    case 6: launch_op<Mdl, 32, 2>(op, a, n, s); break;
    case 7: launch_op<Mdl, 32, 4>(op, a, n, s); break;
    case 8: launch_op<Mdl, 64, 2>(op, a, n, s); break;
    case 9: launch_op<Mdl, 256, 1>(op, a, n, s); break;
    case 10: launch_op<Mdl, 128, 2>(op, a, n, s); break;
    case 11: launch_op<Mdl, 16, 2>(op, a, n, s); break;
    case 12: launch_op<Mdl, 16, 4>(op, a, n, s); break;
    case 13: launch_op<Mdl, 16, 8>(op, a, n, s); break;
    default: return fail(DPF_EUNSUPPORTED, "no kernel class %d", tc.cls);
  }
  LAUNCH_CHECK("step kernel");
  return DPF_OK;
}

template <class Mdl>
static dpf_status engine_rb(const StepArgs& a, double* tmp, float* out, hipStream_t s) {
  constexpr int per = kBlock / kWave;  // outer particles per workgroup
  hipLaunchKernelGGL(k_rb_outer<Mdl>, dim3((a.NT + per - 1) / per), dim3(kBlock), 0, s, a, tmp);
  LAUNCH_CHECK("k_rb_outer");
  hipLaunchKernelGGL(k_rb_finish<Mdl::DX>, dim3(a.n_filters), dim3(kBlock), 0, s, a, (const double*)tmp, out);
  LAUNCH_CHECK("k_rb_finish");
  return DPF_OK;
}

template <class Mdl>
static dpf_status engine_finalize(const StepArgs& a, int F, hipStream_t s) {
  constexpr int DX = Mdl::DX, DZ = Mdl::DZ;
  hipLaunchKernelGGL((k_finalize<DX, DZ>), dim3(F), dim3(fin_block<DX, DZ>()), 0, s, a);
  LAUNCH_CHECK("k_finalize");
  return DPF_OK;
}

template <class Mdl, bool YH>
static dpf_status engine_step_end(int op, const StepArgs& a, const int2* rg, int n_rgroups, int F, const StepEnd& e,
                                  hipStream_t s) {
  constexpr int DX = Mdl::DX, DZ = Mdl::DZ;
  switch (op) {
    case END_POST:
      hipLaunchKernelGGL((k_post<DX, DZ, YH>), dim3(n_rgroups), dim3(kBlock), 0, s, a, rg, e.took, e.next, e.split);
      LAUNCH_CHECK("k_post");
      break;
    case END_FINISH:
      hipLaunchKernelGGL((k_post_end<DX, DZ, YH>), dim3(F), dim3(kBlock), 0, s, a, e.took);
      LAUNCH_CHECK("k_post_end");
      break;
    case END_RUN_STATS:
      hipLaunchKernelGGL((k_run_stats<DX, DZ, YH>), dim3(n_rgroups), dim3(kBlock), 0, s, a, rg);
      LAUNCH_CHECK("k_run_stats");
      break;
    case END_RESOLVE:
      hipLaunchKernelGGL((k_resolve<DX, DZ, YH>), dim3(n_rgroups), dim3(kBlock), 0, s, a, rg, e.next);
      LAUNCH_CHECK("k_resolve");
      break;
  }
  return DPF_OK;
}

// (the predicted observation's partial sums when the step formed them)
template <class Mdl>
static dpf_status engine_post(int op, const StepArgs& a, const int2* rg, int n_rgroups, int F, const StepEnd& e,
                              hipStream_t s) {
  if constexpr (has_yhat<Mdl>()) {
    if (a.yp != nullptr) return engine_step_end<Mdl, true>(op, a, rg, n_rgroups, F, e, s);
  }
  return engine_step_end<Mdl, false>(op, a, rg, n_rgroups, F, e, s);
}

// The engine table entry of model Mdl with parameter derivation DERIVE.
template <class Mdl>
static Engine make_engine(void (*derive)(const double*, std::vector<float>&)) {
  return Engine{Mdl::DX,
                Mdl::DZ,
                Mdl::DY,
                (size_t)Mdl::L::n_raw,
                (size_t)Mdl::L::n_total,
                derive,
                engine_launch<Mdl>,
                learned_model<Mdl>() ? engine_mlp_state<Mdl> : nullptr,
                learned_model<Mdl>() ? engine_mdn_draw<Mdl> : nullptr,
                has_moments<Mdl>(),
                engine_rb<Mdl>,
                engine_finalize<Mdl>,
                engine_post<Mdl>,
                has_yhat<Mdl>(),
                narrow_from<Mdl>(),
                !Mdl::kStreamZ};
}

}  // namespace dpf
