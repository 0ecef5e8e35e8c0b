// Step kernels of the look-ahead DPF (Section 2.2, Fig. 4) and of the plain
// DPF (Section 2, Fig. 2) for many independent filters of uneven sizes.
//
// Data layout in HBM (filter f, outer offset oo = ooff[f], inner offset
// io = ioff[f], sizes N = fN[f], M = fM[f]):
//   x    [DX][NT]            x[d * NT + oo + i]          (SoA, coalesced over i)
//   z    [sum N*DZ*M]         z[(io + i*M) * DZ + d*M + j] ([N][DZ][M] per filter)
//   lam  [sum N*M]            lam[io + i*M + j]           (log qbar, eq:qbar)
//   ell  [sum N*M]            look-ahead / measurement log-weights
//   logw [NT], anc [NT], sel [NT], kpart [NT][DZ]
// x, z and lam are double-buffered; cur[f] says which copy holds the state of
// filter f, so filters that sit a step out keep their state without a copy.
//
// A look-ahead step on its own is the weights kernel, the group statistics of
// the outer weights (filters of several resampling groups), the new-cloud
// kernel and the step end; in a run the new-cloud kernel also computes the next
// step's weights and the previous step's estimates, and only what the outer
// resampling needs stands between two of them.  A plain step likewise: weights,
// statistics, new cloud and estimates on its own, statistics and new cloud in a
// run.
//
// Per-particle kernels run one 256-thread workgroup per tile of 256/SEG
// consecutive outer particles of one filter (a "segment" of SEG lanes per
// particle, lane l handling inner indices l, l+SEG, ..., up to SEG*JPT).
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include "dpf_models.hpp"
#include "dpf_proj.hpp"
#include "dpf_rng.hpp"
#include "dpf_seg.hpp"

namespace dpf {

enum FlagBits : uint32_t {
  F_DEGENERATE_OUTER = 1u,
  F_DEGENERATE_INNER = 2u,
  F_NONFINITE = 4u,
  F_FALLBACK = 8u
};

constexpr int kResGroup = 256;  // outer weights per resampling workgroup
constexpr int kFeatMax = 32;    // input width of the learned-proposal network

// Models whose outer-particle features [x, y, cloud mean, cloud variance] fit
// the network keep the per-particle cloud moments up to date when asked.
template <class Mdl>
constexpr bool has_moments() { return Mdl::DX + Mdl::DY + 2 * Mdl::DZ <= kFeatMax; }

// Models whose predicted observation the look-ahead pass can form (they
// provide obs_mean).
template <class Mdl>
constexpr bool has_yhat() { return Mdl::DY == 1; }

// obs_pre as the plain weights form it, in their kernel and in a run's
// new-cloud kernel (a model of several observed components writes its
// roundings out; one component leaves the compiler no choice).
template <class Mdl>
__device__ __forceinline__ void obs_pre_weights(Prm P, const float* y, const float* x, float* r0) {
  if constexpr (Mdl::DY > 1 && !Mdl::kStreamZ) Mdl::obs_pre_plain(P, y, x, r0);
  else Mdl::obs_pre(P, y, x, r0);
}

// Number of z-free terms of log p(x' | x, z) (px_pre); 1 for models whose
// transition of x ignores z (unused there).
template <class Mdl>
constexpr int npx() {
  if constexpr (Mdl::kXdepZ) return Mdl::NPX;
  else return 1;
}

// Per-filter bookkeeping for the resampling groups.
struct FilterInfo {
  int rg_base;  // first resampling group of the filter
  int ngroup;   // its number of groups
  int pad0, pad1;
};

struct StepArgs {
  const float* prm;
  const int4* tiles;  // (filter, first outer index, tile index within filter, first resampling group)
  const int* fN;
  const int* fM;
  const int* ooff;
  const long long* ioff;
  const FilterInfo* finfo;
  int NT;
  int advance;   // 1: a step (time advances, estimates); 0: initialisation
  uint64_t seed;
  // the filters' progress (a view): time of the state; bit 0 of cur: copy
  // holding the state, bits 1, 2: copy 0 / copy 1 has identity cloud slots,
  // bit 3 (kCurPair): the last step's weights lie in the second ell / logw pair;
  // bit 0 of act: the filter takes the current step (set by the weights
  // kernel), bit 1: it took the previous one
  int* tcur;
  unsigned char* cur;
  unsigned char* act;
  // the view after the step, written by the new-cloud kernel of a look-ahead
  // step (a run's steps alternate between two views, so that every workgroup
  // of a launch reads one while its filters' first tiles write the other).
  // Null: the view above already is the one after the step (the statistics
  // kernel advanced it).
  int* tcur_n;
  unsigned char* cur_n;
  unsigned char* act_n;
  const unsigned char* active;  // [F] or null
  const int* run_Tf;            // [F] or null: filter steps while tcur < min(run_Tf, run_T)
  int run_T;
  const float* Y;
  long long y_tstride;  // y of filter f at time t: Y + (t-1) * y_tstride + f * DY
  float* x[2];
  float* z[2];
  float* lam[2];
  float* ell;
  float* logw;
  int* anc;
  int* sel;      // [NT] selected candidate (look-ahead) / inner ancestor (plain)
  float* kpart;  // [NT][DZ] per-particle sum_j qbar z (plain: of the proposals)
  const float* kpart_prev;  // the previous step's (a run alternates between two)
  double* gstat;  // [resampling groups + 64][4]: group max log w, sum, sum of squares (group scale)
  double* fstat;  // [F][4]: max log w, sum w, sum w^2, degenerate (0/1)
  float* ess;     // [F]
  double* dlogz;  // [F]
  double* loglik;  // [F] cumulative
  uint32_t* flags;  // [F]
  float* est_x;     // [F][DX]
  float* est_z;     // [F][DZ]
  float* trace_x;   // [T][F][DX] or null
  float* trace_z;   // [T][F][DZ] or null
  int n_filters;
  int dy;
  int dx, dz;
  int n_tiles;  // tiles of the class being launched (tile-looping kernels)
  int anc_ready;  // outer ancestors of filters of several resampling groups already in anc
  int n_head;     // head workgroups of a run's new-cloud launch, one per resampling group: the
                  // previous step's estimates
  const int2* rgroups;  // (filter, group) of each resampling workgroup
  const int4* ginfo;    // per resampling group: its filter's (first outer index, N, first group, groups)
  int n_commit;         // learned-step commit workgroups at the head of the launch
  int later_step;       // nested run: a step after its first
  int pair;             // the ell / logw pair this step reads (a run alternates between two)
  int finish;           // step on its own: the last workgroup of a filter finishes it
  int n_comp;           // companions per look-ahead candidate (nested estimator; 0: paired)
  // predicted observation (models with a one-dimensional y), or null: per
  // outer particle sum_j qbar h(xla, zla) of this step's look-ahead draws
  // (yp) and of the next step's (yp_next, written by a fused new-cloud
  // launch); the filter's yhat and its trace
  float* yp;
  float* yp_next;
  float* est_y;    // [F]
  float* trace_y;  // [T][F] or null
  // look-ahead state: cloud slot of each outer particle, per copy.  A step
  // that resamples by copying writes the identity; the learned step writes
  // its outer ancestors instead of moving the clouds.
  int* ind[2];
  float* mom;  // [NT][2 DZ] qbar-weighted cloud mean and variance, or null (not maintained)
  // learned step
  const unsigned char* mlp;  // network blob
  float* mdn;                // [NT][32] network outputs for the current step
  float* xtmp;               // [DX][NT] proposals x_t before resampling
  float* logq;               // [NT] log q of the proposals
  float* kpart_tmp;          // [NT][DZ]
  float* mom_tmp;            // [NT][2 DZ]
  unsigned char* fb;         // [F] 1 where the look-ahead step replaces the learned one; null otherwise
  uint32_t* lflags;          // [F] flags of the learned pass, kept only if it is accepted
  double ess_frac;           // fallback threshold on ESS / N
  // look-ahead run: the new-cloud kernel also computes the next step's
  // look-ahead weights from the clouds it builds (null: it does not), and the
  // estimates kernel records which filters take the next step
  float* ell_next;
  float* logw_next;
  double* gpart;  // [resampling groups][DX + DZ] partial sums of the estimates
  int* fcount;    // [F] workgroups of the step-end kernel done (back to 0 by the last)
};

__device__ __forceinline__ int copy_of(unsigned char c) { return c & 1; }
constexpr int kCurPair = 8;

// Every per-filter value a tile reads, fetched together: the empty asm needs
// them all before the early exits, so the loads go out in one round instead
// of a chain of dependent ones behind each branch.
struct FilterView {
  long long io;
  int N, M, oo, t, ngroup;
  int act, fb, cur;
};

__device__ __forceinline__ FilterView load_filter(const StepArgs& a, int f) {
  FilterView v;
  v.act = a.act[f];
  v.fb = a.fb != nullptr ? a.fb[f] : 1;
  v.N = a.fN[f];
  v.M = a.fM[f];
  v.oo = a.ooff[f];
  v.io = a.ioff[f];
  v.t = a.tcur[f];
  v.cur = a.cur[f];
  v.ngroup = a.finfo[f].ngroup;
  asm volatile("" ::"v"(v.act), "v"(v.fb), "v"(v.N), "v"(v.M), "v"(v.oo), "v"(v.io), "v"(v.t), "v"(v.cur),
               "v"(v.ngroup));
  return v;
}
__device__ __forceinline__ bool ident_slots(unsigned char c, int copy) { return (c >> (1 + copy)) & 1; }

// fz_pre (transition out of time ts) for a whole segment whose lanes share
// the outer particle: lane q of each wave's part of the segment evaluates
// component q once, and the components are broadcast (readlane within a
// wave, lane permutes when two segments share a wave) instead of every lane
// evaluating all of them.
template <class Mdl, int SEG>
__device__ __forceinline__ void fz_pre_seg(Prm P, const float* xp, const float* xn, int ts, float* pre) {
  constexpr int DZ = Mdl::DZ;
  constexpr int W = SEG < 64 ? SEG : 64;
  if constexpr (DZ > W || Mdl::NPRE != DZ) {
    Mdl::fz_pre(P, xp, xn, ts, pre);
  } else {
    const int lane = threadIdx.x & 63;
    const int q = lane % W;
    const float mine = Mdl::fz_pre_k(P, xp, xn, ts, q < DZ ? q : 0);
    if constexpr (W == 64) {
#pragma unroll
      for (int k = 0; k < DZ; ++k) pre[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), k));
    } else {
      const int base = lane - q;
#pragma unroll
      for (int k = 0; k < DZ; ++k) pre[k] = __shfl(mine, base + k);
    }
  }
}

// Minimum waves per SIMD the compiler must leave room for: two for the
// wide-z models (their per-particle arrays would otherwise take the whole
// register file for one wave), no constraint otherwise.
template <class Mdl>
constexpr int min_waves() {
  return Mdl::kStreamZ ? 2 : 1;
}

// Whether filter f takes this step: the caller's mask and the run limits,
// evaluated by the weights kernel (before the time advances) and recorded in
// act[f] for the later kernels of the step.
__device__ __forceinline__ bool step_active(const StepArgs& a, int f) {
  if (a.active != nullptr && a.active[f] == 0) return false;
  const int lim = a.run_Tf ? min(a.run_Tf[f], a.run_T) : a.run_T;
  return a.tcur[f] < lim;
}

template <class Mdl>
__device__ __forceinline__ void load_y(const StepArgs& a, int f, int t, float* y) {
  const float* yp = a.Y + (long long)(t - 1) * a.y_tstride + (long long)f * Mdl::DY;
#pragma unroll
  for (int k = 0; k < Mdl::DY; ++k) y[k] = yp[k];
}

template <class Mdl>
__device__ __forceinline__ const float* y_row(const StepArgs& a, int f, int t) {
  return a.Y + (long long)(t - 1) * a.y_tstride + (long long)f * Mdl::DY;
}

// Online log-sum-exp accumulator (non-finite values are skipped): a new
// maximum rescales the sum, s e^(m - v) + 1, another value adds e^(v - m) --
// the same exponential either way, so no branch.
struct Lse {
  float m = -INFINITY, s = 0.f;
  __device__ __forceinline__ void add(float v) {
    const bool ok = finitef(v), up = v > m;
    const float e = fast_exp(-fabsf(v - m));
    const float t = up ? s * e + 1.0f : s + e;
    s = ok ? t : s;
    m = ok && up ? v : m;
  }
};

// p[i] with a 32-bit byte offset (a wave-uniform p stays in scalar registers).
__device__ __forceinline__ float at32(const float* p, int i) {
  return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(p) + (uint32_t)i * 4u);
}
// A lane's JPT consecutive items from row[j0] on, in loads of up to 16 bytes
// (item by item, each load of a wave would touch every line of the segment's
// row again).  j0 is clamped into the row of n items, so up to JPT - 1 floats
// after the row are read too -- the next row, or the room that the workspace
// leaves after the last one; the caller masks items by ls JPT + r < n.
template <int JPT>
struct Items {
  float v[JPT];
};
template <int JPT>
__device__ __forceinline__ Items<JPT> load_items(const float* row, int j0, int n) {
  return *reinterpret_cast<const Items<JPT>*>(row + min(j0, n - 1));
}
__device__ __forceinline__ void put32(float* p, int i, float v) {
  *reinterpret_cast<float*>(reinterpret_cast<char*>(p) + (uint32_t)i * 4u) = v;
}

template <int SEG>
__device__ __forceinline__ float seg_lse(Lse l, SegScratch& sh) {
  const float m = seg_max<SEG>(l.m, sh);
  const float sc = (l.m == -INFINITY) ? 0.f : l.s * fast_exp(l.m - m);
  const float s = seg_sum<SEG>(sc, sh);
  return (m == -INFINITY) ? -INFINITY : m + fast_log(s);
}

// Log-sum-exp over a narrow segment's items (v[r]: item ls + r SEG, -inf where
// there is none): the bits that a segment of ORD lanes with one item each
// gets, which the narrow class stands in for (these weights decide the
// resampling).
template <int SEG, int JPT, int ORD>
__device__ __forceinline__ float seg_lse_ord(const float* v, SegScratch& sh) {
  float ml = -INFINITY, x[JPT];
#pragma unroll
  for (int r = 0; r < JPT; ++r)
    if (finitef(v[r])) ml = fmaxf(ml, v[r]);
  const float m = seg_max<SEG>(ml, sh);
#pragma unroll
  for (int r = 0; r < JPT; ++r) x[r] = finitef(v[r]) ? fast_exp(v[r] - m) : 0.f;
  const float s = seg_sum_ord<SEG, JPT, ORD>(x);
  return (m == -INFINITY) ? -INFINITY : m + fast_log(s);
}

// A segment's accumulated log-sum-exp and sum: ORD = 0 each lane's items as
// they come (online), then the lanes; 8 or 16 lanes in the order of an ORD-lane
// segment with one item per lane; a wave (item j in lane j % 64) in the order
// of ORD lanes with any: lane j % ORD's items as they come, then its wave's
// lanes, then the waves.
template <int SEG, int JPT, int ORD>
struct SegLse {
  static constexpr bool kOne = ORD > 0 && SEG < kWave;
  static constexpr int NL = ORD > kWave && !kOne ? ORD / kWave : 1;
  Lse l[NL];
  float v[kOne ? JPT : 1];
  __device__ SegLse() {
#pragma unroll
    for (int r = 0; r < (kOne ? JPT : 1); ++r) v[r] = -INFINITY;
  }
  __device__ __forceinline__ void add(int r, float e) {
    if constexpr (kOne) v[r] = e;
    else l[r % NL].add(e);
  }
  __device__ __forceinline__ float get(SegScratch& sh) const {
    if constexpr (kOne) {
      return seg_lse_ord<SEG, JPT, ORD>(v, sh);
    } else if constexpr (NL == 1) {
      return seg_lse<SEG>(l[0], sh);
    } else {
      float m = l[0].m;
#pragma unroll
      for (int w = 1; w < NL; ++w) m = fmaxf(m, l[w].m);
      m = seg_max<SEG>(m, sh);
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < NL; ++w) {
        const float sw = seg_sum<SEG>((l[w].m == -INFINITY) ? 0.f : l[w].s * fast_exp(l[w].m - m), sh);
        s = w == 0 ? sw : s + sw;
      }
      return (m == -INFINITY) ? -INFINITY : m + fast_log(s);
    }
  }
};
template <int SEG, int JPT, int ORD>
struct SegSum {
  static constexpr bool kOne = ORD > 0 && SEG < kWave;
  static constexpr int NL = ORD > kWave && !kOne ? ORD / kWave : 1;
  float v[kOne ? JPT : NL];
  __device__ SegSum() {
#pragma unroll
    for (int r = 0; r < (kOne ? JPT : NL); ++r) v[r] = 0.f;
  }
  __device__ __forceinline__ void add(int r, float q, float h) {
    if constexpr (kOne) v[r] = q * h;
    else v[r % NL] += q * h;
  }
  __device__ __forceinline__ float get(SegScratch& sh) const {
    if constexpr (kOne) {
      return seg_sum_ord<SEG, JPT, ORD>(v);
    } else if constexpr (NL == 1) {
      return seg_sum<SEG>(v[0], sh);
    } else {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < NL; ++w) {
        const float sw = seg_sum<SEG>(v[w], sh);
        s = w == 0 ? sw : s + sw;
      }
      return s;
    }
  }
};

// Block-wide (256 threads) FP64 reductions and scans in a fixed order:
// DPP within each wave, then the four wave results in order.
__device__ __forceinline__ double block_sum_256(double v, double* red4) {
  v = seg_reduce_wave<OpAdd, kWave>(v);
  if ((threadIdx.x & (kWave - 1)) == 0) red4[threadIdx.x / kWave] = v;
  __syncthreads();
  const double r = ((red4[0] + red4[1]) + red4[2]) + red4[3];
  __syncthreads();
  return r;
}

__device__ __forceinline__ double block_scan_incl_256(double v, double* red4) {
  const int w = threadIdx.x / kWave;
  v = seg_scan_wave<kWave>(v);
  if ((threadIdx.x & (kWave - 1)) == kWave - 1) red4[w] = v;
  __syncthreads();
  double pre = 0.0;
  for (int q = 0; q < w; ++q) pre += red4[q];
  __syncthreads();
  return v + pre;
}

// Block-wide stream compaction in thread order: the values of threads with
// pred go to out[0..total); returns total; incl receives the number of pred
// threads up to and including this one.
__device__ __forceinline__ int block_compact(bool pred, int value, int* out, int* wcnt, int* incl) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const unsigned long long b = __ballot(pred);
  const int r = __popcll(b & ((1ull << lane) - 1ull));
  if (lane == 0) wcnt[w] = __popcll(b);
  __syncthreads();
  int off = 0, total = 0;
#pragma unroll
  for (int q = 0; q < kBlock / kWave; ++q) {
    const int c = wcnt[q];
    if (q < w) off += c;
    total += c;
  }
  if (pred) out[off + r] = value;
  if (incl) *incl = off + r + (pred ? 1 : 0);
  __syncthreads();
  return total;
}

// ------------------------------------------------------------ initialisation
// Prior draws [x_0; z_0] ~ N(0, I) (INIT_X at (0, i, 0), INIT_Z at (0, i, j)).
// Look-ahead state: lam_0 = -log M, written to copy 0.  Plain DPF: the prior
// goes to copy 1 with ell = 0 and anc = identity, after which the proposal
// kernel runs with t = 0 (no y_0 is consumed).
template <class Mdl, int SEG, int JPT, bool PLAIN>
static __global__ __launch_bounds__(kBlock) void k_init(StepArgs a) {
  const int4 tile = a.tiles[blockIdx.x];
  const int f = tile.x;
  const int N = a.fN[f], M = a.fM[f];
  const int i = tile.y + threadIdx.x / SEG;
  const int ls = threadIdx.x % SEG;
  if (i >= N) return;
  const int oo = a.ooff[f];
  const long long io = a.ioff[f];
  const Key key = make_key(a.seed, (uint32_t)f);
  const int dst = PLAIN ? 1 : 0;
  if (ls == 0) {
    float x0[Mdl::DX];
    normals<Mdl::DX>(key, 0u, (uint32_t)i, 0u, P_INIT_X, x0);
#pragma unroll
    for (int d = 0; d < Mdl::DX; ++d) a.x[dst][(long long)d * a.NT + oo + i] = x0[d];
    if (PLAIN) a.anc[oo + i] = i;
  }
  const float lam0 = -fast_log((float)M);
  float* zrow = a.z[dst] + (io + (long long)i * M) * Mdl::DZ;
  for (int r = 0; r < JPT; ++r) {
    const int j = ls + r * SEG;
    if (j >= M) break;
    float z0[Mdl::DZ];
    normals<Mdl::DZ>(key, 0u, (uint32_t)i, (uint32_t)j, P_INIT_Z, z0);
#pragma unroll
    for (int d = 0; d < Mdl::DZ; ++d) zrow[d * M + j] = z0[d];
    if (PLAIN)
      a.ell[io + (long long)i * M + j] = 0.f;
    else
      a.lam[dst][io + (long long)i * M + j] = lam0;
  }
}

// ------------------------------------------------------- look-ahead weights
// Fig. 4 steps 1-2: for every (i, j) one candidate x from the j-th inner
// component (LA_X normals at (t, i, j)) and its companion z (LA_Z), then
// ell = lam + log p(y_t | xla, zla) (eq:weightsMC) and the per-particle
// log-sum-exp log w_i.

// log p(y_t | xla, zla) of inner particle (i, j) at time t from its outer x
// and its z; ell = lam + that (la_ell).
//
// The inputs pass through empty asm first: the compiler cannot merge this
// arithmetic with the caller's on the same values, so the weights kernel and
// the new-cloud kernel (a look-ahead run) compile it alike and get the same
// bits.
template <class Mdl, bool H = false>
__device__ __forceinline__ float la_logpy(const StepArgs& a, const Key& key, int t, int i, int j, const float* xi,
                                          const float* zi, const float* yi, float* hout = nullptr) {
  float x[Mdl::DX], z[Mdl::DZ], y[Mdl::DY];
#pragma unroll
  for (int d = 0; d < Mdl::DX; ++d) {
    x[d] = xi[d];
    asm volatile("" : "+v"(x[d]));
  }
#pragma unroll
  for (int d = 0; d < Mdl::DZ; ++d) {
    z[d] = zi[d];
    asm volatile("" : "+v"(z[d]));
  }
#pragma unroll
  for (int d = 0; d < Mdl::DY; ++d) y[d] = yi[d];
  // one draw per candidate: x's normals first, then z's
  float nu[Mdl::DX + Mdl::DZ], xl[Mdl::DX], pre[Mdl::NPRE], zl[Mdl::DZ], r0[Mdl::DY];
  normals<Mdl::DX + Mdl::DZ>(key, (uint32_t)t, (uint32_t)i, (uint32_t)j, P_LA_X, nu);
  Mdl::fx(as_prm(a.prm), x, z, nu, t - 1, xl);
  Mdl::fz_pre(as_prm(a.prm), x, xl, t - 1, pre);
  Mdl::fz_post(as_prm(a.prm), pre, z, nu + Mdl::DX, zl);
  Mdl::obs_pre(as_prm(a.prm), y, xl, r0);
  if constexpr (H) {
    // the noise-free observation of the draw, on opaque copies (no sharing
    // with the likelihood's arithmetic)
    float xh[Mdl::DX], zh[Mdl::DZ];
#pragma unroll
    for (int d = 0; d < Mdl::DX; ++d) {
      xh[d] = xl[d];
      asm volatile("" : "+v"(xh[d]));
    }
#pragma unroll
    for (int d = 0; d < Mdl::DZ; ++d) {
      zh[d] = zl[d];
      asm volatile("" : "+v"(zh[d]));
    }
    Mdl::obs_mean(as_prm(a.prm), xh, zh, hout);
  }
  return Mdl::logpy_post(as_prm(a.prm), r0, zl);
}

// The same for a wide-z model, for the 64 inner particles of a wave at once
// (converged code; lane l's particle j): the candidate's z component by
// component, each pair of components into the matrix-core residual
// (WaveProj; ca its A values, yrow the observation y_t).
template <class Mdl>
__device__ __forceinline__ float la_logpy_wave(const StepArgs& a, const Key& key, int t, int i, int j,
                                               const float* xi, const float* zi, const float* yrow,
                                               const float* ca) {
  static_assert(Mdl::kStreamZ && Mdl::DZ % 2 == 0 && Mdl::DX == 4,
                "la_logpy_wave: wide-z models, DX = 4, DZ even");
  const Prm P = as_prm(a.prm);
  float x[Mdl::DX], z[Mdl::DZ];
#pragma unroll
  for (int d = 0; d < Mdl::DX; ++d) {
    x[d] = xi[d];
    asm volatile("" : "+v"(x[d]));
  }
#pragma unroll
  for (int d = 0; d < Mdl::DZ; ++d) {
    z[d] = zi[d];
    asm volatile("" : "+v"(z[d]));
  }
  // the candidate's draw: block 0 gives x's four normals (and its remnant
  // uniform), z's normals 4 .. 4 + DZ - 1 follow in pairs
  float nu_x[Mdl::DX], xl[Mdl::DX], c[Mdl::NPL];
  const Words w0 = draw(key, (uint32_t)t, (uint32_t)i, (uint32_t)j, P_LA_X, 0u);
  box_muller(w0.w[0], w0.w[1], nu_x[0], nu_x[1]);
  box_muller(w0.w[2], w0.w[3], nu_x[2], nu_x[3]);
  Mdl::fx(P, x, z, nu_x, t - 1, xl);
  Mdl::fz_lite(P, x, xl, t - 1, c);
  WaveProj<Mdl> pj;
  pj.start();
  const float sz = P[Mdl::Layout::sz];
  auto nxt = Mdl::load_pair(P, 0);  // the rows of the next pair, fetched one ahead
  normal_pairs<Mdl::DX, Mdl::DX + Mdl::DZ, true>(
      key, (uint32_t)t, (uint32_t)i, (uint32_t)j, P_LA_X, r24f(w0), [&](int d, float n0, float n1) {
        const int kk = d - Mdl::DX;
        const auto row = nxt;
        if (kk + 2 < Mdl::DZ) nxt = Mdl::load_pair(P, kk / 2 + 1);
        const float z0 = Mdl::fz_post_row(row, 0, sz, Mdl::fz_pre_row(row, 0, c), z, n0, kk);
        const float z1 = Mdl::fz_post_row(row, 1, sz, Mdl::fz_pre_row(row, 1, c), z, n1, kk + 1);
        pj.add(ca[kk / 2], z0, z1);
      });
  return pj.logpy(P, yrow);
}

// lam + g as a separate rounding: g is opaque to the compiler, so no
// multiply inside it is fused into this add (the weights kernel and the
// new-cloud kernel, which adds lam later, get the same bits).
__device__ __forceinline__ float la_ell(float lam, float g) {
  asm volatile("" : "+v"(g));
  return lam + g;
}
template <class Mdl, int SEG, int JPT, int ORD = 0>
__device__ __forceinline__ void la_weights_tile(const StepArgs& a, int ti, bool fallback) {
  __shared__ SegScratch sh;
  const int4 tile = a.tiles[ti];
  const int f = tile.x;
  const int am = a.active != nullptr ? a.active[f] : 1;
  const int tf = a.run_Tf != nullptr ? a.run_Tf[f] : 0x7fffffff;
  asm volatile("" ::"v"(am), "v"(tf));
  const FilterView fv = load_filter(a, f);
  const bool act = am != 0 && fv.t < min(tf, a.run_T);  // step_active
  if (!fallback && tile.z == 0 && threadIdx.x == 0) a.act[f] = act ? 1 : 0;
  if (!act) return;
  const int N = fv.N, M = fv.M;
  const int i = tile.y + threadIdx.x / SEG;
  const int ls = threadIdx.x % SEG;
  const bool vi = i < N;
  const int oo = fv.oo;
  const long long io = fv.io;
  const int t = fv.t + 1;
  const unsigned char cb = (unsigned char)fv.cur;
  const int src = copy_of(cb);
  const Key key = make_key(a.seed, (uint32_t)f);
  const int ci = vi ? (ident_slots(cb, src) ? i : a.ind[src][oo + i]) : 0;

  float y[Mdl::DY], x[Mdl::DX];
  load_y<Mdl>(a, f, t, y);
#pragma unroll
  for (int d = 0; d < Mdl::DX; ++d) x[d] = vi ? a.x[src][(long long)d * a.NT + oo + i] : 0.f;

  const float* zrow = a.z[src] + (io + (long long)ci * M) * Mdl::DZ;
  const float* lrow = a.lam[src] + io + (long long)ci * M;
  float* erow = a.ell + io + (long long)(vi ? i : 0) * M;
  SegLse<SEG, JPT, ORD> acc;
  constexpr bool kH = has_yhat<Mdl>();
  const bool want_h = kH && a.yp != nullptr && !fallback;
  SegSum<SEG, JPT, ORD> hv;  // of the draws' qbar h(xla, zla)
  if constexpr (Mdl::kStreamZ) {
    // wide z: every lane of the wave takes part in the matrix-core residual
    float ca[WaveProj<Mdl>::NA];
    WaveProj<Mdl>::load_a(as_prm(a.prm), ca);
    __shared__ __align__(16) float yrow[Mdl::DY];
    if (threadIdx.x < Mdl::DY) yrow[threadIdx.x] = y_row<Mdl>(a, f, t)[threadIdx.x];
    __syncthreads();
    for (int r = 0; r < JPT; ++r) {
      const int j = ls + r * SEG;
      const bool on = vi && j < M;
      float z[Mdl::DZ];
      int Mr = __builtin_amdgcn_readfirstlane(M);  // opaque: DZ row bases kept over the items would spill
      asm volatile("" : "+s"(Mr));
#pragma unroll
      for (int d = 0; d < Mdl::DZ; ++d) z[d] = on ? at32(zrow + d * Mr, j) : 0.f;
      const float lj = on ? lrow[j] : 0.f;
      const float g = la_logpy_wave<Mdl>(a, key, t, i, on ? j : 0, x, z, yrow, ca);
      if (on) {
        const float e = la_ell(lj, g);
        erow[j] = e;
        acc.add(r, e);
      }
    }
  } else {
#pragma unroll
  for (int r = 0; r < JPT; ++r) {
    const int j = ls + r * SEG;
    if (vi && j < M) {
      float z[Mdl::DZ];
#pragma unroll
      for (int d = 0; d < Mdl::DZ; ++d) z[d] = zrow[d * M + j];
      const float lj = lrow[j];
      float g;
      if (want_h) {
        float h[1];
        g = la_logpy<Mdl, kH>(a, key, t, i, j, x, z, y, h);
        hv.add(r, fast_exp(lj), h[0]);
      } else {
        g = la_logpy<Mdl>(a, key, t, i, j, x, z, y);
      }
      const float e = la_ell(lj, g);
      erow[j] = e;
      acc.add(r, e);
    }
  }
  }
  const float lw = acc.get(sh);
  if (vi && ls == 0) a.logw[oo + i] = lw;
  if (want_h) {
    const float hs = hv.get(sh);
    if (vi && ls == 0) a.yp[oo + i] = hs;
  }
}

// Nested look-ahead weights (Fig. 4 step 1 with N_z' = K companions per
// candidate, eq:weightsMC): candidate m of outer particle i is drawn from
// inner component m as in the paired form (LA_X at (t, i, m)); its K
// companions take ancestors by systematic resampling (U53 LA_B at
// (t, i, m)) of the inner weights conditioned on the candidate,
// kappa_j = lam_j + log p(xla_m | x_i, z_j) (eq:qnobar), and are propagated
// with the inner prior (LA_Z normals k dz .. k dz + dz - 1 at (t, i, m));
// ell_m = lam_m + log (1/K) sum_k p(y_t | xla_m, zla_mk).  When p(x' | x, z)
// does not depend on z the conditioned weights are lam itself: one
// cumulative sum serves every candidate and each lane scores its own
// candidates.  Otherwise the segment walks the candidates in order, forming
// each one's conditioned cumulative sum together and spreading its
// companions over the lanes.
template <class Mdl, int SEG, int JPT, int ORD = 0>
__device__ __forceinline__ void la_weights_nested_tile(const StepArgs& a, int ti) {
  constexpr int DX = Mdl::DX, DZ = Mdl::DZ, DY = Mdl::DY;
  constexpr int NSEG = kBlock / SEG, CAP = SEG * JPT;
  constexpr bool kCond = Mdl::kXdepZ;
  constexpr bool kHoldZ = kCond && JPT * DZ <= 64;  // the lane's cloud stays in registers
  constexpr bool kAux = kCond && Mdl::kAux;
  __shared__ SegScratch sh;
  __shared__ double cdf[NSEG][kCond ? 1 : CAP];
  __shared__ float cz[NSEG][kCond ? CAP : 1][DZ];
  __shared__ float caux[NSEG][kAux ? CAP : 1];
  __shared__ float lms[NSEG][kCond ? CAP : 1];
  // small clouds: each lane's conditioned log-weights of its current
  // candidate, then, per pair of items, the first one's weight and the
  // cumulative weight after the second (the sum between them is one addition:
  // a quarter less LDS than all sums, three workgroups per CU instead of two),
  // [pair][lane]: a lane's entries lie in its own banks whatever the pair
  constexpr bool kCum = kCond && CAP <= 32;
  __shared__ double cum2[kCum ? CAP / 2 : 1][kCum ? kBlock : 1];
  __shared__ float wev[kCum ? CAP / 2 : 1][kCum ? kBlock : 1];
  constexpr bool kH = has_yhat<Mdl>();
  const int4 tile = a.tiles[ti];
  const int f = tile.x;
  const int am = a.active != nullptr ? a.active[f] : 1;
  const int tf = a.run_Tf != nullptr ? a.run_Tf[f] : 0x7fffffff;
  asm volatile("" ::"v"(am), "v"(tf));
  const FilterView fv = load_filter(a, f);
  const bool act = am != 0 && fv.t < min(tf, a.run_T);  // step_active
  // (in a run, bit 1 is the previous step's new-cloud kernel's)
  if (tile.z == 0 && threadIdx.x == 0)
    a.act[f] = (unsigned char)((act ? 1 : 0) | (a.later_step ? a.act[f] & 2 : 0));
  if (!act) return;
  const int N = fv.N, M = fv.M, K = a.n_comp;
  constexpr int CPB = comp_per_block<DZ>();  // companions per block of normals
  const int s = threadIdx.x / SEG;
  const int i = tile.y + s;
  const int ls = threadIdx.x % SEG;
  const bool vi = i < N;
  const int oo = fv.oo;
  const long long io = fv.io;
  const int t = fv.t + 1;
  const unsigned char cb = (unsigned char)fv.cur;
  const int src = copy_of(cb);
  const Key key = make_key(a.seed, (uint32_t)f);
  const int ci = vi ? (ident_slots(cb, src) ? i : a.ind[src][oo + i]) : 0;
  // - log K: with one item per lane the compiler fuses its product into the
  // difference, with several (where it is formed once) not; the classes that
  // stand in for one item do as those
  const float log2K = __builtin_amdgcn_logf((float)K);
  const float logK = fast_log((float)K);
  auto less_log_k = [&](float v) -> float {
    if constexpr (ORD > 0 && ORD <= 128) return __builtin_fmaf(-log2K, 0.6931471805599453f, v);
    else return v - logK;
  };

  float y[DY], x[DX];
  load_y<Mdl>(a, f, t, y);
#pragma unroll
  for (int d = 0; d < DX; ++d) x[d] = vi ? a.x[src][(long long)d * a.NT + oo + i] : 0.f;
  const float* zrow = a.z[src] + (io + (long long)ci * M) * DZ;
  const float* lrow = a.lam[src] + io + (long long)ci * M;
  float* erow = a.ell + io + (long long)(vi ? i : 0) * M;

  // candidates (as in the paired form) and the lanes' inner weights
  float lamv[JPT], xl[JPT][DX];
  float zh[kHoldZ ? JPT : 1][kHoldZ ? DZ : 1];
#pragma unroll
  for (int r = 0; r < JPT; ++r) {
    const int j = ls + r * SEG;
    lamv[r] = -INFINITY;
#pragma unroll
    for (int d = 0; d < DX; ++d) xl[r][d] = 0.f;
    if (vi && j < M) {
      float z[DZ], nu[DX];
#pragma unroll
      for (int d = 0; d < DZ; ++d) z[d] = zrow[d * M + j];
      if constexpr (kHoldZ) {
#pragma unroll
        for (int d = 0; d < DZ; ++d) zh[kHoldZ ? r : 0][kHoldZ ? d : 0] = z[d];
      }
      lamv[r] = lrow[j];
      normals<DX>(key, (uint32_t)t, (uint32_t)i, (uint32_t)j, P_LA_X, nu);
      Mdl::fx(as_prm(a.prm), x, z, nu, t - 1, xl[r]);
      if constexpr (kCond) lms[s][kCond ? j : 0] = lamv[r];
    }
  }
  // predicted observation: sum over the lane's candidates of qbar times the
  // mean of h over their companions
  const bool want_h = kH && a.yp != nullptr;
  const float invK = 1.0f / (float)K;
  SegSum<SEG, JPT, ORD> hv;
  float ev[JPT];
#pragma unroll
  for (int r = 0; r < JPT; ++r) ev[r] = -INFINITY;

  if constexpr (!kCond) {
    // ---- one cumulative sum of the inner weights for every candidate
    float mloc = -INFINITY;
#pragma unroll
    for (int r = 0; r < JPT; ++r)
      if (finitef(lamv[r])) mloc = fmaxf(mloc, lamv[r]);
    const float m0 = seg_max<SEG>(mloc, sh);
    const bool deg = !(m0 > -INFINITY);
    double carry = 0.0;
#pragma unroll
    for (int r = 0; r < JPT; ++r) {
      const int j = ls + r * SEG;
      double w = 0.0;
      if (j < M) w = deg ? 1.0 : (finitef(lamv[r]) ? (double)fast_exp(lamv[r] - m0) : 0.0);
      double tot;
      const double c = seg_scan_incl<SEG>(w, sh, tot);
      cdf[s][r * SEG + ls] = carry + c;
      carry += tot;
    }
    seg_lds_sync<SEG>();
    const double total = cdf[s][M - 1];
#pragma unroll
    for (int r = 0; r < JPT; ++r) {
      const int j = ls + r * SEG;
      if (vi && j < M) {
        float pre[Mdl::NPRE], r0[DY];
        Mdl::fz_pre(as_prm(a.prm), x, xl[r], t - 1, pre);
        Mdl::obs_pre(as_prm(a.prm), y, xl[r], r0);
        const SysPoints pts(uniform53_ab(key, (uint32_t)t, (uint32_t)i, (uint32_t)j, P_LA_B), total, K);
        Lse acck;
        float hk = 0.f;
        for (int k0 = 0; k0 < K; k0 += CPB) {
          float nb[CPB * DZ];
          double P[CPB];
          int bk[CPB];
          normals_kb<DZ>(key, (uint32_t)t, (uint32_t)i, (uint32_t)j, P_LA_Z, k0, nb);
#pragma unroll
          for (int q = 0; q < CPB; ++q) P[q] = k0 + q < K ? pts(k0 + q) : 0.0;
          cdf_find<CAP, CPB>(cdf[s], M, total, P, bk);
#pragma unroll
          for (int q = 0; q < CPB; ++q) {
            const int k = k0 + q;
            if (k >= K) break;
            const int b = bk[q];
            float zg[DZ], zc[DZ];
#pragma unroll
            for (int d = 0; d < DZ; ++d) zg[d] = zrow[d * M + b];
            Mdl::fz_post(as_prm(a.prm), pre, zg, nb + q * DZ, zc);
            acck.add(Mdl::logpy_post(as_prm(a.prm), r0, zc));
            if constexpr (kH) {
              if (want_h) {
                float h[1];
                Mdl::obs_mean(as_prm(a.prm), xl[r], zc, h);
                hk += h[0];
              }
            }
          }
        }
        const float g = (acck.m == -INFINITY) ? -INFINITY : less_log_k(acck.m + fast_log(acck.s));
        ev[r] = la_ell(lamv[r], g);
        if (want_h) hv.add(r, fast_exp(lamv[r]), hk * invK);
      }
    }
  } else {
    // ---- each lane scores its own candidates.  Per candidate, passes over
    // the segment's cloud (staged in LDS, read by every lane at the same
    // index, with what the model needs of each z alone): the largest
    // conditioned log-weight, then the FP64 cumulative sum in inner order.
    // Companion k takes the first index whose cumulative weight exceeds point
    // k; points at or past the total take the last index with positive
    // weight.  Clouds of up to 32 keep the log-weights and the cumulative
    // sums in the lane's LDS column and search it (256 filters of 200 x 20,
    // K = 8: 99 us with the log-weights and their divisions formed again in each
    // pass and a cursor per lane, 58 us now); larger ones form them again.
#pragma unroll
    for (int r = 0; r < JPT; ++r) {
      const int j = ls + r * SEG;
      if (j < M) {
#pragma unroll
        for (int d = 0; d < DZ; ++d)
          cz[s][kCond ? j : 0][d] = vi ? (kHoldZ ? zh[kHoldZ ? r : 0][kHoldZ ? d : 0] : zrow[d * M + j]) : 0.f;
        if constexpr (kAux) caux[s][kAux ? j : 0] = Mdl::aux(cz[s][kCond ? j : 0]);
      }
    }
    // items beyond M: no weight (up to a multiple of four), +inf for the searches
#pragma unroll
    for (int r = 0; r < JPT; ++r) {
      const int j = ls + r * SEG;
      if (j >= M) {
#pragma unroll
        for (int d = 0; d < DZ; ++d) cz[s][kCond ? j : 0][d] = 0.f;
        if constexpr (kAux) caux[s][kAux ? j : 0] = 0.f;
        lms[s][kCond ? j : 0] = -INFINITY;
      }
    }
    if constexpr (kCum) {
      for (int q = (M + 3) / 4 * 2; q < CAP / 2; ++q) cum2[kCum ? q : 0][kCum ? threadIdx.x : 0] = INFINITY;
    }
    seg_lds_sync<SEG>();
    if (vi) {
#pragma unroll
      for (int r = 0; r < JPT; ++r) {
        const int j = ls + r * SEG;
        if (j >= M) continue;
        // conditioned log-weight of inner particle jj given this candidate
        float cpx[Mdl::NPX];
        Mdl::px_pre(as_prm(a.prm), xl[r], x, t - 1, cpx);
        auto kappa = [&](int jj) {
          float zj[DZ], lx;
#pragma unroll
          for (int d = 0; d < DZ; ++d) zj[d] = cz[s][kCond ? jj : 0][d];
          if constexpr (kAux) lx = Mdl::logpx_post_aux(as_prm(a.prm), cpx, zj, caux[s][kAux ? jj : 0]);
          else lx = Mdl::logpx_post(as_prm(a.prm), cpx, zj);
          float kp = lms[s][kCond ? jj : 0] + lx;
          asm volatile("" : "+v"(kp));
          return kp;
        };
        // this lane's columns; they hold the log-weights first (odd items' in
        // the low words of cum2)
        double* const cum = &cum2[0][kCum ? threadIdx.x : 0];
        float* const we = &wev[0][kCum ? threadIdx.x : 0];
        constexpr int CST = kCum ? kBlock : 1;  // entries from one pair to the next
        auto keep = [&](int jj, float kp) {
          if (jj & 1) cum[(jj >> 1) * CST] = __hiloint2double(0, __float_as_int(kp));
          else we[(jj >> 1) * CST] = kp;
        };
        auto kept = [&](int jj) -> float {
          return (jj & 1) ? __int_as_float(__double2loint(cum[(jj >> 1) * CST])) : we[(jj >> 1) * CST];
        };
        // (items by fours, so that their LDS reads and exponentials overlap;
        // those beyond M weigh nothing)
        constexpr int U = CAP % 4 == 0 ? 4 : 1;
        float mx = -INFINITY;
        for (int j4 = 0; j4 < M; j4 += U) {
          float kp[U];
#pragma unroll
          for (int v = 0; v < U; ++v) kp[v] = kappa(j4 + v);
#pragma unroll
          for (int v = 0; v < U; ++v) {
            if constexpr (kCum) keep(j4 + v, kp[v]);
            mx = fmaxf(mx, finitef(kp[v]) ? kp[v] : -INFINITY);
          }
        }
        const bool deg = !(mx > -INFINITY);
        auto weight = [&](int jj) -> float {
          const float kp = kCum ? kept(jj) : kappa(jj);
          const float w = finitef(kp) ? fast_exp(kp - mx) : 0.0f;
          return deg ? (jj < M ? 1.0f : 0.0f) : w;
        };
        double total = 0.0;
        int lastpos = 0;
        for (int j4 = 0; j4 < M; j4 += U) {
          float w[U];
#pragma unroll
          for (int v = 0; v < U; ++v) w[v] = weight(j4 + v);
#pragma unroll
          for (int v = 0; v < U; ++v) {
            total += (double)w[v];
            if constexpr (kCum) {
              if (v & 1) cum[(j4 / 2 + v / 2) * CST] = total;
              else we[(j4 / 2 + v / 2) * CST] = w[v];
            }
            lastpos = w[v] > 0.0f ? j4 + v : lastpos;
          }
        }
        const SysPoints pts(uniform53_ab(key, (uint32_t)t, (uint32_t)i, (uint32_t)j, P_LA_B), total, K);
        float pre[Mdl::NPRE], r0[DY];
        Mdl::fz_pre(as_prm(a.prm), x, xl[r], t - 1, pre);
        Mdl::obs_pre(as_prm(a.prm), y, xl[r], r0);
        Lse acck;
        float hk = 0.f;
        auto emit = [&](int b, const float* nu) {
          float zg[DZ], zc[DZ];
#pragma unroll
          for (int d = 0; d < DZ; ++d) zg[d] = cz[s][kCond ? b : 0][d];
          if constexpr (kAux) Mdl::fz_post_aux(as_prm(a.prm), pre, zg, caux[s][kAux ? b : 0], nu, zc);
          else Mdl::fz_post(as_prm(a.prm), pre, zg, nu, zc);
          acck.add(Mdl::logpy_post(as_prm(a.prm), r0, zc));
          if constexpr (kH) {
            if (want_h) {
              float h[1];
              Mdl::obs_mean(as_prm(a.prm), xl[r], zc, h);
              hk += h[0];
            }
          }
        };
        // (larger clouds) a cursor over the cumulative sum: the points increase
        int jc = -1;
        double c = 0.0;
        for (int k0 = 0; k0 < K; k0 += CPB) {
          float nb[CPB * DZ];
          normals_kb<DZ>(key, (uint32_t)t, (uint32_t)i, (uint32_t)j, P_LA_Z, k0, nb);
          int bk[CPB];
          if constexpr (kCum) {
            // CPB searches of the pairs at once (+inf beyond M), then the pair's
            // first item
            constexpr int NQ = CAP / 2;
            constexpr int S0 = [] {
              int st = 1;
              while (2 * st < NQ) st *= 2;
              return st;
            }();
            double P[CPB];
            const double* at[CPB];
#pragma unroll
            for (int q = 0; q < CPB; ++q) {
              P[q] = k0 + q < K ? pts(k0 + q) : 0.0;
              at[q] = cum[(S0 - 1) * CST] <= P[q] ? cum + (NQ - S0) * CST : cum;
            }
#pragma unroll
            for (int st = S0 / 2; st >= 1; st /= 2) {
#pragma unroll
              for (int q = 0; q < CPB; ++q) at[q] = at[q][(st - 1) * CST] <= P[q] ? at[q] + st * CST : at[q];
            }
#pragma unroll
            for (int q = 0; q < CPB; ++q) {
              const int pr = (int)(at[q] - cum) / CST;
              const double before = pr > 0 ? cum[(pr - 1) * CST] : 0.0;
              const int b = 2 * pr + (before + (double)we[pr * CST] <= P[q] ? 1 : 0);
              bk[q] = P[q] < total ? min(b, M - 1) : lastpos;
            }
          }
#pragma unroll
          for (int q = 0; q < CPB; ++q) {
            const int k = k0 + q;
            if (k >= K) break;
            if constexpr (!kCum) {
              const double P = pts(k);
              while (!(c > P) && jc + 1 < M) {
                ++jc;
                c += (double)weight(jc);
              }
              bk[q] = c > P ? jc : lastpos;
            }
            emit(bk[q], nb + q * DZ);
          }
        }
        const float g = (acck.m == -INFINITY) ? -INFINITY : less_log_k(acck.m + fast_log(acck.s));
        ev[r] = la_ell(lamv[r], g);
        if (want_h) hv.add(r, fast_exp(lamv[r]), hk * invK);
      }
    }
  }
  SegLse<SEG, JPT, ORD> acc;
#pragma unroll
  for (int r = 0; r < JPT; ++r) {
    const int j = ls + r * SEG;
    if (vi && j < M) {
      erow[j] = ev[r];
      acc.add(r, ev[r]);
    }
  }
  const float lw = acc.get(sh);
  if (vi && ls == 0) a.logw[oo + i] = lw;
  if (want_h) {
    const float hs = hv.get(sh);
    if (vi && ls == 0) a.yp[oo + i] = hs;
  }
}

template <class Mdl, int SEG, int JPT, int ORD = 0>
__global__ __launch_bounds__(kBlock) void k_la_weights_nested(StepArgs a) {
  la_weights_nested_tile<Mdl, SEG, JPT, ORD>(a, blockIdx.x);
}

static __device__ bool learned_rejected(const StepArgs& a, int f, int N, float* fred4, double* red4);
static __device__ bool learned_rejected_wave(const StepArgs& a, int f, int N);

// One workgroup per tile.  (A kernel that loops over tiles compiles to
// markedly slower code for the single-tile case, so the learned step's
// fallback has kernels of its own.)
template <class Mdl, int SEG, int JPT, int ORD = 0>
static __global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(min_waves<Mdl>()))) void k_la_weights(StepArgs a) {
  la_weights_tile<Mdl, SEG, JPT, ORD>(a, blockIdx.x, false);
}

// Learned step's fallback, a smaller grid looping over the tiles: each
// workgroup loads its tiles' filters at once, decides per filter whether the
// learned proposals are rejected (the workgroup holding a filter's first
// tile records the decision and the fallback flag), and runs the look-ahead
// weights only for the tiles of rejecting filters.
template <class Mdl, int SEG, int JPT>
static __global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(min_waves<Mdl>()))) void k_la_weights_fallback(StepArgs a) {
  __shared__ int tfl[kBlock], runs[kBlock], todo[kBlock], wcnt[kBlock / kWave];
  __shared__ unsigned char rejr[kBlock];
  __shared__ float fred4[kBlock / kWave];
  __shared__ double red4[kBlock / kWave];
  const int th = threadIdx.x;
  for (int base = blockIdx.x; base < a.n_tiles; base += kBlock * gridDim.x) {
    const int mine = base + th * gridDim.x;
    const bool have = mine < a.n_tiles;
    const int4 tl = have ? a.tiles[mine] : make_int4(-1, 0, 0, 0);
    tfl[th] = tl.x;
    __syncthreads();
    // runs of equal filters (tiles are ordered by filter within a class)
    const bool start = have && (th == 0 || tfl[th - 1] != tl.x);
    int myrun;
    const int nr = block_compact(start, th, runs, wcnt, &myrun);
    // a wave per filter of up to 64 groups, four filters at a time (all of the
    // workgroup one after the other took 8 of this kernel's 12 us where none of
    // 8 filters falls back, now 2)
    for (int r = th / kWave; r < nr; r += kBlock / kWave) {
      const int f = tfl[runs[r]];
      const bool wave = a.finfo[f].ngroup <= kWave;
      const bool rej = wave && step_active(a, f) && learned_rejected_wave(a, f, a.fN[f]);
      if (th % kWave == 0) rejr[r] = wave ? (rej ? 1 : 0) : 2;
    }
    __syncthreads();
    for (int r = 0; r < nr; ++r) {
      if (rejr[r] != 2) continue;
      const int f = tfl[runs[r]];
      const bool rej = step_active(a, f) && learned_rejected(a, f, a.fN[f], fred4, red4);
      __syncthreads();
      if (th == 0) rejr[r] = rej ? 1 : 0;
      __syncthreads();
    }
    const bool rj = have && rejr[myrun - 1] != 0;
    if (have && tl.z == 0) {
      a.fb[tl.x] = rj ? 1 : 0;
      if (rj) {
        atomicOr(&a.flags[tl.x], (uint32_t)F_FALLBACK);
        a.lflags[tl.x] = 0u;
      }
    }
    const int nt = block_compact(rj, mine, todo, wcnt, nullptr);
    for (int q = 0; q < nt; ++q) {
      la_weights_tile<Mdl, SEG, JPT>(a, todo[q], true);
      __syncthreads();
    }
  }
}

// --------------------------------------------------------- plain weights
// Fig. 2 step 1 (eq:approx2 with unit inner weights): ell = log p(y_t | xt, zt),
// log w_i = logsumexp_j ell - log M, and the per-particle partial
// sum_j qbar_ij zt_ij (qbar = softmax_j ell, step 3) for the estimate.
template <class Mdl, int SEG, int JPT, int ORD = 0>
static __global__ __launch_bounds__(kBlock) void k_dpf_weights(StepArgs a) {
  __shared__ SegScratch sh;
  __shared__ float vred[kBlock / kWave][Mdl::DZ];
  const int4 tile = a.tiles[blockIdx.x];
  const int f = tile.x;
  const bool act = step_active(a, f);
  if (tile.z == 0 && threadIdx.x == 0) a.act[f] = act ? 1 : 0;
  if (!act) return;
  const int N = a.fN[f], M = a.fM[f];
  const int i = tile.y + threadIdx.x / SEG;
  const int ls = threadIdx.x % SEG;
  const bool vi = i < N;
  const int oo = a.ooff[f];
  const long long io = a.ioff[f];
  const int t = a.tcur[f] + 1;
  const int src = copy_of(a.cur[f]);

  float y[Mdl::DY], x[Mdl::DX], r0[Mdl::DY];
  load_y<Mdl>(a, f, t, y);
#pragma unroll
  for (int d = 0; d < Mdl::DX; ++d) x[d] = vi ? a.x[src][(long long)d * a.NT + oo + i] : 0.f;
  obs_pre_weights<Mdl>(as_prm(a.prm), y, x, r0);
  const float* zrow = a.z[src] + (io + (long long)(vi ? i : 0) * M) * Mdl::DZ;
  float* erow = a.ell + io + (long long)(vi ? i : 0) * M;
  float ev[JPT];
  SegLse<SEG, JPT, ORD> acc;
#pragma unroll
  for (int r = 0; r < JPT; ++r) {
    const int j = ls + r * SEG;
    ev[r] = -INFINITY;
    if (vi && j < M) {
      float z[Mdl::DZ];
#pragma unroll
      for (int d = 0; d < Mdl::DZ; ++d) z[d] = zrow[d * M + j];
      ev[r] = Mdl::logpy_post(as_prm(a.prm), r0, z);
      erow[j] = ev[r];
      acc.add(r, ev[r]);
    }
  }
  const float lse = acc.get(sh);
  // qbar-weighted cloud mean of the proposals (uniform if degenerate)
  const bool deg = !(lse > -INFINITY);
  float part[Mdl::DZ];
#pragma unroll
  for (int d = 0; d < Mdl::DZ; ++d) part[d] = 0.f;
#pragma unroll
  for (int r = 0; r < JPT; ++r) {
    const int j = ls + r * SEG;
    if (vi && j < M) {
      const float q = deg ? 1.0f / (float)M : (finitef(ev[r]) ? fast_exp(ev[r] - lse) : 0.f);
#pragma unroll
      for (int d = 0; d < Mdl::DZ; ++d) part[d] += q * zrow[d * M + j];
    }
  }
  const float lw = deg ? -INFINITY : lse - fast_log((float)M);
  float* kp = a.kpart + (long long)(oo + i) * Mdl::DZ;
  if constexpr (Mdl::DZ <= 16) {
    int slot;
    const float tot = seg_sum_vec_t<SEG, Mdl::DZ>(part, vred, slot);
    if (vi && slot >= 0) kp[slot] = tot;
  } else {
    seg_sum_vec<SEG, Mdl::DZ>(part, vred);
    if (vi && ls == 0) {
#pragma unroll
      for (int d = 0; d < Mdl::DZ; ++d) kp[d] = part[d];
    }
  }
  if (vi && ls == 0) {
    a.logw[oo + i] = lw;
    if (deg) atomicOr(&a.flags[f], (uint32_t)F_DEGENERATE_INNER);
  }
}

// -------------------------------------------------------- outer resampling
// Systematic resampling of the N outer weights w_i = exp(log w_i - max)
// (Fig. 4 step 3; Fig. 2 step 2), organised around groups of 256 weights.
// Group g carries its own shift m_g = max of its log-weights, the FP64 sum
// s_g of exp(log w_i - m_g) and the sum of squares q_g (one workgroup per
// group, k_res_stats).  A workgroup that needs ancestors combines the
// statistics -- m = max_g m_g, c_g = exp(m_g - m), T_g = c_g s_g, offsets
// B_g = inclusive scan of T -- always with the same code in the same order,
// so every workgroup agrees bit for bit on them; group g's cumulative weights
// are C_i = min(B_g + c_g L_i, B_{g+1}) (L: inclusive FP64 scan of its
// terms), its last one B_{g+1}: monotone, with shared boundaries.  A
// systematic point ((k + u) C_total) / N lies in the first group with
// B_{g+1} > point and takes the first index there with C_i > point (a point
// at or past the total takes the first index reaching the total).  The new
// particles' workgroups resolve their own ancestors this way, so no
// separate selection launch is needed.

// Log-weight source: FP32 log-weights, FP32 exponent of the shifted value.
struct LogSrc {
  const float* lw;
  static constexpr bool kLog = true;
  __device__ float key(int i) const {
    const float v = lw[i];
    return finitef(v) ? v : -INFINITY;
  }
  __device__ double val(int i, float mg) const {
    const float v = lw[i];
    return finitef(v) ? (double)fast_exp(v - mg) : 0.0;
  }
};

// Linear FP64 weights as given (kernel-level primitive).
struct LinSrc {
  const double* w;
  static constexpr bool kLog = false;
  __device__ float key(int) const { return 0.f; }
  __device__ double val(int i, float) const { return w[i]; }
};

__device__ __forceinline__ float block_max_256(float v, float* red4) {
  v = seg_reduce_wave<OpMax, kWave>(v);
  if ((threadIdx.x & (kWave - 1)) == 0) red4[threadIdx.x / kWave] = v;
  __syncthreads();
  const float r = fmaxf(fmaxf(red4[0], red4[1]), fmaxf(red4[2], red4[3]));
  __syncthreads();
  return r;
}

// Scale of group g relative to the global shift, exp(m_g - m) in (0, 1]
// (FP32 exponent widened; every workgroup evaluates it identically).
template <class Src>
__device__ __forceinline__ double group_scale(float mg, float m) {
  if (!Src::kLog) return 1.0;
  return mg > -INFINITY ? (double)fast_exp(mg - m) : 0.0;
}

// Learned step: whether filter f rejects its learned proposals -- no finite
// log-weight, or ESS = (sum w)^2 / sum w^2 below ess_frac * N -- from the
// group statistics of the learned log-weights.  All 256 threads take part;
// every workgroup gets the same answer.
static __device__ bool learned_rejected(const StepArgs& a, int f, int N, float* fred4, double* red4) {
  const int th = threadIdx.x;
  const int G = a.finfo[f].ngroup;
  const double* gs = a.gstat + 4LL * a.finfo[f].rg_base;
  // the three statistics of a group in one memory round (clamped, masked)
  const int thc = min(th, G - 1);
  const double g0 = gs[4 * thc], g1 = gs[4 * thc + 1], g2 = gs[4 * thc + 2];
  const float gm = th < G ? (float)g0 : -INFINITY;
  const float m = block_max_256(gm, fred4);
  if (!(m > -INFINITY)) return true;
  double T = 0.0, Q = 0.0;
  if (th < G) {
    const double c = group_scale<LogSrc>(gm, m);
    T = c * g1;
    Q = (c * c) * g2;
  }
  const double total = block_sum_256(T, red4);
  const double sumsq = block_sum_256(Q, red4);
  return total * total < a.ess_frac * (double)N * sumsq;
}

// The same by one wave (the same sums: beyond 64 groups the others' are 0).
static __device__ bool learned_rejected_wave(const StepArgs& a, int f, int N) {
  const int l = threadIdx.x & (kWave - 1);
  const int G = a.finfo[f].ngroup;
  const double* gs = a.gstat + 4LL * a.finfo[f].rg_base;
  const int lc = min(l, G - 1);
  const double g0 = gs[4 * lc], g1 = gs[4 * lc + 1], g2 = gs[4 * lc + 2];
  const float gm = l < G ? (float)g0 : -INFINITY;
  const float m = seg_reduce_wave<OpMax, kWave>(gm);
  if (!(m > -INFINITY)) return true;
  const double c = l < G ? group_scale<LogSrc>(gm, m) : 0.0;
  const double total = seg_reduce_wave<OpAdd, kWave>(l < G ? c * g1 : 0.0);
  const double sumsq = seg_reduce_wave<OpAdd, kWave>(l < G ? (c * c) * g2 : 0.0);
  return total * total < a.ess_frac * (double)N * sumsq;
}

struct ResScratch {
  double B[kBlock + 1];   // group offsets (at most 256 groups)
  double C[kResGroup];    // cumulative weights of the group being resolved
  double P[kBlock];       // points of this workgroup
  int gsel[kBlock];       // their groups
  int run0[kBlock];       // first point of each run of points sharing a group
  int wcnt[kBlock / kWave];
  double red4[kBlock / kWave];
  float fred4[kBlock / kWave];
};

// Statistics (m_g, s_g, q_g) of group g.
template <class Src>
__device__ void res_group_stat(const Src& src, int n, int g, float& mg, double& sg, double& qg,
                               ResScratch& sh) {
  const int i = g * kResGroup + threadIdx.x;
  const float key = i < n ? src.key(i) : -INFINITY;
  mg = Src::kLog ? block_max_256(key, sh.fred4) : 0.f;
  const double v = (i < n && (!Src::kLog || mg > -INFINITY)) ? src.val(i, mg) : 0.0;
  sg = block_sum_256(v, sh.red4);
  qg = block_sum_256(v * v, sh.red4);
}

// The same from this thread's log-weight lw already loaded (valid: i < n),
// with the same arithmetic as for LogSrc.
__device__ __forceinline__ void res_group_stat_lw(float lw, bool valid, float& mg, double& sg, double& qg,
                                                  ResScratch& sh) {
  const float key = valid && finitef(lw) ? lw : -INFINITY;
  mg = block_max_256(key, sh.fred4);
  const double v = (valid && mg > -INFINITY) ? (finitef(lw) ? (double)fast_exp(lw - mg) : 0.0) : 0.0;
  sg = block_sum_256(v, sh.red4);
  qg = block_sum_256(v * v, sh.red4);
}

struct ResResult {
  float m;       // max log-weight (0 for linear weights or when degenerate)
  double total;  // sum of the weights exp(log w - m)
  double sumsq;  // sum of their squares
  bool deg;      // no finite log-weight: uniform weights were used
  bool nonf;     // some log-weight is neither finite nor -inf (self_cdf; elsewhere the statistics' check)
};

// Ancestors res[j] of the points k0 + j, j < np (np <= 256), from the G group
// statistics gstat [G][4] (m_g, s_g, q_g, -).  want_sumsq: also return the
// sum of squared weights (for the effective sample size).
template <class Src>
__device__ ResResult resolve_points(const Src& src, int n, int n_out, double u, int k0, int np,
                                    const double* gstat, int G, int* res, ResScratch& sh, bool want_sumsq) {
  const int th = threadIdx.x;
  const float gm_t = th < G ? (float)gstat[4 * th] : -INFINITY;
  const float m = Src::kLog ? block_max_256(gm_t, sh.fred4) : 0.f;
  const bool deg = Src::kLog && !(m > -INFINITY);
  double T = 0.0, Q = 0.0;
  if (th < G) {
    if (deg) {
      T = Q = (double)min(kResGroup, n - th * kResGroup);
    } else {
      const double c = group_scale<Src>(gm_t, m);
      T = c * gstat[4 * th + 1];
      Q = (c * c) * gstat[4 * th + 2];
    }
  }
  sh.B[th + 1] = block_scan_incl_256(T, sh.red4);  // its barriers order the writes below
  if (th == 0) sh.B[0] = 0.0;
  const double sumsq = want_sumsq ? block_sum_256(Q, sh.red4) : 0.0;
  __syncthreads();
  const double total = sh.B[G];
  if (th < np) {
    const double P = sys_point(k0 + th, u, total, n_out);
    int lo = 0, hi = G;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (sh.B[mid + 1] > P)
        hi = mid;
      else
        lo = mid + 1;
    }
    if (lo == G) {
      lo = 0;
      hi = G - 1;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (sh.B[mid + 1] >= total)
          hi = mid;
        else
          lo = mid + 1;
      }
    }
    sh.P[th] = P;
    sh.gsel[th] = lo;
  }
  __syncthreads();
  // points are non-decreasing, so their groups are too: list the runs of
  // points per group and visit each distinct group once (few points: a
  // scan by every thread; many: ranks of the run starts by compaction)
  int nruns;
  if (np <= 16) {
    nruns = 0;
    for (int j = 0; j < np; ++j)
      if (j == 0 || sh.gsel[j] != sh.gsel[j - 1]) {
        if (th == 0) sh.run0[nruns] = j;
        ++nruns;
      }
    __syncthreads();
  } else {
    const bool start = th < np && (th == 0 || sh.gsel[th - 1] != sh.gsel[th]);
    nruns = block_compact(start, th, sh.run0, sh.wcnt, nullptr);
  }
  for (int r = 0; r < nruns; ++r) {
    const int j0 = sh.run0[r];
    const int j1 = r + 1 < nruns ? sh.run0[r + 1] : np;
    const int g = sh.gsel[j0];
    const int base = g * kResGroup;
    const int nloc = min(kResGroup, n - base);
    const float mg = Src::kLog ? (float)gstat[4 * g] : 0.f;
    const double cg = deg ? 1.0 : group_scale<Src>(mg, m);
    double v = 0.0;
    if (th < nloc) v = deg ? 1.0 : ((!Src::kLog || mg > -INFINITY) ? src.val(base + th, mg) : 0.0);
    const double L = block_scan_incl_256(v, sh.red4);
    const double Bg = sh.B[g], Bg1 = sh.B[g + 1];
    if (th < nloc) sh.C[th] = (th == nloc - 1) ? Bg1 : fmin(Bg + cg * L, Bg1);
    __syncthreads();
    if (th >= j0 && th < j1) res[th] = base + cdf_search(sh.C, nloc, sh.P[th]);
    __syncthreads();
  }
  ResResult r;
  r.m = deg ? 0.f : m;
  r.total = total;
  r.sumsq = sumsq;
  r.deg = deg;
  r.nonf = false;
  return r;
}

// ------------------------------------------------ wave-level draws (wave 0)
// When a workgroup serves one outer particle, its ancestor and candidate are
// single draws: one wave does them with wave-wide DPP scans (no LDS rounds,
// no barriers) while the other waves get on with independent work.

// Inclusive FP64 scan over the 64 lanes; excl receives the exclusive value.
__device__ __forceinline__ double wave_scan_d(double v, double& excl) {
  const double incl = seg_scan_wave<kWave>(v);
  const double up = __shfl_up(incl, 1);
  excl = (threadIdx.x & (kWave - 1)) == 0 ? 0.0 : up;
  return incl;
}

__device__ __forceinline__ int first_lane(unsigned long long mask) { return __ffsll((long long)mask) - 1; }

// The ancestor of point k0 (one systematic point) from the group statistics
// (lane l holds group l's (m, s, q) in gs), by one wave; G <= 64.  Same rule
// and group offsets B as resolve_points (whose wave 0 computes B with the
// same scan); the group's cumulative weights are summed four per lane then
// scanned across lanes.
template <class Src>
__device__ int resolve_point_w0(const Src& src, int n, int n_out, double u, int k0, const double* gs, int G,
                                bool want_sumsq, ResResult& rr) {
  const int l = threadIdx.x & (kWave - 1);
  const float gm = l < G ? (float)gs[0] : -INFINITY;
  const float m = Src::kLog ? seg_reduce_wave<OpMax, kWave>(gm) : 0.f;
  const bool deg = Src::kLog && !(m > -INFINITY);
  double T = 0.0, Q = 0.0;
  if (l < G) {
    if (deg) {
      T = Q = (double)min(kResGroup, n - l * kResGroup);
    } else {
      const double c = group_scale<Src>(gm, m);
      T = c * gs[1];
      Q = (c * c) * gs[2];
    }
  }
  const double Binc = seg_scan_wave<kWave>(T);  // B[l + 1]
  const double total = readlane_d(Binc, G - 1);
  rr.m = deg ? 0.f : m;
  rr.total = total;
  rr.sumsq = want_sumsq ? seg_reduce_wave<OpAdd, kWave>(Q) : 0.0;
  rr.deg = deg;
  rr.nonf = false;
  const double P = sys_point(k0, u, total, n_out);
  unsigned long long bm = __ballot(l < G && Binc > P);
  if (!bm) bm = __ballot(l < G && Binc >= total);
  const int g = first_lane(bm);
  const int base = g * kResGroup;
  const int nloc = min(kResGroup, n - base);
  const float mg = Src::kLog ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(gm), g)) : 0.f;
  const double cg = deg ? 1.0 : group_scale<Src>(mg, m);
  const double Bg = g > 0 ? readlane_d(Binc, g - 1) : 0.0;
  const double Bg1 = readlane_d(Binc, g);
  // the four weights are read at clamped indices first (loads in flight
  // together; a guarded load would wait inside its own branch), then masked
  double L[4], vv[4], acc = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = 4 * l + q;
    vv[q] = src.val(base + (i < nloc ? i : 0), mg);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = 4 * l + q;
    const double v = i < nloc ? (deg ? 1.0 : ((!Src::kLog || mg > -INFINITY) ? vv[q] : 0.0)) : 0.0;
    acc += v;
    L[q] = acc;
  }
  double ex;
  wave_scan_d(acc, ex);
  double C[4];
  int hit = 4, hit_eq = 4;
#pragma unroll
  for (int q = 3; q >= 0; --q) {
    const int i = 4 * l + q;
    C[q] = (i == nloc - 1) ? Bg1 : fmin(Bg + cg * (ex + L[q]), Bg1);
    if (i < nloc && C[q] > P) hit = q;
    if (i < nloc && C[q] >= Bg1) hit_eq = q;
  }
  bm = __ballot(hit < 4);
  int idx;
  if (bm) {
    const int fl = first_lane(bm);
    idx = 4 * fl + __builtin_amdgcn_readlane(hit, fl);
  } else {
    const int fl = first_lane(__ballot(hit_eq < 4));
    idx = 4 * fl + __builtin_amdgcn_readlane(hit_eq, fl);
  }
  return base + idx;
}

// A filter of one resampling group (N <= 256): every wave that needs its
// ancestors forms the whole cumulative sum itself from the log-weights, four
// consecutive weights per lane -- no statistics launch, no barrier.  C: this
// lane's cumulative weights.
__device__ __forceinline__ ResResult self_cdf(const float* lw, int N, bool want_sumsq, double (&C)[4]) {
  const int l = threadIdx.x & (kWave - 1);
  float v[4];
  float key = -INFINITY;
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = lw[min(4 * l + q, N - 1)];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (4 * l + q < N && finitef(v[q])) key = fmaxf(key, v[q]);
  ResResult rr;
  const float m = seg_reduce_wave<OpMax, kWave>(key);
  rr.deg = !(m > -INFINITY);
  rr.m = rr.deg ? 0.f : m;
  double acc = 0.0, sq = 0.0, L[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double w = 4 * l + q < N ? (rr.deg ? 1.0 : (finitef(v[q]) ? (double)fast_exp(v[q] - m) : 0.0)) : 0.0;
    acc += w;
    sq += w * w;
    L[q] = acc;
  }
  double ex;
  const double incl = wave_scan_d(acc, ex);
  rr.total = readlane_d(incl, kWave - 1);
  rr.sumsq = 0.0;
  rr.nonf = false;
  if (want_sumsq) {
    bool nf = false;
#pragma unroll
    for (int q = 0; q < 4; ++q) nf |= !finitef(v[q]) && !(v[q] == -INFINITY);  // (clamped reads repeat the last)
    rr.sumsq = seg_reduce_wave<OpAdd, kWave>(sq);
    rr.nonf = __ballot(nf) != 0;
  }
  // (monotone, the last one the total)
#pragma unroll
  for (int q = 0; q < 4; ++q) C[q] = 4 * l + q >= N - 1 ? rr.total : fmin(ex + L[q], rr.total);
  return rr;
}

// The first index whose cumulative weight exceeds P (else reaches the total);
// P the same in every lane.
__device__ __forceinline__ int self_point(const double (&C)[4], int N, double total, double P) {
  const int l = threadIdx.x & (kWave - 1);
  int hit = 4, hit_eq = 4;
#pragma unroll
  for (int q = 3; q >= 0; --q) {
    if (4 * l + q < N && C[q] > P) hit = q;
    if (4 * l + q < N && C[q] >= total) hit_eq = q;
  }
  const unsigned long long bm = __ballot(hit < 4);
  const int h = bm ? hit : hit_eq;
  const int fl = first_lane(bm ? bm : __ballot(hit_eq < 4));
  return 4 * fl + __builtin_amdgcn_readlane(h, fl);
}

// The three offsets a new outer particle k's draws start from, U53 at (t, 0, 0)
// of OUTER_U and at (t, k, 0) of `cand` and INNER_U, in every lane of its
// segment: one Philox evaluation (lanes 0, 1, 2 of every quad take one each)
// instead of three, all before the first of them is needed.  Two waves per
// particle or more: each wave its own.
struct OuterDraws {
  double outer, cand, inner;
};
__device__ __forceinline__ OuterDraws outer_draws(Key key, int t, int k, uint32_t cand) {
  const int q = threadIdx.x & 3;
  const Words w = draw(key, (uint32_t)t, q == 0 ? 0u : (uint32_t)k, 0u,
                       q == 0 ? (uint32_t)P_OUTER_U : (q == 1 ? cand : (uint32_t)P_INNER_U), 0u);
  const double u = u53(w.w[0], w.w[1]);
  return OuterDraws{dpp_d<0x00>(u, u), dpp_d<0x55>(u, u), dpp_d<0xAA>(u, u)};
}

// One systematic draw (offset u) over weights exp(e_j - max), j < M (non-
// finite: 0; none finite: uniform), by one wave: each lane sums a chunk of
// CMAX (chunks of more than 16: ceil(M / 64)) consecutive weights, the chunk totals are scanned
// across lanes, and the lane holding the point walks its chunk.  Chunks of
// up to 16 stay in registers; longer ones are read again.
template <int CMAX>
__device__ int select_w0(const float* e, int M, double u, bool& deg_out) {
  constexpr bool kReg = CMAX <= 16;
  constexpr int R = kReg ? CMAX : 1;
  const int l = threadIdx.x & (kWave - 1);
  const int C = kReg ? CMAX : (M + kWave - 1) / kWave;
  const int j0 = l * C;
  const int nv = max(0, min(C, M - j0));  // entries of this lane's chunk
  float ev[R];
  float mloc = -INFINITY;
  if constexpr (kReg) {
    const Items<R> it = load_items<R>(e, j0, M);
#pragma unroll
    for (int q = 0; q < R; ++q) {
      ev[q] = q < nv ? it.v[q] : -INFINITY;
      if (finitef(ev[q])) mloc = fmaxf(mloc, ev[q]);
    }
  } else {
    for (int q = 0; q < nv; ++q) {
      const float v = e[j0 + q];
      if (finitef(v)) mloc = fmaxf(mloc, v);
    }
  }
  const float m = seg_reduce_wave<OpMax, kWave>(mloc);
  const bool deg = !(m > -INFINITY);
  deg_out = deg;
  auto wt = [&](float v) { return deg ? 1.0 : (finitef(v) ? (double)fast_exp(v - m) : 0.0); };
  double acc = 0.0;
  double wv[R];
  if constexpr (kReg) {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      wv[q] = q < nv ? wt(ev[q]) : 0.0;
      acc += wv[q];
    }
  } else {
    for (int q = 0; q < nv; ++q) acc += wt(e[j0 + q]);
  }
  double ex;
  const double incl = wave_scan_d(acc, ex);
  const double total = readlane_d(incl, (M - 1) / C);  // the last lane with entries
  const double P = sys_point(0, u, total, 1);
  // the first lane with entries whose cumulative weight passes the point
  // (else reaches the total); its last entry's cumulative weight is its
  // scanned value, so the walk below always ends inside the chunk
  unsigned long long bm = __ballot(nv > 0 && incl > P);
  const bool clamp = bm == 0;
  if (clamp) bm = __ballot(nv > 0 && incl >= total);
  const int fl = first_lane(bm);
  double cum = ex;
  int hit = -1;
  if constexpr (kReg) {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      cum += wv[q];
      const double cq = q == nv - 1 ? incl : fmin(cum, incl);
      if (q < nv && hit < 0 && (clamp ? cq >= total : cq > P)) hit = j0 + q;
    }
  } else {
    for (int q = 0; q < nv; ++q) {
      cum += wt(e[j0 + q]);
      const double cq = q == nv - 1 ? incl : fmin(cum, incl);
      if (hit < 0 && (clamp ? cq >= total : cq > P)) hit = j0 + q;
    }
  }
  return __builtin_amdgcn_readlane(hit, fl);
}

// Filter-level bookkeeping of the outer resampling (one thread per filter).
static __device__ void res_finish(const StepArgs& a, int f, int t, int N, const ResResult& r) {
  a.fstat[4 * f + 0] = r.deg ? 0.0 : (double)r.m;
  a.fstat[4 * f + 1] = r.total;
  a.fstat[4 * f + 2] = r.sumsq;
  a.fstat[4 * f + 3] = r.deg ? 1.0 : 0.0;
  a.ess[f] = (float)(r.total * r.total / r.sumsq);
  const double dl = r.deg ? -INFINITY : (double)r.m + log(r.total) - log((double)N);
  a.dlogz[f] = dl;
  a.loglik[f] += dl;
  uint32_t fl = r.deg ? (uint32_t)F_DEGENERATE_OUTER : 0u;
  const float* yp = a.Y + (long long)(t - 1) * a.y_tstride + (long long)f * a.dy;
  bool nonf = r.nonf;
#pragma unroll 8
  for (int q = 0; q < a.dy; ++q) nonf |= !finitef(yp[q]);
  if (nonf) fl |= F_NONFINITE;
  if (fl) atomicOr(&a.flags[f], fl);
}

// Group statistics; with advance_time, group 0's workgroup also advances the
// filter's time and flips its state copy (no other workgroup of this launch
// reads them); such a step's weights lie in the first pair.  In the learned step's second pass (fb set) a filter that
// kept its learned proposals keeps the statistics of the first pass.
static __global__ __launch_bounds__(kBlock) void k_res_stats(StepArgs a, const int2* rgroups, int advance_time) {
  __shared__ ResScratch sh;
  const int2 rg = rgroups[blockIdx.x];
  const int4 gi = a.ginfo[blockIdx.x];  // static: the filter's offsets and groups
  const int f = rg.x;
  const int oo = gi.x, N = gi.y, rb = gi.z;
  const int i = rg.y * kResGroup + threadIdx.x;
  // the group's log-weight (clamped index, masked below) and the filter's
  // values in one memory round (a load under a branch would wait inside it)
  const float lw = a.logw[oo + min(i, N - 1)];
  const int ac = a.act[f];
  const int fbv = a.fb != nullptr ? a.fb[f] : 1;
  const int tc = a.tcur[f], cu = a.cur[f];
  asm volatile("" ::"v"(ac), "v"(fbv), "v"(tc), "v"(cu));
  if (!(ac & 1)) return;
  if (fbv == 0) {
    if (advance_time && rg.y == 0 && threadIdx.x == 0) {
      a.tcur[f] = tc + 1;
      a.cur[f] = (unsigned char)((cu ^ 1) & ~kCurPair);
    }
    return;
  }
  float mg;
  double sg, qg;
  res_group_stat_lw(lw, i < N, mg, sg, qg, sh);
  const float v = i < N ? lw : 0.f;
  const int nonf = __syncthreads_or((!finitef(v) && !(v == -INFINITY)) ? 1 : 0);
  if (threadIdx.x == 0) {
    double* gs = a.gstat + 4LL * (rb + rg.y);
    gs[0] = (double)mg;
    gs[1] = sg;
    gs[2] = qg;
    if (nonf) atomicOr(&a.flags[f], (uint32_t)F_NONFINITE);
    if (advance_time && rg.y == 0) {
      a.tcur[f] = tc + 1;
      a.cur[f] = (unsigned char)((cu ^ 1) & ~kCurPair);
    }
  }
}

// Outer ancestors of 256 new particles per workgroup (the grid of k_res_stats,
// after the time advance), by the group-statistics rule of resolve_points;
// group 0 also records the filter's ESS, evidence and flags.  In a learned
// step whose proposals were accepted (fb[f] == 0) the workgroup also
// commits the resampled particles: slot indirection, x, and the per-particle
// moments gathered from the learned pass.
// Learned step with accepted proposals (fb[f] == 0): outer ancestors of 256
// new particles per workgroup b (the grid of k_res_stats) by the
// group-statistics rule of resolve_points, and the commit of the resampled
// particles: the learned pass propagated particle i's cloud into slot i of
// the new copy, so particle k refers to its ancestor's slot; x and the
// per-particle moments are gathered (all loads first).  Group 0 records the
// filter's ESS, evidence and flags.  Filters that fell back are skipped
// (their new-cloud tiles resolve their own ancestors).
template <int DX, int DZ>
__device__ void commit_group(const StepArgs& a, int b) {
  __shared__ ResScratch rsh;
  __shared__ int res[kBlock];
  const int2 rg = a.rgroups[b];
  const int f = rg.x;
  // the filter's values in one memory round (a load under a branch would
  // wait inside it)
  const int ac = a.act[f], fbv = a.fb[f], N = a.fN[f], oo = a.ooff[f], t = a.tcur[f], cu = a.cur[f];
  const int rb = a.finfo[f].rg_base, G = a.finfo[f].ngroup;
  asm volatile("" ::"v"(ac), "v"(fbv), "v"(N), "v"(oo), "v"(t), "v"(cu), "v"(rb), "v"(G));
  if (!ac || fbv) return;
  const int k0 = rg.y * kResGroup;
  const int np = min(kResGroup, N - k0);
  const Key key = make_key(a.seed, (uint32_t)f);
  const double u = uniform53(key, (uint32_t)t, 0u, P_OUTER_U);
  const ResResult rr = resolve_points(LogSrc{a.logw + oo}, N, N, u, k0, np, a.gstat + 4LL * rb, G, res, rsh,
                                      rg.y == 0);
  if (rg.y == 0 && threadIdx.x == 0) res_finish(a, f, t, N, rr);
  const int th = threadIdx.x;
  const int dst = copy_of((unsigned char)cu);
  if (th < np) {
    const long long gk = oo + k0 + th, gp = oo + res[th];
    float xv[DX], kv[DZ], mv[2 * DZ];
#pragma unroll
    for (int d = 0; d < DX; ++d) xv[d] = a.xtmp[(long long)d * a.NT + gp];
#pragma unroll
    for (int d = 0; d < DZ; ++d) kv[d] = a.kpart_tmp[gp * DZ + d];
#pragma unroll
    for (int d = 0; d < 2 * DZ; ++d) mv[d] = a.mom_tmp[gp * 2 * DZ + d];
    a.anc[gk] = res[th];
    a.ind[dst][gk] = res[th];
#pragma unroll
    for (int d = 0; d < DX; ++d) a.x[dst][(long long)d * a.NT + gk] = xv[d];
#pragma unroll
    for (int d = 0; d < DZ; ++d) a.kpart[gk * DZ + d] = kv[d];
    if (a.mom) {
#pragma unroll
      for (int d = 0; d < 2 * DZ; ++d) a.mom[gk * 2 * DZ + d] = mv[d];
    }
    if (k0 == 0 && th == 0) a.cur[f] = (unsigned char)(cu & ~(2 << dst));
  }
  if (rg.y == 0 && th == 0) {
    const uint32_t lf = a.lflags[f];
    if (lf) atomicOr(&a.flags[f], lf);
    a.lflags[f] = 0u;
  }
}

// Estimate q of filter f (x's components, z's, then yhat) of the step that
// ended at time t.
template <int DX, int DZ>
__device__ __forceinline__ void est_store(const StepArgs& a, int f, int t, int q, double e) {
  if (q < DX) {
    a.est_x[f * DX + q] = (float)e;
    if (a.trace_x) a.trace_x[((long long)(t - 1) * a.n_filters + f) * DX + q] = (float)e;
  } else if (q < DX + DZ) {
    a.est_z[f * DZ + q - DX] = (float)e;
    if (a.trace_z) a.trace_z[((long long)(t - 1) * a.n_filters + f) * DZ + q - DX] = (float)e;
  } else {
    a.est_y[f] = (float)e;
    if (a.trace_y) a.trace_y[(long long)(t - 1) * a.n_filters + f] = (float)e;
  }
}

// ---------------------------------------------------------------- estimates
// Estimates of a plain step, xhat = sum_i Wbar_i xt_i and zhat = sum_i Wbar_i
// sum_j qbar z over the proposals weighted at this step (copy xs; their sums
// kp), one workgroup of RB threads per filter: FP64 sums in a fixed order (BS
// threads' strided sums, then DPP and the wave results in order; a smaller
// workgroup takes several of the threads each), so results are reproducible
// and do not depend on the launch.  m, total, deg: of the outer weights.
template <int DX, int DZ>
constexpr int fin_block() { return DX + DZ > 16 ? 256 : 1024; }

template <int DX, int DZ, int RB>
__device__ __forceinline__ void finalize_filter(const StepArgs& a, int f, int N, int oo, int t, const float* xs,
                                                const float* kp, double m, double total, bool deg) {
  constexpr int NV = DX + DZ;
  constexpr int BS = fin_block<DX, DZ>();
  __shared__ double red[NV][BS / kWave];
  for (int v0 = 0; v0 < BS; v0 += RB) {
    double acc[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) acc[q] = 0.0;
    // unrolled so that the loads of several particles are in flight together
    // (same summation order as the plain loop; head workgroups less: their
    // registers are those of the new-cloud kernel)
#pragma unroll RB < BS ? 2 : 4
    for (int i = v0 + threadIdx.x; i < N; i += BS) {
      const float lw = a.logw[oo + i];
      const double w = deg ? 1.0 / N : (finitef(lw) ? (double)fast_exp(lw - (float)m) / total : 0.0);
      for (int d = 0; d < DX; ++d) acc[d] += w * (double)xs[(long long)d * a.NT + oo + i];
      for (int d = 0; d < DZ; ++d) acc[DX + d] += w * (double)kp[(long long)(oo + i) * DZ + d];
    }
    for (int q = 0; q < NV; ++q) {
      const double v = v0 < N ? seg_reduce_wave<OpAdd, kWave>(acc[q]) : 0.0;
      if ((threadIdx.x & (kWave - 1)) == 0) red[q][(v0 + threadIdx.x) / kWave] = v;
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < NV; q += RB) {
    double v = 0.0;
    for (int w = 0; w < BS / kWave; ++w) v += red[q][w];
    est_store<DX, DZ>(a, f, t, q, v);
  }
}

// Of a step on its own, after its new-cloud kernel.
template <int DX, int DZ>
static __global__ __launch_bounds__((fin_block<DX, DZ>())) void k_finalize(StepArgs a) {
  const int f = blockIdx.x;
  if (!a.act[f]) return;
  finalize_filter<DX, DZ, fin_block<DX, DZ>()>(a, f, a.fN[f], a.ooff[f], a.tcur[f], a.x[copy_of(a.cur[f]) ^ 1],
                                               a.kpart, a.fstat[4 * f + 0], a.fstat[4 * f + 1],
                                               a.fstat[4 * f + 3] != 0.0);
}

// Shift and total of resolve_points, in its arithmetic and order.
static __device__ ResResult res_total(int n, const double* gstat, int G) {
  __shared__ double red4[kBlock / kWave], tot;
  __shared__ float fred4[kBlock / kWave];
  const int th = threadIdx.x, thc = min(th, G - 1);
  const double g0 = gstat[4 * thc], g1 = gstat[4 * thc + 1];
  const float gm = th < G ? (float)g0 : -INFINITY;
  ResResult r;
  const float m = block_max_256(gm, fred4);
  r.deg = !(m > -INFINITY);
  r.m = r.deg ? 0.f : m;
  const double T = th >= G ? 0.0 : r.deg ? (double)min(kResGroup, n - th * kResGroup) : group_scale<LogSrc>(gm, m) * g1;
  const double B = block_scan_incl_256(T, red4);
  if (th == G - 1) tot = B;
  __syncthreads();
  r.total = tot;
  r.sumsq = 0.0;
  r.nonf = false;
  return r;
}

// Head workgroup of a plain run's new-cloud launch: filter f's estimates of
// the step being taken (its weights, sums and state copy are the previous
// launch's; this one writes the other buffers).  The weights' total is formed
// as the new-cloud workgroups form it.
template <int DX, int DZ>
__device__ __forceinline__ void est_head_plain(const StepArgs& a, int f) {
  const int act = a.act[f], t = a.tcur[f], N = a.fN[f], oo = a.ooff[f], cu = a.cur[f];
  const FilterInfo fi = a.finfo[f];
  asm volatile("" ::"v"(act), "v"(t), "v"(N), "v"(oo), "v"(cu));
  if (!(act & 1)) return;
  ResResult rr;
  if (fi.ngroup == 1) {
    double C[4];
    rr = self_cdf(a.logw + oo, N, false, C);
  } else {
    rr = res_total(N, a.gstat + 4LL * fi.rg_base, fi.ngroup);
  }
  finalize_filter<DX, DZ, kBlock>(a, f, N, oo, t + 1, a.x[copy_of((unsigned char)cu)], a.kpart_prev,
                                  rr.deg ? 0.0 : (double)rr.m, rr.total, rr.deg);
}

// A plain run of an odd number of steps ends in the other view.
static __global__ __launch_bounds__(kBlock) void k_view_copy(StepArgs a) {
  const int f = blockIdx.x * kBlock + threadIdx.x;
  if (f >= a.n_filters) return;
  a.tcur_n[f] = a.tcur[f];
  a.cur_n[f] = a.cur[f];
  a.act_n[f] = a.act[f];
}

// ------------------------------------------------------- look-ahead step end
// The estimates of a step, xhat = mean_k x_t^(k) and zhat = mean_k sum_j qbar z
// (eq:qbar), and the predicted observation yhat = (1/N) sum_i yp_i: FP64
// partial sums per resampling group (wave sums, then the four waves in order)
// added up in group order -- the same order in every path, so results do not
// depend on how the steps were launched.

// Partial sums of NV values per particle over one group: v[q] this thread's
// (0 beyond the filter's end); thread q < NV returns the group's sum of value
// q (others 0).
template <int NV>
__device__ __forceinline__ double est_partial(const double* v, double (*part)[NV]) {
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const double r = seg_reduce_wave<OpAdd, kWave>(v[q]);
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave][q] = r;
  }
  __syncthreads();
  const int q = threadIdx.x;
  return q < NV ? ((part[0][q] + part[1][q]) + part[2][q]) + part[3][q] : 0.0;
}

// Sum over the filter's groups of partial q (rows of gpart have NV values).
template <int NV>
__device__ __forceinline__ double est_groups(const StepArgs& a, int rb, int G, int q) {
  double e = 0.0;
  // (unrolled: the loads of several groups in flight, added in order)
#pragma unroll 16
  for (int gg = 0; gg < G; ++gg) e += a.gpart[(long long)(rb + gg) * NV + q];
  return e;
}

// Head workgroup of a run's new-cloud launch: while the launch's other
// workgroups take step t + 1, the partial sums of one group's estimates of
// step t (state copy and kpart of the previous launch, which this one does
// not write) and of step t + 1's predicted observation (formed by the
// previous launch).  A filter of one group is finished here, others by
// k_run_stats.  A launch of its own for this took 7 us of a 40 us step, for
// 4096 particles; next to the new clouds it costs nothing measurable.
template <int DX, int DZ, bool YH>
__device__ __forceinline__ void est_head(const StepArgs& a, int b) {
  constexpr int NV = DX + DZ + 1;
  __shared__ double part[kBlock / kWave][NV];
  const int2 rg = a.rgroups[b];
  const int4 gi = a.ginfo[b];
  const int f = rg.x, oo = gi.x, N = gi.y, rb = gi.z, G = gi.w;
  const int act = a.act[f], t = a.tcur[f];
  const unsigned char cb = a.cur[f];
  const bool xz = act & 2, yh = YH && a.yp != nullptr && (act & 1);
  if (!xz && !yh) return;
  const int i = rg.y * kResGroup + threadIdx.x;
  const int ic = min(i, N - 1);
  const double w = 1.0 / N;
  double v[NV];
  const float* xs = a.x[copy_of(cb)];
#pragma unroll
  for (int d = 0; d < DX; ++d) v[d] = (double)xs[(long long)d * a.NT + oo + ic];
#pragma unroll
  for (int d = 0; d < DZ; ++d) v[DX + d] = (double)a.kpart_prev[(long long)(oo + ic) * DZ + d];
  v[NV - 1] = yh ? (double)a.yp[oo + ic] : 0.0;
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = i < N ? w * v[q] : 0.0;
  const double e = est_partial<NV>(v, part);
  const int q = threadIdx.x;
  if (q >= NV) return;
  if (G > 1)
    a.gpart[(long long)(rb + rg.y) * NV + q] = e;
  else if (q < NV - 1 ? xz : yh)
    est_store<DX, DZ>(a, f, q < NV - 1 ? t : t + 1, q, 0.0 + e);
}

// Statistics of the next step's outer log-weights, which the new-cloud kernel
// has already computed (a run), for group g of filter f: gstat and the
// non-finite check.  lw: this thread's weight (any value beyond the end).
__device__ __forceinline__ void next_stats(const StepArgs& a, int f, int row, float lw, bool valid, ResScratch& sh) {
  float mg;
  double sg, qg;
  res_group_stat_lw(lw, valid, mg, sg, qg, sh);
  const float lv = valid ? lw : 0.f;
  const int nonf = __syncthreads_or((!finitef(lv) && !(lv == -INFINITY)) ? 1 : 0);
  if (threadIdx.x == 0) {
    double* gs = a.gstat + 4LL * row;
    gs[0] = (double)mg;
    gs[1] = sg;
    gs[2] = qg;
    if (nonf) atomicOr(&a.flags[f], (uint32_t)F_NONFINITE);
  }
}

// Between two new-cloud launches of a run (handles of up to
// kPostFenceGroups groups, some filter with several): the next step's group
// statistics, and, from the partial sums of the launch's head workgroups, the
// estimates of the step before it and its predicted observation.
// Latency-bound (4 us).
template <int DX, int DZ, bool YH>
static __global__ __launch_bounds__(kBlock) void k_run_stats(StepArgs a, const int2* rgroups) {
  __shared__ ResScratch sh;
  const int2 rg = rgroups[blockIdx.x];
  const int4 gi = a.ginfo[blockIdx.x];
  const int f = rg.x, g = rg.y;
  const int oo = gi.x, N = gi.y, rb = gi.z, G = gi.w;
  const int i = g * kResGroup + threadIdx.x;
  // all loads in one memory round (clamped, masked below)
  const float lwn = a.logw_next[oo + min(i, N - 1)];
  const int act = a.act[f], t = a.tcur[f], act_n = a.act_n[f];
  asm volatile("" ::"v"(lwn), "v"(act), "v"(t), "v"(act_n));
  if (G > 1 && (act_n & 1)) next_stats(a, f, rb + g, lwn, i < N, sh);
  constexpr int NV = DX + DZ + 1;
  const int q = threadIdx.x;
  if (g == 0 && G > 1 && q < NV) {
    const bool on = q < NV - 1 ? (act & 2) : (YH && a.yp != nullptr && (act & 1));
    if (on) est_store<DX, DZ>(a, f, q < NV - 1 ? t : t + 1, q, est_groups<NV>(a, rb, G, q));
  }
}

// End of a look-ahead step taken on its own, of a learned step and of a run
// (and of each step of a run of more than kPostFenceGroups groups; next: also
// the next step's group statistics).  One workgroup per resampling group; a
// filter's last workgroup (found with a counter it resets) adds up the
// partials; with split, k_post_end or k_resolve does.  The view is the one
// after the step; `took` the bit of act that says the filter took it.  When
// tcur_n is given the view is copied there (the handle's own).
template <int DX, int DZ, bool YH>
static __global__ __launch_bounds__(kBlock) void k_post(StepArgs a, const int2* rgroups, int took, int next,
                                                        int split) {
  constexpr int NV = DX + DZ + (YH ? 1 : 0);
  __shared__ ResScratch sh;
  __shared__ double part[kBlock / kWave][NV];
  __shared__ int last;
  const int2 rg = rgroups[blockIdx.x];
  const int4 gi = a.ginfo[blockIdx.x];  // static: the filter's offsets and groups
  const int f = rg.x, g = rg.y;
  const int oo = gi.x, N = gi.y, rb = gi.z, G = gi.w;
  const int i = g * kResGroup + threadIdx.x;
  // loads at a clamped index, masked afterwards (a load guarded by i < N
  // would wait inside its own branch: one memory round per value); the
  // particles' values do not depend on the filter's time, so they are
  // fetched in the same memory round as it (x from both state copies)
  const int ic = min(i, N - 1);
  float raw[NV], xo[DX];
#pragma unroll
  for (int d = 0; d < DX; ++d) {
    raw[d] = a.x[0][(long long)d * a.NT + oo + ic];
    xo[d] = a.x[1][(long long)d * a.NT + oo + ic];
  }
#pragma unroll
  for (int d = 0; d < DZ; ++d) raw[DX + d] = a.kpart[(long long)(oo + ic) * DZ + d];
  if constexpr (YH) raw[NV - 1] = a.yp[oo + ic];
  const float lwn = next ? a.logw_next[oo + ic] : 0.f;
  const int act = a.act[f], t = a.tcur[f], cu = a.cur[f];  // t: the step just taken
  asm volatile("" ::"v"(act), "v"(t), "v"(cu));
  if (a.tcur_n != nullptr && g == 0 && threadIdx.x == 0) {
    a.tcur_n[f] = t;
    a.cur_n[f] = (unsigned char)cu;
    a.act_n[f] = (unsigned char)act;
  }
  if (!(act & took)) return;
  if (copy_of((unsigned char)cu)) {
#pragma unroll
    for (int d = 0; d < DX; ++d) raw[d] = xo[d];
  }
  const double w = 1.0 / N;
  double v[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = i < N ? w * (double)raw[q] : 0.0;
  const double e = est_partial<NV>(v, part);
  if (threadIdx.x < NV) a.gpart[(long long)(rb + g) * NV + threadIdx.x] = e;
  if (next && (act & 1) && G > 1) next_stats(a, f, rb + g, lwn, i < N, sh);
  if (split) return;
  __threadfence();
  if (threadIdx.x == 0) last = atomicAdd(&a.fcount[f], 1) == G - 1;
  __syncthreads();
  if (!last) return;
  __threadfence();
  if (threadIdx.x == 0) a.fcount[f] = 0;
  if (threadIdx.x < NV) est_store<DX, DZ>(a, f, t, threadIdx.x, est_groups<NV>(a, rb, G, threadIdx.x));
}

// With many groups in a launch the cross-workgroup hand-off of k_post (a
// device-scope fence per workgroup writes back the L2 of its XCD) costs more
// than a kernel boundary: k_post runs split (groups only) and this kernel,
// one workgroup per filter, finishes the filters.
template <int DX, int DZ, bool YH>
static __global__ __launch_bounds__(kBlock) void k_post_end(StepArgs a, int took) {
  constexpr int NV = DX + DZ + (YH ? 1 : 0);
  const int f = blockIdx.x;
  const int act = a.act[f], t = a.tcur[f];
  const FilterInfo fi = a.finfo[f];
  if (!(act & took)) return;
  if (threadIdx.x < NV) est_store<DX, DZ>(a, f, t, threadIdx.x, est_groups<NV>(a, fi.rg_base, fi.ngroup, threadIdx.x));
}

// Outer ancestors of every group of 256 new particles of the step about to be
// taken (the view before it), one workgroup per group, for the handles of many
// groups: there each of the new-cloud kernel's workgroups resolving its own
// few particles (a dozen barriers and FP64 scans each) cost more than this
// launch (256 ragged filters of 256 to 4096 particles: 475 us per step, 428 with
// it).  Filters of one group resolve in the new-cloud kernel.
// finish: also the estimates of the step before (the partial sums of k_post).
template <int DX, int DZ, bool YH>
static __global__ __launch_bounds__(kBlock) void k_resolve(StepArgs a, const int2* rgroups, int finish) {
  constexpr int NV = DX + DZ + (YH ? 1 : 0);
  __shared__ ResScratch sh;
  __shared__ int res[kBlock];
  const int2 rg = rgroups[blockIdx.x];
  const int4 gi = a.ginfo[blockIdx.x];
  const int f = rg.x, g = rg.y;
  const int oo = gi.x, N = gi.y, rb = gi.z, G = gi.w;
  const int act = a.act[f], t = a.tcur[f];
  asm volatile("" ::"v"(act), "v"(t));
  if (finish && g == 0 && (act & 2) && threadIdx.x < NV)
    est_store<DX, DZ>(a, f, t, threadIdx.x, est_groups<NV>(a, rb, G, threadIdx.x));
  if (!(act & 1) || G == 1) return;
  const int k0 = g * kResGroup, np = min(kResGroup, N - k0);
  const Key key = make_key(a.seed, (uint32_t)f);
  const double u = uniform53(key, (uint32_t)(t + 1), 0u, P_OUTER_U);
  const ResResult rr = resolve_points(LogSrc{a.logw + oo}, N, N, u, k0, np, a.gstat + 4LL * rb, G, res, sh, g == 0);
  if (g == 0 && threadIdx.x == 0) res_finish(a, f, t + 1, N, rr);
  if (threadIdx.x < np) a.anc[oo + k0 + threadIdx.x] = res[threadIdx.x];
}

// ---------------------------------------------------------------- new cloud
// Look-ahead mode (Fig. 4 step 4): new particle k with parent p = anc[k]
//  * selects candidate c over the parent's ell by one inverse-CDF draw
//    (U53 CAND_U at (t, k, 0)) and regenerates x_t = xla^{(p,c)} from the
//    LA_X normals at (t, p, c) (eq:approx3, sampled by SIR);
//  * conditions the parent's cloud on x_t, kappa_j = lam_pj + log p(x_t |
//    x_p, z_pj) (eq:qnobar), resamples it systematically (INNER_U);
//  * propagates z_t^{(k,j)} = f^z(x_p, x_t, z_{p,b_j}) (NEW_Z at (t, k, j));
//  * applies eq:qbar: lam_t = log p(y_t | x_t, z_t) - logsumexp_j.
// Plain mode (Fig. 2 steps 4-7): a_k ~ Cat(qbar_p) (DPF_ANC_U), a fresh
// x_{t+1} from the a_k-th component (DPF_X at (t, k, 0)), kappa = ell_pj +
// log p(x_{t+1} | x_p, z_pj), systematic inner resampling, DPF_Z normals;
// no measurement update (that happens at the next step).
template <class Mdl, int SEG, int JPT, bool PLAIN, int ORD = 0>
__device__ __forceinline__ void newcloud_tile(const StepArgs& a, int ti) {
  constexpr int DX = Mdl::DX, DZ = Mdl::DZ, DY = Mdl::DY;
  constexpr int NSEG = kBlock / SEG;
  constexpr bool kKeepZ = JPT * DZ <= 64;  // new z stays in registers for the partial sums
  // Wide z: the propagation takes one inner particle at a time (its gathered,
  // noise and new z arrays alone fill most of the registers), passing each
  // one's likelihoods to the later loops through LDS.
  constexpr bool kRoll = DZ >= 32 && JPT > 1;
  constexpr bool kStream = Mdl::kStreamZ;
  __shared__ SegScratch sh;
  __shared__ double cdf[NSEG][SEG * JPT];
  __shared__ float roll_sh[kRoll ? 2 * JPT : 1][kRoll ? kBlock : 1];
  __shared__ float vred[kBlock / kWave][2 * DZ];
  __shared__ int anc_sh[NSEG];
  __shared__ ResScratch rsh;

  const int4 tile = a.tiles[ti];
  const int f = tile.x;
  // group statistics for the wave-level ancestor draw, lane l: group l of
  // the filter (fetched with the filter's values; the array is padded)
  double gst[3] = {0.0, 0.0, 0.0};
  if constexpr (SEG >= kWave) {
    const double* gp = a.gstat + 4LL * (tile.w + (threadIdx.x & (kWave - 1)));
    gst[0] = gp[0];
    gst[1] = gp[1];
    gst[2] = gp[2];
  }
  // the next step's horizon (look-ahead run)
  const int tf_next = (a.ell_next != nullptr && a.run_Tf != nullptr) ? a.run_Tf[f] : 0x7fffffff;
  const FilterView fv = load_filter(a, f);
  // the view holds the filter's progress before the step (act_n given) or after
  const int before = a.act_n != nullptr ? 1 : 0;
  const int t = fv.t + before;  // the step being taken (0 at initialisation)
  const bool act = fv.act & 1;
  const unsigned char cb = (unsigned char)(fv.cur ^ (act ? before : 0));
  const int dst = copy_of(cb), src = dst ^ 1;
  // run: this kernel also computes the next step's weights (Fig. 4 steps 1-2,
  // or Fig. 2 step 1, at t + 1) for the filters that take it; y_{t+1} fetched
  // early.  (The wide-z plain pass keeps its weights kernel.)
  constexpr bool kPlainFuse = PLAIN && !kStream;
  const bool next = (!PLAIN || kPlainFuse) && t < min(tf_next, a.run_T);
  const bool fuse = next && a.ell_next != nullptr;
  if (before && tile.z == 0 && threadIdx.x == 0) {
    // the view after the step (the new clouds are in slot order)
    a.tcur_n[f] = act ? t : fv.t;
    a.cur_n[f] = act ? (unsigned char)((cb & ~kCurPair) | (2 << dst) | (a.pair ? kCurPair : 0)) : (unsigned char)fv.cur;
    a.act_n[f] = act ? (unsigned char)(2 | (next ? 1 : 0)) : (unsigned char)0;
  }
  if (!act) return;
  // learned step with accepted proposals: committed by commit_group
  if (!PLAIN && fv.fb == 0) return;
  float yn[DY];
  if ((!PLAIN || kPlainFuse) && a.ell_next != nullptr) {
    load_y<Mdl>(a, f, min(t, a.run_T - 1) + 1, yn);
  } else if (kPlainFuse) {
#pragma unroll
    for (int d = 0; d < DY; ++d) yn[d] = 0.f;
  }
  const int N = fv.N, M = fv.M;
  const int s = SEG >= kWave ? __builtin_amdgcn_readfirstlane(threadIdx.x / SEG) : threadIdx.x / SEG;
  const int ls = threadIdx.x % SEG;
  const int k = tile.y + s;
  const bool vk = k < N;
  const int oo = fv.oo;
  const long long io = fv.io;
  const Key key = make_key(a.seed, (uint32_t)f);
  const OuterDraws ud = outer_draws(key, t, k, PLAIN ? P_DPF_ANC_U : P_CAND_U);
  // filters of one resampling group form their outer cumulative sum here
  const bool self = a.advance && fv.ngroup == 1;

  // With a wave or more per outer particle, the ancestor and the candidate
  // are single draws done by the segment's first wave with wave-wide scans.
  // The NEW_Z / DPF_Z normals of the inner particles do not depend on them:
  // the segment's other waves draw theirs meanwhile.
  constexpr bool kWaveDraw = SEG >= kWave;
  constexpr bool kEarly = SEG > kWave && JPT * DZ <= 16;
  static_assert(!(kEarly && kStream), "a streamed model draws its noise in the propagation");
  float nue[kEarly ? JPT : 1][DZ];
  // One wave per outer particle: the parent's kappa inputs (lam, or ell in
  // plain mode, and z when p(x'|x, z) depends on z) are fetched together
  // with its ell row for the candidate draw, in the same memory round.
  constexpr bool kPre = SEG == kWave;
  constexpr bool kPreZ = kPre && Mdl::kXdepZ;
  constexpr bool kXZ = Mdl::kXdepZ;
  constexpr int NPX = npx<Mdl>();
  float kpre[kPre ? JPT : 1];
  float zpre[kPreZ ? JPT : 1][kPreZ ? DZ : 1];
#pragma unroll
  for (int r = 0; r < (kPre ? JPT : 1); ++r) {
    kpre[r] = 0.f;
#pragma unroll
    for (int d = 0; d < (kPreZ ? DZ : 1); ++d) zpre[r][d] = 0.f;
  }
  int p, c, pc;
  bool deg1;
  float xp[DX], xn[DX];
  if constexpr (kWaveDraw) {
    // ---- 0-2. ancestor, candidate and new x by the segment's first wave --
    __shared__ int pc_sh[NSEG][2];
    __shared__ float xw_sh[NSEG][DX];
    __shared__ int d1_sh[NSEG];
    const int G = fv.ngroup;
    const bool resolve = a.advance && !a.anc_ready && !self;
    const bool blk = resolve && G > kWave;  // many groups: the whole workgroup resolves
    if (blk) {
      const ResResult rr = resolve_points(LogSrc{a.logw + oo}, N, N, ud.outer, tile.y, min(NSEG, N - tile.y),
                                          a.gstat + 4LL * a.finfo[f].rg_base, G, anc_sh, rsh, tile.z == 0);
      if (tile.z == 0 && threadIdx.x == 0) res_finish(a, f, t, N, rr);
    }
    int pw = 0, cw = 0, pcw = 0;
    bool d1 = false;
    float xpw[DX], xw[DX];
#pragma unroll
    for (int d = 0; d < DX; ++d) xpw[d] = xw[d] = 0.f;
    if (ls < kWave && vk) {
      const bool first = tile.z == 0 && s == 0;
      if (self) {
        double C[4];
        const ResResult rr = self_cdf(a.logw + oo, N, first, C);
        pw = self_point(C, N, rr.total, sys_point(k, ud.outer, rr.total, N));
        if (first && ls == 0) res_finish(a, f, t, N, rr);
      } else if (blk) {
        pw = anc_sh[s];
      } else if (resolve) {
        ResResult rr;
        pw = resolve_point_w0(LogSrc{a.logw + oo}, N, N, ud.outer, k, gst, G, first, rr);
        if (first && ls == 0) res_finish(a, f, t, N, rr);
      } else {
        pw = a.advance ? a.anc[oo + k] : k;  // identity at initialisation
      }
      // the parent's slot and x do not depend on the candidate: fetched first
      pcw = (PLAIN || ident_slots(cb, src)) ? pw : a.ind[src][oo + pw];
#pragma unroll
      for (int d = 0; d < DX; ++d) xpw[d] = a.x[src][(long long)d * a.NT + oo + pw];
      const float* zpw = a.z[src] + (io + (long long)pcw * M) * DZ;
      if constexpr (kPre) {
        const float* kr = PLAIN ? a.ell + io + (long long)pw * M : a.lam[src] + io + (long long)pcw * M;
        const Items<JPT> ki = load_items<JPT>(kr, ls * JPT, M);
#pragma unroll
        for (int r = 0; r < JPT; ++r) kpre[r] = ki.v[r];
        if constexpr (kPreZ) {
#pragma unroll
          for (int d = 0; d < DZ; ++d) {
            const Items<JPT> zi = load_items<JPT>(zpw + d * M, ls * JPT, M);
#pragma unroll
            for (int r = 0; r < JPT; ++r) zpre[kPreZ ? r : 0][kPreZ ? d : 0] = zi.v[r];
          }
        }
      }
      // candidate (look-ahead) / inner ancestor (plain) over the parent's ell
      cw = select_w0<(SEG * JPT + kWave - 1) / kWave>(a.ell + io + (long long)pw * M, M, ud.cand, d1);
      // every lane of the wave computes the new x (same counters)
      float zc[DZ], nu[DX];
      if constexpr (kPreZ) {
        // z of the candidate: held by lane cw / JPT in its slot cw % JPT
        const int rr = cw % JPT;
#pragma unroll
        for (int d = 0; d < DZ; ++d) {
          float v = zpre[0][kPreZ ? d : 0];
#pragma unroll
          for (int r = 1; r < JPT; ++r)
            if (rr == r) v = zpre[kPreZ ? r : 0][kPreZ ? d : 0];
          zc[d] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), cw / JPT));
        }
      } else {
#pragma unroll
        for (int d = 0; d < DZ; ++d) zc[d] = zpw[d * M + cw];
      }
      if (PLAIN)
        normals<DX>(key, (uint32_t)t, (uint32_t)k, 0u, P_DPF_X, nu);
      else
        normals<DX>(key, (uint32_t)t, (uint32_t)pw, (uint32_t)cw, P_LA_X, nu);
      Mdl::fx(as_prm(a.prm), xpw, zc, nu, PLAIN ? t : t - 1, xw);
      if (ls == 0) {
        if (!a.anc_ready || self) a.anc[oo + k] = pw;
        a.sel[oo + k] = cw;
#pragma unroll
        for (int d = 0; d < DX; ++d) a.x[dst][(long long)d * a.NT + oo + k] = xw[d];
      }
    }
    if constexpr (SEG == kWave) {
      p = __builtin_amdgcn_readfirstlane(pw);
      c = cw;
      pc = __builtin_amdgcn_readfirstlane(pcw);
      deg1 = d1;
#pragma unroll
      for (int d = 0; d < DX; ++d) {
        xn[d] = xw[d];
        xp[d] = xpw[d];
      }
    } else {
      if (ls == 0) {
#pragma unroll
        for (int d = 0; d < DX; ++d) xw_sh[s][d] = xw[d];
        pc_sh[s][0] = pw;
        pc_sh[s][1] = cw;
        d1_sh[s] = d1 ? 1 : 0;
      }
      if constexpr (kEarly) {
#pragma unroll
        for (int r = 0; r < JPT; ++r) {
          const int jj = ls + r * SEG;
          if (jj < M) normals<DZ>(key, (uint32_t)t, (uint32_t)k, (uint32_t)jj, PLAIN ? P_DPF_Z : P_NEW_Z, nue[r]);
        }
      }
      __syncthreads();
      p = __builtin_amdgcn_readfirstlane(pc_sh[s][0]);
      c = pc_sh[s][1];
      deg1 = d1_sh[s] != 0;
#pragma unroll
      for (int d = 0; d < DX; ++d) xn[d] = xw_sh[s][d];
      pc = (PLAIN || ident_slots(cb, src)) ? p : a.ind[src][oo + p];
#pragma unroll
      for (int d = 0; d < DX; ++d) xp[d] = a.x[src][(long long)d * a.NT + oo + p];
    }
  } else {
  // ---- 0. outer ancestors of this tile's new particles -------------------
  // (resolved here, also for the learned step's fallback filters)
  p = 0;
  if (self) {
    // each wave its own particles'
    double C[4];
    const bool first = tile.z == 0 && threadIdx.x < kWave;
    const ResResult rr = self_cdf(a.logw + oo, N, first, C);
    constexpr int NSW = kWave / SEG;
    const int s0 = s - s % NSW;
#pragma unroll
    for (int q = 0; q < NSW; ++q) {
      const int kq = tile.y + s0 + q;
      const int pq = kq < N ? self_point(C, N, rr.total, sys_point(kq, ud.outer, rr.total, N)) : 0;
      if (s == s0 + q) p = pq;
    }
    if (first && threadIdx.x == 0) res_finish(a, f, t, N, rr);
  } else {
    if (a.advance && !a.anc_ready) {
      const int np = min(NSEG, N - tile.y);
      const ResResult rr = resolve_points(LogSrc{a.logw + oo}, N, N, ud.outer, tile.y, np, a.gstat + 4LL * tile.w,
                                          fv.ngroup, anc_sh, rsh, tile.z == 0);
      if (tile.z == 0 && threadIdx.x == 0) res_finish(a, f, t, N, rr);
      __syncthreads();
      p = vk ? anc_sh[s] : 0;
    } else if (vk) {
      p = a.advance ? a.anc[oo + k] : k;  // identity at initialisation
    }
  }
  if (vk && ls == 0 && (!a.anc_ready || self)) a.anc[oo + k] = p;
  pc = (PLAIN || ident_slots(cb, src)) ? p : a.ind[src][oo + p];
#pragma unroll
  for (int d = 0; d < DX; ++d) xp[d] = a.x[src][(long long)d * a.NT + oo + p];
  const float* zp0 = a.z[src] + (io + (long long)pc * M) * DZ;
  const float* ep = a.ell + io + (long long)p * M;

  // ---- 1. selection over the parent's ell (candidate / ancestor) --------
  // (lane ls: JPT consecutive items; one scan over the lanes, then each lane
  // counts its cumulative weights up to the point)
  float ev[JPT];
  float mloc = -INFINITY;
  const Items<JPT> ei = load_items<JPT>(ep, ls * JPT, M);
#pragma unroll
  for (int r = 0; r < JPT; ++r) {
    const int j = ls * JPT + r;
    ev[r] = (vk && j < M) ? ei.v[r] : -INFINITY;
    if (finitef(ev[r])) mloc = fmaxf(mloc, ev[r]);
  }
  const float m1 = seg_max<SEG>(mloc, sh);
  deg1 = !(m1 > -INFINITY);
  double acc1 = 0.0;
#pragma unroll
  for (int r = 0; r < JPT; ++r) {
    const int j = ls * JPT + r;
    ev[r] = j < M ? (deg1 ? 1.0f : (finitef(ev[r]) ? fast_exp(ev[r] - m1) : 0.0f)) : 0.0f;
    acc1 += (double)ev[r];
  }
  double ex1, in1;
  seg_scan_wave_both<SEG>(acc1, ex1, in1);
  const double tot1 = seg_last<SEG>(in1);
  const double P1 = ud.cand * tot1;
  // first index whose cumulative weight exceeds the point (a point at the
  // total: the first that reaches it)
  float below = 0.f, short1 = 0.f;
  {
    double cum = ex1;
#pragma unroll
    for (int r = 0; r < JPT; ++r) {
      cum += (double)ev[r];
      const double C = r == JPT - 1 ? in1 : fmin(cum, in1);
      const bool in = ls * JPT + r < M;
      below += in && C <= P1 ? 1.f : 0.f;
      short1 += in && C < tot1 ? 1.f : 0.f;
    }
  }
  c = (int)seg_reduce_wave<OpAdd, SEG>(below);
  if (__ballot(c >= M)) {
    const int c2 = (int)seg_reduce_wave<OpAdd, SEG>(short1);
    c = c >= M ? min(c2, M - 1) : c;
  }
  if (vk && ls == 0) a.sel[oo + k] = c;

  // ---- 2. the new outer particle (every lane of the segment the same) ----
  {
    float zc[DZ], nu[DX], xo[DX];
#pragma unroll
    for (int d = 0; d < DZ; ++d) zc[d] = zp0[d * M + c];
    if (PLAIN)
      normals<DX>(key, (uint32_t)t, (uint32_t)k, 0u, P_DPF_X, nu);
    else
      normals<DX>(key, (uint32_t)t, (uint32_t)p, (uint32_t)c, P_LA_X, nu);
    // (opaque on both sides: products shared with the conditioning below
    // would change what is fused, hence the rounding)
#pragma unroll
    for (int d = 0; d < DX; ++d) {
      xo[d] = xp[d];
      asm volatile("" : "+v"(xo[d]));
    }
    Mdl::fx(as_prm(a.prm), xo, zc, nu, PLAIN ? t : t - 1, xn);
#pragma unroll
    for (int d = 0; d < DX; ++d) asm volatile("" : "+v"(xn[d]));
    if (vk && ls == 0) {
#pragma unroll
      for (int d = 0; d < DX; ++d) a.x[dst][(long long)d * a.NT + oo + k] = xn[d];
    }
  }

  }
  // the new clouds are written in slot order: the slots of copy dst become
  // the identity
  if (!PLAIN && !before && tile.z == 0 && threadIdx.x == 0 && !ident_slots(cb, dst))
    a.cur[f] = (unsigned char)(cb | (2 << dst));
  const float* zp = a.z[src] + (io + (long long)pc * M) * DZ;
  const float* ep = a.ell + io + (long long)p * M;
  (void)c;

  // ---- 3. x-conditioned inner weights and local systematic resampling ---
  // (lane ls: JPT consecutive inner particles)
  const float* lp = a.lam[src] + io + (long long)pc * M;
  float ev[JPT];
  float mk = -INFINITY;
  float cpx[kXZ ? NPX : 1];
  if constexpr (kXZ) Mdl::px_pre(as_prm(a.prm), xn, xp, PLAIN ? t : t - 1, cpx);
  Items<kPre ? 1 : JPT> ki;
  Items<kXZ && !kPre ? JPT : 1> zi[kXZ && !kPre ? DZ : 1];
  if constexpr (!kPre) {
    ki = load_items<JPT>(PLAIN ? ep : lp, ls * JPT, M);
    if constexpr (kXZ) {
#pragma unroll
      for (int d = 0; d < DZ; ++d) zi[d] = load_items<JPT>(zp + d * M, ls * JPT, M);
    }
  }
#pragma unroll
  for (int r = 0; r < JPT; ++r) {
    const int j = ls * JPT + r;
    if (vk && j < M) {
      float kap = kPre ? kpre[kPre ? r : 0] : ki.v[kPre ? 0 : r];
      if constexpr (kXZ) {
        float zj[DZ];
#pragma unroll
        for (int d = 0; d < DZ; ++d)
          zj[d] = kPreZ ? zpre[kPreZ ? r : 0][kPreZ ? d : 0] : zi[kPre ? 0 : d].v[kPre ? 0 : r];
        kap += Mdl::logpx_post(as_prm(a.prm), cpx, zj);
      }
      ev[r] = kap;
      if (finitef(kap)) mk = fmaxf(mk, kap);
    } else {
      ev[r] = -INFINITY;
    }
  }
  const float m2 = seg_max<SEG>(mk, sh);
  const bool deg2 = !(m2 > -INFINITY);
#pragma unroll
  for (int r = 0; r < JPT; ++r)
    ev[r] = ls * JPT + r < M ? (deg2 ? 1.0f : (finitef(ev[r]) ? fast_exp(ev[r] - m2) : 0.0f)) : 0.0f;
  seg_cdf<SEG, JPT>(ev, cdf[s], sh);
  seg_lds_sync<SEG>();
  const double tot2 = cdf[s][M - 1];
  const SysPoints pts(ud.inner, tot2, M);
  // inner ancestors of this lane's new particles ls, ls + SEG, ...
  int anc2[kRoll ? 1 : JPT];
  if constexpr (!kRoll) {
    double P[JPT];
#pragma unroll
    for (int r = 0; r < JPT; ++r) {
      const int jj = ls + r * SEG;
      P[r] = jj < M ? pts(jj) : 0.0;
    }
    cdf_find<SEG * JPT, JPT>(cdf[s], M, tot2, P, anc2);
  }

  // ---- 4. gather + propagate (+ measurement update in look-ahead mode) ---
  // (plain: t is the step just taken and the proposal is for t + 1)
  // Wide z, a wave or more per particle: component q of the shared part stays
  // in lane q and is read from there when its turn comes (64 scalars held at
  // once spilled).
  constexpr bool kPreLane = kStream && SEG >= kWave && DZ <= kWave;
  float pre[kPreLane ? 1 : Mdl::NPRE];
  if constexpr (kPreLane) {
    const int q = threadIdx.x & (kWave - 1);
    pre[0] = Mdl::fz_pre_k(as_prm(a.prm), xp, xn, PLAIN ? t : t - 1, q < DZ ? q : 0);
  } else {
    fz_pre_seg<Mdl, SEG>(as_prm(a.prm), xp, xn, PLAIN ? t : t - 1, pre);
  }
  auto pre_at = [&](int d) -> float {
    if constexpr (kPreLane) return readlane_f(pre[0], d);
    else return pre[kPreLane ? 0 : d];
  };
  float y[DY], r0[DY];
  if (!PLAIN) {
    load_y<Mdl>(a, f, t, y);
    Mdl::obs_pre(as_prm(a.prm), y, xn, r0);
  }
  if constexpr (kPlainFuse) {
    // (opaque: nothing is shared with the propagation, whose bits, and the
    // weights', are those of the kernels on their own)
    float xo[DX];
#pragma unroll
    for (int d = 0; d < DX; ++d) {
      xo[d] = xn[d];
      asm volatile("" : "+v"(xo[d]));
    }
    // (not under `if (fuse)`: products in another block than their sums would
    // stay unfused)
    obs_pre_weights<Mdl>(as_prm(a.prm), yn, xo, r0);
  }
  float* zdst = a.z[dst] + (io + (long long)k * M) * DZ;
  float llv[JPT], gn[JPT];
  float zkeep[kKeepZ ? JPT : 1][DZ];
  // predicted observation of the next step (fused run, when requested)
  constexpr bool kH = !PLAIN && has_yhat<Mdl>();
  const bool want_h = kH && fuse && a.yp_next != nullptr;
  float hn[kH ? JPT : 1];
  SegLse<SEG, JPT, ORD> acc;
  // wide z: the new z of every lane of the wave goes through the matrix-core
  // residual together (lanes without a particle carry zeros)
  float ca[kStream ? Mdl::DZ / 2 : 1];
  __shared__ __align__(16) float y_sh[kStream ? 2 : 1][kStream ? DY : 4];  // y_t, y_{t+1}
  if constexpr (kStream) {
    WaveProj<Mdl>::load_a(as_prm(a.prm), ca);
    if (!PLAIN && threadIdx.x < 2 * DY) {
      const int h = threadIdx.x / DY, q = threadIdx.x % DY;
      y_sh[h][kStream ? q : 0] = y_row<Mdl>(a, f, h ? min(t, a.run_T - 1) + 1 : t)[q];
    }
    __syncthreads();
  }
#pragma unroll kRoll ? 1 : JPT
  for (int r = 0; r < JPT; ++r) {
    const int jj = ls + r * SEG;
    float lv = -INFINITY, gv = 0.f;
    if constexpr (kStream) {
      // Bound by the vector units: at N = 16384, M = 1024, DZ = 64 vector
      // instructions fill some 3 of a step's 3.5 ms (two generators, 132 normals
      // and two mixtures of 32 terms a particle), FP32 matrix products 1 ms,
      // mostly under them.  A run of 4 steps with its export takes 18.5 ms; 22.0
      // when the rows came as single scalars, y and the likelihood's form were
      // looked up term by term and each pair of components was stored under a
      // mask of its own and by 64-bit addresses.
      const bool on = vk && jj < M;
      int b;
      if constexpr (kRoll) {
        const double P[1] = {jj < M ? pts(jj) : 0.0};
        int bb[1];
        cdf_find<SEG * JPT, 1>(cdf[s], M, tot2, P, bb);
        b = bb[0];
      } else {
        b = anc2[kRoll ? 0 : r];
      }
      float zg[DZ], zn[DZ];
      int Mr = __builtin_amdgcn_readfirstlane(M);  // opaque: 2 DZ row bases kept over the items would spill
      asm volatile("" : "+s"(Mr));
#pragma unroll
      for (int d = 0; d < DZ; ++d) zg[d] = on ? at32(zp + d * Mr, b) : 0.f;
      const Prm P = as_prm(a.prm);
      WaveProj<Mdl> pj;
      pj.start();
      const float sz = P[Mdl::Layout::sz];
      auto nxt = Mdl::load_pair(P, 0);  // the rows of the next pair, fetched one ahead
      normal_pairs<0, DZ, false>(key, (uint32_t)t, (uint32_t)k, (uint32_t)jj, PLAIN ? P_DPF_Z : P_NEW_Z, 0.f,
                                 [&](int d, float n0, float n1) {
                                   const auto row = nxt;
                                   if (d + 2 < DZ) nxt = Mdl::load_pair(P, d / 2 + 1);
                                   zn[d] = Mdl::fz_post_row(row, 0, sz, pre_at(d), zg, n0, d);
                                   zn[d + 1] = Mdl::fz_post_row(row, 1, sz, pre_at(d + 1), zg, n1, d + 1);
                                   if (!PLAIN) pj.add(ca[d / 2], zn[d], zn[d + 1]);
                                 });
      if (on) {
#pragma unroll
        for (int d = 0; d < DZ; ++d) put32(zdst + d * Mr, jj, zn[d]);
      }
      if constexpr (kKeepZ) {
#pragma unroll
        for (int d = 0; d < DZ; ++d) zkeep[kKeepZ ? r : 0][d] = zn[d];
      }
      if (!PLAIN) {
        const float l0 = pj.logpy(P, y_sh[0]);
        // the next step's look-ahead likelihood of these new inner particles
        const float g0 = fuse ? la_logpy_wave<Mdl>(a, key, t + 1, k, jj, xn, zn, y_sh[kStream ? 1 : 0], ca) : 0.f;
        if (on) {
          lv = l0;
          gv = g0;
          acc.add(r, lv);
        }
      }
    } else if (vk && jj < M) {
      const int b = anc2[kRoll ? 0 : r];
      float zg[DZ], zn[DZ], nu[DZ];
#pragma unroll
      for (int d = 0; d < DZ; ++d) zg[d] = at32(zp + d * M, b);
      if constexpr (kEarly) {
#pragma unroll
        for (int d = 0; d < DZ; ++d) nu[d] = nue[kEarly ? r : 0][d];
      } else {
        normals<DZ>(key, (uint32_t)t, (uint32_t)k, (uint32_t)jj, PLAIN ? P_DPF_Z : P_NEW_Z, nu);
      }
      Mdl::fz_post(as_prm(a.prm), pre, zg, nu, zn);
#pragma unroll
      for (int d = 0; d < DZ; ++d) put32(zdst + d * M, jj, zn[d]);
      if (!PLAIN) {
        lv = Mdl::logpy_post(as_prm(a.prm), r0, zn);
      } else if (kPlainFuse && fuse) {
        float zo[DZ];
#pragma unroll
        for (int d = 0; d < DZ; ++d) {
          zo[d] = zn[d];
          asm volatile("" : "+v"(zo[d]));
        }
        lv = Mdl::logpy_post(as_prm(a.prm), r0, zo);
        acc.add(r, lv);
      }
      if constexpr (kKeepZ) {
#pragma unroll
        for (int d = 0; d < DZ; ++d) zkeep[kKeepZ ? r : 0][d] = zn[d];
      }
      if (!PLAIN) {
        acc.add(r, lv);
        // the next step's look-ahead likelihood of this new inner particle
        // (ALU work that overlaps the gathers of the others)
        if (want_h) {
          float h[1];
          gv = la_logpy<Mdl, kH>(a, key, t + 1, k, jj, xn, zn, yn, h);
          hn[kH ? r : 0] = h[0];
        } else if (fuse) {
          gv = la_logpy<Mdl>(a, key, t + 1, k, jj, xn, zn, yn);
        }
      }
    }
    if constexpr (kRoll) {
      roll_sh[2 * r][threadIdx.x] = lv;
      roll_sh[2 * r + 1][threadIdx.x] = gv;
    } else {
      llv[r] = lv;
      gn[r] = gv;
    }
  }
  if constexpr (kRoll) {
    // (each thread reads back its own slots)
#pragma unroll
    for (int r = 0; r < JPT; ++r) {
      llv[r] = roll_sh[2 * r][threadIdx.x];
      gn[r] = roll_sh[2 * r + 1][threadIdx.x];
    }
  }
  uint32_t fl = (deg1 || deg2) ? (uint32_t)F_DEGENERATE_INNER : 0u;
  if (!PLAIN) {
    const float lse = acc.get(sh);
    const bool deg3 = !(lse > -INFINITY);
    if (deg3) fl |= F_DEGENERATE_INNER;
    float* ldst = a.lam[dst] + io + (long long)k * M;
    constexpr int NP = has_moments<Mdl>() ? 2 * DZ : DZ;
    const bool want_mom = has_moments<Mdl>() && a.mom != nullptr;
    float part[NP];
    float lamv[JPT];
#pragma unroll
    for (int d = 0; d < NP; ++d) part[d] = 0.f;
#pragma unroll
    for (int r = 0; r < JPT; ++r) {
      const int jj = ls + r * SEG;
      lamv[r] = 0.f;
      if (vk && jj < M) {
        const float lam = deg3 ? -fast_log((float)M) : (finitef(llv[r]) ? llv[r] - lse : -INFINITY);
        lamv[r] = lam;
        ldst[jj] = lam;
        const float q = deg3 ? 1.0f / (float)M : (finitef(llv[r]) ? fast_exp(lam) : 0.f);
#pragma unroll
        for (int d = 0; d < DZ; ++d) {
          const float zv = kKeepZ ? zkeep[kKeepZ ? r : 0][d] : zdst[d * M + jj];
          part[d] += q * zv;
          if constexpr (NP == 2 * DZ) part[DZ + d] += want_mom ? q * zv * zv : 0.f;
        }
      }
    }
    float* kp = a.kpart + (long long)(oo + k) * DZ;
    if constexpr (NP <= 16) {
      // transpose reduction: each owning lane stores its slot
      int slot;
      if (want_mom) {
        const float tot = seg_sum_vec_t<SEG, NP>(part, reinterpret_cast<float(*)[NP]>(&vred[0][0]), slot);
        const float mean = seg_vec_fetch<SEG, NP>(tot, slot >= DZ ? slot - DZ : -1);
        if (vk && slot >= 0) {
          float* mp = a.mom + (long long)(oo + k) * 2 * DZ;
          if (slot < DZ) {
            kp[slot] = tot;
            mp[slot] = tot;
          } else {
            mp[slot] = fmaxf(tot - mean * mean, 0.f);
          }
        }
      } else {
        const float tot = seg_sum_vec_t<SEG, DZ>(part, reinterpret_cast<float(*)[DZ]>(&vred[0][0]), slot);
        if (vk && slot >= 0) kp[slot] = tot;
      }
    } else {
      seg_sum_vec<SEG, DZ>(part, reinterpret_cast<float(*)[DZ]>(&vred[0][0]));
      if (vk && ls == 0) {
#pragma unroll
        for (int d = 0; d < DZ; ++d) kp[d] = part[d];
      }
    }
    // ---- 5. look-ahead run: the next step's weights ell = lam + g, in the
    // weights kernel's lane layout and summation order
    if (fuse) {
      float* en = a.ell_next + io + (long long)(vk ? k : 0) * M;
      SegLse<SEG, JPT, ORD> acc2;
      SegSum<SEG, JPT, ORD> hv;
#pragma unroll
      for (int r = 0; r < JPT; ++r) {
        const int jj = ls + r * SEG;
        if (vk && jj < M) {
          const float e = la_ell(lamv[r], gn[r]);
          en[jj] = e;
          acc2.add(r, e);
          if (want_h) hv.add(r, fast_exp(lamv[r]), hn[kH ? r : 0]);
        }
      }
      const float lw = acc2.get(sh);
      if (vk && ls == 0) a.logw_next[oo + k] = lw;
      if (want_h) {
        const float hs = hv.get(sh);
        if (vk && ls == 0) a.yp_next[oo + k] = hs;
      }
    }
  }
  if constexpr (kPlainFuse) {
    // the next step's weights and weighted sums, as k_dpf_weights forms them
    if (fuse) {
      const float lse = acc.get(sh);
      const bool degw = !(lse > -INFINITY);
      if (degw) fl |= F_DEGENERATE_INNER;
      float* en = a.ell_next + io + (long long)(vk ? k : 0) * M;
      float part[DZ];
#pragma unroll
      for (int d = 0; d < DZ; ++d) part[d] = 0.f;
#pragma unroll
      for (int r = 0; r < JPT; ++r) {
        const int jj = ls + r * SEG;
        if (vk && jj < M) {
          en[jj] = llv[r];
          const float q = degw ? 1.0f / (float)M : (finitef(llv[r]) ? fast_exp(llv[r] - lse) : 0.f);
#pragma unroll
          for (int d = 0; d < DZ; ++d) part[d] += q * (kKeepZ ? zkeep[kKeepZ ? r : 0][d] : zdst[d * M + jj]);
        }
      }
      float* kp = a.kpart + (long long)(oo + k) * DZ;
      int slot;
      const float tot = seg_sum_vec_t<SEG, DZ>(part, reinterpret_cast<float(*)[DZ]>(&vred[0][0]), slot);
      if (vk && slot >= 0) kp[slot] = tot;
      if (vk && ls == 0) a.logw_next[oo + k] = degw ? -INFINITY : lse - fast_log((float)M);
    }
  }
  if (vk && ls == 0 && fl) atomicOr(&a.flags[f], fl);
}

// End of a step on its own where every filter has one group and the launch few
// workgroups: a filter's last workgroup (of its tiles, and in a plain step of
// its head workgroup) forms a look-ahead step's estimates as k_post does and
// makes the view after the step the handle's own: a launch less (two in a plain
// step).  Every wave releases its stores before the count; the last workgroup
// acquires after it.
template <class Mdl, int SEG, bool PLAIN>
__device__ __forceinline__ void finish_step(const StepArgs& a, int f) {
  constexpr int DX = Mdl::DX, DZ = Mdl::DZ;
  constexpr bool YH = has_yhat<Mdl>() && !PLAIN;
  constexpr int NV = DX + DZ + (YH ? 1 : 0);
  constexpr int NSEG = kBlock / SEG;
  __shared__ double part[kBlock / kWave][NV];
  __shared__ int last;
  const int N = a.fN[f], oo = a.ooff[f];
  __threadfence();
  __syncthreads();
  if (threadIdx.x == 0) last = atomicAdd(&a.fcount[f], 1) == (N + NSEG - 1) / NSEG + (PLAIN ? 1 : 0) - 1;
  __syncthreads();
  if (!last) return;
  __threadfence();
  const int t = a.tcur_n[f], act = a.act_n[f], cu = a.cur_n[f];
  if (!PLAIN && (act & 2)) {
    const int i = min((int)threadIdx.x, N - 1);
    const double w = 1.0 / N;
    double v[NV];
    const float* xs = a.x[copy_of((unsigned char)cu)];
#pragma unroll
    for (int d = 0; d < DX; ++d) v[d] = (double)xs[(long long)d * a.NT + oo + i];
#pragma unroll
    for (int d = 0; d < DZ; ++d) v[DX + d] = (double)a.kpart[(long long)(oo + i) * DZ + d];
    if constexpr (YH) v[NV - 1] = a.yp != nullptr ? (double)a.yp[oo + i] : 0.0;
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = (int)threadIdx.x < N ? w * v[q] : 0.0;
    const double e = est_partial<NV>(v, part);
    const int q = threadIdx.x;
    if (q < DX + DZ || (YH && q < NV && a.yp != nullptr)) est_store<DX, DZ>(a, f, t, q, 0.0 + e);
  }
  if (threadIdx.x == 0) {
    a.fcount[f] = 0;
    a.tcur[f] = t;
    a.cur[f] = (unsigned char)cu;
    a.act[f] = (unsigned char)act;
  }
}

// With the wide inner state the children of one parent (neighbouring tiles
// after the ordered resampling) run on one XCD and read the parent's cloud
// through one L2.
template <class Mdl, int SEG, int JPT, bool PLAIN, int ORD = 0>
static __global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(min_waves<Mdl>()))) void k_newcloud(StepArgs a) {
  if ((int)blockIdx.x < a.n_head) {
    if constexpr (!PLAIN) est_head<Mdl::DX, Mdl::DZ, has_yhat<Mdl>()>(a, blockIdx.x);
    else if constexpr (!Mdl::kStreamZ) {
      est_head_plain<Mdl::DX, Mdl::DZ>(a, blockIdx.x);
      if (a.finish) finish_step<Mdl, SEG, PLAIN>(a, blockIdx.x);
    }
    return;
  }
  const int b = (int)blockIdx.x - a.n_head;
  const int ti = Mdl::kStreamZ ? xcd_contiguous_tile(b, (int)gridDim.x - a.n_head) : b;
  newcloud_tile<Mdl, SEG, JPT, PLAIN, ORD>(a, ti);
  if constexpr (!Mdl::kStreamZ) {
    if (a.finish) finish_step<Mdl, SEG, PLAIN>(a, a.tiles[ti].x);
  }
}

// Learned step: the new clouds of the filters that fell back only (smaller
// grid looping over the tiles, tiles checked at once).
template <class Mdl, int SEG, int JPT>
static __global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(min_waves<Mdl>()))) void k_newcloud_fallback(StepArgs a) {
  constexpr bool PLAIN = false;
  // the first n_commit workgroups commit the filters that kept their
  // learned proposals
  if ((int)blockIdx.x < a.n_commit) {
    commit_group<Mdl::DX, Mdl::DZ>(a, blockIdx.x);
    return;
  }
  const int bid = blockIdx.x - a.n_commit, nb = gridDim.x - a.n_commit;
  __shared__ int todo[kBlock], wcnt[kBlock / kWave];
  for (int base = bid; base < a.n_tiles; base += kBlock * nb) {
    const int mine = base + threadIdx.x * nb;
    // tile, then both of its filter's bytes in one round (clamped, masked)
    const int f = a.tiles[min(mine, a.n_tiles - 1)].x;
    const int ac = a.act[f], fbv = a.fb[f];
    const bool need = mine < a.n_tiles && ac && fbv;
    const int nt = block_compact(need, mine, todo, wcnt, nullptr);
    for (int q = 0; q < nt; ++q) {
      newcloud_tile<Mdl, SEG, JPT, PLAIN>(a, todo[q]);
      __syncthreads();
    }
  }
}

}  // namespace dpf
