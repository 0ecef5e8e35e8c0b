// Small service kernels: per-filter reset, activity mask for multi-step
// runs, state export / import, and the kernel-level primitives exposed for
// testing (raw Philox words, normals, systematic resampling) -- the latter
// call the same device functions as the step kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dpf_kernels.hpp"

namespace dpf {

// t = 0, state in copy 0 (the plain DPF's initial proposals are written
// there from the prior held in copy 1), flags and evidence cleared.  keep: the
// bits of cur that stay (where the last step's weights lie).
static __global__ void k_reset(int* tcur, unsigned char* cur, unsigned char* act, uint32_t* flags, double* loglik,
                        uint32_t* lflags, int* fcount, int F, int keep) {
  const int f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= F) return;
  tcur[f] = 0;
  fcount[f] = 0;
  cur[f] = (unsigned char)(6 | (keep ? cur[f] & keep : 0));  // copy 0; identity cloud slots in both copies
  act[f] = 1;
  flags[f] = 0u;
  loglik[f] = 0.0;
  lflags[f] = 0u;
}

static __global__ __launch_bounds__(kBlock) void k_zero(float* p, long long n) {
  for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < n; e += (long long)gridDim.x * kBlock) p[e] = 0.f;
}

// Element e of an array of per-filter segments: find the filter by binary
// search over the offsets (the arrays are sized by the host).
__device__ __forceinline__ int filter_of(const long long* off, int F, long long e) {
  int lo = 0, hi = F - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= e)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// x is [DX][NT]: element e = d * NT + g, filter by g.
static __global__ void k_state_copy_x(float* ext, float* buf0, float* buf1, const unsigned char* cur,
                               const long long* ooff64, int F, int NT, int DX, int dir) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (long long)NT * DX) return;
  const int f = filter_of(ooff64, F, e % NT);
  float* buf = (cur[f] & 1) ? buf1 : buf0;
  if (dir == 0)
    ext[e] = buf[e];
  else
    buf0[e] = ext[e];
}

// The estimates of a handle to up to five arrays of the caller, in one launch:
// a step served by itself is bound by its launches, and five copies took
// longer than the step's kernels.  Words of 4 bytes (nothing is asked of the
// arrays beyond what their types ask).
constexpr int kEstArrays = 5;
struct EstCopy {
  uint32_t* dst[kEstArrays];
  const uint32_t* src[kEstArrays];
  long long end[kEstArrays];  // words of this array and those before it
};
static __global__ __launch_bounds__(kBlock) void k_estimate_copy(EstCopy e) {
  const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
  long long first = 0;
#pragma unroll
  for (int q = 0; q < kEstArrays; ++q) {
    if (i >= first && i < e.end[q]) e.dst[q][i - first] = e.src[q][i - first];
    first = e.end[q];
  }
}

// ---- state export and import: one launch
// The external state is [t (F words, padded to tb bytes)][x][z][lam] in the
// layouts of the workspace.  Workgroup (b, y) moves the y-th of gridDim.y
// equal shares of resampling group b's outer particles: their clouds are
// dz M and M contiguous floats each, one run for the whole share when the
// copy is in slot order (always so on import, which fills copy 0).  The copy
// is memory-bound; whole runs moved 16 bytes at a time, with the group's
// offsets from the static tables, replace a per-element search and 64-bit
// divisions (16384 x 1024 x 64, 4.36 GB: 4.6 ms before, 1.6 ms or 5.3 TB/s now).
struct StateIo {
  char* ext;
  size_t tb;
  float* x[2];
  float* z[2];
  float* lam[2];
  const int* ind[2];
  int* tcur;
  unsigned char* cur;
  uint32_t* flags;
  double* loglik;
  const int2* rgroups;
  const int4* ginfo;
  const int* fM;
  const long long* ioff;
  int F, NT, dx, dz;
  long long NMT;
};

// n floats, all 256 threads: 16 bytes per thread and load where source and
// destination have the same place within 16 bytes (the head and tail single),
// else 4 bytes.
__device__ __forceinline__ void copy_run(float* dst, const float* src, long long n) {
  const int th = threadIdx.x;
  long long done = 0;
  if ((((uintptr_t)dst ^ (uintptr_t)src) & 15) == 0) {
    const long long head = min(n, (long long)((16 - ((uintptr_t)src & 15)) & 15) / 4);
    if (th < head) dst[th] = src[th];
    const long long n4 = (n - head) / 4;
    const float4* s4 = reinterpret_cast<const float4*>(src + head);
    float4* d4 = reinterpret_cast<float4*>(dst + head);
#pragma unroll 4
    for (long long e = th; e < n4; e += kBlock) d4[e] = s4[e];
    done = head + 4 * n4;
  }
#pragma unroll 4
  for (long long e = done + th; e < n; e += kBlock) dst[e] = src[e];
}

template <bool IMPORT>
static __global__ __launch_bounds__(kBlock) void k_state_io(StateIo a) {
  const int2 rg = a.rgroups[blockIdx.x];
  const int4 gi = a.ginfo[blockIdx.x];
  const int f = rg.x, oo = gi.x, N = gi.y;
  const long long io = a.ioff[f];
  const int M = a.fM[f];
  const int cb = IMPORT ? 6 : a.cur[f];  // (an import fills copy 0 in slot order)
  const int c = copy_of((unsigned char)cb);
  const bool ident = ident_slots((unsigned char)cb, c);
  float* ex = reinterpret_cast<float*>(a.ext + a.tb);
  float* ez = ex + (size_t)a.NT * a.dx;
  float* el = ez + (size_t)a.NMT * a.dz;
  // this share's particles [i0, i1) of the group
  const int g0 = rg.y * kResGroup, ng = min(kResGroup, N - g0);
  const int per = (ng + gridDim.y - 1) / gridDim.y;
  const int i0 = g0 + min(ng, (int)blockIdx.y * per), i1 = g0 + min(ng, ((int)blockIdx.y + 1) * per);
  if (blockIdx.y == 0) {
    for (int d = 0; d < a.dx; ++d) {
      float* e = ex + (size_t)d * a.NT + oo + g0;
      float* w = a.x[c] + (size_t)d * a.NT + oo + g0;
      if ((int)threadIdx.x < ng) {
        if constexpr (IMPORT) w[threadIdx.x] = e[threadIdx.x];
        else e[threadIdx.x] = w[threadIdx.x];
      }
    }
    int* et = reinterpret_cast<int*>(a.ext);
    if (rg.y == 0 && threadIdx.x == 0) {
      if constexpr (IMPORT) {
        a.tcur[f] = et[f];
        a.cur[f] = (unsigned char)(6 | (a.cur[f] & kCurPair));
        a.flags[f] = 0u;
        a.loglik[f] = 0.0;
      } else {
        et[f] = a.tcur[f];
      }
    }
    // zeros in the padding of the time header
    if (!IMPORT && blockIdx.x == 0 && threadIdx.x < (int)(a.tb / 4) - a.F) et[a.F + threadIdx.x] = 0;
  }
  if (i0 >= i1) return;
  const long long zw = (long long)M * a.dz;
  if constexpr (IMPORT) {
    copy_run(a.z[0] + io * a.dz + i0 * zw, ez + io * a.dz + i0 * zw, (i1 - i0) * zw);
    copy_run(a.lam[0] + io + (long long)i0 * M, el + io + (long long)i0 * M, (long long)(i1 - i0) * M);
  } else if (ident) {
    copy_run(ez + io * a.dz + i0 * zw, a.z[c] + io * a.dz + i0 * zw, (i1 - i0) * zw);
    copy_run(el + io + (long long)i0 * M, a.lam[c] + io + (long long)i0 * M, (long long)(i1 - i0) * M);
  } else {
    for (int i = i0; i < i1; ++i) {
      const long long sl = a.ind[c][oo + i];
      copy_run(ez + io * a.dz + i * zw, a.z[c] + io * a.dz + sl * zw, zw);
      copy_run(el + io + (long long)i * M, a.lam[c] + io + sl * M, M);
    }
  }
}

// Moves the weights of the filters whose last step's lie in the second pair
// (kCurPair) into the first, which then holds every filter's: of the groups'
// inner particles (inner) or of their outer ones.  Workgroups as in k_state_io.
// Calls repeat safely: the second pair and the bits stay as they are.
static __global__ __launch_bounds__(kBlock) void k_last_weights(const unsigned char* cur, const int2* rgroups,
                                                                const int4* ginfo, const int* fM,
                                                                const long long* ioff, const float* second,
                                                                float* first, int inner) {
  const int2 rg = rgroups[blockIdx.x];
  const int4 gi = ginfo[blockIdx.x];
  const int f = rg.x, oo = gi.x, N = gi.y;
  if (!(cur[f] & kCurPair)) return;
  const int g0 = rg.y * kResGroup, ng = min(kResGroup, N - g0);
  const int per = (ng + gridDim.y - 1) / gridDim.y;
  const int i0 = g0 + min(ng, (int)blockIdx.y * per), i1 = g0 + min(ng, ((int)blockIdx.y + 1) * per);
  const long long M = inner ? fM[f] : 1, at = (inner ? ioff[f] : (long long)oo) + i0 * M;
  copy_run(first + at, second + at, (i1 - i0) * M);
}

// ---------------------------------------------------------------- primitives
static __global__ void k_philox_words(Key key, const uint32_t* ctr, long long n, uint32_t* out) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const Words w = philox(key, ctr[4 * e], ctr[4 * e + 1], ctr[4 * e + 2], ctr[4 * e + 3]);
#pragma unroll
  for (int q = 0; q < 4; ++q) out[4 * e + q] = w.w[q];
}

template <int D>
static __global__ void k_normals_grid(Key key, uint32_t t, uint32_t purpose, int na, int nb, float* out) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (long long)na * nb) return;
  const int a = (int)(e / nb), b = (int)(e % nb);
  float v[D];
  normals<D>(key, t, (uint32_t)a, (uint32_t)b, purpose, v);
#pragma unroll
  for (int d = 0; d < D; ++d) out[e * D + d] = v[d];
}

// Systematic resampling of one FP64 weight vector by the outer-resampling
// code of the step (group statistics, then points resolved 256 per
// workgroup by the same device function the new-cloud kernel uses).
static __global__ __launch_bounds__(kBlock) void k_prim_res_stats(const double* w, int n, double* gstat) {
  __shared__ ResScratch sh;
  float mg;
  double sg, qg;
  res_group_stat(LinSrc{w}, n, blockIdx.x, mg, sg, qg, sh);
  if (threadIdx.x == 0) {
    gstat[4 * blockIdx.x + 0] = (double)mg;
    gstat[4 * blockIdx.x + 1] = sg;
    gstat[4 * blockIdx.x + 2] = qg;
  }
}

static __global__ __launch_bounds__(kBlock) void k_prim_res_select(const double* w, int n, int n_out, double u,
                                                            const double* gstat, int* out) {
  __shared__ ResScratch sh;
  __shared__ int res[kBlock];
  const int G = (n + kResGroup - 1) / kResGroup;
  const int k0 = blockIdx.x * kBlock;
  const int np = min(kBlock, n_out - k0);
  resolve_points(LinSrc{w}, n, n_out, u, k0, np, gstat, G, res, sh, false);
  if (threadIdx.x < np) out[k0 + threadIdx.x] = res[threadIdx.x];
}

// One segment per (S index); the cdf build and search are those of k_newcloud.
template <int SEG, int JPT>
static __global__ __launch_bounds__(kBlock) void k_seg_systematic_prim(const double* wt, int S, int n,
                                                                 int n_out, const double* u,
                                                                 int* out) {
  constexpr int NSEG = kBlock / SEG;
  __shared__ SegScratch sh;
  __shared__ double cdf[NSEG][SEG * JPT];
  const int s = threadIdx.x / SEG;
  const int ls = threadIdx.x % SEG;
  const int g = blockIdx.x * NSEG + s;
  const bool vg = g < S;
  double w[JPT], P[JPT];
  int res[JPT];
#pragma unroll
  for (int r = 0; r < JPT; ++r) {
    const int j = ls * JPT + r;
    w[r] = (vg && j < n) ? wt[(long long)g * n + j] : 0.0;
  }
  seg_cdf<SEG, JPT>(w, cdf[s], sh);
  __syncthreads();
  if (!vg) return;
  const double uu = u[g];
  const double total = cdf[s][n - 1];
#pragma unroll
  for (int r = 0; r < JPT; ++r) {
    const int k = ls + r * SEG;
    P[r] = k < n_out ? sys_point(k, uu, total, n_out) : 0.0;
  }
  cdf_find<SEG * JPT, JPT>(cdf[s], n, total, P, res);
#pragma unroll
  for (int r = 0; r < JPT; ++r) {
    const int k = ls + r * SEG;
    if (k < n_out) out[(long long)g * n_out + k] = res[r];
  }
}

}  // namespace dpf
