// Learned proposal network: a mixture density network over x_t that stands
// in for the Monte Carlo optimal-proposal estimate of eq:approx3.
//
// Network: 32 (features, zero padded) -> 256 -> 256 -> 32 outputs (20 used:
// 4 mixture logits, 4 x 2 means, 4 x 2 log standard deviations), tanh-form
// GELU after both hidden layers.  Matrix products run on the gfx950 matrix
// cores, v_mfma_f32_16x16x32_bf16: BF16 operands (round to nearest even),
// FP32 accumulation.  Lane l of a wave holds, for a 16 x 16 x 32 step,
//   A: row l % 16, k = 8 (l / 16) .. 8 (l / 16) + 7   (8 bf16, 16 bytes)
//   B: col l % 16, the same 8 k                         (8 bf16, 16 bytes)
//   D: col l % 16, rows 4 (l / 16) .. 4 (l / 16) + 3    (4 floats)
// so both operands are read as 16-byte vectors from k-contiguous storage:
// weights as [out][in] (and transposed copies for the backward pass),
// activations row-major in LDS, and in HBM, where the batch is the contraction
// index (weight gradients), blocked by 32 batch rows: [B / 32][columns][32],
// so that an operand fragment is 1 KB of contiguous memory.
//
// Row tiles: a 256-thread workgroup (4 waves) owns 16 rows of the batch (the
// network on a large handle's state up to four such tiles: MlpTiles);
// wave w computes hidden columns 64 w .. 64 w + 63.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dpf_models.hpp"
#include "dpf_seg.hpp"

namespace dpf {

constexpr int kMlpIn = 32;
constexpr int kMlpHid = 256;
constexpr int kMlpOut = 32;
constexpr int kMix = 4;
constexpr int kMlpRows = 16;
constexpr float kLogSdMin = -6.907755278982137f;  // log 1e-3
constexpr float kLogSdMax = 6.907755278982137f;   // log 1e3

// Device blob of the network (bytes): BF16 weights [out][in], FP32 biases,
// and the feature standardisation (mean, standard deviation).
struct MlpBlobLayout {
  static constexpr size_t W1 = 0;                                  // bf16 [256][32]
  static constexpr size_t W2 = W1 + kMlpHid * kMlpIn * 2;          // bf16 [256][256]
  static constexpr size_t W3 = W2 + kMlpHid * kMlpHid * 2;         // bf16 [32][256]
  static constexpr size_t b1 = W3 + kMlpOut * kMlpHid * 2;         // f32 [256]
  static constexpr size_t b2 = b1 + kMlpHid * 4;                   // f32 [256]
  static constexpr size_t b3 = b2 + kMlpHid * 4;                   // f32 [32]
  static constexpr size_t fmean = b3 + kMlpOut * 4;                // f32 [32]
  static constexpr size_t fstd = fmean + kMlpIn * 4;               // f32 [32]
  static constexpr size_t bytes = fstd + kMlpIn * 4;
};

// FP32 parameter vector (training masters, Adam moments, gradients).
struct MlpParamLayout {
  static constexpr int W1 = 0;                          // [256][32]
  static constexpr int b1 = W1 + kMlpHid * kMlpIn;      // [256]
  static constexpr int W2 = b1 + kMlpHid;               // [256][256]
  static constexpr int b2 = W2 + kMlpHid * kMlpHid;     // [256]
  static constexpr int W3 = b2 + kMlpHid;               // [32][256]
  static constexpr int b3 = W3 + kMlpOut * kMlpHid;     // [32]
  static constexpr int n = b3 + kMlpOut;
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short bf16_t;

// Round to nearest even; NaN stays NaN (the card's own conversion; by integer
// arithmetic it was a third of a hidden layer's vector instructions).
__device__ __forceinline__ bf16_t f2bf(float v) { return __builtin_bit_cast(bf16_t, (__bf16)v); }

__device__ __forceinline__ bf16x8 ld8(const bf16_t* p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p));
}

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

constexpr float kGeluC = 0.7978845608028654f;  // sqrt(2 / pi)
constexpr float kGeluA = 0.044715f;

__device__ __forceinline__ float gelu_f(float a) {
  const float th = tanh_f(kGeluC * (a + kGeluA * a * a * a));
  return 0.5f * a * (1.0f + th);
}
__device__ __forceinline__ float gelu_grad_f(float a) {
  const float th = tanh_f(kGeluC * (a + kGeluA * a * a * a));
  const float du = kGeluC * (1.0f + 3.0f * kGeluA * a * a);
  return 0.5f * (1.0f + th) + 0.5f * a * (1.0f - th * th) * du;
}

// LDS row strides (bf16 elements), padded by 16 bytes so that the 16 rows
// of an operand fragment fall on distinct banks.
constexpr int kInStride = kMlpIn + 8;
constexpr int kHidStride = kMlpHid + 8;

struct alignas(16) MlpShared {
  bf16_t x0[kMlpRows][kInStride];
  bf16_t h1[kMlpRows][kHidStride];
  bf16_t h2[kMlpRows][kHidStride];
  float part[2][kMlpRows][16];
  float o[kMlpRows][kMlpOut + 1];  // outputs of the tile (for an epilogue per row)
};

// Weight fragments and biases of one wave, loaded before the layer inputs
// are ready so that the three layers find their operands in registers.
// Wave w owns the NT column tiles 16 NT w .. of the hidden layers (16 / NT
// waves) and, waves 0 to 3 in the output layer, column tile w & 1 over k-steps
// 4 (w >> 1) .. 4 (w >> 1) + 3.
template <int NT>
struct MlpFrags {
  bf16x8 w1[1][NT];
  bf16x8 w2[8][NT];
  bf16x8 w3[4];
  float b1[NT], b2[NT], b3;
};

// Fragment order of a weight matrix [n][k] with 16 NTL rows n: element (n, k)
// at the place where the lane that needs it reads, so that a fragment is 1 KB
// of contiguous memory instead of 16 pieces of 64 bytes a row apart.  All
// workgroups fetch the same weights at once, and those pieces met on few L2
// channels: the training kernel spent 9 us of its 20 on the 156 KB.  Used for
// the training copies and the handle's copy of the network; the public blob
// keeps its row-major layout.
__device__ __forceinline__ int frag_at(int n, int k, int ntl) {
  return ((k / 32 * ntl + n / 16) * 64 + (k / 8) % 4 * 16 + n % 16) * 8 + k % 8;
}

// The fragment of k-step ks and row tile tile, lane l, row-major (leading
// dimension ld) or in fragment order.
template <bool FRAG>
__device__ __forceinline__ bf16x8 ld_frag(const bf16_t* W, int ks, int tile, int ntl, int ld) {
  const int l = threadIdx.x & 63;
  if constexpr (FRAG) return ld8(W + ((ks * ntl + tile) * 64 + l) * 8);
  else return ld8(W + (size_t)(16 * tile + (l & 15)) * ld + 32 * ks + 8 * (l >> 4));
}

template <int NT, bool FRAG>
__device__ __forceinline__ void mlp_load_frags(const bf16_t* W1, const bf16_t* W2, const bf16_t* W3,
                                               const unsigned char* blob, MlpFrags<NT>& fr) {
  using BL = MlpBlobLayout;
  const float* b1 = reinterpret_cast<const float*>(blob + BL::b1);
  const float* b2 = reinterpret_cast<const float*>(blob + BL::b2);
  const float* b3 = reinterpret_cast<const float*>(blob + BL::b3);
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int lr = l & 15;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    fr.w1[0][nt] = ld_frag<FRAG>(W1, 0, NT * w + nt, 16, kMlpIn);
    fr.b1[nt] = b1[16 * (NT * w + nt) + lr];
    fr.b2[nt] = b2[16 * (NT * w + nt) + lr];
  }
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) fr.w2[ks][nt] = ld_frag<FRAG>(W2, ks, NT * w + nt, 16, kMlpHid);
  }
  const int k3 = 4 * ((w >> 1) & 1);
#pragma unroll
  for (int q = 0; q < 4; ++q) fr.w3[q] = ld_frag<FRAG>(W3, k3 + q, w & 1, 2, kMlpHid);
  fr.b3 = b3[16 * (w & 1) + lr];
}

// From a blob: the caller's (row-major) or a handle's (fragment order).
template <int NT, bool FRAG>
__device__ __forceinline__ void mlp_load_blob(const unsigned char* blob, MlpFrags<NT>& fr) {
  using BL = MlpBlobLayout;
  mlp_load_frags<NT, FRAG>(reinterpret_cast<const bf16_t*>(blob + BL::W1),
                           reinterpret_cast<const bf16_t*>(blob + BL::W2),
                           reinterpret_cast<const bf16_t*>(blob + BL::W3), blob, fr);
}

// Batch-blocked operands of the weight gradients: row b of column n of a
// matrix with N columns.  (As [N][B] each column was a power-of-two stride
// away from the next: the fragments' 64-byte pieces fell on few memory
// channels: 13.5 us for the weight-gradient kernel of batch 4096, 8.4 us
// blocked.)
constexpr int kBatchBlk = 32;
__device__ __forceinline__ size_t blk_at(int b, int n, int N) {
  return ((size_t)(b / kBatchBlk) * N + n) * kBatchBlk + b % kBatchBlk;
}

// Four bf16 of consecutive batch rows (8-byte aligned).
__device__ __forceinline__ void store_rows4(bf16_t* p, const bf16_t* h) {
  *reinterpret_cast<uint2*>(p) = make_uint2(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16));
}

// Hidden layer: rows of `in` (LDS, K = KIN) times the wave's weight
// fragments plus bias, GELU, rounded into `out` (LDS).  With TRAIN the
// pre-activations stay in a[NT][4] (column tile, row: this lane's D elements)
// and the outputs also go to the batch-blocked h_t (the tile's rows from
// row0), four rows per 8-byte store.
template <int NT, int KIN, int SIN, bool TRAIN>
__device__ __forceinline__ void mlp_hidden(const bf16_t (*in)[SIN], const bf16x8 (*wf)[NT], const float* bias,
                                           bf16_t (*out)[kHidStride], int row0 = 0, float (*a)[4] = nullptr,
                                           bf16_t* h_t = nullptr) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int lr = l & 15, lk = 8 * (l >> 4);
  f32x4 acc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < KIN / 32; ++ks) {
    const bf16x8 a = ld8(&in[lr][32 * ks + lk]);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = mfma16(a, wf[ks][nt], acc[nt]);
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int n = 16 * (NT * w + nt) + lr;
    const float bn = bias[nt];
    bf16_t h[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v = acc[nt][r] + bn;
      h[r] = f2bf(gelu_f(v));
      out[4 * (l >> 4) + r][n] = h[r];
      if constexpr (TRAIN) a[nt][r] = v;
    }
    if constexpr (TRAIN) store_rows4(h_t + blk_at(row0 + 4 * (l >> 4), n, kMlpHid), h);
  }
}

// Output layer of the 16 rows in sh.h2 -> sh.o (and out [rows][32] when
// given): 2 column tiles x 8 k-steps, split over the 4 waves.
template <int NT>
__device__ __forceinline__ void mlp_out_layer(const MlpFrags<NT>& fr, MlpShared& sh, int row0, int nrows, float* out) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int lr = l & 15, lk = 8 * (l >> 4);
  const int nt = w & 1, kh = w >> 1;
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < 4; ++q) acc = mfma16(ld8(&sh.h2[lr][32 * (4 * (kh & 1) + q) + lk]), fr.w3[q], acc);
  if (kh == 1) {
#pragma unroll
    for (int r = 0; r < 4; ++r) sh.part[nt][4 * (l >> 4) + r][lr] = acc[r];
  }
  __syncthreads();
  if (kh == 0) {
    const int n = 16 * nt + lr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 4 * (l >> 4) + r;
      const float v = (acc[r] + sh.part[nt][row][lr]) + fr.b3;
      sh.o[row][n] = v;
      if (out && row < nrows) out[(size_t)(row0 + row) * kMlpOut + n] = v;
    }
  }
}

// The three layers for the 16 rows in sh.x0; outputs [rows][32] FP32.
template <int NT>
__device__ __forceinline__ void mlp_rows(const MlpFrags<NT>& fr, MlpShared& sh, int row0, int nrows, float* out) {
  mlp_hidden<NT, kMlpIn, kInStride, false>(sh.x0, fr.w1, fr.b1, sh.h1);
  __syncthreads();
  mlp_hidden<NT, kMlpHid, kHidStride, false>(sh.h1, fr.w2, fr.b2, sh.h2);
  __syncthreads();
  mlp_out_layer(fr, sh, row0, nrows, out);
}

// The same for RT row tiles at once (4 waves): one buffer for both hidden
// layers, each read whole before its successor is written.
template <int RT>
struct alignas(16) MlpTiles {
  bf16_t x0[16 * RT][kInStride];
  bf16_t h[16 * RT][kHidStride];
  float part[2][16 * RT][16];
  float o[16 * RT][kMlpOut + 1];
};
template <int RT, int KIN, int SIN>
__device__ __forceinline__ void mlp_hidden_tiles(const bf16_t (*in)[SIN], const bf16x8 (*wf)[4], const f32x4* bias,
                                                 bf16_t (*out)[kHidStride]) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int lr = l & 15, lk = 8 * (l >> 4);
  // (weights as the A operand: a lane's four D elements are consecutive
  // columns of one row, an 8-byte store)
  f32x4 acc[RT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) acc[rt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int ks = 0; ks < KIN / 32; ++ks) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const bf16x8 a = ld8(&in[16 * rt + lr][32 * ks + lk]);
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) acc[rt][nt] = mfma16(wf[ks][nt], a, acc[rt][nt]);
    }
  }
  __syncthreads();  // in may be out
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      bf16_t h[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) h[r] = f2bf(gelu_f(acc[rt][nt][r] + bias[nt][r]));
      store_rows4(&out[16 * rt + lr][16 * (4 * w + nt) + 4 * (l >> 4)], h);
    }
  }
  __syncthreads();
}
template <int RT>
__device__ __forceinline__ void mlp_tiles(const MlpFrags<4>& fr, const unsigned char* blob, MlpTiles<RT>& sh, int row0,
                                          int nrows, float* out) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  f32x4 b1[4], b2[4];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    const int n = 16 * (4 * w + nt) + 4 * (l >> 4);
    b1[nt] = *reinterpret_cast<const f32x4*>(blob + MlpBlobLayout::b1 + 4 * n);
    b2[nt] = *reinterpret_cast<const f32x4*>(blob + MlpBlobLayout::b2 + 4 * n);
  }
  mlp_hidden_tiles<RT, kMlpIn, kInStride>(sh.x0, fr.w1, b1, sh.h);
  mlp_hidden_tiles<RT, kMlpHid, kHidStride>(sh.h, fr.w2, b2, sh.h);
  const int lr = l & 15, lk = 8 * (l >> 4);
  const int nt = w & 1, kh = w >> 1;
  f32x4 acc[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    acc[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 4; ++q)
      acc[rt] = mfma16(ld8(&sh.h[16 * rt + lr][32 * (4 * kh + q) + lk]), fr.w3[q], acc[rt]);
    if (kh == 1) {
#pragma unroll
      for (int r = 0; r < 4; ++r) sh.part[nt][16 * rt + 4 * (l >> 4) + r][lr] = acc[rt][r];
    }
  }
  __syncthreads();
  if (kh == 0) {
    const int n = 16 * nt + lr;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * rt + 4 * (l >> 4) + r;
        const float v = (acc[rt][r] + sh.part[nt][row][lr]) + fr.b3;
        sh.o[row][n] = v;
        if (out && row < nrows) out[(size_t)(row0 + row) * kMlpOut + n] = v;
      }
    }
  }
}

// Standardised FP32 features X [B][32] -> outputs [B][32].
static __global__ __launch_bounds__(kBlock) void k_mlp_fwd_x(const unsigned char* blob, const float* X, int B,
                                                      float* out) {
  __shared__ MlpShared sh;
  MlpFrags<4> fr;
  mlp_load_blob<4, false>(blob, fr);
  const int row0 = blockIdx.x * kMlpRows;
  const int nrows = min(kMlpRows, B - row0);
  for (int e = threadIdx.x; e < kMlpRows * kMlpIn; e += kBlock) {
    const int r = e / kMlpIn, c = e % kMlpIn;
    const bf16_t v = r < nrows ? f2bf(X[(size_t)(row0 + r) * kMlpIn + c]) : (bf16_t)0;
    sh.x0[r][c] = v;
  }
  __syncthreads();
  mlp_rows(fr, sh, row0, nrows, out);
}

// ---------------------------------------------------------------- MDN
// Output row: logits [0, 4), means [4, 4 + 4 DX) as [component][d], log
// standard deviations [4 + 4 DX, 4 + 8 DX) likewise, clamped to
// [log 1e-3, log 1e3].
template <int DX>
struct Mdn {
  static constexpr int kMu = kMix, kSd = kMix + kMix * DX, kUsed = kMix + 2 * kMix * DX;
  static_assert(kUsed <= kMlpOut, "mixture does not fit the output layer");
};

__device__ __forceinline__ float clamp_sd(float s) { return fminf(fmaxf(s, kLogSdMin), kLogSdMax); }

// log q(x) of the mixture in row o.
template <int DX>
__device__ float mdn_logpdf(const float* o, const float* x) {
  using Q = Mdn<DX>;
  float lmax = -INFINITY;
#pragma unroll
  for (int c = 0; c < kMix; ++c) lmax = fmaxf(lmax, o[c]);
  float se = 0.f;
#pragma unroll
  for (int c = 0; c < kMix; ++c) se += fast_exp(o[c] - lmax);
  const float lse_l = lmax + fast_log(se);
  float e[kMix], emax = -INFINITY;
#pragma unroll
  for (int c = 0; c < kMix; ++c) {
    float q = 0.f;
#pragma unroll
    for (int d = 0; d < DX; ++d) {
      const float s = clamp_sd(o[Q::kSd + c * DX + d]);
      const float z = (x[d] - o[Q::kMu + c * DX + d]) * fast_exp(-s);
      q += -0.5f * z * z - s - 0.5f * kLn2Pi;
    }
    e[c] = (o[c] - lse_l) + q;
    emax = fmaxf(emax, e[c]);
  }
  float s2 = 0.f;
#pragma unroll
  for (int c = 0; c < kMix; ++c) s2 += fast_exp(e[c] - emax);
  return emax + fast_log(s2);
}

// ------------------------------------------- training: forward and backward
// One 16-row tile of the batch per workgroup goes through the forward pass,
// the gradient of the mean mixture NLL and the backward pass through layers
// 3 and 2 in one launch: the pre-activations stay in the lanes that need them
// again (the backward products have the forward ones' lane layout), the
// outputs and their gradient in LDS.  What leaves the workgroup is what the
// weight gradients contract over the batch (layer inputs and gradients,
// BF16, batch-blocked) and the tile's partial sums of the bias gradients
// and the loss.  The tile is bound by its own chain (two 128 KB weight
// fetches from L2, five barriers, 64 GELU terms per lane), not by the matrix
// cores; the transposed W2 is requested before the output layer so that it
// arrives behind it.  Batch 4096 (256 tiles, one per CU): forward 14.8 us,
// gradient 8.7 us and backward 22.8 us as three launches with the
// pre-activations in HBM, 11.8 us now.  Each XCD takes a contiguous run of
// tiles: two tiles share each 64-byte line of the batch-blocked outputs, and
// dealt to different L2s they cost 4.3 us more.
constexpr int kTrainNT = 2;  // column tiles per wave
constexpr int kTrainThreads = kWave * 16 / kTrainNT;

struct MlpTrainArgs {
  const unsigned char* blob;
  const float* X;    // [.][32] standardised features
  const float* xt;   // [.][2] targets
  const int* idx;    // rows of X and xt that make up the batch, or null: rows 0 .. B - 1
  long long n_src;   // rows of X and xt (with idx; an index outside gives a row of NaNs)
  const bf16_t* W1;   // weights in fragment order
  const bf16_t* W2;
  const bf16_t* W3;
  const bf16_t* W3t;  // transposed weights [256][32] and [256][256] likewise
  const bf16_t* W2t;
  bf16_t* x0t;        // batch-blocked, 32 columns
  bf16_t* h1t;        // 256
  bf16_t* h2t;        // 256
  bf16_t* gt;         // 32
  bf16_t* da2t;       // 256
  bf16_t* da1t;       // 256
  float* b1_part;     // [tiles][256]
  float* b2_part;     // [tiles][256]
  float* b3_part;     // [tiles][32]
  double* loss_part;  // [tiles]
  int B;              // a multiple of 16
};

// Sum of a tile's 16 rows in the order of a DPP row reduction: quads of rows
// as (0 + 1) + (2 + 3), then the quads likewise.
template <class T, class F>
__device__ __forceinline__ T rows16_sum(F&& v) {
  T q[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) q[k] = (v(4 * k) + v(4 * k + 1)) + (v(4 * k + 2) + v(4 * k + 3));
  return (q[0] + q[1]) + (q[2] + q[3]);
}

// Value of the quad's lane K in all four lanes.
template <int K>
__device__ __forceinline__ float quad_get(float v) {
  return dpp_f<K * 0x55>(v, v);
}

// Gradient of the mean NLL (divided by B) w.r.t. the outputs o [16][..] of a
// tile, by one wave: lane 4 r + c takes component c of row r (sums over the
// components run in component order).  g: FP32 and gb: BF16 rows; nll [16].
template <int DX>
__device__ __forceinline__ void mdn_grad_tile(const float (*o)[kMlpOut + 1], float (*xt)[DX], int B,
                                              float (*g)[kMlpOut + 1], bf16_t (*gb)[kInStride], double* nll) {
  using Q = Mdn<DX>;
  const int l = threadIdx.x & 63;
  const int row = l >> 2, c = l & 3;
  const float oc = o[row][c];
  const float lmax = fmaxf(fmaxf(quad_get<0>(oc), quad_get<1>(oc)), fmaxf(quad_get<2>(oc), quad_get<3>(oc)));
  const float e1 = fast_exp(oc - lmax);
  float se = 0.f;
  se += quad_get<0>(e1);
  se += quad_get<1>(e1);
  se += quad_get<2>(e1);
  se += quad_get<3>(e1);
  const float lse_l = lmax + fast_log(se);
  float zz[DX], sd_inv[DX];
  float q = 0.f;
#pragma unroll
  for (int d = 0; d < DX; ++d) {
    const float s = clamp_sd(o[row][Q::kSd + c * DX + d]);
    sd_inv[d] = fast_exp(-s);
    zz[d] = (xt[row][d] - o[row][Q::kMu + c * DX + d]) * sd_inv[d];
    q += -0.5f * zz[d] * zz[d] - s - 0.5f * kLn2Pi;
  }
  const float ell = (oc - lse_l) + q;
  const float emax = fmaxf(fmaxf(quad_get<0>(ell), quad_get<1>(ell)), fmaxf(quad_get<2>(ell), quad_get<3>(ell)));
  const float e2 = fast_exp(ell - emax);
  float s2 = 0.f;
  s2 += quad_get<0>(e2);
  s2 += quad_get<1>(e2);
  s2 += quad_get<2>(e2);
  s2 += quad_get<3>(e2);
  const float L = emax + fast_log(s2);
  const float invB = 1.0f / (float)B;
  const float gam = fast_exp(ell - L);
  const float pi = fast_exp(oc - lse_l);
  auto put = [&](int col, float v) {
    g[row][col] = v;
    gb[row][col] = f2bf(v);
  };
  put(c, (pi - gam) * invB);
#pragma unroll
  for (int d = 0; d < DX; ++d) {
    const float sr = o[row][Q::kSd + c * DX + d];
    const bool inside = sr > kLogSdMin && sr < kLogSdMax;
    put(Q::kMu + c * DX + d, -gam * zz[d] * sd_inv[d] * invB);
    put(Q::kSd + c * DX + d, inside ? -gam * (zz[d] * zz[d] - 1.0f) * invB : 0.f);
  }
  // the columns beyond the mixture's
#pragma unroll
  for (int k = 0; k < (kMlpOut - Q::kUsed) / kMix; ++k) put(Q::kUsed + kMix * k + c, 0.f);
  if (c == 0) nll[row] = -(double)L;
}

// Weight fragments of a backward product (KIN deep) of wave w's column tiles
// from the transposed weights Wt [256][KIN] in fragment order.
template <int NT, int KIN>
__device__ __forceinline__ void mlp_load_back(const bf16_t* Wt, bf16x8 (*wf)[NT]) {
  const int w = threadIdx.x >> 6;
#pragma unroll
  for (int ks = 0; ks < KIN / 32; ++ks) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) wf[ks][nt] = ld_frag<true>(Wt, ks, NT * w + nt, 16, KIN);
  }
}

// d = (rows of `in`) x Wt^T for the wave's columns, times gelu'(a); the
// BF16 result goes to `out` (LDS, optional) and batch-blocked to dt, its FP32
// column sums to bpart.
template <int NT, int KIN, int SIN>
__device__ __forceinline__ void mlp_back_layer(const bf16_t (*in)[SIN], const bf16x8 (*wf)[NT], const float (*a)[4],
                                               bf16_t (*out)[kHidStride], bf16_t* dt, float* bpart, int row0) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int lr = l & 15, lk = 8 * (l >> 4);
  f32x4 acc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < KIN / 32; ++ks) {
    const bf16x8 av = ld8(&in[lr][32 * ks + lk]);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = mfma16(av, wf[ks][nt], acc[nt]);
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int n = 16 * (NT * w + nt) + lr;
    float cs = 0.f;
    bf16_t h[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float v = acc[nt][r] * gelu_grad_f(a[nt][r]);
      asm volatile("" : "+v"(v));  // the rounded product, not a fused sum
      cs += v;
      h[r] = f2bf(v);
      if (out) out[4 * (l >> 4) + r][n] = h[r];
    }
    store_rows4(dt + blk_at(row0 + 4 * (l >> 4), n, kMlpHid), h);
    // the four row groups of the column: lanes lr, lr+16, lr+32, lr+48
    cs += __shfl_xor(cs, 16);
    cs += __shfl_xor(cs, 32);
    if (l < 16) bpart[n] = cs;
  }
}

// BLOB: the forward pass takes its weights from the caller's blob, which between
// calls is the caller's to rewrite; else from the workspace's fragment-order
// copies, which the step before in the same call has just written (batch 4096:
// 23 us a step from the blob's rows, 21 from the copies).
template <int DX, bool BLOB>
static __global__ __launch_bounds__(kTrainThreads) void k_mlp_train(MlpTrainArgs p) {
  __shared__ MlpShared sh;
  __shared__ float g_sh[kMlpRows][kMlpOut + 1];
  __shared__ alignas(16) bf16_t gb_sh[kMlpRows][kInStride];
  __shared__ float xt_sh[kMlpRows][DX];
  __shared__ double nll_sh[kMlpRows];
  constexpr int NT = kTrainNT;
  const int th = threadIdx.x, w = th >> 6;
  const int tile = xcd_contiguous_tile(blockIdx.x, gridDim.x), row0 = tile * kMlpRows, B = p.B;
  // source row of tile row r (-1: index out of range)
  auto src_row = [&](int r) -> long long {
    if (!p.idx) return row0 + r;
    const long long q = p.idx[row0 + r];
    return q >= 0 && q < p.n_src ? q : -1;
  };
  // the tile's rows first (the barrier waits for them), then the weights
  static_assert(kMlpRows * kMlpIn % kTrainThreads == 0, "whole rounds of the tile's features");
  constexpr int NX = kMlpRows * kMlpIn / kTrainThreads;
  float xv[NX], tv = 0.f;
#pragma unroll
  for (int q = 0; q < NX; ++q) {
    const int e = th + q * kTrainThreads;
    const long long r = src_row(e / kMlpIn);
    xv[q] = r >= 0 ? p.X[(size_t)r * kMlpIn + e % kMlpIn] : NAN;
  }
  if (th < kMlpRows * DX) {
    const long long r = src_row(th / DX);
    tv = r >= 0 ? p.xt[(size_t)r * DX + th % DX] : NAN;
  }
  MlpFrags<NT> fr;
  if constexpr (BLOB) mlp_load_blob<NT, false>(p.blob, fr);
  else mlp_load_frags<NT, true>(p.W1, p.W2, p.W3, p.blob, fr);
#pragma unroll
  for (int q = 0; q < NX; ++q) {
    const int e = th + q * kTrainThreads;
    sh.x0[e / kMlpIn][e % kMlpIn] = f2bf(xv[q]);
  }
  if (th < kMlpRows * DX) xt_sh[th / DX][th % DX] = tv;
  __syncthreads();
  // batch-blocked copy of a [16][32] tile: column th / 4, four rows
  auto put_t = [&](const bf16_t (*m)[kInStride], bf16_t* out) {
    if (th < kMlpIn * (kMlpRows / 4)) {
      const int c = th >> 2, r = 4 * (th & 3);
      const bf16_t h[4] = {m[r][c], m[r + 1][c], m[r + 2][c], m[r + 3][c]};
      store_rows4(out + blk_at(row0 + r, c, kMlpIn), h);
    }
  };
  put_t(sh.x0, p.x0t);
  float a1[NT][4], a2[NT][4];
  mlp_hidden<NT, kMlpIn, kInStride, true>(sh.x0, fr.w1, fr.b1, sh.h1, row0, a1, p.h1t);
  __syncthreads();
  mlp_hidden<NT, kMlpHid, kHidStride, true>(sh.h1, fr.w2, fr.b2, sh.h2, row0, a2, p.h2t);
  bf16x8 w3t[1][NT], w2t[8][NT];
  mlp_load_back<NT, kMlpOut>(p.W3t, w3t);
  mlp_load_back<NT, kMlpHid>(p.W2t, w2t);
  __syncthreads();
  mlp_out_layer(fr, sh, row0, kMlpRows, nullptr);
  __syncthreads();
  if (w == 0) mdn_grad_tile<DX>(sh.o, xt_sh, B, g_sh, gb_sh, nll_sh);
  __syncthreads();
  put_t(gb_sh, p.gt);
  if (th >= 2 * kWave && th < 2 * kWave + kMlpOut) {
    const int c = th - 2 * kWave;
    p.b3_part[(size_t)tile * kMlpOut + c] = rows16_sum<float>([&](int r) { return g_sh[r][c]; });
  }
  if (th == 3 * kWave) p.loss_part[tile] = rows16_sum<double>([&](int r) { return nll_sh[r]; });
  // (h1 is free again: every wave is past the second layer)
  mlp_back_layer<NT, kMlpOut, kInStride>(gb_sh, w3t, a2, sh.h1, p.da2t, p.b2_part + (size_t)tile * kMlpHid, row0);
  __syncthreads();
  mlp_back_layer<NT, kMlpHid, kHidStride>(sh.h1, w2t, a1, nullptr, p.da1t, p.b1_part + (size_t)tile * kMlpHid, row0);
}

// The training copies of the weights, all in fragment order: W1, W2, W3 and
// the transposed W2, W3 of the backward products.
struct MlpTrainWeights {
  bf16_t* W1;
  bf16_t* W2;
  bf16_t* W3;
  bf16_t* W2t;
  bf16_t* W3t;
};

// ---------------------------------------------------------------- Adam
// Gradient = ordered sum of the partials, Adam update of the FP32 master
// (moments m, v), BF16 / FP32 copies into the blob and the training copies.
struct AdamArgs {
  float* p;  // masters [n]
  float* m;  // [n]
  float* v;  // [n]
  float* grad_out;  // [n] or null
  unsigned char* blob;
  MlpTrainWeights tw;
  const bf16_t* At[3];  // W1, W2, W3: gradients at the layer's outputs, batch-blocked
  const bf16_t* Ht[3];  // and the layer's inputs
  const float* b1_part;   // [tiles][256]
  const float* b2_part;
  int tiles;
  const float* b3_part;     // [tiles][32]
  const double* loss_part;  // [tiles]
  float* loss;
  int B;
  float lr, bc1, bc2;  // bias corrections 1 - beta^t
  int update;          // 0: gradients only
};

constexpr float kAdamB1 = 0.9f, kAdamB2 = 0.999f, kAdamEps = 1e-8f;

// Writes parameter e of the FP32 vector into the blob and, where given, the
// training copies.
__device__ __forceinline__ void mlp_store_param(int e, float val, unsigned char* blob, const MlpTrainWeights& tw) {
  using PL = MlpParamLayout;
  using BL = MlpBlobLayout;
  if (e < PL::b1) {
    const bf16_t h = f2bf(val);
    reinterpret_cast<bf16_t*>(blob + BL::W1)[e] = h;
    if (tw.W1) tw.W1[frag_at(e / kMlpIn, e % kMlpIn, 16)] = h;
  } else if (e < PL::W2) {
    reinterpret_cast<float*>(blob + BL::b1)[e - PL::b1] = val;
  } else if (e < PL::b2) {
    const int q = e - PL::W2;
    const bf16_t h = f2bf(val);
    reinterpret_cast<bf16_t*>(blob + BL::W2)[q] = h;
    if (tw.W2) {
      tw.W2[frag_at(q / kMlpHid, q % kMlpHid, 16)] = h;
      tw.W2t[frag_at(q % kMlpHid, q / kMlpHid, 16)] = h;
    }
  } else if (e < PL::W3) {
    reinterpret_cast<float*>(blob + BL::b2)[e - PL::b2] = val;
  } else if (e < PL::b3) {
    const int q = e - PL::W3;
    const bf16_t h = f2bf(val);
    reinterpret_cast<bf16_t*>(blob + BL::W3)[q] = h;
    if (tw.W3) {
      tw.W3[frag_at(q / kMlpHid, q % kMlpHid, 2)] = h;
      tw.W3t[frag_at(q % kMlpHid, q / kMlpHid, 16)] = h;
    }
  } else {
    reinterpret_cast<float*>(blob + BL::b3)[e - PL::b3] = val;
  }
}

// Parameter e's master and moments, fetched ahead of its gradient.
struct AdamState {
  float p, m, v;
};
__device__ __forceinline__ AdamState adam_load(const AdamArgs& a, int e) {
  if (!a.update) return AdamState{};
  return AdamState{a.p[e], a.m[e], a.v[e]};
}

// Parameter e of the FP32 vector with gradient g.
__device__ __forceinline__ void adam_param(const AdamArgs& a, int e, float g, const AdamState& st) {
  if (a.grad_out) a.grad_out[e] = g;
  if (!a.update) return;
  const float m = kAdamB1 * st.m + (1.0f - kAdamB1) * g;
  const float v = kAdamB2 * st.v + (1.0f - kAdamB2) * g * g;
  a.m[e] = m;
  a.v[e] = v;
  const float mh = m / a.bc1, vh = v / a.bc2;
  const float p = st.p - a.lr * mh / (sqrtf(vh) + kAdamEps);
  a.p[e] = p;
  mlp_store_param(e, p, a.blob, a.tw);
}

// Sum of the partials of one 256-row group (16 consecutive tiles from t0,
// absent ones 0): four tiles as (0 + 1) + (2 + 3), the four results in order.
template <class T, class F>
__device__ __forceinline__ T group16_sum(int t0, int tiles, F&& part) {
  T v[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) v[k] = part(min(t0 + k, tiles - 1));
#pragma unroll
  for (int k = 0; k < 16; ++k) v[k] = t0 + k < tiles ? v[k] : T(0);
  T r[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) r[k] = (v[4 * k] + v[4 * k + 1]) + (v[4 * k + 2] + v[4 * k + 3]);
  return ((r[0] + r[1]) + r[2]) + r[3];
}

// ---------------------------------------------- weight gradients and Adam
// One launch: kWgTiles workgroups of one 16 x 16 tile of the three weight
// matrices each, dW[m][n] = sum_b A[b][m] H[b][n], then the tile's Adam update;
// kAdamB workgroups of 32 hidden biases (the batch tiles' column sums, fetched
// by all threads at once into LDS and added there in tile order); one for the
// output biases and the loss (256-row groups, then the groups in order).
//
// The batch is split into chunks of kWgChunk rows, one wave each (eight
// chunks at a time, a chunk's operands all in flight before its products),
// and the waves' FP32 tiles are added in chunk order through LDS: with the
// chunks' partial matrices in HBM and Adam a launch of its own, batch 4096
// took 13.1 + 9.8 us, 10 us now.  What is left is latency (operands come
// from the Infinity Cache, written by other XCDs) and 64 bytes per clock into
// each CU.  Each XCD takes a contiguous run of tiles, so that a row of tiles
// shares its A columns in one L2.
constexpr int kWgChunk = 512;
constexpr int kWgWaves = 8;
constexpr int kWgThreads = kWgWaves * kWave;
constexpr int kWgTiles1 = kMlpHid * kMlpIn / 256, kWgTiles2 = kMlpHid * kMlpHid / 256,
              kWgTiles3 = kMlpOut * kMlpHid / 256;
constexpr int kWgTiles = kWgTiles1 + kWgTiles2 + kWgTiles3;
constexpr int kAdamBiases = 32;
constexpr int kAdamB = 2 * kMlpHid / kAdamBiases;
constexpr int kAdamGrid = kWgTiles + kAdamB + 1;
constexpr int kAdamTiles = 256;  // batch tiles (or groups) staged at a time

__device__ __forceinline__ void wgrad_tile(const AdamArgs& a, int tile) {
  using PL = MlpParamLayout;
  __shared__ float red[kWgWaves][16][17];
  // matrix j of M x N (N / 16 tiles in a row of tiles), its first parameter
  int j = 0, M = kMlpHid, N = kMlpIn, e0 = PL::W1;
  if (tile >= kWgTiles1) {
    tile -= kWgTiles1;
    j = 1;
    N = kMlpHid;
    e0 = PL::W2;
    if (tile >= kWgTiles2) {
      tile -= kWgTiles2;
      j = 2;
      M = kMlpOut;
      e0 = PL::W3;
    }
  }
  const int m0 = 16 * (tile / (N / 16)), n0 = 16 * (tile % (N / 16));
  const int th = threadIdx.x, l = th & 63, w = th >> 6;
  const int lr = l & 15, lk = 8 * (l >> 4);
  const bf16_t* ap = a.At[j] + (m0 + lr) * kBatchBlk + lk;
  const bf16_t* hp = a.Ht[j] + (n0 + lr) * kBatchBlk + lk;
  const size_t as = M, hs = N;  // elements per batch row
  const int e = e0 + (m0 + (th >> 4)) * N + n0 + (th & 15);  // (th < 256)
  AdamState st = {};
  if (th < 256) st = adam_load(a, e);
  float g = 0.f;
  for (int c0 = 0; c0 * kWgChunk < a.B; c0 += kWgWaves) {
    const int b0 = min(a.B, (c0 + w) * kWgChunk), b1 = min(a.B, b0 + kWgChunk);
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int KS = kWgChunk / 32;
    if (b1 - b0 == kWgChunk) {
      bf16x8 av[KS], hv[KS];
#pragma unroll
      for (int q = 0; q < KS; ++q) {
        av[q] = ld8(ap + (b0 + 32 * q) * as);
        hv[q] = ld8(hp + (b0 + 32 * q) * hs);
      }
      __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the products
#pragma unroll
      for (int q = 0; q < KS; ++q) acc = mfma16(av[q], hv[q], acc);
    } else {
      for (int b = b0; b < b1; b += 32) acc = mfma16(ld8(ap + b * as), ld8(hp + b * hs), acc);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) red[w][4 * (l >> 4) + r][lr] = acc[r];
    __syncthreads();
    if (th < 256) {
      const int nc = min(kWgWaves, (a.B - c0 * kWgChunk + kWgChunk - 1) / kWgChunk);
#pragma unroll
      for (int q = 0; q < kWgWaves; ++q)
        if (q < nc) g += red[q][th >> 4][th & 15];
    }
    __syncthreads();
  }
  if (th < 256) adam_param(a, e, g, st);
}

static __global__ __launch_bounds__(kWgThreads) void k_mlp_wgrad_adam(AdamArgs a) {
  using PL = MlpParamLayout;
  const int th = threadIdx.x, blk = blockIdx.x;
  if (blk < kWgTiles) {
    wgrad_tile(a, xcd_contiguous_tile(blk, kWgTiles));
    return;
  }
  __shared__ float sm[kAdamTiles][kAdamBiases];
  __shared__ double dsm[kAdamTiles];
  const int c = th % kAdamBiases, q0 = th / kAdamBiases;
  constexpr int NQ = kWgThreads / kAdamBiases;
  if (blk < kWgTiles + kAdamB) {
    const int col = (blk - kWgTiles) * kAdamBiases;  // over b1 then b2
    const bool second = col >= kMlpHid;
    const float* bp = (second ? a.b2_part : a.b1_part) + (second ? col - kMlpHid : col) + c;
    float g = 0.f;
    for (int t0 = 0; t0 < a.tiles; t0 += kAdamTiles) {
      const int nt = min(kAdamTiles, a.tiles - t0);
      float v[kAdamTiles / NQ];
#pragma unroll
      for (int k = 0; k < kAdamTiles / NQ; ++k)
        v[k] = bp[(size_t)(t0 + min(q0 + k * NQ, nt - 1)) * kMlpHid];
#pragma unroll
      for (int k = 0; k < kAdamTiles / NQ; ++k) sm[q0 + k * NQ][c] = v[k];
      __syncthreads();
      if (th < kAdamBiases) {
#pragma unroll 16
        for (int t = 0; t < nt; ++t) g += sm[t][c];
      }
      __syncthreads();
    }
    if (th < kAdamBiases) {
      const int e = (second ? PL::b2 + col - kMlpHid : PL::b1 + col) + c;
      adam_param(a, e, g, adam_load(a, e));
    }
    return;
  }
  const int groups = (a.tiles + 15) / 16;
  float g = 0.f;
  double s = 0.0;
  for (int g0 = 0; g0 < groups; g0 += kAdamTiles) {
    const int ng = min(kAdamTiles, groups - g0);
    for (int k = q0; k < ng; k += NQ)
      sm[k][c] = group16_sum<float>(16 * (g0 + k), a.tiles,
                                    [&](int t) { return a.b3_part[(size_t)t * kMlpOut + c]; });
    if (a.loss && th < ng)
      dsm[th] = group16_sum<double>(16 * (g0 + th), a.tiles, [&](int t) { return a.loss_part[t]; });
    __syncthreads();
    if (th < kAdamBiases) {
      for (int k = 0; k < ng; ++k) g += sm[k][c];
    }
    if (a.loss && th == kWgThreads - 1) {
      for (int k = 0; k < ng; ++k) s += dsm[k];
    }
    __syncthreads();
  }
  static_assert(kMlpOut == kAdamBiases, "one output bias per lane");
  if (th < kMlpOut) adam_param(a, PL::b3 + c, g, adam_load(a, PL::b3 + c));
  if (a.loss && th == kWgThreads - 1) *a.loss = (float)(s / a.B);
}

// Masters -> blob (and the training copies when given), plus the feature
// standardisation.
static __global__ void k_mlp_pack(const float* params, const float* fmean, const float* fstd, unsigned char* blob,
                           MlpTrainWeights tw) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < MlpParamLayout::n) mlp_store_param(e, params[e], blob, tw);
  if (e < kMlpIn) {
    reinterpret_cast<float*>(blob + MlpBlobLayout::fmean)[e] = fmean[e];
    reinterpret_cast<float*>(blob + MlpBlobLayout::fstd)[e] = fstd[e];
  }
}

// A blob (in the workspace) -> a handle's: the weights in fragment order, the
// rest as it is.
static __global__ void k_mlp_to_handle(const unsigned char* src, unsigned char* dst) {
  using BL = MlpBlobLayout;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  constexpr int n1 = kMlpHid * kMlpIn, n2 = kMlpHid * kMlpHid, n3 = kMlpOut * kMlpHid;
  constexpr int nf = (int)(BL::bytes - BL::b1) / 4;
  const bf16_t* sw = reinterpret_cast<const bf16_t*>(src);
  bf16_t* dw = reinterpret_cast<bf16_t*>(dst);
  if (e < n1) dw[frag_at(e / kMlpIn, e % kMlpIn, 16)] = sw[e];
  if (e < n2) dw[n1 + frag_at(e / kMlpHid, e % kMlpHid, 16)] = sw[n1 + e];
  if (e < n3) dw[n1 + n2 + frag_at(e / kMlpHid, e % kMlpHid, 2)] = sw[n1 + n2 + e];
  if (e < nf) reinterpret_cast<uint32_t*>(dst + BL::b1)[e] = reinterpret_cast<const uint32_t*>(src + BL::b1)[e];
}

}  // namespace dpf
