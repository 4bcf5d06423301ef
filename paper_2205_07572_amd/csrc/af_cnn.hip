// af_cnn.hip -- learned regrid tagger on gfx950 (a project addition, not part
// of the paper's method).
//
// Network: three 3x3 convolutions (zero "same" padding, 16x16 inputs,
// nin -> 32 -> 32 -> 32 channels, ReLU), global average pooling, linear head
// 32 -> 3 (coarsen / keep / refine), softmax cross-entropy.  Parameters are
// FP32 masters packed as W1[co][ci][3][3], b1, W2, b2, W3, b3, Wh[3][32], bh.
//
// One block holds one 16x16 sample at a time in LDS and takes it through the
// whole network, and in training back again: the convolutions are implicit
// GEMMs on v_mfma_f32_16x16x32_bf16 (BF16 operands, FP32 accumulation) that
// read their operands from LDS; bias, ReLU, pooling, head and loss are FP32.
// Nothing but the input, the logits and one row of gradient sums per block
// crosses HBM.  A second kernel adds the blocks' rows, a third is Adam.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <string>
#include <vector>

#include "af.h"
#include "af_internal.h"

namespace af {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kImg = 16, kPix = 256, kWidth = 32, kClasses = 3;

// FP32 -> BF16, round to nearest even (NaN and Inf pass through).
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return uint16_t(u >> 16);
  u += 0x7fffu + ((u >> 16) & 1u);
  return uint16_t(u >> 16);
}

// ---------------------------------------------------------------------------
// The network on one sample at a time (k_cnn).
//
// LDS holds images channel-innermost with a zero ring, [18][18][channels]
// BF16 (the first layer's channels padded to CP, a multiple of 8), and the
// weights as [co][tap * channels + ci] with a row pitch of an odd number of
// 16-byte units.  A wave takes two image rows: a 16x16 tile's A rows are the
// 16 pixels of an image row, its B rows 16 output channels, and a lane's 8
// k values are 8 channels of one pixel of one tap, one 16-byte LDS load.
// The k steps run in ascending order of (tap, channel).
//
// Training goes on in the same block.  For layer l it needs the upstream
// gradient G = dA relu'(z) (the signs of z stay in registers), twice: G
// channel-innermost for the input gradient, where the products of a tap are
// one k step of 32 output channels, and G^T [co][pixel] for the weight
// gradient, whose k runs over pixels.  The weight gradient's other operand is
// the layer's input as [ci][18 rows][pitch 24], so that 8 pixels of a row are
// one 16-byte load; a tap's shift by one column is an alignment of that load
// with the dword beside it.  G overwrites the layer's input image once its
// transpose is made.  Weight gradients stay in registers over all samples of
// a block (5 accumulator tiles a layer and wave) and leave as one row of
// sums per block.
//
// What bounds it: the chain of k loops, epilogues and barriers of one sample
// per CU (a product of the largest layer is 9 MFMA steps); 11 MFLOP of a
// sample's forward pass are about 1 us of a CU's BF16 rate.  Measured: a
// training step of 256 samples (with Adam) 53.6 us, the tagging of 1792
// leaves 83 us in this kernel.  Before, with im2col matrices, GEMMs and
// elementwise kernels in HBM: 6424 us (5556 of them in a one-block sum of
// 8192 bias rows, 545 in the GEMMs) and 290 us.
// ---------------------------------------------------------------------------
constexpr int kCnnThreads = 512, kCnnWaves = kCnnThreads / 64;
static_assert(kCnnWaves * 2 == kImg, "a wave takes two image rows");
constexpr int kRing = kImg + 2, kRingPix = kRing * kRing;
constexpr int kTapsW = 9 * kWidth;            // k extent of layers 2 and 3
constexpr int kPitchW = kTapsW + 8;           // their weight rows (592 bytes)
constexpr int kPitchWt = kWidth + 8;          // rows of W^T [tap * 32 + ci][co] (80 bytes)
constexpr int kPitchG = kPix + 8;             // rows of G^T (528 bytes)
constexpr int kXtRow = 24, kPitchXt = kRing * kXtRow + 8;  // transposed input: pixel x at column x + 8 (880 bytes)
constexpr int kPitchA3 = kWidth + 1;
constexpr int kCnnRows = 256;                 // blocks of a launch: one per CU
// a block's row of gradient sums: [layer][tap][co][ci], biases [layer][co],
// then loss, Wh [3][32], bh [3]
constexpr int kPartW = 9 * kWidth * kWidth, kPartB = 3 * kPartW, kPartH = kPartB + 3 * kWidth;
constexpr int kPartN = kPartH + 1 + kClasses * kWidth + kClasses;
constexpr int kPart = (kPartN + 63) / 64 * 64;

struct CnnOffsets {
  int w[3], b[3], wh, bh;
};

struct CnnArgs {
  const float* params;   // packed FP32 parameters
  CnnOffsets off;
  const float* x;        // [B][nin][16][16]
  int nin, B;
  float* logits;         // [B][3] or null
  const int32_t* labels; // training
  float* acts;           // null or [3][B*256][32]: pre-activations
  float* dacts;          // null or [3][B*256][32]: gradients of the post-ReLU outputs
  float* part;           // training: [gridDim.x][kPart]
};

template <int CP, bool TRAIN>
struct CnnLds {
  static constexpr int STEPS1 = (9 * CP + 31) / 32;
  static constexpr int PITCH1 = STEPS1 * 32 + 8;  // 16 bytes times an odd number, as kPitchW
  static constexpr int WFWD = kWidth * PITCH1 + 2 * kWidth * kPitchW;
  static_assert(!TRAIN || (WFWD >= kTapsW * kPitchWt + kWidth * kPitchG && WFWD >= 2 * kPix * kPitchA3),
                "the backward operands and the last layer fit the forward weights' place");
  alignas(16) uint16_t w[WFWD];
  alignas(16) uint16_t x0[kRingPix * CP];
  alignas(16) uint16_t a1[kRingPix * kWidth];
  alignas(16) uint16_t a2[kRingPix * kWidth];
  alignas(16) uint16_t xt[TRAIN ? kWidth * kPitchXt : 8];
  float a3[TRAIN ? 4 : kPix * kPitchA3];  // training: in the weights' place
  float bias[3][kWidth], wh[kClasses * kWidth], bh[4], pooled[kWidth], lg[4], red[kCnnWaves][kWidth];
};

// acc += the convolution of image rows 2 wave, 2 wave + 1 (C channels).
template <int C>
__device__ __forceinline__ void cnn_conv(const uint16_t* img, const uint16_t* w, int wave, int lane,
                                         f32x4 (&acc)[2][2]) {
  constexpr int K = 9 * C, STEPS = (K + 31) / 32, PITCH = STEPS * 32 + 8;
  const int g = lane >> 4, c = lane & 15;
  const u16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll 3
  for (int s = 0; s < STEPS; ++s) {
    const int ks = s * 32 + 8 * g;
    const bool valid = STEPS * 32 == K || ks < K;  // past K the weights are zero, the image must not be NaN
    const int tap = valid ? ks / C : 0, ci = valid ? ks - tap * C : 0;
    const int ty = tap / 3, tx = tap - 3 * ty;
    bf16x8 a[2], b[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const u16x8 v = *reinterpret_cast<const u16x8*>(img + ((2 * wave + t + ty) * kRing + c + tx) * C + ci);
      a[t] = __builtin_bit_cast(bf16x8, valid ? v : zero8);
      b[t] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(w + (t * 16 + c) * PITCH + ks));
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int n = 0; n < 2; ++n) acc[t][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t], b[n], acc[t][n], 0, 0, 0);
  }
}

// Weight gradient tiles of one layer: acc[k] (+)= G^T X of tap T0 + k for
// output channels 16 coh .. and input channels 16 cih .., over the sample's
// pixels (8 k steps of two image rows).
template <int T0, int NTAP>
__device__ __forceinline__ void cnn_wgrad(const uint16_t* gt, const uint16_t* xt, int coh, int cih, int lane,
                                          f32x4 (&acc)[5]) {
  const int g = lane >> 4, c = lane & 15;
  const uint16_t* const ga = gt + (coh * 16 + c) * kPitchG + 8 * g;
  const uint16_t* const xa = xt + (cih * 16 + c) * kPitchXt + (g >> 1) * kXtRow + 8 + 8 * (g & 1);
#pragma unroll 1
  for (int s = 0; s < kImg / 2; ++s) {
    const bf16x8 a = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(ga + 32 * s));
#pragma unroll
    for (int ty = T0 / 3; ty <= (T0 + NTAP - 1) / 3; ++ty) {
      const uint16_t* const p = xa + (2 * s + ty) * kXtRow;
      const u32x4 d = *reinterpret_cast<const u32x4*>(p);
      const unsigned lo = *reinterpret_cast<const unsigned*>(p - 2), hi = *reinterpret_cast<const unsigned*>(p + 8);
#pragma unroll
      for (int tx = 0; tx < 3; ++tx) {
        const int k = 3 * ty + tx - T0;
        if (k < 0 || k >= NTAP) continue;
        u32x4 v = d;
        if (tx == 0) {
          v[0] = __builtin_amdgcn_alignbit(d[0], lo, 16);
          v[1] = __builtin_amdgcn_alignbit(d[1], d[0], 16);
          v[2] = __builtin_amdgcn_alignbit(d[2], d[1], 16);
          v[3] = __builtin_amdgcn_alignbit(d[3], d[2], 16);
        } else if (tx == 2) {
          v[0] = __builtin_amdgcn_alignbit(d[1], d[0], 16);
          v[1] = __builtin_amdgcn_alignbit(d[2], d[1], 16);
          v[2] = __builtin_amdgcn_alignbit(d[3], d[2], 16);
          v[3] = __builtin_amdgcn_alignbit(hi, d[3], 16);
        }
        acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, v), acc[k], 0, 0, 0);
      }
    }
  }
}

// out = the input gradient of image rows 2 wave, 2 wave + 1: each tap's
// product over the 32 output channels, added in ascending order of the taps.
__device__ __forceinline__ void cnn_dgrad(const uint16_t* gi, const uint16_t* wt, int wave, int lane,
                                          f32x4 (&out)[2][2]) {
  const int g = lane >> 4, c = lane & 15;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int n = 0; n < 2; ++n) out[t][n] = zero;
#pragma unroll 3
  for (int tap = 0; tap < 9; ++tap) {
    const int ty = tap / 3, tx = tap - 3 * ty;
    bf16x8 a[2], b[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      a[t] = __builtin_bit_cast(
          bf16x8, *reinterpret_cast<const u16x8*>(gi + ((2 * wave + t + 2 - ty) * kRing + c + 2 - tx) * kWidth + 8 * g));
      b[t] = __builtin_bit_cast(bf16x8,
                                *reinterpret_cast<const u16x8*>(wt + (tap * kWidth + t * 16 + c) * kPitchWt + 8 * g));
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int n = 0; n < 2; ++n)
        out[t][n] += __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t], b[n], zero, 0, 0, 0);
  }
}

// Transposed copy of an image of C channels, [ci][row][x + 8]; its ring
// columns and rows stay zero.
template <int C>
__device__ __forceinline__ void cnn_transpose(const uint16_t* img, uint16_t* xt, int tid) {
#pragma unroll 1
  for (int e = tid; e < kPix * (C / 8); e += kCnnThreads) {
    const int p = e & (kPix - 1), c0 = (e / kPix) * 8;
    const int y = p / kImg, x = p % kImg;
    const u16x8 v = *reinterpret_cast<const u16x8*>(img + ((y + 1) * kRing + x + 1) * C + c0);
#pragma unroll
    for (int k = 0; k < 8; ++k) xt[(c0 + k) * kPitchXt + (y + 1) * kXtRow + x + 8] = v[k];
  }
}

// BF16 weights of a layer with cin input channels, [co][tap * C + ci] with
// the given row pitch.
template <int C>
__device__ __forceinline__ void cnn_weights(const float* W, int cin, int pitch, uint16_t* w, int tid) {
#pragma unroll 6
  for (int e = tid; e < kWidth * cin * 9; e += kCnnThreads) {
    const int co = e / (cin * 9), r = e - co * cin * 9, ci = r / 9, tap = r - ci * 9;
    w[co * pitch + tap * C + ci] = f2bf(W[e]);
  }
}

// W^T [tap * 32 + ci][co] of a layer with 32 input channels.
__device__ __forceinline__ void cnn_weights_t(const float* W, uint16_t* wt, int tid) {
#pragma unroll 6
  for (int e = tid; e < kWidth * kTapsW; e += kCnnThreads) {
    const int co = e / kTapsW, r = e - co * kTapsW, ci = r / 9, tap = r - ci * 9;
    wt[(tap * kWidth + ci) * kPitchWt + co] = f2bf(W[e]);
  }
}

template <int CP, bool TRAIN>
__global__ __launch_bounds__(kCnnThreads) void k_cnn(const CnnArgs A) {
  using L_t = CnnLds<CP, TRAIN>;
  __shared__ L_t S;
  const int tid0 = threadIdx.x;
  uint16_t* const w1 = S.w;
  uint16_t* const w2 = w1 + kWidth * L_t::PITCH1;
  uint16_t* const w3 = w2 + kWidth * kPitchW;
  float* const a3 = TRAIN ? reinterpret_cast<float*>(S.w) : S.a3;
  uint16_t* const wt = S.w;                       // training, backward
  uint16_t* const gt = S.w + kTapsW * kPitchWt;

  auto zero = [&](uint16_t* p, int n) {  // n even
#pragma unroll 1
    for (int e = tid0; e < n / 2; e += kCnnThreads) reinterpret_cast<unsigned*>(p)[e] = 0;
  };
  auto weights = [&](int tid) {  // w1's padding (channels past nin, k past 9 CP) must be zero
    cnn_weights<CP>(A.params + A.off.w[0], A.nin, L_t::PITCH1, w1, tid);
    cnn_weights<kWidth>(A.params + A.off.w[1], kWidth, kPitchW, w2, tid);
    cnn_weights<kWidth>(A.params + A.off.w[2], kWidth, kPitchW, w3, tid);
  };
  zero(S.x0, kRingPix * CP);
  zero(S.a1, kRingPix * kWidth);
  zero(S.a2, kRingPix * kWidth);
  if (TRAIN) zero(S.xt, kWidth * kPitchXt);
  if (tid0 < 3 * kWidth) S.bias[tid0 / kWidth][tid0 % kWidth] = A.params[A.off.b[tid0 / kWidth] + tid0 % kWidth];
  if (tid0 < kClasses * kWidth) S.wh[tid0] = A.params[A.off.wh + tid0];
  if (tid0 < kClasses) S.bh[tid0] = A.params[A.off.bh + tid0];
  if (!TRAIN) {
    zero(w1, kWidth * L_t::PITCH1);
    __syncthreads();
    weights(tid0);
  }

  f32x4 gw[3][5];  // weight gradients, TRAIN
  float gb[3][2] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
  float gh[kClasses] = {0.f, 0.f, 0.f}, gbh = 0.f, gloss = 0.f;
  if (TRAIN)
#pragma unroll
    for (int l = 0; l < 3; ++l)
#pragma unroll
      for (int k = 0; k < 5; ++k) gw[l][k] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int b = blockIdx.x; b < A.B; b += gridDim.x) {
    // opaque to the compiler, so that the addresses made from it are not all
    // kept in registers across the sample loop (they spilled)
    int tid = tid0;
    asm volatile("" : "+v"(tid));
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int g = lane >> 4, c = lane & 15;
    const int coh = wave & 1, cih = (wave >> 1) & 1;
    if (TRAIN) {  // the last sample's backward pass used the weights' place
      __syncthreads();
      zero(w1, kWidth * L_t::PITCH1);
    }
    __syncthreads();
    if (TRAIN) weights(tid);
    for (int e = tid; e < kPix * (CP / 8); e += kCnnThreads) {
      const int p = e & (kPix - 1), c0 = (e / kPix) * 8;
      u16x8 v;
#pragma unroll
      for (int k = 0; k < 8; ++k)
        v[k] = c0 + k < A.nin ? f2bf(A.x[(size_t(b) * A.nin + c0 + k) * kPix + p]) : uint16_t(0);
      *reinterpret_cast<u16x8*>(S.x0 + ((p / kImg + 1) * kRing + p % kImg + 1) * CP + c0) = v;
    }
    __syncthreads();

    // ---- forward.  zpos[l]: bit t * 8 + n * 4 + r set where the lane's z > 0
    unsigned zpos[3];
    auto layer = [&](int l, f32x4 (&acc)[2][2], uint16_t* out) {
      unsigned m = 0;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int y = 2 * wave + t, x = 4 * g + r, ch = n * 16 + c;
            const float z = acc[t][n][r] + S.bias[l][ch];
            const bool pos = z > 0.f;
            acc[t][n][r] = pos ? z : 0.f;
            if (pos) m |= 1u << (t * 8 + n * 4 + r);
            if (out) out[((y + 1) * kRing + x + 1) * kWidth + ch] = f2bf(acc[t][n][r]);
            if (A.acts) A.acts[((size_t(l) * A.B + b) * kPix + y * kImg + x) * kWidth + ch] = z;
          }
      zpos[l] = m;
    };
    f32x4 acc[2][2];
    auto clear = [&]() {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    clear();
    cnn_conv<CP>(S.x0, w1, wave, lane, acc);
    layer(0, acc, S.a1);
    __syncthreads();
    clear();
    cnn_conv<kWidth>(S.a1, w2, wave, lane, acc);
    layer(1, acc, S.a2);
    __syncthreads();
    clear();
    cnn_conv<kWidth>(S.a2, w3, wave, lane, acc);
    layer(2, acc, nullptr);
    if (TRAIN) __syncthreads();  // a3 takes the weights' place
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          a3[((2 * wave + t) * kImg + 4 * g + r) * kPitchA3 + n * 16 + c] = acc[t][n][r];
    __syncthreads();

    // ---- head: the pooled mean adds the pixels in order
    if (tid < kWidth) {
      float s = 0.f;
#pragma unroll 16
      for (int p = 0; p < kPix; ++p) s += a3[p * kPitchA3 + tid];
      S.pooled[tid] = s * (1.0f / kPix);
    }
    __syncthreads();
    if (tid < kClasses) {
      float s = S.bh[tid];
      for (int k = 0; k < kWidth; ++k) s += S.wh[tid * kWidth + k] * S.pooled[k];
      S.lg[tid] = s;
      if (A.logits) A.logits[size_t(b) * kClasses + tid] = s;
    }
    if (!TRAIN) continue;  // pooled is written again several barriers later
    __syncthreads();
    // softmax cross-entropy: every thread forms dl, then dA of the pooling
    // for its two channels
    const int lab = min(max(int(A.labels[b]), 0), kClasses - 1);
    const float mx = fmaxf(S.lg[0], fmaxf(S.lg[1], S.lg[2]));
    float den = 0.f;
    for (int k = 0; k < kClasses; ++k) den += expf(S.lg[k] - mx);
    float dl[kClasses];
    for (int k = 0; k < kClasses; ++k) dl[k] = (expf(S.lg[k] - mx) / den - (k == lab ? 1.f : 0.f)) / A.B;
    if (tid == 0) gloss += -(S.lg[lab] - mx - logf(den)) / A.B;
    if (tid < kWidth)
      for (int k = 0; k < kClasses; ++k) gh[k] += dl[k] * S.pooled[tid];
    if (tid < kClasses) gbh += dl[tid];
    f32x4 dA[2][2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      float dp = 0.f;
      for (int k = 0; k < kClasses; ++k) dp += dl[k] * S.wh[k * kWidth + n * 16 + c];
      dp *= 1.0f / kPix;
#pragma unroll
      for (int t = 0; t < 2; ++t) dA[t][n] = f32x4{dp, dp, dp, dp};
    }

    // ---- backward.  put: G = dA relu'(z) of layer l into G^T and, where
    // gi is given, channel-innermost
    auto put = [&](int l, uint16_t* gi) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          const int y = 2 * wave + t, ch = n * 16 + c;
          u16x4 h;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float v = (zpos[l] >> (t * 8 + n * 4 + r)) & 1u ? dA[t][n][r] : 0.f;
            h[r] = f2bf(v);
            gb[l][n] += v;
            if (gi) gi[((y + 1) * kRing + 4 * g + r + 1) * kWidth + ch] = h[r];
            if (A.dacts)
              A.dacts[((size_t(l) * A.B + b) * kPix + y * kImg + 4 * g + r) * kWidth + ch] = dA[t][n][r];
          }
          *reinterpret_cast<u16x4*>(gt + ch * kPitchG + y * kImg + 4 * g) = h;
        }
    };
    auto wgrad = [&](f32x4 (&acc)[5]) {
      if (wave < kCnnWaves / 2)
        cnn_wgrad<0, 5>(gt, S.xt, coh, cih, lane, acc);
      else
        cnn_wgrad<5, 4>(gt, S.xt, coh, cih, lane, acc);
    };
    __syncthreads();  // a3 has been read
#pragma unroll
    for (int l = 2; l >= 1; --l) {
      uint16_t* const in = l == 2 ? S.a2 : S.a1;
      cnn_weights_t(A.params + A.off.w[l], wt, tid);
      cnn_transpose<kWidth>(in, S.xt, tid);
      __syncthreads();
      put(l, in);
      __syncthreads();
      wgrad(gw[l]);
      cnn_dgrad(in, wt, wave, lane, dA);
      __syncthreads();
    }
    cnn_transpose<CP>(S.x0, S.xt, tid);
    put(0, nullptr);
    __syncthreads();
    if (16 * cih < CP) wgrad(gw[0]);
  }

  if (!TRAIN) return;
  // ---- the block's row of sums
  const int tid = tid0, wave = tid >> 6, lane = tid & 63;
  const int g = lane >> 4, c = lane & 15;
  const int coh = wave & 1, cih = (wave >> 1) & 1;
  float* const P = A.part + size_t(blockIdx.x) * kPart;
  const int tap0 = wave < kCnnWaves / 2 ? 0 : 5, ntap = wave < kCnnWaves / 2 ? 5 : 4;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
#pragma unroll
    for (int k = 0; k < 5; ++k)
      if (k < ntap)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          P[l * kPartW + ((tap0 + k) * kWidth + coh * 16 + 4 * g + r) * kWidth + cih * 16 + c] = gw[l][k][r];
    // bias: over the wave's pixels, then the waves in order
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      float v = gb[l][n];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (g == 0) S.red[wave][n * 16 + c] = v;
    }
    __syncthreads();
    if (tid < kWidth) {
      float s = 0.f;
      for (int k = 0; k < kCnnWaves; ++k) s += S.red[k][tid];
      P[kPartB + l * kWidth + tid] = s;
    }
    __syncthreads();
  }
  if (tid == 0) P[kPartH] = gloss;
  if (tid < kWidth)
    for (int k = 0; k < kClasses; ++k) P[kPartH + 1 + k * kWidth + tid] = gh[k];
  if (tid < kClasses) P[kPartH + 1 + kClasses * kWidth + tid] = gbh;
}

// grad (packed order) and loss: the blocks' rows added in a fixed order, four
// runs of rows side by side and then their sums.
__global__ __launch_bounds__(256) void k_cnn_grad(const float* part, int rows, CnnOffsets off, int nin, float* grad,
                                                  float* loss) {
  __shared__ float red[4][64];
  const int e = blockIdx.x * 64 + (threadIdx.x & 63), q = threadIdx.x >> 6;
  const int per = (rows + 3) / 4, r1 = min(rows, (q + 1) * per);
  float s = 0.f;
#pragma unroll 8
  for (int r = q * per; r < r1; ++r) s += part[size_t(r) * kPart + e];
  red[q][threadIdx.x & 63] = s;
  __syncthreads();
  if (q != 0 || e >= kPartN) return;
  s = (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
  if (e < kPartB) {
    const int l = e / kPartW, f = e - l * kPartW;
    const int tap = f / (kWidth * kWidth), co = f / kWidth % kWidth, ci = f % kWidth;
    const int cin = l == 0 ? nin : kWidth;
    if (ci < cin) grad[off.w[l] + (co * cin + ci) * 9 + tap] = s;
  } else if (e < kPartH) {
    grad[off.b[(e - kPartB) / kWidth] + (e - kPartB) % kWidth] = s;
  } else if (e == kPartH) {
    *loss = s;
  } else if (e <= kPartH + kClasses * kWidth) {
    grad[off.wh + e - kPartH - 1] = s;
  } else {
    grad[off.bh + e - kPartH - 1 - kClasses * kWidth] = s;
  }
}

template <bool TRAIN>
static hipError_t launch_cnn(int cp, const CnnArgs& A, int blocks, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>(blocks)), thr(kCnnThreads);
  switch (cp) {
    case 8: hipLaunchKernelGGL((k_cnn<8, TRAIN>), grid, thr, 0, st, A); break;
    case 16: hipLaunchKernelGGL((k_cnn<16, TRAIN>), grid, thr, 0, st, A); break;
    case 24: hipLaunchKernelGGL((k_cnn<24, TRAIN>), grid, thr, 0, st, A); break;
    case 32: hipLaunchKernelGGL((k_cnn<32, TRAIN>), grid, thr, 0, st, A); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

__global__ void k_adam(float* p, float* m1, float* m2, const float* g, int n, float lr, float b1, float b2, float eps,
                       float c1, float c2) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
    const float gi = g[e];
    const float a = b1 * m1[e] + (1.f - b1) * gi;
    const float v = b2 * m2[e] + (1.f - b2) * gi * gi;
    m1[e] = a;
    m2[e] = v;
    p[e] -= lr * (a / c1) / (sqrtf(v / c2) + eps);
  }
}

// Features of leaves (m = 16): 12 channels (p,u,v) x (avg, corner, xedge,
// yedge) of the owned DOFs of every interior cell, and one channel with the
// leaf level; each standardised with (x - mean[c]) * inv_std[c].
template <typename T>
struct DofPtrs {
  const T* p[2][4];
};

// One block per leaf, one thread per cell: the leaf's level and the channel's
// plane are uniform and four channels are in flight (one thread per element,
// with three 64-bit divisions each, on 1792 leaves: 18 us, now
// 11).
template <typename T>
__global__ __launch_bounds__(kPix) void k_features(const DofPtrs<T> D, uint32_t mask, int npatch, int pitch, int ncomp,
                                                   const int32_t* plevel, int first, const float* mean,
                                                   const float* inv_std, int nin, float* x) {
  constexpr int U = 4;
  const int leaf = first + int(blockIdx.x), l = plevel[leaf];
  const int p = threadIdx.x, i = p % kImg, j = p / kImg;
  float* const out = x + size_t(blockIdx.x) * nin * kPix + p;
  for (int c0 = 0; c0 < nin; c0 += U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ch = c0 + u;
      v[u] = ch >= 12 ? float(l) : 0.f;
      if (ch < nin && ch < 12 && ch / 4 < ncomp)
        v[u] = float(D.p[(mask >> l) & 1][ch % 4][((size_t(ch / 4) * npatch + leaf) * (kImg + 5) + (j + kGhost)) * pitch +
                                                  (i + kGhost)]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ch = c0 + u;
      if (ch < nin) out[size_t(ch) * kPix] = (v[u] - mean[ch]) * inv_std[ch];
    }
  }
}

// Learned tags with the plain criterion as fallback: refine if either says
// refine; coarsen only if both say coarsen; a non-finite output uses the
// plain tag.  Level limits as for the plain tagger.
__global__ void k_combine_tags(const float* logits, const int8_t* plain, const int32_t* plevel, int first, int n,
                               int lmax, int8_t* out, int8_t* learned) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= n) return;
  const float* L = logits + b * kClasses;
  const int leaf = first + b;
  const int8_t pt = plain[leaf];
  int8_t t;
  if (!isfinite(L[0]) || !isfinite(L[1]) || !isfinite(L[2])) {
    t = pt;
    if (learned) learned[leaf] = 2;  // marks a fallback
  } else {
    const int cls = (L[2] > L[1] && L[2] > L[0]) ? 2 : (L[0] > L[1] ? 0 : 1);
    const int8_t lt = int8_t(cls - 1);
    if (learned) learned[leaf] = lt;
    if (lt == 1 || pt == 1) t = 1;
    else if (lt == -1 && pt == -1) t = -1;
    else t = 0;
  }
  const int l = plevel[leaf];
  if (t == 1 && l >= lmax) t = 0;
  if (t == -1 && l == 0) t = 0;
  out[leaf] = t;
}

}  // namespace af

// ===========================================================================
// Host side
// ===========================================================================
using namespace af;

struct af_cnn {
  int nin, cp1, nparams;
  CnnOffsets off;
  float* d_params = nullptr;  // FP32 masters
  float* d_m1 = nullptr;
  float* d_m2 = nullptr;
  float* d_grad = nullptr;
  // workspace for up to cap samples, one block: inputs and logits of af_cnn_tag,
  // and the rows of gradient sums of af_cnn_loss_grad's blocks
  int cap = 0;
  float* d_feat = nullptr;
  float* d_logits = nullptr;
  float* d_part = nullptr;
  float* d_norm = nullptr;  // mean[nin], inv_std[nin]
};

namespace {
thread_local std::string g_cnn_err;
af_status cfail(af_status s, const std::string& m) {
  g_cnn_err = m;
  return s;
}
#define CNN_HIP(call)                                                                                   \
  do {                                                                                                  \
    hipError_t e_ = (call);                                                                             \
    if (e_ != hipSuccess) return cfail(AF_ERR_DEVICE, std::string(#call ": ") + hipGetErrorString(e_)); \
  } while (0)

int grid_for(long n) { return int(std::min<long>((n + 255) / 256, 8192)); }

// The workspace of every entry point for n samples: after one call of any of
// them the others allocate nothing up to that size (and can be captured).
af_status ensure_batch(af_cnn* c, int n) {
  if (n <= c->cap) return AF_OK;
  (void)hipFree(c->d_feat);
  c->d_feat = c->d_logits = c->d_part = nullptr;
  c->cap = 0;
  const size_t feat = size_t(n) * c->nin * kPix, part = size_t(std::min(n, kCnnRows)) * kPart;
  CNN_HIP(hipMalloc(&c->d_feat, (feat + part + size_t(n) * kClasses) * 4));
  c->d_part = c->d_feat + feat;
  c->d_logits = c->d_part + part;
  c->cap = n;
  return AF_OK;
}

CnnArgs cnn_args(const af_cnn* c, const float* x, int B) {
  CnnArgs A{};
  A.params = c->d_params;
  A.off = c->off;
  A.x = x;
  A.nin = c->nin;
  A.B = B;
  return A;
}

}  // namespace

extern "C" {

const char* af_cnn_last_error(void) { return g_cnn_err.c_str(); }

af_status af_cnn_create(int32_t nin, af_cnn** out) {
  if (!out || nin < 1 || nin > 32) return cfail(AF_ERR_ARG, "nin must be in [1, 32]");
  auto c = std::make_unique<af_cnn>();
  c->nin = nin;
  c->cp1 = (nin + 7) / 8 * 8;
  int o = 0;
  for (int l = 0; l < 3; ++l) {
    const int cin = l == 0 ? nin : kWidth;
    c->off.w[l] = o;
    o += kWidth * cin * 9;
    c->off.b[l] = o;
    o += kWidth;
  }
  c->off.wh = o;
  o += kClasses * kWidth;
  c->off.bh = o;
  o += kClasses;
  c->nparams = o;
  CNN_HIP(hipMalloc(&c->d_params, size_t(o) * 4));
  CNN_HIP(hipMalloc(&c->d_m1, size_t(o) * 4));
  CNN_HIP(hipMalloc(&c->d_m2, size_t(o) * 4));
  CNN_HIP(hipMalloc(&c->d_grad, size_t(o) * 4));
  CNN_HIP(hipMemset(c->d_params, 0, size_t(o) * 4));
  CNN_HIP(hipMemset(c->d_m1, 0, size_t(o) * 4));
  CNN_HIP(hipMemset(c->d_m2, 0, size_t(o) * 4));
  CNN_HIP(hipMalloc(&c->d_norm, size_t(2) * nin * 4));
  std::vector<float> norm(2 * nin, 0.f);
  for (int i = 0; i < nin; ++i) norm[nin + i] = 1.f;
  CNN_HIP(hipMemcpy(c->d_norm, norm.data(), norm.size() * 4, hipMemcpyHostToDevice));
  *out = c.release();
  return AF_OK;
}

af_status af_cnn_destroy(af_cnn* c) {
  if (!c) return AF_OK;
  (void)hipFree(c->d_params);
  (void)hipFree(c->d_m1);
  (void)hipFree(c->d_m2);
  (void)hipFree(c->d_grad);
  (void)hipFree(c->d_feat);
  (void)hipFree(c->d_norm);
  delete c;
  return AF_OK;
}

int32_t af_cnn_num_params(const af_cnn* c) { return c ? c->nparams : -1; }

af_status af_cnn_set_params(af_cnn* c, const float* host) {
  if (!c || !host) return cfail(AF_ERR_ARG, "null argument");
  CNN_HIP(hipMemcpy(c->d_params, host, size_t(c->nparams) * 4, hipMemcpyHostToDevice));
  CNN_HIP(hipMemset(c->d_m1, 0, size_t(c->nparams) * 4));
  CNN_HIP(hipMemset(c->d_m2, 0, size_t(c->nparams) * 4));
  return AF_OK;
}

af_status af_cnn_get_params(const af_cnn* c, float* host) {
  if (!c || !host) return cfail(AF_ERR_ARG, "null argument");
  CNN_HIP(hipMemcpy(host, c->d_params, size_t(c->nparams) * 4, hipMemcpyDeviceToHost));
  return AF_OK;
}

af_status af_cnn_set_normalization(af_cnn* c, const float* mean, const float* inv_std) {
  if (!c || !mean || !inv_std) return cfail(AF_ERR_ARG, "null argument");
  std::vector<float> v(mean, mean + c->nin);
  v.insert(v.end(), inv_std, inv_std + c->nin);
  CNN_HIP(hipMemcpy(c->d_norm, v.data(), v.size() * 4, hipMemcpyHostToDevice));
  return AF_OK;
}

af_status af_cnn_forward(af_cnn* c, const float* x, int32_t B, float* logits, float* acts, hipStream_t st) {
  if (!c || !x || !logits || B <= 0) return cfail(AF_ERR_ARG, "bad argument");
  af_status s = ensure_batch(c, B);
  if (s != AF_OK) return s;
  CnnArgs A = cnn_args(c, x, B);
  A.logits = logits;
  A.acts = acts;
  CNN_HIP(launch_cnn<false>(c->cp1, A, std::min(B, kCnnRows), st));
  return AF_OK;
}

af_status af_cnn_loss_grad(af_cnn* c, const float* x, const int32_t* labels, int32_t B, float* loss, float* grad,
                           float* dacts, hipStream_t st) {
  if (!c || !x || !labels || !loss || B <= 0) return cfail(AF_ERR_ARG, "bad argument");
  af_status s = ensure_batch(c, B);
  if (s != AF_OK) return s;
  const int rows = std::min(B, kCnnRows);
  CnnArgs A = cnn_args(c, x, B);
  A.labels = labels;
  A.dacts = dacts;
  A.part = c->d_part;
  CNN_HIP(launch_cnn<true>(c->cp1, A, rows, st));
  // every entry of the gradient and the loss is written (no accumulation across calls)
  hipLaunchKernelGGL(k_cnn_grad, dim3(kPart / 64), dim3(256), 0, st, c->d_part, rows, c->off, c->nin,
                     grad ? grad : c->d_grad, loss);
  CNN_HIP(hipGetLastError());
  return AF_OK;
}

af_status af_cnn_adam_step(af_cnn* c, const float* grad, float lr, int32_t t, hipStream_t st) {
  if (!c || t < 1) return cfail(AF_ERR_ARG, "bad argument");
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - std::pow(b1, float(t)), c2 = 1.f - std::pow(b2, float(t));
  hipLaunchKernelGGL(k_adam, dim3(grid_for(c->nparams)), dim3(256), 0, st, c->d_params, c->d_m1, c->d_m2,
                     grad ? grad : c->d_grad, c->nparams, lr, b1, b2, 1e-8f, c1, c2);
  CNN_HIP(hipGetLastError());
  return AF_OK;
}

}  // extern "C"

// Feature extraction and learned tagging need the AF context and hierarchy;
// they are implemented with the accessors below (defined in af_api.cpp).
struct AfTagView {
  bool fp32;
  int ncomp, m, npatch, pitch, lmax, nleaves;
  const void* dof0[4];
  const void* dof1[4];
  const int32_t* plevel;
};
extern "C" af_status af_internal_tag_view(const af_ctx* ctx, const af_hier* h, const af_state* bufs, AfTagView* v);

namespace {
// One block per leaf, at most 2^23 a launch: a grid is limited to 2^32
// threads (beyond it the count wraps without an error).
template <typename T>
void launch_features(const AfTagView& v, uint32_t mask, const float* norm, int nin, float* x, hipStream_t st) {
  DofPtrs<T> D;
  for (int k = 0; k < 4; ++k) {
    D.p[0][k] = static_cast<const T*>(v.dof0[k]);
    D.p[1][k] = static_cast<const T*>(v.dof1[k]);
  }
  constexpr int kLeaves = 1 << 23;
  for (int first = 0; first < v.nleaves; first += kLeaves)
    hipLaunchKernelGGL(k_features<T>, dim3(unsigned(std::min(v.nleaves - first, kLeaves))), dim3(kPix), 0, st, D, mask,
                       v.npatch, v.pitch, v.ncomp, v.plevel, first, norm, norm + nin, nin,
                       x + size_t(first) * nin * kPix);
}
}  // namespace

extern "C" {

af_status af_cnn_features(af_ctx* ctx, af_cnn* c, const af_hier* h, const af_state* bufs, uint32_t mask,
                          float* x, hipStream_t st) {
  if (!ctx || !c || !h || !x) return cfail(AF_ERR_ARG, "null argument");
  AfTagView v;
  af_status s = af_internal_tag_view(ctx, h, bufs, &v);
  if (s != AF_OK) return cfail(s, "af_cnn_features: bad context, hierarchy or buffers");
  if (v.m != kImg) return cfail(AF_ERR_ARG, "af_cnn_features: the tagger takes 16x16 patches");
  if (v.nleaves <= 0) return AF_OK;
  if (v.fp32) launch_features<float>(v, mask, c->d_norm, c->nin, x, st);
  else launch_features<double>(v, mask, c->d_norm, c->nin, x, st);
  CNN_HIP(hipGetLastError());
  return AF_OK;
}

af_status af_cnn_tag(af_ctx* ctx, af_cnn* c, const af_hier* h, const af_state* bufs, uint32_t mask,
                     const int8_t* plain, int8_t* tags, int8_t* learned, hipStream_t st) {
  if (!ctx || !c || !h || !plain || !tags) return cfail(AF_ERR_ARG, "null argument");
  AfTagView v;
  af_status s = af_internal_tag_view(ctx, h, bufs, &v);
  if (s != AF_OK) return cfail(s, "af_cnn_tag: bad context, hierarchy or buffers");
  if ((s = ensure_batch(c, v.nleaves)) != AF_OK) return s;
  if ((s = af_cnn_features(ctx, c, h, bufs, mask, c->d_feat, st)) != AF_OK) return s;
  if ((s = af_cnn_forward(c, c->d_feat, v.nleaves, c->d_logits, nullptr, st)) != AF_OK) return s;
  hipLaunchKernelGGL(k_combine_tags, dim3((v.nleaves + 255) / 256), dim3(256), 0, st, c->d_logits, plain, v.plevel,
                     0, v.nleaves, v.lmax, tags, learned);
  CNN_HIP(hipGetLastError());
  return AF_OK;
}

}  // extern "C"
