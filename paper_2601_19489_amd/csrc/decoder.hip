// Anchor (neural-Gaussian) decoder of Sec. 2.3 on BF16 matrix cores
// (v_mfma_f32_16x16x32_bf16), FP32 accumulation.
//
// Per anchor i and camera centre c: x = [feat_i (32), unit(c - pos_i) (3)]
// rounded to BF16. Three heads h (opacity, colour, covariance), each
// z_h = W1_h x + b1_h, h_h = bf16(max(z_h, 0)), y_h = W2_h h_h + b2_h.
// Child j of anchor i (Gaussian j A + i): opacity max(0, tanh y_op[j]),
// rgb sigmoid(y_col[3j ..]), scale scaling[3 ..] sigmoid(y_cov[7j ..]),
// quaternion y_cov[7j+3 .. 7j+6] normalised, mean pos + offsets[3j ..]
// scaling[0 ..].
//
// Backward: BF16 rounding is taken as the identity (straight-through) and
// the rounded operands of the forward are reused. The gradient operand of
// every backward product (dL/dy, dL/dz, FP32) enters the BF16 matrix core
// as two terms hi + lo with hi = bf16(v), lo = bf16(v - hi), which keeps
// about 16 bits of it.
//
// Matrix-core operand layout (16x16x32, wave64; lane l, m = l % 16,
// kq = l / 16): A (16 x 32) lane holds A[m][8 kq .. 8 kq + 7]; B (32 x 16)
// lane holds B[8 kq .. 8 kq + 7][m]; D (16 x 16) lane holds
// D[4 kq .. 4 kq + 3][m].
#include <math.h>

#include <mutex>

#include "common.h"

namespace gs {

namespace {

constexpr int kKids = GS_ANCHOR_CHILDREN;  // 10
constexpr int kFeat = GS_ANCHOR_FEAT;      // 32
constexpr int kIn = kFeat + 3;             // 35 inputs
constexpr int kHid = 32;                   // hidden units per head
constexpr int kHidAll = 3 * kHid;          // 96
constexpr int kOut = 110;                  // 10 + 30 + 70 outputs
constexpr int kTile = 64;                  // anchors per workgroup iteration
// LDS row strides (elements): BF16 inputs and hidden units, FP32 outputs
constexpr int kXS = 72, kHS = 104, kYS = 161, kZS = 97, kDS = 65;
constexpr int kTS = 72;  // transposed BF16 copies (a row per input or hidden unit)
// Padded output columns: head h occupies columns 32 h .. 32 h + 31 (op,
// colour) and 64 .. 159 (covariance); the forward computes 16, 32 and 80 of
// them, the backward reads 32, 32 and 96.
__host__ __device__ constexpr int head_base(int h) { return 32 * h; }
__host__ __device__ constexpr int head_row(int h) {
  return h == 0 ? 0 : h == 1 ? 10 : h == 2 ? 40 : 110;
}
__host__ __device__ constexpr int head_len(int h) { return head_row(h + 1) - head_row(h); }
// The 50 padding columns: 10 .. 31, 62, 63, 134 .. 159.
__host__ __device__ constexpr int pad_col(int p) {
  return p < 22 ? 10 + p : p < 24 ? 62 + (p - 22) : 134 + (p - 24);
}
constexpr int kBwdThreads = 1024;          // the backward's workgroup
// Per-workgroup partial sums in the workspace: dW1 [96][48], dW2 [160][32]
// (padded rows), db1 [96], db2 [160].
constexpr int kWsW1 = 0, kWsW2 = kWsW1 + kHidAll * 48, kWsB1 = kWsW2 + 160 * kHid,
              kWsB2 = kWsB1 + kHidAll, kWsFloats = kWsB2 + 160;
constexpr int kMaxBlocks = 256;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// Round to nearest even: two values in one v_cvt_pk_bf16_f32, the first in the
// low half.
__device__ __forceinline__ uint32_t f2bf2(float a, float b) {
  const bf16x2 h = __builtin_convertvector((f32x2{a, b}), bf16x2);
  return __builtin_bit_cast(uint32_t, h);
}
__device__ __forceinline__ uint16_t f2bf(float f) { return (uint16_t)f2bf2(f, f); }

__device__ __forceinline__ bf16x8 pack8(const uint16_t (&h)[8]) {
  union {
    uint16_t s[8];
    bf16x8 v;
  } u;
#pragma unroll
  for (int e = 0; e < 8; ++e) u.s[e] = h[e];
  return u.v;
}

__device__ __forceinline__ bf16x8 lds8(const uint16_t* p) {  // 16-byte aligned
  union {
    uint4 q;
    bf16x8 v;
  } u;
  u.q = *reinterpret_cast<const uint4*>(p);
  return u.v;
}

// Two FP32 values split into BF16 hi and lo terms.
__device__ __forceinline__ void split2(float a, float b, uint32_t& hi, uint32_t& lo) {
  hi = f2bf2(a, b);
  lo = f2bf2(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xFFFF0000u));
}

// 8 FP32 values at p[0], p[stride], ... split into BF16 hi and lo terms.
__device__ __forceinline__ void split8(const float* p, int stride, bf16x8& hi, bf16x8& lo) {
  union {
    uint32_t q[4];
    bf16x8 v;
  } h, l;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    split2(p[2 * e * stride], p[(2 * e + 1) * stride], h.q[e], l.q[e]);
  hi = h.v;
  lo = l.v;
}

__device__ __forceinline__ bf16x8 gather8(const uint16_t* p, int stride) {
  uint16_t h[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) h[e] = p[e * stride];
  return pack8(h);
}

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float sigm(float x) { return 1.f / (1.f + expf(-x)); }

// BF16 copies of the weights, staged once per workgroup in LDS (in the
// space the tile loop uses later): W1 padded to 64 inputs [96][64] at s,
// W2 in padded rows [160][32] at s + 96 * 64. Ends with a barrier.
constexpr int kStageW2 = kHidAll * 64;
__device__ void stage_weights(const float* __restrict__ w1, const float* __restrict__ w2,
                              uint16_t* s) {
  constexpr int kP1 = (kHidAll * kIn + kBwdThreads - 1) / kBwdThreads;
  constexpr int kP2 = (kOut * kHid + kBwdThreads - 1) / kBwdThreads;
  const int tid = threadIdx.x;
  float v1[kP1], v2[kP2];  // every load issued before the first is used
#pragma unroll
  for (int q = 0; q < kP1; ++q) v1[q] = w1[min(tid + q * kBwdThreads, kHidAll * kIn - 1)];
#pragma unroll
  for (int q = 0; q < kP2; ++q) v2[q] = w2[min(tid + q * kBwdThreads, kOut * kHid - 1)];
#pragma unroll
  for (int q = 0; q < kP1; ++q) {
    const int e = tid + q * kBwdThreads;
    if (e < kHidAll * kIn) s[e / kIn * 64 + e % kIn] = f2bf(v1[q]);
  }
#pragma unroll
  for (int q = 0; q < kP2; ++q) {
    const int e = tid + q * kBwdThreads, r = e / kHid;
    const int hd = r < head_row(1) ? 0 : r < head_row(2) ? 1 : 2;
    if (e < kOut * kHid)
      s[kStageW2 + (head_base(hd) + r - head_row(hd)) * kHid + e % kHid] = f2bf(v2[q]);
  }
  for (int e = tid; e < kHidAll * (64 - kIn); e += kBwdThreads)
    s[e / (64 - kIn) * 64 + kIn + e % (64 - kIn)] = 0;
  for (int e = tid; e < 50 * kHid; e += kBwdThreads)  // the padding rows
    s[kStageW2 + pad_col(e / kHid) * kHid + e % kHid] = 0;
  __syncthreads();
}

// The backward runs 16 wavefronts per tile: wavefront w takes rows
// 16 (w % 4) .. + 15 and quarter h = w / 4 of every product's N-tiles, so it
// holds a quarter of the weight operands (three eighths where the tiles do not
// divide by four).
// layer 1: hidden N-tiles h and, for h < 2, 4 + h
// layer-2 output tiles in order (head, N-tile): 0: (0,0), 1-2: (1,0..1),
// 3-7: (2,0..4); quarter h computes tiles 2 h and 2 h + 1
// dL/dh: h = 0, 1: both N-tiles of head h; h = 2, 3: N-tile h - 2 of head 2
// dL/dx: N-tile h for h < 2
__host__ __device__ constexpr int l2_head(int t) { return t == 0 ? 0 : t < 3 ? 1 : 2; }
__host__ __device__ constexpr int l2_ntile(int t) { return t == 0 ? 0 : t < 3 ? t - 1 : t - 3; }

struct FwdWQuarter {
  bf16x8 w1[2][2];  // [hidden N-tile][K-step]
  bf16x8 w2[2];     // output tiles
};

__device__ void load_fwd_weights(const uint16_t* s, int h, FwdWQuarter& W) {
  const int l = threadIdx.x & 63, m = l & 15, kq = l >> 4;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int k = 0; k < 2; ++k)
      W.w1[j][k] = lds8(s + (16 * min(h + 4 * j, 5) + m) * 64 + 32 * k + 8 * kq);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int t = 2 * h + j;
    W.w2[j] = lds8(s + kStageW2 + (head_base(l2_head(t)) + 16 * l2_ntile(t) + m) * kHid + 8 * kq);
  }
}

struct BwdWQuarter {
  // h < 2: W2^T, N-tiles 0, 1 of head h, then W1^T, K-steps 0 .. 2 (hidden
  // 32 s ..) of N-tile h; else W2^T, K-steps 0 .. 2 of N-tile h - 2 of head 2
  bf16x8 t[5];
};

__device__ void load_bwd_weights(const uint16_t* s, int h, BwdWQuarter& W) {
  const int l = threadIdx.x & 63, m = l & 15, kq = l >> 4;
#pragma unroll
  for (int t = 0; t < 5; ++t) {
    const int hd = h < 2 ? h : 2, k = h < 2 ? 0 : t, nt = h < 2 ? t : h - 2;
    if (h < 2 ? t < 2 : t < 3)  // uniform
      W.t[t] = gather8(s + kStageW2 + (head_base(hd) + 32 * k + 8 * kq) * kHid + 16 * nt + m, kHid);
    else
      W.t[t] = gather8(s + (32 * max(t - 2, 0) + 8 * kq) * 64 + 16 * (h & 1) + m, 64);
  }
}

struct DecIn {
  const float *feat, *pos, *offsets, *scaling, *w1, *b1, *w2, *b2;
  int64_t A;
  double cx, cy, cz;  // camera centre
};

// Zero the padding columns 35 .. 71 of the input rows (never written again).
__device__ void zero_x_pad(uint16_t* sX) {
  for (int e = threadIdx.x; e < kTile * (kXS - kIn); e += (int)blockDim.x)
    sX[(e / (kXS - kIn)) * kXS + kIn + e % (kXS - kIn)] = 0;
}

// The biases, copied once per workgroup into LDS (read per N-tile in the
// tile loop: a global load there is one memory round trip per tile). Ends
// with a barrier.
struct Bias {
  float b1[kHidAll];
  float b2[kOut];
};

__device__ void stage_bias(const DecIn& in, Bias& B) {
  for (int e = threadIdx.x; e < kHidAll; e += (int)blockDim.x) B.b1[e] = in.b1[e];
  for (int e = threadIdx.x; e < kOut; e += (int)blockDim.x) B.b2[e] = in.b2[e];
  __syncthreads();
}

// The forward. A wavefront takes 16 anchors at a time and keeps them in
// registers: products are formed transposed (weights as the A operand, anchors
// as the columns of B and D), so lane (m, kq) loads the inputs 8 kq .. 8 kq + 7
// of anchor m straight from memory, layer 1 leaves it hidden units 4 kq .. + 3
// of each 16 in D, two lane swaps turn those into the 8 kq .. + 7 that layer 2
// takes, and the rows of W2 are dealt out so that D rows 4 kq .. + 3 of an
// output tile are one child's opacity and colour, scale or quaternion: what a
// child needs is in one lane, and nothing waits for another wavefront.
// Output tile t holds slots 4 t .. 4 t + 3 of four rows: slots 0 .. 9 opacity
// and colour (two heads, hence two products) of child `slot`, 12 .. 21 its
// scale (and mean), 22 .. 31 its quaternion.
//
// What bounds it: memory latency (two rounds of 16 wavefronts a compute unit
// at 100k anchors), behind 84 MB to read and write. Against 64 anchors per
// workgroup of four wavefronts that exchanged every layer through LDS, two
// workgroups a compute unit: 49 -> 23 us at 100k anchors (3.6 TB/s), 17.4 ->
// 9.5 us at 2k. Workgroups of 512, two a compute unit: the same.
constexpr int kFwdThreads = 1024;
constexpr int kFwdRows = 16;         // anchors per wavefront
constexpr int kWS = 40;              // LDS row stride of the weights (elements)
constexpr int kOutTiles = 8;

// W2 row of row r (0 .. 15) of output tile t, -1: padding.
__device__ __forceinline__ int out_row(int t, int r) {
  const int slot = 4 * t + (r >> 2), i = r & 3;
  if (slot < kKids) return i == 0 ? slot : head_row(1) + 3 * slot + i - 1;
  if (slot < 12) return -1;
  if (slot < 22) return i < 3 ? head_row(2) + 7 * (slot - 12) + i : -1;
  return head_row(2) + 7 * (slot - 22) + 3 + i;
}

__global__ void __launch_bounds__(kFwdThreads) k_decode_fwd(DecIn in, float* __restrict__ means,
                                                            float* __restrict__ scales,
                                                            float* __restrict__ quats,
                                                            float* __restrict__ opac,
                                                            float* __restrict__ rgb) {
  __shared__ __align__(16) uint16_t sW1[kHidAll * kWS];    // inputs 35 .. 39 zero
  __shared__ __align__(16) uint16_t sW2[(kOut + 1) * kWS];  // row kOut zero
  __shared__ __align__(16) float sB1[kHidAll], sB2[kOutTiles * 16];
  const int tid = threadIdx.x, l = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t A = in.A, N = A * kKids;
  const int64_t step = (int64_t)gridDim.x * (kFwdThreads / kWave) * kFwdRows;
  // two neighbouring groups of 16 (a 128-byte line of every array) to a
  // workgroup, whose chiplet then reads the line once (groups dealt singly:
  // 57 instead of 28 MB read at 100k anchors); wavefronts 2 w, 2 w + 1 of every
  // workgroup before 2 w + 2 of any, so few anchors still go to many compute
  // units
  int64_t a0 = (((int64_t)(w >> 1) * gridDim.x + blockIdx.x) * 2 + (w & 1)) * kFwdRows;
  float fv[8], pv[3];
  const auto fetch = [&](int m, int kq) {  // anchor inputs (past the end: the last anchor's)
    const int64_t ai = a0 + m < A ? a0 + m : A - 1;
#pragma unroll
    for (int e = 0; e < 8; ++e) fv[e] = in.feat[(8 * kq + e) * A + ai];
#pragma unroll
    for (int d = 0; d < 3; ++d) pv[d] = in.pos[d * A + ai];
  };
  fetch(l & 15, l >> 4);
  {  // the weights, every load issued before the first is used
    constexpr int kP1 = (kHidAll * kIn + kFwdThreads - 1) / kFwdThreads;
    constexpr int kP2 = (kOut * kHid + kFwdThreads - 1) / kFwdThreads;
    float v1[kP1], v2[kP2];
#pragma unroll
    for (int q = 0; q < kP1; ++q) v1[q] = in.w1[min(tid + q * kFwdThreads, kHidAll * kIn - 1)];
#pragma unroll
    for (int q = 0; q < kP2; ++q) v2[q] = in.w2[min(tid + q * kFwdThreads, kOut * kHid - 1)];
    if (tid < kHidAll) sB1[tid] = in.b1[tid];
    if (tid < kOutTiles * 16) {
      const int r = out_row(tid >> 4, tid & 15);
      sB2[tid] = r >= 0 ? in.b2[r] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < kP1; ++q) {
      const int e = tid + q * kFwdThreads;
      if (e < kHidAll * kIn) sW1[e / kIn * kWS + e % kIn] = f2bf(v1[q]);
    }
#pragma unroll
    for (int q = 0; q < kP2; ++q) {
      const int e = tid + q * kFwdThreads;
      if (e < kOut * kHid) sW2[e / kHid * kWS + e % kHid] = f2bf(v2[q]);
    }
    for (int e = tid; e < kHidAll * (kWS - kIn); e += kFwdThreads)
      sW1[e / (kWS - kIn) * kWS + kIn + e % (kWS - kIn)] = 0;
    if (tid < kWS) sW2[kOut * kWS + tid] = 0;
    __syncthreads();
  }
  const bf16x8 none = lds8(sW2 + kOut * kWS);  // zeros
  for (; a0 < A; a0 += step) {
    // the weights are read where they are used: the compiler must not see that
    // they are the same in every turn, or it keeps them all in registers
    int lane = l;
    asm volatile("" : "+v"(lane));
    const int m = lane & 15, kq = lane >> 4;
    const int64_t ai = a0 + m < A ? a0 + m : A - 1;
    const bool live = a0 + m < A;
    // what the children need of the anchor (child 4 t + kq of output tile 3 + t)
    float off[3][3], so[3], ss[3], pos[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      so[d] = in.scaling[d * A + ai];
      ss[d] = in.scaling[(3 + d) * A + ai];
      pos[d] = pv[d];
#pragma unroll
      for (int t = 0; t < 3; ++t)
        off[t][d] = in.offsets[(3 * min(4 * t + kq, kKids - 1) + d) * A + ai];
    }
    bf16x8 x0, x1 = none;
    {
      uint16_t h[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) h[e] = f2bf(fv[e]);
      x0 = pack8(h);
      if (kq == 0) {
#pragma clang fp contract(off)
        const double d0 = in.cx - (double)pv[0];
        const double d1 = in.cy - (double)pv[1];
        const double d2 = in.cz - (double)pv[2];
        const double nrm = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
        const uint16_t g[8] = {f2bf((float)(d0 / nrm)), f2bf((float)(d1 / nrm)),
                               f2bf((float)(d2 / nrm)), 0, 0, 0, 0, 0};
        x1 = pack8(g);
      }
    }
    // layer 1, and the hidden units as layer 2's operands
    bf16x8 hid[3];
#pragma unroll
    for (int hd = 0; hd < 3; ++hd) {
      uint32_t p[2][2];  // [16 units][pair]: units 4 kq, + 1 and + 2, + 3
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int nt = 2 * hd + u, row = 16 * nt + m;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = mfma(lds8(sW1 + row * kWS + 8 * kq), x0, acc);
        acc = mfma(lds8(kq == 0 ? sW1 + row * kWS + kFeat : sW2 + kOut * kWS), x1, acc);
        const float4 bb = *reinterpret_cast<const float4*>(sB1 + 16 * nt + 4 * kq);
        p[u][0] = f2bf2(fmaxf(acc[0] + bb.x, 0.f), fmaxf(acc[1] + bb.y, 0.f));
        p[u][1] = f2bf2(fmaxf(acc[2] + bb.z, 0.f), fmaxf(acc[3] + bb.w, 0.f));
      }
      typedef unsigned u2 __attribute__((ext_vector_type(2)));
      union {
        uint32_t q[4];
        bf16x8 v;
      } o;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        // rows of 16 lanes: (0 1 2 3), (0' 1' 2' 3') -> (0 1 0' 1'), (2 3 2' 3')
        // -> (0 2 0' 2'), (1 3 1' 3')
        const u2 a = __builtin_amdgcn_permlane32_swap(p[0][c], p[1][c], false, false);
        const u2 b = __builtin_amdgcn_permlane16_swap(a.x, a.y, false, false);
        o.q[c] = b.x;
        o.q[2 + c] = b.y;
      }
      hid[hd] = o.v;
    }
    a0 += step;
    if (a0 < A) fetch(m, kq);  // the next anchors', behind the rest
    a0 -= step;
#pragma unroll
    for (int t = 0; t < kOutTiles; ++t) {
      const int r = out_row(t, m);
      const uint16_t* wr = sW2 + (r >= 0 ? r : kOut) * kWS + 8 * kq;
      const bf16x8 wv = lds8(wr);
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      if (t < 3) {
        // row 4 i of the tile: opacity (head 0); the others: colour (head 1). Each
        // head has a sum of its own, so that an infinite hidden unit stays in it.
        const f32x4 op = mfma(wv, hid[0], acc);
        acc = mfma(wv, hid[1], acc);
        acc[0] = op[0];
      } else {
        acc = mfma(wv, hid[2], acc);
      }
      const float4 bb = *reinterpret_cast<const float4*>(sB2 + 16 * t + 4 * kq);
      const float y0 = acc[0] + bb.x, y1 = acc[1] + bb.y, y2 = acc[2] + bb.z,
                  y3 = acc[3] + bb.w;
      const int slot = 4 * t + kq;
      if (!live) continue;
      if (slot < kKids) {
        const int64_t g = slot * A + ai;
        opac[g] = fmaxf(tanhf(y0), 0.f);
        rgb[g] = sigm(y1);
        rgb[N + g] = sigm(y2);
        rgb[2 * N + g] = sigm(y3);
      } else if (slot >= 12 && slot < 22) {
        const int64_t g = (slot - 12) * A + ai;
        scales[g] = ss[0] * sigm(y0);
        scales[N + g] = ss[1] * sigm(y1);
        scales[2 * N + g] = ss[2] * sigm(y2);
#pragma unroll
        for (int d = 0; d < 3; ++d)
          means[d * N + g] = pos[d] + off[min(max(t - 3, 0), 2)][d] * so[d];
      } else if (slot >= 22) {
        const int64_t g = (slot - 22) * A + ai;
        const float inv = 1.f / sqrtf(y0 * y0 + y1 * y1 + y2 * y2 + y3 * y3);
        quats[g] = y0 * inv;
        quats[N + g] = y1 * inv;
        quats[2 * N + g] = y2 * inv;
        quats[3 * N + g] = y3 * inv;
      }
    }
  }
}

struct DecGrad {
  const float *dmeans, *dscales, *dquats, *dopac, *drgb;  // child-Gaussian gradients
  float *dfeat, *doffsets, *dscaling;                     // per-anchor outputs (may be null)
  float* ws;                                              // per-workgroup partial sums
  int accumulate;
};

// The forward of one tile of anchors a0 .. a0 + 63 for the backward's 16
// wavefronts: sX (BF16 inputs), sH (BF16 hidden units), sY (FP32 y + b2 in
// padded columns), divided as above. Ends with a barrier.
__device__ void tile_forward(const DecIn& in, const Bias& B, int64_t a0, int tid, int h,
                             const FwdWQuarter& W, uint16_t* sX, uint16_t* sH, float* sY,
                             uint16_t* sXT, uint16_t* sHT) {
  const int64_t A = in.A;
  {
    constexpr int kPer = kFeat * kTile / kBwdThreads;  // 2
    static_assert(kFeat * kTile % kBwdThreads == 0, "whole rounds");
    float fv[kPer];  // every load issued before the first is used
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int e = tid + q * kBwdThreads, k = e / kTile, m = e % kTile;
      const int64_t ai = a0 + m;
      fv[q] = in.feat[k * A + (ai < A ? ai : a0)];  // a0 < A: a valid row
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int e = tid + q * kBwdThreads, k = e / kTile, m = e % kTile;
      const uint16_t v = a0 + m < A ? f2bf(fv[q]) : (uint16_t)0;
      sX[m * kXS + k] = v;
      sXT[k * kTS + m] = v;
    }
  }
  if (tid < kTile) {
#pragma clang fp contract(off)
    const int64_t ai = a0 + tid;
    uint16_t d3[3] = {0, 0, 0};
    if (ai < A) {
      const double d0 = in.cx - (double)in.pos[ai];
      const double d1 = in.cy - (double)in.pos[A + ai];
      const double d2 = in.cz - (double)in.pos[2 * A + ai];
      const double nrm = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
      d3[0] = f2bf((float)(d0 / nrm));
      d3[1] = f2bf((float)(d1 / nrm));
      d3[2] = f2bf((float)(d2 / nrm));
    }
    for (int j = 0; j < 3; ++j) {
      sX[tid * kXS + kFeat + j] = d3[j];
      sXT[(kFeat + j) * kTS + tid] = d3[j];
    }
  }
  __syncthreads();
  const int l = tid & 63, wr = (tid >> 6) & 3, m = l & 15, kq = l >> 4;
  const int row = 16 * wr + m;
  const bf16x8 xa0 = lds8(sX + row * kXS + 8 * kq);
  const bf16x8 xa1 = lds8(sX + row * kXS + 32 + 8 * kq);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (h + 4 * j > 5) continue;  // uniform
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = mfma(xa0, W.w1[j][0], acc);
    acc = mfma(xa1, W.w1[j][1], acc);
    const int hid = 16 * (h + 4 * j) + m;
    const float bb = B.b1[hid];
    uint32_t v[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
      v[i] = f2bf2(fmaxf(acc[2 * i] + bb, 0.f), fmaxf(acc[2 * i + 1] + bb, 0.f));
#pragma unroll
    for (int i = 0; i < 4; ++i)
      sH[(16 * wr + 4 * kq + i) * kHS + hid] = (uint16_t)(v[i / 2] >> (16 * (i & 1)));
    *reinterpret_cast<uint2*>(sHT + hid * kTS + 16 * wr + 4 * kq) = make_uint2(v[0], v[1]);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int t = 2 * h + j, hd = l2_head(t), nt = l2_ntile(t);
    const bf16x8 ha = lds8(sH + row * kHS + kHid * hd + 8 * kq);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = mfma(ha, W.w2[j], acc);
    const int local = 16 * nt + m;
    const float bb = local < head_len(hd) ? B.b2[head_row(hd) + local] : 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      sY[(16 * wr + 4 * kq + i) * kYS + head_base(hd) + local] = acc[i] + bb;
  }
  __syncthreads();
}

__device__ __forceinline__ void put(float* p, float v, int accumulate) {
  if (accumulate) *p += v; else *p = v;
}

// The backward. One workgroup a compute unit takes a tile of 64 anchors at a
// time through the phases below; every weight-gradient sum adds the anchors of
// its workgroup in order, so the grid and the tiles decide its bits.
// What bounds it: a phase's LDS traffic and conversions, one after the other
// between barriers (61% of the wavefronts' cycles are waits, a third of the
// rest LDS). 99.6 -> 85.5 us at 100k anchors: BF16 conversions by instruction
// instead of integer arithmetic 6 us, loads ahead of the tile's forward and 16
// wavefronts instead of 8 4 us, and the weight gradients' operands read 16
// bytes at a time from transposed copies, instead of gathered (and dL/dz split
// anew) by every tile that takes them, 5 us.
__global__ void __launch_bounds__(kBwdThreads) k_decode_bwd(DecIn in, DecGrad gr) {
  __shared__ __align__(16) uint16_t sX[kTile * kXS];
  __shared__ __align__(16) uint16_t sH[kTile * kHS];
  __shared__ __align__(16) float sY[kTile * kYS];   // y, then dL/dy in place
  __shared__ float sZ[kTile * kZS];   // dL/dz
  __shared__ float sD[kFeat * kDS];   // dL/dfeat, transposed for coalesced writes
  __shared__ float sP[3][kKids][kTile];  // dL/dscale sigmoid(y)
  // What the weight gradients take along the anchors, 8 at a time: inputs,
  // hidden units and dL/dz in its two terms, transposed as they are written
  __shared__ __align__(16) uint16_t sXT[48 * kTS], sHT[kHidAll * kTS], sZh[kHidAll * kTS],
      sZl[kHidAll * kTS];
  __shared__ Bias sB;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = w & 3, h = w >> 2;  // row block and N-tile quarter of this wavefront
  FwdWQuarter Wf;
  BwdWQuarter Wb;
  stage_bias(in, sB);
  stage_weights(in.w1, in.w2, reinterpret_cast<uint16_t*>(sY));
  load_fwd_weights(reinterpret_cast<const uint16_t*>(sY), h, Wf);
  load_bwd_weights(reinterpret_cast<const uint16_t*>(sY), h, Wb);
  zero_x_pad(sX);
  for (int e = threadIdx.x; e < (48 - kIn) * kTS; e += kBwdThreads) sXT[kIn * kTS + e] = 0;
  __syncthreads();
  const int64_t A = in.A, N = A * kKids;
  // weight-gradient tiles of this wavefront: W2 (8 x 2 tiles) w; W1 (6 x 3
  // tiles) w, and the last two for wavefronts 8 and 9 (which have no dL/dx)
  f32x4 accW2 = {0.f, 0.f, 0.f, 0.f}, accW1[2] = {accW2, accW2};
  const auto w1_tile = [&](int q) { return q == 0 ? w : w == 8 || w == 9 ? w + 8 : 18; };
  float dbias = 0.f;  // bt 0..159: b2 padded column; 160..255: b1 unit
  const int bt = (int)threadIdx.x - (kBwdThreads - 160 - kHidAll);
  for (int64_t a0 = (int64_t)blockIdx.x * kTile; a0 < A; a0 += (int64_t)gridDim.x * kTile) {
    // the addresses below are formed anew in every turn: kept, they would take
    // the registers of the reads ahead
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int l = tid & 63, m = l & 15, kq = l >> 4;
    // What the elementwise part needs, read ahead of the tile's forward: the
    // (child, anchor) items of the first ten wavefronts, and for three others,
    // one axis d each, the offsets' part, which does not depend on the outputs
    // (in the same registers).
    float q[2 * kKids], sc = 0.f;
    const auto read_item = [&](int it) {
      const int j = it / kTile;
      const int64_t ai = a0 + it % kTile < A ? a0 + it % kTile : A - 1, g = j * A + ai;
      q[0] = gr.dopac[g];
#pragma unroll
      for (int c = 0; c < 3; ++c) q[1 + c] = gr.drgb[c * N + g];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        q[4 + a] = gr.dscales[a * N + g];
        q[7 + a] = in.scaling[(3 + a) * A + ai];
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) q[10 + c] = gr.dquats[c * N + g];
    };
    static_assert(kTile == kWave && kKids + 3 <= kBwdThreads / kWave, "a wavefront per child");
    if (w < kKids) read_item(tid);
    const int d = w - kKids;
    const bool axis = d >= 0 && d < 3;
    if (axis) {
      const int64_t ai = a0 + l < A ? a0 + l : A - 1;
      sc = in.scaling[d * A + ai];
#pragma unroll
      for (int j = 0; j < kKids; ++j) {
        q[j] = gr.dmeans[d * N + j * A + ai];
        q[kKids + j] = in.offsets[(3 * j + d) * A + ai];
      }
    }
    tile_forward(in, sB, a0, tid, h, Wf, sX, sH, sY, sXT, sHT);
    // dL/dy in place of y (one (child, anchor) item per thread; zero
    // for absent anchors), and the items' dL/dscale sigmoid(y) for the scaling
    // gradient
    const auto item = [&](int it) {
      const int j = it / kTile, mm = it % kTile;
      const int64_t ai = a0 + mm;
      float* y = sY + mm * kYS;
      float* yc = y + 32 + 3 * j;
      float* yv = y + 64 + 7 * j;
      if (ai >= A) {
        y[j] = 0.f;
        for (int c = 0; c < 3; ++c) yc[c] = 0.f;
        for (int c = 0; c < 7; ++c) yv[c] = 0.f;
        return;
      }
      const float th = tanhf(y[j]);
      y[j] = th > 0.f ? q[0] * (1.f - th * th) : 0.f;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float s = sigm(yc[c]);
        yc[c] = q[1 + c] * s * (1.f - s);
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const float s = sigm(yv[a]);
        sP[a][j][mm] = q[4 + a] * s;
        yv[a] = q[4 + a] * q[7 + a] * s * (1.f - s);
      }
      const float r0 = yv[3], r1 = yv[4], r2 = yv[5], r3 = yv[6];
      const float nrm = sqrtf(r0 * r0 + r1 * r1 + r2 * r2 + r3 * r3);
      const float n0 = r0 / nrm, n1 = r1 / nrm, n2 = r2 / nrm, n3 = r3 / nrm;
      const float d0 = q[10], d1 = q[11], d2 = q[12], d3 = q[13];
      const float dot = n0 * d0 + n1 * d1 + n2 * d2 + n3 * d3;
      yv[3] = (d0 - n0 * dot) / nrm;
      yv[4] = (d1 - n1 * dot) / nrm;
      yv[5] = (d2 - n2 * dot) / nrm;
      yv[6] = (d3 - n3 * dot) / nrm;
    };
    if (w < kKids) item(tid);
    if (axis && a0 + l < A) {
      const int64_t ai = a0 + l;
      if (gr.doffsets)
#pragma unroll
        for (int j = 0; j < kKids; ++j)
          put(gr.doffsets + (3 * j + d) * A + ai, q[j] * sc, gr.accumulate);
      float g_off = 0.f;
#pragma unroll
      for (int j = 0; j < kKids; ++j) g_off += q[j] * q[kKids + j];
      if (gr.dscaling) put(gr.dscaling + d * A + ai, g_off, gr.accumulate);
    }
    // padded columns
    for (int it = tid; it < kTile * 50; it += kBwdThreads) {
      sY[it / 50 * kYS + pad_col(it % 50)] = 0.f;
    }
    __syncthreads();
    if (axis && gr.dscaling && a0 + l < A) {
      float g_sc = 0.f;
#pragma unroll
      for (int j = 0; j < kKids; ++j) g_sc += sP[d][j][l];
      put(gr.dscaling + (3 + d) * A + a0 + l, g_sc, gr.accumulate);
    }
    const int row = 16 * wr + m;
    // dL/dh = W2^T dy per head, through the ReLU into dL/dz
    {
      const auto to_z = [&](int hid, const f32x4& acc) {
        float z[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 16 * wr + 4 * kq + i;
          z[i] = sH[r * kHS + hid] != 0 ? acc[i] : 0.f;
          sZ[r * kZS + hid] = z[i];
        }
        uint32_t zh[2], zl[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) split2(z[2 * i], z[2 * i + 1], zh[i], zl[i]);
        const int at = hid * kTS + 16 * wr + 4 * kq;
        *reinterpret_cast<uint2*>(sZh + at) = make_uint2(zh[0], zh[1]);
        *reinterpret_cast<uint2*>(sZl + at) = make_uint2(zl[0], zl[1]);
      };
      bf16x8 hi, lo;
      if (h < 2) {
        split8(sY + row * kYS + head_base(h) + 8 * kq, 1, hi, lo);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          f32x4 acc = {0.f, 0.f, 0.f, 0.f};
          acc = mfma(hi, Wb.t[nt], acc);
          acc = mfma(lo, Wb.t[nt], acc);
          to_z(kHid * h + 16 * nt + m, acc);
        }
      } else {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          split8(sY + row * kYS + head_base(2) + 32 * s + 8 * kq, 1, hi, lo);
          acc = mfma(hi, Wb.t[s], acc);
          acc = mfma(lo, Wb.t[s], acc);
        }
        to_z(kHid * 2 + 16 * (h - 2) + m, acc);
      }
    }
    __syncthreads();
    // dL/dfeat = (W1^T dz)[0..31], inputs 16 h .. 16 h + 15
    if (h < 2) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        bf16x8 hi, lo;
        split8(sZ + row * kZS + 32 * s + 8 * kq, 1, hi, lo);
        acc = mfma(hi, Wb.t[2 + s], acc);
        acc = mfma(lo, Wb.t[2 + s], acc);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) sD[(16 * h + m) * kDS + 16 * wr + 4 * kq + i] = acc[i];
    }
    // weight gradients over this tile (K = anchors, two 32-anchor steps)
    {
      const int mt = w >> 1, nt = w & 1, hd = l2_head(mt);
      const int colb = head_base(hd) + 16 * l2_ntile(mt);
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int k0 = 32 * s + 8 * kq;
        bf16x8 hi, lo;
        split8(sY + k0 * kYS + colb + m, kYS, hi, lo);
        const bf16x8 b = lds8(sHT + (kHid * hd + 16 * nt + m) * kTS + k0);
        accW2 = mfma(hi, b, accW2);
        accW2 = mfma(lo, b, accW2);
      }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int idx = w1_tile(q);
      if (idx < 18) {
        const int mt = idx / 3, nt = idx % 3;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const int k0 = 32 * s + 8 * kq;
          const bf16x8 hi = lds8(sZh + (16 * mt + m) * kTS + k0);
          const bf16x8 lo = lds8(sZl + (16 * mt + m) * kTS + k0);
          const bf16x8 b = lds8(sXT + (16 * nt + m) * kTS + k0);
          accW1[q] = mfma(hi, b, accW1[q]);
          accW1[q] = mfma(lo, b, accW1[q]);
        }
      }
    }
    // the bias sums: by the last wavefronts, of which most have one tile less
    if (bt >= 0 && bt < 160) {
#pragma unroll 16
      for (int r = 0; r < kTile; ++r) dbias += sY[r * kYS + bt];
    } else if (bt >= 160) {
#pragma unroll 16
      for (int r = 0; r < kTile; ++r) dbias += sZ[r * kZS + bt - 160];
    }
    __syncthreads();
    if (gr.dfeat)
      for (int e = tid; e < kFeat * kTile; e += kBwdThreads) {
        const int k = e / kTile, mm = e % kTile;
        const int64_t ai = a0 + mm;
        if (ai < A) put(gr.dfeat + k * A + ai, sD[k * kDS + mm], gr.accumulate);
      }
    __syncthreads();
  }
  // partial sums of this workgroup
  const int l = threadIdx.x & 63, m = l & 15, kq = l >> 4;
  float* ws = gr.ws + (int64_t)blockIdx.x * kWsFloats;
  {
    const int mt = w >> 1, nt = w & 1, colb = head_base(l2_head(mt)) + 16 * l2_ntile(mt);
#pragma unroll
    for (int i = 0; i < 4; ++i) ws[kWsW2 + (colb + 4 * kq + i) * kHid + 16 * nt + m] = accW2[i];
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int idx = w1_tile(q);
    if (idx < 18) {
      const int mt = idx / 3, nt = idx % 3;
#pragma unroll
      for (int i = 0; i < 4; ++i) ws[kWsW1 + (16 * mt + 4 * kq + i) * 48 + 16 * nt + m] = accW1[q][i];
    }
  }
  if (bt >= 0 && bt < 160) ws[kWsB2 + bt] = dbias;
  else if (bt >= 160) ws[kWsB1 + bt - 160] = dbias;
}

// Sum of the per-workgroup partials (deterministic): a block takes 32
// parameters; thread group g (of 8) sums the partials of workgroups g, g + 8,
// ... in order, then the 8 group sums are added in group order.
constexpr int kRedParams = 32, kRedGroups = 8;
__global__ void __launch_bounds__(kRedParams* kRedGroups) k_decode_reduce(
    const float* __restrict__ ws, int nblk, float* __restrict__ dw1, float* __restrict__ db1,
    float* __restrict__ dw2, float* __restrict__ db2, int accumulate) {
  __shared__ float part[kRedGroups][kRedParams];
  const int lp = threadIdx.x % kRedParams, grp = threadIdx.x / kRedParams;
  const int t = blockIdx.x * kRedParams + lp;
  int src = -1;
  float* dst = nullptr;
  if (t < kHidAll * kIn) {
    src = kWsW1 + (t / kIn) * 48 + t % kIn;
    dst = dw1 + t;
  } else if (t < kHidAll * kIn + kHidAll) {
    const int h = t - kHidAll * kIn;
    src = kWsB1 + h;
    dst = db1 + h;
  } else if (t < kHidAll * kIn + kHidAll + kOut * kHid) {
    const int u = t - kHidAll * kIn - kHidAll, r = u / kHid, c = u % kHid;
    const int hd = r < 10 ? 0 : r < 40 ? 1 : 2;
    src = kWsW2 + (head_base(hd) + r - head_row(hd)) * kHid + c;
    dst = dw2 + u;
  } else if (t < kHidAll * kIn + kHidAll + kOut * kHid + kOut) {
    const int r = t - kHidAll * kIn - kHidAll - kOut * kHid;
    const int hd = r < 10 ? 0 : r < 40 ? 1 : 2;
    src = kWsB2 + head_base(hd) + r - head_row(hd);
    dst = db2 + r;
  }
  float s = 0.f;
  if (src >= 0) {
#pragma unroll 4
    for (int b = grp; b < nblk; b += kRedGroups) s += ws[(int64_t)b * kWsFloats + src];
  }
  part[grp][lp] = s;
  __syncthreads();
  if (grp == 0 && src >= 0) {
    float tot = 0.f;
#pragma unroll
    for (int k = 0; k < kRedGroups; ++k) tot += part[k][lp];
    put(dst, tot, accumulate);
  }
}

constexpr int kParamCount = kHidAll * kIn + kHidAll + kOut * kHid + kOut;

int decode_blocks(int64_t A) {
  const int64_t tiles = (A + kTile - 1) / kTile;
  return (int)(tiles < kMaxBlocks ? tiles : kMaxBlocks);
}

bool anchors_ok(const gs_anchors* a) {
  return a && a->feat && a->pos && a->offsets && a->scaling;
}
bool mlp_ok(const gs_mlp* p) { return p && p->w1 && p->b1 && p->w2 && p->b2; }

DecIn make_in(const gs_anchors* a, int64_t A, const gs_mlp* p, const CamDev& cd) {
  DecIn in;
  in.feat = a->feat; in.pos = a->pos; in.offsets = a->offsets; in.scaling = a->scaling;
  in.w1 = p->w1; in.b1 = p->b1; in.w2 = p->w2; in.b2 = p->b2;
  in.A = A;
  in.cx = cd.campos[0]; in.cy = cd.campos[1]; in.cz = cd.campos[2];
  return in;
}

}  // namespace

}  // namespace gs

using namespace gs;

extern "C" gs_status gs_anchor_decode_fwd(const gs_anchors* anchors, int64_t n_anchors,
                                          const gs_mlp* mlp, const gs_camera* cam,
                                          gs_gaussians* out, void* stream) {
  CamDev cd;
  if (n_anchors < 0 || n_anchors > ((int64_t)1 << 28) || !make_cam(cam, &cd)) return GS_EINVAL;
  if (n_anchors == 0) return GS_OK;
  if (!anchors_ok(anchors) || !mlp_ok(mlp) || !out || !out->means || !out->log_scales ||
      !out->quats || !out->opacity_logits || !out->sh)
    return GS_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const DecIn in = make_in(anchors, n_anchors, mlp, cd);
  const int64_t groups = (n_anchors + kFwdRows - 1) / kFwdRows;
  const int nb = (int)(groups < 512 ? (groups + 1) / 2 : 256);
  GS_TIMED("decode_fwd", st,
           k_decode_fwd<<<nb, kFwdThreads, 0, st>>>(in, out->means, out->log_scales, out->quats,
                                                 out->opacity_logits, out->sh));
  GS_CHECK_LAUNCH();
  return GS_OK;
}

extern "C" gs_status gs_anchor_decode_workspace(int64_t n_anchors, size_t* bytes) {
  if (n_anchors < 0 || !bytes) return GS_EINVAL;
  *bytes = (size_t)decode_blocks(n_anchors) * kWsFloats * sizeof(float);
  return GS_OK;
}

namespace gs {
namespace {

// The backward's two launches on a caller-given partial-sum buffer `ws` of
// decode_blocks(A) * kWsFloats floats (every launched workgroup writes all of
// its partials, so the buffer needs no clearing). `timed`: bracket the
// launches with the launch timer (which creates events; the allocation-free
// entry point passes false).
gs_status decode_bwd_launch(const gs_anchors* anchors, int64_t n_anchors, const gs_mlp* mlp,
                            const CamDev& cd, const gs_gaussians* dchild, gs_anchors* danchors,
                            gs_mlp* dmlp, float* ws, int32_t accumulate, hipStream_t st,
                            bool timed) {
  const int nb = decode_blocks(n_anchors);
  if (n_anchors > 0) {
    const DecIn in = make_in(anchors, n_anchors, mlp, cd);
    DecGrad gr;
    gr.dmeans = dchild->means; gr.dscales = dchild->log_scales; gr.dquats = dchild->quats;
    gr.dopac = dchild->opacity_logits; gr.drgb = dchild->sh;
    gr.dfeat = danchors->feat; gr.doffsets = danchors->offsets; gr.dscaling = danchors->scaling;
    gr.ws = ws;
    gr.accumulate = accumulate;
    if (timed)
      GS_TIMED("decode_bwd", st, k_decode_bwd<<<nb, kBwdThreads, 0, st>>>(in, gr));
    else
      k_decode_bwd<<<nb, kBwdThreads, 0, st>>>(in, gr);
    GS_CHECK_LAUNCH();
  }
  const int rb = div_up(kParamCount, kRedParams);
  const int rnb = n_anchors > 0 ? nb : 0;
  if (timed)
    GS_TIMED("decode_reduce", st,
             k_decode_reduce<<<rb, kRedParams * kRedGroups, 0, st>>>(
                 ws, rnb, dmlp->w1, dmlp->b1, dmlp->w2, dmlp->b2, accumulate));
  else
    k_decode_reduce<<<rb, kRedParams * kRedGroups, 0, st>>>(ws, rnb, dmlp->w1, dmlp->b1,
                                                            dmlp->w2, dmlp->b2, accumulate);
  GS_CHECK_LAUNCH();
  return GS_OK;
}

// Arguments shared by both backward entry points: GS_EINVAL checks.
bool decode_bwd_args_ok(const gs_anchors* anchors, int64_t n_anchors, const gs_mlp* mlp,
                        const gs_camera* cam, const gs_gaussians* dchild,
                        const gs_anchors* danchors, const gs_mlp* dmlp, int32_t accumulate,
                        CamDev* cd) {
  if (n_anchors < 0 || n_anchors > ((int64_t)1 << 28) || !make_cam(cam, cd) ||
      (accumulate != 0 && accumulate != 1) || !mlp_ok(dmlp))
    return false;
  if (n_anchors > 0 &&
      (!anchors_ok(anchors) || !mlp_ok(mlp) || !dchild || !dchild->means ||
       !dchild->log_scales || !dchild->quats || !dchild->opacity_logits || !dchild->sh ||
       !danchors))
    return false;
  return true;
}

}  // namespace
}  // namespace gs

extern "C" gs_status gs_anchor_decode_bwd(const gs_anchors* anchors, int64_t n_anchors,
                                          const gs_mlp* mlp, const gs_camera* cam,
                                          const gs_gaussians* dchild, gs_anchors* danchors,
                                          gs_mlp* dmlp, void* workspace, size_t workspace_bytes,
                                          int32_t accumulate, void* stream) {
  CamDev cd;
  if (!decode_bwd_args_ok(anchors, n_anchors, mlp, cam, dchild, danchors, dmlp, accumulate, &cd))
    return GS_EINVAL;
  const int nb = decode_blocks(n_anchors);
  if (n_anchors > 0 &&
      (!workspace || workspace_bytes < (size_t)nb * kWsFloats * sizeof(float)))
    return GS_ECAPACITY;
  return decode_bwd_launch(anchors, n_anchors, mlp, cd, dchild, danchors, dmlp,
                           (float*)workspace, accumulate, (hipStream_t)stream, true);
}

// ---------------------------------------------------------------------------
// Allocation-free backward: the per-workgroup partials live in a fixed
// device array of the library instead of a caller workspace. The array is
// sized for the largest grid the backward launches (kMaxBlocks workgroups,
// whatever the anchor count), so every A the backward accepts fits.
static __device__ __align__(256) float scratch[kMaxBlocks * kWsFloats];
static_assert(sizeof(scratch) == GS_DECODE_SCRATCH_BYTES, "header states the scratch size");

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch[kMaxDevices] = {};  // device address of `scratch`, per device

// The address of the current device's copy of `scratch`, looked up once per
// device (with that device current) and kept; never the array's host-side
// name, which is no device address.
gs_status scratch_on_current_device(float** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return GS_EHIP;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return GS_EHIP;
    g_scratch[dev] = static_cast<float*>(p);
  }
  *out = g_scratch[dev];
  return GS_OK;
}
}  // namespace

extern "C" gs_status gs_anchor_decode_bwd_noalloc(const gs_anchors* anchors, int64_t n_anchors,
                                                  const gs_mlp* mlp, const gs_camera* cam,
                                                  const gs_gaussians* dchild,
                                                  gs_anchors* danchors, gs_mlp* dmlp,
                                                  int32_t accumulate, void* stream) {
  CamDev cd;
  if (!decode_bwd_args_ok(anchors, n_anchors, mlp, cam, dchild, danchors, dmlp, accumulate, &cd))
    return GS_EINVAL;
  if ((size_t)decode_blocks(n_anchors) * kWsFloats > sizeof(scratch) / sizeof(float))
    return GS_ECAPACITY;
  float* ws = nullptr;
  const gs_status st = scratch_on_current_device(&ws);
  if (st != GS_OK) return st;
  return decode_bwd_launch(anchors, n_anchors, mlp, cd, dchild, danchors, dmlp, ws, accumulate,
                           (hipStream_t)stream, false);
}
