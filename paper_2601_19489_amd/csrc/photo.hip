// Photometric loss of Eq. 5 for one view, E = (1 - lambda) L1 + lambda
// (1 - SSIM), and its image gradient; the pruning-score accumulation of
// Eq. 6. SSIM per colour channel under an 11 x 11 Gaussian window (sigma
// 1.5, normalised) with zero padding, C1 = 0.01^2, C2 = 0.03^2; SSIM and L1
// are means over channels and pixels.
//
// Forward: one workgroup per 32 x 32 output tile of one channel. The 42 x 42
// input patch of both images goes to LDS, a horizontal 11-tap pass writes the
// five window sums (x, y, x^2, y^2, xy) per patch row and output column to
// LDS, and a vertical pass finishes them per pixel. With the gradient
// requested, each pixel also writes the three partials of its SSIM term with
// respect to the window's mean, second moment and cross moment of x; the
// backward correlates those maps with the same window (it is symmetric) and
// combines them with x and y at the pixel.
//
// What bounds it: VALU issue (some 130 operations per pixel forward, 70
// backward); before, it was the LDS, of which every output read all of its
// window's values. So a thread forms eight neighbouring columns of a row, or
// four neighbouring rows of a column, from values it reads once (6 + 18 LDS
// words per pixel forward, where 29 + 55 were read), each sum over the taps in
// the order it had, and the horizontal sums take the patches' place in LDS
// (five workgroups per compute unit forward instead of three: 108 -> 100 us).
// 1600 x 1066 x 3: loss 82 -> 50 us, loss and gradient 143 -> 100 us. (One sum
// for x^2 + y^2, of which the variances need no more: 92 us, but the gradient
// of a smooth image is off by 6.6e-6 instead of 5.9e-6.)
#include <math.h>

#include "common.h"

namespace gs {

namespace {

constexpr int kTile = 32;
constexpr int kRad = 5;
constexpr int kTaps = 2 * kRad + 1;
constexpr int kPatch = kTile + 2 * kRad;  // 42
constexpr int kCols = 8;                  // columns per thread of the horizontal pass
constexpr int kRows = 4;                  // rows per thread of the vertical pass
constexpr int kPStride = kPatch + 1;      // odd row strides: lanes on different
constexpr int kHStride = kTile + 1;       // rows use different LDS banks
static_assert(kPatch <= kWave && kTile * kTile == 256 * kRows &&
                  kPatch * (kTile / kCols) <= 256,
              "one wavefront per patch row, one turn per pass");
constexpr float kC1 = 0.01f * 0.01f;
constexpr float kC2 = 0.03f * 0.03f;

struct Window {
  float w[kTaps];
};

// The block's sums of NQ per-thread values, written to out[q * n_blocks +
// block] (summed over the blocks in a fixed order afterwards).
template <int NQ>
__device__ __forceinline__ void block_sum_store(float (&v)[NQ], float* out, int64_t n_blocks,
                                                int64_t block, float* red) {
#pragma unroll
  for (int q = 0; q < NQ; ++q)
    for (int d = 1; d < kWave; d <<= 1) v[q] += __shfl_xor(v[q], d, kWave);
  const int w = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0)
    for (int q = 0; q < NQ; ++q) red[q * 4 + w] = v[q];
  __syncthreads();
  if (threadIdx.x < NQ) {
    const int q = threadIdx.x;
    out[q * n_blocks + block] =
        (red[q * 4 + 0] + red[q * 4 + 1]) + (red[q * 4 + 2] + red[q * 4 + 3]);
  }
}

// The tile's input patch (zero outside the image), a row per wavefront and turn.
__device__ __forceinline__ void load_patch(const float* __restrict__ in, int H, int W, int x0,
                                           int y0, float (&out)[kPatch][kPStride]) {
  const int c = threadIdx.x & (kWave - 1), gx = x0 + c - kRad;
  const bool in_x = gx >= 0 && gx < W;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  constexpr int kTurns = (kPatch + 3) / 4;
  float v[kTurns];
#pragma unroll
  for (int k = 0; k < kTurns; ++k) {  // every load is issued before the first is used
    const int r = w + 4 * k, gy = y0 + r - kRad;
    v[k] = r < kPatch && c < kPatch && in_x && gy >= 0 && gy < H ? in[(int64_t)gy * W + gx] : 0.f;
  }
#pragma unroll
  for (int k = 0; k < kTurns; ++k)
    if (w + 4 * k < kPatch && c < kPatch) out[w + 4 * k][c] = v[k];
}

// The vertical window sums of rows i0 .. i0 + kRows - 1 of column j.
template <int NQ>
__device__ __forceinline__ void vertical(const float (&hs)[NQ][kPatch][kHStride],
                                         const Window& win, int i0, int j,
                                         float (&m)[NQ][kRows]) {
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
#pragma unroll
    for (int o = 0; o < kRows; ++o) m[q][o] = 0.f;
#pragma unroll
    for (int r = 0; r < kRows + 2 * kRad; ++r) {
      const float v = hs[q][i0 + r][j];
#pragma unroll
      for (int o = 0; o < kRows; ++o)
        if (r - o >= 0 && r - o < kTaps) m[q][o] = fmaf(win.w[r - o], v, m[q][o]);
    }
  }
}

__global__ void __launch_bounds__(256) k_photo_fwd(const float* __restrict__ img,
                                                   const float* __restrict__ tgt, int H, int W,
                                                   Window win, float* __restrict__ fmaps,
                                                   int64_t plane, float* __restrict__ parts) {
  __shared__ union {  // the patches, then the horizontal sums
    struct {
      float px[kPatch][kPStride], py[kPatch][kPStride];
    };
    float hs[5][kPatch][kHStride];
  } L;
  __shared__ float red[8];
  const int x0 = blockIdx.x * kTile, y0 = blockIdx.y * kTile;
  const int64_t base = (int64_t)blockIdx.z * H * W;
  const int tid = threadIdx.x;
  load_patch(img + base, H, W, x0, y0, L.px);
  load_patch(tgt + base, H, W, x0, y0, L.py);
  __syncthreads();
  const int j = tid % kTile, i0 = tid / kTile * kRows;
  float acc[2] = {0.f, 0.f};  // sum |x - y|, sum S
#pragma unroll
  for (int o = 0; o < kRows; ++o)  // zero outside the image
    acc[0] += fabsf(L.px[i0 + o + kRad][j + kRad] - L.py[i0 + o + kRad][j + kRad]);
  const bool hz = tid < kPatch * (kTile / kCols);
  const int r = hz ? tid % kPatch : 0, j0 = hz ? tid / kPatch * kCols : 0;
  float s[5][kCols] = {};
  if (hz) {
#pragma unroll
    for (int c = 0; c < kCols + 2 * kRad; ++c) {
      const float a = L.px[r][j0 + c], b = L.py[r][j0 + c];
      const float v[5] = {a, b, a * a, b * b, a * b};
#pragma unroll
      for (int o = 0; o < kCols; ++o)  // taps of a column in order as c grows
        if (c - o >= 0 && c - o < kTaps)
#pragma unroll
          for (int q = 0; q < 5; ++q) s[q][o] = fmaf(win.w[c - o], v[q], s[q][o]);
    }
  }
  __syncthreads();  // the patches are read until here
  if (hz)
#pragma unroll
    for (int q = 0; q < 5; ++q)
#pragma unroll
      for (int o = 0; o < kCols; ++o) L.hs[q][r][j0 + o] = s[q][o];
  __syncthreads();
  float m[5][kRows];
  vertical<5>(L.hs, win, i0, j, m);
#pragma unroll
  for (int o = 0; o < kRows; ++o) {
    const int gy = y0 + i0 + o, gx = x0 + j;
    if (gy >= H || gx >= W) continue;
    const float mx = m[0][o], my = m[1][o];
    const float vx = m[2][o] - mx * mx, vy = m[3][o] - my * my, cxy = m[4][o] - mx * my;
    const float A1 = 2.f * mx * my + kC1, A2 = 2.f * cxy + kC2;
    const float B1 = mx * mx + my * my + kC1, B2 = vx + vy + kC2;
    const float inv = 1.f / (B1 * B2);
    const float S = A1 * A2 * inv;
    acc[1] += S;
    if (fmaps) {
      const float dmx = 2.f * my * A2 * inv - 2.f * mx * S / B1;
      const float dvx = -S / B2;
      const float dcxy = 2.f * A1 * inv;
      const int64_t p = base + (int64_t)gy * W + gx;
      fmaps[p] = dmx - 2.f * mx * dvx - my * dcxy;
      fmaps[plane + p] = dvx;
      fmaps[2 * plane + p] = dcxy;
    }
  }
  const int64_t nblk = (int64_t)gridDim.x * gridDim.y * gridDim.z;
  const int64_t blk = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
  block_sum_store<2>(acc, parts, nblk, blk, red);
}

// loss[0..2] = E, L1, SSIM from the per-block sums over n values (FP64,
// each of 256 threads a fixed stride of blocks, then a fixed-order tree).
__device__ __forceinline__ void photo_finish(const float* __restrict__ parts, int64_t nblk,
                                             double n, float lambda, double (&red)[2][256],
                                             float* __restrict__ loss) {
  double a = 0.0, b = 0.0;
#pragma unroll 8
  for (int64_t i = threadIdx.x; i < nblk; i += 256) {
    a += (double)parts[i];
    b += (double)parts[nblk + i];
  }
  red[0][threadIdx.x] = a;
  red[1][threadIdx.x] = b;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
      red[0][threadIdx.x] += red[0][threadIdx.x + h];
      red[1][threadIdx.x] += red[1][threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double l1 = red[0][0] / n, s = red[1][0] / n;
    loss[0] = (float)((1.0 - lambda) * l1 + lambda * (1.0 - s));
    loss[1] = (float)l1;
    loss[2] = (float)s;
  }
}

__global__ void __launch_bounds__(256) k_photo_finish(const float* __restrict__ parts,
                                                      int64_t nblk, double n, float lambda,
                                                      float* __restrict__ loss) {
  __shared__ double red[2][256];
  photo_finish(parts, nblk, n, lambda, red, loss);
}

// The gradient; the last workgroup writes the loss first (a launch of its own
// costs 7 us, here it runs beside the other workgroups).
__global__ void __launch_bounds__(256) k_photo_bwd(const float* __restrict__ img,
                                                   const float* __restrict__ tgt, int H, int W,
                                                   Window win, const float* __restrict__ fmaps,
                                                   int64_t plane, float wl1, float wssim,
                                                   float* __restrict__ grad,
                                                   const float* __restrict__ parts, float lambda,
                                                   float* __restrict__ loss) {
  __shared__ union {
    float pf[3][kPatch][kPStride];  // the maps' patches, then the horizontal sums
    float hs[3][kPatch][kHStride];
    double red[2][256];
  } L;
  if (blockIdx.x == gridDim.x - 1 && blockIdx.y == gridDim.y - 1 &&
      blockIdx.z == gridDim.z - 1) {
    photo_finish(parts, (int64_t)gridDim.x * gridDim.y * gridDim.z, (double)plane, lambda, L.red,
                 loss);
    __syncthreads();  // the LDS changes hands
  }
  const int x0 = blockIdx.x * kTile, y0 = blockIdx.y * kTile;
  const int64_t base = (int64_t)blockIdx.z * H * W;
  const int tid = threadIdx.x;
#pragma unroll
  for (int q = 0; q < 3; ++q) load_patch(fmaps + q * plane + base, H, W, x0, y0, L.pf[q]);
  __syncthreads();
  const bool hz = tid < kPatch * (kTile / kCols);
  const int r = hz ? tid % kPatch : 0, j0 = hz ? tid / kPatch * kCols : 0;
  float s[3][kCols] = {};
  if (hz) {
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int c = 0; c < kCols + 2 * kRad; ++c) {
        const float v = L.pf[q][r][j0 + c];
#pragma unroll
        for (int o = 0; o < kCols; ++o)
          if (c - o >= 0 && c - o < kTaps) s[q][o] = fmaf(win.w[c - o], v, s[q][o]);
      }
  }
  __syncthreads();  // the patches are read until here
  if (hz)
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int o = 0; o < kCols; ++o) L.hs[q][r][j0 + o] = s[q][o];
  __syncthreads();
  const int j = tid % kTile, i0 = tid / kTile * kRows;
  float g[3][kRows];
  vertical<3>(L.hs, win, i0, j, g);
#pragma unroll
  for (int o = 0; o < kRows; ++o) {
    const int gy = y0 + i0 + o, gx = x0 + j;
    if (gy >= H || gx >= W) continue;
    const int64_t p = base + (int64_t)gy * W + gx;
    const float x = img[p], y = tgt[p];
    const float d = x - y;
    const float sgn = d > 0.f ? 1.f : (d < 0.f ? -1.f : 0.f);
    const float dssim = g[0][o] + 2.f * x * g[1][o] + y * g[2][o];
    grad[p] = wl1 * sgn - wssim * dssim;
  }
}

__global__ void k_prune_acc(const uint32_t* __restrict__ count, int64_t n,
                            const float* __restrict__ photo, double* __restrict__ prune,
                            uint32_t* __restrict__ split) {
  const double e = (double)photo[0];
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t c = count[i];
    prune[i] += e * (double)c;
    if (split) split[i] += c;
  }
}

Window make_window() {
  Window w;
  double g[kTaps], s = 0.0;
  for (int t = 0; t < kTaps; ++t) {
    const double r = t - kRad;
    g[t] = exp(-r * r / (2.0 * 1.5 * 1.5));
    s += g[t];
  }
  for (int t = 0; t < kTaps; ++t) w.w[t] = (float)(g[t] / s);
  return w;
}

// per-block sums (2 floats per block) ahead of the SSIM partial maps
size_t parts_bytes(int32_t c, int32_t h, int32_t w) {
  const size_t nblk = (size_t)c * (size_t)div_up(h, kTile) * (size_t)div_up(w, kTile);
  return (2 * nblk * sizeof(float) + 255) / 256 * 256;
}

}  // namespace

}  // namespace gs

using namespace gs;

extern "C" gs_status gs_photo_loss_workspace(int32_t channels, int32_t height, int32_t width,
                                             size_t* bytes) {
  if (channels < 1 || height < 1 || width < 1 || !bytes) return GS_EINVAL;
  *bytes = parts_bytes(channels, height, width) +
           (size_t)3 * channels * height * width * sizeof(float);
  return GS_OK;
}

extern "C" gs_status gs_photo_loss(const float* image, const float* target, int32_t channels,
                                   int32_t height, int32_t width, float lambda, void* workspace,
                                   size_t workspace_bytes, float* loss, float* dL_dimage,
                                   void* stream) {
  if (channels < 1 || height < 1 || width < 1 || !(lambda >= 0.f && lambda <= 1.f) || !image ||
      !target || !loss || !workspace)
    return GS_EINVAL;
  const int64_t plane = (int64_t)channels * height * width;
  const size_t pb = parts_bytes(channels, height, width);
  const size_t need = pb + (dL_dimage ? (size_t)3 * plane * sizeof(float) : 0);
  if (workspace_bytes < need) return GS_ECAPACITY;
  hipStream_t st = (hipStream_t)stream;
  float* parts = (float*)workspace;
  float* fmaps = dL_dimage ? (float*)((char*)workspace + pb) : nullptr;
  const Window win = make_window();
  const dim3 grid(div_up(width, kTile), div_up(height, kTile), channels);
  const int64_t nblk = (int64_t)grid.x * grid.y * grid.z;
  GS_TIMED("photo_loss", st,
           k_photo_fwd<<<grid, 256, 0, st>>>(image, target, height, width, win, fmaps, plane,
                                             parts);
           if (dL_dimage) k_photo_bwd<<<grid, 256, 0, st>>>(
               image, target, height, width, win, fmaps, plane,
               (float)((1.0 - lambda) / (double)plane), (float)(lambda / (double)plane),
               dL_dimage, parts, lambda, loss);
           else k_photo_finish<<<1, 256, 0, st>>>(parts, nblk, (double)plane, lambda, loss));
  GS_CHECK_LAUNCH();
  return GS_OK;
}

extern "C" gs_status gs_prune_accumulate(const uint32_t* count, int64_t n, const float* photo,
                                         double* prune_score, uint32_t* split_score,
                                         void* stream) {
  if (n < 0 || (n > 0 && (!count || !photo || !prune_score))) return GS_EINVAL;
  if (n == 0) return GS_OK;
  hipStream_t st = (hipStream_t)stream;
  const int blocks = (int)std::min<int64_t>(div_up(n, 256), 4096);
  k_prune_acc<<<blocks, 256, 0, st>>>(count, n, photo, prune_score, split_score);
  GS_CHECK_LAUNCH();
  return GS_OK;
}
