// Per-tile compositing (Sec. 2.1, second step) and its backward (Sec. 2.2).
//
// Forward: one workgroup per tile; each lane owns PX pixels. The tile's
// sorted splat records are gathered through `vals` into LDS in batches;
// every wavefront walks the batch's splats that reach its pixels front to
// back. The workgroup stops as soon as every pixel has reached T < 1e-4.
//
// Backward: one wavefront per region of a tile, PX pixels per lane, walking the
// tile's list back to front from each pixel's last contributor. The transmittance
// in front of each splat is recomputed as T / (1 - alpha) from the stored
// final transmittance (nothing per splat is stored by the forward), and the
// colour and depth behind it are accumulated on the way. The per-splat
// gradient components are summed over the wavefront and parked in LDS, and
// after each batch one FP64 atomic add per (splat, component) carries the
// region's total.
//
// The FP32 arithmetic here may be contracted to FMAs; alpha is computed by
// the same expression (explicit fmaf) in both kernels, so the backward
// replays exactly the forward's alphas.
#include <math.h>

#include <type_traits>

#include "binning.h"
#include "common.h"
#include "sort.h"

namespace gs {

constexpr float kAlphaMax = 0.99f;
constexpr float kTStop = 1e-4f;
constexpr float kNegHalfLog2e = -0.72134752044448170f;  // -log2(e) / 2

// G = exp(-Q/2) as one v_exp_f32
__device__ __forceinline__ float gauss(float Q) {
  return __builtin_amdgcn_exp2f(Q * kNegHalfLog2e);
}

struct SplatQ {
  float Q, mag, dx, dy;
};

__device__ __forceinline__ SplatQ eval_q(float px, float py, float u, float v, float a, float b2,
                                         float c) {
  SplatQ r;
  r.dx = px - u;
  r.dy = py - v;
  const float s1 = a * r.dx;
  const float t1 = c * r.dy;
  const float td = t1 * r.dy;
  r.Q = fmaf(r.dx, fmaf(b2, r.dy, s1), td);
  r.mag = fmaf(s1, r.dx, td);
  return r;
}

// q > t in FP64, the definition of the skip decision.
__device__ __forceinline__ bool skips_f64(float t, float px, float py, float u, float v, float a,
                                          float b, float c) {
#pragma clang fp contract(off)
  const double dx = (double)px - (double)u;
  const double dy = (double)py - (double)v;
  const double q = dx * ((double)a * dx + 2.0 * ((double)b * dy)) + dy * ((double)c * dy);
  return q > (double)t;
}

__device__ __attribute__((noinline)) bool splat_skips_exact(float t, float px, float py, float u,
                                                            float v, float a, float b, float c) {
  return skips_f64(t, px, py, u, v, a, b, c);
}

// Which cells of a tile a splat can blend in. A cell is a block of CW x CH
// pixels, one per lane of a wavefront; the splat is left out of a cell when
// Q > t at all of its pixel centres, so leaving it out changes nothing.
//
// The smallest Q over the cell's rectangle of pixel centres lies on one of
// its edges that face the centroid (Q grows along every ray from it), and on
// an edge at -b d / c (or / a) clamped to it, so
// two evaluations of Q give it; any other point of the rectangle would give a
// larger value, so an inexact minimiser errs by the square of its error. The
// FP32 value is within 8 u (1 + r) / (1 - r) of the exact one, relatively
// (the bound of skip_band, the minimiser and the rectangle's own rounding
// included), and the band is 16 u (1 + r) / (1 - r) t: a value above
// t + band means Q > t at every pixel centre of the cell. An infinite band
// (degenerate and non-finite records) keeps every cell.
//
// What it saves: a splat of a trained scene covers a few pixels, so it blends
// in 8 to 25% of its tile's pixels and reaches 1.7 to 2.5 of a 16-pixel tile's
// four cells (measured at 123k to 1M Gaussians of about their spacing's size;
// 3.8 on the surface scene).
template <int CW, int CH>
__device__ __forceinline__ bool cell_reached(float x0, float y0, float u, float v, float a,
                                             float b2, float c, float kx, float ky, float lim) {
#pragma clang fp contract(fast)
  const float dx0 = x0 + 0.5f - u, dx1 = x0 + ((float)CW - 0.5f) - u;
  const float dy0 = y0 + 0.5f - v, dy1 = y0 + ((float)CH - 0.5f) - v;
  const float ex = __builtin_amdgcn_fmed3f(0.f, dx0, dx1);  // the facing edges
  const float ey = __builtin_amdgcn_fmed3f(0.f, dy0, dy1);
  const float y = __builtin_amdgcn_fmed3f(ky * ex, dy0, dy1);
  const float x = __builtin_amdgcn_fmed3f(kx * ey, dx0, dx1);
  const float q1 = fmaf(ex, fmaf(b2, y, a * ex), (c * y) * y);
  const float q2 = fmaf(x, fmaf(b2, ey, a * x), (c * ey) * ey);
  return !(fminf(q1, q2) > lim);
}

// Bit i: cell i of the tile at (x0, y0) is reached; X(i), Y(i) the cell's
// pixel offsets in the tile.
template <int CW, int CH, int NCELL, class CellX, class CellY>
__device__ __forceinline__ uint32_t cells_reached(float x0, float y0, float4 r0, float c, float t,
                                                  float band, CellX X, CellY Y) {
  const float a = r0.z, b = r0.w;
  const float ky = -b * __builtin_amdgcn_rcpf(c), kx = -b * __builtin_amdgcn_rcpf(a);
  // centroids out of the range in which the squares below stay finite: every cell
  const float lim = fabsf(r0.x) + fabsf(r0.y) < 1e15f ? t + band : __builtin_huge_valf();
  const float b2 = b + b;
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < NCELL; ++i)
    if (cell_reached<CW, CH>(x0 + (float)X(i), y0 + (float)Y(i), r0.x, r0.y, a, b2, c, kx, ky,
                             lim))
      m |= 1u << i;
  return m;
}

// A splat whose colour or depth is not finite (or so large that their sum is
// not) has to leave the pixels that do not blend it as they are, which a weight
// of 0 does not. A wavefront whose batch of the list holds such a splat
// walks that batch splat by splat, under the mask of the pixels that blend it.
// (The mask in the ordinary walk costs the forward 2 to 15%, a branch around
// the odd splats of a group 1 to 12%, a walk of its own under 1%.)
constexpr uint32_t kOddSplat = 1u << 31;  // among the cells' bits
__device__ __forceinline__ bool odd_splat(float4 r1, float4 r2) {  // (c, t, o, z), (r, g, b, -)
  return !(fabsf(r2.x) + fabsf(r2.y) + fabsf(r2.z) + fabsf(r1.w) < __builtin_huge_valf());
}

// 2 x + (the lane's bit of m), one instruction.
__device__ __forceinline__ uint32_t shift_in(uint32_t x, uint64_t m) {
  uint32_t r;
  uint64_t carry;
  asm("v_addc_co_u32 %0, %1, %2, %2, %3" : "=v"(r), "=s"(carry) : "v"(x), "s"(m));
  return r;
}

constexpr int kFwdBatch = 256;  // splats per LDS batch in the forward (default)
constexpr int kFwdGroup = 4;    // splats a wavefront evaluates together (fwd_tile)
// A batch in LDS, and per wavefront the byte offsets (16 per entry) of the
// batch's splats that reach its cells. Entry NB holds a splat that blends
// nowhere: it fills up a wavefront's last group.
template <int NB, int NTH>
struct FwdLdsT {
  // (u, v, a, 2 b), (c, t - band, t + band, o), (r, g, b, z)
  float4 s0[NB + 1], s1[NB + 1], s2[NB + 1];
  float t[NB + 1];
  uint32_t cells[NB + 1];
  alignas(16) uint32_t list[NTH / kWave][NB + kFwdGroup];
};

// The forward's cells: 8 x 8 pixels, one per lane (lane l at column l % 8 and
// row l / 8), numbered along a Z curve over the tile; wavefront w holds cells
// w PX .. w PX + PX - 1.
struct FwdCells {
  __host__ __device__ static constexpr int x(int i) { return 8 * ((i & 1) | ((i >> 1) & 2)); }
  __host__ __device__ static constexpr int y(int i) {
    return 8 * (((i >> 1) & 1) | ((i >> 2) & 2));
  }
};

// Stage the record of Gaussian g (g >= n: a splat that blends nowhere, since
// its t < 0 skips it) as entry q, with the cells of the TILE x TILE tile at
// (x0, y0) that it reaches (and kOddSplat).
template <int TILE, class Lds>
__device__ __forceinline__ void fwd_stage(Lds& L, int q, const float* __restrict__ splats,
                                          uint32_t g, int64_t n, float x0, float y0) {
  float4 r0 = make_float4(0.f, 0.f, 1.f, 0.f), r1 = make_float4(1.f, -1.f, 0.f, 0.f);
  float4 r2 = make_float4(0.f, 0.f, 0.f, 0.f);
  float band = 0.f;
  uint32_t cells = 0;
  if ((int64_t)g < n) {
    const float4* r = reinterpret_cast<const float4*>(splats + (size_t)g * GS_SPLAT_FLOATS);
    r0 = r[0];
    r1 = r[1];
    r2 = r[2];
    band = skip_band(r0.z, r0.w, r1.x, r1.y);
    cells = cells_reached<8, 8, TILE * TILE / 64>(x0, y0, r0, r1.x, r1.y, band, FwdCells::x,
                                                  FwdCells::y);
  }
  L.t[q] = r1.y;
  L.cells[q] = (int64_t)g < n && odd_splat(r1, r2) ? cells | kOddSplat : cells;
  L.s0[q] = make_float4(r0.x, r0.y, r0.z, r0.w + r0.w);  // exact
  L.s1[q] = make_float4(r1.x, r1.y - band, r1.y + band, r1.z);
  L.s2[q] = make_float4(r2.x, r2.y, r2.z, r1.w);
}

// The forward that writes its tile lists (from the binning's column runs):
// the batch's Gaussian ids and the block-scan words.
template <int NB, int NTH>
struct DefLds {
  static constexpr int R = 2;  // runs per thread per scan step
  uint32_t sid[NB];
  uint32_t wcnt[2][R][NTH / kWave];  // per-wavefront counts, double-buffered by step
  uint32_t next;
};

// Where a tile's list continues in the column runs: segment `seg` (global
// index), its next run r and run end r1, and the next list position pos.
// The column's segments sf .. se - 1 and runs c0 .. c1 - 1; a window of NTH
// segments from wb on, thread t holding the first list position in row ty
// of segment wb + t (hs; 0xFFFFFFFF past se).
struct DefCursor {
  uint32_t seg, r, r1, pos;
  uint32_t sf, se, c0, c1, wb, hs;
};

__device__ __forceinline__ void def_window(const RunLists& rl, DefCursor& c, int tiles_y, int ty) {
  const uint32_t s = c.wb + threadIdx.x;
  c.hs = s < c.se ? rl.hist[(int64_t)s * tiles_y + ty] : 0xFFFFFFFFu;
}

// Point the cursor at the segment holding list position pos of row ty: the
// last one whose first position in the row is at most pos (a segment with
// no entry in the row shares its first position with the next one), found
// with one block count over the window (moved on when the whole window lies
// at or below pos). se if that is below min_seg (the seek always moves
// forward), which happens only on a list that the run tables do not hold
// (never for tables of the same binning).
template <int NTH>
__device__ __forceinline__ void def_seek(const RunLists& rl, DefCursor& c, int tiles_y, int ty,
                                         uint32_t pos, uint32_t min_seg) {
  uint32_t seg;
  for (;;) {
    const uint32_t k = __builtin_amdgcn_readfirstlane(
        (uint32_t)__syncthreads_count(c.hs <= pos));  // leading segments (monotone)
    if (k == (uint32_t)NTH && c.wb + NTH < c.se) {
      c.wb += NTH;
      def_window(rl, c, tiles_y, ty);
      continue;
    }
    seg = k > 0 && c.wb + k - 1 >= min_seg ? c.wb + k - 1 : c.se;
    break;
  }
  c.seg = seg;
  c.pos = pos;
  if (seg < c.se) {
    c.r = c.c0 + (seg - c.sf) * (uint32_t)kSegRuns;
    c.r1 = min(c.r + (uint32_t)kSegRuns, c.c1);
  } else {
    c.r = c.r1 = 0;
  }
}

// The cursor of a tile (column tx, row ty) at its first list position.
template <int NTH>
__device__ __forceinline__ void def_start(const RunLists& rl, DefCursor& c, int tx, int tiles_y,
                                          int ty, uint32_t start) {
  c.sf = rl.segfirst[tx];
  c.se = rl.segfirst[tx + 1];
  c.c0 = rl.cstart[tx];
  c.c1 = rl.cstart[tx + 1];
  c.wb = c.sf;
  def_window(rl, c, tiles_y, ty);
  def_seek<NTH>(rl, c, tiles_y, ty, start, c.sf);
}

// The next cnt entries of the tile's list (row ty of column tx): the runs
// from the cursor on that cover row ty, in run order (= list order), into
// L.sid[0 .. cnt) and vals[c.pos ..]. Each step scans R NTH runs (run
// c.r + k NTH + t in slot k of thread t) with one barrier: the per-wavefront
// counts alternate between two buffers, so a step's counts are not
// overwritten before every thread has read them. A run left over when the
// batch fills is taken by the next batch. Entries that the tables do not
// hold (never for tables of the same binning) get the id 0xFFFFFFFF, an
// absent splat.
template <int NB, int NTH>
__device__ __forceinline__ void def_fill(const RunLists& rl, DefLds<NB, NTH>& D, DefCursor& c,
                                         int tx, int tiles_y, int ty, int cnt,
                                         uint32_t* __restrict__ vals) {
  constexpr int R = DefLds<NB, NTH>::R, NW = NTH / kWave;
  const int lane = threadIdx.x & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int filled = 0, buf = 0;
  bool full = false;
  while (filled < cnt) {
    if (c.r >= c.r1) {  // segment used up: the one holding the next position
      if (c.seg >= c.se) break;
      def_seek<NTH>(rl, c, tiles_y, ty, c.pos, c.seg + 1);
      if (c.seg >= c.se) break;
    }
    bool cov[R];
    uint32_t gid[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {  // loads first
      const uint32_t rr = c.r + k * NTH + threadIdx.x;
      const uint2 q = rr < c.r1 ? rl.runs[rr] : make_uint2(0u, 0u);
      gid[k] = q.x;
      cov[k] = (uint32_t)ty - (q.y & 0xFFFFu) < (q.y >> 16);
    }
    uint64_t bal[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      bal[k] = __ballot(cov[k]);
      if (lane == 0) D.wcnt[buf][k][w] = (uint32_t)__popcll(bal[k]);
    }
    __syncthreads();
    // the counts are uniform (per block, and below w per wavefront): scalar
    uint32_t total = 0, rank[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      uint32_t before = 0, tk = 0;
#pragma unroll
      for (int v = 0; v < NW; ++v) {
        const uint32_t x = __builtin_amdgcn_readfirstlane(D.wcnt[buf][k][v]);
        before += v < w ? x : 0u;
        tk += x;
      }
      rank[k] = total + before +
                __builtin_amdgcn_mbcnt_hi((uint32_t)(bal[k] >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)bal[k], 0u));
      total += tk;
    }
    const uint32_t need = (uint32_t)(cnt - filled);
    const uint32_t take = min(total, need);
#pragma unroll
    for (int k = 0; k < R; ++k) {
      if (cov[k] && rank[k] < take) {
        D.sid[filled + (int)rank[k]] = gid[k];
        vals[c.pos + rank[k]] = gid[k];
      }
      if (cov[k] && rank[k] == take) D.next = (uint32_t)(k * NTH) + threadIdx.x;  // first not taken
    }
    c.pos += take;
    filled += (int)take;
    buf ^= 1;
    if (total > need) {
      full = true;
      break;
    }
    c.r = min(c.r + (uint32_t)(R * NTH), c.r1);
  }
  for (int q = filled + (int)threadIdx.x; q < cnt; q += NTH) D.sid[q] = 0xFFFFFFFFu;
  __syncthreads();
  if (full) c.r += __builtin_amdgcn_readfirstlane(D.next);
}

// Checkpoints of the per-splat backward (the design the paper adopts): the
// forward state (T, C0, C1, C2, D) of every pixel before list positions 0,
// 32, 64, ..., laid out [tile][bucket][5][TILE * TILE].
constexpr int kCkptInterval = 32;
constexpr int kCkptVals = 5;

// Forward of one tile (column-major id `tile`) by the whole workgroup; with
// CKPT it also writes the checkpoints of the pixels still compositing at
// each interval boundary below nbk buckets, and sets *ovf if a pixel blends
// a splat at a list position of bucket nbk or later.
// With DEF the lists come from the binning's run tables `rl` (deferred
// binning) and the forward writes each batch's entries to `dvals` (vals is
// not read): every list position up to the last one staged, which covers
// every pixel's n_contrib.
//
// What bounds it: VALU issue where the lists are dense (27 operations per
// pixel and splat; at 1M Gaussians of the surface scene a splat of a list
// reaches 96% of its tile's cells), and the serial walk of the longest lists
// where splats are small (a third to a half of the cells reached). So a
// wavefront owns whole 8 x 8 cells and walks only the splats that reach them,
// four at a time: the shapes, Q and alpha of one splat do not wait for the
// blend of the one before, and the colours are read into the registers that
// the shapes needed. Decisions are 64-bit lane masks in scalar registers, and
// the position of a pixel's last blend is one bit per splat walked. Against
// one splat per step over 16 x 4 strips, all of the list: 393 -> 299 us at
// 1920x1080, 344 -> 254 us at 1600x1066 (1M Gaussians, lists as the binning
// left them), 332 -> 138 us at 300k Gaussians of about their spacing's size.
// Groups of two: 303, 260 and 151 us; four with the colours read together
// with the shapes (96 registers): 321, 281 and 133 us.
template <int TILE, int PX, bool CKPT = false, int NB = kFwdBatch, bool DEF = false>
__device__ __forceinline__ void fwd_tile(FwdLdsT<NB, TILE * TILE / PX>& L, int tile,
                                         const float* __restrict__ splats,
                                         const uint32_t* __restrict__ vals,
                                         const uint32_t* __restrict__ ranges, int64_t n, int W,
                                         int H, int tiles_y, float bg0, float bg1, float bg2,
                                         float* __restrict__ image, float* __restrict__ depth,
                                         float* __restrict__ T_final,
                                         uint32_t* __restrict__ n_contrib,
                                         float* __restrict__ ckpt = nullptr, int nbk = 0,
                                         uint32_t* __restrict__ ovf = nullptr,
                                         DefLds<NB, TILE * TILE / PX>* DL = nullptr,
                                         RunLists rl = {}, uint32_t* __restrict__ dvals = nullptr) {
#pragma clang fp contract(fast)
  constexpr int NTH = TILE * TILE / PX;
  constexpr int G = kFwdGroup;
  static_assert(G == 4 && NB % G == 0, "a group's list entries are one 16-byte word");
  const int tx = tile / tiles_y, ty = tile % tiles_y;
  const float x0 = (float)(tx * TILE), y0 = (float)(ty * TILE);
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  uint32_t* const list = L.list[wv];
  const uint32_t start = ranges[tile], end = ranges[tile + 1];
  float px[PX], py[PX], T[PX], C0[PX], C1[PX], C2[PX], D[PX];
  uint32_t last[PX];   // one past the list position of the last blended splat
  uint64_t done[PX];   // the lanes whose pixel j takes no more splats
  bool alldone = true;  // uniform
#pragma unroll
  for (int j = 0; j < PX; ++j) {
    const int x = tx * TILE + FwdCells::x(wv * PX + j) + lane % 8;
    const int y = ty * TILE + FwdCells::y(wv * PX + j) + lane / 8;
    px[j] = (float)x + 0.5f;
    py[j] = (float)y + 0.5f;
    T[j] = 1.f; C0[j] = C1[j] = C2[j] = D[j] = 0.f; last[j] = 0;
    done[j] = __ballot(!(x < W && y < H));
    alldone = alldone && done[j] == ~0ull;
  }
  if (threadIdx.x == 0) fwd_stage<TILE>(L, NB, splats, 0u, 0, 0.f, 0.f);  // the filler
  DefCursor cur{};
  if constexpr (DEF) {
    if (start < end) def_start<NTH>(rl, cur, tx, tiles_y, ty, start);
  }
  for (uint32_t b = start; b < end; b += NB) {
    if (__syncthreads_count(!alldone) == 0) break;
    const int cnt = (int)min((uint32_t)NB, end - b);
    if constexpr (DEF) def_fill<NB, NTH>(rl, *DL, cur, tx, tiles_y, ty, cnt, dvals);
    for (int q = threadIdx.x; q < cnt; q += NTH) {
      uint32_t g;
      if constexpr (DEF) g = DL->sid[q]; else g = vals[b + q];
      fwd_stage<TILE>(L, q, splats, g, n, x0, y0);
    }
    __syncthreads();
    if (alldone) continue;
    // the wavefront's list: the splats that reach its cells, in order (with
    // CKPT every splat, since a checkpoint is due at fixed positions)
    int m = 0;
    uint64_t odd = 0;
    for (int base = 0; base < cnt; base += kWave) {
      constexpr uint32_t kMine = (1u << PX) - 1u;
      const int q = base + lane;
      const uint32_t cells = L.cells[min(q, NB)];
      const bool reach = q < cnt && (CKPT || ((cells >> (wv * PX)) & kMine) != 0u);
      const uint64_t bal = __ballot(reach);
      odd |= __ballot(reach && (cells & kOddSplat) != 0u);
      if (reach)
        list[m + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                           __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u))] =
            16u * (uint32_t)q;
      m += (int)__popcll(bal);
    }
    if (lane < G) list[m + lane] = 16u * NB;
    __builtin_amdgcn_wave_barrier();  // a wavefront's LDS operations complete in order
    const uint32_t rel = b - start;
    // the checkpoint due before the splat at list position pos, if any
    const auto checkpoint = [&](uint32_t pos) {
      if (!CKPT || pos % kCkptInterval != 0) return;
      const uint32_t bk = pos / kCkptInterval;
#pragma unroll
      for (int j = 0; j < PX; ++j) {
        if (__builtin_amdgcn_inverse_ballot_w64(done[j]) || bk >= (uint32_t)nbk) continue;
        constexpr int NP = TILE * TILE;
        const int pi = (FwdCells::y(wv * PX + j) + lane / 8) * TILE + FwdCells::x(wv * PX + j) +
                       lane % 8;
        float* c = ckpt + ((size_t)tile * nbk + bk) * kCkptVals * NP + pi;
        c[0] = T[j];
        c[NP] = C0[j];
        c[2 * NP] = C1[j];
        c[3 * NP] = C2[j];
        c[4 * NP] = D[j];
      }
    };
    if (odd != 0) {  // splat by splat, the same operations in the same order
#pragma unroll 1
      for (int i = 0; i < m && !alldone; ++i) {
        const int q = (int)(list[i] / 16u);
        const uint32_t pos = rel + (uint32_t)q;
        const float4 a0 = L.s0[q], a1 = L.s1[q], a2 = L.s2[q];
        checkpoint(pos);
        alldone = true;
#pragma unroll
        for (int j = 0; j < PX; ++j) {
          const float Q = eval_q(px[j], py[j], a0.x, a0.y, a0.z, a0.w, a1.x).Q;
          uint64_t skip = __ballot(Q > a1.z);
          if (~(skip | __ballot(Q <= a1.y)) != 0)
            skip = __ballot(skips_f64(L.t[q], px[j], py[j], a0.x, a0.y, a0.z, 0.5f * a0.w, a1.x));
          const float al = fminf(kAlphaMax, a1.w * gauss(Q));
          const float Tn = T[j] * (1.f - al);
          const uint64_t low = __ballot(Tn < kTStop);
          const uint64_t none = skip | done[j] | low;  // no blend
          done[j] |= low & ~skip;
          if (!__builtin_amdgcn_inverse_ballot_w64(none)) {
            const float w = al * T[j];
            C0[j] = fmaf(a2.x, w, C0[j]);
            C1[j] = fmaf(a2.y, w, C1[j]);
            C2[j] = fmaf(a2.z, w, C2[j]);
            D[j] = fmaf(a2.w, w, D[j]);
            T[j] = Tn;
            last[j] = pos + 1u;
            if (CKPT && pos >= (uint32_t)nbk * kCkptInterval) atomicOr(ovf, 1u);
          }
          alldone = alldone && done[j] == ~0ull;
        }
      }
      continue;
    }
    for (int i0 = 0; i0 < m && !alldone; i0 += 32) {
      const int i1 = min(i0 + 32, m);
      uint32_t hist[PX];  // per splat walked, newest in bit 0: not blended
#pragma unroll
      for (int j = 0; j < PX; ++j) hist[j] = ~0u;
      int i = i0;
      for (; i < i1 && !alldone; i += G) {
        uint32_t off[G];
        float4 a0[G], a1[G], a2[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
          off[g] = list[i + g];
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
          a0[g] = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(L.s0) + off[g]);
          a1[g] = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(L.s1) + off[g]);
        }
        float Q[G][PX];
        uint64_t skip[G][PX], near = 0;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int j = 0; j < PX; ++j) {
            Q[g][j] = eval_q(px[j], py[j], a0[g].x, a0[g].y, a0[g].z, a0[g].w, a1[g].x).Q;
            skip[g][j] = __ballot(Q[g][j] > a1[g].z);
            near |= ~(skip[g][j] | __ballot(Q[g][j] <= a1[g].y));
          }
        if (near != 0) {  // a few groups in a thousand: the FP64 decision
          asm volatile("");  // not to be computed ahead of the branch
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const int q = (int)(off[g] / 16u);
            const float4 e0 = L.s0[q], e1 = L.s1[q];
            const float t = L.t[q];
#pragma unroll
            for (int j = 0; j < PX; ++j)
              skip[g][j] =
                  __ballot(skips_f64(t, px[j], py[j], e0.x, e0.y, e0.z, 0.5f * e0.w, e1.x));
          }
        }
        // the colours are read only now, into the registers that the shapes
        // needed until here, while alpha is formed
#pragma unroll
        for (int g = 0; g < G; ++g)
          a2[g] = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(L.s2) + off[g]);
        float al[G][PX];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int j = 0; j < PX; ++j) al[g][j] = fminf(kAlphaMax, a1[g].w * gauss(Q[g][j]));
#pragma unroll
        for (int g = 0; g < G; ++g) {
          if (CKPT && off[g] < 16u * NB) checkpoint(rel + off[g] / 16u);
          // the step in select form: every pixel runs it, and a skipped,
          // stopped or finished pixel changes nothing (no divergent branches)
          alldone = true;
#pragma unroll
          for (int j = 0; j < PX; ++j) {
            const float Tn = T[j] * (1.f - al[g][j]);
            const uint64_t low = __ballot(Tn < kTStop);
            const uint64_t none = skip[g][j] | done[j] | low;  // no blend
            done[j] |= low & ~skip[g][j];
            const bool nb = __builtin_amdgcn_inverse_ballot_w64(none);
            // weight 0 when not blending: adding c * 0 leaves the sums unchanged
            // (c is finite: no odd splat here)
            const float w = nb ? 0.f : al[g][j] * T[j];
            C0[j] = fmaf(a2[g].x, w, C0[j]);
            C1[j] = fmaf(a2[g].y, w, C1[j]);
            C2[j] = fmaf(a2[g].z, w, C2[j]);
            D[j] = fmaf(a2[g].w, w, D[j]);
            T[j] = nb ? T[j] : Tn;
            hist[j] = shift_in(hist[j], none);
            // a blend in a bucket without a checkpoint: the backward would need it
            if (CKPT && !nb && rel + off[g] / 16u >= (uint32_t)nbk * kCkptInterval)
              atomicOr(ovf, 1u);
            alldone = alldone && done[j] == ~0ull;
          }
        }
      }
      // the newest clear bit of hist is the last blend: the splat that many
      // before the last one walked
#pragma unroll
      for (int j = 0; j < PX; ++j)
        if (~hist[j] != 0u) last[j] = rel + list[i - 1 - __builtin_ctz(~hist[j])] / 16u + 1u;
    }
  }
  const size_t HW = (size_t)H * W;
#pragma unroll
  for (int j = 0; j < PX; ++j) {
    const int x = tx * TILE + FwdCells::x(wv * PX + j) + lane % 8;
    const int y = ty * TILE + FwdCells::y(wv * PX + j) + lane / 8;
    if (x < W && y < H) {
      const size_t p = (size_t)y * W + x;
      image[p] = fmaf(T[j], bg0, C0[j]);
      image[HW + p] = fmaf(T[j], bg1, C1[j]);
      image[2 * HW + p] = fmaf(T[j], bg2, C2[j]);
      depth[p] = D[j];
      T_final[p] = T[j];
      n_contrib[p] = last[j];
    }
  }
}

// Wavefronts per SIMD the forward is compiled for. 7 (72 registers, nothing
// spilled) against 8 (64, a few registers of the staging spilled) at 16-pixel
// tiles: 299 against 300 us on the 1920x1080 view of the surface scene, 138
// against 145 us at 300k Gaussians of about their spacing's size. 32-pixel
// tiles have 16 wavefronts to a workgroup: two of them need 8 (372 against 455
// us with one). With several pixels per lane the registers of the ordinary walk
// decide, and the walk of odd splats has to do with as many (32-pixel tiles, four
// pixels, lists given: 3 and 142 registers 355 us, 4 and 128 339 us on the surface
// scene).
constexpr int fwd_waves(int tile, int px, bool lists = false) {
  return px == 4 ? (lists ? 4 : 3) : px == 2 ? 1 : tile == 32 ? 8 : 7;
}

template <int TILE, int PX>
__global__ void __launch_bounds__(TILE* TILE / PX)
__attribute__((amdgpu_waves_per_eu(fwd_waves(TILE, PX, true)))) k_render_fwd(
    const float* __restrict__ splats, const uint32_t* __restrict__ vals,
    const uint32_t* __restrict__ ranges, int64_t n, int W, int H, int tiles_y, float bg0,
    float bg1, float bg2, float* __restrict__ image, float* __restrict__ depth,
    float* __restrict__ T_final, uint32_t* __restrict__ n_contrib) {
  __shared__ FwdLdsT<kFwdBatch, TILE * TILE / PX> L;
  fwd_tile<TILE, PX>(L, blockIdx.x, splats, vals, ranges, n, W, H, tiles_y, bg0, bg1, bg2, image,
                     depth, T_final, n_contrib);
}

template <int TILE, int PX>
__global__ void __launch_bounds__(TILE* TILE / PX)
__attribute__((amdgpu_waves_per_eu(fwd_waves(TILE, PX)))) k_render_fwd_def(
    const float* __restrict__ splats, RunLists rl, uint32_t* __restrict__ vals,
    const uint32_t* __restrict__ ranges, int64_t n, int W, int H, int tiles_y, float bg0,
    float bg1, float bg2, float* __restrict__ image, float* __restrict__ depth,
    float* __restrict__ T_final, uint32_t* __restrict__ n_contrib) {
  __shared__ FwdLdsT<kFwdBatch, TILE * TILE / PX> L;
  __shared__ DefLds<kFwdBatch, TILE * TILE / PX> DL;
  fwd_tile<TILE, PX, false, kFwdBatch, true>(L, blockIdx.x, splats, nullptr, ranges, n, W, H,
                                             tiles_y, bg0, bg1, bg2, image, depth, T_final,
                                             n_contrib, nullptr, 0, nullptr, &DL, rl, vals);
}

__global__ void __launch_bounds__(256) k_render_fwd_ckpt(
    const float* __restrict__ splats, const uint32_t* __restrict__ vals,
    const uint32_t* __restrict__ ranges, int64_t n, int W, int H, int tiles_y, float bg0,
    float bg1, float bg2, float* __restrict__ image, float* __restrict__ depth,
    float* __restrict__ T_final, uint32_t* __restrict__ n_contrib, float* __restrict__ ckpt,
    int nbk, uint32_t* __restrict__ ovf) {
  __shared__ FwdLdsT<kFwdBatch, 256> L;
  fwd_tile<16, 1, true>(L, blockIdx.x, splats, vals, ranges, n, W, H, tiles_y, bg0, bg1, bg2,
                        image, depth, T_final, n_contrib, ckpt, nbk, ovf);
}

// Inclusive scans over each half (32 lanes) of the wavefront with DPP: row
// shifts within 16-lane rows, then row 0 (2) carried into row 1 (3).
__device__ __forceinline__ float half_incl_sum(float x) {
  x += dpp_mov<0x111>(0.f, x);
  x += dpp_mov<0x112>(0.f, x);
  x += dpp_mov<0x114>(0.f, x);
  x += dpp_mov<0x118>(0.f, x);
  x += dpp_mov<0x142, 0xa>(0.f, x);
  return x;
}
__device__ __forceinline__ float half_incl_prod(float x) {
  x *= dpp_mov<0x111>(1.f, x);
  x *= dpp_mov<0x112>(1.f, x);
  x *= dpp_mov<0x114>(1.f, x);
  x *= dpp_mov<0x118>(1.f, x);
  x *= dpp_mov<0x142, 0xa>(1.f, x);
  return x;
}
// the value of the next lower lane of the half (1 for its first lane)
__device__ __forceinline__ float half_shift_prod(float x, int lane) {
  const float y = dpp_mov<0x138>(1.f, x);  // wave_shr:1
  return (lane & 31) ? y : 1.f;
}

// Per-splat backward with checkpoints (the paper's design, as an ablation of
// the pixel-parallel backward below): one workgroup per 16 x 16 tile; each
// wavefront takes buckets of 32 list positions, one splat per lane of each
// half, and walks the tile's pixels two at a time (one per half). A lane
// rebuilds the transmittance in front of its splat from the bucket's
// checkpoint and the product of (1 - alpha) over the lower lanes, and the
// colour behind it from the image minus the checkpoint colour and the
// blended colour of the lanes up to it (DPP scans), and accumulates its
// splat's gradient over all pixels in registers (as moments for the conic
// and centroid); the halves are combined and each (splat, tile) gets one
// atomic per component.
template <bool DEPTH>
__global__ void __launch_bounds__(256) k_render_bwd_ckpt(
    const float* __restrict__ splats, const uint32_t* __restrict__ vals,
    const uint32_t* __restrict__ ranges, int W, int H, int tiles_y,
    const float* __restrict__ image, const float* __restrict__ depth,
    const uint32_t* __restrict__ n_contrib, const float* __restrict__ ckpt, int nbk,
    const float* __restrict__ dL_dimage, const float* __restrict__ dL_ddepth,
    double* __restrict__ grad2d, int64_t n) {
#pragma clang fp contract(fast)
  constexpr int TILE = 16, NP = TILE * TILE;
  __shared__ float pim[3][NP], pdc[3][NP], pdep[NP], pdd[NP];
  __shared__ uint32_t pnc[NP];
  __shared__ uint32_t smax;
  const int tile = blockIdx.x;
  const int tx = tile / tiles_y, ty = tile % tiles_y;
  const uint32_t start = ranges[tile], end = ranges[tile + 1];
  const size_t HW = (size_t)H * W;
  {
    const int t = threadIdx.x;
    const int x = tx * TILE + t % TILE, y = ty * TILE + t / TILE;
    const bool in = x < W && y < H;
    const size_t p = (size_t)y * W + x;
    pnc[t] = in ? n_contrib[p] : 0u;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      pim[c][t] = in ? image[c * HW + p] : 0.f;
      pdc[c][t] = in ? dL_dimage[c * HW + p] : 0.f;
    }
    pdep[t] = (DEPTH && in) ? depth[p] : 0.f;
    pdd[t] = (DEPTH && in && dL_ddepth) ? dL_ddepth[p] : 0.f;
    if (t == 0) smax = 0;
    __syncthreads();
    if (pnc[t]) atomicMax(&smax, pnc[t]);
    __syncthreads();
  }
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const int h = lane >> 5;
  const uint32_t nbt = (smax + kCkptInterval - 1) / kCkptInterval;
  for (uint32_t b = (uint32_t)w; b < nbt; b += 256 / kWave) {
    const uint32_t pos = b * kCkptInterval + (uint32_t)(lane & 31);
    const bool has = pos < smax && start + pos < end;
    uint32_t g = 0xFFFFFFFFu;
    float4 a0 = make_float4(0.f, 0.f, 1.f, 0.f), a1 = make_float4(1.f, -1.f, 0.f, 0.f);
    float4 a2 = make_float4(0.f, 0.f, 0.f, 0.f);
    if (has) {
      g = vals[start + pos];
      if ((int64_t)g < n) {
        const float4* r = reinterpret_cast<const float4*>(splats + (size_t)g * GS_SPLAT_FLOATS);
        a0 = r[0];
        a1 = r[1];
        a2 = r[2];
      }
    }
    const float b2 = a0.w + a0.w;
    float M00 = 0.f, Mx = 0.f, My = 0.f, Mxx = 0.f, Mxy = 0.f, Myy = 0.f;
    float gc0 = 0.f, gc1 = 0.f, gc2 = 0.f, gz = 0.f;
    for (int it = 0; it < NP / 2; ++it) {
      const int pi = 2 * it + h;
      const uint32_t nc = pnc[pi];
      float Tb = 0.f, Cb0 = 0.f, Cb1 = 0.f, Cb2 = 0.f, Db = 0.f;
      // the pixel composites in this bucket (and its checkpoint exists: a
      // caller's bucket count below the forward's need gives wrong values,
      // never an access outside the buffer)
      if (b * kCkptInterval < nc && b < (uint32_t)nbk) {
        const float* c = ckpt + ((size_t)tile * nbk + b) * kCkptVals * NP + pi;
        Tb = c[0];
        Cb0 = c[NP];
        Cb1 = c[2 * NP];
        Cb2 = c[3 * NP];
        if (DEPTH) Db = c[4 * NP];
      }
      const float pxf = (float)(tx * TILE + pi % TILE) + 0.5f;
      const float pyf = (float)(ty * TILE + pi / TILE) + 0.5f;
      const SplatQ q = eval_q(pxf, pyf, a0.x, a0.y, a0.z, b2, a1.x);
      const bool act = has && pos < nc &&
                       !splat_skips(q.Q, q.mag, a1.y, pxf, pyf, a0.x, a0.y, a0.z, a0.w, a1.x);
      const float G = act ? gauss(q.Q) : 0.f;
      const float oG = a1.z * G;
      const float al = fminf(kAlphaMax, oG);
      const float om = 1.f - al;
      const float Ti = Tb * half_shift_prod(half_incl_prod(om), lane);
      const float wgt = al * Ti;
      const float C0i = Cb0 + half_incl_sum(a2.x * wgt);
      const float C1i = Cb1 + half_incl_sum(a2.y * wgt);
      const float C2i = Cb2 + half_incl_sum(a2.z * wgt);
      const float rinv = __builtin_amdgcn_rcpf(om);
      const float d0 = pdc[0][pi], d1 = pdc[1][pi], d2 = pdc[2][pi];
      // colour (with background) behind the splat = image - blended up to it
      float acc = d0 * (Ti * a2.x - (pim[0][pi] - C0i) * rinv) +
                  d1 * (Ti * a2.y - (pim[1][pi] - C1i) * rinv) +
                  d2 * (Ti * a2.z - (pim[2][pi] - C2i) * rinv);
      gc0 += d0 * wgt;
      gc1 += d1 * wgt;
      gc2 += d2 * wgt;
      if (DEPTH) {
        const float Di = Db + half_incl_sum(a1.w * wgt);
        const float dd = pdd[pi];
        acc += dd * (Ti * a1.w - (pdep[pi] - Di) * rinv);
        gz += dd * wgt;
      }
      const float tg = (act && oG <= kAlphaMax) ? acc * G : 0.f;
      const float tx_ = tg * q.dx, ty_ = tg * q.dy;
      M00 += tg;
      Mx += tx_;
      My += ty_;
      Mxx = fmaf(tx_, q.dx, Mxx);
      Mxy = fmaf(tx_, q.dy, Mxy);
      Myy = fmaf(ty_, q.dy, Myy);
    }
    float v[10] = {M00, Mx, My, Mxx, Mxy, Myy, gc0, gc1, gc2, gz};
#pragma unroll
    for (int c = 0; c < 10; ++c) v[c] += __shfl_xor(v[c], 32, kWave);
    // lanes l and l + 32 now hold the same sums for splat l & 31
    constexpr int NC = GS_GRAD2D_COMPONENTS;
    const float o = a1.z, a = a0.z, bb = a0.w, cc = a1.x;
    float out[NC];
    out[0] = o * (a * v[1] + bb * v[2]);
    out[1] = o * (bb * v[1] + cc * v[2]);
    out[2] = -0.5f * o * v[3];
    out[3] = -o * v[4];
    out[4] = -0.5f * o * v[5];
    out[5] = v[0];
    out[6] = v[6];
    out[7] = v[7];
    out[8] = v[8];
    out[9] = v[9];
    const uint32_t gv = (has && (int64_t)g < n) ? g : 0xFFFFFFFFu;
    // one lane per (splat, component), so that an instruction's atomic adds
    // fall in the consecutive records of a few splats; the values come from
    // the splat's lane by wave shuffles
#pragma unroll
    for (int r = 0; r < 32 * NC / kWave; ++r) {
      const int e = r * kWave + lane, sl = e / NC, c = e - NC * sl;
      float val = 0.f;
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        const float t = __shfl(out[k], sl, kWave);
        if (k == c) val = t;
      }
      const uint32_t gs = (uint32_t)__shfl((int)gv, sl, kWave);
      if (gs != 0xFFFFFFFFu && val != 0.f)
        unsafeAtomicAdd(grad2d + (size_t)gs * NC + c, (double)val);
    }
  }
}

// Row sums of eight values by reduce-scatter over a row of 16 lanes: the
// values are halved between partner lanes three times (partners differ in
// lane bit 0, then bit 1, then by a rotation of 4, which flips bit 2) and
// the last partners (rotation by 8) are added. Lane l ends with the row sum
// of v[rs_slot(l)], rs_slot(l) = 4 (l & 1) + 2 ((l >> 1) & 1) + ((l >> 2) & 1),
// in 22 operations where eight all-reduces take 32. b0..b2 are lane bits
// 0..2 and every lane of the row must be active.
__device__ __forceinline__ float row_reduce_scatter8(const float* v, bool b0, bool b1, bool b2) {
  float r1[4], r2[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float keep = b0 ? v[i + 4] : v[i], send = b0 ? v[i] : v[i + 4];
    r1[i] = keep + dpp_mov<0xB1>(0.f, send);  // partner lane ^ 1
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float keep = b1 ? r1[i + 2] : r1[i], send = b1 ? r1[i] : r1[i + 2];
    r2[i] = keep + dpp_mov<0x4E>(0.f, send);  // partner lane ^ 2
  }
  const float keep = b2 ? r2[1] : r2[0], send = b2 ? r2[0] : r2[1];
  const float r3 = keep + dpp_mov<0x124>(0.f, send);  // row_ror:4
  return r3 + dpp_mov<0x128>(0.f, r3);                 // row_ror:8
}

__host__ __device__ constexpr int rs_slot(int l) {
  return 4 * (l & 1) + 2 * ((l >> 1) & 1) + ((l >> 2) & 1);
}

// Sum of x over the four rows of 16 lanes, row 0 first, in every row.
__device__ __forceinline__ float rows_sum(float x) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  const uint32_t u = __float_as_uint(x);
  const u2 h = __builtin_amdgcn_permlane32_swap(u, u, false, false);      // rows 0 1 0 1, 2 3 2 3
  const u2 a = __builtin_amdgcn_permlane16_swap(h.x, h.x, false, false);  // row 0, row 1
  const u2 b = __builtin_amdgcn_permlane16_swap(h.y, h.y, false, false);  // row 2, row 3
  return ((__uint_as_float(a.x) + __uint_as_float(a.y)) + __uint_as_float(b.x)) +
         __uint_as_float(b.y);
}

// The backward's unit of work is a region of 16 x 4 PX pixels of a tile (8 x 8
// for 8-pixel tiles), walked by one wavefront on its own: PX cells of 16 x 4
// pixels, one pixel per lane (lane l at column l % 16 and row l / 16), stacked
// so that a lane's pixels share their column. (8 x 8 cells would be reached
// about 11% less often, but a lane's pixels would not share dx.)
constexpr int kBwdBatch = 64;  // list entries a wavefront stages at a time, one per lane
constexpr int kBwdGroup = 2;   // splats evaluated together with one pixel per lane

// The staged splats that reach the region, in list order. Entry kBwdBatch holds
// a splat that blends nowhere: it fills up the last group.
struct BwdLds {
  // (u, v, a, b), (c, t - band, t + band, o), (r, g, b, z)
  float4 s0[kBwdBatch + 1], s1[kBwdBatch + 1], s2[kBwdBatch + 1];
  float t[kBwdBatch + 1];
  uint32_t sid[kBwdBatch + 1], pos[kBwdBatch + 1], cells[kBwdBatch + 1];
  float red[GS_GRAD2D_COMPONENTS][kBwdBatch + 1];  // the region's sums per splat
};

template <int TILE>
constexpr int bwd_cell_width() { return TILE < 16 ? TILE : 16; }
// regions of a tile with PX cells each, and their pixel offsets in the tile
template <int TILE, int PX>
constexpr int bwd_regions() { return TILE * TILE / (64 * PX); }
template <int TILE, int PX>
__device__ __forceinline__ int bwd_region_x(int r) {
  return TILE < 32 ? 0 : 16 * (r & 1);
}
template <int TILE, int PX>
__device__ __forceinline__ int bwd_region_y(int r) {
  return 4 * PX * (TILE < 32 ? r : r >> 1);
}

// One (splat, pixel) term of the backward, from the splat's G = exp(-Q / 2)
// (0: the pixel does not blend it): the pixel's T and U are moved in front of
// the splat; tg is dL/dQ / (-o / 2), w the blend weight. The order of every
// operation is written out, here and in the sums below, so that the gradients
// do not depend on which of the walks forms them.
// The first half does not need T and U: x = alpha, y = 1 / (1 - alpha), z = the
// splat's colour (and depth) along dL/dC, w = G (-1: alpha is clamped).
template <bool DEPTH>
__device__ __forceinline__ float4 bwd_pixel_shape(float G, float o, float4 a2, float dC0,
                                                  float dC1, float dC2, float dD) {
#pragma clang fp contract(off)
  const float oG = o * G;
  const float al = fminf(kAlphaMax, oG);
  float dcc = fmaf(dC2, a2.z, fmaf(dC0, a2.x, dC1 * a2.y));
  if (DEPTH) dcc = fmaf(dD, a2.w, dcc);
  return make_float4(al, __builtin_amdgcn_rcpf(1.f - al), dcc, oG <= kAlphaMax ? G : -1.f);
}
__device__ __forceinline__ void bwd_pixel_blend(float4 p, float& T, float& U, float& tg,
                                                float& w) {
#pragma clang fp contract(off)
  const float Tb = T * p.y;  // transmittance in front of this splat
  w = p.x * Tb;
  const float dal = p.y * fmaf(T, p.z, -U);
  tg = p.w >= 0.f ? dal * p.w : 0.f;  // no gradient through the clamp
  U = fmaf(w, p.z, U);
  T = Tb;
}
template <bool DEPTH>
__device__ __forceinline__ void bwd_pixel(float G, float o, float4 a2, float dC0, float dC1,
                                          float dC2, float dD, float& T, float& U, float& tg,
                                          float& w) {
  bwd_pixel_blend(bwd_pixel_shape<DEPTH>(G, o, a2, dC0, dC1, dC2, dD), T, U, tg, w);
}

// The lane's sums over its PX pixels: m0, m1, m2 of tg and its ey, ey^2 moments,
// c of the colour and depth terms. Pixels that do not blend have tg = w = 0.
template <int PX, bool DEPTH>
__device__ __forceinline__ void bwd_lane_sums(const float* tg, const float* w, const float* ey,
                                              const float* dC0, const float* dC1,
                                              const float* dC2, const float* dD, float& m0,
                                              float& m1, float& m2, float* c) {
#pragma clang fp contract(off)
  c[0] = dC0[0] * w[0];
  c[1] = dC1[0] * w[0];
  c[2] = dC2[0] * w[0];
  c[3] = DEPTH ? dD[0] * w[0] : 0.f;
  m0 = tg[0];
  m1 = PX > 1 ? fmaf(ey[0], tg[0], ey[PX > 1 ? 1 : 0] * tg[PX > 1 ? 1 : 0]) : ey[0] * tg[0];
  m2 = (ey[0] * tg[0]) * ey[0];
#pragma unroll
  for (int j = 1; j < PX; ++j) {
    c[0] = fmaf(dC0[j], w[j], c[0]);
    c[1] = fmaf(dC1[j], w[j], c[1]);
    c[2] = fmaf(dC2[j], w[j], c[2]);
    if (DEPTH) c[3] = fmaf(dD[j], w[j], c[3]);
    m0 = m0 + tg[j];
    if (j > 1) m1 = fmaf(ey[j], tg[j], m1);
    m2 = fmaf(ey[j] * tg[j], ey[j], m2);
  }
}

// The sums of a splat over the wavefront, from the lane's own sums (m0, m1, m2
// of tg and its ey, ey^2 moments; c of the colour and depth terms), into
// red[.][k]: within the rows of 16 lanes by DPP, then over the rows in their
// order by lane swaps. (Measured and slower: the nine sums as products with one-hot columns
// on the matrix cores, 16x16x4 FP32, 765 against 550 us for the image-space
// backward of the 1M-Gaussian 1600x1066 step: nine dependent products of 32
// cycles a splat; scattering over the rows first, eight operations fewer but
// each waiting for the last, 560 us.)
template <bool DEPTH, int N>
__device__ __forceinline__ void bwd_reduce(float (&red)[GS_GRAD2D_COMPONENTS][N], int k, int lane,
                                           float4 a0, float cc,
                                           float o, float ex, float m0, float m1, float m2,
                                           const float* c) {
#pragma clang fp contract(off)
  const int l16 = lane & 15;
  // dL/dQ = -o/2 tg: centroid and conic terms from the moments
  const float nho = -0.5f * o;
  float g[8];
  g[0] = nho * fmaf(a0.z * ex, m0, a0.w * m1);  // times -2 in the region's sum
  g[1] = nho * fmaf(a0.w * ex, m0, cc * m1);    // times -2 in the region's sum
  g[2] = ((ex * ex) * nho) * m0;
  g[3] = (ex * nho) * m1;                       // times 2 in the region's sum
  g[4] = nho * m2;
  g[5] = m0;
  g[6] = c[0];
  g[7] = c[1];
  // lanes 0..7 of a row hold the reduce-scattered sums, lane 8 (and 9) those
  // of components 8 (and 9)
  const float rs = row_reduce_scatter8(g, l16 & 1, l16 & 2, l16 & 4);
  float out = row_sum16(c[2]);
  if (DEPTH) {
    const float s9 = row_sum16(c[3]);
    if (l16 == 9) out = s9;
  }
  out = rows_sum(l16 < 8 ? rs : out);
  if (lane < (DEPTH ? 10 : 9)) red[lane < 8 ? rs_slot(lane) : lane][k] = out;
}

// Backward of one region of the tile whose list starts at `start` (region
// origin x0, y0). What bounds it: VALU issue where the lists are dense (some
// 45 operations per pixel and splat with four pixels per lane, the sums over
// the wavefront included), the walk of the longest lists where splats are
// small. So a wavefront stages only the splats that reach its region, reads a
// list entry's record a batch ahead, and skips the cells that a splat does
// not reach; splats that reach more than half of them take the pixels of a lane
// side by side (from two of four cells on, three, or all four only: 806, 808
// and 825 us at 300k Gaussians of about their spacing's size without a tile
// order, 650, 646 and 647 us for the surface scene); with one pixel per lane two
// splats are evaluated together, so that only T and U pass from one to the next.
// With the long regions of bwd_region_coop, against one wavefront per tile
// walking the whole list: 873 -> 335 us (300k Gaussians of about their spacing's
// size, 1600x1066), 1476 -> 525 us (1M children of 100k anchors), 272 -> 73 us
// (1000 Gaussians, 64x64), 583 -> 558 us (1M Gaussians of the surface scene,
// 1600x1066). With 96 registers for five wavefronts a SIMD (a few spilled): 581
// us for the last. Fewer pixels per lane mean more regions to a tile, each with
// its own adds: with one (16-pixel tiles) 626 -> 270 us on the first scene, but
// 1280 -> 1450 us on the last.
template <int TILE, int PX, bool DEPTH>
__device__ __forceinline__ void bwd_region(BwdLds& L, int x0, int y0, uint32_t start,
                                           const float* __restrict__ splats,
                                           const uint32_t* __restrict__ vals, int W, int H,
                                           float bg0, float bg1, float bg2,
                                           const float* __restrict__ T_final,
                                           const uint32_t* __restrict__ n_contrib,
                                           const float* __restrict__ dL_dimage,
                                           const float* __restrict__ dL_ddepth,
                                           double* __restrict__ grad2d, int64_t n) {
#pragma clang fp contract(fast)
  constexpr int NB = kBwdBatch, NC = GS_GRAD2D_COMPONENTS;
  constexpr int CW = bwd_cell_width<TILE>(), CH = 64 / CW;
  static_assert(NB == kWave, "a batch is one entry per lane");
  const int lane = threadIdx.x & (kWave - 1);
  const size_t HW = (size_t)H * W;
  float py[PX], T[PX], dC0[PX], dC1[PX], dC2[PX], dD[PX];
  // U = dL/dC . (colour, depth) of everything behind the current splat
  // (background included): dL/dalpha (1 - alpha) = T (dL/dC . c) - U
  float U[PX];
  uint32_t nc[PX];
  uint32_t most = 0;
  const int x = x0 + lane % CW;
  const float px = (float)x + 0.5f;
#pragma unroll
  for (int j = 0; j < PX; ++j) {
    const int y = y0 + j * CH + lane / CW;
    py[j] = (float)y + 0.5f;
    T[j] = 1.f; dC0[j] = dC1[j] = dC2[j] = dD[j] = 0.f; nc[j] = 0;
    if (x < W && y < H) {
      const size_t p = (size_t)y * W + x;
      T[j] = T_final[p];
      nc[j] = n_contrib[p];
      dC0[j] = dL_dimage[p];
      dC1[j] = dL_dimage[HW + p];
      dC2[j] = dL_dimage[2 * HW + p];
      if (DEPTH) dD[j] = dL_ddepth ? dL_ddepth[p] : 0.f;
    }
    U[j] = T[j] * (dC0[j] * bg0 + dC1[j] * bg1 + dC2[j] * bg2);  // background depth is 0
    most = max(most, nc[j]);
  }
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) most = max(most, (uint32_t)__shfl_xor((int)most, d, kWave));
  most = __builtin_amdgcn_readfirstlane(most);
  if (most == 0) return;  // nothing blended: no record is read
  if (lane == 0) {  // the filler: t < 0 skips it
    L.s0[NB] = make_float4(0.f, 0.f, 1.f, 0.f);
    L.s1[NB] = make_float4(1.f, -1.f, -1.f, 0.f);
    L.s2[NB] = make_float4(0.f, 0.f, 0.f, 0.f);
    L.t[NB] = -1.f;
    L.pos[NB] = 0xFFFFFFFFu;
  }
  // the list from its last entry that blends down, NB entries at a time; lane
  // l takes entry lo + l of [lo, hi). The record of the next batch and the id
  // of the one after are read while a batch is worked on.
  const auto entry = [&](int lo, int hi) {
    return lo + lane < hi ? vals[start + (uint32_t)max(lo + lane, 0)] : 0xFFFFFFFFu;
  };
  const auto record = [&](uint32_t g, float4* r) {
    const float4* p = reinterpret_cast<const float4*>(splats + ((int64_t)g < n ? (size_t)g : 0) *
                                                                   GS_SPLAT_FLOATS);
    r[0] = p[0];
    r[1] = p[1];
    r[2] = p[2];
  };
  int hi = (int)most, lo = max(hi - NB, 0);
  uint32_t gid = entry(lo, hi);
  float4 rec[3];
  record(gid, rec);
  uint32_t gid1 = entry(max(lo - NB, 0), lo);
  bool odd = false;  // from the first odd splat on: U may not be finite behind it
  while (hi > 0) {
    // stage: the entries that reach the region, compacted in list order
    uint32_t cells = 0;  // an id past n (never for a correct list) reaches nothing
    float band = 0.f;
    if ((int64_t)gid < n) {
      band = skip_band(rec[0].z, rec[0].w, rec[1].x, rec[1].y);
      cells = cells_reached<CW, CH, PX>((float)x0, (float)y0, rec[0], rec[1].x, rec[1].y, band,
                                        [](int) { return 0; }, [](int i) { return CH * i; });
    }
    const uint64_t reach = __ballot(cells != 0);
    odd = odd || __ballot(cells != 0 && odd_splat(rec[1], rec[2])) != 0;
    const int m = (int)__popcll(reach);
    if (cells != 0) {
      const int k = (int)__builtin_amdgcn_mbcnt_hi(
          (uint32_t)(reach >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)reach, 0u));
      L.s0[k] = rec[0];
      L.s1[k] = make_float4(rec[1].x, rec[1].y - band, rec[1].y + band, rec[1].z);
      L.s2[k] = make_float4(rec[2].x, rec[2].y, rec[2].z, rec[1].w);
      L.t[k] = rec[1].y;
      L.sid[k] = gid;
      L.pos[k] = (uint32_t)(lo + lane);
      if (PX > 1) L.cells[k] = cells;
    }
    __builtin_amdgcn_wave_barrier();  // a wavefront's LDS operations complete in order
    hi = lo;
    lo = max(lo - NB, 0);
    gid = gid1;
    record(gid, rec);
    gid1 = entry(max(lo - NB, 0), lo);
    uint64_t hit = 0;  // the staged splats that some pixel blends
    if constexpr (PX > 1) {
      const uint32_t mine = lane < m ? L.cells[lane] : 0u;
      uint64_t has[PX];
#pragma unroll
      for (int j = 0; j < PX; ++j) has[j] = __ballot((mine >> j) & 1u);
      const uint64_t most_cells = odd ? 0ull : __ballot(__builtin_popcount(mine) > PX / 2);
      for (int k = m - 1; k >= 0; --k) {
        const uint32_t pos = L.pos[k];  // position in the tile list
        const float4 a0 = L.s0[k], a1 = L.s1[k], a2 = L.s2[k];
        const float b2 = a0.w + a0.w;
        const float ex = px - a0.x;
        const float aex = a0.z * ex;
        uint64_t act[PX], some = 0, near = 0;
        float Q[PX], ey[PX], tg[PX], w[PX];
        // beside: more than half of the cells are reached, and the pixels of a
        // lane go side by side (those of a cell that is not reached are skipped
        // by Q > t); otherwise, and from the first odd splat on, the reached
        // cells one after the other, under the mask of the pixels that blend
        const auto shapes = [&](auto beside) {
#pragma unroll
          for (int j = 0; j < PX; ++j) {
            act[j] = 0;
            ey[j] = py[j] - a0.y;
            if (!beside.value && !((has[j] >> k) & 1ull)) continue;  // uniform
            const float t1 = a1.x * ey[j];
            const float td = t1 * ey[j];
            Q[j] = fmaf(ex, fmaf(b2, ey[j], aex), td);  // same value as eval_q
            const uint64_t skip = __ballot(Q[j] > a1.z);
            near |= ~(skip | __ballot(Q[j] <= a1.y));
            act[j] = __ballot(pos < nc[j]) & ~skip;
            some |= act[j];
          }
        };
        const auto terms = [&](auto beside) {
#pragma unroll
          for (int j = 0; j < PX; ++j) {
            tg[j] = w[j] = 0.f;
            const bool on = __builtin_amdgcn_inverse_ballot_w64(act[j]);
            if (!beside.value) {
              if (on) {
                asm volatile("");  // masked, not selected
                bwd_pixel<DEPTH>(gauss(Q[j]), a1.w, a2, dC0[j], dC1[j], dC2[j], dD[j], T[j], U[j],
                                 tg[j], w[j]);
              }
              continue;
            }
            // an inactive pixel runs the same arithmetic with alpha = 0: no change
            const float G = gauss(on ? Q[j] : __builtin_huge_valf());
            bwd_pixel<DEPTH>(G, a1.w, a2, dC0[j], dC1[j], dC2[j], dD[j], T[j], U[j], tg[j],
                             w[j]);
          }
        };
        const bool beside = (most_cells >> k) & 1ull;
        if (beside) shapes(std::true_type{}); else shapes(std::false_type{});
        if (near != 0) {  // a few splats in a thousand: the FP64 decision
          asm volatile("");  // not to be computed ahead of the branch
          some = 0;
#pragma unroll
          for (int j = 0; j < PX; ++j) {
            const bool skip = skips_f64(L.t[k], px, py[j], a0.x, a0.y, a0.z, a0.w, a1.x);
            act[j] = __ballot(pos < nc[j] && !skip);
            some |= act[j];
          }
        }
        if (some == 0) continue;
        hit |= 1ull << k;
        float m0, m1, m2, c[4];
        if (beside) {
          terms(std::true_type{});
          bwd_lane_sums<PX, DEPTH>(tg, w, ey, dC0, dC1, dC2, dD, m0, m1, m2, c);
        } else {
          terms(std::false_type{});
          bwd_lane_sums<PX, DEPTH>(tg, w, ey, dC0, dC1, dC2, dD, m0, m1, m2, c);
        }
        bwd_reduce<DEPTH>(L.red, k, lane, a0, a1.x, a1.w, ex, m0, m1, m2, c);
      }
    } else if (odd) {  // splat by splat, the same operations in the same order
#pragma unroll 1
      for (int k = m - 1; k >= 0; --k) {
        const uint32_t pos = L.pos[k];
        const float4 a0 = L.s0[k], a1 = L.s1[k], a2 = L.s2[k];
        const float ex = px - a0.x, ey = py[0] - a0.y;
        const float Q = eval_q(px, py[0], a0.x, a0.y, a0.z, a0.w + a0.w, a1.x).Q;
        uint64_t skip = __ballot(Q > a1.z);
        if (~(skip | __ballot(Q <= a1.y)) != 0)
          skip = __ballot(skips_f64(L.t[k], px, py[0], a0.x, a0.y, a0.z, a0.w, a1.x));
        const uint64_t act = __ballot(pos < nc[0]) & ~skip;
        if (act == 0) continue;
        hit |= 1ull << k;
        float tg = 0.f, w = 0.f, m0, m1, m2, c[4];
        if (__builtin_amdgcn_inverse_ballot_w64(act))
          bwd_pixel<DEPTH>(gauss(Q), a1.w, a2, dC0[0], dC1[0], dC2[0], dD[0], T[0], U[0], tg, w);
        bwd_lane_sums<1, DEPTH>(&tg, &w, &ey, dC0, dC1, dC2, dD, m0, m1, m2, c);
        bwd_reduce<DEPTH>(L.red, k, lane, a0, a1.x, a1.w, ex, m0, m1, m2, c);
      }
    } else {
      constexpr int G = kBwdGroup;
      for (int k0 = m - 1; k0 >= 0; k0 -= G) {
        int k[G];
        float4 a0[G], a1[G], a2[G];
        float Q[G], ex[G], ey[G];
        uint64_t act[G], near = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
          k[g] = k0 - g >= 0 ? k0 - g : NB;
          a0[g] = L.s0[k[g]];
          a1[g] = L.s1[k[g]];
          a2[g] = L.s2[k[g]];
          const uint32_t pos = L.pos[k[g]];
          ex[g] = px - a0[g].x;
          ey[g] = py[0] - a0[g].y;
          const float t1 = a1[g].x * ey[g];
          const float td = t1 * ey[g];
          Q[g] = fmaf(ex[g], fmaf(a0[g].w + a0[g].w, ey[g], a0[g].z * ex[g]), td);
          const uint64_t skip = __ballot(Q[g] > a1[g].z);
          near |= ~(skip | __ballot(Q[g] <= a1[g].y));
          act[g] = __ballot(pos < nc[0]) & ~skip;
        }
        if (near != 0) {
          asm volatile("");
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const bool skip = skips_f64(L.t[k[g]], px, py[0], a0[g].x, a0[g].y, a0[g].z, a0[g].w,
                                        a1[g].x);
            act[g] = __ballot(L.pos[k[g]] < nc[0] && !skip);
          }
        }
        float tg[G], w[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const float Gs = gauss(
              __builtin_amdgcn_inverse_ballot_w64(act[g]) ? Q[g] : __builtin_huge_valf());
          bwd_pixel<DEPTH>(Gs, a1[g].w, a2[g], dC0[0], dC1[0], dC2[0], dD[0], T[0], U[0], tg[g],
                           w[g]);
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
          if (act[g] == 0) continue;  // uniform
          hit |= 1ull << k[g];
          float m0, m1, m2, c[4];
          bwd_lane_sums<1, DEPTH>(&tg[g], &w[g], &ey[g], dC0, dC1, dC2, dD, m0, m1, m2, c);
          bwd_reduce<DEPTH>(L.red, k[g], lane, a0[g], a1[g].x, a1[g].w, ex[g], m0, m1, m2, c);
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
    // one atomic per (splat, component) for this region, one lane per pair, so
    // that the lanes of an instruction cover the consecutive components of a
    // few splats (a few cache lines of the per-splat records). Without depth,
    // component 9 has no gradient.
    constexpr int NCU = DEPTH ? NC : NC - 1;
    for (int e = lane; e < m * NCU; e += kWave) {
      const int q = e / NCU, c = e - q * NCU;
      if (!((hit >> q) & 1ull)) continue;
      float a = L.red[c][q];
      if (c < 2) a *= -2.f;  // exact: powers of two
      if (c == 3) a *= 2.f;
      if (a != 0.f) unsafeAtomicAdd(grad2d + (size_t)L.sid[q] * NC + c, (double)a);
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// A region of four cells whose walk is long goes to a workgroup of NW = 4 or 8
// wavefronts, a cell of 16 x 4 pixels to each or to two of them, 16 list
// entries at a time, in three steps. The shapes of a cell's splats depend on
// nothing before them: with 8 wavefronts, two share a cell's entries. Then
// one wavefront per cell walks T and U through them, six operations an entry.
// Then the wavefronts share out the entries and form their sums from the four
// cells' values, in the order in which one wavefront with four pixels per lane
// forms them, so the gradients are the same to the bit. With 4 wavefronts a
// cell's own walks T and U as it goes, and it is about 1.6 times the work of
// one wavefront where every splat reaches every cell, hence only for long
// walks.
template <int NW>
struct BwdCoopLds {
  static constexpr int kWaves = NW, B = 16;  // list entries at a time
  using Px = std::conditional_t<NW == 8, float4, float2>;
  float4 s0[kWave + 1], s1[kWave + 1], s2[kWave + 1];  // as in BwdLds, by list entry
  float t[kWave + 1];
  uint32_t sid[kWave + 1], cells[kWave + 1];
  Px px[B][4][kWave];      // by entry, cell and lane: (tg, w), before that the shape
  uint32_t hit[2][NW];     // by wavefront: the batch's entries that some pixel blends
  float red[GS_GRAD2D_COMPONENTS][B];
  uint32_t most[4];
};

template <int NW, bool DEPTH>
__device__ __forceinline__ void bwd_region_coop(BwdCoopLds<NW>& L, int x0, int y0, uint32_t start,
                                                const float* __restrict__ splats,
                                                const uint32_t* __restrict__ vals, int W, int H,
                                                float bg0, float bg1, float bg2,
                                                const float* __restrict__ T_final,
                                                const uint32_t* __restrict__ n_contrib,
                                                const float* __restrict__ dL_dimage,
                                                const float* __restrict__ dL_ddepth,
                                                double* __restrict__ grad2d, int64_t n) {
#pragma clang fp contract(fast)
  constexpr int NC = GS_GRAD2D_COMPONENTS, NCU = DEPTH ? NC : NC - 1;
  constexpr int B = BwdCoopLds<NW>::B, G = kBwdGroup;
  static_assert(NW == 4 || NW == 8, "one or two wavefronts to a cell");
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int cell = wv & 3;
  const size_t HW = (size_t)H * W;
  const int x = x0 + lane % 16;
  const float px = (float)x + 0.5f;
  // the upstream gradients of the four cells (for the sums), and the state of
  // this wavefront's own
  float py[4], dC0[4], dC1[4], dC2[4], dD[4];
  float T = 1.f, U = 0.f;
  uint32_t nc = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int y = y0 + j * 4 + lane / 16;
    py[j] = (float)y + 0.5f;
    dC0[j] = dC1[j] = dC2[j] = dD[j] = 0.f;
    if (x < W && y < H) {
      const size_t p = (size_t)y * W + x;
      dC0[j] = dL_dimage[p];
      dC1[j] = dL_dimage[HW + p];
      dC2[j] = dL_dimage[2 * HW + p];
      if (DEPTH) dD[j] = dL_ddepth ? dL_ddepth[p] : 0.f;
      if (j == cell) {
        T = T_final[p];
        nc = n_contrib[p];
      }
    }
  }
  float my_py = py[0], e0 = dC0[0], e1 = dC1[0], e2 = dC2[0], e3 = dD[0];
#pragma unroll
  for (int j = 1; j < 4; ++j)
    if (cell == j) {  // uniform
      my_py = py[j];
      e0 = dC0[j];
      e1 = dC1[j];
      e2 = dC2[j];
      e3 = dD[j];
    }
  U = T * (e0 * bg0 + e1 * bg1 + e2 * bg2);
  uint32_t most = nc;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) most = max(most, (uint32_t)__shfl_xor((int)most, d, kWave));
  if (lane == 0 && wv < 4) L.most[wv] = most;
  if (threadIdx.x == 0) {  // the filler: t < 0 skips it
    L.s0[kWave] = make_float4(0.f, 0.f, 1.f, 0.f);
    L.s1[kWave] = make_float4(1.f, -1.f, -1.f, 0.f);
    L.s2[kWave] = make_float4(0.f, 0.f, 0.f, 0.f);
    L.t[kWave] = -1.f;
  }
  __syncthreads();
  most = max(max(L.most[0], L.most[1]), max(L.most[2], L.most[3]));
  most = __builtin_amdgcn_readfirstlane(most);
  // 64 entries of the list at a time, staged by the wavefronts in turn (the
  // next 64 are read by another wavefront while these are worked on)
  uint32_t gid = 0xFFFFFFFFu;
  float4 rec[3];
  const auto fetch = [&](int lo, int hi) {
    gid = lo + lane < hi ? vals[start + (uint32_t)(lo + lane)] : 0xFFFFFFFFu;
    const float4* p = reinterpret_cast<const float4*>(
        splats + ((int64_t)gid < n ? (size_t)gid : 0) * GS_SPLAT_FLOATS);
    rec[0] = p[0];
    rec[1] = p[1];
    rec[2] = p[2];
  };
  int hi = (int)most, lo = max(hi - kWave, 0);
  if (wv == 0 && hi > 0) fetch(lo, hi);
  for (int turn = 0; hi > 0; ++turn) {
    if (wv == turn % NW) {
      uint32_t cells = 0;  // an id past n (never for a correct list) reaches nothing
      if ((int64_t)gid < n) {
        float band = skip_band(rec[0].z, rec[0].w, rec[1].x, rec[1].y);
        cells = cells_reached<16, 4, 4>((float)x0, (float)y0, rec[0], rec[1].x, rec[1].y, band,
                                        [](int) { return 0; }, [](int i) { return 4 * i; });
        if (odd_splat(rec[1], rec[2])) band = __builtin_huge_valf();  // to the FP64 decision
        L.s0[lane] = rec[0];
        L.s1[lane] = make_float4(rec[1].x, rec[1].y - band, rec[1].y + band, rec[1].z);
        L.s2[lane] = make_float4(rec[2].x, rec[2].y, rec[2].z, rec[1].w);
        L.t[lane] = rec[1].y;
        L.sid[lane] = gid;
      }
      L.cells[lane] = cells;
    }
    const int nlo = max(lo - kWave, 0);
    if (wv == (turn + 1) % NW && lo > 0) fetch(nlo, lo);
    __syncthreads();
    const uint64_t mine = __ballot((L.cells[lane] >> cell) & 1u);
    for (int b0 = (hi - lo - 1) / B * B, par = 0; b0 >= 0; b0 -= B, par ^= 1) {
      // the shapes of the cell's entries of this batch, G at a time
      uint32_t todo = (uint32_t)(mine >> b0) & ((1u << B) - 1u), hit = 0;
      if (NW == 8) todo &= wv < 4 ? 0x5555u : 0xAAAAu;
      while (todo != 0) {
        int k[G];
        float4 a0[G], a1[G], a2[G];
        float Q[G];
        uint64_t act[G], near = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const int kb = 31 - __builtin_clz(todo | 1u);
          k[g] = todo != 0 ? b0 + kb : kWave;
          todo &= ~(1u << kb);
          a0[g] = L.s0[k[g]];
          a1[g] = L.s1[k[g]];
          a2[g] = L.s2[k[g]];
          const float ex = px - a0[g].x, ey = my_py - a0[g].y;
          const float t1 = a1[g].x * ey;
          const float td = t1 * ey;
          Q[g] = fmaf(ex, fmaf(a0[g].w + a0[g].w, ey, a0[g].z * ex), td);  // as eval_q
          const uint64_t skip = __ballot(Q[g] > a1[g].z);
          near |= ~(skip | __ballot(Q[g] <= a1[g].y));
          act[g] = __ballot((uint32_t)(lo + k[g]) < nc) & ~skip;
        }
        if (near != 0) {  // a few groups in a thousand: the FP64 decision
          asm volatile("");  // not to be computed ahead of the branch
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const bool on = (uint32_t)(lo + k[g]) < nc &&
                            !skips_f64(L.t[k[g]], px, my_py, a0[g].x, a0[g].y, a0[g].z, a0[g].w,
                                       a1[g].x);
            act[g] = __ballot(on);
            // the other pixels pass unchanged whatever the splat's colour
            a2[g] = make_float4(on ? a2[g].x : 0.f, on ? a2[g].y : 0.f, on ? a2[g].z : 0.f,
                                on ? a2[g].w : 0.f);
          }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
          if (act[g] == 0) continue;  // uniform (the filler's t < 0 leaves it inactive)
          const bool on = __builtin_amdgcn_inverse_ballot_w64(act[g]);
          const float Gs = gauss(on ? Q[g] : __builtin_huge_valf());
          float4 p = bwd_pixel_shape<DEPTH>(Gs, a1[g].w, a2[g], e0, e1, e2, e3);
          p.w = on ? p.w : -1.f;  // no gradient from the others, whatever their U
          if constexpr (NW == 8) {
            L.px[k[g] - b0][cell][lane] = p;
          } else {
            float2 tw;
            bwd_pixel_blend(p, T, U, tw.x, tw.y);
            L.px[k[g] - b0][cell][lane] = tw;
          }
          hit |= 1u << (k[g] - b0);
        }
      }
      if (lane == 0) L.hit[par][wv] = hit;
      __syncthreads();
      uint32_t hits[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        hits[j] = __builtin_amdgcn_readfirstlane(
            L.hit[par][j] | (NW == 8 ? L.hit[par][NW - 4 + j] : 0u));
      if (NW == 8 && wv < 4) {  // T and U through the cell's entries, last first
        uint32_t left = wv == 0 ? hits[0] : wv == 1 ? hits[1] : wv == 2 ? hits[2] : hits[3];
        constexpr int R = 4;  // entries read together
        while (left != 0) {
          int k[R];
          float4 p[R];
#pragma unroll
          for (int g = 0; g < R; ++g) {
            k[g] = left != 0 ? 31 - __builtin_clz(left) : -1;
            if (left != 0) left &= ~(1u << k[g]);
            if constexpr (NW == 8) p[g] = L.px[max(k[g], 0)][cell][lane];
          }
#pragma unroll
          for (int g = 0; g < R; ++g) {
            if (k[g] < 0) break;  // uniform
            float tg, w;
            bwd_pixel_blend(p[g], T, U, tg, w);
            *reinterpret_cast<float2*>(&L.px[k[g]][cell][lane]) = make_float2(tg, w);
          }
        }
      }
      if (NW == 8) __syncthreads();
      // the sums: entry q by wavefront q % NW
      const uint32_t any = hits[0] | hits[1] | hits[2] | hits[3];
#pragma unroll
      for (int q = wv; q < B; q += NW) {
        if (!((any >> q) & 1u)) continue;  // uniform
        const uint32_t of = ((hits[0] >> q) & 1u) | ((hits[1] >> q) & 1u) << 1 |
                            ((hits[2] >> q) & 1u) << 2 | ((hits[3] >> q) & 1u) << 3;
        const float4 a0 = L.s0[b0 + q], a1 = L.s1[b0 + q];
        float tg[4], w[4], ey[4], m0, m1, m2, c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          // a cell without a blend adds zeros
          const float2 tw = (of >> j) & 1u ? *reinterpret_cast<const float2*>(&L.px[q][j][lane])
                                           : make_float2(0.f, 0.f);
          tg[j] = tw.x;
          w[j] = tw.y;
          ey[j] = py[j] - a0.y;
        }
        bwd_lane_sums<4, DEPTH>(tg, w, ey, dC0, dC1, dC2, dD, m0, m1, m2, c);
        const float ex = px - a0.x;
        bwd_reduce<DEPTH>(L.red, q, lane, a0, a1.x, a1.w, ex, m0, m1, m2, c);
      }
      __syncthreads();
      for (int e = threadIdx.x; e < B * NCU; e += NW * kWave) {
        const int q = e / NCU, c = e - q * NCU;
        if (!((any >> q) & 1u)) continue;
        float a = L.red[c][q];
        if (c < 2) a *= -2.f;  // exact: powers of two
        if (c == 3) a *= 2.f;
        if (a != 0.f) unsafeAtomicAdd(grad2d + (size_t)L.sid[b0 + q] * NC + c, (double)a);
      }
    }
    __syncthreads();  // the entries are read until here
    hi = lo;
    lo = nlo;
  }
}

// A launch ends when its longest walk does, and all its walks together fill
// the chip for about (their sum) x 0.5 cycles, at some 1000 cycles per splat
// of a walk by a single wavefront: a walk above 1 / 3072 of the sum is long
// (the sum is taken from four quantiles of the sorted tiles' work). Measured
// at 1 / 2048, 1 / 3072, 1 / 4096 and with no region long: 340, 335, 340 and
// 749 us at 300k Gaussians of about their spacing's size, 540, 536, 509 and
// 1151 us at 1M children of 100k anchors, 573, 558, 595 and 615 us at 1M
// Gaussians of the surface scene (1600x1066 each).
__device__ __forceinline__ uint32_t bwd_long_walk(const uint32_t* order, const uint32_t* work,
                                                  int nt, int regions) {
  uint32_t s = 0;
#pragma unroll
  for (int i = 1; i < 8; i += 2) s += work[order[(int)((int64_t)nt * i / 8)]];
  return (uint32_t)((uint64_t)s * (uint32_t)regions / 12288u);
}
constexpr int kBwdSplit = 2048;  // regions, heaviest first, that may get a workgroup

// The backward's launch: with four cells per region and the tiles' order known,
// workgroups 0 .. split - 1 each look at one of the first regions and take it if
// its tile's walk is long; the workgroups after them take the other regions,
// one per wavefront.
template <int NW, bool SPLIT>
union BwdShared {
  BwdLds one[NW];
  BwdCoopLds<NW> coop;
};
template <int NW>
union BwdShared<NW, false> {
  BwdLds one[NW];
};
// Launches of at most this many regions have 8 wavefronts to a workgroup, the
// others (and the batched one) 4: where the walk of a workgroup decides, 8 are
// faster, where the chip is full their third step costs more than it saves. 4
// against 8: 90 and 73 us (16 regions), 153 and 122 us (144), 101 and 92 us
// (950), 274 and 257 us (3600); 328 and 360 us, 527 and 746 us (6700 regions,
// 300k Gaussians of about their spacing's size and 1M children of anchors).
// The line lies somewhere between those two sizes, and it counts empty regions
// too: where most of a large view is empty, 8 would be faster (100k Gaussians
// in 65 tiles of a 1920x1080 view, 8160 regions: 1710 us with 4, 1452 with 8,
// 5249 with one wavefront to a tile), but the launch is chosen before the lists
// are known.
constexpr int64_t kBwdFewRegions = 4096;
template <int TILE, int PX>
constexpr bool bwd_can_split() { return PX == 4 && TILE >= 16; }
template <int TILE, int PX>
__host__ __device__ inline int bwd_split(int nt, bool ordered) {
  const int r = nt * bwd_regions<TILE, PX>();
  return !bwd_can_split<TILE, PX>() || !ordered ? 0 : r < kBwdSplit ? r : kBwdSplit;
}

// Region r of rank order: of tile order[r / R]; its part r % R.
template <int TILE, int PX, bool DEPTH, class Shared>
__device__ __forceinline__ void bwd_one(Shared& L, int tile, int part,
                                        const float* __restrict__ splats,
                                        const uint32_t* __restrict__ vals,
                                        const uint32_t* __restrict__ ranges, int W, int H,
                                        int tiles_y, float bg0, float bg1, float bg2,
                                        const float* __restrict__ T_final,
                                        const uint32_t* __restrict__ n_contrib,
                                        const float* __restrict__ dL_dimage,
                                        const float* __restrict__ dL_ddepth,
                                        double* __restrict__ grad2d, int64_t n) {
  const int x0 = tile / tiles_y * TILE + bwd_region_x<TILE, PX>(part);
  const int y0 = tile % tiles_y * TILE + bwd_region_y<TILE, PX>(part);
  if constexpr (!std::is_same<Shared, BwdLds>::value)
    bwd_region_coop<Shared::kWaves, DEPTH>(L, x0, y0, ranges[tile], splats, vals, W, H, bg0, bg1,
                                           bg2, T_final, n_contrib, dL_dimage, dL_ddepth, grad2d,
                                           n);
  else
    bwd_region<TILE, PX, DEPTH>(L, x0, y0, ranges[tile], splats, vals, W, H, bg0, bg1, bg2,
                                T_final, n_contrib, dL_dimage, dL_ddepth, grad2d, n);
}

// order, work: the tiles heaviest first and each tile's largest n_contrib
// (null: tile-id order, one wavefront per region).
// Two pixels per lane without depth: 80 registers, six wavefronts per SIMD.
template <int TILE, int PX, bool DEPTH, int NW>
__global__ void __launch_bounds__(NW* kWave)
__attribute__((amdgpu_waves_per_eu(PX == 2 && !DEPTH ? 6 : 1))) k_render_bwd(
    const float* __restrict__ splats, const uint32_t* __restrict__ vals,
    const uint32_t* __restrict__ ranges, int W, int H, int nt, int tiles_y, float bg0, float bg1,
    float bg2, const float* __restrict__ T_final, const uint32_t* __restrict__ n_contrib,
    const float* __restrict__ dL_dimage, const float* __restrict__ dL_ddepth,
    double* __restrict__ grad2d, int64_t n, const uint32_t* __restrict__ order,
    const uint32_t* __restrict__ work) {
  __shared__ BwdShared<NW, bwd_can_split<TILE, PX>()> L;
  constexpr int R = bwd_regions<TILE, PX>();
  const int split = bwd_split<TILE, PX>(nt, order != nullptr);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const bool first = (int)blockIdx.x < split;
  const int item = first ? (int)blockIdx.x : ((int)blockIdx.x - split) * NW + wv;
  if (item >= nt * R) return;
  const int rank = item / R;
  const int tile = order ? (int)order[rank] : rank;
  const bool is_long = item < split && work[tile] > bwd_long_walk(order, work, nt, nt * R);
  if (first != is_long) return;
  if constexpr (bwd_can_split<TILE, PX>()) {
    if (first) {
      bwd_one<TILE, PX, DEPTH>(L.coop, tile, item % R, splats, vals, ranges, W, H, tiles_y, bg0,
                               bg1, bg2, T_final, n_contrib, dL_dimage, dL_ddepth, grad2d, n);
      return;
    }
  }
  bwd_one<TILE, PX, DEPTH>(L.one[wv], tile, item % R, splats, vals, ranges, W, H, tiles_y, bg0,
                           bg1, bg2, T_final, n_contrib, dL_dimage, dL_ddepth, grad2d, n);
}

// Longest-first tile order for the backward. The backward of a tile walks
// its list down from the largest n_contrib of its pixels, so that number is
// the tile's work; starting the heaviest tiles first keeps them out of the
// launch's tail. work[t] = max n_contrib over tile t (one workgroup a tile).
template <int TILE>
__global__ void __launch_bounds__(256) k_tile_work(const uint32_t* __restrict__ n_contrib, int W,
                                                   int H, int tiles_y,
                                                   uint32_t* __restrict__ work) {
  __shared__ uint32_t wmax[256 / kWave];
  const int tile = blockIdx.x, tx = tile / tiles_y, ty = tile % tiles_y;
  uint32_t m = 0;
  for (int i = threadIdx.x; i < TILE * TILE; i += 256) {
    const int x = tx * TILE + i % TILE, y = ty * TILE + i / TILE;
    if (x < W && y < H) m = max(m, n_contrib[(size_t)y * W + x]);
  }
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d, kWave));
  if ((threadIdx.x & (kWave - 1)) == 0) wmax[threadIdx.x / kWave] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < 256 / kWave; ++w) m = max(m, wmax[w]);
    work[tile] = m;
  }
}

// 1024 work classes, exact below 512 splats, 8 wide above (up to 4600).
__device__ __forceinline__ uint32_t work_class(uint32_t w) {
  return w < 512u ? w : min(512u + ((w - 512u) >> 3), 1023u);
}

// Counting sort of the nt tiles by descending work class (one workgroup);
// tiles of one class keep no particular order.
__global__ void __launch_bounds__(1024) k_tile_rank(const uint32_t* __restrict__ work, int nt,
                                                    uint32_t* __restrict__ order) {
  constexpr int kHeld = 8;  // classes held in registers per thread (nt <= 8192)
  __shared__ uint32_t cnt[1024];
  __shared__ uint32_t wsum[1024 / kWave];
  cnt[threadIdx.x] = 0;
  uint32_t cls[kHeld];
#pragma unroll
  for (int j = 0; j < kHeld; ++j) {
    const int t = threadIdx.x + j * 1024;
    cls[j] = t < nt ? work_class(work[t]) : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kHeld; ++j)
    if (threadIdx.x + j * 1024 < nt) atomicAdd(&cnt[cls[j]], 1u);
  for (int t = threadIdx.x + kHeld * 1024; t < nt; t += 1024)
    atomicAdd(&cnt[work_class(work[t])], 1u);
  __syncthreads();
  // thread i holds class 1023 - i, so the exclusive scan gives descending offsets
  const uint32_t c = cnt[1023 - threadIdx.x];
  uint32_t total;
  const uint32_t off = block_exclusive_scan<1024>(c, wsum, total);
  cnt[1023 - threadIdx.x] = off;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kHeld; ++j) {
    const int t = threadIdx.x + j * 1024;
    if (t < nt) order[atomicAdd(&cnt[cls[j]], 1u)] = (uint32_t)t;
  }
  for (int t = threadIdx.x + kHeld * 1024; t < nt; t += 1024)
    order[atomicAdd(&cnt[work_class(work[t])], 1u)] = (uint32_t)t;
}

// Eq. 4 counts: the forward's decisions replayed per tile; for every splat
// of the list, the number of masked pixels of the tile that blend it is
// added to its score with one atomic per (splat, tile).
//
// A pixel's decisions depend on no other pixel, so only masked pixels are
// replayed: a wavefront owns one 8 x 8 cell as in fwd_tile, drops out where
// nothing is masked or once its masked pixels have stopped, and walks the
// splats that reach the cell, four at a time, counting in lane i the blends
// of the i-th splat of its list (VALU issue bounds it: some 15 operations per
// pixel and splat). Against every pixel, splat and strip of the tile one
// after the other: 1096 -> 249 us (1M Gaussians grown on the fit scene, mean
// of three 1600x1066 views).
template <int TILE>
__global__ void __launch_bounds__(TILE* TILE) k_split_score(
    const float* __restrict__ splats, const uint32_t* __restrict__ vals,
    const uint32_t* __restrict__ ranges, int64_t n, int W, int H, int tiles_y,
    const uint8_t* __restrict__ mask, uint32_t* __restrict__ score) {
#pragma clang fp contract(fast)
  constexpr int NTH = TILE * TILE, NB = 256, G = kFwdGroup;
  __shared__ FwdLdsT<NB, NTH> L;
  __shared__ uint32_t sid[NB], cnt[NB + 1];
  const int tile = blockIdx.x;
  const int tx = tile / tiles_y, ty = tile % tiles_y;
  const uint32_t start = ranges[tile], end = ranges[tile + 1];
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int x = tx * TILE + FwdCells::x(wv) + lane % 8, y = ty * TILE + FwdCells::y(wv) + lane / 8;
  const float px = (float)x + 0.5f, py = (float)y + 0.5f;
  const uint64_t masked = __ballot(x < W && y < H && mask[(size_t)y * W + x] != 0);
  uint64_t done = ~masked;  // the lanes that take no more splats
  float T = 1.f;
  uint32_t* const list = L.list[wv];
  if (threadIdx.x == 0) fwd_stage<TILE>(L, NB, splats, 0u, 0, 0.f, 0.f);  // the filler
  for (uint32_t b = start; b < end; b += NB) {
    if (__syncthreads_count(done != ~0ull) == 0) break;
    const int nb = (int)min((uint32_t)NB, end - b);
    for (int q = threadIdx.x; q < nb; q += NTH) {
      const uint32_t g = vals[b + q];
      cnt[q] = 0;
      sid[q] = g;
      fwd_stage<TILE>(L, q, splats, g, n, (float)(tx * TILE), (float)(ty * TILE));
    }
    __syncthreads();
    if (done != ~0ull) {
      int m = 0;
      for (int base = 0; base < nb; base += kWave) {
        const int q = base + lane;
        const bool reach = q < nb && ((L.cells[min(q, NB)] >> wv) & 1u) != 0u;
        const uint64_t bal = __ballot(reach);
        if (reach)
          list[m + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u))] =
              16u * (uint32_t)q;
        m += (int)__popcll(bal);
      }
      if (lane < G) list[m + lane] = 16u * NB;
      __builtin_amdgcn_wave_barrier();  // a wavefront's LDS operations complete in order
      for (int i0 = 0; i0 < m && done != ~0ull; i0 += kWave) {
        const int i1 = min(i0 + kWave, m);
        uint32_t blends = 0;  // of splat i0 + lane
        for (int i = i0; i < i1 && done != ~0ull; i += G) {
          uint32_t off[G];
          float4 a0[G], a1[G];
          float Q[G], al[G];
          uint64_t skip[G], near = 0;
#pragma unroll
          for (int g = 0; g < G; ++g) off[g] = list[i + g];
#pragma unroll
          for (int g = 0; g < G; ++g) {
            a0[g] = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(L.s0) + off[g]);
            a1[g] = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(L.s1) + off[g]);
          }
#pragma unroll
          for (int g = 0; g < G; ++g) {
            Q[g] = eval_q(px, py, a0[g].x, a0[g].y, a0[g].z, a0[g].w, a1[g].x).Q;
            skip[g] = __ballot(Q[g] > a1[g].z);
            near |= ~(skip[g] | __ballot(Q[g] <= a1[g].y));
          }
          if (near != 0) {  // a few groups in a thousand: the FP64 decision
            asm volatile("");  // not to be computed ahead of the branch
#pragma unroll
            for (int g = 0; g < G; ++g)
              skip[g] = __ballot(skips_f64(L.t[off[g] / 16u], px, py, a0[g].x, a0[g].y, a0[g].z,
                                           0.5f * a0[g].w, a1[g].x));
          }
#pragma unroll
          for (int g = 0; g < G; ++g) al[g] = fminf(kAlphaMax, a1[g].w * gauss(Q[g]));
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const float Tn = T * (1.f - al[g]);
            const uint64_t low = __ballot(Tn < kTStop);
            const uint64_t none = skip[g] | done | low;  // no blend
            done |= low & ~skip[g];
            T = __builtin_amdgcn_inverse_ballot_w64(none) ? T : Tn;
            blends = __builtin_amdgcn_inverse_ballot_w64(1ull << (i - i0 + g))
                         ? (uint32_t)__popcll(~none) : blends;
          }
        }
        if (i0 + lane < i1 && blends != 0) atomicAdd(&cnt[list[i0 + lane] / 16u], blends);
      }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < nb; q += NTH)
      if (cnt[q] && (int64_t)sid[q] < n) atomicAdd(score + sid[q], cnt[q]);
  }
}

// ---------------------------------------------------------------------------
// Batched views: one persistent launch per phase. The (view, tile) work items
// of all views form one queue (view by view, tiles in id order); every
// workgroup takes the next item with one atomic on a device counter until
// the queue is empty.
struct ViewSet {
  int n_views, total;
  int start[GS_MAX_VIEWS + 1];  // first work item of each view
  int W[GS_MAX_VIEWS], H[GS_MAX_VIEWS], tiles_y[GS_MAX_VIEWS];
  const float* splats[GS_MAX_VIEWS];
  const uint32_t* vals[GS_MAX_VIEWS];
  const uint32_t* ranges[GS_MAX_VIEWS];
  float* image[GS_MAX_VIEWS];
  float* depth[GS_MAX_VIEWS];
  float* T_final[GS_MAX_VIEWS];
  uint32_t* n_contrib[GS_MAX_VIEWS];
  const float* dL_dimage[GS_MAX_VIEWS];
  const float* dL_ddepth[GS_MAX_VIEWS];
  double* grad2d[GS_MAX_VIEWS];
  RunLists rl[GS_MAX_VIEWS];  // the deferred binning's run tables (deferred forward only)
};

// Next work item for the whole workgroup (-1 when the queue is empty).
__device__ __forceinline__ int next_item(uint32_t* queue, int total, int* s_item) {
  if (threadIdx.x == 0) *s_item = (int)atomicAdd(queue, 1u);
  __syncthreads();
  const int it = *s_item;
  __syncthreads();
  return it < total ? it : -1;
}

__device__ __forceinline__ int view_of(const ViewSet& vs, int it) {
  int v = 0;
  while (v + 1 < vs.n_views && it >= vs.start[v + 1]) ++v;
  return v;
}

template <int TILE, int PX, int NB>
__global__ void __launch_bounds__(TILE* TILE / PX)
__attribute__((amdgpu_waves_per_eu(fwd_waves(TILE, PX)))) k_render_fwd_batched(
    ViewSet vs, int64_t n, float bg0, float bg1, float bg2, uint32_t* queue) {
  __shared__ FwdLdsT<NB, TILE * TILE / PX> L;
  __shared__ int s_item;
  for (int it; (it = next_item(queue, vs.total, &s_item)) >= 0;) {
    const int v = view_of(vs, it);
    fwd_tile<TILE, PX, false, NB>(L, it - vs.start[v], vs.splats[v], vs.vals[v], vs.ranges[v], n, vs.W[v],
                       vs.H[v], vs.tiles_y[v], bg0, bg1, bg2, vs.image[v], vs.depth[v],
                       vs.T_final[v], vs.n_contrib[v]);
  }
}

// The batched forward on the lists of the deferred binning (one run table
// per view); each view's vals receives the list positions it stages.
template <int TILE, int PX, int NB>
__global__ void __launch_bounds__(TILE* TILE / PX)
__attribute__((amdgpu_waves_per_eu(fwd_waves(TILE, PX)))) k_render_fwd_batched_def(
    ViewSet vs, int64_t n, float bg0, float bg1, float bg2, uint32_t* queue) {
  __shared__ FwdLdsT<NB, TILE * TILE / PX> L;
  __shared__ DefLds<NB, TILE * TILE / PX> DL;
  __shared__ int s_item;
  for (int it; (it = next_item(queue, vs.total, &s_item)) >= 0;) {
    const int v = view_of(vs, it);
    uint32_t* vals = const_cast<uint32_t*>(vs.vals[v]);  // the caller's (writable) list array
    fwd_tile<TILE, PX, false, NB, true>(L, it - vs.start[v], vs.splats[v], vals, vs.ranges[v], n,
                                        vs.W[v], vs.H[v], vs.tiles_y[v], bg0, bg1, bg2,
                                        vs.image[v], vs.depth[v], vs.T_final[v], vs.n_contrib[v],
                                        nullptr, 0, nullptr, &DL, vs.rl[v], vals);
  }
}

// The backward's regions from one queue: first those that may be long, by the
// workgroup together, then the rest, each wavefront on its own.
template <int TILE, int PX, bool DEPTH>
__global__ void __launch_bounds__(4 * kWave) k_render_bwd_batched(
    ViewSet vs, int64_t n, float bg0, float bg1, float bg2, uint32_t* queue,
    const uint32_t* __restrict__ order, const uint32_t* __restrict__ work) {
  __shared__ BwdShared<4, bwd_can_split<TILE, PX>()> L;
  __shared__ int s_item;
  constexpr int R = bwd_regions<TILE, PX>();
  const int total = vs.total * R, split = bwd_split<TILE, PX>(vs.total, order != nullptr);
  const uint32_t long_walk = split > 0 ? bwd_long_walk(order, work, vs.total, total) : 0u;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int q = -1;
  if constexpr (bwd_can_split<TILE, PX>()) {
    while ((q = next_item(queue, split + total, &s_item)) >= 0 && q < split) {
      const int it = (int)order[q / R];
      if (work[it] <= long_walk) continue;
      const int v = view_of(vs, it);
      bwd_one<TILE, PX, DEPTH>(L.coop, it - vs.start[v], q % R, vs.splats[v], vs.vals[v],
                               vs.ranges[v], vs.W[v], vs.H[v], vs.tiles_y[v], bg0, bg1, bg2,
                               vs.T_final[v], vs.n_contrib[v], vs.dL_dimage[v], vs.dL_ddepth[v],
                               vs.grad2d[v], n);
    }
    if (q < 0) return;  // the queue is empty
    __syncthreads();    // the regions' LDS changes hands
  }
  // the item taken last is the first wavefront's
  for (bool have = bwd_can_split<TILE, PX>() && wv == 0;; have = false) {
    if (!have) {
      uint32_t k = 0;
      if ((threadIdx.x & (kWave - 1)) == 0) k = atomicAdd(queue, 1u);
      q = (int)__builtin_amdgcn_readfirstlane(k);
    }
    const int item = q - split;
    if (item < 0) continue;  // never: the queue is past the split regions here
    if (item >= total) return;
    const int it = order ? (int)order[item / R] : item / R;
    if (item < split && work[it] > long_walk) continue;  // done by a workgroup
    const int v = view_of(vs, it);
    bwd_one<TILE, PX, DEPTH>(L.one[wv], it - vs.start[v], item % R, vs.splats[v], vs.vals[v],
                             vs.ranges[v], vs.W[v], vs.H[v], vs.tiles_y[v], bg0, bg1, bg2,
                             vs.T_final[v], vs.n_contrib[v], vs.dL_dimage[v], vs.dL_ddepth[v],
                             vs.grad2d[v], n);
  }
}

__global__ void k_reset_queue(uint32_t* q) { *q = 0u; }

// k_tile_work over the (view, tile) items of a batch: work[it] = largest
// n_contrib of the item's pixels.
template <int TILE>
__global__ void __launch_bounds__(256) k_tile_work_views(ViewSet vs, uint32_t* __restrict__ work) {
  __shared__ uint32_t wmax[256 / kWave];
  const int it = blockIdx.x, v = view_of(vs, it), tile = it - vs.start[v];
  const int W = vs.W[v], H = vs.H[v], tx = tile / vs.tiles_y[v], ty = tile % vs.tiles_y[v];
  const uint32_t* nc = vs.n_contrib[v];
  uint32_t m = 0;
  for (int i = threadIdx.x; i < TILE * TILE; i += 256) {
    const int x = tx * TILE + i % TILE, y = ty * TILE + i / TILE;
    if (x < W && y < H) m = max(m, nc[(size_t)y * W + x]);
  }
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d, kWave));
  if ((threadIdx.x & (kWave - 1)) == 0) wmax[threadIdx.x / kWave] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < 256 / kWave; ++w) m = max(m, wmax[w]);
    work[it] = m;
  }
}

__global__ void k_zero_f64(double* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

gs_status launch_preprocess_bwd(const gs_gaussians* g, int64_t n, int deg, const CamDev& cam,
                                const double* grad2d, gs_gaussians* grads, int accumulate,
                                hipStream_t st);
gs_status launch_preprocess_bwd_adam(gs_gaussians* g, int64_t n, int deg, const CamDev& cam,
                                     const double* grad2d, const gs_adam_params* adam,
                                     hipStream_t st);
gs_status launch_preprocess_bwd_views(const gs_gaussians* g, int64_t n, int deg,
                                      const CamDev* cams, const double* const* grad2d,
                                      int n_views, gs_gaussians* grads, int accumulate,
                                      hipStream_t st);

}  // namespace gs

using namespace gs;

extern "C" gs_status gs_render_fwd(const float* splats, int64_t n, const uint32_t* vals,
                                   const uint32_t* ranges, const gs_camera* cam, const float* bg,
                                   float* image, float* depth, float* T_final,
                                   uint32_t* n_contrib, void* stream) {
  CamDev cd;
  if (n < 0 || !make_cam(cam, &cd) || !ranges || !bg || !image || !depth || !T_final ||
      !n_contrib)
    return GS_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const int nt = cd.tiles_x * cd.tiles_y;
  const int px = tuning().fwd_px;
#define GS_FWD(TL, PXV)                                                                        \
  k_render_fwd<TL, PXV><<<nt, TL * TL / PXV, 0, st>>>(splats, vals, ranges, n, cd.W, cd.H,  \
                                                      cd.tiles_y, bg[0], bg[1], bg[2], image, \
                                                      depth, T_final, n_contrib)
  GS_TIMED("render_fwd", st, if (cd.tile == 8) GS_FWD(8, 1);
           else if (cd.tile == 16) {
             if (px == 4) GS_FWD(16, 4); else if (px == 2) GS_FWD(16, 2); else GS_FWD(16, 1);
           } else {
             if (px == 4) GS_FWD(32, 4); else if (px == 2) GS_FWD(32, 2); else GS_FWD(32, 1);
           });
#undef GS_FWD
  GS_CHECK_LAUNCH();
  return GS_OK;
}

extern "C" gs_status gs_render_fwd_deferred(const float* splats, int64_t n, const void* workspace,
                                            size_t workspace_bytes, int64_t capacity,
                                            uint32_t* vals, const uint32_t* ranges,
                                            const gs_camera* cam, const float* bg, float* image,
                                            float* depth, float* T_final, uint32_t* n_contrib,
                                            void* stream) {
  CamDev cd;
  if (n < 0 || capacity < 0 || !make_cam(cam, &cd) || !ranges || !bg || !image || !depth ||
      !T_final || !n_contrib || (capacity > 0 && !vals))
    return GS_EINVAL;
  RunLists rl;
  if (!run_lists(workspace, workspace_bytes, n, capacity, cd.tiles_x, cd.tiles_y, &rl))
    return GS_ECAPACITY;
  hipStream_t st = (hipStream_t)stream;
  const int nt = cd.tiles_x * cd.tiles_y;
  const int px = tuning().fwd_px;
#define GS_FWD(TL, PXV)                                                                        \
  k_render_fwd_def<TL, PXV><<<nt, TL * TL / PXV, 0, st>>>(splats, rl, vals, ranges, n, cd.W,  \
                                                          cd.H, cd.tiles_y, bg[0], bg[1],     \
                                                          bg[2], image, depth, T_final,       \
                                                          n_contrib)
  GS_TIMED("render_fwd", st, if (cd.tile == 8) GS_FWD(8, 1);
           else if (cd.tile == 16) {
             if (px == 4) GS_FWD(16, 4); else if (px == 2) GS_FWD(16, 2); else GS_FWD(16, 1);
           } else {
             if (px == 4) GS_FWD(32, 4); else if (px == 2) GS_FWD(32, 2); else GS_FWD(32, 1);
           });
#undef GS_FWD
  GS_CHECK_LAUNCH();
  return GS_OK;
}

// The image-space backward of gs_render_bwd and gs_render_bwd_adam: grad2d
// zeroed, the tile order measured (when asked), then one launch over the
// tiles accumulating grad2d.
static gs_status image_bwd(int64_t n, const CamDev& cd, const float* splats, const uint32_t* vals,
                           const uint32_t* ranges, const float* bg, const float* T_final,
                           const uint32_t* n_contrib, const float* dL_dimage,
                           const float* dL_ddepth, double* grad2d, uint32_t* tile_order,
                           hipStream_t st) {
  k_zero_f64<<<div_up(n * GS_GRAD2D_COMPONENTS, 256), 256, 0, st>>>(grad2d,
                                                                     n * GS_GRAD2D_COMPONENTS);
  GS_CHECK_LAUNCH();
  const int nt = cd.tiles_x * cd.tiles_y;
  const int px = tuning().bwd_px;
  const uint32_t* order = nullptr;
  if (tile_order) {  // [0, nt): the order; [nt, 2 nt): per-tile work
    uint32_t* work = tile_order + nt;
    GS_TIMED("tile_order", st, {
      if (cd.tile == 8) k_tile_work<8><<<nt, 256, 0, st>>>(n_contrib, cd.W, cd.H, cd.tiles_y, work);
      else if (cd.tile == 16) k_tile_work<16><<<nt, 256, 0, st>>>(n_contrib, cd.W, cd.H, cd.tiles_y, work);
      else k_tile_work<32><<<nt, 256, 0, st>>>(n_contrib, cd.W, cd.H, cd.tiles_y, work);
      k_tile_rank<<<1, 1024, 0, st>>>(work, nt, tile_order);
    });
    GS_CHECK_LAUNCH();
    order = tile_order;
  }
#define GS_BWD3(TL, PXV, DEP, NW)                                                              \
  k_render_bwd<TL, PXV, DEP, NW><<<bwd_split<TL, PXV>(nt, order != nullptr) +                  \
                                       div_up((int64_t)nt * bwd_regions<TL, PXV>(), NW),       \
                                   NW * kWave, 0, st>>>(                                       \
      splats, vals, ranges, cd.W, cd.H, nt, cd.tiles_y, bg[0], bg[1], bg[2], T_final,          \
      n_contrib, dL_dimage, dL_ddepth, grad2d, n, order, order ? tile_order + nt : nullptr)
#define GS_BWD2(TL, PXV, DEP)                                                                  \
  if (bwd_can_split<TL, PXV>() && order && nt * bwd_regions<TL, PXV>() <= kBwdFewRegions)      \
    GS_BWD3(TL, PXV, DEP, (bwd_can_split<TL, PXV>() ? 8 : 4));                                 \
  else GS_BWD3(TL, PXV, DEP, 4)
#define GS_BWD(TL, PXV) \
  if (dL_ddepth) { GS_BWD2(TL, PXV, true); } else { GS_BWD2(TL, PXV, false); }
  GS_TIMED("render_bwd", st, if (cd.tile == 8) { GS_BWD(8, 1); }
           else if (cd.tile == 16) {
             if (px == 4) { GS_BWD(16, 4); } else if (px == 2) { GS_BWD(16, 2); }
             else { GS_BWD(16, 1); }
           } else {
             if (px == 4) { GS_BWD(32, 4); } else { GS_BWD(32, 2); }
           });
#undef GS_BWD
#undef GS_BWD2
#undef GS_BWD3
  GS_CHECK_LAUNCH();
  return GS_OK;
}

extern "C" gs_status gs_render_bwd(const gs_gaussians* g, int64_t n, int32_t sh_degree,
                                   const gs_camera* cam, const float* splats,
                                   const uint32_t* vals, const uint32_t* ranges, const float* bg,
                                   const float* T_final, const uint32_t* n_contrib,
                                   const float* dL_dimage, const float* dL_ddepth, double* grad2d,
                                   gs_gaussians* grads, int32_t accumulate, uint32_t* tile_order,
                                   void* stream) {
  CamDev cd;
  if (n < 0 || sh_degree < GS_DIRECT || sh_degree > 3 || !make_cam(cam, &cd) || !ranges || !bg ||
      !T_final || !n_contrib || !dL_dimage || !grad2d || !aligned16(grad2d) || !g || !grads)
    return GS_EINVAL;
  if (n == 0) return GS_OK;
  hipStream_t st = (hipStream_t)stream;
  const gs_status s = image_bwd(n, cd, splats, vals, ranges, bg, T_final, n_contrib, dL_dimage,
                                dL_ddepth, grad2d, tile_order, st);
  if (s != GS_OK) return s;
  return launch_preprocess_bwd(g, n, sh_degree, cd, grad2d, grads, accumulate, st);
}

static bool gaussians_set(const gs_gaussians& g) {
  return g.means && g.log_scales && g.quats && g.opacity_logits && g.sh;
}

extern "C" gs_status gs_render_bwd_adam(gs_gaussians* g, int64_t n, int32_t sh_degree,
                                        const gs_camera* cam, const float* splats,
                                        const uint32_t* vals, const uint32_t* ranges,
                                        const float* bg, const float* T_final,
                                        const uint32_t* n_contrib, const float* dL_dimage,
                                        const float* dL_ddepth, double* grad2d,
                                        const gs_adam_params* adam, uint32_t* tile_order,
                                        void* stream) {
  CamDev cd;
  if (n < 0 || sh_degree < GS_DIRECT || sh_degree > 3 || !make_cam(cam, &cd) || !ranges || !bg ||
      !T_final || !n_contrib || !dL_dimage || !grad2d || !aligned16(grad2d) || !g || !adam ||
      !adam->step)
    return GS_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  if (n > 0) {
    if (!gaussians_set(*g) || !gaussians_set(adam->m) || !gaussians_set(adam->v))
      return GS_EINVAL;
    gs_status s = image_bwd(n, cd, splats, vals, ranges, bg, T_final, n_contrib, dL_dimage,
                            dL_ddepth, grad2d, tile_order, st);
    if (s != GS_OK) return s;
    s = launch_preprocess_bwd_adam(g, n, sh_degree, cd, grad2d, adam, st);
    if (s != GS_OK) return s;
  }
  return launch_step_advance(adam->step, st);
}

extern "C" gs_status gs_render_fwd_ckpt(const float* splats, int64_t n, const uint32_t* vals,
                                        const uint32_t* ranges, const gs_camera* cam,
                                        const float* bg, float* image, float* depth,
                                        float* T_final, uint32_t* n_contrib, float* ckpt,
                                        int32_t ckpt_buckets, uint32_t* ckpt_overflow,
                                        void* stream) {
  CamDev cd;
  if (n < 0 || !make_cam(cam, &cd) || cd.tile != 16 || ckpt_buckets < 1 || !ranges || !bg ||
      !image || !depth || !T_final || !n_contrib || !ckpt || !ckpt_overflow)
    return GS_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const int nt = cd.tiles_x * cd.tiles_y;
  GS_TIMED("render_fwd", st,
           k_render_fwd_ckpt<<<nt, 256, 0, st>>>(splats, vals, ranges, n, cd.W, cd.H, cd.tiles_y,
                                                 bg[0], bg[1], bg[2], image, depth, T_final,
                                                 n_contrib, ckpt, ckpt_buckets, ckpt_overflow));
  GS_CHECK_LAUNCH();
  return GS_OK;
}

extern "C" gs_status gs_render_bwd_ckpt(const gs_gaussians* g, int64_t n, int32_t sh_degree,
                                        const gs_camera* cam, const float* splats,
                                        const uint32_t* vals, const uint32_t* ranges,
                                        const float* image, const float* depth,
                                        const uint32_t* n_contrib, const float* ckpt,
                                        int32_t ckpt_buckets, const float* dL_dimage,
                                        const float* dL_ddepth, double* grad2d,
                                        gs_gaussians* grads, int32_t accumulate, void* stream) {
  CamDev cd;
  if (n < 0 || sh_degree < GS_DIRECT || sh_degree > 3 || !make_cam(cam, &cd) || cd.tile != 16 ||
      ckpt_buckets < 1 || !ranges || !image || !n_contrib || !ckpt || !dL_dimage || !grad2d ||
      !aligned16(grad2d) ||
      !g || !grads || (dL_ddepth && !depth))
    return GS_EINVAL;
  if (n == 0) return GS_OK;
  hipStream_t st = (hipStream_t)stream;
  k_zero_f64<<<div_up(n * GS_GRAD2D_COMPONENTS, 256), 256, 0, st>>>(grad2d,
                                                                     n * GS_GRAD2D_COMPONENTS);
  GS_CHECK_LAUNCH();
  const int nt = cd.tiles_x * cd.tiles_y;
  GS_TIMED("render_bwd", st, if (dL_ddepth) {
    k_render_bwd_ckpt<true><<<nt, 256, 0, st>>>(splats, vals, ranges, cd.W, cd.H, cd.tiles_y,
                                                image, depth, n_contrib, ckpt, ckpt_buckets,
                                                dL_dimage, dL_ddepth, grad2d, n);
  } else {
    k_render_bwd_ckpt<false><<<nt, 256, 0, st>>>(splats, vals, ranges, cd.W, cd.H, cd.tiles_y,
                                                 image, depth, n_contrib, ckpt, ckpt_buckets,
                                                 dL_dimage, nullptr, grad2d, n);
  });
  GS_CHECK_LAUNCH();
  return launch_preprocess_bwd(g, n, sh_degree, cd, grad2d, grads, accumulate, st);
}

extern "C" gs_status gs_split_score(const float* splats, int64_t n, const uint32_t* vals,
                                    const uint32_t* ranges, const gs_camera* cam,
                                    const uint8_t* mask, uint32_t* score, void* stream) {
  CamDev cd;
  if (n < 0 || !make_cam(cam, &cd) || !ranges || !mask || !score || (n > 0 && !splats))
    return GS_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const int nt = cd.tiles_x * cd.tiles_y;
#define GS_SCORE(TL) \
  k_split_score<TL><<<nt, TL * TL, 0, st>>>(splats, vals, ranges, n, cd.W, cd.H, cd.tiles_y, mask, score)
  GS_TIMED("split_score", st, if (cd.tile == 8) GS_SCORE(8); else if (cd.tile == 16) GS_SCORE(16);
           else GS_SCORE(32));
#undef GS_SCORE
  GS_CHECK_LAUNCH();
  return GS_OK;
}

// ---------------------------------------------------------------------------
namespace {

int cu_count() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cached[dev]) {
    int c = 0;
    if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c <= 0)
      c = 256;
    cached[dev] = c;
  }
  return cached[dev];
}

// Validates a view batch for the render phases; fills the work queue layout.
bool make_view_set(const gs_view* views, int32_t n_views, bool bwd, ViewSet* vs, int* tile,
                   bool* any_depth) {
  if (!views || n_views < 1 || n_views > GS_MAX_VIEWS) return false;
  vs->n_views = n_views;
  vs->start[0] = 0;
  *any_depth = false;
  for (int v = 0; v < n_views; ++v) {
    CamDev cd;
    const gs_view& w = views[v];
    if (!make_cam(&w.cam, &cd)) return false;
    if (v == 0) *tile = cd.tile;
    if (cd.tile != *tile) return false;
    if (!w.ranges || !w.T_final || !w.n_contrib) return false;
    if (!bwd && (!w.image || !w.depth)) return false;
    if (bwd && (!w.dL_dimage || !w.grad2d || !aligned16(w.grad2d))) return false;
    vs->W[v] = cd.W;
    vs->H[v] = cd.H;
    vs->tiles_y[v] = cd.tiles_y;
    vs->splats[v] = w.splats;
    vs->vals[v] = w.vals;
    vs->ranges[v] = w.ranges;
    vs->image[v] = w.image;
    vs->depth[v] = w.depth;
    vs->T_final[v] = w.T_final;
    vs->n_contrib[v] = w.n_contrib;
    vs->dL_dimage[v] = w.dL_dimage;
    vs->dL_ddepth[v] = w.dL_ddepth;
    vs->grad2d[v] = w.grad2d;
    if (w.dL_ddepth) *any_depth = true;
    vs->start[v + 1] = vs->start[v] + cd.tiles_x * cd.tiles_y;
  }
  vs->total = vs->start[n_views];
  return true;
}

int persistent_grid(int total, int wgs_per_cu) {
  const int g = cu_count() * wgs_per_cu;
  return g < total ? g : total;
}

}  // namespace

extern "C" gs_status gs_render_fwd_batched(int64_t n, const gs_view* views, int32_t n_views,
                                           const float* bg, uint32_t* queue, void* stream) {
  ViewSet vs;
  int tile = 16;
  bool any_depth;
  if (n < 0 || !bg || !queue || !make_view_set(views, n_views, false, &vs, &tile, &any_depth))
    return GS_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const int px = tuning().fwd_px;
  const int grid = persistent_grid(vs.total, tuning().persist_wgs);
  k_reset_queue<<<1, 1, 0, st>>>(queue);
  GS_CHECK_LAUNCH();
  const int fb = tuning().fwd_batch;
#define GS_FWDB3(TL, PXV, NBV)                                                                   \
  k_render_fwd_batched<TL, PXV, NBV><<<grid, TL * TL / PXV, 0, st>>>(vs, n, bg[0], bg[1], bg[2], \
                                                                     queue)
#define GS_FWDB(TL, PXV)                                 \
  do {                                                   \
    if (fb == 64) GS_FWDB3(TL, PXV, 64);                 \
    else if (fb == 128) GS_FWDB3(TL, PXV, 128);          \
    else GS_FWDB3(TL, PXV, 256);                         \
  } while (0)
  GS_TIMED("render_fwd", st, if (tile == 8) GS_FWDB(8, 1);
           else if (tile == 16) {
             if (px == 4) GS_FWDB(16, 4); else if (px == 2) GS_FWDB(16, 2); else GS_FWDB(16, 1);
           } else {
             if (px == 4) GS_FWDB(32, 4); else if (px == 2) GS_FWDB(32, 2); else GS_FWDB(32, 1);
           });
#undef GS_FWDB
#undef GS_FWDB3
  GS_CHECK_LAUNCH();
  return GS_OK;
}

extern "C" gs_status gs_render_fwd_batched_deferred(int64_t n, const gs_view* views,
                                                    int32_t n_views, const void* const* workspaces,
                                                    const size_t* workspace_bytes, const float* bg,
                                                    uint32_t* queue, void* stream) {
  ViewSet vs;
  int tile = 16;
  bool any_depth;
  if (n < 0 || !bg || !queue || !workspaces || !workspace_bytes ||
      !make_view_set(views, n_views, false, &vs, &tile, &any_depth))
    return GS_EINVAL;
  for (int v = 0; v < n_views; ++v) {
    const gs_view& w = views[v];
    if (w.capacity < 0 || (w.capacity > 0 && !w.vals)) return GS_EINVAL;
    CamDev cd;
    if (!make_cam(&w.cam, &cd)) return GS_EINVAL;
    if (!run_lists(workspaces[v], workspace_bytes[v], n, w.capacity, cd.tiles_x, cd.tiles_y,
                   &vs.rl[v]))
      return GS_ECAPACITY;
  }
  hipStream_t st = (hipStream_t)stream;
  const int px = tuning().fwd_px;
  const int grid = persistent_grid(vs.total, tuning().persist_wgs);
  k_reset_queue<<<1, 1, 0, st>>>(queue);
  GS_CHECK_LAUNCH();
  const int fb = tuning().fwd_batch;
#define GS_FWDB3(TL, PXV, NBV)                                                               \
  k_render_fwd_batched_def<TL, PXV, NBV><<<grid, TL * TL / PXV, 0, st>>>(vs, n, bg[0], bg[1], \
                                                                         bg[2], queue)
#define GS_FWDB(TL, PXV)                                 \
  do {                                                   \
    if (fb == 64) GS_FWDB3(TL, PXV, 64);                 \
    else if (fb == 128) GS_FWDB3(TL, PXV, 128);          \
    else GS_FWDB3(TL, PXV, 256);                         \
  } while (0)
  GS_TIMED("render_fwd", st, if (tile == 8) GS_FWDB(8, 1);
           else if (tile == 16) {
             if (px == 4) GS_FWDB(16, 4); else if (px == 2) GS_FWDB(16, 2); else GS_FWDB(16, 1);
           } else {
             if (px == 4) GS_FWDB(32, 4); else if (px == 2) GS_FWDB(32, 2); else GS_FWDB(32, 1);
           });
#undef GS_FWDB
#undef GS_FWDB3
  GS_CHECK_LAUNCH();
  return GS_OK;
}

extern "C" gs_status gs_render_bwd_batched(const gs_gaussians* g, int64_t n, int32_t sh_degree,
                                           const gs_view* views, int32_t n_views,
                                           const float* bg, uint32_t* queue,
                                           gs_gaussians* grads, int32_t accumulate,
                                           uint32_t* tile_order, void* stream) {
  ViewSet vs;
  int tile = 16;
  bool any_depth;
  if (n < 0 || sh_degree < GS_DIRECT || sh_degree > 3 || !bg || !queue || !g || !grads ||
      (accumulate != 0 && accumulate != 1) ||
      !make_view_set(views, n_views, true, &vs, &tile, &any_depth))
    return GS_EINVAL;
  if (n == 0) return GS_OK;
  hipStream_t st = (hipStream_t)stream;
  for (int v = 0; v < n_views; ++v) {
    k_zero_f64<<<div_up(n * GS_GRAD2D_COMPONENTS, 256), 256, 0, st>>>(vs.grad2d[v],
                                                                       n * GS_GRAD2D_COMPONENTS);
    GS_CHECK_LAUNCH();
  }
  const int px = tuning().bwd_px;
  k_reset_queue<<<1, 1, 0, st>>>(queue);
  GS_CHECK_LAUNCH();
  const uint32_t* order = nullptr;
  if (tile_order && vs.total > 0) {  // [0, total): the order; [total, 2 total): the work
    uint32_t* work = tile_order + vs.total;
    GS_TIMED("tile_order", st, {
      if (tile == 8) k_tile_work_views<8><<<vs.total, 256, 0, st>>>(vs, work);
      else if (tile == 16) k_tile_work_views<16><<<vs.total, 256, 0, st>>>(vs, work);
      else k_tile_work_views<32><<<vs.total, 256, 0, st>>>(vs, work);
      k_tile_rank<<<1, 1024, 0, st>>>(work, vs.total, tile_order);
    });
    GS_CHECK_LAUNCH();
    order = tile_order;
  }
#define GS_BWDB2(TL, PXV, DEP)                                                          \
  k_render_bwd_batched<TL, PXV, DEP><<<                                                 \
      persistent_grid(bwd_split<TL, PXV>(vs.total, order != nullptr) +                  \
                          vs.total * bwd_regions<TL, PXV>(),                            \
                      div_up(tuning().persist_wgs * bwd_regions<TL, PXV>(),             \
                             4)),                                        \
      4 * kWave, 0, st>>>(vs, n, bg[0], bg[1], bg[2], queue, order,                         \
                      order ? tile_order + vs.total : nullptr)
#define GS_BWDB(TL, PXV) \
  if (any_depth) GS_BWDB2(TL, PXV, true); else GS_BWDB2(TL, PXV, false)
  GS_TIMED("render_bwd", st, if (tile == 8) { GS_BWDB(8, 1); }
           else if (tile == 16) {
             if (px == 4) { GS_BWDB(16, 4); } else if (px == 2) { GS_BWDB(16, 2); }
             else { GS_BWDB(16, 1); }
           } else {
             if (px == 4) { GS_BWDB(32, 4); } else { GS_BWDB(32, 2); }
           });
#undef GS_BWDB
#undef GS_BWDB2
  GS_CHECK_LAUNCH();
  CamDev cds[GS_MAX_VIEWS];
  const double* g2[GS_MAX_VIEWS];
  for (int v = 0; v < n_views; ++v) {
    make_cam(&views[v].cam, &cds[v]);
    g2[v] = vs.grad2d[v];
  }
  return launch_preprocess_bwd_views(g, n, sh_degree, cds, g2, n_views, grads, accumulate, st);
}
