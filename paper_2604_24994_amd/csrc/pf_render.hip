// Rendering: tile rasteriser and ray walk over a built scene.
//
// Raster, per view (Sec. 3.2, rasterization; appendix B order):
//   k_view_count  per cell: power distance from the camera centre (the sort
//                 key) and the tile rectangle of its ball
//   scan          cell offsets into the pair list
//   k_view_emit   (tile, key<<32 | cell) pairs + tile histogram
//   scan/scatter  counting sort by tile
//   k_tile_sort   per tile, sort by (key, cell) in LDS (bitonic, global
//                 memory fallback for long lists)
//   k_split_plan  which tiles go to which of the two composites
//   k_raster      one 256-thread workgroup per 16x16 tile, one lane per
//                 pixel, each wave an 8x8 quadrant walking the tile's list
//                 front to back; the list and the cells' records are staged
//                 in LDS 256 entries at a time by the whole workgroup, and
//                 cells that miss the quadrant are dropped 64 at a time
//   k_raster_split  tiles with long lists: sixteen waves per 8x8 quadrant
// Trace, per view (Sec. 3.2, ray tracing; appendix C):
//   k_start_*     argmin power distance from the camera centre
//   k_trace       one lane per ray; per step the piece of the current cell
//                 (same device code as the rasteriser) and the exit face in one
//                 pass over its faces; colours evaluated for many rays at once
#include "pf_internal.hpp"
#include "pf_render.hpp"
#include "pf_shade.hpp"

#include <algorithm>
#include <cmath>
#include <vector>

namespace pf {
namespace {

__device__ inline uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr double RECT_PAD = 1e-2;   // pixels

// Pixels by which a ball's bounds on the image are widened.  A ray's direction
// is M v (M the camera's 3x3 matrix), while the bounds come from v' = M^T e of
// the centre e, which is M^-1 e + E M^-1 e with E = M^T M - 1: a rotation
// rounded to float32 moves them by less than 1e-3 pixels, a matrix written with
// a few digits, or with an axis scaled a little, by up to some pixels.  Where
// the shift (|E| and the ray's own float32 rounding, times the pixels per unit
// of angle at the image's corner) may reach half of RECT_PAD, the pad is a pixel.
double rect_pad(const pf_camera& c) {
  double e2 = 0.0;
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      double d = i == j ? -1.0 : 0.0;
      for (int r = 0; r < 3; ++r) d += (double)c.c2w[4 * r + i] * (double)c.c2w[4 * r + j];
      e2 += d * d;
    }
  double scale;
  if (c.model == 0) {
    const double x = std::max(std::fabs((double)c.cx), std::fabs(c.width - (double)c.cx)) / c.fx;
    const double y = std::max(std::fabs((double)c.cy), std::fabs(c.height - (double)c.cy)) / c.fy;
    scale = std::max(c.fx, c.fy) * (1.0 + x * x + y * y);
  } else {
    scale = c.f_fish * (double)c.theta_max / std::sin(std::min((double)c.theta_max, 3.0));
  }
  return (std::sqrt(e2) + 1.2e-7) * scale <= 0.5 * RECT_PAD ? RECT_PAD : 1.0;
}

// Tile rectangle of a ball (camera-space centre X,Y,Z, radius rho).
__device__ bool ball_rect(const pf_camera& c, double pad, double X, double Y, double Z, double rho, int tiles_x,
                          int tiles_y, int& x0, int& x1, int& y0, int& y1) {
  const double W = c.width, H = c.height;
  double ulo, uhi, vlo, vhi;
  bool full = false;
  if (c.model == 0) {
    if (Z + rho <= 0.0) return false;
    if (Z - rho <= 1e-9 * (1.0 + fabs(Z))) {
      full = true;
    } else {
      const double zz = Z * Z - rho * rho;
      const double sx = rho * sqrt(fmax(0.0, X * X + zz));
      const double sy = rho * sqrt(fmax(0.0, Y * Y + zz));
      const double kxl = (X * Z - sx) / zz, kxh = (X * Z + sx) / zz;
      const double kyl = (Y * Z - sy) / zz, kyh = (Y * Z + sy) / zz;
      ulo = (double)c.fx * kxl + (double)c.cx;
      uhi = (double)c.fx * kxh + (double)c.cx;
      vlo = (double)c.fy * kyl + (double)c.cy;
      vhi = (double)c.fy * kyh + (double)c.cy;
    }
  } else {
    const double Lc = sqrt(X * X + Y * Y + Z * Z);
    if (Lc <= rho * (1.0 + 1e-9)) {
      full = true;
    } else {
      const double beta = asin(fmin(1.0, rho / Lc));
      const double thc = acos(fmax(-1.0, fmin(1.0, Z / Lc)));
      const double tmax = (double)c.theta_max;
      if (thc - beta > tmax) return false;
      const double f = (double)c.f_fish;
      const double thi = fmin(tmax, thc + beta);
      const double rhi = f * thi;
      if (thc <= beta || thc + beta >= M_PI) {
        ulo = c.cx - rhi; uhi = c.cx + rhi;
        vlo = c.cy - rhi; vhi = c.cy + rhi;
      } else {
        const double tlo = fmax(0.0, thc - beta);
        const double rlo = f * tlo;
        const double phc = atan2(Y, X);
        const double dph = asin(fmin(1.0, sin(beta) / sin(thc)));
        const double pa = phc - dph, pb = phc + dph;
        ulo = vlo = INFINITY;
        uhi = vhi = -INFINITY;
        const double ph[2] = {pa, pb}, rr[2] = {rlo, rhi};
        for (int i = 0; i < 2; ++i)
          for (int j = 0; j < 2; ++j) {
            const double u = c.cx + rr[j] * cos(ph[i]), v = c.cy + rr[j] * sin(ph[i]);
            ulo = fmin(ulo, u); uhi = fmax(uhi, u);
            vlo = fmin(vlo, v); vhi = fmax(vhi, v);
          }
        // axis-aligned extremes of the outer arc inside [pa, pb]
        for (int q = -4; q <= 4; ++q) {
          const double a = q * (M_PI / 2);
          if (a > pa && a < pb) {
            const double u = c.cx + rhi * cos(a), v = c.cy + rhi * sin(a);
            ulo = fmin(ulo, u); uhi = fmax(uhi, u);
            vlo = fmin(vlo, v); vhi = fmax(vhi, v);
          }
        }
      }
    }
  }
  if (full) {
    x0 = 0; x1 = tiles_x - 1;
    y0 = 0; y1 = tiles_y - 1;
    return true;
  }
  // pixels whose centre (p + 1/2) may lie in [lo, hi] (a ball between two pixel
  // centres has none), padded by rect_pad
  const double pxl = ceil(ulo - 0.5 - pad), pxh = floor(uhi - 0.5 + pad);
  const double pyl = ceil(vlo - 0.5 - pad), pyh = floor(vhi - 0.5 + pad);
  if (!(pxh >= 0.0 && pyh >= 0.0 && pxl <= W - 1 && pyl <= H - 1 && pxl <= pxh && pyl <= pyh)) return false;
  x0 = (int)fmax(0.0, floor(fmax(pxl, 0.0) / TILE));
  x1 = (int)fmin((double)(tiles_x - 1), floor(fmin(pxh, W - 1) / TILE));
  y0 = (int)fmax(0.0, floor(fmax(pyl, 0.0) / TILE));
  y1 = (int)fmin((double)(tiles_y - 1), floor(fmin(pyh, H - 1) / TILE));
  return x0 <= x1 && y0 <= y1;
}

struct ViewArgs {
  pf_camera cam;
  int tiles_x, tiles_y;
  double pad;   // rect_pad
};

// One camera of a batched raster call: its tiles are numbered from
// tile_base and its pixels from pix_base across the whole batch.
struct ViewDev {
  ViewArgs v;
  long long tile_base;
  long long pix_base;
  int view_id;   // camera index within the call
};

// A ball that crosses the plane of a pinhole camera (camera outside the
// ball) has no bounded screen rectangle; the pixel rays that meet it are
// those within the cone of half-angle asin(rho/|c|) around the direction c
// to its centre.  A tile is kept when the angle between its centre ray and
// c is at most that half-angle plus the tile's own angular radius.
struct Cone {
  double ax, ay, az;   // unit direction to the centre, camera axes
  double cmin;         // cosine of the widened half-angle
};

__device__ inline bool cone_tile(const pf_camera& c, const Cone& k, int tx, int ty) {
  const double dx = ((double)(tx * TILE) + 0.5 * TILE - (double)c.cx) / (double)c.fx;
  const double dy = ((double)(ty * TILE) + 0.5 * TILE - (double)c.cy) / (double)c.fy;
  const double dot = dx * k.ax + dy * k.ay + k.az;
  // dot / |d| >= cmin, without the square root
  if (k.cmin <= 0.0 && dot >= 0.0) return true;
  const double d2 = dx * dx + dy * dy + 1.0;
  return k.cmin >= 0.0 ? (dot >= 0.0 && dot * dot >= k.cmin * k.cmin * d2) : (dot * dot <= k.cmin * k.cmin * d2);
}

// Tile footprint of a cell's ball in a view: 0 none, 1 the rectangle
// [x0, x1] x [y0, y1], 2 the tiles of that rectangle (all of the view)
// accepted by cone_tile(k).
__device__ inline int cell_rect(const ViewArgs& v, const float4 g, int& x0, int& x1, int& y0, int& y1,
                                Cone& k) {
  if (!(g.w >= 0.0f)) return 0;
  const float* m = v.cam.c2w;
  const double ex = (double)g.x - m[3], ey = (double)g.y - m[7], ez = (double)g.z - m[11];
  const double X = m[0] * ex + m[4] * ey + m[8] * ez;
  const double Y = m[1] * ex + m[5] * ey + m[9] * ez;
  const double Z = m[2] * ex + m[6] * ey + m[10] * ez;
  const double r = (double)g.w * (1.0 + 1e-5) + 1e-7;
  if (!ball_rect(v.cam, v.pad, X, Y, Z, r, v.tiles_x, v.tiles_y, x0, x1, y0, y1)) return 0;
  if (v.cam.model == 0 && Z - r <= 1e-9 * (1.0 + fabs(Z))) {
    const double L = sqrt(X * X + Y * Y + Z * Z);
    if (L > r * (1.0 + 1e-9)) {
      // tile angular radius: half diagonal of a tile plus the one-pixel pad
      const double tile_ang = (0.5 * TILE + 1.0) * 1.4142135623730951 / fmin((double)v.cam.fx, (double)v.cam.fy);
      const double ang = asin(r / L) + tile_ang + 1e-6;
      k.ax = X / L;
      k.ay = Y / L;
      k.az = Z / L;
      k.cmin = ang >= M_PI ? -1.0 : cos(ang);
      return 2;
    }
  }
  return 1;
}

// What live_ball takes.
struct BallArgs {
  const float4* geo;
  const float* cull;
  float4* ball;
  const float* ball_top;
  const float* tex;
};

// The cells' balls for a group of several views (live_ball).
__global__ void k_live_ball(BallArgs b, int64_t n, float4* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool grown;
  if (i < n) out[i] = live_ball(b.geo, b.cull, b.ball, b.ball_top, b.tex, i, grown);
}

// blockIdx.y = view; one thread per (view, cell).
// Cells whose footprint needs the per-tile cone test are listed in
// cone_list (as view * n + cell) and counted by k_cone_count.
// LIVE (one view): the balls are formed here; else k_live_ball did.
template <bool LIVE>
__global__ void k_view_count(const ViewDev* __restrict__ views, BallArgs b, float4* __restrict__ live,
                             const float* __restrict__ power, int64_t n, uint32_t* __restrict__ cnt,
                             uint32_t* __restrict__ key, uint32_t* __restrict__ cone_list,
                             uint32_t* __restrict__ cone_n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const ViewArgs& v = views[blockIdx.y].v;
  const int64_t o = (int64_t)blockIdx.y * n + i;
  const float4 g = b.geo[i];
  int x0, x1, y0, y1;
  Cone k;
  uint32_t c = 0;
  float4 bl;
  if constexpr (LIVE) {
    bool grown;
    bl = live[i] = live_ball(b.geo, b.cull, b.ball, b.ball_top, b.tex, i, grown);
  } else {
    bl = live[i];
  }
  const int mode = cell_rect(v, bl, x0, x1, y0, y1, k);
  if (o == 0) cnt[(int64_t)gridDim.y * n] = 0;   // (the scan's last entry)
  if (mode == 1) {
    c = (uint32_t)((x1 - x0 + 1) * (y1 - y0 + 1));
  } else if (mode == 2) {
    cone_list[atomicAdd(cone_n, 1u)] = (uint32_t)o;
  }
  cnt[o] = c;
  const float* m = v.cam.c2w;
  const double ex = (double)m[3] - g.x, ey = (double)m[7] - g.y, ez = (double)m[11] - g.z;
  key[o] = order_key((float)(ex * ex + ey * ey + ez * ez - (double)power[i]));
}

// blockIdx.y = view; a lane per (view, cell).  A wave emits its cells'
// pixel rectangles together: after a scan of the pair counts over the wave,
// it writes 64 pairs at a time, pair p taken by the lane whose run holds p,
// so that a cell whose footprint covers many tiles is spread over the wave
// rather than holding it, and the stores of a step are contiguous.  A
// cell's pairs keep the order of its rectangle (rows of tiles, then tiles).
__global__ void __launch_bounds__(256) k_view_emit(const ViewDev* __restrict__ views, const float4* __restrict__ ball, int64_t n,
                                                   const uint32_t* __restrict__ off, const uint32_t* __restrict__ key,
                                                   uint32_t* __restrict__ ptile, unsigned long long* __restrict__ pval,
                                                   uint32_t* __restrict__ tile_cnt) {
  __shared__ int s_end[4][64];   // end of each lane's run of the wave's pairs
  __shared__ int s_x0[4][64], s_y0[4][64], s_w[4][64];
  __shared__ uint32_t s_o[4][64];
  __shared__ unsigned long long s_val[4][64];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const ViewDev& vd = views[blockIdx.y];
  int nt = 0, x0 = 0, x1 = -1, y0 = 0, y1 = -1;
  uint32_t o = 0;
  unsigned long long val = 0;
  if (i < n) {
    const int64_t oi = (int64_t)blockIdx.y * n + i;
    Cone k;
    const int mode = cell_rect(vd.v, ball[i], x0, x1, y0, y1, k);
    if (mode == 1) {   // (cone footprints: k_cone_emit)
      nt = (x1 - x0 + 1) * (y1 - y0 + 1);
      o = off[oi];
      val = ((unsigned long long)key[oi] << 32) | (uint32_t)i;
    }
  }
  int end = nt;
  for (int d = 1; d < 64; d <<= 1) {
    const int t = __shfl_up(end, d, 64);
    if (lane >= d) end += t;
  }
  const int total = __shfl(end, 63, 64);
  s_end[wv][lane] = end;
  s_x0[wv][lane] = x0;
  s_y0[wv][lane] = y0;
  s_w[wv][lane] = x1 - x0 + 1;
  s_o[wv][lane] = o;
  s_val[wv][lane] = val;
  __syncthreads();
  const uint32_t tbase = (uint32_t)vd.tile_base;
  const int tiles_x = vd.v.tiles_x;
  for (int base = 0; base < total; base += 64) {
    const int p = base + lane;
    if (p >= total) break;
    // owner: the first lane whose run ends after p
    int lo = 0, hi = 63;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (s_end[wv][mid] > p) hi = mid;
      else lo = mid + 1;
    }
    const int r = p - (lo == 0 ? 0 : s_end[wv][lo - 1]);
    const int w = s_w[wv][lo];
    const int ty = s_y0[wv][lo] + r / w, tx = s_x0[wv][lo] + r % w;
    const uint32_t t = tbase + (uint32_t)(ty * tiles_x + tx);
    const uint32_t at = s_o[wv][lo] + (uint32_t)r;
    ptile[at] = t;
    pval[at] = s_val[wv][lo];
    atomicAdd(&tile_cnt[t], 1u);
  }
}

// One workgroup per listed (view, cell): its threads test the tiles of the
// view in parallel.  The grid may be larger than the list (cone_n).  (A grid of
// fixed size whose workgroups take cells in turn keeps 165 instead of 62 registers
// and took 0.66 and 0.45 ms instead of 0.35 for 8 views of a 1M-cell scene.)
__global__ void __launch_bounds__(256) k_cone_count(const ViewDev* __restrict__ views,
                                                    const float4* __restrict__ ball, int64_t n,
                                                    const uint32_t* __restrict__ cone_list,
                                                    const uint32_t* __restrict__ cone_n,
                                                    uint32_t* __restrict__ cnt) {
  __shared__ uint32_t part[4];
  if (blockIdx.x >= *cone_n) return;
  const uint32_t o = cone_list[blockIdx.x];
  const int64_t i = (int64_t)(o % (uint64_t)n);
  const ViewArgs& v = views[o / (uint64_t)n].v;
  int x0, x1, y0, y1;
  Cone k;
  (void)cell_rect(v, ball[i], x0, x1, y0, y1, k);
  const int tw = x1 - x0 + 1, nt = tw * (y1 - y0 + 1);
  uint32_t c = 0;
  for (int t = threadIdx.x; t < nt; t += 256) c += cone_tile(v.cam, k, x0 + t % tw, y0 + t / tw) ? 1u : 0u;
  for (int sh = 32; sh > 0; sh >>= 1) c += __shfl_xor(c, sh, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) cnt[o] = part[0] + part[1] + part[2] + part[3];
}

__global__ void __launch_bounds__(256) k_cone_emit(const ViewDev* __restrict__ views, const float4* __restrict__ ball, int64_t n,
                                                   const uint32_t* __restrict__ off, const uint32_t* __restrict__ key,
                                                   const uint32_t* __restrict__ cone_list,
                                                   const uint32_t* __restrict__ cone_n,
                                                   uint32_t* __restrict__ ptile, unsigned long long* __restrict__ pval,
                                                   uint32_t* __restrict__ tile_cnt) {
  __shared__ uint32_t wsum[4];
  if (blockIdx.x >= *cone_n) return;
  const uint32_t o = cone_list[blockIdx.x];
  const int64_t i = (int64_t)(o % (uint64_t)n);
  const ViewDev& vd = views[o / (uint64_t)n];
  int x0, x1, y0, y1;
  Cone k;
  (void)cell_rect(vd.v, ball[i], x0, x1, y0, y1, k);
  const int tw = x1 - x0 + 1, nt = tw * (y1 - y0 + 1);
  const unsigned long long val = ((unsigned long long)key[o] << 32) | (uint32_t)i;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t base = off[o];
  for (int t0 = 0; t0 < nt; t0 += 256) {
    const int t = t0 + threadIdx.x;
    const int tx = x0 + t % tw, ty = y0 + t / tw;
    const bool pass = t < nt && cone_tile(vd.v.cam, k, tx, ty);
    const uint64_t m = __ballot(pass);
    if (lane == 0) wsum[wv] = (uint32_t)__popcll(m);
    __syncthreads();
    uint32_t before = 0, total = 0;
    for (int w = 0; w < 4; ++w) {
      before += w < wv ? wsum[w] : 0u;
      total += wsum[w];
    }
    if (pass) {
      const uint32_t pos = base + before + (uint32_t)__popcll(m & lt);
      const uint32_t tile = (uint32_t)(vd.tile_base + ty * vd.v.tiles_x + tx);
      ptile[pos] = tile;
      pval[pos] = val;
      atomicAdd(&tile_cnt[tile], 1u);
    }
    base += total;
    __syncthreads();
  }
}

__global__ void k_tile_scatter(const uint32_t* __restrict__ ptile, const unsigned long long* __restrict__ pval,
                               int64_t np, const uint32_t* __restrict__ tile_off, uint32_t* __restrict__ fill,
                               unsigned long long* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= np) return;
  const uint32_t t = ptile[i];
  const uint32_t pos = tile_off[t] + atomicAdd(&fill[t], 1u);
  out[pos] = pval[i];
}

constexpr int SORT_THREADS = 256;
constexpr int SORT_LDS = 4096;

// One stage (k, j) of a bitonic network in its "flip" form (every comparator
// puts the smaller value at the lower index) over buf[0, n), n <= n2 a power of
// two: the missing tail counts as +infinity and is never touched.
template <int THREADS>
__device__ inline void bitonic_stage(unsigned long long* buf, uint32_t n, uint32_t n2, uint32_t k, uint32_t j) {
  for (uint32_t t = threadIdx.x; t < n2 / 2; t += THREADS) {
    // t-th comparator of this stage: lower index i has bit j clear
    const uint32_t i = ((t & ~(j - 1)) << 1) | (t & (j - 1));   // (j a power of two)
    const uint32_t p = (j == (k >> 1)) ? (i ^ (k - 1)) : (i + j);
    if (p < n) {
      const unsigned long long x = buf[i], y = buf[p];
      if (y < x) {
        buf[i] = y;
        buf[p] = x;
      }
    }
  }
  __syncthreads();
}

// Ascending sort of one tile's segment in LDS; tiles with longer lists are
// noted in long_list (*long_n of them) for k_tile_sort_long.
__global__ void __launch_bounds__(SORT_THREADS) k_tile_sort(unsigned long long* __restrict__ vals,
                                                            const uint32_t* __restrict__ tile_off,
                                                            uint32_t* __restrict__ long_list,
                                                            uint32_t* __restrict__ long_n) {
  __shared__ unsigned long long sh[SORT_LDS];
  const uint32_t a = tile_off[blockIdx.x], b = tile_off[blockIdx.x + 1];
  const uint32_t n = b - a;
  if (n <= 1) return;
  if (n > SORT_LDS) {
    if (threadIdx.x == 0) long_list[atomicAdd(long_n, 1u)] = blockIdx.x;
    return;
  }
  uint32_t n2 = 1;
  while (n2 < n) n2 <<= 1;
  for (uint32_t i = threadIdx.x; i < n; i += SORT_THREADS) sh[i] = vals[a + i];
  __syncthreads();
  for (uint32_t k = 2; k <= n2; k <<= 1)
    for (uint32_t j = k >> 1; j > 0; j >>= 1) bitonic_stage<SORT_THREADS>(sh, n, n2, k, j);
  for (uint32_t i = threadIdx.x; i < n; i += SORT_THREADS) vals[a + i] = sh[i];
}

constexpr int SORT_LONG_THREADS = 1024;
constexpr uint32_t SORT_LONG_LDS = 16384;

// The lists beyond SORT_LDS entries, a workgroup each, in turn: sixteen waves
// and 128 kB of LDS.  Runs of SORT_LONG_LDS entries are sorted in LDS; beyond
// that, only the stages whose comparators span two runs (one or two per doubling)
// work in global memory, the rest of each merge is done run by run in LDS again.
// The network is bound by the latency of its stages.  For four views up to
// 1920x1080 at 1,048,576 cells (lists of up to 44 thousand) the sorts take
// 0.79 ms; 2.6 with all stages of a long list in global memory and 256 threads.
__global__ void __launch_bounds__(SORT_LONG_THREADS) k_tile_sort_long(unsigned long long* __restrict__ vals,
                                                                      const uint32_t* __restrict__ tile_off,
                                                                      const uint32_t* __restrict__ long_list,
                                                                      const uint32_t* __restrict__ long_n) {
  __shared__ unsigned long long sh[SORT_LONG_LDS];
  const uint32_t count = *long_n;
  for (uint32_t l = blockIdx.x; l < count; l += gridDim.x) {
    const uint32_t tile = long_list[l];
    const uint32_t n = tile_off[tile + 1] - tile_off[tile];
    unsigned long long* v = vals + tile_off[tile];
    uint32_t n2 = 1;
    while (n2 < n) n2 <<= 1;
    // all stages (k, j) with k in (k0, k1] and j below SORT_LONG_LDS, run by run
    auto runs = [&](uint32_t k0, uint32_t k1) {
      for (uint32_t r = 0; r < n; r += SORT_LONG_LDS) {
        const uint32_t m = min(n - r, SORT_LONG_LDS), m2 = min(n2, SORT_LONG_LDS);
        for (uint32_t i = threadIdx.x; i < m; i += SORT_LONG_THREADS) sh[i] = v[r + i];
        __syncthreads();
        for (uint32_t k = 2 * k0; k <= k1; k <<= 1)
          for (uint32_t j = min(k, SORT_LONG_LDS) >> 1; j > 0; j >>= 1)
            bitonic_stage<SORT_LONG_THREADS>(sh, m, m2, k, j);
        for (uint32_t i = threadIdx.x; i < m; i += SORT_LONG_THREADS) v[r + i] = sh[i];
        __syncthreads();
      }
    };
    runs(1, min(n2, SORT_LONG_LDS));
    for (uint32_t k = 2 * SORT_LONG_LDS; k <= n2; k <<= 1) {
      for (uint32_t j = k >> 1; j >= SORT_LONG_LDS; j >>= 1) bitonic_stage<SORT_LONG_THREADS>(v, n, n2, k, j);
      runs(k >> 1, k);
    }
  }
}

struct SceneDev {
  const float4* geo;
  const float4* nrm;
  const float4* ball;
  const int32_t* row;
  const int32_t* nrast;
  const int32_t* col;
  const float4* plane;
  const float* rgb;
  const float* tex;
  float tau;
};

// A cell's ball relative to the camera centre, its radius widened by what the
// float32 test below can be off (a few 1e-7 of the centre's distance).
__device__ inline float4 ball_from(const float4 ball, double ox, double oy, double oz) {
  const float x = (float)((double)ball.x - ox), y = (float)((double)ball.y - oy), z = (float)((double)ball.z - oz);
  return make_float4(x, y, z, ball.w + 1e-6f * (fabsf(x) + fabsf(y) + fabsf(z)));
}

// Whether the ray meets the ball's line of sight (the line through the camera
// centre): squared distance of the centre from the line below the radius'.
__device__ inline bool ball_hit(const RayD& R, const float4 b) {
  const float t = b.x * R.fx + b.y * R.fy + b.z * R.fz;
  const float qx = fmaf(-t, R.fx, b.x), qy = fmaf(-t, R.fy, b.y), qz = fmaf(-t, R.fz, b.z);
  return qx * qx + qy * qy + qz * qz < b.w * b.w;
}

constexpr int RB = 256;     // tile-list entries staged in LDS per batch
constexpr int RBLK = 256;   // record slots reserved per wave at a time
constexpr int SBLK = SEG_BLOCK;   // segment slots reserved per wave at a time

__device__ inline unsigned long long bcast64(unsigned long long x) {
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)x);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(x >> 32));
  return ((unsigned long long)hi << 32) | lo;
}

__device__ inline void tile_pixel(int tiles_x, int& px, int& py, int tile = -1) {
  if (tile < 0) tile = blockIdx.x;
  const int tx = tile % tiles_x, ty = tile / tiles_x;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  px = tx * TILE + (w & 1) * 8 + (lane & 7);
  py = ty * TILE + (w >> 1) * 8 + (lane >> 3);
}

// Record buffers of a store-mode pass and the slots a wave holds of them.
struct RecOut {
  int4* ri;
  float4* rf;
  float* rt;
  unsigned long long* counter;
  int4* seg;
  int64_t cap, seg_cap;
};

struct WaveSlots {
  long long rblk = 0, sblk = 0;   // next slots of the current record / segment block
  long long cblk = -1;            // first slot (header) of the current segment block
  int rleft = 0, sleft = 0;
};

// Appends the records of the lanes in m (one cell's contributions over the
// wave's pixels, all lanes active): slots come from the wave's own blocks; a
// new block is reserved with one global atomic when the current one cannot
// take the append.
__device__ inline void append_records(const RecOut& O, WaveSlots& W, uint64_t m, int lane, uint64_t lt, int ci, int pix,
                                      int view_bind, float alpha, float r, float g, float b, float T, int& head) {
  const int cnt = __popcll(m);
  if (cnt > W.rleft) {
    unsigned long long bk = 0;
    if (lane == 0) bk = atomicAdd(&O.counter[0], (unsigned long long)RBLK);
    W.rblk = (long long)bcast64(bk);
    W.rleft = RBLK;
  }
  if (W.sleft == 0) {
    unsigned long long bk = 0;
    if (lane == 0) bk = atomicAdd(&O.counter[1], (unsigned long long)SBLK);
    const long long nb = (long long)bcast64(bk);
    // the block's header links it to the wave's previous block
    if (lane == 0 && nb < O.seg_cap) O.seg[nb] = make_int4(-1, (int)W.cblk, 0, 0);
    W.cblk = nb;
    W.sblk = nb + 1;
    W.sleft = SBLK - 1;
  }
  const long long base = W.rblk, sg = W.sblk;
  W.rblk += cnt;
  W.rleft -= cnt;
  W.sblk += 1;
  W.sleft -= 1;
  if (lane == 0 && sg < O.seg_cap && base + cnt <= O.cap)
    O.seg[sg] = make_int4(ci, (int)base, (int)(uint32_t)m, (int)(uint32_t)(m >> 32));
  if ((m >> lane) & 1ull) {
    const long long slot = base + __popcll(m & lt);
    if (slot < O.cap) {
      O.ri[slot] = make_int4(ci, pix, head, view_bind);
      O.rf[slot] = make_float4(alpha, r, g, b);
      O.rt[slot] = T;
      head = (int)slot;
    }
  }
}

// Ends a wave's segment list: unused slots of its last block are marked
// empty (mask 0); *tail receives the block and the slots used in it.
__device__ inline void close_segments(const RecOut& O, const WaveSlots& W, int lane, int2* tail) {
  for (int j = lane; j < W.sleft; j += 64)
    if (W.sblk + j < O.seg_cap) O.seg[W.sblk + j] = make_int4(0, 0, 0, 0);
  if (lane == 0) *tail = make_int2((int)W.cblk, SBLK - W.sleft);
}

// View of a tile of the group: the last one whose tiles start at or before it.
__device__ inline const ViewDev& tile_view(const ViewDev* __restrict__ views, int nview, int64_t gtile) {
  int lo = 0, hi = nview - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (views[mid].tile_base <= (long long)gtile) lo = mid; else hi = mid - 1;
  }
  return views[lo];
}

__device__ inline float wave_min_f(float x) {
  for (int o = 32; o > 0; o >>= 1) x = fminf(x, __shfl_xor(x, o, 64));
  return x;
}
__device__ inline float wave_add_f(float x) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Cone around the rays of a wave's 8x8 pixels (unit axis a, half-angle with
// cosine ct and sine st; the apex is the camera centre).  A cell's ball can only be met by
// one of those rays if it reaches the cone, which ray_cone_meets tests for
// 64 cells at a time, one per lane; the exact per-pixel test follows for
// the cells that pass, so the test only has to err on the side of passing.
struct RayCone {
  float ax, ay, az, ct, st;
};

__device__ inline RayCone ray_cone(const RayD& R, bool use) {
  RayCone C;
  const float sx = wave_add_f(use ? R.fx : 0.0f), sy = wave_add_f(use ? R.fy : 0.0f),
              sz = wave_add_f(use ? R.fz : 0.0f);
  const float n2 = sx * sx + sy * sy + sz * sz;
  const float inv = n2 > 0.0f ? 1.0f / sqrtf(n2) : 0.0f;
  C.ax = sx * inv;
  C.ay = sy * inv;
  C.az = sz * inv;
  // sine of the largest angle to a ray, from the cross product (accurate for
  // small angles), a little widened
  const float ux = C.ay * R.fz - C.az * R.fy, uy = C.az * R.fx - C.ax * R.fz, uz = C.ax * R.fy - C.ay * R.fx;
  const float s2 = -wave_min_f(use ? -(ux * ux + uy * uy + uz * uz) : 0.0f);
  const float dmin = wave_min_f(use ? C.ax * R.fx + C.ay * R.fy + C.az * R.fz : 1.0f);
  // a cone of more than about 60 degrees (images of a few pixels) is not used
  const bool ok = dmin > 0.5f && inv > 0.0f;
  C.st = ok ? sqrtf(s2) * (1.0f + 1e-4f) + 2e-6f : 2.0f;
  C.ct = ok ? sqrtf(fmaxf(0.0f, 1.0f - C.st * C.st)) : 0.0f;
  return C;
}

// Whether the ball b (ball_from) may reach the cone: the distance of its centre from the cone's surface, |c x a| ct - (c.a) st with c the centre
// relative to the apex, is at most rho (it is negative inside; a centre
// nearer to the apex than to the surface is further away than that).  The
// margin covers the rounding of the products (a few 1e-7 |c|).
__device__ inline bool ray_cone_meets(const RayCone& C, const float4 b) {
  if (C.st > 1.0f) return true;
  const float par = b.x * C.ax + b.y * C.ay + b.z * C.az;
  const float ux = b.y * C.az - b.z * C.ay, uy = b.z * C.ax - b.x * C.az, uz = b.x * C.ay - b.y * C.ax;
  const float perp = fsqrt(ux * ux + uy * uy + uz * uz);
  const float far = fabsf(b.x) + fabsf(b.y) + fabsf(b.z);
  return !(perp * C.ct - par * C.st > b.w * (1.0f + 1e-5f) + 2e-6f * far + 1e-7f);
}

// Pixels of a wave as points u = (d.b1, d.b2) / (d.a) of the plane at unit
// distance along the axis a of its cone, b1 and b2 completing a to a frame.
// A ball whose centre projects to w at depth z = c.a meets the ray of u only
// if |c x d| <= rho, and |c x d|^2 >= z^2 |w - u|^2 / (1 + |u|^2), so the
// nearest of the 64 points decides whether any ray of the wave can meet it:
// balls that fall between the pixel centres are dropped, 64 cells at a time.
struct RayGrid {
  float b1x, b1y, b1z, b2x, b2y, b2z, k;   // k = 1 + largest |u|^2
};

__device__ inline RayGrid ray_grid(const RayD& R, const RayCone& C, bool use, float2& u) {
  RayGrid G;
  onb(C.ax, C.ay, C.az, G.b1x, G.b1y, G.b1z, G.b2x, G.b2y, G.b2z);
  const float par = R.fx * C.ax + R.fy * C.ay + R.fz * C.az;
  const float inv = use && par > 0.0f ? 1.0f / par : 0.0f;
  // (a pixel without a ray is put out of reach)
  u.x = use ? (R.fx * G.b1x + R.fy * G.b1y + R.fz * G.b1z) * inv : 1e18f;
  u.y = use ? (R.fx * G.b2x + R.fy * G.b2y + R.fz * G.b2z) * inv : 1e18f;
  const float m = -wave_min_f(use ? -(u.x * u.x + u.y * u.y) : 0.0f);
  G.k = (1.0f + m) * (1.0f + 1e-5f);
  return G;
}

// Whether the ball may meet one of the rays u[0..63] (pairs of points).
__device__ inline bool ray_grid_meets(const RayCone& C, const RayGrid& G, const float4* u2, const float4 b) {
  if (C.st > 1.0f) return true;
  const float cx = b.x, cy = b.y, cz = b.z;
  const float r = b.w * (1.0f + 1e-5f) + 2e-6f * (fabsf(cx) + fabsf(cy) + fabsf(cz)) + 1e-7f;
  const float depth = cx * C.ax + cy * C.ay + cz * C.az;
  if (!(depth > 2.0f * r)) return true;   // around or behind the camera
  const float inv = 1.0f / depth;
  const float wx = (cx * G.b1x + cy * G.b1y + cz * G.b1z) * inv, wy = (cx * G.b2x + cy * G.b2y + cz * G.b2z) * inv;
  float best = INFINITY;
#pragma unroll 4
  for (int j = 0; j < 32; ++j) {
    const float4 p = u2[j];
    const float ex = wx - p.x, ey = wy - p.y, gx = wx - p.z, gy = wy - p.w;
    best = fminf(best, fminf(ex * ex + ey * ey, gx * gx + gy * gy));
  }
  return !(best * depth * depth > r * r * G.k);
}

// COUNT: the work counters of the composite are added to counters[0..5]
// (RASTER_COUNTERS): pixel-cell tests, sphere hits, contributions, and the
// (wave, cell) steps that tested, that computed a piece, that shaded.
struct RasterCounts {
  unsigned long long test = 0, hit = 0, contrib = 0, step = 0, step_hit = 0, step_shade = 0;
  __device__ void add(unsigned long long* __restrict__ c) const {
    if ((threadIdx.x & 63) == 0) {
      atomicAdd(&c[0], test);
      atomicAdd(&c[1], hit);
      atomicAdd(&c[2], contrib);
      atomicAdd(&c[3], step);
      atomicAdd(&c[4], step_hit);
      atomicAdd(&c[5], step_shade);
    }
  }
};

// Which tiles of a launch go to k_raster_split: those whose list is longer
// than plan[PLAN_LEN], listed (longest first, by classes of 1/8 of a power of
// two) in plan[PLAN_LIST ...], plan[PLAN_COUNT] of them; plan[PLAN_NEXT] is the
// queue of k_raster_split, zeroed here.
//
// The cost of a launch that leaves lists up to length t to k_raster is taken as
//   max(CHAIN t, D + CHAIN_SHARE CHAIN t) + S,
// D the cost in k_raster of the lists up to t (DENSE_TILE + DENSE_ENTRY len each)
// and S that in k_raster_split of the others (SPLIT_TILE + SPLIT_ENTRY len, less per
// entry beyond SPLIT_KNEE): k_raster's longest list is walked by one wave per
// quadrant, half of it while the others run, and it is cheap per tile;
// k_raster_split works off one quadrant per CU at a time, which costs it more
// per tile and per entry, but a list is sixteen times shorter.  The t of the
// least cost is taken.  The constants (microseconds) are fitted to 43 launches of
// 1k to 1M cells, 100x100 to 1920x1080, one to eight views, each through either
// kernel alone: of 128x128 at 1,024 cells 0.165 or 0.054 ms, of 256x256 at
// 1,048,576 6.6 or 0.71, of four mixed views up to 1920x1080 there 38 or 9.0, of
// 1280x720 at 262,144 1.69 or 1.52 (1.26 as planned); of 2 views of 1027x1048 at
// 2,561 0.34 or 0.49, of 3 of 1920x1080 at 60,000 2.6 or 5.6, of 8 of 1600x1066
// at 1,048,576 24 or 41.
constexpr int PLAN_LEN = 0, PLAN_COUNT = 1, PLAN_NEXT = 2, PLAN_LIST = 4;
constexpr int PLAN_THREADS = 1024, PLAN_CLASSES = 256;
constexpr float CHAIN = 2.5f, CHAIN_SHARE = 0.5f, DENSE_TILE = 0.02f, DENSE_ENTRY = 2.75e-3f;
constexpr float SPLIT_TILE = 0.118f, SPLIT_ENTRY = 4.5e-3f, SPLIT_KNEE = 100.0f, SPLIT_LONG = 2.7e-3f;

// Length class: lengths below 16 by themselves, then eight classes per power
// of two; class_max is the largest length of a class.
__device__ inline int len_class(uint32_t len) {
  if (len < 16) return (int)len;
  const int e = 31 - __clz(len);
  return 16 + 8 * (e - 4) + (int)((len >> (e - 3)) & 7u);
}
__device__ inline uint32_t class_max(int c) {
  if (c < 16) return (uint32_t)c;
  const int e = (c - 16) / 8 + 4, f = (c - 16) % 8;
  return (uint32_t)((((unsigned long long)(9 + f)) << (e - 3)) - 1);
}

__global__ void __launch_bounds__(PLAN_THREADS) k_split_plan(const uint32_t* __restrict__ tile_off, int64_t tile_first,
                                                             int64_t count, uint32_t* __restrict__ plan) {
  constexpr int REP = 8;   // copies of the histogram (fewer lanes meet on one word)
  __shared__ uint32_t s_n[REP][PLAN_CLASSES], s_sum[REP][PLAN_CLASSES];
  __shared__ uint32_t s_pos[PLAN_CLASSES];
  __shared__ uint32_t s_part[4];
  __shared__ float s_partc[4][2];
  __shared__ float s_cost[4];
  __shared__ int s_cls[4], s_best;
  __shared__ uint32_t s_count;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, rep = t & (REP - 1);
  for (int k = t; k < REP * PLAN_CLASSES; k += PLAN_THREADS) {
    (&s_n[0][0])[k] = 0;
    (&s_sum[0][0])[k] = 0;
  }
  __syncthreads();
  // (eight loads in flight per thread)
  auto each = [&](auto&& fn) {
    for (int64_t i0 = 0; i0 < count; i0 += 8 * PLAN_THREADS) {
      uint32_t len[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int64_t i = i0 + k * PLAN_THREADS + t;
        len[k] = i < count ? tile_off[tile_first + i + 1] - tile_off[tile_first + i] : 0u;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (len[k]) fn((uint32_t)(i0 + k * PLAN_THREADS + t), len[k]);
    }
  };
  each([&](uint32_t, uint32_t len) {
    const int c = len_class(len);
    atomicAdd(&s_n[rep][c], 1u);
    atomicAdd(&s_sum[rep][c], len);
  });
  __syncthreads();
  // a thread per class: prefix sums of the lists and their entries, and the
  // least cost with its class
  uint32_t n = 0, n_in = 0;
  float dense = 0.0f, split = 0.0f;   // of the lists up to the class, either way
  if (t < PLAN_CLASSES) {
    uint32_t sum = 0;
    for (int r = 0; r < REP; ++r) {
      n += s_n[r][t];
      sum += s_sum[r][t];
    }
    const float fn = (float)n, fl = (float)sum, head = fminf(fl, fn * SPLIT_KNEE);
    n_in = n;
    dense = DENSE_TILE * fn + DENSE_ENTRY * fl;
    split = SPLIT_TILE * fn + SPLIT_ENTRY * head + SPLIT_LONG * (fl - head);
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t a = __shfl_up(n_in, d, 64);
      const float b = __shfl_up(dense, d, 64), c = __shfl_up(split, d, 64);
      if (lane >= d) {
        n_in += a;
        dense += b;
        split += c;
      }
    }
    if (lane == 63) {
      s_part[wave] = n_in;
      s_partc[wave][0] = dense;
      s_partc[wave][1] = split;
    }
  }
  __syncthreads();
  const uint32_t n_all = s_part[0] + s_part[1] + s_part[2] + s_part[3];
  const float split_all = ((s_partc[0][1] + s_partc[1][1]) + s_partc[2][1]) + s_partc[3][1];
  if (t < PLAN_CLASSES) {
    for (int w = 0; w < wave; ++w) {
      n_in += s_part[w];
      dense += s_partc[w][0];
      split += s_partc[w][1];
    }
    // (class 0, no lists of any length: everything is split)
    const float chain = CHAIN * (float)class_max(t);
    float cost = n || t == 0 ? fmaxf(chain, dense + CHAIN_SHARE * chain) + (split_all - split) : INFINITY;
    int cls = t;
    for (int o = 32; o > 0; o >>= 1) {
      const float c2 = __shfl_xor(cost, o, 64);
      const int k2 = __shfl_xor(cls, o, 64);
      if (c2 < cost || (c2 == cost && k2 > cls)) {
        cost = c2;
        cls = k2;
      }
    }
    if (lane == 0) {
      s_cost[wave] = cost;
      s_cls[wave] = cls;
    }
    s_pos[t] = n_all - n_in;   // lists of the longer classes come first
  }
  __syncthreads();
  if (t == 0) {
    int w = 0;
    for (int k = 1; k < 4; ++k)
      if (s_cost[k] <= s_cost[w]) w = k;
    s_best = s_cls[w];
    s_count = 0;
    plan[PLAN_LEN] = class_max(s_cls[w]);
    plan[PLAN_NEXT] = 0;
  }
  __syncthreads();
  if (t == s_best) {
    s_count = n_all - n_in;
    plan[PLAN_COUNT] = n_all - n_in;
  }
  __syncthreads();
  const int bc = s_best;
  if (s_count == 0) return;
  each([&](uint32_t i, uint32_t len) {
    const int c = len_class(len);
    if (c > bc) plan[PLAN_LIST + atomicAdd(&s_pos[c], 1u)] = i;
  });
}

// Seven waves per SIMD (at most 72 VGPRs) are asked for explicitly: the
// compiler's own choice lands a few registers above, at six.  Tiles whose
// list is longer than plan[PLAN_LEN] are left to k_raster_split.
template <bool STORE, bool COUNT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(7)))
k_raster(const ViewDev* __restrict__ views, int nview, SceneDev S, const unsigned long long* __restrict__ list,
         const uint32_t* __restrict__ tile_off, float t_min, float* __restrict__ rgba_all, int4* __restrict__ rec_ri,
         float4* __restrict__ rec_rf, float* __restrict__ rec_rt, int32_t* __restrict__ rec_head,
         unsigned long long* __restrict__ rec_counter, int4* __restrict__ rec_seg, int2* __restrict__ rec_wtail,
         int64_t wtail_base, int64_t rec_cap, int64_t seg_cap,
         int64_t tile_first, const uint32_t* __restrict__ plan,
         unsigned long long* __restrict__ counters) {
  // the tile's sorted cells are staged RB at a time: list entry and the cell
  // record fields every lane needs, loaded by the whole workgroup at once
  __shared__ int s_ci[RB];
  __shared__ float4 s_geo[RB];
  __shared__ float4 s_nrm[RB];
  __shared__ float4 s_ball[RB];   // ball_from
  __shared__ int s_row[RB];
  __shared__ int s_nr[RB];
  __shared__ int s_more[4];
  __shared__ RayCone s_cone[4];   // per wave
  const RecOut O{rec_ri, rec_rf, rec_rt, rec_counter, rec_seg, rec_cap, seg_cap};

  // one workgroup per work item (a tile of one of the launch's views); the
  // hardware dispatcher hands the next item to whichever CU frees up, so the
  // tiles of all views of a call (the requests of a serving batch) share
  // the CUs.  (A persistent loop over items held twice the registers and
  // halved the occupancy.)
  const int64_t item = blockIdx.x;
  const int64_t gtile = tile_first + item;
  const uint32_t e0 = tile_off[gtile], e1 = tile_off[gtile + 1];
  if (e1 - e0 > plan[PLAN_LEN]) return;
  const ViewDev& vd = tile_view(views, nview, gtile);
  const ViewArgs& v = vd.v;
  float* rgba = rgba_all + 4 * vd.pix_base;
  int px, py;
  tile_pixel(v.tiles_x, px, py, (int)(gtile - vd.tile_base));
  const bool inside = px < v.cam.width && py < v.cam.height;
  const RayD R = make_ray(v.cam, px + 0.5, py + 0.5);
  bool live = inside && R.valid;
  float T = 1.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f;
  int head = -1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const int pix = py * v.cam.width + px;
  WaveSlots W;
  RasterCounts N;
  {
    const RayCone cone = ray_cone(R, live);
    if (lane == 0) s_cone[wave] = cone;
  }
  for (uint32_t b0 = e0; b0 < e1; b0 += RB) {
    {
      const uint32_t e = b0 + threadIdx.x;
      if (e < e1) {
        const int c = (int)(uint32_t)list[e];
        s_ci[threadIdx.x] = c;
        s_geo[threadIdx.x] = S.geo[c];
        s_nrm[threadIdx.x] = S.nrm[c];
        s_ball[threadIdx.x] = ball_from(S.ball[c], R.ox, R.oy, R.oz);
        s_row[threadIdx.x] = S.row[c];
        s_nr[threadIdx.x] = S.nrast[c];
      }
    }
    __syncthreads();
    // the cells whose ball can meet a ray of the wave's quadrant, found 64 at
    // a time, one per lane; only those are tested pixel by pixel
    const int nb = (int)min((uint32_t)RB, e1 - b0);
#pragma unroll 1
    for (int k0 = 0; k0 < nb; k0 += 64) {
      uint64_t todo;
      {
        const RayCone cone = s_cone[wave];
        const int q = k0 + lane;
        todo = __ballot(q < nb && ray_cone_meets(cone, s_ball[q]));
      }
      for (; todo; todo &= todo - 1) {
        if (!__any(live)) break;
        const int q = k0 + __ffsll((long long)todo) - 1;
        const int ci = __builtin_amdgcn_readfirstlane(s_ci[q]);
        const bool hit = live && ball_hit(R, s_ball[q]);
        if constexpr (COUNT) {
          N.test += (unsigned long long)__popcll(__ballot(live));
          N.hit += (unsigned long long)__popcll(__ballot(hit));
          ++N.step;
        }
        if (!__any(hit)) continue;
        if constexpr (COUNT) ++N.step_hit;
        const float4 g = s_geo[q];
        const ufloat_p tx = uniform_ptr(S.tex + (int64_t)ci * (KD * TEXW));
        Piece P;
        P.alpha = 0.0f;
        float r = 0.0f, gg = 0.0f, b = 0.0f;
        if (hit) {
          const Local L = make_local(R, g.x, g.y, g.z);
          P = piece_geometry(R, L, g.w, uniform_ptr(S.plane + __builtin_amdgcn_readfirstlane(s_row[q])),
                             __builtin_amdgcn_readfirstlane(s_nr[q]), s_nrm[q], tx, S.tau);
        }
        const bool contrib = hit && P.alpha > 0.0f;
        if (__any(contrib))
          radiance_wave(S.tex + (int64_t)ci * (KD * TEXW), tx, uniform_ptr(S.rgb + 3 * (int64_t)ci), contrib, P.ux, P.uy,
                        R.fx, R.fy, R.fz, S.tau, r, gg, b);
        if constexpr (COUNT) {
          const uint64_t mc = __ballot(contrib);
          N.contrib += (unsigned long long)__popcll(mc);
          N.step_shade += mc ? 1ull : 0ull;
        }
        if constexpr (STORE) {
          const uint64_t m = __ballot(contrib);
          if (m)
            append_records(O, W, m, lane, lt, ci, pix, pack_view_bind(vd.view_id, P.bind0, P.bind1), P.alpha, r, gg, b,
                           T, head);
        }
        if (contrib) {
          const float wgt = T * P.alpha;
          cr += wgt * r;
          cg += wgt * gg;
          cb += wgt * b;
          T *= (1.0f - P.alpha);
        }
        live = live && (T >= t_min);
      }
    }
    const bool wl = __any(live);
    if (lane == 0) s_more[wave] = wl ? 1 : 0;
    __syncthreads();
    const bool more = (s_more[0] | s_more[1] | s_more[2] | s_more[3]) != 0;
    __syncthreads();
    if (!more) break;
  }
  if (inside) {
    float* o = rgba + 4 * ((int64_t)py * v.cam.width + px);
    o[0] = cr;
    o[1] = cg;
    o[2] = cb;
    o[3] = 1.0f - T;
    if constexpr (STORE) rec_head[vd.pix_base + pix] = head;
  }
  if constexpr (STORE) close_segments(O, W, lane, rec_wtail + (wtail_base + item) * 4 + wave);
  if constexpr (COUNT) N.add(counters);
}

// Waits until *p >= v (32-bit counters in LDS written by another wave of the
// workgroup); returns false if *stop became 0 first.
__device__ inline bool lds_wait(const int* p, int v, const unsigned long long* stop) {
  while (__hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < v) {
    if (stop && __hip_atomic_load(stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == 0ull) return false;
    __builtin_amdgcn_s_sleep(1);
  }
  return true;
}

// The same composite for the tiles with long lists: a workgroup of NW waves
// per 8x8 quadrant of a tile.  Opacity and colour of a (pixel, cell) pair do
// not depend on the cells in front of it, so NW - 1 waves evaluate the cells
// of the list, each taking the next one over the quadrant's 64 pixels, and
// one wave composites their results in list order: the arithmetic of a
// pixel is that of k_raster, operation for operation.  The list is first
// reduced, a step of 64 NW entries at a time and one cell per lane, to the
// cells whose ball can meet one of the quadrant's rays; those are queued.
//
// A tile's list is a serial chain for its four waves in k_raster: with few
// tiles, or a few long ones among many, the chip idles behind those chains.
//
// Results pass through a ring of RING slots in LDS: a slot holds cell j of
// the queue once s_flag of the slot reads base + j + 1, and is free for cell
// j + RING once s_done > base + j (base: cells of the earlier steps).  The
// evaluating waves take cells in order and the compositing wave waits for
// them in order, so the first cell not yet composited is always being
// evaluated in a slot of its own, and both sides finish; when no pixel is
// left (s_live = 0) the evaluating waves stop waiting for slots.  The
// workgroups take the quadrants of the plan's tiles from a queue, longest
// lists first.
constexpr int NW = 16;
template <bool STORE, bool COUNT>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4)))
k_raster_split(const ViewDev* __restrict__ views, int nview, SceneDev S, const unsigned long long* __restrict__ list,
               const uint32_t* __restrict__ tile_off, float t_min, float* __restrict__ rgba_all,
               int4* __restrict__ rec_ri, float4* __restrict__ rec_rf, float* __restrict__ rec_rt,
               int32_t* __restrict__ rec_head, unsigned long long* __restrict__ rec_counter,
               int4* __restrict__ rec_seg, int2* __restrict__ rec_wtail, int64_t wtail_base, int64_t rec_cap,
               int64_t seg_cap, int64_t tile_first, uint32_t* plan, unsigned long long* __restrict__ counters) {
  constexpr int CH = 64 * NW;      // list entries culled at a time
  constexpr int RING = 2 * NW;
  __shared__ int q_ci[CH];
  __shared__ float4 q_geo[CH];
  __shared__ float4 q_nrm[CH];
  __shared__ float4 q_ball[CH];   // ball_from
  __shared__ int q_row[CH];
  __shared__ int q_nr[CH];
  __shared__ float4 s_res[RING][64];               // (alpha, colour) per pixel
  __shared__ int s_bind[STORE ? RING : 1][64];
  __shared__ unsigned long long s_mask[RING];      // the pixels the cell contributes to
  __shared__ int s_cell[RING];
  __shared__ int s_flag[RING];
  __shared__ int s_done;                           // cells composited
  __shared__ int s_next;                           // next cell of the queue to evaluate
  __shared__ unsigned long long s_live;            // pixels not yet opaque
  __shared__ int s_cnt[NW];
  __shared__ float4 s_u2[32];                      // the pixels as points (RayGrid)
  __shared__ RayCone s_cone;
  __shared__ RayGrid s_grid;
  __shared__ uint32_t s_item;
  static_assert(RING <= 64, "flags cleared by one wave");

  const uint32_t n_items = 4 * plan[PLAN_COUNT];
  RasterCounts N;
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(&plan[PLAN_NEXT], 1u);
    __syncthreads();
    const uint32_t qi = __builtin_amdgcn_readfirstlane(s_item);
    if (qi >= n_items) break;
    const int64_t item = plan[PLAN_LIST + qi / 4];
    const int quad = qi & 3;
    const int64_t gtile = tile_first + item;
    const ViewDev& vd = tile_view(views, nview, gtile);
    const ViewArgs& v = vd.v;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ltile = (int)(gtile - vd.tile_base);
    const int px = (ltile % v.tiles_x) * TILE + (quad & 1) * 8 + (lane & 7);
    const int py = (ltile / v.tiles_x) * TILE + (quad >> 1) * 8 + (lane >> 3);
    const bool inside = px < v.cam.width && py < v.cam.height;
    const RayD R = make_ray(v.cam, px + 0.5, py + 0.5);
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const uint32_t e0 = tile_off[gtile], e1 = tile_off[gtile + 1];
    if (wave == 0) {
      const bool use = inside && R.valid;
      const RayCone cone = ray_cone(R, use);
      float2 u;
      const RayGrid grid = ray_grid(R, cone, use, u);
      ((float2*)s_u2)[lane] = u;
      const uint64_t l = __ballot(use);
      if (lane == 0) {
        s_cone = cone;
        s_grid = grid;
        s_live = l;
        s_done = 0;
        s_next = 0;
      }
      if (lane < RING) s_flag[lane] = 0;
    }
    __syncthreads();

    // Queues the cells of the list entries [b0, b0 + CH) that can meet a ray
    // of the quadrant; returns their number (all waves take part).
    auto cull = [&](uint32_t b0) -> int {
      const uint32_t e = b0 + threadIdx.x;
      int c = -1;
      float4 bl = make_float4(0.0f, 0.0f, 0.0f, -1.0f);
      if (e < e1) {
        c = (int)(uint32_t)list[e];
        bl = ball_from(S.ball[c], R.ox, R.oy, R.oz);
      }
      const RayCone cone = s_cone;
      bool keep = c >= 0 && ray_cone_meets(cone, bl);
      if (keep) keep = ray_grid_meets(cone, s_grid, s_u2, bl);
      const uint64_t km = __ballot(keep);
      if (lane == 0) s_cnt[wave] = __popcll(km);
      float4 g = make_float4(0.0f, 0.0f, 0.0f, 0.0f), nr4 = g;
      int row = 0, nrast = 0;
      if (keep) {
        g = S.geo[c];
        nr4 = S.nrm[c];
        row = S.row[c];
        nrast = S.nrast[c];
      }
      __syncthreads();
      int at = __popcll(km & lt), total = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const int n = s_cnt[w];
        at += w < wave ? n : 0;
        total += n;
      }
      if (keep) {
        q_ci[at] = c;
        q_geo[at] = g;
        q_nrm[at] = nr4;
        q_ball[at] = bl;
        q_row[at] = row;
        q_nr[at] = nrast;
      }
      __syncthreads();
      return __builtin_amdgcn_readfirstlane(total);
    };

    int base = 0;   // cells queued by the earlier steps
    if (wave == 0) {
      // --- the compositing wave
      const RecOut O{rec_ri, rec_rf, rec_rt, rec_counter, rec_seg, rec_cap, seg_cap};
      bool live = inside && R.valid;
      float T = 1.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f;
      int head = -1;
      const int pix = py * v.cam.width + px;
      WaveSlots W;
      uint64_t lm = __ballot(live);
      for (uint32_t b0 = e0; b0 < e1; b0 += CH) {
        const int nq = cull(b0);
        for (int j = 0; j < nq && lm; ++j) {
          const int slot = (base + j) % RING;
          lds_wait(&s_flag[slot], base + j + 1, nullptr);
          const uint64_t m = bcast64(s_mask[slot]) & lm;
          if (m) {
            const bool contrib = (m >> lane) & 1ull;
            const float4 c = s_res[slot][lane];
            if constexpr (COUNT) {
              N.contrib += (unsigned long long)__popcll(m);
              ++N.step_shade;
            }
            if constexpr (STORE)
              append_records(O, W, m, lane, lt, __builtin_amdgcn_readfirstlane(s_cell[slot]), pix, s_bind[slot][lane],
                             c.x, c.y, c.z, c.w, T, head);
            if (contrib) {
              const float wgt = T * c.x;
              cr += wgt * c.y;
              cg += wgt * c.z;
              cb += wgt * c.w;
              T *= (1.0f - c.x);
            }
            live = live && (T >= t_min);
            lm = __ballot(live);
          }
          if (lane == 0) {
            __hip_atomic_store(&s_live, (unsigned long long)lm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_store(&s_done, base + j + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
          __builtin_amdgcn_wave_barrier();
        }
        base += nq;
        __syncthreads();
        if (lane == 0) s_next = 0;
        __builtin_amdgcn_wave_barrier();
        if (!lm) break;
      }
      if (inside) {
        float* o = rgba_all + 4 * (vd.pix_base + (int64_t)py * v.cam.width + px);
        o[0] = cr;
        o[1] = cg;
        o[2] = cb;
        o[3] = 1.0f - T;
        if constexpr (STORE) rec_head[vd.pix_base + pix] = head;
      }
      if constexpr (STORE) close_segments(O, W, lane, rec_wtail + (wtail_base + item) * 4 + quad);
    } else {
      // --- the evaluating waves
      for (uint32_t b0 = e0; b0 < e1; b0 += CH) {
        const int nq = cull(b0);
        for (;;) {
          int j = 0;
          if (lane == 0) j = atomicAdd(&s_next, 1);
          __builtin_amdgcn_wave_barrier();
          j = __builtin_amdgcn_readfirstlane(j);
          if (j >= nq) break;
          const int ci = __builtin_amdgcn_readfirstlane(q_ci[j]);
          const float4 g = q_geo[j];
          // (pixels only leave the set, so an older value costs work, not results)
          const uint64_t lm = bcast64(
              __hip_atomic_load(&s_live, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
          if (!lm) break;
          const bool hit = ((lm >> lane) & 1ull) && ball_hit(R, q_ball[j]);
          if constexpr (COUNT) {
            const uint64_t hm = __ballot(hit);
            N.test += (unsigned long long)__popcll(lm);
            N.hit += (unsigned long long)__popcll(hm);
            ++N.step;
            N.step_hit += hm ? 1ull : 0ull;
          }
          Piece P;
          P.alpha = 0.0f;
          float r = 0.0f, gg = 0.0f, b = 0.0f;
          const ufloat_p tx = uniform_ptr(S.tex + (int64_t)ci * (KD * TEXW));
          if (hit) {
            const Local L = make_local(R, g.x, g.y, g.z);
            P = piece_geometry(R, L, g.w, uniform_ptr(S.plane + __builtin_amdgcn_readfirstlane(q_row[j])),
                                     __builtin_amdgcn_readfirstlane(q_nr[j]), q_nrm[j], tx, S.tau);
          }
          const bool contrib = hit && P.alpha > 0.0f;
          const uint64_t m = __ballot(contrib);
          if (m)
            radiance_wave(S.tex + (int64_t)ci * (KD * TEXW), tx, uniform_ptr(S.rgb + 3 * (int64_t)ci), contrib, P.ux,
                          P.uy, R.fx, R.fy, R.fz, S.tau, r, gg, b);
          const int slot = (base + j) % RING;
          if (!lds_wait(&s_done, base + j - RING + 1, &s_live)) break;
          if (contrib) {
            s_res[slot][lane] = make_float4(P.alpha, r, gg, b);
            if constexpr (STORE) s_bind[slot][lane] = pack_view_bind(vd.view_id, P.bind0, P.bind1);
          }
          if (lane == 0) {
            s_mask[slot] = m;
            s_cell[slot] = ci;
          }
          // (the wave's LDS writes complete in order before the flag is set)
          if (lane == 0)
            __hip_atomic_store(&s_flag[slot], base + j + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
          // the wave stays together across the loop's end: without this the
          // lanes other than 0 are sent past the next iteration's lane-0
          // branch before lane 0 has taken its next cell
          __builtin_amdgcn_wave_barrier();
        }
        base += nq;
        __syncthreads();
        if (!__hip_atomic_load(&s_live, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) break;
      }
    }
    __syncthreads();   // (the shared state is set up anew for the next quadrant)
  }
  if constexpr (COUNT) N.add(counters);
}

// Total records listed by the segments (the block reservation leaves unused
// record slots, so the reserved count is an upper bound).
__global__ void __launch_bounds__(256) k_seg_total(const int4* __restrict__ seg, int64_t nseg,
                                                   unsigned long long* __restrict__ total) {
  __shared__ unsigned long long part[4];
  unsigned long long acc = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nseg; i += (int64_t)gridDim.x * blockDim.x)
    acc += (unsigned long long)seg_count(seg[i]);
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(total, part[0] + part[1] + part[2] + part[3]);
}

// argmin over cells with a non-empty power cell of pow(o, p_i) in float64;
// ties go to the lower index.  Stage 1: per block; stage 2: one block.
// On the way, the balls that the texture has outgrown since the build are
// replaced in place (live_ball): a ball that covers the whole bounded cell stays
// right whatever the texture becomes, and passes of several streams that find
// one outgrown all write the same value.
__global__ void __launch_bounds__(256) k_start_partial(const float* __restrict__ p, const float* __restrict__ w,
                                                       const int32_t* __restrict__ flags, int64_t n, double ox,
                                                       double oy, double oz, BallArgs b, double* __restrict__ pk,
                                                       long long* __restrict__ pi) {
  double best = INFINITY;
  long long bi = -1;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    if (flags[i] & FLAG_EMPTY_POWER) continue;
    const double ex = ox - p[3 * i], ey = oy - p[3 * i + 1], ez = oz - p[3 * i + 2];
    const double k = ex * ex + ey * ey + ez * ez - (double)w[i];
    if (k < best || (k == best && (bi < 0 || i < bi))) {
      best = k;
      bi = i;
    }
    bool grown;
    const float4 bl = live_ball(b.geo, b.cull, b.ball, b.ball_top, b.tex, i, grown);
    if (grown) b.ball[i] = bl;
  }
  __shared__ double sk[256];
  __shared__ long long si[256];
  sk[threadIdx.x] = best;
  si[threadIdx.x] = bi;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      const double k2 = sk[threadIdx.x + s];
      const long long i2 = si[threadIdx.x + s];
      if (i2 >= 0 && (si[threadIdx.x] < 0 || k2 < sk[threadIdx.x] || (k2 == sk[threadIdx.x] && i2 < si[threadIdx.x]))) {
        sk[threadIdx.x] = k2;
        si[threadIdx.x] = i2;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    pk[blockIdx.x] = sk[0];
    pi[blockIdx.x] = si[0];
  }
}

__global__ void __launch_bounds__(256) k_start_final(const double* __restrict__ pk, const long long* __restrict__ pi,
                                                     int nb, int32_t* __restrict__ out) {
  __shared__ double sk[256];
  __shared__ long long si[256];
  double best = INFINITY;
  long long bi = -1;
  for (int b = threadIdx.x; b < nb; b += 256) {
    if (pi[b] >= 0 && (bi < 0 || pk[b] < best || (pk[b] == best && pi[b] < bi))) {
      best = pk[b];
      bi = pi[b];
    }
  }
  sk[threadIdx.x] = best;
  si[threadIdx.x] = bi;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      const double k2 = sk[threadIdx.x + s];
      const long long i2 = si[threadIdx.x + s];
      if (i2 >= 0 && (si[threadIdx.x] < 0 || k2 < sk[threadIdx.x] || (k2 == sk[threadIdx.x] && i2 < si[threadIdx.x]))) {
        sk[threadIdx.x] = k2;
        si[threadIdx.x] = i2;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = (int32_t)si[0];
}

// Face loads a ray of the walk has in flight (with four and with two, before
// the radiance was deferred: 5.74 and 5.80 ms for 921600 rays of 67 cells in a
// 1M-cell scene, 0.85 and 0.93 ms for a fisheye view of 16k cells).
constexpr int WALK_FACES = 4;
// Contributions a ray of the walk may have pending (of 6, 8, 10, 12 the ring of
// ten was best or within 2% for both views: 4.5, 3.98, 3.96, 4.15 ms and 0.81,
// 0.69, 0.68, 0.60 ms; sixteen, which leaves one wave per SIMD less, 5.2 and
// 0.62 ms), and the ratio of what they cost: a ray-by-ray evaluation of all
// pending rays takes about as long as twelve evaluations of one cell (ratio 4,
// 8, 16, 32: 3.96, 3.84, 3.79, 3.74 ms and 0.68, 0.69, 0.70, 0.77 ms).
constexpr int WALK_QUEUE = 10;
constexpr int WALK_GROUP = 12;

// One lane per ray.  STORE: every contribution is also written as a record (as
// the store-mode rasteriser does) with a one-record segment; rec_seg must be
// zeroed by the caller (unused slots of the wave's segment blocks keep an empty
// mask).
// A step reads every face of the cell once, for the piece and for the exit
// together.  Opacity decides how far a ray goes, colour does not: a contribution's
// texture point and weight wait in the ray's LDS ring until it is full.  Then
// either all rays of the wave that hold that cell, now or some contributions
// ago, are shaded at once on the matrix cores from one coalesced read of its
// texture, or, where few do, every ray's oldest contribution with per-lane reads.
// What bounds it are the instructions it issues (84% of the SIMDs' cycles over 8
// views of 1600x1066), a part of its lanes idle, and the waits for a step's dependent
// loads (44% of its waves' cycles); the ring's LDS (40,960 bytes) and the registers
// leave four waves per SIMD, two in the record-writing form (51,200 bytes, whose
// three workgroups per CU the register allocation does not use).
// 921600 rays through 1M cells (67 cells, 18 faces each, 22 contributions per
// ray): 8.9 ms with two face passes and the radiance in place, 5.7 ms with one,
// 3.7 ms with the radiance deferred (1.9 ms of it the faces, 0.6 the opacity);
// a 300 x 300 fisheye of 16k cells 1.48, 0.85 and 0.67 ms.
// COUNT: the walk's work counters are added to counters[0..5]
// (TRACE_COUNTERS): rays walked, cells walked, pieces computed (sphere
// hits), contributions, exit faces scanned, and the most cells one ray
// walked (maximum).
template <bool STORE, bool COUNT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_trace(ViewArgs v, int64_t tile_first, SceneDev S, const int32_t* __restrict__ start,
                                               float t_min, int max_steps, float* __restrict__ rgba,
                                               unsigned long long* __restrict__ truncated, int view,
                                               int4* __restrict__ rec_ri, float4* __restrict__ rec_rf,
                                               float* __restrict__ rec_rt, int32_t* __restrict__ rec_head,
                                               unsigned long long* __restrict__ rec_counter,
                                               int4* __restrict__ rec_seg, int64_t rec_cap, int64_t seg_cap,
                                               unsigned long long* __restrict__ counters) {
  int px, py;
  tile_pixel(v.tiles_x, px, py, (int)(tile_first + blockIdx.x));
  const bool inside = px < v.cam.width && py < v.cam.height;
  const RayD R = make_ray(v.cam, px + 0.5, py + 0.5);
  bool live = inside && R.valid;
  float T = 1.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f;
  int cell = start[0];
  int prev = -1;
  double t_cur = 0.0;
  bool cut = false;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const int pix = py * v.cam.width + px;
  int head = -1;
  // the wave's current record / segment blocks; the lanes still walking
  // update them together
  long long rblk = 0, sblk = 0;
  int rleft = 0, sleft = 0;
  unsigned long long n_pieces = 0, n_contrib = 0, n_faces = 0;
  int n_steps = 0;
  const bool walked = live && cell >= 0;
  // contributions whose radiance is still to be evaluated, a ring per ray with
  // holes: bit d of `held` marks slot d, `slot` is the next one
  __shared__ float4 s_pend[4][WALK_QUEUE][64];             // cell, texture point, weight
  __shared__ int s_rec[4][STORE ? WALK_QUEUE : 1][64];     // STORE: its record, or -1
  unsigned held = 0;
  int slot = 0;
  // adds the colour of slot d's contribution
  auto add = [&](int d, float wgt, float r, float gg, float b) {
    cr = fmaf(wgt, r, cr);
    cg = fmaf(wgt, gg, cg);
    cb = fmaf(wgt, b, cb);
    held &= ~(1u << d);
    if constexpr (STORE) {
      const int rec = s_rec[wave][d][lane];
      if (rec >= 0) {
        float* o = reinterpret_cast<float*>(rec_rf + rec);
        o[1] = r;
        o[2] = gg;
        o[3] = b;
      }
    }
  };
  // evaluates pending contributions, among them the oldest of the first ray
  // in `due` (a wave-uniform mask of rays that hold one)
  auto shade = [&](uint64_t due) {
    // the ray's oldest pending contribution
    const unsigned rot = (held >> slot) | (held << (WALK_QUEUE - slot));
    int d = slot + (rot ? __ffs((int)rot) - 1 : 0);
    d = d < WALK_QUEUE ? d : d - WALK_QUEUE;
    const float4 own = s_pend[wave][d][lane];
    const int c = __builtin_amdgcn_readlane(__float_as_int(own.x), __ffsll((long long)due) - 1);
    int dc = -1;
#pragma unroll
    for (int j = 0; j < WALK_QUEUE; ++j)
      if ((held >> j & 1u) && __float_as_int(s_pend[wave][j][lane].x) == c) dc = j;
    float r, gg, b;
    if (WALK_GROUP * __popcll(__ballot(dc >= 0)) >= __popcll(__ballot(held != 0u))) {
      const bool on = dc >= 0;
      const float4 p = s_pend[wave][max(dc, 0)][lane];
      const float ux = on ? p.y : 0.0f, uy = on ? p.z : 0.0f;
      const float* tx = S.tex + (int64_t)c * (KD * TEXW);
      radiance_wave(tx, uniform_ptr(tx), uniform_ptr(S.rgb + 3 * (int64_t)c), on, ux, uy, R.fx, R.fy, R.fz, S.tau, r,
                    gg, b);
      if (on) add(dc, p.w, r, gg, b);
    } else if (held != 0u) {
      const int own_c = __float_as_int(own.x);
      radiance_lane(S.tex + (int64_t)own_c * (KD * TEXW), S.rgb + 3 * (int64_t)own_c, own.y, own.z, R.fx, R.fy, R.fz,
                    S.tau, r, gg, b);
      add(d, own.w, r, gg, b);
    }
  };
  bool going = walked && max_steps > 0;
  cut = walked && max_steps == 0;
  int step = 0;
  while (__any(going)) {
    // every ray that goes on needs a free slot
    uint64_t full;
    while ((full = __ballot(going && (held >> slot & 1u))) != 0ull) {
      shade(full);
      __builtin_amdgcn_wave_barrier();
    }
    if (going) {
      going = false;   // set again where the walk goes on
      const float4 g = S.geo[cell];
      const Local L = make_local(R, g.x, g.y, g.z);
      const float4 bl = S.ball[cell];
      const int f0 = S.row[cell], nf = S.row[cell + 1] - f0;
      const float* tx = S.tex + (int64_t)cell * (KD * TEXW);
      // one pass over the faces clips the piece (the same arithmetic as the
      // rasteriser's; raster faces come first) and finds the exit: the nearest
      // face ahead of the current position that the ray leaves through, and the
      // second nearest, which is the exit where the nearest is the face the ray
      // came through (its neighbour is read for the winner alone)
      const double D = (double)g.w * (double)g.w - L.qq;
      const bool piece = D > 0.0 && bl.w >= 0.0f && ball_hit(R, ball_from(bl, R.ox, R.oy, R.oz));
      const int nr = piece ? S.nrast[cell] : 0;
      const float sq = piece ? fsqrt((float)D) : 0.0f;
      Interval I = {-sq, sq, -1, -1};
      const float s_cur = (float)(t_cur + L.b);
      const float s_min = s_cur - 1e-6f * (1.0f + fabsf(s_cur));
      const float nqx = -L.qx, nqy = -L.qy, nqz = -L.qz;
      float best = INFINITY, second = INFINITY;
      int bf = -1, sf = -1;
      auto face = [&](const float4 pl, int f) {
        const float a = face_slope(R, pl);
        const float s = face_offset(pl, nqx, nqy, nqz) * frcp(a);
        clip_face(I, a, s, f < nr, f);
        const bool ahead = a > 0.0f && s >= s_min && f < nf;
        const bool lt1 = ahead && s < best, lt2 = ahead && s < second;
        second = lt1 ? best : (lt2 ? s : second);
        sf = lt1 ? bf : (lt2 ? f : sf);
        best = lt1 ? s : best;
        bf = lt1 ? f : bf;
      };
      const float4* __restrict__ pf = S.plane + f0;
      for (int f = 0; f < nf; f += WALK_FACES) {
        float4 pl[WALK_FACES];
#pragma unroll
        for (int j = 0; j < WALK_FACES; ++j) pl[j] = pf[min(f + j, nf - 1)];
#pragma unroll
        for (int j = 0; j < WALK_FACES; ++j) face(pl[j], f + j);
      }
      bool contrib = false;
      Piece P;
      if (piece) {
        P = piece_dense<false>(R, L, I, S.nrm[cell], tx, S.tau);
        contrib = P.alpha > 0.0f;
      }
      if constexpr (COUNT) {
        n_pieces += (bl.w >= 0.0f && ball_hit(R, ball_from(bl, R.ox, R.oy, R.oz))) ? 1ull : 0ull;
        n_contrib += contrib ? 1ull : 0ull;
      }
      int rec = -1;
      if constexpr (STORE) {
        const uint64_t m = __ballot(contrib);
        if (m) {
          const int leader = __ffsll((long long)__ballot(true)) - 1;
          const int cnt = __popcll(m);
          if (cnt > rleft) {
            unsigned long long bk = 0;
            if (lane == leader) bk = atomicAdd(&rec_counter[0], (unsigned long long)RBLK);
            rblk = (long long)bcast64(bk);
            rleft = RBLK;
          }
          if (cnt > sleft) {
            unsigned long long bk = 0;
            if (lane == leader) bk = atomicAdd(&rec_counter[1], (unsigned long long)RBLK);
            sblk = (long long)bcast64(bk);
            sleft = RBLK;
          }
          if (contrib) {
            const long long rs = rblk + __popcll(m & lt), sg = sblk + __popcll(m & lt);
            if (rs < rec_cap) {
              rec_ri[rs] = make_int4(cell, pix, head, pack_view_bind(view, P.bind0, P.bind1));
              reinterpret_cast<float*>(rec_rf + rs)[0] = P.alpha;   // (the colour follows)
              rec_rt[rs] = T;
              head = rec = (int)rs;
              if (sg < seg_cap) rec_seg[sg] = make_int4(cell, (int)rs, 1, 0);   // mask 1: one record
            }
          }
          rblk += cnt;
          rleft -= cnt;
          sblk += cnt;
          sleft -= cnt;
        }
      }
      if (contrib) {
        s_pend[wave][slot][lane] = make_float4(__int_as_float(cell), P.ux, P.uy, T * P.alpha);
        if constexpr (STORE) s_rec[wave][slot][lane] = rec;
        held |= 1u << slot;
        slot = slot + 1 < WALK_QUEUE ? slot + 1 : 0;
        T *= (1.0f - P.alpha);
      }
      bool on = !(T < t_min);
      if (on) {
        if constexpr (COUNT) n_faces += (unsigned long long)nf;
        int nx = bf >= 0 ? S.col[f0 + bf] : prev;
        if (nx == prev && sf >= 0) {
          best = second;
          bf = sf;
          nx = S.col[f0 + bf];
        }
        if (nx == prev) {
          // no such face: the full scan, which takes the nearest exit of all where
          // none is ahead
          best = INFINITY;
          float best_any = INFINITY;
          int bf_any = -1;
          bf = -1;
          for (int f = 0; f < nf; ++f) {
            if (S.col[f0 + f] == prev) continue;
            const float4 pl = pf[f];
            const float a = face_slope(R, pl);
            if (!(a > 0.0f)) continue;
            const float s = face_offset(pl, nqx, nqy, nqz) * frcp(a);
            if (s < best_any) { best_any = s; bf_any = f; }
            if (s >= s_min && s < best) { best = s; bf = f; }
          }
          if (bf < 0) { bf = bf_any; best = best_any; }
          nx = bf >= 0 ? S.col[f0 + bf] : -1;
        }
        on = bf >= 0;
        if (on) {
          t_cur = fmax(t_cur, (double)best - L.b);
          on = nx >= 0;   // (else it left the domain box)
        }
        if (on) {
          prev = cell;
          cell = nx;
          ++step;
          going = step < max_steps;
          cut = !going;
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  uint64_t rest;
  while ((rest = __ballot(held != 0u)) != 0ull) {
    shade(rest);
    __builtin_amdgcn_wave_barrier();
  }
  n_steps = walked ? step + (step < max_steps ? 1 : 0) : 0;
  if (inside) {
    float* o = rgba + 4 * ((int64_t)py * v.cam.width + px);
    o[0] = cr;
    o[1] = cg;
    o[2] = cb;
    o[3] = 1.0f - T;
    if constexpr (STORE) rec_head[pix] = head;
  }
  const uint64_t bc = __ballot(cut);
  if ((threadIdx.x & 63) == 0 && bc) atomicAdd(truncated, (unsigned long long)__popcll(bc));
  if constexpr (COUNT) {
    unsigned long long w_steps = (unsigned long long)n_steps, w_pieces = n_pieces, w_contrib = n_contrib,
                       w_faces = n_faces;
    int w_max = n_steps;
    for (int o = 32; o > 0; o >>= 1) {
      w_steps += __shfl_xor(w_steps, o, 64);
      w_pieces += __shfl_xor(w_pieces, o, 64);
      w_contrib += __shfl_xor(w_contrib, o, 64);
      w_faces += __shfl_xor(w_faces, o, 64);
      w_max = max(w_max, __shfl_xor(w_max, o, 64));
    }
    const uint64_t bw = __ballot(walked);
    if (lane == 0) {
      atomicAdd(&counters[0], (unsigned long long)__popcll(bw));
      atomicAdd(&counters[1], w_steps);
      atomicAdd(&counters[2], w_pieces);
      atomicAdd(&counters[3], w_contrib);
      atomicAdd(&counters[4], w_faces);
      atomicMax(&counters[5], (unsigned long long)w_max);
    }
  }
}

BallArgs ball_args(const Scene& sc) { return {sc.geo, sc.cull, sc.ball, sc.ball_top, sc.prm.tex}; }

SceneDev scene_dev(const Scene& sc, const float4* ball) {
  SceneDev d;
  d.geo = sc.geo;
  d.nrm = sc.nrm;
  d.ball = ball;
  d.row = sc.row;
  d.nrast = sc.nrast;
  d.col = sc.col;
  d.plane = sc.plane;
  d.rgb = sc.prm.rgb;
  d.tex = sc.prm.tex;
  d.tau = sc.prm.tau;
  return d;
}

template <typename T>
struct Buf {
  T* p = nullptr;
  hipStream_t s;
  explicit Buf(hipStream_t st) : s(st) {}
  ~Buf() { if (p) pf::pool_free(p, s); }
  hipError_t alloc(size_t count) { return pf::pool_alloc((void**)&p, sizeof(T) * (count ? count : 1), s); }
};

}  // namespace

bool camera_ok(const pf_camera& c, std::string* why) {
  if (c.model != 0 && c.model != 1) { *why = "camera model must be 0 or 1"; return false; }
  if (c.width < 1 || c.height < 1 || (int64_t)c.width * c.height > (1ll << 31) / 4) {
    *why = "camera size out of range"; return false;
  }
  for (int i = 0; i < 12; ++i)
    if (!std::isfinite(c.c2w[i])) { *why = "non-finite camera matrix"; return false; }
  if (c.model == 0 && !(c.fx > 0 && c.fy > 0 && std::isfinite(c.cx) && std::isfinite(c.cy))) {
    *why = "pinhole intrinsics must be finite with fx, fy > 0"; return false;
  }
  if (c.model == 1 && !(c.f_fish > 0 && c.theta_max > 0 && c.theta_max <= 3.14159274f)) {
    *why = "fisheye needs f_fish > 0 and 0 < theta_max <= pi"; return false;
  }
  return true;
}

int raster_group_size(int64_t n, int ncam) {
  // views are processed in groups so that the per-(view, cell) scan fits 32 bits
  return (int)std::max<int64_t>(1, std::min<int64_t>(ncam, ((int64_t)1 << 28) / n));
}

int64_t view_tiles(const pf_camera& c) {
  return (int64_t)((c.width + TILE - 1) / TILE) * ((c.height + TILE - 1) / TILE);
}

namespace {

// Consecutive arrays in one allocation, each on a 256-byte boundary.
struct Arena {
  int64_t bytes = 0;
  int64_t add(int64_t count, int64_t size) {
    const int64_t at = bytes;
    bytes += (std::max<int64_t>(count, 1) * size + 255) & ~(int64_t)255;
    return at;
  }
};

// A group's arrays that are sized by its cells and tiles, and those sized by
// its pairs: two allocations (an allocation's release records an event; with one
// for each of the thirteen arrays the releases of a small render took as long as
// its kernels).  The arrays that start as zeros are neighbours.
struct GroupLayout {
  Arena fixed, pairs;
  int64_t views, ball, cnt, key, off, cone_list, plan, toff, zero, tcnt, fill, cone_n, long_n, zero_end, ptile, pval,
      sorted, long_list;
  GroupLayout(int64_t n, int nv, int64_t ntiles, int64_t np) {
    const int64_t nvc = (int64_t)nv * n;
    views = fixed.add(nv, sizeof(ViewDev));
    ball = fixed.add(n, sizeof(float4));
    cnt = fixed.add(nvc + 1, 4);
    key = fixed.add(nvc, 4);
    off = fixed.add(nvc + 1, 4);
    cone_list = fixed.add(nvc, 4);
    plan = fixed.add(PLAN_LIST + ntiles, 4);
    toff = fixed.add(ntiles + 1, 4);
    zero = tcnt = fixed.add(ntiles + 1, 4);
    fill = fixed.add(ntiles, 4);
    cone_n = fixed.add(1, 4);
    long_n = fixed.add(1, 4);
    zero_end = fixed.bytes;
    ptile = pairs.add(np, 4);
    pval = pairs.add(np, 8);
    sorted = pairs.add(np, 8);
    long_list = pairs.add(np / (SORT_LDS + 1), 4);
  }
};

}  // namespace

int64_t raster_group_bytes(int64_t n, int nv, int64_t ntiles, int64_t np) {
  const int64_t nvc = (int64_t)nv * n;
  const GroupLayout l(n, nv, ntiles, np);
  return l.fixed.bytes + l.pairs.bytes + scan_scratch_bytes(nvc + 1) + scan_scratch_bytes(ntiles + 1);
}

namespace {

// The binned tile lists of one group of views (every buffer lives until
// the group is done).
struct Group {
  int c0 = 0, nv = 0;
  int64_t ntiles = 0, tiles_before = 0, pix_before = 0;
  uint32_t np = 0;
  Buf<char> fixed, pairs;
  template <typename T>
  struct Part {
    T* p = nullptr;
  };
  Part<ViewDev> views;
  Part<float4> ball;
  Part<uint32_t> cnt, key, off, tcnt, toff, fill, cone_list, cone_n, long_n, ptile, plan, long_list;
  Part<unsigned long long> pval, sorted;
  explicit Group(hipStream_t s) : fixed(s), pairs(s) {}
};

// Cull and count (count_only: stops after the pair count), then emit,
// bucket by tile and sort each tile's list.
pf_status bin_group(Scene& sc, const pf_camera* cams, Group& G, hipStream_t s, bool count_only) {
  const int64_t n = sc.n;
  const int nv = G.nv;
  std::vector<ViewDev> hv(nv);
  int64_t ntiles = 0, pix = G.pix_before;
  for (int v = 0; v < nv; ++v) {
    const pf_camera& cam = cams[G.c0 + v];
    hv[v].v.cam = cam;
    hv[v].v.tiles_x = (cam.width + TILE - 1) / TILE;
    hv[v].v.tiles_y = (cam.height + TILE - 1) / TILE;
    hv[v].v.pad = rect_pad(cam);
    hv[v].tile_base = ntiles;
    hv[v].pix_base = pix;
    hv[v].view_id = G.c0 + v;
    ntiles += (int64_t)hv[v].v.tiles_x * hv[v].v.tiles_y;
    pix += (int64_t)cam.width * cam.height;
  }
  G.ntiles = ntiles;
  const int64_t nvc = (int64_t)nv * n;
  {
    const GroupLayout l(n, nv, ntiles, 0);
    PF_HIP_TRY(G.fixed.alloc(l.fixed.bytes));
    char* p = G.fixed.p;
    G.views.p = (ViewDev*)(p + l.views);
    G.ball.p = (float4*)(p + l.ball);
    G.cnt.p = (uint32_t*)(p + l.cnt);
    G.key.p = (uint32_t*)(p + l.key);
    G.off.p = (uint32_t*)(p + l.off);
    G.cone_list.p = (uint32_t*)(p + l.cone_list);
    G.plan.p = (uint32_t*)(p + l.plan);
    G.toff.p = (uint32_t*)(p + l.toff);
    G.tcnt.p = (uint32_t*)(p + l.tcnt);
    G.fill.p = (uint32_t*)(p + l.fill);
    G.cone_n.p = (uint32_t*)(p + l.cone_n);
    G.long_n.p = (uint32_t*)(p + l.long_n);
    PF_HIP_TRY(hipMemsetAsync(p + l.zero, 0, (size_t)(l.zero_end - l.zero), s));
  }
  PF_HIP_TRY(hipMemcpyAsync(G.views.p, hv.data(), sizeof(ViewDev) * nv, hipMemcpyHostToDevice, s));
  const dim3 g((unsigned)((n + 255) / 256), (unsigned)nv);
  {
    // one view's threads form its balls themselves (for 256x256 at 1,048,576
    // cells 48 us in one launch, 25 and 35 in two); with more views each ball
    // is formed once
    ProfScope ps("k_view_count", s);
    if (nv == 1) {
      k_view_count<true><<<g, 256, 0, s>>>(G.views.p, ball_args(sc), G.ball.p, sc.prm.power, n, G.cnt.p, G.key.p,
                                           G.cone_list.p, G.cone_n.p);
    } else {
      k_live_ball<<<g.x, 256, 0, s>>>(ball_args(sc), n, G.ball.p);
      PF_HIP_TRY(hipGetLastError());
      k_view_count<false><<<g, 256, 0, s>>>(G.views.p, ball_args(sc), G.ball.p, sc.prm.power, n, G.cnt.p, G.key.p,
                                            G.cone_list.p, G.cone_n.p);
    }
  }
  PF_HIP_TRY(hipGetLastError());
  // A workgroup per cell that could be listed where those that find nothing
  // cost less than learning the number (16,384 of them 8 us, a synchronisation
  // and a copy 20 to 30); else as many as there are.
  uint32_t gcone = (uint32_t)nvc;
  if (nvc > 16384) {
    PF_HIP_TRY(hipMemcpyAsync(&gcone, G.cone_n.p, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    PF_HIP_TRY(hipStreamSynchronize(s));
  }
  if (gcone) {
    k_cone_count<<<gcone, 256, 0, s>>>(G.views.p, G.ball.p, n, G.cone_list.p, G.cone_n.p, G.cnt.p);
    PF_HIP_TRY(hipGetLastError());
  }
  PF_HIP_TRY(exclusive_scan_u32(G.cnt.p, G.off.p, nvc + 1, nullptr, s));
  uint32_t np = 0;
  PF_HIP_TRY(hipMemcpyAsync(&np, G.off.p + nvc, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
  PF_HIP_TRY(hipStreamSynchronize(s));
  G.np = np;
  double ppc = (double)np / (double)nvc;   // sizing hint (renders may run on several threads)
  __atomic_store(&sc.pairs_per_cell, &ppc, __ATOMIC_RELAXED);
  if (count_only) return PF_OK;
  {
    const GroupLayout l(n, nv, ntiles, np);
    PF_HIP_TRY(G.pairs.alloc(l.pairs.bytes));
    G.ptile.p = (uint32_t*)(G.pairs.p + l.ptile);
    G.pval.p = (unsigned long long*)(G.pairs.p + l.pval);
    G.sorted.p = (unsigned long long*)(G.pairs.p + l.sorted);
    G.long_list.p = (uint32_t*)(G.pairs.p + l.long_list);
  }
  {
    ProfScope ps("k_view_emit", s);
    k_view_emit<<<g, 256, 0, s>>>(G.views.p, G.ball.p, n, G.off.p, G.key.p, G.ptile.p, G.pval.p, G.tcnt.p);
    if (gcone)
      k_cone_emit<<<gcone, 256, 0, s>>>(G.views.p, G.ball.p, n, G.off.p, G.key.p, G.cone_list.p, G.cone_n.p,
                                        G.ptile.p, G.pval.p, G.tcnt.p);
  }
  PF_HIP_TRY(hipGetLastError());
  PF_HIP_TRY(exclusive_scan_u32(G.tcnt.p, G.toff.p, ntiles + 1, nullptr, s));
  if (np) {
    k_tile_scatter<<<(unsigned)((np + 255) / 256), 256, 0, s>>>(G.ptile.p, G.pval.p, np, G.toff.p, G.fill.p,
                                                               G.sorted.p);
    PF_HIP_TRY(hipGetLastError());
    ProfScope ps("k_tile_sort", s);
    k_tile_sort<<<(unsigned)ntiles, SORT_THREADS, 0, s>>>(G.sorted.p, G.toff.p, G.long_list.p, G.long_n.p);
    PF_HIP_TRY(hipGetLastError());
    const uint32_t most = np / (SORT_LDS + 1);   // lists that can be that long
    if (most)
      k_tile_sort_long<<<std::min(most, 256u), SORT_LONG_THREADS, 0, s>>>(G.sorted.p, G.toff.p, G.long_list.p,
                                                                        G.long_n.p);
    PF_HIP_TRY(hipGetLastError());
  }
  return PF_OK;
}

template <bool STORE, bool COUNT>
void launch_raster(Scene& sc, Group& G, float t_min, float* rgba, hipStream_t s, const RecBuf& rb, int64_t first,
                   int64_t count, int64_t wtail_base, unsigned long long* counters) {
  k_split_plan<<<1, PLAN_THREADS, 0, s>>>(G.toff.p, first, count, G.plan.p);
  // (one workgroup of sixteen waves per CU is resident)
  k_raster_split<STORE, COUNT><<<(unsigned)std::min<int64_t>(4 * count, 256), 64 * NW, 0, s>>>(
      G.views.p, G.nv, scene_dev(sc, G.ball.p), G.sorted.p, G.toff.p, t_min, rgba, rb.ri, rb.rf, rb.rt, rb.head, rb.counter,
      rb.seg, rb.wtail, wtail_base, rb.cap, rb.seg_cap, first, G.plan.p, counters);
  k_raster<STORE, COUNT><<<(unsigned)count, 256, 0, s>>>(
      G.views.p, G.nv, scene_dev(sc, G.ball.p), G.sorted.p, G.toff.p, t_min, rgba, rb.ri, rb.rf, rb.rt, rb.head, rb.counter,
      rb.seg, rb.wtail, wtail_base, rb.cap, rb.seg_cap, first, G.plan.p, counters);
}

// Composite of the group's tiles [first, first + count) (one launch, one
// workgroup per tile); with records, the wave segment tails go to
// rec->wtail from index wtail_base.
pf_status composite(Scene& sc, Group& G, float t_min, float* rgba, hipStream_t s, const RecBuf* rec,
                    int64_t first, int64_t count, int64_t wtail_base, unsigned long long* counters) {
  if (count <= 0) return PF_OK;
  ProfScope ps(rec ? "k_raster_store" : "k_raster", s);
  if (rec) {
    if (counters) launch_raster<true, true>(sc, G, t_min, rgba, s, *rec, first, count, wtail_base, counters);
    else launch_raster<true, false>(sc, G, t_min, rgba, s, *rec, first, count, wtail_base, nullptr);
  } else {
    if (counters) launch_raster<false, true>(sc, G, t_min, rgba, s, RecBuf{}, first, count, 0, counters);
    else launch_raster<false, false>(sc, G, t_min, rgba, s, RecBuf{}, first, count, 0, nullptr);
  }
  PF_HIP_TRY(hipGetLastError());
  return PF_OK;
}

}  // namespace

pf_status raster_views(Scene& sc, const pf_camera* cams, int ncam, float t_min, float* rgba, hipStream_t s,
                       const RecBuf* rec, const GroupFn* fn, unsigned long long* counters) {
  const int group = raster_group_size(sc.n, ncam);
  int64_t pix_done = 0, tiles_done = 0;
  for (int c0 = 0; c0 < ncam; c0 += group) {
    Group G(s);
    G.c0 = c0;
    G.nv = std::min(group, ncam - c0);
    G.tiles_before = tiles_done;
    G.pix_before = pix_done;
    pf_status st = bin_group(sc, cams, G, s, false);
    if (st != PF_OK) return st;
    if (fn) {
      const GroupComposite run = [&](int64_t first, int64_t count, const RecBuf* r) {
        return composite(sc, G, t_min, rgba, s, r, first, count, 0, counters);
      };
      st = (*fn)(tiles_done, G.ntiles, run);
    } else {
      st = composite(sc, G, t_min, rgba, s, rec, 0, G.ntiles, tiles_done, counters);
    }
    if (st != PF_OK) return st;
    tiles_done += G.ntiles;
    for (int v = 0; v < G.nv; ++v) pix_done += (int64_t)cams[c0 + v].width * cams[c0 + v].height;
  }
  return PF_OK;
}

pf_status raster_workspace(Scene& sc, const pf_camera* cams, int ncam, hipStream_t s, int64_t* bytes) {
  const int group = raster_group_size(sc.n, ncam);
  int64_t worst = 0, pix_done = 0;
  for (int c0 = 0; c0 < ncam; c0 += group) {
    Group G(s);
    G.c0 = c0;
    G.nv = std::min(group, ncam - c0);
    G.pix_before = pix_done;
    const pf_status st = bin_group(sc, cams, G, s, true);
    if (st != PF_OK) return st;
    worst = std::max(worst, raster_group_bytes(sc.n, G.nv, G.ntiles, G.np));
    for (int v = 0; v < G.nv; ++v) pix_done += (int64_t)cams[c0 + v].width * cams[c0 + v].height;
  }
  *bytes = worst;
  return PF_OK;
}

pf_status seg_record_total(const int4* seg, int64_t nseg, unsigned long long* total_dev, hipStream_t s) {
  PF_HIP_TRY(hipMemsetAsync(total_dev, 0, sizeof(unsigned long long), s));
  if (nseg > 0) {
    const unsigned nb = (unsigned)std::min<int64_t>(1024, (nseg + 255) / 256);
    k_seg_total<<<nb, 256, 0, s>>>(seg, nseg, total_dev);
    PF_HIP_TRY(hipGetLastError());
  }
  return PF_OK;
}

pf_status trace_view(const Scene& sc, const pf_camera& cam, float t_min, int max_steps, float* rgba,
                     unsigned long long* trunc_dev, hipStream_t s, const RecBuf* rec, int view, int64_t pix_base,
                     int64_t tile_first, int64_t tile_count, const TraceScratch* scratch,
                     unsigned long long* counters) {
  const int64_t n = sc.n;
  ViewArgs v;
  v.cam = cam;
  v.tiles_x = (cam.width + TILE - 1) / TILE;
  v.tiles_y = (cam.height + TILE - 1) / TILE;
  v.pad = 0.0;   // (no tile lists)
  const int64_t ntiles = tile_count >= 0 ? tile_count : (int64_t)v.tiles_x * v.tiles_y - tile_first;
  if (ntiles <= 0) return PF_OK;
  const int nb = (int)std::min<int64_t>(TRACE_START_BLOCKS, (n + 255) / 256);
  Buf<double> pk_own(s);
  Buf<long long> pi_own(s);
  Buf<int32_t> start_own(s);
  double* pk = scratch ? scratch->pk : nullptr;
  long long* pi = scratch ? scratch->pi : nullptr;
  int32_t* start = scratch ? scratch->start : nullptr;
  if (!scratch) {
    PF_HIP_TRY(pk_own.alloc(nb));
    PF_HIP_TRY(pi_own.alloc(nb));
    PF_HIP_TRY(start_own.alloc(1));
    pk = pk_own.p;
    pi = pi_own.p;
    start = start_own.p;
  }
  k_start_partial<<<nb, 256, 0, s>>>(sc.prm.p, sc.prm.power, sc.flags, n, cam.c2w[3], cam.c2w[7], cam.c2w[11],
                                     ball_args(sc), pk, pi);
  PF_HIP_TRY(hipGetLastError());
  k_start_final<<<1, 256, 0, s>>>(pk, pi, nb, start);
  PF_HIP_TRY(hipGetLastError());
  ProfScope ps(rec ? "k_trace_store" : "k_trace", s);
  if (rec) {
    const RecBuf& rb = *rec;
    if (counters)
      k_trace<true, true><<<(unsigned)ntiles, 256, 0, s>>>(v, tile_first, scene_dev(sc, sc.ball), start, t_min, max_steps,
                                                           rgba, trunc_dev, view, rb.ri, rb.rf, rb.rt,
                                                           rb.head + pix_base, rb.counter, rb.seg, rb.cap, rb.seg_cap,
                                                           counters);
    else
      k_trace<true, false><<<(unsigned)ntiles, 256, 0, s>>>(v, tile_first, scene_dev(sc, sc.ball), start, t_min, max_steps,
                                                            rgba, trunc_dev, view, rb.ri, rb.rf, rb.rt,
                                                            rb.head + pix_base, rb.counter, rb.seg, rb.cap,
                                                            rb.seg_cap, nullptr);
  } else if (counters) {
    k_trace<false, true><<<(unsigned)ntiles, 256, 0, s>>>(v, tile_first, scene_dev(sc, sc.ball), start, t_min, max_steps, rgba,
                                                          trunc_dev, 0, nullptr, nullptr, nullptr, nullptr, nullptr,
                                                          nullptr, 0, 0, counters);
  } else {
    k_trace<false, false><<<(unsigned)ntiles, 256, 0, s>>>(v, tile_first, scene_dev(sc, sc.ball), start, t_min, max_steps,
                                                           rgba, trunc_dev, 0, nullptr, nullptr, nullptr, nullptr,
                                                           nullptr, nullptr, 0, 0, nullptr);
  }
  PF_HIP_TRY(hipGetLastError());
  return PF_OK;
}

}  // namespace pf
