// Scene build: face adjacency of the power diagram clipped to the domain
// box, a ball around each cell's dense part and hidden-cell flags.
//
// What is computed: for every cell i the faces of
//   Pi_i = { x : |x-p_i|^2 - w_i <= |x-p_j|^2 - w_j }  (appendix B)
// inside the domain box; these are the regular-triangulation edges the ray
// walk crosses (appendix C).  Faces whose plane lies within r_i of p_i are
// listed first: only they can cut the bounded cell Pi_i n B(p_i, r_i) that
// the rasteriser composites (Sec. 3.2).
//
// How (gfx950): sites are Morton-sorted and grouped into an implicit 64-ary
// tree (leaves of 64 consecutive sites; each node keeps an AABB and the
// largest weight below it).  One wave64 owns one cell and holds its convex
// polytope in registers as up to 128 vertices, two per lane, each vertex the
// intersection of three planes with positive orientation det(m_a,m_b,m_c).
// Clipping by a plane removes the vertices beyond it and re-triangulates the
// cavity: every edge (a,b) from a removed vertex to a kept one yields the new
// vertex (a,b,k).  An LDS table maps directed edges to vertex slots.
// Candidates come nearest-first from the cell's own leaf, then from a tree
// walk that prunes a node when no site in its box can be closer in power
// than p_i to any current vertex:  dist(v,box)^2 - maxw >= |v-p_i|^2 - w_i.
// Everything in the clipper is float64 in cell-local coordinates (FP64 runs
// at the unpacked FP32 rate on CDNA).
#include "pf_internal.hpp"

#include <type_traits>
#include <vector>

namespace pf {
namespace {

constexpr int PM_MID = 128;       // plane capacity of the second pass (edge table in LDS)
constexpr int SPL_MID = 4;        // vertex slots per lane of the second pass
constexpr int PM_BIG = 256;       // plane capacity of the third pass (edge table in HBM)
constexpr int SPL_BIG = 8;        // vertex slots per lane of the third pass
// traversal stack: the unvisited siblings along one root-to-leaf path,
// (levels - 2) x 63 + 64 + the root's children: 190 entries at 16M sites
constexpr int STACK = 192;
constexpr int WIT = 8;           // per empty cell: four planes that prove it empty, then seeds (write_witness)
constexpr int64_t ELIM_MIN = 24000;   // cells from which the empty ones are taken out first (build_scene_impl)
constexpr int RING_K = 16;        // rank of the leaf mate that sets the first ring radius
// Upper bound on candidate clips plus node visits per cell; a cell that
// reaches it is reported as over capacity instead of running on.
constexpr int WORK_LIMIT = 1 << 22;


__device__ inline uint32_t spread10(uint32_t v) {
  v &= 1023u;
  v = (v | (v << 16)) & 0x030000FFu;
  v = (v | (v << 8)) & 0x0300F00Fu;
  v = (v | (v << 4)) & 0x030C30C3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

__device__ inline float wave_min(float x) {
  for (int o = 32; o > 0; o >>= 1) x = fminf(x, __shfl_xor(x, o, 64));
  return x;
}
__device__ inline float wave_max(float x) {
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
  return x;
}
// Wave-wide reductions of a double with DPP moves (all 64 lanes active):
// butterflies within rows of 16 lanes, then the row broadcasts of lanes 15
// and 31 leave the result in lane 63, which is read back to every lane.
template <int CTRL, int ROW_MASK>
__device__ inline double dpp_d(double x, double old) {
  const long long xb = __double_as_longlong(x), ob = __double_as_longlong(old);
  const int lo = __builtin_amdgcn_update_dpp((int)ob, (int)xb, CTRL, ROW_MASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(ob >> 32), (int)(xb >> 32), CTRL, ROW_MASK, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ inline double lane63_d(double x) {
  const long long xb = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)xb, 63), hi = __builtin_amdgcn_readlane((int)(xb >> 32), 63);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ inline double wave_max_d(double x) {
  x = fmax(x, dpp_d<0xB1, 0xf>(x, -INFINITY));    // quad perm [1,0,3,2]
  x = fmax(x, dpp_d<0x4E, 0xf>(x, -INFINITY));    // quad perm [2,3,0,1]
  x = fmax(x, dpp_d<0x141, 0xf>(x, -INFINITY));   // row half mirror
  x = fmax(x, dpp_d<0x140, 0xf>(x, -INFINITY));   // row mirror
  x = fmax(x, dpp_d<0x142, 0xa>(x, -INFINITY));   // row bcast 15
  x = fmax(x, dpp_d<0x143, 0xc>(x, -INFINITY));   // row bcast 31
  return lane63_d(x);
}
__device__ inline double wave_sum_d(double x) {
  x += dpp_d<0xB1, 0xf>(x, 0.0);
  x += dpp_d<0x4E, 0xf>(x, 0.0);
  x += dpp_d<0x141, 0xf>(x, 0.0);
  x += dpp_d<0x140, 0xf>(x, 0.0);
  x += dpp_d<0x142, 0xa>(x, 0.0);
  x += dpp_d<0x143, 0xc>(x, 0.0);
  return lane63_d(x);
}

// Per-block partial bounds of the spheres and weights:
// [minx,miny,minz,maxx,maxy,maxz,maxw,minr] per block.
__global__ void __launch_bounds__(256) k_bounds(const float* __restrict__ p, const float* __restrict__ w,
                                                const float* __restrict__ r, int64_t n,
                                                float* __restrict__ part) {
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  float wmax = -INFINITY, rmin = INFINITY;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    float ri = r[i];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      float c = p[3 * i + a];
      lo[a] = fminf(lo[a], c - ri);
      hi[a] = fmaxf(hi[a], c + ri);
    }
    wmax = fmaxf(wmax, w[i]);
    rmin = fminf(rmin, ri);
  }
  __shared__ float red[4][8];
  float v[8] = {lo[0], lo[1], lo[2], hi[0], hi[1], hi[2], wmax, rmin};
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    bool is_min = (q < 3) || (q == 7);
    v[q] = is_min ? wave_min(v[q]) : wave_max(v[q]);
    if (lane == 0) red[wv][q] = v[q];
  }
  __syncthreads();
  if (threadIdx.x < 8) {
    int q = threadIdx.x;
    bool is_min = (q < 3) || (q == 7);
    float a = red[0][q];
    for (int k = 1; k < 4; ++k) a = is_min ? fminf(a, red[k][q]) : fmaxf(a, red[k][q]);
    part[blockIdx.x * 8 + q] = a;
  }
}

__global__ void k_morton(const float* __restrict__ p, int64_t n, float3 lo, float3 inv,
                         uint32_t* __restrict__ keys, uint32_t* __restrict__ vals) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint32_t q[3];
  float l[3] = {lo.x, lo.y, lo.z}, s[3] = {inv.x, inv.y, inv.z};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float t = (p[3 * i + a] - l[a]) * s[a];
    t = fminf(fmaxf(t, 0.0f), 1023.0f);
    q[a] = (uint32_t)t;
  }
  keys[i] = spread10(q[0]) | (spread10(q[1]) << 1) | (spread10(q[2]) << 2);
  vals[i] = (uint32_t)i;
}

__global__ void k_gather_sites(const float* __restrict__ p, const float* __restrict__ w,
                               const float* __restrict__ r, const uint32_t* __restrict__ order, int64_t n,
                               float4* __restrict__ sp, int32_t* __restrict__ sidx, float* __restrict__ srad) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  uint32_t i = order[k];
  sp[k] = make_float4(p[3 * i], p[3 * i + 1], p[3 * i + 2], w[i]);
  sidx[k] = (int32_t)i;
  srad[k] = r[i];
}

// One wave per parent node: AABB and max weight of up to 64 children.
__global__ void __launch_bounds__(64) k_tree_level(const float4* __restrict__ sp, const float* __restrict__ srad,
                                                   const float4* __restrict__ clo, const float4* __restrict__ chi,
                                                   int64_t nchild, float4* __restrict__ olo,
                                                   float4* __restrict__ ohi) {
  const int lane = threadIdx.x;
  const int64_t c = (int64_t)blockIdx.x * 64 + lane;
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY}, w = -INFINITY;
  float rmax = 0.0f;
  if (c < nchild) {
    if (sp) {
      float4 s = sp[c];
      lo[0] = hi[0] = s.x;
      lo[1] = hi[1] = s.y;
      lo[2] = hi[2] = s.z;
      w = s.w;
      rmax = srad ? srad[c] : 0.0f;
    } else {
      float4 a = clo[c], b = chi[c];
      lo[0] = a.x; lo[1] = a.y; lo[2] = a.z; w = a.w;
      hi[0] = b.x; hi[1] = b.y; hi[2] = b.z;
      rmax = b.w;
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    lo[a] = wave_min(lo[a]);
    hi[a] = wave_max(hi[a]);
  }
  w = wave_max(w);
  rmax = wave_max(rmax);
  if (lane == 0) {
    olo[blockIdx.x] = make_float4(lo[0], lo[1], lo[2], w);
    ohi[blockIdx.x] = make_float4(hi[0], hi[1], hi[2], rmax);
  }
}

// ---------------------------------------------------------------------------
// Clipper of one cell, run by one wave.  SPL vertex slots per lane (64*SPL
// vertices), PM plane capacity; the directed-edge -> vertex-slot table has
// PM*PM entries of type EOT and lives in LDS (small variant) or in a per-cell
// HBM workspace (large variant, for the few cells of very high degree).

template <int SPL, int PM>
struct Shared {
  double pl[PM][4];               // planes (m.x, m.y, m.z, h), cell-local
  int nb[PM];                     // neighbour (original index) or -1-f
  union {                         // never live at the same time (one wave per block)
    int tid[64 * SPL];            // packed plane triples of the vertices being written
    float key[64];                // per-lane ordering keys
  };
  double tpos[64 * SPL][3];       // the vertices
  double bd[8];                   // bounds of the polytope (update_bounds)
  int stack[STACK];
  unsigned char used[PM];
  unsigned short remap[PM];
  unsigned short hole[64 * SPL];  // slots of the vertices that the current clip removes
  unsigned short edge[64 * SPL];  // plane pairs of the edges it cuts
  unsigned char ord[64];          // lanes of the flagged candidates in processing order
  int last;                       // the site whose plane emptied the cell
};

// EMPTY_HERE: emptied by a coincident site (no plane); EMPTY_VOID: a dropped cell
enum ClipResult { NOCUT = 0, CUT = 1, EMPTY = 2, OVER_V = 3, OVER_P = 4, OVER_W = 5, OVER_S = 6, EMPTY_HERE = 7,
                  EMPTY_VOID = 8 };

__device__ inline bool is_over(int st) { return st >= OVER_V && st <= OVER_S; }
__device__ inline bool is_empty(int st) { return st == EMPTY || st >= EMPTY_HERE; }

template <int SPL>
struct Poly {
  int id[SPL];                    // packed (a | b<<8 | c<<16), slot lane + 64*s
  double x[SPL], y[SPL], z[SPL];  // vertex positions
  int ntri;                       // wave-uniform vertex count
  bool stale;                     // the bounds in Shared are those of an earlier (larger) polytope
};

// Shared::bd: max |v|^2 and its root, the vertex centroid, the largest squared
// distance from it and its root, and |centroid| + that root (roots rounded up)
constexpr int BD_R2 = 0, BD_R = 1, BD_CX = 2, BD_CY = 3, BD_CZ = 4, BD_RC2 = 5, BD_RC = 6, BD_CN = 7;

// Square root for bounds only: the hardware's (about 24 bits), which callers
// widen by SQRT_UP or SQRT_DOWN.
__device__ inline double sqrt_about(double x) { return __builtin_amdgcn_sqrt(x); }
constexpr double SQRT_UP = 1.0 + 1e-6, SQRT_DOWN = 1.0 - 1e-6;

__device__ inline int lane_int(int x, int src) { return __builtin_amdgcn_readlane(x, src); }
__device__ inline float lane_float(float x, int src) { return __int_as_float(lane_int(__float_as_int(x), src)); }
__device__ inline double lane_double(double x, int src) {
  const long long b = __double_as_longlong(x);
  return __longlong_as_double(((long long)lane_int((int)(b >> 32), src) << 32) | (unsigned int)lane_int((int)b, src));
}

__device__ inline void unpack(int id, int& a, int& b, int& c) {
  a = id & 255;
  b = (id >> 8) & 255;
  c = (id >> 16) & 255;
}


template <int PM, typename EOT>
__device__ inline void reg_edges(EOT* eo, int id, int slot) {
  int a, b, c;
  unpack(id, a, b, c);
  eo[a * PM + b] = (EOT)slot;
  eo[b * PM + c] = (EOT)slot;
  eo[c * PM + a] = (EOT)slot;
}

// Point where planes a, b and (m, h) meet; returns the determinant of the
// normals (positive for the triple of a vertex).
template <int SPL, int PM>
__device__ inline double plane_triple(const Shared<SPL, PM>& S, int a, int b, double mx, double my, double mz,
                                      double h, double& x, double& y, double& z) {
  const double ax = S.pl[a][0], ay = S.pl[a][1], az = S.pl[a][2], ah = S.pl[a][3];
  const double bx = S.pl[b][0], by = S.pl[b][1], bz = S.pl[b][2], bh = S.pl[b][3];
  // c23 = b x k, c31 = k x a, c12 = a x b
  const double c23x = by * mz - bz * my, c23y = bz * mx - bx * mz, c23z = bx * my - by * mx;
  const double c31x = my * az - mz * ay, c31y = mz * ax - mx * az, c31z = mx * ay - my * ax;
  const double c12x = ay * bz - az * by, c12y = az * bx - ax * bz, c12z = ax * by - ay * bx;
  const double det = ax * c23x + ay * c23y + az * c23z;
  const double inv = 1.0 / det;
  x = (ah * c23x + bh * c31x + h * c12x) * inv;
  y = (ah * c23y + bh * c31y + h * c12y) * inv;
  z = (ah * c23z + bh * c31z + h * c12z) * inv;
  return det;
}

template <int SPL, int PM>
__device__ inline void update_bounds(Shared<SPL, PM>& S, Poly<SPL>& P) {
  const int lane = threadIdx.x;
  double m = 0.0, sx = 0.0, sy = 0.0, sz = 0.0;
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    if (lane + 64 * s < P.ntri) {
      m = fmax(m, P.x[s] * P.x[s] + P.y[s] * P.y[s] + P.z[s] * P.z[s]);
      sx += P.x[s];
      sy += P.y[s];
      sz += P.z[s];
    }
  }
  const double r2 = wave_max_d(m);
  const double inv = 1.0 / (double)P.ntri;
  const double cx = wave_sum_d(sx) * inv, cy = wave_sum_d(sy) * inv, cz = wave_sum_d(sz) * inv;
  double mc = 0.0;
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    if (lane + 64 * s < P.ntri) {
      const double dx = P.x[s] - cx, dy = P.y[s] - cy, dz = P.z[s] - cz;
      mc = fmax(mc, dx * dx + dy * dy + dz * dz);
    }
  }
  const double rc2 = wave_max_d(mc);
  if (lane == 0) {
    S.bd[BD_R2] = r2;
    S.bd[BD_R] = sqrt_about(r2) * SQRT_UP;
    S.bd[BD_CX] = cx; S.bd[BD_CY] = cy; S.bd[BD_CZ] = cz;
    S.bd[BD_RC2] = rc2;
    S.bd[BD_RC] = sqrt_about(rc2) * SQRT_UP;
    S.bd[BD_CN] = (sqrt_about(cx * cx + cy * cy + cz * cz) + sqrt_about(rc2)) * SQRT_UP;
  }
  __syncthreads();
  P.stale = false;
}

template <int SPL, int PM, typename EOT>
__device__ int compact_planes(Shared<SPL, PM>& S, EOT* eo, Poly<SPL>& P, int nplanes);

// Vertices that lie on a plane up to rounding are kept: sites on a grid give planes
// that only touch the polytope.  (Decided by rounding, the vertices beyond such a plane need not be connected,
// and two pairs of edges then share an entry of the edge table.)  Relative to the
// reach of the polytope, or of a larger one before it (tol = CUT_TOL times that);
// a vertex is off by some 1e-16 of it, and a tenth of CUT_TOL passes the tests too.
// With this and the look for equal planes below, k_clip takes 7.40 instead of 7.29 ms
// in a rebuild of 1,048,576 cells.
constexpr double CUT_TOL = 1e-13;

// Clip the polytope by the plane (m, h) of site orig.  A plane that cuts is
// stored as number nplanes (the caller counts it).  Vertices that stay keep
// their slots and their edges; the new ones, one per cut edge and computed one
// per lane, take the slots of the removed ones and then those behind the last.
template <int SPL, int PM, typename EOT>
__device__ ClipResult clip(Shared<SPL, PM>& S, EOT* eo, Poly<SPL>& P, int& nplanes, int orig, double mx, double my,
                           double mz, double h, double tol) {
  constexpr int NT = 64 * SPL;
  const int lane = threadIdx.x;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const double slack = tol * (fabs(mx) + fabs(my) + fabs(mz)), limit = h + slack, well = h + 1e4 * slack;
  bool out[SPL], deep = false;
  uint64_t ob[SPL];
  int nout = 0;
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    const double at = mx * P.x[s] + my * P.y[s] + mz * P.z[s];
    out[s] = lane + 64 * s < P.ntri && at > limit;
    deep = deep || (out[s] && at > well);
    ob[s] = __ballot(out[s]);
    nout += __popcll(ob[s]);
  }
  if (nout == 0) return NOCUT;
  if (!__any(deep)) {
    // hardly a cut: perhaps the plane of a site at the place of one taken before (the
    // same normal and no smaller an offset), which cuts nothing
    bool same = false;
    for (int q = lane; q < nplanes; q += 64)
      same = same || (S.pl[q][0] == mx && S.pl[q][1] == my && S.pl[q][2] == mz && S.pl[q][3] <= h);
    if (__any(same)) return NOCUT;
  }
  if (nplanes == PM) {
    nplanes = compact_planes(S, eo, P, nplanes);
    if (nplanes == PM) return OVER_P;
  }
  const int kp = nplanes;
  if (lane == 0) {
    S.pl[kp][0] = mx; S.pl[kp][1] = my; S.pl[kp][2] = mz; S.pl[kp][3] = h;
    S.nb[kp] = orig;
  }
  if (nout == P.ntri) {
    __syncthreads();
    return EMPTY;
  }

  // the edges it cuts: from a removed vertex to a kept one
  bool e[3 * SPL];
  int ex[3 * SPL], ey[3 * SPL];
  int my_new = 0;
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    int a, b, c;
    unpack(P.id[s], a, b, c);
    const int xs[3] = {a, b, c}, ys[3] = {b, c, a};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      ex[3 * s + q] = xs[q];
      ey[3 * s + q] = ys[q];
      bool keep_opp = false;
      if (out[s]) {
        const int opp = (int)eo[ys[q] * PM + xs[q]] & (NT - 1);
        uint64_t m = ob[0];
#pragma unroll
        for (int t = 1; t < SPL; ++t) m = (opp >> 6) == t ? ob[t] : m;
        keep_opp = ((m >> (opp & 63)) & 1ull) == 0ull;
      }
      e[3 * s + q] = out[s] && keep_opp;
      my_new += e[3 * s + q] ? 1 : 0;
    }
  }
  // exclusive prefix sum and total of my_new (< 2^NB) from one ballot per bit
  constexpr int NB = SPL <= 2 ? 3 : SPL <= 5 ? 4 : 5;
  int excl = 0, n_new = 0;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const uint64_t bm = __ballot((my_new >> b) & 1);
    excl += __popcll(bm & lt) << b;
    n_new += __popcll(bm) << b;
  }
  const int n_old = P.ntri, n_tot = n_old - nout + n_new;
  if (n_tot > NT) return OVER_V;
  int hbase = 0;
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    if (out[s]) S.hole[hbase + __popcll(ob[s] & lt)] = (unsigned short)(lane + 64 * s);
    hbase += __popcll(ob[s]);
  }
#pragma unroll
  for (int q = 0; q < 3 * SPL; ++q)
    if (e[q]) S.edge[excl++] = (unsigned short)(ex[q] | (ey[q] << 8));
  __syncthreads();
  for (int j = lane; j < n_new; j += 64) {
    const int ed = S.edge[j], a = ed & 255, b = ed >> 8;
    const int slot = j < nout ? S.hole[j] : n_old + (j - nout);
    double x, y, z;
    plane_triple(S, a, b, mx, my, mz, h, x, y, z);
    S.tid[slot] = a | (b << 8) | (kp << 16);
    S.tpos[slot][0] = x; S.tpos[slot][1] = y; S.tpos[slot][2] = z;
  }
  if (n_new < nout) {
    // fewer new than removed: the kept vertices behind the new end move into
    // the holes left over (which lie before it: hole j is at most the number
    // of kept vertices plus j)
    int kb = n_new;
#pragma unroll
    for (int s = 0; s < SPL; ++s) {
      const bool move = lane + 64 * s < n_old && !out[s] && lane + 64 * s >= n_tot;
      const uint64_t mb = __ballot(move);
      if (move) {
        const int slot = S.hole[kb + __popcll(mb & lt)];
        S.tid[slot] = P.id[s];
        S.tpos[slot][0] = P.x[s]; S.tpos[slot][1] = P.y[s]; S.tpos[slot][2] = P.z[s];
      }
      kb += __popcll(mb);
    }
  }
  __syncthreads();
  P.ntri = n_tot;
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    const int t = lane + 64 * s;
    if (t < n_tot && (out[s] || t >= n_old)) {
      P.id[s] = S.tid[t];
      P.x[s] = S.tpos[t][0]; P.y[s] = S.tpos[t][1]; P.z[s] = S.tpos[t][2];
      reg_edges<PM>(eo, P.id[s], t);
    }
  }
  __syncthreads();
  P.stale = true;
  return CUT;
}

// Whether the bisector plane (m, h) can reach the polytope: it must come
// within the bounding ball around the vertex centroid (or p_i coincides
// with the other site).
template <int SPL, int PM>
__device__ inline bool may_cut(const Shared<SPL, PM>& S, double mx, double my, double mz, double mm, double h) {
  const double t = h - (mx * S.bd[BD_CX] + my * S.bd[BD_CY] + mz * S.bd[BD_CZ]);
  return t < 0.0 || t * t < S.bd[BD_RC2] * mm || mm == 0.0;
}

struct Cand {
  double mx, my, mz, mm, h;
  int orig;
  bool ok;
};

__device__ inline Cand load_cand(const float4* __restrict__ sp, const int32_t* __restrict__ sidx, int64_t j,
                                 bool valid, double px, double py, double pz, double wi) {
  Cand c;
  c.ok = valid;
  c.mx = c.my = c.mz = c.mm = c.h = 0.0;
  c.orig = -1;
  if (valid) {
    float4 s = sp[j];
    c.mx = (double)s.x - px;
    c.my = (double)s.y - py;
    c.mz = (double)s.z - pz;
    c.mm = c.mx * c.mx + c.my * c.my + c.mz * c.mz;
    c.h = 0.5 * (c.mm + wi - (double)s.w);
    c.orig = sidx ? sidx[j] : -1;
  }
  return c;
}

// Drops planes that no longer bound the polytope and renumbers the rest,
// so that the plane capacity limits live faces only.  Returns the new plane
// count.
template <int SPL, int PM, typename EOT>
__device__ int compact_planes(Shared<SPL, PM>& S, EOT* eo, Poly<SPL>& P, int nplanes) {
  constexpr int NR = (PM + 63) / 64;
  const int lane = threadIdx.x;
  for (int q = lane; q < PM; q += 64) S.used[q] = 0;
  __syncthreads();
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    if (lane + 64 * s < P.ntri) {
      int a, b, c;
      unpack(P.id[s], a, b, c);
      S.used[a] = 1; S.used[b] = 1; S.used[c] = 1;
    }
  }
  __syncthreads();
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  bool u[NR];
  int dst[NR];
  double pl[NR][4];
  int nbv[NR];
  int base = 0;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int q = lane + 64 * r;
    u[r] = q < nplanes && q < PM && S.used[q];
    const uint64_t m = __ballot(u[r]);
    dst[r] = base + __popcll(m & lt);
    base += __popcll(m);
    if (u[r]) {
      for (int c = 0; c < 4; ++c) pl[r][c] = S.pl[q][c];
      nbv[r] = S.nb[q];
      S.remap[q] = (unsigned short)dst[r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if (u[r]) {
      for (int c = 0; c < 4; ++c) S.pl[dst[r]][c] = pl[r][c];
      S.nb[dst[r]] = nbv[r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    if (lane + 64 * s < P.ntri) {
      int a, b, c;
      unpack(P.id[s], a, b, c);
      P.id[s] = S.remap[a] | (S.remap[b] << 8) | (S.remap[c] << 16);
    }
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < SPL; ++s)
    if (lane + 64 * s < P.ntri) reg_edges<PM>(eo, P.id[s], lane + 64 * s);
  __syncthreads();
  return base;
}

// Whether the plane (m, h) cuts off a vertex of the current polytope (the
// vertex list after the last clip is in S.tpos).
template <int SPL, int PM>
__device__ inline bool cuts_vertices(const Shared<SPL, PM>& S, int ntri, double mx, double my, double mz,
                                     double h) {
  for (int t = 0; t < ntri; ++t)
    if (mx * S.tpos[t][0] + my * S.tpos[t][1] + mz * S.tpos[t][2] > h) return true;
  return false;
}

// Number of flagged lanes whose key orders before this lane's (ties by
// lane); keys of the wave in S.key.
template <int SPL, int PM>
__device__ inline int lane_rank(const Shared<SPL, PM>& S, uint64_t flagged, float key) {
  const int lane = threadIdx.x;
  int rank = 0;
  while (flagged) {
    const int t = __ffsll((long long)flagged) - 1;
    flagged &= flagged - 1;
    const float kt = S.key[t];
    rank += (kt < key || (kt == key && t < lane)) ? 1 : 0;
  }
  return rank;
}

// Maximum over the wave, in every lane (all lanes active).
__device__ inline float wave_max_dpp(float x) {
  const int lowest = __float_as_int(-INFINITY);
  auto step = [&](int moved) { x = fmaxf(x, __int_as_float(moved)); };
  step(__builtin_amdgcn_update_dpp(lowest, __float_as_int(x), 0xB1, 0xf, 0xf, false));    // quad perm [1,0,3,2]
  step(__builtin_amdgcn_update_dpp(lowest, __float_as_int(x), 0x4E, 0xf, 0xf, false));    // quad perm [2,3,0,1]
  step(__builtin_amdgcn_update_dpp(lowest, __float_as_int(x), 0x141, 0xf, 0xf, false));   // row half mirror
  step(__builtin_amdgcn_update_dpp(lowest, __float_as_int(x), 0x140, 0xf, 0xf, false));   // row mirror
  step(__builtin_amdgcn_update_dpp(lowest, __float_as_int(x), 0x142, 0xa, 0xf, false));   // row bcast 15
  step(__builtin_amdgcn_update_dpp(lowest, __float_as_int(x), 0x143, 0xc, 0xf, false));   // row bcast 31
  return __int_as_float(lane_int(__float_as_int(x), 63));
}

constexpr int FEW = 8;   // candidates up to which a batch is clipped one by one without a test of all

// Processes one batch of candidates (one per lane).  The polytope only
// shrinks, so a candidate whose plane misses the ball around it, or every
// current vertex, can never cut later and is dropped; the others are clipped
// in order of their bisector's offset from p_i (most constraining first).
// Candidates among the first nwl seeds (lane q % 64 of wl[q / 64]) were taken
// before.  Returns false when the cell became empty or overflowed (state in
// status).
template <int SPL, int PM, typename EOT, int NWL>
__device__ bool process_batch(Shared<SPL, PM>& S, EOT* eo, Poly<SPL>& P, int& nplanes, int& status, const Cand& c,
                              int self_orig, int& work, const int (&wl)[NWL], int nwl) {
  const int lane = threadIdx.x;
  if (P.stale) update_bounds(S, P);
  const double tol = CUT_TOL * S.bd[BD_R];
  bool f = c.ok && may_cut(S, c.mx, c.my, c.mz, c.mm, c.h);
  uint64_t fm = __ballot(f);
  if (fm == 0ull) return true;
  if (nwl > 0) {
#pragma unroll
    for (int r = 0; r < NWL; ++r)
      for (int q = 0; q < min(nwl - 64 * r, 64); ++q) f = f && lane_int(wl[r], q) != c.orig;
    fm = __ballot(f);
    if (fm == 0ull) return true;
  }
  // Many candidates: first the plane furthest on the wrong side of the vertex
  // centroid, again and again, each cutting off the larger part.  (By offset
  // alone, an empty cell of a build from scratch took 54 clips and another one
  // 83.)  Then, or when they are few, those left in order of their offset.
  bool deepest = __popcll(fm) > FEW;
  const double rm = c.mm > 0.0 ? __builtin_amdgcn_rsq(c.mm) : 0.0;
  int nflag = __popcll(fm), r = -1;
  for (;;) {
    int src;
    if (deepest) {
      if (P.stale) update_bounds(S, P);
      const float v = !f ? -INFINITY
                      : c.mm == 0.0 ? INFINITY
                                    : (float)((c.mx * S.bd[BD_CX] + c.my * S.bd[BD_CY] + c.mz * S.bd[BD_CZ] - c.h) * rm);
      const float best = wave_max_dpp(v);
      if (best > 0.0f) {
        src = __ffsll((long long)__ballot(v == best)) - 1;
        if (lane == src) f = false;
      } else {
        // clip() begins with the test against the vertices; here it is made
        // for all candidates at once, one per lane
        f = f && cuts_vertices(S, P.ntri, c.mx, c.my, c.mz, c.h);
        fm = __ballot(f);
        if (fm == 0ull) return true;
        nflag = __popcll(fm);
        deepest = false;
        continue;
      }
    } else {
      if (r < 0) {
        r = 0;
        if (nflag > 1) {
          // most constraining first: the plane's offset from p_i, h/|m|
          // (coincident sites first)
          const float okey = c.mm > 0.0 ? (float)(c.h * rm) : -INFINITY;
          S.key[lane] = f ? okey : INFINITY;
          __syncthreads();
          if (f) S.ord[lane_rank(S, fm, okey)] = (unsigned char)lane;
        } else if (f) {
          S.ord[0] = (unsigned char)lane;
        }
        __syncthreads();
      }
      if (r == nflag) return true;
      src = __builtin_amdgcn_readfirstlane((int)S.ord[r]);
      ++r;
    }
    if (++work > WORK_LIMIT) {
      status = OVER_W;
      return false;
    }
    const double mx = lane_double(c.mx, src), my = lane_double(c.my, src), mz = lane_double(c.mz, src),
                 h = lane_double(c.h, src);
    const int orig = lane_int(c.orig, src);
    if (mx == 0.0 && my == 0.0 && mz == 0.0) {
      // coincident sites: the one with the smaller weight (or, on a tie,
      // the larger index) owns nothing
      if (h < 0.0 || (h == 0.0 && orig < self_orig)) {
        status = EMPTY_HERE;
        if (lane == 0) S.last = orig;
        return false;
      }
      continue;
    }
    const ClipResult res = clip(S, eo, P, nplanes, orig, mx, my, mz, h, tol);
    if (res == CUT) {
      ++nplanes;
    } else if (res == EMPTY || is_over(res)) {
      status = res;
      return false;
    }
  }
}

// Why a cell is empty, for the next build: out[0] is the site whose plane
// left nothing of the polytope, out[1..3] the planes of the polytope's vertex
// nearest to it.  That vertex minimises m.x over the polytope (m the emptying
// plane's normal), so its planes with non-negative weights balance m, and no
// point satisfies the four planes (k_witness checks exactly that for the new
// positions).  Box face f is stored as -2 - f, no plane as -1; out[4..7] are
// the most recent planes before it.  All lanes take part.
template <int SPL, int PM>
__device__ void write_witness(const Shared<SPL, PM>& S, const Poly<SPL>& P, int nplanes, int status,
                              int32_t* __restrict__ out) {
  const int lane = threadIdx.x;
  auto code = [](int nb) { return nb < 0 ? nb - 1 : nb; };
  if (status == EMPTY_HERE) {   // a site at the same place with a larger weight
    if (lane < WIT) out[lane] = lane == 0 ? S.last : -1;
    return;
  }
  const double mx = S.pl[nplanes][0], my = S.pl[nplanes][1], mz = S.pl[nplanes][2];
  double best = INFINITY;
  int id = 0;
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    if (lane + 64 * s < P.ntri) {
      const double d = mx * P.x[s] + my * P.y[s] + mz * P.z[s];
      if (d < best) {
        best = d;
        id = P.id[s];
      }
    }
  }
  const double least = -wave_max_d(-best);
  const int src = __ffsll((long long)__ballot(best == least)) - 1;
  id = __shfl(id, src, 64);
  int a, b, c;
  unpack(id, a, b, c);
  if (lane < WIT) {
    const int q = lane == 0 ? nplanes : lane == 1 ? a : lane == 2 ? b : lane == 3 ? c : nplanes - (lane - 3);
    // (no plane twice: as seeds they are clipped one after the other)
    const bool twice = lane > 3 && (q == a || q == b || q == c);
    out[lane] = q >= 0 && q < PM && !twice ? code(S.nb[q]) : -1;
  }
}

// A ball around the part of the cell that can contribute to an image: the
// polytope where (x - p).n <= disp, inside the sphere, disp the sites' largest
// displacement or 0.
// (The displaced face lies within the sites' displacements, so the dense side
// does not reach past that plane; a ray along the face counts the side below
// the undisplaced one.)  Its corners are the vertices on that side and the
// points where the edges across the plane meet it.  The smaller of two balls
// is taken: around p, of the sphere's radius at most, or around the middle of
// the corners' box.  Cell-local centre and radius (no margin), radius -1 when
// there are no corners.  All lanes take part.
template <int SPL, int PM, typename EOT>
__device__ float4 dense_ball(const Shared<SPL, PM>& S, const EOT* eo, const Poly<SPL>& P,
                             const float* __restrict__ normal, float disp, float r) {
  constexpr int NT = 64 * SPL;
  const int lane = threadIdx.x;
  // (a normal whose float32 unit vector (k_prep) is not finite cuts nothing off:
  // every comparison of the piece with its face is false)
  const float fx = normal[0], fy = normal[1], fz = normal[2], finv = 1.0f / sqrtf(fx * fx + fy * fy + fz * fz);
  const bool face = fabsf(fx * finv) + fabsf(fy * finv) + fabsf(fz * finv) < INFINITY;
  const double ax = fx, ay = fy, az = fz;
  const double inv = 1.0 / sqrt(ax * ax + ay * ay + az * az);
  const double nx = face ? ax * inv : 0.0, ny = face ? ay * inv : 0.0, nz = face ? az * inv : 0.0;
  const double top = face ? (double)disp * (1.0 + 1e-5) + 1e-7 * (double)r : INFINITY;
  uint64_t above[SPL];
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    const int t = lane + 64 * s;
    above[s] = __ballot(t < P.ntri && !(nx * P.x[s] + ny * P.y[s] + nz * P.z[s] <= top));
  }
  auto corners = [&](auto&& fn) {
#pragma unroll
    for (int s = 0; s < SPL; ++s) {
      if (lane + 64 * s >= P.ntri) continue;
      if (!((above[s] >> lane) & 1ull)) {
        fn((float)P.x[s], (float)P.y[s], (float)P.z[s]);
        continue;
      }
      int a, b, c;
      unpack(P.id[s], a, b, c);
      const int xs[3] = {a, b, c}, ys[3] = {b, c, a};
      const double h0 = nx * P.x[s] + ny * P.y[s] + nz * P.z[s] - top;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const int opp = (int)eo[ys[q] * PM + xs[q]] & (NT - 1);
        uint64_t m = above[0];
#pragma unroll
        for (int t = 1; t < SPL; ++t) m = (opp >> 6) == t ? above[t] : m;
        if ((m >> (opp & 63)) & 1ull) continue;
        const double ox = S.tpos[opp][0], oy = S.tpos[opp][1], oz = S.tpos[opp][2];
        const double h1 = nx * ox + ny * oy + nz * oz - top;   // <= 0 < h0
        const double f = h0 * __builtin_amdgcn_rcp(h0 - h1);
        fn((float)(P.x[s] + f * (ox - P.x[s])), (float)(P.y[s] + f * (oy - P.y[s])),
           (float)(P.z[s] + f * (oz - P.z[s])));
      }
    }
  };
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY}, far = -1.0f;
  corners([&](float x, float y, float z) {
    lo[0] = fminf(lo[0], x); hi[0] = fmaxf(hi[0], x);
    lo[1] = fminf(lo[1], y); hi[1] = fmaxf(hi[1], y);
    lo[2] = fminf(lo[2], z); hi[2] = fmaxf(hi[2], z);
    far = fmaxf(far, x * x + y * y + z * z);
  });
  far = wave_max_dpp(far);
  if (far < 0.0f) return make_float4(0.0f, 0.0f, 0.0f, -1.0f);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    lo[a] = -wave_max_dpp(-lo[a]);
    hi[a] = wave_max_dpp(hi[a]);
  }
  const float cx = 0.5f * (lo[0] + hi[0]), cy = 0.5f * (lo[1] + hi[1]), cz = 0.5f * (lo[2] + hi[2]);
  float fc = 0.0f;
  corners([&](float x, float y, float z) {
    fc = fmaxf(fc, (x - cx) * (x - cx) + (y - cy) * (y - cy) + (z - cz) * (z - cz));
  });
  const float rc = sqrtf(wave_max_dpp(fc)), rp = fminf(r, sqrtf(far));
  return rc < rp ? make_float4(cx, cy, cz, rc) : make_float4(0.0f, 0.0f, 0.0f, rp);
}

// MODE 0: all cells, sorted position k = blockIdx.x, faces at stride
// FACE_CAP by original index, edge table in LDS.  MODE 1: the cells listed
// in klist (sorted positions), faces at stride PM_BIG in slot blockIdx.x
// (recorded in bigslot), edge table in LDS.  MODE 2: listed cells that
// already own a slot, edge table in an HBM workspace (for PM*PM too large
// for LDS).
// sp, sidx and the tree hold the n sites that take part; wsp, wspos (all wn
// sites, by original index) are where the previous build's seeds are read.
template <int SPL, int PM, int MODE>
__global__ void __launch_bounds__(64) k_clip(const float4* __restrict__ sp, const int32_t* __restrict__ sidx,
                                             int64_t n, const float4* __restrict__ nlo,
                                             const float4* __restrict__ nhi, Levels lv, float3 bmin,
                                             float3 bmax, const float* __restrict__ radius,
                                             const int32_t* __restrict__ klist, unsigned short* __restrict__ eo_g,
                                             int32_t* __restrict__ faces, int32_t* __restrict__ bigslot,
                                             int32_t* __restrict__ counts, int32_t* __restrict__ nrast,
                                             float* __restrict__ cull, int32_t* __restrict__ flags,
                                             const int32_t* __restrict__ wrow, const int32_t* __restrict__ wcol,
                                             const int32_t* __restrict__ wtri,
                                             const int32_t* __restrict__ wwit, const float4* __restrict__ wsp,
                                             const int32_t* __restrict__ wspos, int64_t wn,
                                             int32_t* __restrict__ wit_out, const float* __restrict__ normal,
                                             const float* __restrict__ tex, float4* __restrict__ ball,
                                             float* __restrict__ ball_top) {
  constexpr bool LISTED = MODE >= 1, EO_HBM = MODE == 2;
  using EOT = typename std::conditional<(64 * SPL > 256), unsigned short, unsigned char>::type;
  static_assert(EO_HBM ? std::is_same<EOT, unsigned short>::value : true, "HBM edge table holds 16-bit slots");
  __shared__ Shared<SPL, PM> S;
  __shared__ EOT eo_lds[EO_HBM ? 1 : PM * PM];
  EOT* eo;
  if constexpr (EO_HBM) eo = (EOT*)(eo_g + (int64_t)blockIdx.x * PM * PM);
  else eo = eo_lds;
  const int lane = threadIdx.x;
  const int64_t k = LISTED ? (int64_t)klist[blockIdx.x] : (int64_t)blockIdx.x;
  const float4 me = sp[k];
  const int32_t self = sidx[k];
  const double px = me.x, py = me.y, pz = me.z, wi = me.w;
  const double ri = radius[self];

  // distances to the faces of the domain box
  const double bh[6] = {(double)bmax.x - px, px - (double)bmin.x, (double)bmax.y - py,
                        py - (double)bmin.y, (double)bmax.z - pz, pz - (double)bmin.z};
  Poly<SPL> P;
  int nplanes = 6;
  // a dropped cell (weight -inf) has an empty power cell and cuts no other
  int status = wi > -INFINITY ? CUT : EMPTY_VOID;
  int work = 0;

  // phase 1, from a previous build: a cell that had faces starts from its
  // previous neighbours (sites that moved little keep most of them), then one
  // unrestricted traversal certifies it; a cell that was empty starts from
  // the sites that emptied it, which usually empty it again at once.
  // Otherwise (or if that fails) the own leaf (Morton neighbours) and rings.
  const int64_t leaf = k / LEAF;
  const int wb = (MODE <= 1 && wrow) ? wrow[self] : 0;
  const int wcnt = (MODE <= 1 && wrow) ? wrow[self + 1] - wb : 0;
  const bool warm = wcnt > 0;
  constexpr int NWL = MODE == 0 ? 1 : (PM + 63) / 64;
  int wl[NWL];   // the seeds already taken, spread over the lanes
  int nwl = 0;
#pragma unroll
  for (int r = 0; r < NWL; ++r) wl[r] = -1;
  double dmax = 0.0;

  // The previous faces and vertices (as triples of faces) at once: all planes
  // and, one per lane, the points where each triple's planes meet now.  When
  // every point lies inside every other plane and the box, the points are
  // vertices of the polytope of these planes, and all of them: each has its
  // three edges leading to others of the list, as before, and a polytope's
  // vertices are connected.  (Else the planes are taken one by one.  At
  // 1,048,576 cells moved by 1e-4, 15 clips of a start from the box took
  // 110,000 cycles.)
  bool whole = false;
  if (MODE <= 1 && status == CUT && warm && wcnt <= PM && 2 * wcnt - 4 <= 64 * SPL && wtri[2 * (int64_t)wb] >= 0) {
    const int F = wcnt, V = 2 * F - 4;
    uint64_t boxes = 0;   // box faces among the faces
    for (int f0 = 0; f0 < F; f0 += 64) {
      const int f = f0 + lane;
      int v = 0;
      if (f < F) {
        v = wcol[wb + f];
        double mx = 0.0, my = 0.0, mz = 0.0, h = INFINITY;
        if (v >= 0 && v < wn) {
          const float4 q = wsp[wspos[v]];
          mx = (double)q.x - px;
          my = (double)q.y - py;
          mz = (double)q.z - pz;
          h = 0.5 * (mx * mx + my * my + mz * mz + wi - (double)q.w);
        } else if (v < 0 && v >= -6) {
          const int bf = -1 - v, ax = bf >> 1;
          const double sgn = (bf & 1) ? -1.0 : 1.0;
          mx = ax == 0 ? sgn : 0.0;
          my = ax == 1 ? sgn : 0.0;
          mz = ax == 2 ? sgn : 0.0;
          h = ax == 0 ? (bf & 1 ? bh[1] : bh[0]) : ax == 1 ? (bf & 1 ? bh[3] : bh[2]) : (bf & 1 ? bh[5] : bh[4]);
        }
        S.pl[f][0] = mx; S.pl[f][1] = my; S.pl[f][2] = mz; S.pl[f][3] = h;
        S.nb[f] = v;
      }
#pragma unroll
      for (int r = 0; r < NWL; ++r)
        if (f0 == 64 * r) wl[r] = f < F ? v : -1;
#pragma unroll
      for (int q = 0; q < 6; ++q)
        if (__any(f < F && v == -1 - q)) boxes |= 1ull << q;
    }
    __syncthreads();
    bool bad = false;
    int tri[SPL];
#pragma unroll
    for (int s = 0; s < SPL; ++s) {
      const int t = lane + 64 * s;
      P.id[s] = tri[s] = 0;
      P.x[s] = P.y[s] = P.z[s] = 0.0;
      if (t < V) {
        tri[s] = wtri[2 * (int64_t)wb + t];
        int a, b, c;
        unpack(tri[s], a, b, c);
        bad = bad || tri[s] < 0 || a >= F || b >= F || c >= F;
        if (!bad) {
          const double det = plane_triple(S, a, b, S.pl[c][0], S.pl[c][1], S.pl[c][2], S.pl[c][3], P.x[s], P.y[s],
                                          P.z[s]);
          bad = !(det > 0.0);
          const double q[6] = {P.x[s], -P.x[s], P.y[s], -P.y[s], P.z[s], -P.z[s]};
#pragma unroll
          for (int f = 0; f < 6; ++f) bad = bad || (!((boxes >> f) & 1ull) && !(q[f] < bh[f]));
        }
      }
    }
    if (!__any(bad)) {
      for (int f = 0; f < F; ++f) {
        const double mx = S.pl[f][0], my = S.pl[f][1], mz = S.pl[f][2], h = S.pl[f][3];
#pragma unroll
        for (int s = 0; s < SPL; ++s) {
          int a, b, c;
          unpack(tri[s], a, b, c);
          bad = bad || (lane + 64 * s < V && f != a && f != b && f != c &&
                        !(mx * P.x[s] + my * P.y[s] + mz * P.z[s] < h));
        }
        if (__any(bad)) break;
      }
    }
    whole = !__any(bad);
    if (whole) {
      P.ntri = V;
      P.stale = true;
      nplanes = F;
      nwl = F;
      dmax = INFINITY;
#pragma unroll
      for (int s = 0; s < SPL; ++s) {
        if (lane + 64 * s < V) {
          P.id[s] = tri[s];
          S.tpos[lane + 64 * s][0] = P.x[s];
          S.tpos[lane + 64 * s][1] = P.y[s];
          S.tpos[lane + 64 * s][2] = P.z[s];
          reg_edges<PM>(eo, tri[s], lane + 64 * s);
        }
      }
    }
    __syncthreads();
  }
  // more faces than this pass holds: left to the next one
  if (MODE <= 1 && status == CUT && wcnt > PM) status = OVER_P;

  if (!whole) {
    // the domain box as the initial polytope
    if (lane < 6) {
      const int ax = lane >> 1;
      const double sgn = (lane & 1) ? -1.0 : 1.0;
      S.pl[lane][0] = ax == 0 ? sgn : 0.0;
      S.pl[lane][1] = ax == 1 ? sgn : 0.0;
      S.pl[lane][2] = ax == 2 ? sgn : 0.0;
      S.pl[lane][3] = ax == 0 ? (lane & 1 ? bh[1] : bh[0]) : ax == 1 ? (lane & 1 ? bh[3] : bh[2])
                                                                   : (lane & 1 ? bh[5] : bh[4]);
      S.nb[lane] = -1 - lane;
    }
    P.ntri = 8;
    P.stale = true;
#pragma unroll
    for (int s = 0; s < SPL; ++s) {
      P.id[s] = 0;
      P.x[s] = P.y[s] = P.z[s] = 0.0;
    }
    if (lane < 8) {
      const int sx = (lane & 1) ? -1 : 1, sy = (lane & 2) ? -1 : 1, sz = (lane & 4) ? -1 : 1;
      const int X = sx > 0 ? 0 : 1, Y = sy > 0 ? 2 : 3, Z = sz > 0 ? 4 : 5;
      // orientation det(m_X, m_Y, m_Z) = sx*sy*sz
      P.id[0] = (sx * sy * sz > 0) ? (X | (Y << 8) | (Z << 16)) : (Y | (X << 8) | (Z << 16));
      P.x[0] = sx > 0 ? bh[0] : -bh[1];
      P.y[0] = sy > 0 ? bh[2] : -bh[3];
      P.z[0] = sz > 0 ? bh[4] : -bh[5];
      S.tpos[lane][0] = P.x[0]; S.tpos[lane][1] = P.y[0]; S.tpos[lane][2] = P.z[0];
    }
    __syncthreads();
    if (lane < 8) reg_edges<PM>(eo, P.id[0], lane);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NWL; ++r) wl[r] = -1;
    if (MODE <= 1 && wrow && status == CUT && (warm || wwit)) {
      const int ns = warm ? min(wcnt, 64) : WIT;
      const int v = lane < ns ? (warm ? wcol[wb + lane] : wwit[(int64_t)self * WIT + lane]) : -1;
      const bool ok = v >= 0 && v < wn && v != self;
      Cand c = load_cand(wsp, nullptr, ok ? (int64_t)wspos[v] : 0, ok, px, py, pz, wi);
      c.orig = ok ? v : -1;
      process_batch(S, eo, P, nplanes, status, c, self, work, wl, 0);
      wl[0] = c.orig;
      nwl = ns;
      if (warm) dmax = INFINITY;
    }
  }
  if (!warm && status == CUT) {
    const int64_t j = leaf * LEAF + lane;
    bool ok = j < n && j != k;
    double d2 = INFINITY;
    if (ok) {
      const float4 q = sp[j];
      const double dx = (double)q.x - px, dy = (double)q.y - py, dz = (double)q.z - pz;
      d2 = dx * dx + dy * dy + dz * dz;
    }
    // first ring radius: the RING_K-th nearest leaf mate, at most r_i (a
    // Morton leaf can straddle a jump of the curve and span the scene)
    const uint64_t okm = __ballot(ok);
    S.key[lane] = ok ? (float)d2 : INFINITY;
    __syncthreads();
    const int target = min(RING_K, __popcll(okm) - 1);
    const uint64_t sel = __ballot(ok && lane_rank(S, okm, (float)d2) == target);
    __syncthreads();
    const double dk = sel ? __shfl(d2, __ffsll((long long)sel) - 1, 64) : 0.0;
    dmax = fmax(fmin(sqrt(dk), ri), 1e-6);
    const Cand c = load_cand(sp, sidx, j, ok, px, py, pz, wi);
    process_batch(S, eo, P, nplanes, status, c, self, work, wl, nwl);
  }

  // phase 2: the other sites in rings [dmin, dmax) of doubling radius, which
  // brings near sites first across the whole tree and keeps the transient
  // polytope small.  Each ring walks the tree depth first, most constraining
  // child first, pruning by the current polytope; a ring that left no
  // prunable work beyond dmax ends the search.
  double dmin = 0.0;
  while (status == CUT) {
    bool skipped = false;
    int top = 1;
    if (lane == 0) S.stack[0] = (lv.n << 24) | 0;
    __syncthreads();
    while (top > 0 && status == CUT) {
      if (++work > WORK_LIMIT) {
        status = OVER_W;
        break;
      }
      const int ent = __builtin_amdgcn_readfirstlane(S.stack[top - 1]);
      --top;
      const int L = ent >> 24;
      const long long idx = ent & 0xFFFFFF;
      if (P.stale) update_bounds(S, P);
      if (L == 1) {
        if (idx == leaf && !warm) continue;
        const int64_t j = idx * LEAF + lane;
        const bool ok = j < n && j != k;
        Cand c = load_cand(sp, sidx, j, ok, px, py, pz, wi);
        if (dmax < INFINITY || dmin > 0.0) {
          const bool beyond = ok && c.mm >= dmax * dmax;
          if (__ballot(beyond && may_cut(S, c.mx, c.my, c.mz, c.mm, c.h)) != 0ull) skipped = true;
          c.ok = ok && !beyond && c.mm >= dmin * dmin;
        }
        if (!process_batch(S, eo, P, nplanes, status, c, self, work, wl, nwl)) break;
        continue;
      }
      // children are nodes of level L-1
      const long long cnum = lv.cnt[L - 1];
      const long long cidx = idx * 64 + lane;
      const bool valid = cidx < cnum;
      float4 bl = make_float4(0.0f, 0.0f, 0.0f, 0.0f), bu = bl;   // (box and largest weight, in bl.w)
      bool keep = false;
      double dkey = INFINITY;
      if (valid) {
        bl = nlo[lv.off[L - 1] + cidx];
        bu = nhi[lv.off[L - 1] + cidx];
        const double lx = (double)bl.x - px, ly = (double)bl.y - py, lz = (double)bl.z - pz, W = bl.w;
        const double hx = (double)bu.x - px, hy = (double)bu.y - py, hz = (double)bu.z - pz;
        // ball around p_i
        const double dx = fmax(0.0, fmax(lx, -hx)), dy = fmax(0.0, fmax(ly, -hy)), dz = fmax(0.0, fmax(lz, -hz));
        const double D = sqrt_about(dx * dx + dy * dy + dz * dz) * SQRT_DOWN;
        const double R = S.bd[BD_R];
        const bool far0 = D > R && (D - R) * (D - R) - W >= S.bd[BD_R2] - wi;
        // ball around the vertex centroid
        const double cx = S.bd[BD_CX], cy = S.bd[BD_CY], cz = S.bd[BD_CZ];
        const double ex = fmax(0.0, fmax(lx - cx, cx - hx)), ey = fmax(0.0, fmax(ly - cy, cy - hy));
        const double ez = fmax(0.0, fmax(lz - cz, cz - hz));
        const double Dc = sqrt_about(ex * ex + ey * ey + ez * ez) * SQRT_DOWN, Rc = S.bd[BD_RC], cn = S.bd[BD_CN];
        const bool far1 = Dc > Rc && (Dc - Rc) * (Dc - Rc) - W >= cn * cn - wi;
        keep = !(far0 || far1);
        if (keep && D >= dmax) {
          skipped = true;   // wait for a later ring
          keep = false;
        }
        // lower bound of the bisector offset h/|m| of any site in the box
        if (keep) dkey = (D * D + wi - W) / (2.0 * fmax(D, 1e-12));
      }
      if (__ballot(valid && skipped) != 0ull) skipped = true;
      // exact per-vertex test: can any site in the box beat p_i at a vertex of
      // the current polytope?  For a few boxes the lanes are the vertices and
      // the boxes are taken in turn, for many the other way round.
      const uint64_t km = __ballot(keep);
      uint64_t cm = 0;
      if (2 * __popcll(km) <= P.ntri) {
        for (uint64_t m = km; m; m &= m - 1) {
          const int src = __ffsll((long long)m) - 1;
          const double lx = (double)lane_float(bl.x, src) - px, ly = (double)lane_float(bl.y, src) - py,
                       lz = (double)lane_float(bl.z, src) - pz, W = lane_float(bl.w, src);
          const double hx = (double)lane_float(bu.x, src) - px, hy = (double)lane_float(bu.y, src) - py,
                       hz = (double)lane_float(bu.z, src) - pz;
          bool cut = false;
#pragma unroll
          for (int s = 0; s < SPL; ++s) {
            if (lane + 64 * s < P.ntri) {
              const double vx = P.x[s], vy = P.y[s], vz = P.z[s];
              const double dx = fmax(0.0, fmax(lx - vx, vx - hx));
              const double dy = fmax(0.0, fmax(ly - vy, vy - hy));
              const double dz = fmax(0.0, fmax(lz - vz, vz - hz));
              cut = cut || dx * dx + dy * dy + dz * dz - W < vx * vx + vy * vy + vz * vz - wi;
            }
          }
          if (__any(cut)) cm |= 1ull << src;
        }
      } else {
        bool cut = false;
        if (keep) {
          const double lx = (double)bl.x - px, ly = (double)bl.y - py, lz = (double)bl.z - pz, W = bl.w;
          const double hx = (double)bu.x - px, hy = (double)bu.y - py, hz = (double)bu.z - pz;
          for (int t = 0; t < P.ntri && !cut; ++t) {
            const double vx = S.tpos[t][0], vy = S.tpos[t][1], vz = S.tpos[t][2];
            const double dx = fmax(0.0, fmax(lx - vx, vx - hx));
            const double dy = fmax(0.0, fmax(ly - vy, vy - hy));
            const double dz = fmax(0.0, fmax(lz - vz, vz - hz));
            cut = dx * dx + dy * dy + dz * dz - W < vx * vx + vy * vy + vz * vz - wi;
          }
        }
        cm = __ballot(cut);
      }
      if (cm != 0ull) {
        const int nc = __popcll(cm);
        if (top + nc > STACK) {
          status = OVER_S;
          break;
        }
        // most constraining child (smallest offset bound) on top of the stack
        const bool cut = (cm >> lane) & 1ull;
        S.key[lane] = cut ? (float)dkey : INFINITY;
        __syncthreads();
        if (cut) S.stack[top + nc - 1 - lane_rank(S, cm, (float)dkey)] = ((L - 1) << 24) | (int)(idx * 64 + lane);
        top += nc;
      }
      __syncthreads();
    }
    if (!skipped) break;
    // rings double until they lie beyond every vertex of the polytope; the
    // remaining sites can then only cut through their weight, and one
    // unrestricted traversal certifies the cell
    dmin = dmax;
    if (P.stale) update_bounds(S, P);
    dmax = (dmin * dmin >= S.bd[BD_R2]) ? INFINITY : 2.0 * dmax;
  }

  // --- outputs
  int32_t* out;
  if constexpr (MODE == 0) {
    out = faces + (int64_t)self * FACE_CAP;
  } else if constexpr (MODE == 1) {
    out = faces + (int64_t)blockIdx.x * PM_BIG;
    if (lane == 0) bigslot[self] = (int32_t)blockIdx.x;
  } else {
    out = faces + (int64_t)bigslot[self] * PM_BIG;
  }
  if (is_empty(status) || is_over(status)) {
    if (status == EMPTY || status == EMPTY_HERE)
      write_witness(S, P, nplanes, status, wit_out + (int64_t)self * WIT);
    else if (lane < WIT)
      wit_out[(int64_t)self * WIT + lane] = -1;
    if (lane == 0) {
      counts[self] = 0;
      nrast[self] = 0;
      cull[self] = -1.0f;
      ball[self] = make_float4(0.0f, 0.0f, 0.0f, -1.0f);
      const int why = status == OVER_V ? FLAG_OVER_VERTS : status == OVER_P ? FLAG_OVER_PLANES
                    : status == OVER_W ? FLAG_OVER_WORK : FLAG_OVER_STACK;
      flags[self] = status == EMPTY_HERE ? FLAG_EMPTY_POWER | FLAG_SAME_PLACE
                    : is_empty(status)   ? FLAG_EMPTY_POWER
                                         : (FLAG_OVERFLOW | why);
    }
    return;
  }
  // the largest displacement of the cell's face (loaded here, used at the end)
  const float disp = lane < KD ? site_top(tex + ((int64_t)self * KD + lane) * TEXW) : -INFINITY;
  for (int q = lane; q < PM; q += 64) S.used[q] = 0;
  __syncthreads();
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    if (lane + 64 * s < P.ntri) {
      int a, b, c;
      unpack(P.id[s], a, b, c);
      S.used[a] = 1; S.used[b] = 1; S.used[c] = 1;
    }
  }
  __syncthreads();
  // categories: 0 raster neighbour face, 1 other neighbour face, 2 box face
  constexpr int NR = (PM + 63) / 64;
  int cat[NR];
  double viol = -INFINITY;  // max over faces of the signed distance of p_i outside
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int q = lane + 64 * r;
    cat[r] = 3;
    if (q < nplanes && S.used[q]) {
      if (S.nb[q] < 0) {
        cat[r] = 2;
      } else {
        const double mx = S.pl[q][0], my = S.pl[q][1], mz = S.pl[q][2], h = S.pl[q][3];
        const double mn = sqrt(mx * mx + my * my + mz * mz);
        cat[r] = (fabs(h) <= ri * mn * (1.0 + 1e-6)) ? 0 : 1;
        viol = fmax(viol, -h / mn);
      }
    }
  }
  // faces by category, each category in increasing neighbour order (the
  // order in which the planes were taken does not show in the output)
#pragma unroll
  for (int r = 0; r < NR; ++r)
    if (lane + 64 * r < PM) S.used[lane + 64 * r] = (unsigned char)cat[r];
  __syncthreads();
  int cbase[3] = {0, 0, 0};
#pragma unroll
  for (int r = 0; r < NR; ++r)
    for (int ccat = 0; ccat < 3; ++ccat) cbase[ccat] += __popcll(__ballot(cat[r] == ccat));
  const int nr = cbase[0];
  const int base = cbase[0] + cbase[1] + cbase[2];
  cbase[2] = cbase[0] + cbase[1];
  cbase[1] = cbase[0];
  cbase[0] = 0;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int q = lane + 64 * r;
    if (cat[r] < 3) {
      const int me = S.nb[q];
      int pos = 0;
      for (int t = 0; t < nplanes; ++t)
        pos += (S.used[t] == cat[r] && (S.nb[t] < me || (S.nb[t] == me && t < q))) ? 1 : 0;
      out[cbase[cat[r]] + pos] = me;
      S.remap[q] = (unsigned short)(cbase[cat[r]] + pos);
    }
  }
  // the vertices as triples of faces (in output order) behind the faces, for
  // the next build, where the row has room
  constexpr int ROW = MODE == 0 ? FACE_CAP : PM_BIG;
  if (3 * base - 4 <= ROW) {
    __syncthreads();
    const bool simple = P.ntri == 2 * base - 4;   // (else a degenerate polytope: none)
#pragma unroll
    for (int s = 0; s < SPL; ++s) {
      const int t = lane + 64 * s;
      int a, b, c;
      unpack(P.id[s], a, b, c);
      if (t < 2 * base - 4)
        out[base + t] = simple ? S.remap[a] | (S.remap[b] << 8) | (S.remap[c] << 16) : -1;
    }
  }
  viol = wave_max_d(viol);
  if (P.stale) update_bounds(S, P);
  const double R = sqrt(S.bd[BD_R2]);
  const float top = fmaxf(wave_max_dpp(disp), 0.0f);
  const float4 bl = dense_ball(S, eo, P, normal + 3 * (int64_t)self, top, (float)ri);
  if (lane == 0) {
    counts[self] = base;
    nrast[self] = nr;
    const bool hidden = viol > ri;
    const float rcull = (float)fmin(ri, R * (1.0 + 1e-6));
    cull[self] = hidden ? -1.0f : rcull;
    float4 wide = widened_ball((float)(px + bl.x), (float)(py + bl.y), (float)(pz + bl.z), bl.w,
                               fabs(px) + fabs(py) + fabs(pz));
    if (hidden || bl.w < 0.0f) wide.w = -1.0f;
    ball[self] = wide;
    // (as large as the whole cell's, it does not depend on the displacements)
    ball_top[self] = bl.w >= rcull ? INFINITY : top;
    flags[self] = 0;
  }
}


// Connectivity loss over the Cech graph (supplementary material, loss
// functions): one wave per cell i walks the site tree for the spheres that
// overlap B(p_i, r_i) (nodes pruned by box distance > r_i + largest radius
// below).  With ov_ij = r_i + r_j - d_ij, each overlapping pair appears in
// L(i) and in L(j), so the derivative of the total with respect to r_i is
// 4 lambda sum_j ov_ij and with respect to p_i is
// 4 lambda sum_j ov_ij (p_j - p_i)/d_ij; every cell adds only its own
// gradient, so no atomics touch a neighbour.
__global__ void __launch_bounds__(64) k_connect(const float4* __restrict__ sp, const float* __restrict__ srad,
                                                const int32_t* __restrict__ sidx, int64_t n,
                                                const float4* __restrict__ nlo, const float4* __restrict__ nhi,
                                                Levels lv, float lambda, float* __restrict__ gp,
                                                float* __restrict__ gr, double* __restrict__ loss,
                                                unsigned int* __restrict__ overflow) {
  __shared__ int stack[STACK];
  const int lane = threadIdx.x;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const int64_t k = blockIdx.x;
  const float4 me = sp[k];
  const double px = me.x, py = me.y, pz = me.z, ri = srad[k];
  double lsum = 0.0, gsum = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
  int top = 1;
  if (lane == 0) stack[0] = (lv.n << 24) | 0;
  __syncthreads();
  while (top > 0) {
    const int ent = stack[top - 1];
    --top;
    const int L = ent >> 24;
    const long long idx = ent & 0xFFFFFF;
    if (L == 1) {
      const int64_t j = idx * LEAF + lane;
      if (j < n && j != k) {
        const float4 q = sp[j];
        const double dx = (double)q.x - px, dy = (double)q.y - py, dz = (double)q.z - pz;
        const double rs = ri + (double)srad[j];
        const double d2 = dx * dx + dy * dy + dz * dz;
        if (d2 < rs * rs) {
          const double d = sqrt(d2);
          const double ov = rs - d;
          lsum += ov * ov;
          gsum += ov;
          if (d > 0.0) {   // d ov / d p_i = (p_j - p_i) / d
            gx += ov * dx / d;
            gy += ov * dy / d;
            gz += ov * dz / d;
          }
        }
      }
      continue;
    }
    const long long cidx = idx * 64 + lane;
    bool keep = false;
    if (cidx < lv.cnt[L - 1]) {
      const float4 a = nlo[lv.off[L - 1] + cidx], b = nhi[lv.off[L - 1] + cidx];
      const double ex = fmax(0.0, fmax((double)a.x - px, px - (double)b.x));
      const double ey = fmax(0.0, fmax((double)a.y - py, py - (double)b.y));
      const double ez = fmax(0.0, fmax((double)a.z - pz, pz - (double)b.z));
      const double reach = ri + (double)b.w;
      keep = ex * ex + ey * ey + ez * ez < reach * reach;
    }
    const uint64_t m = __ballot(keep);
    const int nc = __popcll(m);
    if (top + nc > STACK) {
      if (lane == 0) atomicAdd(overflow, 1u);
      break;
    }
    if (keep) stack[top + __popcll(m & lt)] = ((L - 1) << 24) | (int)cidx;
    top += nc;
    __syncthreads();
  }
  lsum = wave_sum_d(lsum);
  gsum = wave_sum_d(gsum);
  gx = wave_sum_d(gx);
  gy = wave_sum_d(gy);
  gz = wave_sum_d(gz);
  if (lane == 0) {
    const int32_t self = sidx[k];
    const double f = 4.0 * (double)lambda;
    if (gr && gsum != 0.0) atomicAdd(gr + self, (float)(f * gsum));
    if (gp && (gx != 0.0 || gy != 0.0 || gz != 0.0)) {
      atomicAdd(gp + 3 * (int64_t)self, (float)(f * gx));
      atomicAdd(gp + 3 * (int64_t)self + 1, (float)(f * gy));
      atomicAdd(gp + 3 * (int64_t)self + 2, (float)(f * gz));
    }
    if (loss && lsum != 0.0) atomicAdd(loss, (double)lambda * lsum);
  }
}

// Cells that the previous build found empty and whose witness planes still
// leave nothing of them: a lane per cell.  With the four planes (m, h) in the
// cell's frame, weights l >= 0 on the last three with m_0 + sum l m = 0 and
// h_0 + sum l h < 0 prove that no x has m.x <= h for all four, so the power
// cell is empty whatever the other sites are.  The weights are rounded, and
// where the normals are nearly coplanar little of them is left (sites moved
// into one plane: det is what a fused multiply-add leaves of zero), so the
// proof is made for the weights as they are: with e = m_0 + sum l m, every x of
// the cell has e.x <= h_0 + sum l h, and within the domain box e.x is at least
// -(|e_x| X + |e_y| Y + |e_z| Z).  Below that, less the rounding of e and of the
// offsets h and a margin, nothing is left whatever the l are; a cell that misses
// it is clipped like any other.  keep[k] (sorted position) says which cells are left; for
// the others the outputs of an empty cell are written.
__global__ void __launch_bounds__(256) k_witness(const float4* __restrict__ sp, const int32_t* __restrict__ sidx,
                                                 const int32_t* __restrict__ spos, int64_t n, float3 bmin, float3 bmax,
                                                 const int32_t* __restrict__ wit, int32_t* __restrict__ wit_out,
                                                 int32_t* __restrict__ counts, int32_t* __restrict__ nrast,
                                                 float* __restrict__ cull, float4* __restrict__ ball,
                                                 int32_t* __restrict__ flags, uint32_t* __restrict__ keep) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int32_t self = sidx[k];
  const int4* wr = (const int4*)(wit + (int64_t)self * WIT);
  const int4 w0 = wr[0];
  bool gone = false, here = false;
  if (w0.x != -1) {
    const float4 me = sp[k];
    const double px = me.x, py = me.y, pz = me.z, wi = me.w;
    bool ok = wi > -INFINITY;
    // offset h of plane v; H: the magnitudes it is formed from
    auto plane = [&](int v, double& mx, double& my, double& mz, double& H) -> double {
      mx = my = mz = H = 0.0;
      if (v >= 0 && v < n && v != self) {
        const float4 q = sp[spos[v]];
        mx = (double)q.x - px;
        my = (double)q.y - py;
        mz = (double)q.z - pz;
        const double mm = mx * mx + my * my + mz * mz;
        H = mm + fabs(wi) + fabs((double)q.w);
        return 0.5 * (mm + wi - (double)q.w);
      }
      if (v <= -2 && v >= -7) {
        const int f = -2 - v, ax = f >> 1;
        const double sgn = (f & 1) ? -1.0 : 1.0;
        mx = ax == 0 ? sgn : 0.0;
        my = ax == 1 ? sgn : 0.0;
        mz = ax == 2 ? sgn : 0.0;
        const double lim = (f & 1) ? (ax == 0 ? bmin.x : ax == 1 ? bmin.y : bmin.z)
                                   : (ax == 0 ? bmax.x : ax == 1 ? bmax.y : bmax.z);
        const double at = ax == 0 ? px : ax == 1 ? py : pz;
        H = fabs(lim) + fabs(at);
        return sgn * (lim - at);
      }
      ok = false;
      return 0.0;
    };
    double x0, y0, z0, H0;
    const double h0 = plane(w0.x, x0, y0, z0, H0);
    if (ok && x0 == 0.0 && y0 == 0.0 && z0 == 0.0) {
      gone = here = h0 < 0.0 || (h0 == 0.0 && w0.x < self);   // coincident sites
    } else if (ok) {
      double xa, ya, za, xb, yb, zb, xc, yc, zc, Ha, Hb, Hc;
      const double ha = plane(w0.y, xa, ya, za, Ha), hb = plane(w0.z, xb, yb, zb, Hb), hc = plane(w0.w, xc, yc, zc, Hc);
      // (cross products of the pairs, determinant, weights by Cramer's rule)
      const double bcx = yb * zc - zb * yc, bcy = zb * xc - xb * zc, bcz = xb * yc - yb * xc;
      const double cax = yc * za - zc * ya, cay = zc * xa - xc * za, caz = xc * ya - yc * xa;
      const double abx = ya * zb - za * yb, aby = za * xb - xa * zb, abz = xa * yb - ya * xb;
      const double det = xa * bcx + ya * bcy + za * bcz;
      if (ok && det != 0.0) {
        const double inv = -1.0 / det;
        const double la = (x0 * bcx + y0 * bcy + z0 * bcz) * inv, lb = (x0 * cax + y0 * cay + z0 * caz) * inv,
                     lc = (x0 * abx + y0 * aby + z0 * abz) * inv;
        const double v = h0 + la * ha + lb * hb + lc * hc;
        const double scale = fabs(h0) + fabs(la * ha) + fabs(lb * hb) + fabs(lc * hc);
        // e, and the rounding of its sums and of the h (a few units of 1.1e-16)
        auto left = [&](double m0, double ma, double mb, double mc) {
          return fabs(m0 + la * ma + lb * mb + lc * mc) +
                 1e-15 * (fabs(m0) + fabs(la * ma) + fabs(lb * mb) + fabs(lc * mc));
        };
        const double reach = left(x0, xa, xb, xc) * fmax(fabs((double)bmin.x - px), fabs((double)bmax.x - px)) +
                             left(y0, ya, yb, yc) * fmax(fabs((double)bmin.y - py), fabs((double)bmax.y - py)) +
                             left(z0, za, zb, zc) * fmax(fabs((double)bmin.z - pz), fabs((double)bmax.z - pz));
        const double round_h = 1e-15 * (H0 + la * Ha + lb * Hb + lc * Hc);
        gone = la >= 0.0 && lb >= 0.0 && lc >= 0.0 && v < -(1e-8 * scale + reach + round_h);
      }
    }
  }
  keep[k] = gone ? 0u : 1u;
  if (gone) {
    int4* o = (int4*)(wit_out + (int64_t)self * WIT);
    o[0] = w0;
    o[1] = wr[1];
    counts[self] = 0;
    nrast[self] = 0;
    cull[self] = -1.0f;
    ball[self] = make_float4(0.0f, 0.0f, 0.0f, -1.0f);
    flags[self] = here ? FLAG_EMPTY_POWER | FLAG_SAME_PLACE : FLAG_EMPTY_POWER;
  }
}
static_assert(WIT == 8, "k_witness copies a cell's witnesses as two int4");

// The sites that are left, in Morton order, and where each one is.
__global__ void k_keep_sites(const float4* __restrict__ sp, const int32_t* __restrict__ sidx, int64_t n,
                             const uint32_t* __restrict__ keep, const uint32_t* __restrict__ pos,
                             float4* __restrict__ osp, int32_t* __restrict__ osidx, int32_t* __restrict__ ospos) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n || !keep[k]) return;
  const uint32_t q = pos[k];
  osp[q] = sp[k];
  osidx[q] = sidx[k];
  ospos[sidx[k]] = (int32_t)q;
}

__global__ void k_list_overflow(const int32_t* __restrict__ flags, const int32_t* __restrict__ spos, int64_t n,
                                int32_t* __restrict__ klist, unsigned int* __restrict__ nlist) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && (flags[i] & FLAG_OVERFLOW)) klist[atomicAdd(nlist, 1u)] = spos[i];
}

__global__ void k_inverse(const int32_t* __restrict__ sidx, int64_t n, int32_t* __restrict__ spos) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) spos[sidx[k]] = (int32_t)k;
}

// The cell that owns the place of site v: v itself, or, where v is empty because
// of a site at the same place (its witness), that one in turn.
__device__ inline int place_owner(int v, const int32_t* __restrict__ flags, const int32_t* __restrict__ wit) {
  // (each is heavier than the one before, or as heavy and of lower index)
  while (flags[v] & FLAG_SAME_PLACE) v = wit[(int64_t)v * WIT];
  return v;
}

// Float planes of a face: the bisector with site v, face f of the domain box.
__device__ inline float4 site_plane(const float* __restrict__ p, const float* __restrict__ w, double px, double py,
                                    double pz, double wi, int v) {
  const double mx = (double)p[3 * (int64_t)v] - px, my = (double)p[3 * (int64_t)v + 1] - py,
               mz = (double)p[3 * (int64_t)v + 2] - pz;
  const double h = 0.5 * (mx * mx + my * my + mz * mz + wi - (double)w[v]);
  return make_float4((float)mx, (float)my, (float)mz, (float)h);
}
__device__ inline float4 box_plane(float3 bmin, float3 bmax, double px, double py, double pz, int f) {
  const int ax = f >> 1;
  const bool low = f & 1;
  const float sgn = low ? -1.0f : 1.0f;
  const double at = ax == 0 ? px : ax == 1 ? py : pz;
  const double lim = low ? at - (ax == 0 ? (double)bmin.x : ax == 1 ? (double)bmin.y : (double)bmin.z)
                         : (ax == 0 ? (double)bmax.x : ax == 1 ? (double)bmax.y : (double)bmax.z) - at;
  return make_float4(ax == 0 ? sgn : 0.0f, ax == 1 ? sgn : 0.0f, ax == 2 ? sgn : 0.0f, (float)lim);
}

// Final adjacency: sixteen lanes per cell copy its faces and vertex triples
// (tri: two words per face, -1 first where the build kept no triples) and form
// the planes.  Two sites at one place give a cell the same plane twice, and the
// clip keeps the one it met first: where there are such sites (TIES) a face is
// given to the place's owner, and the faces of such a cell are put in order again
// (without triples).  (To look at every face's neighbour for it took 0.07 of 0.22
// ms at 1,048,576 cells.)
template <bool TIES>
__global__ void __launch_bounds__(256) k_fill(const float* __restrict__ p, const float* __restrict__ w, int64_t n,
                                              const int32_t* __restrict__ faces_tmp,
                                              const int32_t* __restrict__ faces_big,
                                              const int32_t* __restrict__ bigslot, const uint32_t* __restrict__ row,
                                              const int32_t* __restrict__ counts, const int32_t* __restrict__ nrast,
                                              const int32_t* __restrict__ flags, const int32_t* __restrict__ wit,
                                              float3 bmin, float3 bmax, int32_t* __restrict__ col,
                                              float4* __restrict__ plane, int32_t* __restrict__ tri) {
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;
  const int l = threadIdx.x & 15;
  if (i >= n) return;
  const int c = counts[i];
  if (c <= 0) return;
  const double px = p[3 * i], py = p[3 * i + 1], pz = p[3 * i + 2], wi = w[i];
  const uint32_t off = row[i];
  const int b = bigslot[i];
  const int32_t* src = b >= 0 ? faces_big + (int64_t)b * PM_BIG : faces_tmp + i * FACE_CAP;
  const int room = b >= 0 ? PM_BIG : FACE_CAP;
  auto put = [&](int at, int v) {
    col[off + at] = v;
    plane[off + at] = v >= 0 ? site_plane(p, w, px, py, pz, wi, v) : box_plane(bmin, bmax, px, py, pz, -1 - v);
  };
  bool given = false;
  for (int f = l; f < c; f += 16) {
    const int v = src[f];
    if constexpr (TIES) given = given || (v >= 0 && (flags[v] & FLAG_SAME_PLACE));
    put(f, v);
  }
  const bool any = TIES && ((__ballot(given) >> (threadIdx.x & 48)) & 0xFFFFu);
  if (any) {
    // the place of a face within its category: raster faces, other cells', the box's
    const int nr = nrast[i];
    for (int f = l; f < c; f += 16) {
      if (src[f] < 0) continue;
      const int v = place_owner(src[f], flags, wit);
      const int g0 = f < nr ? 0 : nr, g1 = f < nr ? nr : c;
      int at = g0;
      for (int g = g0; g < g1; ++g) {
        if (src[g] < 0) continue;
        const int u = place_owner(src[g], flags, wit);
        at += (u < v || (u == v && g < f)) ? 1 : 0;
      }
      put(at, v);
    }
  }
  int32_t* to = tri + 2 * (int64_t)off;
  if (c >= 4 && 3 * c - 4 <= room && !any) {
    for (int t = l; t < 2 * c - 4; t += 16) to[t] = src[c + t];
  } else if (l == 0) {
    to[0] = -1;
  }
}

__device__ inline float softplus_f(float x) { return x > 20.0f ? x : log1pf(expf(x)); }

// Packed records; a cell of zero density (e.g. an empty Steiner cell, whose
// logit is -inf) is never binned for the raster: it cannot contribute.
__global__ void k_prep(const float* __restrict__ p, const float* __restrict__ r, const float* __restrict__ nrm,
                       const float* __restrict__ lam, float sigma_scale, int64_t n, float4* __restrict__ geo,
                       float4* __restrict__ onrm, float* __restrict__ cull, float4* __restrict__ ball) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  geo[i] = make_float4(p[3 * i], p[3 * i + 1], p[3 * i + 2], r[i]);
  const float nx = nrm[3 * i], ny = nrm[3 * i + 1], nz = nrm[3 * i + 2];
  const float inv = 1.0f / sqrtf(nx * nx + ny * ny + nz * nz);
  const float sigma = sigma_scale * softplus_f(lam[i]);
  onrm[i] = make_float4(nx * inv, ny * inv, nz * inv, sigma);
  if (!(sigma > 0.0f)) {
    cull[i] = -1.0f;
    ball[i].w = -1.0f;
  }
}

// out: [hidden, overflow, over-vertices, over-planes, over-work, over-stack, same place]
__global__ void k_count_flags(const int32_t* __restrict__ flags, const float* __restrict__ cull, int64_t n,
                              unsigned long long* __restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int f = i < n ? flags[i] : 0;
  const bool b[7] = {i < n && cull[i] < 0.0f,        (f & FLAG_OVERFLOW) != 0,  (f & FLAG_OVER_VERTS) != 0,
                     (f & FLAG_OVER_PLANES) != 0,    (f & FLAG_OVER_WORK) != 0, (f & FLAG_OVER_STACK) != 0,
                     (f & FLAG_SAME_PLACE) != 0};
#pragma unroll
  for (int q = 0; q < 7; ++q) {
    const uint64_t m = __ballot(b[q]);
    if ((threadIdx.x & 63) == 0 && m) atomicAdd(&out[q], (unsigned long long)__popcll(m));
  }
}

template <typename T>
struct DevBuf {
  T* p = nullptr;
  hipStream_t s;
  explicit DevBuf(hipStream_t st) : s(st) {}
  ~DevBuf() { if (p) pf::pool_free(p, s); }
  hipError_t alloc(size_t count) { return pf::pool_alloc((void**)&p, sizeof(T) * (count ? count : 1), s); }
  void reset() {
    if (p) pf::pool_free(p, s);
    p = nullptr;
  }
};

// Zero-density cells that overflowed every build pass are dropped: their
// sorted-site weight becomes -inf, so a rebuild gives them an empty power
// cell and lets them cut no other cell.
__global__ void k_drop_void(const int32_t* __restrict__ flags, const int32_t* __restrict__ spos,
                            const float* __restrict__ lam, float sigma_scale, int64_t n, float4* __restrict__ sp,
                            unsigned int* __restrict__ ndrop) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n || !(flags[i] & FLAG_OVERFLOW)) return;
  if (sigma_scale * softplus_f(lam[i]) > 0.0f) return;
  sp[spos[i]].w = -INFINITY;
  atomicAdd(ndrop, 1u);
}

}  // namespace

pf_status connect_loss_impl(const Scene& sc, float lambda, const pf_grads& g, double* loss_dev, hipStream_t s) {
  if (!sc.t_sp) {
    set_error("pf_connect_loss: the scene has no site tree");
    return PF_ERR_INVALID;
  }
  DevBuf<unsigned int> ovf(s);
  PF_HIP_TRY(ovf.alloc(1));
  PF_HIP_TRY(hipMemsetAsync(ovf.p, 0, sizeof(unsigned int), s));
  {
    ProfScope ps("k_connect", s);
    k_connect<<<(unsigned)sc.n, 64, 0, s>>>(sc.t_sp, sc.t_srad, sc.t_sidx, sc.n, sc.t_lo, sc.t_hi, sc.t_lv, lambda,
                                            g.p, g.radius, loss_dev, ovf.p);
  }
  PF_HIP_TRY(hipGetLastError());
  unsigned int h = 0;
  PF_HIP_TRY(hipMemcpyAsync(&h, ovf.p, sizeof(h), hipMemcpyDeviceToHost, s));
  PF_HIP_TRY(hipStreamSynchronize(s));
  if (h) {
    set_error("pf_connect_loss: " + std::to_string(h) + " cells exceeded the traversal stack");
    return PF_ERR_OVERFLOW;
  }
  return PF_OK;
}

void free_scene(Scene* sc, hipStream_t s, bool async) {
  void* ptrs[] = {sc->geo,  sc->nrm,    sc->cull, sc->ball,   sc->ball_top, sc->flags, sc->row,  sc->nrast, sc->col,
                  sc->plane, sc->t_sp, sc->t_sidx, sc->t_srad, sc->t_lo, sc->t_hi, sc->wit, sc->tri};
  // synchronous: renders on any stream may still read the arrays
  if (!async) (void)hipDeviceSynchronize();
  for (void* q : ptrs)
    if (q) pf::pool_free(q, async ? s : nullptr);
  sc->geo = sc->nrm = nullptr;
  sc->cull = nullptr;
  sc->ball = nullptr;
  sc->ball_top = nullptr;
  sc->flags = sc->row = sc->nrast = sc->col = nullptr;
  sc->plane = nullptr;
  sc->t_sp = sc->t_lo = sc->t_hi = nullptr;
  sc->t_sidx = nullptr;
  sc->t_srad = nullptr;
  sc->wit = nullptr;
  sc->tri = nullptr;
}

pf_status build_scene_impl(const pf_params& prm, const pf_build_opts& opt, hipStream_t s, Scene* sc,
                           const Scene* prev) {
  const int64_t n = prm.n;
  // warm start from a previous build of the same cells
  const bool use_prev = prev && prev->n == n && prev->row && prev->col && prev->tri;
  const int32_t* warm_row = use_prev ? prev->row : nullptr;
  const int32_t* warm_col = use_prev ? prev->col : nullptr;
  const int32_t* warm_wit = use_prev ? prev->wit : nullptr;
  const int32_t* warm_tri = use_prev ? prev->tri : nullptr;
  sc->n = n;
  sc->prm = prm;

  // bounds of the spheres
  const int nbk = (int)std::min<int64_t>(1024, (n + 255) / 256);
  DevBuf<float> part(s);
  PF_HIP_TRY(part.alloc((size_t)nbk * 8));
  k_bounds<<<nbk, 256, 0, s>>>(prm.p, prm.power, prm.radius, n, part.p);
  PF_HIP_TRY(hipGetLastError());
  std::vector<float> hp((size_t)nbk * 8);
  PF_HIP_TRY(hipMemcpyAsync(hp.data(), part.p, sizeof(float) * hp.size(), hipMemcpyDeviceToHost, s));
  PF_HIP_TRY(hipStreamSynchronize(s));
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  float rmin = INFINITY;
  for (int b = 0; b < nbk; ++b) {
    for (int a = 0; a < 3; ++a) {
      lo[a] = std::min(lo[a], hp[b * 8 + a]);
      hi[a] = std::max(hi[a], hp[b * 8 + 3 + a]);
    }
    rmin = std::min(rmin, hp[b * 8 + 7]);
  }
  for (int a = 0; a < 3; ++a) {
    if (!std::isfinite(lo[a]) || !std::isfinite(hi[a])) {
      set_error("pf_build_scene: non-finite site or radius");
      return PF_ERR_INVALID;
    }
  }
  if (!(rmin > 0.0f)) {
    set_error("pf_build_scene: radii must be positive");
    return PF_ERR_INVALID;
  }
  const bool user_box = opt.box_min[0] <= opt.box_max[0];
  const float pad = opt.box_pad > 0.0f ? opt.box_pad : 0.01f;
  for (int a = 0; a < 3; ++a) {
    float l = lo[a], h = hi[a];
    if (user_box) {
      l = std::min(l, opt.box_min[a]);
      h = std::max(h, opt.box_max[a]);
    }
    const float ext = std::max(h - l, 1e-6f);
    sc->box_min[a] = l - pad * ext;
    sc->box_max[a] = h + pad * ext;
  }
  const float3 bmin = make_float3(sc->box_min[0], sc->box_min[1], sc->box_min[2]);
  const float3 bmax = make_float3(sc->box_max[0], sc->box_max[1], sc->box_max[2]);

  // Morton order of the sites
  DevBuf<uint32_t> keys(s), order(s);
  PF_HIP_TRY(keys.alloc(n));
  PF_HIP_TRY(order.alloc(n));
  const float3 inv = make_float3(1024.0f / (bmax.x - bmin.x), 1024.0f / (bmax.y - bmin.y),
                                 1024.0f / (bmax.z - bmin.z));
  const unsigned g256 = (unsigned)((n + 255) / 256);
  k_morton<<<g256, 256, 0, s>>>(prm.p, n, bmin, inv, keys.p, order.p);
  PF_HIP_TRY(hipGetLastError());
  PF_HIP_TRY(radix_sort_u32(keys.p, order.p, n, 30, s));
  // the sorted sites and the tree stay with the scene (sphere-overlap queries)
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->t_sp, sizeof(float4) * n, s));
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->t_sidx, sizeof(int32_t) * n, s));
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->t_srad, sizeof(float) * n, s));
  struct { float4* p; } sp{sc->t_sp};
  struct { int32_t* p; } sidx{sc->t_sidx};
  k_gather_sites<<<g256, 256, 0, s>>>(prm.p, prm.power, prm.radius, order.p, n, sp.p, sidx.p, sc->t_srad);
  PF_HIP_TRY(hipGetLastError());

  // implicit 64-ary tree over n sorted sites: per node the box of its sites,
  // their largest weight and largest sphere radius
  auto build_tree = [&](const float4* sites, const float* srad, int64_t count, Levels& lvl, float4*& lo_p,
                        float4*& hi_p) -> pf_status {
    lvl = Levels{};
    lvl.cnt[0] = count;
    long long total_nodes = 0;
    int L = 0;
    do {
      ++L;
      if (L > MAXLVL) {
        set_error("pf_build_scene: too many sites for the build tree");
        return PF_ERR_UNSUPPORTED;
      }
      lvl.cnt[L] = (lvl.cnt[L - 1] + 63) / 64;
      lvl.off[L] = total_nodes;
      total_nodes += lvl.cnt[L];
    } while (lvl.cnt[L] > 1);
    lvl.n = L;
    if (lo_p) pf::pool_free(lo_p, s);
    if (hi_p) pf::pool_free(hi_p, s);
    lo_p = hi_p = nullptr;
    PF_HIP_TRY(pf::pool_alloc((void**)&lo_p, sizeof(float4) * total_nodes, s));
    PF_HIP_TRY(pf::pool_alloc((void**)&hi_p, sizeof(float4) * total_nodes, s));
    for (int l = 1; l <= lvl.n; ++l) {
      const bool from_sites = l == 1;
      k_tree_level<<<(unsigned)lvl.cnt[l], 64, 0, s>>>(from_sites ? sites : nullptr, from_sites ? srad : nullptr,
                                                       from_sites ? nullptr : lo_p + lvl.off[l - 1],
                                                       from_sites ? nullptr : hi_p + lvl.off[l - 1],
                                                       lvl.cnt[l - 1], lo_p + lvl.off[l], hi_p + lvl.off[l]);
      PF_HIP_TRY(hipGetLastError());
    }
    return PF_OK;
  };
  {
    const pf_status st = build_tree(sp.p, sc->t_srad, n, sc->t_lv, sc->t_lo, sc->t_hi);
    if (st != PF_OK) return st;
  }

  // per-cell clipping
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->cull, sizeof(float) * n, s));
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->ball, sizeof(float4) * n, s));
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->ball_top, sizeof(float) * n, s));
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->flags, sizeof(int32_t) * n, s));
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->wit, sizeof(int32_t) * WIT * n, s));
  PF_HIP_TRY(hipMemsetAsync(sc->wit, 0xFF, sizeof(int32_t) * WIT * n, s));
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->nrast, sizeof(int32_t) * n, s));
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->row, sizeof(int32_t) * (n + 1), s));
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->geo, sizeof(float4) * n, s));
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->nrm, sizeof(float4) * n, s));
  DevBuf<int32_t> faces_tmp(s), counts(s), bigslot(s), spos(s), klist(s), faces_big(s);
  DevBuf<unsigned short> eo_big(s);
  DevBuf<unsigned int> nbig_d(s), ndrop_d(s);
  PF_HIP_TRY(faces_tmp.alloc((size_t)n * FACE_CAP));
  PF_HIP_TRY(counts.alloc(n + 1));
  PF_HIP_TRY(bigslot.alloc(n));
  PF_HIP_TRY(spos.alloc(n));
  PF_HIP_TRY(klist.alloc(n));
  PF_HIP_TRY(nbig_d.alloc(1));
  PF_HIP_TRY(ndrop_d.alloc(1));
  k_inverse<<<g256, 256, 0, s>>>(sidx.p, n, spos.p);
  PF_HIP_TRY(hipGetLastError());
  auto list_overflow = [&](const int32_t* pos, unsigned int& count) -> pf_status {
    PF_HIP_TRY(hipMemsetAsync(nbig_d.p, 0, sizeof(unsigned int), s));
    k_list_overflow<<<g256, 256, 0, s>>>(sc->flags, pos, n, klist.p, nbig_d.p);
    PF_HIP_TRY(hipGetLastError());
    PF_HIP_TRY(hipMemcpyAsync(&count, nbig_d.p, sizeof(count), hipMemcpyDeviceToHost, s));
    PF_HIP_TRY(hipStreamSynchronize(s));
    return PF_OK;
  };
  // The sites and the tree that the cells are clipped against: all of them,
  // or, after a previous build, those left once the cells that k_witness shows
  // to be still empty are out.  An empty power cell cuts no other cell (at
  // every point some other site is nearer in power), so the others come out
  // the same without it, and most sites can be empty: 70% at 1,048,576 cells,
  // where k_clip took 19.9 ms with them and 12.7 without (k_witness 0.12).
  // Below ELIM_MIN cells the extra launches and the count read back cost more
  // than they save: pf_update_scene after moves of 1e-4 takes, with and without,
  // 0.92 and 0.84 ms at 16,384 cells uniform in a cube (1.06 and 0.99 in the
  // mixture of surfaces), 1.05 and 1.00 (1.23 and 1.25) at 24,000, 1.13 and 1.13
  // (1.95 and 2.13) at 32,768, 1.34 and 1.54 (2.40 and 2.97) at 65,536.
  // (Without a previous build, clipping each cell against its
  // own leaf first finds too few of them: 7.1 ms to shorten 14.6 by 1.8 at
  // 300,000 cells.)
  struct Part {
    const float4* sp;
    const int32_t* sidx;
    const int32_t* spos;
    int64_t n;
    Levels lv;
    const float4 *lo, *hi;
  };
  const Part whole{sc->t_sp, sc->t_sidx, spos.p, n, sc->t_lv, sc->t_lo, sc->t_hi};
  Part used = whole;
  DevBuf<uint32_t> keep(s), keep_pos(s), n_keep(s);
  DevBuf<float4> k_sp(s), k_lo(s), k_hi(s);
  DevBuf<int32_t> k_sidx(s), k_spos(s);
  if (warm_wit && n >= ELIM_MIN) {
    PF_HIP_TRY(keep.alloc(n));
    PF_HIP_TRY(keep_pos.alloc(n));
    PF_HIP_TRY(n_keep.alloc(1));
    {
      ProfScope ps("k_witness", s);
      k_witness<<<g256, 256, 0, s>>>(sp.p, sidx.p, spos.p, n, bmin, bmax, warm_wit, sc->wit, counts.p, sc->nrast,
                                     sc->cull, sc->ball, sc->flags, keep.p);
    }
    PF_HIP_TRY(hipGetLastError());
    PF_HIP_TRY(exclusive_scan_u32(keep.p, keep_pos.p, n, n_keep.p, s));
    uint32_t left = 0;
    PF_HIP_TRY(hipMemcpyAsync(&left, n_keep.p, sizeof(left), hipMemcpyDeviceToHost, s));
    PF_HIP_TRY(hipStreamSynchronize(s));
    used.n = left;
    if (left) {
      PF_HIP_TRY(k_sp.alloc(left));
      PF_HIP_TRY(k_sidx.alloc(left));
      PF_HIP_TRY(k_spos.alloc(n));
      k_keep_sites<<<g256, 256, 0, s>>>(sp.p, sidx.p, n, keep.p, keep_pos.p, k_sp.p, k_sidx.p, k_spos.p);
      PF_HIP_TRY(hipGetLastError());
      const pf_status st = build_tree(k_sp.p, nullptr, left, used.lv, k_lo.p, k_hi.p);
      if (st != PF_OK) return st;
      used.sp = k_sp.p;
      used.sidx = k_sidx.p;
      used.spos = k_spos.p;
      used.lo = k_lo.p;
      used.hi = k_hi.p;
    }
  }
  // all passes; repeated (at most 3 more times) while zero-density cells
  // overflow and are dropped (then with every site: a cell may have been
  // shown empty by one that is dropped)
  sc->n_dropped = 0;
  for (int attempt = 0;; ++attempt) {
  PF_HIP_TRY(hipMemsetAsync(bigslot.p, 0xFF, sizeof(int32_t) * n, s));
  if (used.n) {
    ProfScope ps_clip("k_clip", s);
    k_clip<2, FACE_CAP, 0><<<(unsigned)used.n, 64, 0, s>>>(used.sp, used.sidx, used.n, used.lo, used.hi, used.lv, bmin,
                                                           bmax, prm.radius, nullptr, nullptr, faces_tmp.p, nullptr,
                                                           counts.p, sc->nrast, sc->cull, sc->flags, warm_row,
                                                           warm_col, warm_tri, warm_wit, sp.p, spos.p, n, sc->wit,
                                                           prm.normal, prm.tex, sc->ball, sc->ball_top);
  }
  PF_HIP_TRY(hipGetLastError());
  // second pass (twice the capacity, edge table still in LDS) for the cells
  // that overflowed, third pass (4x, edge table in HBM) for what is left
  unsigned int nbig = 0;
  {
    const pf_status st = list_overflow(used.spos, nbig);
    if (st != PF_OK) return st;
  }
  sc->n_big = nbig;
  faces_big.reset();
  eo_big.reset();
  if (nbig) {
    PF_HIP_TRY(faces_big.alloc((size_t)nbig * PM_BIG));
    {
      ProfScope ps_big("k_clip_mid", s);
      k_clip<SPL_MID, PM_MID, 1><<<nbig, 64, 0, s>>>(used.sp, used.sidx, used.n, used.lo, used.hi, used.lv, bmin, bmax,
                                                    prm.radius, klist.p, nullptr, faces_big.p, bigslot.p, counts.p,
                                                    sc->nrast, sc->cull, sc->flags, warm_row, warm_col, warm_tri, warm_wit,
                                                    sp.p, spos.p, n, sc->wit, prm.normal, prm.tex, sc->ball, sc->ball_top);
    }
    PF_HIP_TRY(hipGetLastError());
    unsigned int nbig3 = 0;
    const pf_status st = list_overflow(used.spos, nbig3);
    if (st != PF_OK) return st;
    if (nbig3) {
      PF_HIP_TRY(eo_big.alloc((size_t)nbig3 * PM_BIG * PM_BIG));
      ProfScope ps_big("k_clip_big", s);
      k_clip<SPL_BIG, PM_BIG, 2><<<nbig3, 64, 0, s>>>(used.sp, used.sidx, used.n, used.lo, used.hi, used.lv, bmin, bmax,
                                                     prm.radius, klist.p, eo_big.p, faces_big.p, bigslot.p, counts.p,
                                                     sc->nrast, sc->cull, sc->flags, nullptr, nullptr, nullptr, nullptr, nullptr,
                                                     nullptr, 0, sc->wit, prm.normal, prm.tex, sc->ball, sc->ball_top);
      PF_HIP_TRY(hipGetLastError());
    }
  }
  if (attempt == 3) break;
  unsigned int ndrop = 0;
  PF_HIP_TRY(hipMemsetAsync(ndrop_d.p, 0, sizeof(unsigned int), s));
  k_drop_void<<<g256, 256, 0, s>>>(sc->flags, spos.p, prm.occ_logit, prm.sigma_scale, n, sp.p, ndrop_d.p);
  PF_HIP_TRY(hipGetLastError());
  PF_HIP_TRY(hipMemcpyAsync(&ndrop, ndrop_d.p, sizeof(ndrop), hipMemcpyDeviceToHost, s));
  PF_HIP_TRY(hipStreamSynchronize(s));
  if (ndrop == 0) break;
  sc->n_dropped += ndrop;
  used = whole;
  }

  k_prep<<<g256, 256, 0, s>>>(prm.p, prm.radius, prm.normal, prm.occ_logit, prm.sigma_scale, n, sc->geo,
                              sc->nrm, sc->cull, sc->ball);
  PF_HIP_TRY(hipGetLastError());
  DevBuf<unsigned long long> cnt(s);
  PF_HIP_TRY(cnt.alloc(7));
  PF_HIP_TRY(hipMemsetAsync(cnt.p, 0, 7 * sizeof(unsigned long long), s));
  k_count_flags<<<g256, 256, 0, s>>>(sc->flags, sc->cull, n, cnt.p);
  PF_HIP_TRY(hipGetLastError());
  PF_HIP_TRY(hipMemsetAsync(counts.p + n, 0, sizeof(int32_t), s));
  PF_HIP_TRY(exclusive_scan_u32((const uint32_t*)counts.p, (uint32_t*)sc->row, n + 1, nullptr, s));
  uint32_t total = 0;
  unsigned long long hc[7] = {0, 0, 0, 0, 0, 0, 0};
  PF_HIP_TRY(hipMemcpyAsync(&total, sc->row + n, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
  PF_HIP_TRY(hipMemcpyAsync(hc, cnt.p, sizeof(hc), hipMemcpyDeviceToHost, s));
  PF_HIP_TRY(hipStreamSynchronize(s));
  sc->n_faces = total;
  sc->n_hidden = (int64_t)hc[0];
  sc->n_overflow = (int64_t)hc[1];
  if (sc->n_overflow) {
    set_error("pf_build_scene: " + std::to_string(sc->n_overflow) + " of " + std::to_string(n) +
              " cells exceeded a per-cell capacity (vertices " + std::to_string(hc[2]) + ", planes " +
              std::to_string(hc[3]) + ", work " + std::to_string(hc[4]) + ", stack " + std::to_string(hc[5]) +
              "; " + std::to_string(sc->n_big) + " cells took the high-degree pass)");
    return PF_ERR_OVERFLOW;
  }
  // capacity in steps of 2^18 faces: rebuilds of similar size reuse the pool's blocks
  const size_t fcap = ((size_t)total + (1u << 18)) & ~(size_t)((1u << 18) - 1);
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->col, sizeof(int32_t) * fcap, s));
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->plane, sizeof(float4) * fcap, s));
  PF_HIP_TRY(pf::pool_alloc((void**)&sc->tri, sizeof(int32_t) * 2 * fcap, s));
  auto fill = hc[6] ? k_fill<true> : k_fill<false>;
  fill<<<(unsigned)((n + 15) / 16), 256, 0, s>>>(prm.p, prm.power, n, faces_tmp.p, faces_big.p, bigslot.p,
                                                  (const uint32_t*)sc->row, counts.p, sc->nrast, sc->flags, sc->wit,
                                                  bmin, bmax, sc->col, sc->plane, sc->tri);
  PF_HIP_TRY(hipGetLastError());
  PF_HIP_TRY(hipStreamSynchronize(s));
  return PF_OK;
}

}  // namespace pf
