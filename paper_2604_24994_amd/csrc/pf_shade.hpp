// Per-(ray, cell) device math shared by the rasteriser, the ray walk and the
// backward pass, so that the two renderers evaluate every contribution's
// geometry with the same arithmetic.  One product differs: the slope of the last
// raster face where their number is odd (piece_geometry), by which opacities
// differ in the last bits at 0.1% of the pixels.  Colours agree up to rounding: a
// wave that shades one cell, always in the rasteriser and mostly in the walk, takes
// the lobe softmaxes without the max shift (radiance_wave), a ray by itself with it
// (radiance_lane).
//
// Numerics: the ray is generated in float64 and, per cell, re-expressed in
// the cell's local frame in float64: q = closest-approach offset from p_i,
// s = t - t_closest, so that x(t) - p_i = q + s d.  All lengths below are
// then small numbers near the cell, computed in float32 (IEEE division and
// square root are replaced by the hardware reciprocal and square root,
// <= 1 ulp).  The sphere discriminant is
// formed in float64 (it cancels near tangency).
#pragma once

#include <hip/hip_runtime.h>

#include "pf_internal.hpp"

namespace pf {

struct RayD {
  double ox, oy, oz;   // camera centre
  double dx, dy, dz;   // unit direction
  float fx, fy, fz;    // direction rounded to float
  bool valid;
};

// Equidistant fisheye: camera-frame direction at polar angle th of the
// pixel offset (ex, ey), rho = |(ex, ey)|.  Out of line, so that the float64
// sine and cosine constants stay in this function instead of occupying
// registers across the loops of the kernels that generate rays.
__device__ __attribute__((noinline)) double3 fisheye_dir(double ex, double ey, double rho, double th) {
  const double st = sin(th);
  double3 d;
  d.x = rho > 0.0 ? st * ex / rho : 0.0;
  d.y = rho > 0.0 ? st * ey / rho : 0.0;
  d.z = cos(th);
  return d;
}

// Ray through pixel-centre coordinates (u, v).
__device__ inline RayD make_ray(const pf_camera& c, double u, double v) {
  RayD r;
  double dcx, dcy, dcz;
  r.valid = true;
  if (c.model == 0) {
    dcx = (u - (double)c.cx) / (double)c.fx;
    dcy = (v - (double)c.cy) / (double)c.fy;
    dcz = 1.0;
  } else {
    const double ex = u - (double)c.cx, ey = v - (double)c.cy;
    const double rho = sqrt(ex * ex + ey * ey);
    const double th = rho / (double)c.f_fish;
    r.valid = th <= (double)c.theta_max;
    const double3 d = fisheye_dir(ex, ey, rho, th);
    dcx = d.x;
    dcy = d.y;
    dcz = d.z;
  }
  const float* m = c.c2w;
  double wx = (double)m[0] * dcx + (double)m[1] * dcy + (double)m[2] * dcz;
  double wy = (double)m[4] * dcx + (double)m[5] * dcy + (double)m[6] * dcz;
  double wz = (double)m[8] * dcx + (double)m[9] * dcy + (double)m[10] * dcz;
  // 1/|w|: hardware reciprocal square root refined by two Newton steps
  const double w2 = wx * wx + wy * wy + wz * wz;
  double inv = __builtin_amdgcn_rsq(w2);
  inv = inv * fma(-0.5 * w2 * inv, inv, 1.5);
  inv = inv * fma(-0.5 * w2 * inv, inv, 1.5);
  r.dx = wx * inv;
  r.dy = wy * inv;
  r.dz = wz * inv;
  r.ox = m[3];
  r.oy = m[7];
  r.oz = m[11];
  r.fx = (float)r.dx;
  r.fy = (float)r.dy;
  r.fz = (float)r.dz;
  return r;
}

__device__ inline float frcp(float x) { return __builtin_amdgcn_rcpf(x); }
// Hardware square root (<= 1 ulp; the correctly rounded expansion costs a
// dozen instructions).
__device__ inline float fsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// Read-only data whose address is the same in every lane of the wave, read
// through the scalar cache: a pointer to the constant address space says so
// whatever else the kernel writes (for an ordinary pointer the compiler has to
// prove that no earlier store or atomic touches the data, and reads it into
// vector registers, once per lane, when it cannot).  The data must not be
// written while the kernel runs.
typedef float vec4f __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) float* ufloat_p;
typedef const __attribute__((address_space(4))) vec4f* uvec4_p;
__device__ inline ufloat_p uniform_ptr(const float* p) { return (ufloat_p)p; }
__device__ inline uvec4_p uniform_ptr(const float4* p) { return (uvec4_p)p; }
__device__ inline float4 load4(uvec4_p p) {
  const vec4f v = *p;
  return make_float4(v.x, v.y, v.z, v.w);
}

constexpr float LOG2E_F = 1.4426950408889634f;

// exp(x - shift) as one fused multiply-add and the hardware exp2, with
// shift_l2 = shift * log2(e) formed once per softmax.
__device__ inline float exp_shifted(float x, float shift_l2) {
  return __builtin_amdgcn_exp2f(fmaf(x, LOG2E_F, -shift_l2));
}

// Local frame of the ray at a cell: q (float), beta = s at t = 0, and the
// squared closest-approach distance in float64.
struct Local {
  float qx, qy, qz;
  float beta;
  double qq;
  double b;          // float64 beta
  double dqx, dqy, dqz;  // float64 q
};

__device__ inline Local make_local(const RayD& R, float px, float py, float pz) {
  Local L;
  const double ocx = R.ox - (double)px, ocy = R.oy - (double)py, ocz = R.oz - (double)pz;
  const double b = ocx * R.dx + ocy * R.dy + ocz * R.dz;
  const double qx = ocx - b * R.dx, qy = ocy - b * R.dy, qz = ocz - b * R.dz;
  L.qx = (float)qx;
  L.qy = (float)qy;
  L.qz = (float)qz;
  L.dqx = qx;
  L.dqy = qy;
  L.dqz = qz;
  L.qq = qx * qx + qy * qy + qz * qz;
  L.b = b;
  L.beta = (float)b;
  return L;
}

// h - q.m of face plane (m, h) = pl as one fused chain from h, given -q: the
// ray x = p_i + q + s d meets the plane at s = (h - q.m) / (d.m).
__device__ inline float face_offset(const float4 pl, float nqx, float nqy, float nqz) {
  return fmaf(nqz, pl.z, fmaf(nqy, pl.y, fmaf(nqx, pl.x, pl.w)));
}

// Duff et al., "Building an Orthonormal Basis, Revisited" (JCGT 2017).
__device__ inline void onb(float nx, float ny, float nz, float& t1x, float& t1y, float& t1z, float& t2x,
                           float& t2y, float& t2z) {
  const float sign = copysignf(1.0f, nz);
  const float a = -frcp(sign + nz);   // |sign + nz| >= 1
  const float b = nx * ny * a;
  t1x = 1.0f + sign * nx * nx * a;
  t1y = sign * b;
  t1z = -sign * nx;
  t2x = b;
  t2y = sign + ny * ny * a;
  t2z = -ny;
}

// Softmax of up to 8 base-2 logits z into p (normalised in place by the
// caller): p_k = 2^z_k, returned sum.  The logits are exponentiated
// unshifted (2^z is exact in float range), and only when the sum leaves
// [2^-100, 2^100] (a logit near the range's ends) are they shifted by their
// largest, as a softmax usually is; *shift receives the shift (0 or that
// largest logit).  Saves the max and the subtraction on every call.
template <int N>
__device__ inline float softmax2_sum(const float (&z)[N], float (&p)[N], float* shift) {
  float sum = 0.0f;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    p[k] = __builtin_amdgcn_exp2f(z[k]);
    sum += p[k];
  }
  float sh = 0.0f;
  if (!(sum >= 0x1p-100f && sum <= 0x1p100f)) {
    sh = z[0];
#pragma unroll
    for (int k = 1; k < N; ++k) sh = fmaxf(sh, z[k]);
    sum = 0.0f;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      p[k] = __builtin_amdgcn_exp2f(z[k] - sh);
      sum += p[k];
    }
  }
  *shift = sh;
  return sum;
}

// a b + c d with one rounding less (written out where two kernels have to
// agree to the last bit: the compiler may fuse either product).
__device__ inline float dot2(float a, float b, float c, float d) { return fmaf(a, b, c * d); }

// a.b for the geometry of a piece, fused in a fixed order: a piece's ends, and
// with them which rays graze it, must not depend on the kernel around it.
__device__ inline float dot3(float ax, float ay, float az, float bx, float by, float bz) {
  return fmaf(az, bz, fmaf(ax, bx, ay * by));
}

// Soft-Voronoi weights over the K detail sites at face point u (Sec. 3.4,
// Eq. svdisp / Eq. svrad).  The logits are shifted by tau*|u| and written as
//   |u - s_k| - |u| = (|s_k|^2 - 2 u.s_k) / (|u - s_k| + |u|),
// which keeps them accurate when u is far from the sites (grazing rays).
// STRIDE: floats from one site's (s, d) to the next.
template <int STRIDE = TEXW, typename FP>
__device__ inline void sv_weights(FP tx, float ux, float uy, float tau, float* w) {
  const float un = fsqrt(dot2(ux, ux, uy, uy));
  float mx = -INFINITY;
#pragma unroll
  for (int k = 0; k < KD; ++k) {
    const float sx = tx[k * STRIDE + 0], sy = tx[k * STRIDE + 1];
    const float ex = ux - sx, ey = uy - sy;
    const float dist = fsqrt(dot2(ex, ex, ey, ey));
    const float num = fmaf(-2.0f, dot2(ux, sx, uy, sy), dot2(sx, sx, sy, sy));
    const float den = dist + un;
    const float q = num * frcp(den);   // (unconditional, so that the choice is no branch)
    const float e = den > 0.0f ? q : 0.0f;
    w[k] = -tau * e;
    mx = fmaxf(mx, w[k]);
  }
  float sum = 0.0f;
  const float mxl = mx * LOG2E_F;
#pragma unroll
  for (int k = 0; k < KD; ++k) {
    w[k] = exp_shifted(w[k], mxl);
    sum += w[k];
  }
  const float inv = frcp(sum);
#pragma unroll
  for (int k = 0; k < KD; ++k) w[k] *= inv;
}

// Sums of detail site t's M Spherical-Voronoi lobes for direction g = d log2(e):
// *sum = sum_m 2^(a_m.g - shift), (sr, sg, sb) = sum_m 2^(a_m.g - shift) c_m;
// returns the base-2 shift (softmax2_sum).
__device__ inline float sv_lobes(const float* __restrict__ t, float gx, float gy, float gz, float& sum, float& sr,
                                 float& sg, float& sb) {
  float lg[MA], e[MA], sh;
#pragma unroll
  for (int m = 0; m < MA; ++m) lg[m] = t[3 + 3 * m] * gx + t[4 + 3 * m] * gy + t[5 + 3 * m] * gz;
  sum = softmax2_sum(lg, e, &sh);
  sr = sg = sb = 0.0f;
#pragma unroll
  for (int m = 0; m < MA; ++m) {
    sr += e[m] * t[3 + 3 * MA + 3 * m];
    sg += e[m] * t[4 + 3 * MA + 3 * m];
    sb += e[m] * t[5 + 3 * MA + 3 * m];
  }
  return sh;
}

// Geometry of one (ray, cell) piece: bounded interval, dipole split and
// opacity.  faces/nfaces: the cell's raster faces.  Returns alpha (0 when
// the piece is empty) and the texture point u, plus what the backward needs.
struct Piece {
  float alpha;
  float ux, uy;       // texture point in the face frame
  float s0, s1;       // bounded interval (local s)
  float j0, j1;       // dense part
  int bind0, bind1;   // binding constraint of s0 / s1: -1 sphere, -2 camera, f >= 0 face index
  float den, sx, sbar, delta;
  float t1x, t1y, t1z, t2x, t2y, t2z;
};

// A ray's interval within a cell while the faces clip it.
struct Interval {
  float s0, s1;
  int b0, b1;
};

// Exit (a >= 0) and entry (a < 0) bounds of face f, met at s = offset / a, by
// selects rather than branches.  a = d.m + 0 is never -0, so a face parallel
// to the ray (a = +0) gives s = bb * (1/+0): -inf when the ray lies on its
// outer side (bb < 0), which empties the interval, +inf (or NaN for bb = 0)
// otherwise, which leaves it.  Once empty, an interval stays empty.
__device__ inline void clip_face(Interval& I, float a, float s, bool on, int f) {
  const bool exits = a >= 0.0f;
  const bool out = on && exits && s < I.s1;
  const bool in = on && !exits && s > I.s0;
  I.s1 = out ? s : I.s1;
  I.b1 = out ? f : I.b1;
  I.s0 = in ? s : I.s0;
  I.b0 = in ? f : I.b0;
}

// d.m + 0 of face plane (m, h) = pl.
__device__ inline float face_slope(const RayD& R, const float4 pl) {
  return fmaf(R.fz, pl.z, fmaf(R.fy, pl.y, R.fx * pl.x)) + 0.0f;
}

// The piece of an interval that the sphere and the faces have clipped.
// WAVE_CELL: every lane of the wave evaluates the same cell (the rasteriser):
// before the displacement weights, it tests whether the dense part is empty
// for every displacement the sites allow (for the walk's per-lane loads that
// test costs more than it saves).  Either way alpha is the same.
template <bool WAVE_CELL, typename FP>
__device__ inline Piece piece_dense(const RayD& R, const Local& L, Interval I, float4 nrm, FP tx, float tau) {
  Piece P;
  P.alpha = 0.0f;
  P.ux = P.uy = 0.0f;
  if (L.beta > I.s0) { I.s0 = L.beta; I.b0 = -2; }
  const float s0 = I.s0, s1 = I.s1, fx = R.fx, fy = R.fy, fz = R.fz;
  P.s0 = s0;
  P.s1 = s1;
  P.bind0 = I.b0;
  P.bind1 = I.b1;
  if (!(s0 < s1)) return P;

  // dipole face with displacement (Sec. 3.3, Sec. 3.4)
  const float nx = nrm.x, ny = nrm.y, nz = nrm.z;
  onb(nx, ny, nz, P.t1x, P.t1y, P.t1z, P.t2x, P.t2y, P.t2z);
  const float den = dot3(fx, fy, fz, nx, ny, nz);
  const float qn = dot3(L.qx, L.qy, L.qz, nx, ny, nz);
  const float qt1 = dot3(L.qx, L.qy, L.qz, P.t1x, P.t1y, P.t1z);
  const float qt2 = dot3(L.qx, L.qy, L.qz, P.t2x, P.t2y, P.t2z);
  const float dt1 = dot3(fx, fy, fz, P.t1x, P.t1y, P.t1z);
  const float dt2 = dot3(fx, fy, fz, P.t2x, P.t2y, P.t2z);
  P.den = den;
  float j0 = s0, j1 = s1;
  if (den != 0.0f) {
    const float idn = frcp(den);
    // The displacement is a convex combination of the sites' d_k, so the
    // displaced face lies between the faces moved by min d_k and max d_k.
    // When even the face moved by max d_k leaves [s0, s1] on the empty side
    // (beyond s1 going in, before s0 going out), the dense part is empty
    // whatever the weights: alpha = 0 without evaluating them.  The test
    // keeps a relative margin far above the rounding of the exact path, so
    // it only fires where that path gives an empty dense part too.
    if constexpr (WAVE_CELL) {
      float dmax = tx[2], dabs = fabsf(tx[2]);
#pragma unroll
      for (int k = 1; k < KD; ++k) {
        dmax = fmaxf(dmax, tx[k * TEXW + 2]);
        dabs = fmaxf(dabs, fabsf(tx[k * TEXW + 2]));
      }
      const float bound = (dmax + 1e-5f * dabs - qn) * idn;
      const float tol = 1e-4f * (fabsf(s0) + fabsf(s1) + fabsf(bound)) + 1e-30f;
      if (den > 0.0f ? bound + tol <= s0 : bound - tol >= s1) return P;
    }
    const float sbar = -qn * idn;
    float w[KD];
    sv_weights(tx, qt1 + sbar * dt1, qt2 + sbar * dt2, tau, w);
    float delta = 0.0f;
#pragma unroll
    for (int k = 0; k < KD; ++k) delta += w[k] * tx[k * TEXW + 2];
    const float sxx = (delta - qn) * idn;
    if (den > 0.0f) j1 = fminf(s1, sxx);
    else j0 = fmaxf(s0, sxx);
    P.ux = qt1 + sxx * dt1;
    P.uy = qt2 + sxx * dt2;
    P.sx = sxx;
    P.sbar = sbar;
    P.delta = delta;
  } else {
    const float sm = 0.5f * (s0 + s1);
    P.ux = qt1 + sm * dt1;
    P.uy = qt2 + sm * dt2;
    P.sx = 0.0f;
    P.sbar = 0.0f;
    P.delta = 0.0f;
    if (!(qn < 0.0f)) j1 = j0;
  }
  P.j0 = j0;
  P.j1 = j1;
  const float ell = fmaxf(j1 - j0, 0.0f);
  P.alpha = 1.0f - __expf(-nrm.w * ell);
  return P;
}

// The rasteriser's piece: the cell's faces are read through the scalar cache,
// two per step from one wave-uniform address, and the wave leaves the face loop
// as soon as no lane's interval is left.
template <typename VP, typename FP>
__device__ inline Piece piece_geometry(const RayD& R, const Local& L, float r, VP faces, int nfaces, float4 nrm, FP tx,
                                       float tau) {
  const double D = (double)r * (double)r - L.qq;
  if (D <= 0.0) {
    Piece P;
    P.alpha = 0.0f;
    P.ux = P.uy = 0.0f;
    P.bind0 = P.bind1 = -1;
    P.s0 = 1.0f;
    P.s1 = 0.0f;
    return P;
  }
  const float sq = fsqrt((float)D);
  Interval I = {-sq, sq, -1, -1};
  const float nqx = -L.qx, nqy = -L.qy, nqz = -L.qz;
  auto clip = [&](const float4 pl, float a, int f) {
    clip_face(I, a, face_offset(pl, nqx, nqy, nqz) * frcp(a), true, f);
  };
  int f = 0;
  bool more = nfaces >= 2;
  float4 c0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), c1 = c0;
  if (more) {
    c0 = load4(faces);
    c1 = load4(faces + 1);
  }
  while (more) {
    const float4 p0 = c0, p1 = c1;
    const int fn = f + 2;
    if (fn + 2 <= nfaces) {   // the next pair is loaded while this one is tested
      const VP fp = faces + __builtin_amdgcn_readfirstlane(fn);
      c0 = load4(fp);
      c1 = load4(fp + 1);
    }
    clip(p0, face_slope(R, p0), f);
    clip(p1, face_slope(R, p1), f + 1);
    f = fn;
    more = f + 2 <= nfaces && __any(I.s0 < I.s1);
  }
  if (f + 1 == nfaces) {
    // (its slope rounded as the other products here.  With face_slope, raster and
    // walk have the same opacities bit for bit, but other rays graze such a face,
    // and the gradient of power moved by 2e-5 of its norm in one training step of
    // eight: too far for what it gives.)
    const float4 pl = load4(faces + __builtin_amdgcn_readfirstlane(f));
    clip(pl, dot3(R.fx, R.fy, R.fz, pl.x, pl.y, pl.z) + 0.0f, f);
  }
  return piece_dense<true>(R, L, I, nrm, tx, tau);
}

// A cell's Spherical-Voronoi axes and colours spread over the wave as the A
// operands of 4x4x1 FP32 MFMAs (sixteen blocks of four rows, lane 4 b + i
// holding row i of block b; every instruction broadcasts one block to all):
// lane l of ax[c] holds component c of axis km = l (site km / 8, axis km % 8),
// and lane l of col[v] component l % 4 of the colour of km = 16 v + l / 4, with
// a one in the place of the fourth component.  All 64 lanes must take part.
struct WaveTex {
  float ax[3], col[4];
};

__device__ inline WaveTex wave_tex(const float* __restrict__ tx) {
  const int lane = threadIdx.x & 63;
  WaveTex W;
  const float* a = tx + (lane >> 3) * TEXW + 3 + 3 * (lane & 7);
#pragma unroll
  for (int c = 0; c < 3; ++c) W.ax[c] = a[c];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int km = 16 * v + (lane >> 2), c = lane & 3;
    W.col[v] = c < 3 ? tx[(km >> 3) * TEXW + 3 + 3 * MA + 3 * (km & 7) + c] : 1.0f;
  }
  return W;
}

// Sums of site K's lobes for the lane's direction g = d log2(e), as
// (sum_m e_m c_m, sum_m e_m), e_m = 2^(a_m . g).  The B operands and the
// results have one pixel (record) per lane, as everywhere else, so both
// contractions, 8 x 3 and 4 x 8 per lane, run on the matrix cores with the
// same products and the same order of additions as multiply-adds in the lane.
template <int K>
__device__ inline vec4f wave_lobes(const WaveTex& W, float gx, float gy, float gz) {
  const vec4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
  vec4f l0 = __builtin_amdgcn_mfma_f32_4x4x1f32(W.ax[0], gx, zero, 4, 2 * K, 0);
  vec4f l1 = __builtin_amdgcn_mfma_f32_4x4x1f32(W.ax[0], gx, zero, 4, 2 * K + 1, 0);
  l0 = __builtin_amdgcn_mfma_f32_4x4x1f32(W.ax[1], gy, l0, 4, 2 * K, 0);
  l1 = __builtin_amdgcn_mfma_f32_4x4x1f32(W.ax[1], gy, l1, 4, 2 * K + 1, 0);
  l0 = __builtin_amdgcn_mfma_f32_4x4x1f32(W.ax[2], gz, l0, 4, 2 * K, 0);
  l1 = __builtin_amdgcn_mfma_f32_4x4x1f32(W.ax[2], gz, l1, 4, 2 * K + 1, 0);
  constexpr int B = 8 * (K & 1);   // block of the site's first colour
  const float c = W.col[K >> 1];
  vec4f s = zero;
  s = __builtin_amdgcn_mfma_f32_4x4x1f32(c, __builtin_amdgcn_exp2f(l0[0]), s, 4, B + 0, 0);
  s = __builtin_amdgcn_mfma_f32_4x4x1f32(c, __builtin_amdgcn_exp2f(l0[1]), s, 4, B + 1, 0);
  s = __builtin_amdgcn_mfma_f32_4x4x1f32(c, __builtin_amdgcn_exp2f(l0[2]), s, 4, B + 2, 0);
  s = __builtin_amdgcn_mfma_f32_4x4x1f32(c, __builtin_amdgcn_exp2f(l0[3]), s, 4, B + 3, 0);
  s = __builtin_amdgcn_mfma_f32_4x4x1f32(c, __builtin_amdgcn_exp2f(l1[0]), s, 4, B + 4, 0);
  s = __builtin_amdgcn_mfma_f32_4x4x1f32(c, __builtin_amdgcn_exp2f(l1[1]), s, 4, B + 5, 0);
  s = __builtin_amdgcn_mfma_f32_4x4x1f32(c, __builtin_amdgcn_exp2f(l1[2]), s, 4, B + 6, 0);
  s = __builtin_amdgcn_mfma_f32_4x4x1f32(c, __builtin_amdgcn_exp2f(l1[3]), s, 4, B + 7, 0);
  return s;
}
static_assert(KD == 8 && MA == 8, "wave_tex and wave_lobes: 64 site-axis pairs, two colour blocks of eight");

// Radiance at texture point u for direction d: base colour plus the
// soft-Voronoi blend of the detail sites' Spherical-Voronoi colours, for a wave
// that shades one cell (all lanes take part, those outside `on` get an
// unspecified colour).  The lobes are exponentiated in base 2 without the
// max shift; where a site's sum leaves [2^-100, 2^100], the colour is evaluated
// again with each site's logits shifted by their largest (as in
// softmax2_sum).  That rare pass runs over the sites in a loop that is not
// unrolled, so that its texture reads are its own.
template <typename FP>
__device__ inline void radiance_wave(const float* __restrict__ tex, FP tx, FP rgb, bool on, float ux, float uy, float fx,
                                     float fy, float fz, float tau, float& cr, float& cg, float& cb) {
  const WaveTex W = wave_tex(tex);
  float w[KD];
  sv_weights(tx, ux, uy, tau, w);
  const float gx = fx * LOG2E_F, gy = fy * LOG2E_F, gz = fz * LOG2E_F;
  cr = rgb[0];
  cg = rgb[1];
  cb = rgb[2];
  bool in_range = true;
  auto add = [&](const vec4f s, float wk) {
    in_range = in_range && s[3] >= 0x1p-100f && s[3] <= 0x1p100f;
    const float sc = wk * frcp(s[3]);
    cr += sc * s[0];
    cg += sc * s[1];
    cb += sc * s[2];
  };
  add(wave_lobes<0>(W, gx, gy, gz), w[0]);
  add(wave_lobes<1>(W, gx, gy, gz), w[1]);
  add(wave_lobes<2>(W, gx, gy, gz), w[2]);
  add(wave_lobes<3>(W, gx, gy, gz), w[3]);
  add(wave_lobes<4>(W, gx, gy, gz), w[4]);
  add(wave_lobes<5>(W, gx, gy, gz), w[5]);
  add(wave_lobes<6>(W, gx, gy, gz), w[6]);
  add(wave_lobes<7>(W, gx, gy, gz), w[7]);
  if (on && !in_range) {
    cr = rgb[0];
    cg = rgb[1];
    cb = rgb[2];
#pragma unroll 1
    for (int k = 0; k < KD; ++k) {
      float wk = w[0];
#pragma unroll
      for (int j = 1; j < KD; ++j) wk = (k == j) ? w[j] : wk;
      const FP t = tx + k * TEXW;
      float mx = -INFINITY;
      for (int m = 0; m < MA; ++m) mx = fmaxf(mx, dot3(t[3 + 3 * m], t[4 + 3 * m], t[5 + 3 * m], gx, gy, gz));
      float sum = 0.0f, sr = 0.0f, sg = 0.0f, sb = 0.0f;
      for (int m = 0; m < MA; ++m) {
        const float e =
            __builtin_amdgcn_exp2f(dot3(t[3 + 3 * m], t[4 + 3 * m], t[5 + 3 * m], gx, gy, gz) - mx);
        sum += e;
        sr += e * t[3 + 3 * MA + 3 * m];
        sg += e * t[4 + 3 * MA + 3 * m];
        sb += e * t[5 + 3 * MA + 3 * m];
      }
      const float sc = wk * frcp(sum);
      cr += sc * sr;
      cg += sc * sg;
      cb += sc * sb;
    }
  }
}

// The same with a cell per lane, the texture read per lane (the walk, where too
// few rays of the wave hold the cell at once): every softmax shifted by its
// largest logit, which keeps fewer values live than the unshifted form with its
// rare shifted pass.
__device__ inline void radiance_lane(const float* __restrict__ tx, const float* __restrict__ rgb, float ux, float uy,
                                     float fx, float fy, float fz, float tau, float& cr, float& cg, float& cb) {
  float w[KD];
  sv_weights(tx, ux, uy, tau, w);
  cr = rgb[0];
  cg = rgb[1];
  cb = rgb[2];
#pragma unroll
  for (int k = 0; k < KD; ++k) {
    const float* t = tx + k * TEXW;
    float lg[MA];
    float mx = -INFINITY;
#pragma unroll
    for (int m = 0; m < MA; ++m) {
      lg[m] = t[3 + 3 * m] * fx + t[4 + 3 * m] * fy + t[5 + 3 * m] * fz;
      mx = fmaxf(mx, lg[m]);
    }
    float sum = 0.0f, sr = 0.0f, sg = 0.0f, sb = 0.0f;
    const float mxl = mx * LOG2E_F;
#pragma unroll
    for (int m = 0; m < MA; ++m) {
      const float e = exp_shifted(lg[m], mxl);
      sum += e;
      sr += e * t[3 + 3 * MA + 3 * m];
      sg += e * t[4 + 3 * MA + 3 * m];
      sb += e * t[5 + 3 * MA + 3 * m];
    }
    const float sc = w[k] * frcp(sum);
    cr += sc * sr;
    cg += sc * sg;
    cb += sc * sb;
  }
}

}  // namespace pf
