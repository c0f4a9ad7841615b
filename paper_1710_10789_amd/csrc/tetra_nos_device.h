// Device-side building blocks of the number-of-states kernel (gfx950). Internal header.
//
// Integrated corner weights w_l of the five energy cases of Sec. II.C of Guterding & Jeschke
// (arXiv:1710.10789), in the notation of tetra_device.h, and the grid indices at which a
// tetrahedron-band's number of states changes.
#pragma once

#include "tetra_device.h"
#include "tetra_spline.h"

namespace tetra {

// Integrated corner weights w_l (Sec. II.C), for the number of states, in the local variables of
// tetra_device.h:
//   first case   w1 = K x^3 (4 - x S),  w_l = K x^4 r_l1 (l = 2, 3, 4)
//   third case   w_l = V - K' y^4 r_4l (l = 1, 2, 3),  w4 = V - K' y^3 (4 - y S')
//   middle case  w_l(z) = w_l(E2) + sum_k c_lk z^(k+1) / (k+1): the integral from E2 of the cubic
//                dw_l/dE (the expansion written out at corner_dos_B_coeffs), with w_l(E2) the first
//                case's value at x = E21.
// The kernels add increments w_l(E_j) - w_l(E_{j-1}); with bins much narrower than the tetrahedron they are small
// differences of values up to V = V_T/(4 V_G), and FP32 evaluation leaves them a relative error of about 1e-7 E41/de,
// FP64 about 1e-16 E41/de. They use the FP64 volumes below (nos_volumes, corner_nos) and energy_index. The forms per
// case, in FP32 (TetSetup) and FP64 (NosSetup), and the steps found from FP32 frames (shift_frames, step_window) are a
// second writing of the same weights and steps that only checks on the host call.

__host__ __device__ __forceinline__ void corner_nos_A(const TetSetup& c, float x, float w[4]) {
  const float t = c.kA * x * x * x;
  const float u = t * x;
  w[0] = t * (4.0f - x * c.sA);
  w[1] = u * c.r21;
  w[2] = u * c.r31;
  w[3] = u * c.r41;
}

// coef[l][k] is the z^k coefficient of w_{l+1} on the middle case (k = 0..4).
__host__ __device__ __forceinline__ void corner_nos_B_coeffs(const TetSetup& c, float V, float coef[4][5]) {
  float g[4][4];
  corner_dos_B_coeffs(c, V, g);
  // first-case values at x = a = E21, written with a * r21 = 1 so that a = 0 gives zeros
  const float a = c.e21, ka2 = V * c.r31 * c.r41 * a * a;
  coef[0][0] = ka2 * (3.0f - a * c.r31 - a * c.r41);
  coef[1][0] = ka2;
  coef[2][0] = ka2 * a * c.r31;
  coef[3][0] = ka2 * a * c.r41;
#pragma unroll
  for (int l = 0; l < 4; ++l) {
    coef[l][1] = g[l][0];
    coef[l][2] = 0.5f * g[l][1];
    coef[l][3] = (1.0f / 3.0f) * g[l][2];
    coef[l][4] = 0.25f * g[l][3];
  }
}

__host__ __device__ __forceinline__ void corner_nos_B_poly(const float coef[4][5], float z, float w[4]) {
#pragma unroll
  for (int l = 0; l < 4; ++l)
    w[l] = __builtin_fmaf(
        __builtin_fmaf(__builtin_fmaf(__builtin_fmaf(coef[l][4], z, coef[l][3]), z, coef[l][2]), z, coef[l][1]), z,
        coef[l][0]);
}

__host__ __device__ __forceinline__ void corner_nos_C(const TetSetup& c, float V, float y, float w[4]) {
  const float t = c.kC * y * y * y;
  const float u = t * y;
  w[0] = V - u * c.r41;
  w[1] = V - u * c.r42;
  w[2] = V - u * c.r43;
  w[3] = V - t * (4.0f - y * c.sC);
}

// The integrated weights by volumes, in FP64 from the sorted corner energies and six reciprocals (few
// registers, no cancellation): the part below E of a tetrahedron is one tetrahedron in the first case,
// three in the middle one, the whole less one in the third, and each of those carries a quarter of its
// volume per vertex, shared out by the vertex's barycentric coordinates. V = V_T/(4 V_G).
struct NosVolumes {
  float e[4];
  double r21, r31, r41, r32, r42, r43;
};
__host__ __device__ __forceinline__ NosVolumes nos_volumes(const float e[4]) {
  NosVolumes c;
  for (int l = 0; l < 4; ++l) c.e[l] = e[l];
  // Reciprocals of zero differences are not finite; the case that would use them is never selected.
  auto inverse = [&](int i, int j) { return rcp64((double)c.e[i] - (double)c.e[j]); };
  c.r21 = inverse(1, 0);
  c.r31 = inverse(2, 0);
  c.r41 = inverse(3, 0);
  c.r32 = inverse(2, 1);
  c.r42 = inverse(3, 1);
  c.r43 = inverse(3, 2);
  return c;
}
__host__ __device__ __forceinline__ void corner_nos(const NosVolumes& c, double V, double E, double w[4]) {
  const double x = E - c.e[0], y = c.e[3] - E;
  if (!(y > 0.0)) {
    w[0] = w[1] = w[2] = w[3] = V;
  } else if (!(x > 0.0)) {
    w[0] = w[1] = w[2] = w[3] = 0.0;
  } else if (E <= c.e[1]) {
    const double a = x * c.r21, b = x * c.r31, d = x * c.r41, f = V * a * b * d;
    w[0] = f * (4.0 - a - b - d);
    w[1] = f * a;
    w[2] = f * b;
    w[3] = f * d;
  } else if (E <= c.e[2]) {
    const double z = E - c.e[1], r13 = x * c.r31, r14 = x * c.r41, r23 = z * c.r32, r24 = z * c.r42;
    const double s23 = 1.0 - r23, s24 = 1.0 - r24;
    const double a = V * r13 * r14 * s24, b = V * r13 * r24 * s23, d = V * r23 * r24;
    w[0] = a * (3.0 - r13 - r14) + b * (2.0 - r13) + d;
    w[1] = a * s24 + b * (s24 + s23) + d * (1.0 + s23 + s24);
    w[2] = a * r13 + b * (r13 + r23) + d * r23;
    w[3] = a * (r14 + r24) + b * r24 + d * r24;
  } else {
    const double a = y * c.r41, b = y * c.r42, d = y * c.r43, f = V * a * b * d;
    w[0] = V - f * a;
    w[1] = V - f * b;
    w[2] = V - f * d;
    w[3] = V - f * (4.0 - a - b - d);
  }
}

// The first grid index j with E_j at or above (above = false) or above (true) e, on E_j = e0 + (j + joff) de: the
// rounded quotient, put right by the sign of e - E_j, which the fused product gives exactly (e - e0 of two FP32
// values and the product's 46 bits are exact). Without it a flat tetrahedron on a grid energy whose quotient
// rounds up, such as 32.8125 / 4.6875, is full one energy before its step is looked for. Kept inside [lo, top].
__host__ __device__ __forceinline__ double energy_index(float e, double e0, double de, double inv_de, double joff,
                                                      bool above, double lo, double top) {
  const double x = (double)e - e0, u = x * inv_de - joff;
  if (!(u > lo)) return lo;
  if (!(u < top)) return top;
  double j = ceil(u);
  if (fabs(u - rint(u)) > 1.0e-6) return fmin(j, top);  // no rounding reaches the next index
  auto past = [&](double i) {
    const double r = __builtin_fma(-(i + joff), de, x);  // e - E_i
    return above ? r < 0.0 : r <= 0.0;
  };
  if (!past(j)) j += 1.0;
  else if (past(j - 1.0)) j -= 1.0;
  return fmin(j, top);
}

// FP64 constants of one tetrahedron-band (checks on the host only).
struct NosSetup {
  double x0, z0, y0;  // grid index 0 in the local frames: E_0 - E1, E_0 - E2, E4 - E_0
  double e21, e31, e41, e32, e42;
  double r21, r31, r41, r32, r42, r43;
  double kA, sA, kC, sC;
};

// e sorted ascending; grid E_j = e0 + (j + joff) de. Differences of FP32 values are exact in FP64.
__host__ __device__ __forceinline__ NosSetup nos_setup(const float e[4], float e0, float joff, float de, double V) {
  NosSetup c;
  const double E0 = (double)e0 + (double)joff * (double)de;
  c.x0 = E0 - (double)e[0];
  c.z0 = E0 - (double)e[1];
  c.y0 = (double)e[3] - E0;
  c.e21 = (double)e[1] - (double)e[0];
  c.e31 = (double)e[2] - (double)e[0];
  c.e41 = (double)e[3] - (double)e[0];
  c.e32 = (double)e[2] - (double)e[1];
  c.e42 = (double)e[3] - (double)e[1];
  // Reciprocals of zero differences are infinite; the case that would use them is never selected.
  c.r21 = 1.0 / c.e21;
  c.r31 = 1.0 / c.e31;
  c.r41 = 1.0 / c.e41;
  c.r32 = 1.0 / c.e32;
  c.r42 = 1.0 / c.e42;
  c.r43 = 1.0 / ((double)e[3] - (double)e[2]);
  c.kA = V * c.r21 * c.r31 * c.r41;
  c.sA = c.r21 + c.r31 + c.r41;
  c.kC = V * c.r41 * c.r42 * c.r43;
  c.sC = c.r41 + c.r42 + c.r43;
  return c;
}

__host__ __device__ __forceinline__ void corner_nos_A(const NosSetup& c, double x, double w[4]) {
  const double t = c.kA * x * x * x;
  const double u = t * x;
  w[0] = t * (4.0 - x * c.sA);
  w[1] = u * c.r21;
  w[2] = u * c.r31;
  w[3] = u * c.r41;
}

// coef[l][k] is the z^k coefficient of w_{l+1} on the middle case (k = 0..4).
__host__ __device__ __forceinline__ void corner_nos_B_coeffs(const NosSetup& c, double V, double coef[4][5]) {
  const double a = c.e21, b = c.e32, cc = c.e42;
  const double rb = c.r32, rc = c.r42, rbc = rb * rc;
  const double k1 = V * c.r31 * c.r41, k31 = k1 * c.r31, k41 = k1 * c.r41, k3141 = k31 * c.r41;
  const double ab = a * b, ac = a * cc, bc = b * cc, aa = a * a, bb = b * b, c2 = cc * cc;
  // the cubic dw_l/dE = sum_k g_lk z^k (same expansion as corner_dos_B_coeffs)
  const double g[4][4] = {
      {4.0 * a * (ab + ac + 2.0 * bc) * k3141, -12.0 * (aa - bc) * k3141, -12.0 * (2.0 * a + b + cc) * k3141,
       4.0 * (aa + 2.0 * ab + 2.0 * ac + bb + bc + c2) * rbc * k3141},
      {4.0 * a * k1, 12.0 * k1, -12.0 * (a + b + cc) * rbc * k1, 4.0 * (ab + ac + bb + bc + c2) * rbc * rbc * k1},
      {4.0 * aa * k31, 12.0 * a * k31, 12.0 * k31, -4.0 * (aa + 2.0 * ab + ac + bb + 2.0 * bc) * rb * rbc * k31},
      {4.0 * aa * k41, 12.0 * a * k41, 12.0 * k41, -4.0 * (aa + ab + 2.0 * ac + 2.0 * bc + c2) * rc * rbc * k41}};
  // first-case values at x = a = E21, written with a * r21 = 1 so that a = 0 gives zeros
  const double ka2 = k1 * a * a;
  coef[0][0] = ka2 * (3.0 - a * c.r31 - a * c.r41);
  coef[1][0] = ka2;
  coef[2][0] = ka2 * a * c.r31;
  coef[3][0] = ka2 * a * c.r41;
#pragma unroll
  for (int l = 0; l < 4; ++l) {
    coef[l][1] = g[l][0];
    coef[l][2] = 0.5 * g[l][1];
    coef[l][3] = (1.0 / 3.0) * g[l][2];
    coef[l][4] = 0.25 * g[l][3];
  }
}

__host__ __device__ __forceinline__ void corner_nos_B_poly(const double coef[4][5], double z, double w[4]) {
#pragma unroll
  for (int l = 0; l < 4; ++l) w[l] = (((coef[l][4] * z + coef[l][3]) * z + coef[l][2]) * z + coef[l][1]) * z + coef[l][0];
}

__host__ __device__ __forceinline__ void corner_nos_C(const NosSetup& c, double V, double y, double w[4]) {
  const double t = c.kC * y * y * y;
  const double u = t * y;
  w[0] = V - u * c.r41;
  w[1] = V - u * c.r42;
  w[2] = V - u * c.r43;
  w[3] = V - t * (4.0 - y * c.sC);
}

// Moves the energy origin of the local frames by s (the energies become E_j = e0 + s + j*de); s = -de/2
// gives the midpoints between grid energies. Each head absorbs s exactly, the rounding goes to the tail.
__host__ __device__ __forceinline__ void shift_frames(TetSetup& c, float s) {
  float hi, lo;
  two_sum(c.d_hi, s, hi, lo);
  c.d_hi = hi;
  c.d_lo += lo;
  two_sum(c.f_hi, s, hi, lo);
  c.f_hi = hi;
  c.f_lo += lo;
  two_sum(c.h_hi, s, hi, lo);
  c.h_hi = hi;
  c.h_lo += lo;
}

// Steps of one tetrahedron-band's number of states on the grid E_j = e0 + (j + joff) de, with the
// frames of c shifted by joff*de: ja = first j with x_j > 0 (E_j > E1), js = first j with x_j >= E41
// (E_j >= E4), exact from estimates and the local frame. Indices below 0 or beyond the grid are only
// determined as such (the estimates are clamped to [-2, 3e7]).
__host__ __device__ __forceinline__ void step_window(const TetSetup& c, float e1, float e4, float e0, float joff,
                                                     float de, float inv_de, int& ja, int& js) {
  const float big = 3.0e7f;
  const float t1 = fminf(fmaxf((e1 - e0) * inv_de - joff, -2.0f), big);
  const float t4 = fminf(fmaxf((e4 - e0) * inv_de - joff, -2.0f), big);
  ja = (int)floorf(t1) + 1;
  js = (int)ceilf(t4);
  if (!(local_x(c, ja, de) > 0.0f)) ++ja;
  else if (local_x(c, ja - 1, de) > 0.0f) --ja;
  if (!(local_x(c, js, de) >= c.e41)) ++js;
  else if (local_x(c, js - 1, de) >= c.e41) --js;
}

}  // namespace tetra
