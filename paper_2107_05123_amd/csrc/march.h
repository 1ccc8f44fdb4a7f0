// The pressure-Poisson leaf operator as a march along the last axis.
//
// A lane walks one column of leaves.  Between two leaves it keeps the node
// layer they share with its phase field and its differences along x and y
// already transformed in x and y, and on the way out the contributions to
// that layer still in the transformed space, so these transforms run once per
// node layer instead of once for each of the two leaves that share it.
//
// Two-point transform.  The Q1 values at the Gauss points -+1/sqrt(3) are
// w (a + c b) and w (c a + b), w = (1 + 1/sqrt3)/2, c = 2 - sqrt3.  The
// transforms below leave w out (two fused multiply-adds each); w^3 of the
// phase field goes into its nodal scaling, w^4 of trial and test function
// into the coefficient.
//
// Coefficient 1/rho(clamp(phi)): with s = (1 + phi)/2 the pull back is a
// clamp to [0, 1], which the hardware applies for free as the output
// modifier of the multiply-add that forms s, and rho = rho- + (rho+ - rho-) s
// holds the light phase exactly.
#pragma once
#include <hip/hip_runtime.h>

namespace chns {
namespace march {

constexpr double kC = 0.26794919243112270647;  // 2 - sqrt(3)
constexpr double kW = 0.78867513459481288225;  // (1 + 1/sqrt(3))/2

__device__ __forceinline__ double mad(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float mad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double sat(double v) { return fmin(fmax(v, 0.0), 1.0); }
__device__ __forceinline__ float sat(float v) { return __builtin_amdgcn_fmed3f(v, 0.0f, 1.0f); }
// hardware estimate (better than 2^-20) and one third-order step: the error
// e^3 is below 2^-60 (three multiply-adds; two Newton steps take four)
__device__ __forceinline__ double recip(double r) {
  const double y = __builtin_amdgcn_rcp(r);
  const double e = __builtin_fma(-r, y, 1.0);
  return __builtin_fma(y, __builtin_fma(e, e, e), y);
}
__device__ __forceinline__ float recip(float r) { return __builtin_amdgcn_rcpf(r); }
// Four reciprocals.  FP64 with `joint`: that of the product, multiplied back
// (nine products and one refined estimate instead of four, each result off by
// two more roundings); the fourth powers of the arguments have to stay inside
// the double range.
__device__ __forceinline__ void recip4(double* r, bool joint) {
  if (joint) {
    const double a = r[0], b = r[1], c = r[2], d = r[3];
    const double ab = a * b, cd = c * d;
    const double t = recip(ab * cd);
    const double iab = t * cd, icd = t * ab;
    r[0] = iab * b;
    r[1] = iab * a;
    r[2] = icd * d;
    r[3] = icd * c;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = recip(r[i]);
  }
}
__device__ __forceinline__ void recip4(float* r, bool) {
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = recip(r[i]);
}
// stored phase field (FP64: phi, FP32: 1 + phi) -> w^3 s, s = (1 + phi)/2
__device__ __forceinline__ double phase_node(double v) {
  constexpr double k = 0.5 * kW * kW * kW;
  return __builtin_fma(v, k, k);
}
__device__ __forceinline__ float phase_node(float v) { return v * (float)(0.5 * kW * kW * kW); }

// (a, b) -> (a + c b, c a + b); symmetric, so also its own transpose
template <typename T>
__device__ __forceinline__ void tf(T a, T b, T& u, T& v) {
  u = mad(T(kC), b, a);
  v = mad(T(kC), a, b);
}

// coefficient 1/(A s + B) of one level, with det J, the gradients' scales and
// w^4 of trial and test function folded in (3D: rho/F, F = h w^4/8)
template <typename T>
struct PpCoef {
  T A, B;
  bool joint;
};
// r = rho-/rho+
template <typename T>
__device__ __forceinline__ PpCoef<T> pp_coef3(double r, int lev, bool joint) {
  const double f = ldexp(8.0 / (kW * kW * kW * kW), lev);
  return {T((1.0 - r) * f), T(r * f), joint};
}
// joint reciprocals (recip4) for density ratios up to 1e50 either way
__host__ __device__ inline bool pp_joint(double r) { return r > 1e-50 && r < 1e50; }

// Corner order of a layer: (x, y), (x+1, y), (x, y+1), (x+1, y+1).
//
// Differences are taken between nodal values, before any transform: for a
// smooth field they are then exact up to the field's own rounding.
template <typename T>
struct PpMarch {
  // last node layer: corner values, differences along x (at the Gauss points
  // gy) and along y (at gx), phase field at the Gauss columns (gx + 2 gy)
  T U[4], X[2], Y[2], P[4];
  // contributions of the leaf below to that layer: along z at the Gauss
  // columns, along x (per gy) and along y (per gx)
  T aV[4], aX[2], aY[2];

  // 2 x 2 nodal values of a layer -> values at its Gauss columns
  __device__ __forceinline__ static void plane(T a, T b, T c, T d, T* v) {
    T a0, a1, b0, b1;
    tf(a, b, a0, a1);
    tf(c, d, b0, b1);
    tf(a0, b0, v[0], v[2]);
    tf(a1, b1, v[1], v[3]);
  }
  __device__ __forceinline__ static void layer(const T* u, const T* p, T* x, T* y, T* ph) {
    tf(u[1] - u[0], u[3] - u[2], x[0], x[1]);
    tf(u[2] - u[0], u[3] - u[1], y[0], y[1]);
    plane(phase_node(p[0]), phase_node(p[1]), phase_node(p[2]), phase_node(p[3]), ph);
  }

  __device__ __forceinline__ void start(const T* u, const T* p) {
    layer(u, p, X, Y, P);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      U[i] = u[i];
      aV[i] = T(0);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) aX[i] = aY[i] = T(0);
  }

  // contributions in the transformed space -> the layer's corners
  __device__ __forceinline__ static void corners(const T* v, const T* x, const T* y, T* r) {
    T a0, a1, b0, b1, d0, d1;
    tf(v[0], v[2], a0, b0);
    tf(v[1], v[3], a1, b1);
    a0 -= y[0];
    b0 += y[0];
    a1 -= y[1];
    b1 += y[1];
    tf(a0, a1, r[0], r[1]);
    tf(b0, b1, r[2], r[3]);
    tf(x[0], x[1], d0, d1);
    r[0] -= d0;
    r[1] += d0;
    r[2] -= d1;
    r[3] += d1;
  }

  // the leaf between the last layer and the layer (u, p): r takes the last
  // layer's corner sums (this leaf and the one below).  next() runs once the corners are consumed: the place to
  // load the following layer into the same registers.
  template <class NEXT>
  __device__ __forceinline__ void step(const T* u, const T* p, const PpCoef<T>& c, T* r, const NEXT& next) {
    T v[4], x[2], y[2], ph[4], k0[4], k1[4];
    layer(u, p, x, y, ph);
    plane(u[0] - U[0], u[1] - U[1], u[2] - U[2], u[3] - U[3], v);
#pragma unroll
    for (int q = 0; q < 4; ++q) U[q] = u[q];
    next();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      k0[q] = mad(c.A, sat(mad(T(kC), ph[q], P[q])), c.B);
      k1[q] = mad(c.A, sat(mad(T(kC), P[q], ph[q])), c.B);
      P[q] = ph[q];
    }
    recip4(k0, c.joint);
    recip4(k1, c.joint);
    T g0, g1, cX[2], cY[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      // along x: constant in gx, i = gy
      tf(X[i], x[i], g0, g1);
      g0 *= k0[2 * i] + k0[2 * i + 1];
      g1 *= k1[2 * i] + k1[2 * i + 1];
      cX[i] = mad(T(kC), g1, aX[i] + g0);
      aX[i] = mad(T(kC), g0, g1);
      X[i] = x[i];
      // along y: constant in gy, i = gx
      tf(Y[i], y[i], g0, g1);
      g0 *= k0[i] + k0[i + 2];
      g1 *= k1[i] + k1[i + 2];
      cY[i] = mad(T(kC), g1, aY[i] + g0);
      aY[i] = mad(T(kC), g0, g1);
      Y[i] = y[i];
    }
    T cV[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const T g = v[q] * (k0[q] + k1[q]);
      cV[q] = aV[q] - g;
      aV[q] = g;
    }
    corners(cV, cX, cY, r);
  }

  // corner sums of the last layer of the march
  __device__ __forceinline__ void finish(T* r) { corners(aV, aX, aY, r); }
};

}  // namespace march
}  // namespace chns
