// Matrix-free Q1 operator applies on bricks of octree leaves (gfx950).
//
// y = P^T (sum_e K_e) P x without assembling anything:
//   * a brick is an aligned cube of B^d leaves of one level; one wavefront
//     owns 64/B^(d-1) bricks and walks them layer by layer along the last
//     axis, one leaf column per lane;
//   * each node layer of a brick is gathered once into LDS through the
//     brick's node table; hanging entries are interpolated from their parents
//     on the fly (the constraint P, paper Sec. 4.3 and Fig. 1 caption);
//   * every lane evaluates its leaf with sum-factorised 2-point Gauss
//     quadrature (the element operators below);
//   * leaf results are summed per node in LDS in a fixed order; nodes inside
//     a brick are written straight to y, nodes on a brick face go to a slot
//     buffer, and a second pass (k_combine) adds the slots of every shared
//     node in a fixed order, applying P^T for hanging entries.  No atomics:
//     the result is bitwise reproducible.
#include <algorithm>
#include <mutex>

#include "brick_geom.h"
#include "chns_internal.h"
#include "elem_chns.h"
#include "pp_tile.h"

namespace chns {
namespace {

// Slot buffer of the allocation-free apply (chns_apply_operator_noalloc):
// one per GPU, held until the process ends.  In host code `scratch` names a
// host-side stand-in; kernels get the device address from scratch_address().
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// ------------------------------------------------------------ arithmetic
__device__ __forceinline__ double rcp_t(double r) {
  // hardware estimate refined by two Newton steps (error well below 1e-15)
  double y = __builtin_amdgcn_rcp(r);
  double e = __builtin_fma(-r, y, 1.0);
  y = __builtin_fma(y, e, y);
  e = __builtin_fma(-r, y, 1.0);
  return __builtin_fma(y, e, y);
}
__device__ __forceinline__ float rcp_t(float r) { return __builtin_amdgcn_rcpf(r); }
// 1/sqrt(x) for x > 0: hardware estimate refined by two Newton steps
// y <- y + y (1 - x y^2) / 2 (FP64), the hardware value alone in FP32
__device__ __forceinline__ double rsqrt_t(double x) {
  double y = __builtin_amdgcn_rsq(x);
  double e = __builtin_fma(-x * y, y, 1.0);
  y = __builtin_fma(0.5 * y, e, y);
  e = __builtin_fma(-x * y, y, 1.0);
  return __builtin_fma(0.5 * y, e, y);
}
__device__ __forceinline__ float rsqrt_t(float x) { return __builtin_amdgcn_rsqf(x); }
// fused multiply-add in the operands' own precision (__builtin_fma is the
// double one: float operands would be widened and the result narrowed)
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// 1D two-node / two-Gauss-point transform, scaled by 1/w: (a, b) nodal values
// -> (a + c b, c a + b) = values at xi = -1/sqrt3, +1/sqrt3 over w, with
// w = (1 + 1/sqrt3)/2 and c = 2 - sqrt3: two multiply-adds (sum, difference
// and one multiply-add for each point took four operations; the transforms
// are half of the momentum leaf's FP64 work).  The matrix is symmetric, so the
// same transform also applies the transpose.  The powers of w are folded into
// the forms' constants.
template <typename T>
__device__ __forceinline__ void pair_tf(T& a, T& b) {
  T u, v;
  march::tf(a, b, u, v);
  a = u;
  b = v;
}
// w^n
template <int N>
constexpr double kWp = march::kW * kWp<N - 1>;
template <>
inline constexpr double kWp<0> = 1.0;
// A constant with its rounding to T beside it.  An FP32 constant is off by up
// to 2^-25, the same for every leaf: where the constant only scales values, a
// bias of the whole result (the Cahn-Hilliard Jacobian at 32^3 leaves was 7.3e-8
// from 64 bits with plain constants, 6.0e-8 with these).
template <typename T>
struct Const2 {
  T hi, lo;
};
template <typename T>
__host__ __device__ constexpr Const2<T> const2(double v) {
  return {T(v), T(v - (double)T(v))};
}
// times 2^e
template <typename T>
__device__ __forceinline__ Const2<T> scaled(Const2<T> c, int e) {
  return {T(ldexp(c.hi, e)), T(ldexp(c.lo, e))};
}
__device__ __forceinline__ double times(double v, Const2<double> c) { return v * c.hi; }
__device__ __forceinline__ float times(float v, Const2<float> c) { return fma_t(v, c.hi, v * c.lo); }

// Phase field of the mixture laws: s = (1 + phi)/2, its pull back a clamp to
// [0, 1], rho = rho- + (rho+ - rho-) s.  The stored field (FP64 phi, FP32 1 +
// phi) becomes w^d s at the corners, before the transforms, so that the light
// phase, s = 0, is held exactly; taken from phi after them, rho- came out of a
// difference of two rounded halves, and the 2D pressure apply at density ratio
// 1000 on 64^2 leaves was 9e-14 from extended precision instead of 1.5e-16.
template <int DIM>
__device__ __forceinline__ double phase_s(double v) {
  constexpr double k = 0.5 * kWp<DIM>;
  return __builtin_fma(v, k, k);
}
template <int DIM>
__device__ __forceinline__ float phase_s(float v) {
  return times(v, const2<float>(0.5 * kWp<DIM>));
}

template <int N, int BIT, typename T>
__device__ __forceinline__ void stage(T* v) {
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (!(i & BIT)) pair_tf(v[i], v[i | BIT]);
}
template <int DIM, typename T>
__device__ __forceinline__ void all_stages(T* v) {
  constexpr int N = 1 << DIM;
  stage<N, 1>(v);
  stage<N, 2>(v);
  if constexpr (DIM == 3) stage<N, 4>(v);
}
__host__ __device__ constexpr int insert0(int r, int d) { return (r & ((1 << d) - 1)) | ((r >> d) << (d + 1)); }

// --------------------------------------------------------- element operators
// Folded constants: with values scaled by w^-d through the stages, the Gauss
// weights (1), det J = (h/2)^d, the (2/h)^2 of two gradients and the powers of
// w collapse into per-level constants, so c_q = 1/rho(s_q) costs one fma, one
// clamp and one reciprocal per Gauss point, and one fma per corner for s.

// Pressure Poisson: y_a = sum_q detJ (2/h)^2 c_q gradN_a . grad x,
// c_q = 1/rho(clamp(phi_q)) (Def. 2, VMS pressure Poisson; pull back remark).
template <int DIM, typename T, bool RCP = true>
__device__ __forceinline__ void elem_pp_coef(const T* ph, T A, T Bc, T* c) {
  constexpr int NC = 1 << DIM;
#pragma unroll
  for (int i = 0; i < NC; ++i) c[i] = phase_s<DIM>(ph[i]);
  all_stages<DIM>(c);
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    // coefficient 1 / (A s + B) (pressure) or A s + B (viscosity)
    const T lin = fma_t(A, march::sat(c[i]), Bc);
    c[i] = RCP ? rcp_t(lin) : lin;
  }
}
template <int DIM, typename T>
__device__ __forceinline__ void elem_pp_apply(const T* x, const T* c, T* y) {
  constexpr int NC = 1 << DIM, H = NC / 2;
#pragma unroll
  for (int i = 0; i < NC; ++i) y[i] = T(0);
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    T g[H];
#pragma unroll
    for (int r = 0; r < H; ++r) {
      const int lo = insert0(r, d), hi = lo | (1 << d);
      g[r] = x[hi] - x[lo];
    }
    stage<H, 1>(g);
    if constexpr (H > 2) stage<H, 2>(g);
#pragma unroll
    for (int r = 0; r < H; ++r) {
      const int lo = insert0(r, d), hi = lo | (1 << d);
      g[r] *= (c[lo] + c[hi]);
    }
    stage<H, 1>(g);
    if constexpr (H > 2) stage<H, 2>(g);
#pragma unroll
    for (int r = 0; r < H; ++r) {
      const int lo = insert0(r, d), hi = lo | (1 << d);
      y[hi] += g[r];
      y[lo] -= g[r];
    }
  }
}

template <int DIM, typename T, bool RCP = true>
__device__ __forceinline__ void elem_pp(const T* x, const T* ph, T A, T Bc, T* y) {
  T c[1 << DIM];
  elem_pp_coef<DIM, T, RCP>(ph, A, Bc, c);
  elem_pp_apply<DIM, T>(x, c, y);
}

// Mass: y_a = sum_q detJ r_q N_a (N . x), r_q = rho(clamp(phi_q)) or 1.
template <int DIM, typename T, bool RHO>
__device__ __forceinline__ void elem_mass_coef(const T* ph, T A, T Bc, T* r) {
  constexpr int NC = 1 << DIM;
  if constexpr (RHO) {
#pragma unroll
    for (int i = 0; i < NC; ++i) r[i] = phase_s<DIM>(ph[i]);
    all_stages<DIM>(r);
#pragma unroll
    for (int i = 0; i < NC; ++i) r[i] = fma_t(A, march::sat(r[i]), Bc);
  } else {
#pragma unroll
    for (int i = 0; i < NC; ++i) r[i] = Bc;
  }
}
template <int DIM, typename T>
__device__ __forceinline__ void elem_mass_apply(const T* x, const T* r, T* y) {
  constexpr int NC = 1 << DIM;
#pragma unroll
  for (int i = 0; i < NC; ++i) y[i] = x[i];
  all_stages<DIM>(y);
#pragma unroll
  for (int i = 0; i < NC; ++i) y[i] *= r[i];
  all_stages<DIM>(y);
}

// ------------------------------------------------------------ op traits
// NI gathered input fields (the vector x; wall nodes read as zero when
// MASK), NCF coefficient fields, NO output fields; WALL: 0 no special rows,
// 1 identity rows on the walls (y = x), 2 zero rows on the walls.
enum OpKind {
  K_PP = 0, K_MASS = 1, K_MASS_RHO = 2, K_CH_RES = 3, K_CH_JAC = 4, K_VP = 5, K_VP_RHS = 6, K_PP_RHS = 7,
  K_VU_RHS = 8, K_ENERGY = 9, K_PPS = 10, K_VPS = 11, K_DIAG = 12
};
template <int OP, int DIM>
struct Traits;
#define CHNS_TRAITS(OPK, ni, ncf, no, mask, wall)                  \
  template <int DIM>                                               \
  struct Traits<OPK, DIM> {                                        \
    static constexpr int NI = ni, NCF = ncf, NO = no, WALL = wall; \
    static constexpr bool MASK = mask;                             \
  };
CHNS_TRAITS(K_PP, 1, 1, 1, false, 0)
CHNS_TRAITS(K_MASS, 1, 0, 1, false, 0)
CHNS_TRAITS(K_MASS_RHO, DIM, 1, DIM, true, 1)
CHNS_TRAITS(K_CH_RES, 2, 2 + DIM, 2, false, 0)
CHNS_TRAITS(K_CH_JAC, 2, 1 + DIM, 2, false, 0)
CHNS_TRAITS(K_VP, DIM, 2 + DIM, DIM, true, 1)
CHNS_TRAITS(K_VP_RHS, 0, 3 * DIM + 3, DIM, false, 2)
CHNS_TRAITS(K_PP_RHS, 0, 4 * DIM + 3, 1, false, 0)
CHNS_TRAITS(K_VU_RHS, 0, 4 * DIM + 4, DIM, false, 2)
CHNS_TRAITS(K_ENERGY, 0, 2 + DIM, 1, false, 0)
CHNS_TRAITS(K_PPS, 1, 1, 1, false, 0)  // pressure operator + shift * mass
CHNS_TRAITS(K_VPS, 1, 1, 1, false, 0)  // scalar momentum: K_{eta/(2 Re)} + M_{rho/dt}
CHNS_TRAITS(K_DIAG, 1, 1, 1, false, 0)  // diagonal of the scalar operators (the input is the node entry itself)
#undef CHNS_TRAITS

constexpr int kMaxCoef = kMaxCoefFields;

// Constants of the Cahn-Hilliard Jacobian and the momentum form, evaluated on
// the host: kernel arguments sit in scalar registers, where the divisions that
// form them would leave 28 vector registers occupied through the march.
template <typename T>
struct FormConst {
  T idt;                     // 1 / dt
  Const2<T> kphi, kmu;       // Jacobian: stiffness of phi and mu over h^(d-2)
  T ra, rb, rwa, rwb;        // momentum: rho = ra s + rb, the same times w^2d
  T kea, keb, cgp, cJ;       // gamma^2 k, grad eta~, gamma J / (2 Pe) (el_vp)
  T tau_c, va, vb, vc;       // 4 / dt^2, eta / Re = va s + vb, C_I d
};
template <int DIM, typename T>
FormConst<T> form_const(const Phys& P, double rm, double em);

template <typename T>
struct BrickArgs {
  const int32_t* table;
  const int8_t* level;
  int64_t count;
  int64_t slot_base;
  int nbnd;
  int64_t n;        // field stride of x and y
  int64_t n_slots;  // field stride of slots
  const T* x;
  const T* cf[kMaxCoef];  // coefficient fields (stride n each)
  T* y;
  T* slots;
  const int32_t* hang;
  const uint8_t* wall;
  double ratio, eta_ratio;  // rho-/rho+, eta-/eta+
  Phys phys;                // physical parameters of the CHNS forms
  double* partials;    // fused x.y partial per block, or null
  const int* done;
  // damped-Jacobi sweep (pressure operator): y = x + sm_w sm_d (sm_r - A x)
  const T* sm_r;
  const T* sm_d;
  T sm_w;
  double shift;  // K_PPS: mass shift
  int diag_of;   // K_DIAG: the operator's form
  FormConst<T> fc;  // K_CH_JAC, K_VP
  // structured (uniform, lexicographically numbered) meshes: node indices are
  // computed from the brick anchor instead of read from the table
  const int32_t* anchor;  // 3 per brick, integer node coordinates
  int64_t sy, sz;         // index strides of y and z
  int32_t side;           // nodes per edge - 1
  // table meshes, 3D 8^3 bricks: eight block bases per brick (base[0] < 0:
  // use the table), from which the node numbers are computed
  const int32_t* abase;
};

// -------------------------------------------------- CHNS element routines
// (corner arrays as in elem_chns.h; w = det J, gs = 2/h)
template <int DIM>
__device__ __forceinline__ void el_ch_res(const double (*x)[1 << DIM], const double (*c)[1 << DIM], const Phys& P,
                                          double gs, double w, double (*y)[1 << DIM]) {
  constexpr int NC = 1 << DIM;
  double pt[NC], mt[NC], dp[NC];
#pragma unroll
  for (int a = 0; a < NC; ++a) {
    pt[a] = 0.5 * (x[0][a] + c[0][a]);
    mt[a] = 0.5 * (x[1][a] + c[1][a]);
    dp[a] = x[0][a] - c[0][a];
    y[0][a] = 0.0;
    y[1][a] = 0.0;
  }
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const double ptq = QP<DIM>::val(pt, q), dpq = QP<DIM>::val(dp, q), mtq = QP<DIM>::val(mt, q);
    double gpt[DIM], gmt[DIM], fl[DIM], fm[DIM];
    QP<DIM>::grad(pt, q, gs, gpt);
    QP<DIM>::grad(mt, q, gs, gmt);
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      const double ut = QP<DIM>::val(c[2 + d], q);
      fl[d] = w * (-ut * ptq + gmt[d] / (P.Pe * P.Cn));
      fm[d] = w * P.Cn * P.Cn * gpt[d];
    }
    const double fphi = w * dpq / P.dt, fmu = w * (dpsi(ptq) - mtq);
#pragma unroll
    for (int a = 0; a < NC; ++a) {
      double s0 = refN<DIM>(q, a) * fphi, s1 = refN<DIM>(q, a) * fmu;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        const double gN = gs * refD<DIM>(q, a, d);
        s0 += gN * fl[d];
        s1 += gN * fm[d];
      }
      y[0][a] += s0;
      y[1][a] += s1;
    }
  }
}

// right-hand sides: coefficient layout phi~, mu~, u^ (DIM), u^k (DIM), p^k,
// then v (DIM) and p^{k+1}, and last the body force f_v (DIM; zero except for
// manufactured solutions), which is the known right-hand side of the momentum
// equation: (w, f_v) in the velocity prediction and -f_v inside R_m
template <int DIM>
__device__ __forceinline__ void el_vp_rhs(const double (*c)[1 << DIM], const Phys& P, double gs, double w,
                                          double (*y)[1 << DIM]) {
  constexpr int NC = 1 << DIM;
  const double* uh[DIM];
#pragma unroll
  for (int d = 0; d < DIM; ++d) uh[d] = c[2 + d];
  const double* pk = c[2 + 2 * DIM];
  constexpr int FV = 3 + 2 * DIM;  // first body-force row
#pragma unroll
  for (int f = 0; f < DIM; ++f)
#pragma unroll
    for (int a = 0; a < NC; ++a) y[f][a] = 0.0;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    MomQ<DIM> M;
    M.init(P, c[0], c[1], uh, q, gs);
    double gp[DIM];
    QP<DIM>::grad(pk, q, gs, gp);
#pragma unroll
    for (int i = 0; i < DIM; ++i) {
      const double* uk = c[2 + DIM + i];
      const double ui = QP<DIM>::val(uk, q);
      double gui[DIM];
      QP<DIM>::grad(uk, q, gs, gui);
      const double kort = kort_i<DIM>(c[0], q, i, gs, M.gphi);
      const double fvi = QP<DIM>::val(c[FV + i], q);
      const double rk = M.rknown(P, i, ui, gui, gp, kort) - fvi;
      const double g = i == P.gaxis ? -1.0 : 0.0;
      const double fN = w * (M.rho * ui / P.dt - 0.5 * M.rho * M.dot(M.uh, gui) - M.dot(M.J, gui) / (2.0 * P.Pe) -
                             gp[i] + M.rho * g / P.Fr + fvi);
      double fG[DIM];
#pragma unroll
      for (int d = 0; d < DIM; ++d) fG[d] = w * (-M.eta * gui[d] / (2.0 * P.Re) + P.Cn / P.We * M.gphi[i] * M.gphi[d]);
      const double fst = -w * M.tau * rk;
#pragma unroll
      for (int a = 0; a < NC; ++a) {
        double gN[DIM];
        gradN<DIM>(q, a, gs, gN);
        y[i][a] += refN<DIM>(q, a) * fN + M.dot(gN, fG) + M.s(P, gN) * fst;
      }
    }
  }
}

template <int DIM>
__device__ __forceinline__ void el_pp_rhs(const double (*c)[1 << DIM], const Phys& P, double gs, double w,
                                          double (*y)[1 << DIM]) {
  constexpr int NC = 1 << DIM;
  const double* uh[DIM];
#pragma unroll
  for (int d = 0; d < DIM; ++d) uh[d] = c[2 + d];
  const double* pk = c[2 + 2 * DIM];
  constexpr int FV = 3 + 3 * DIM;  // first body-force row
#pragma unroll
  for (int a = 0; a < NC; ++a) y[0][a] = 0.0;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    MomQ<DIM> M;
    M.init(P, c[0], c[1], uh, q, gs);
    double gp[DIM], fG[DIM];
    QP<DIM>::grad(pk, q, gs, gp);
    double div = 0.0;
#pragma unroll
    for (int i = 0; i < DIM; ++i) {
      const double* v = c[3 + 2 * DIM + i];
      const double* uk = c[2 + DIM + i];
      double gv[DIM], gui[DIM];
      QP<DIM>::grad(v, q, gs, gv);
      QP<DIM>::grad(uk, q, gs, gui);
      div += gv[i];
      const double rl = M.rlin(P, QP<DIM>::val(v, q), gv);
      const double rk = M.rknown(P, i, QP<DIM>::val(uk, q), gui, gp, kort_i<DIM>(c[0], q, i, gs, M.gphi)) -
                        QP<DIM>::val(c[FV + i], q);
      fG[i] = w * (-(2.0 / P.dt) * M.tau * (rl + rk) / M.rho + gp[i] / M.rho);
    }
    const double fN = -w * (2.0 / P.dt) * div;
#pragma unroll
    for (int a = 0; a < NC; ++a) {
      double gN[DIM];
      gradN<DIM>(q, a, gs, gN);
      y[0][a] += refN<DIM>(q, a) * fN + M.dot(gN, fG);
    }
  }
}

template <int DIM>
__device__ __forceinline__ void el_vu_rhs(const double (*c)[1 << DIM], const Phys& P, double gs, double w,
                                          double (*y)[1 << DIM]) {
  constexpr int NC = 1 << DIM;
  const double* uh[DIM];
#pragma unroll
  for (int d = 0; d < DIM; ++d) uh[d] = c[2 + d];
  const double* pk = c[2 + 2 * DIM];
  const double* pn = c[3 + 3 * DIM];
  constexpr int FV = 4 + 3 * DIM;  // first body-force row
#pragma unroll
  for (int f = 0; f < DIM; ++f)
#pragma unroll
    for (int a = 0; a < NC; ++a) y[f][a] = 0.0;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    MomQ<DIM> M;
    M.init(P, c[0], c[1], uh, q, gs);
    double gp[DIM], gpn[DIM];
    QP<DIM>::grad(pk, q, gs, gp);
    QP<DIM>::grad(pn, q, gs, gpn);
#pragma unroll
    for (int i = 0; i < DIM; ++i) {
      const double* v = c[3 + 2 * DIM + i];
      const double* uk = c[2 + DIM + i];
      double gv[DIM], gui[DIM];
      QP<DIM>::grad(v, q, gs, gv);
      QP<DIM>::grad(uk, q, gs, gui);
      const double vq = QP<DIM>::val(v, q);
      const double rl = M.rlin(P, vq, gv);
      const double rk = M.rknown(P, i, QP<DIM>::val(uk, q), gui, gp, kort_i<DIM>(c[0], q, i, gs, M.gphi)) -
                        QP<DIM>::val(c[FV + i], q);
      const double f = w * (M.rho * vq - M.tau * (rl + rk) - 0.5 * P.dt * (gpn[i] - gp[i]));
#pragma unroll
      for (int a = 0; a < NC; ++a) y[i][a] += refN<DIM>(q, a) * f;
    }
  }
}

// energy density of the leaf, split equally over its corners:
// 1/2 rho |u|^2 + (psi + Cn^2/2 |grad phi|^2)/(Cn We) + rho y / Fr
// (coefficients: phi, the vertical coordinate, u)
template <int DIM>
__device__ __forceinline__ void el_energy(const double (*c)[1 << DIM], const Phys& P, double gs, double w,
                                          double (*y)[1 << DIM]) {
  constexpr int NC = 1 << DIM;
  double e = 0.0;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const double ph = QP<DIM>::val(c[0], q);
    const double rho = P.alpha * pull_back(ph) + P.beta;
    double g[DIM];
    QP<DIM>::grad(c[0], q, gs, g);
    double uu = 0.0, gg = 0.0;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      const double u = QP<DIM>::val(c[2 + d], q);
      uu += u * u;
      gg += g[d] * g[d];
    }
    e += w * (0.5 * rho * uu + (psi(ph) + 0.5 * P.Cn * P.Cn * gg) / (P.Cn * P.We) + rho * QP<DIM>::val(c[1], q) / P.Fr);
  }
#pragma unroll
  for (int a = 0; a < NC; ++a) y[0][a] = e / NC;
}

// ---------------------------------------- heavy forms, corners read on demand
// The Cahn-Hilliard Jacobian and the VMS momentum operator read many fields;
// their element routines take the corner values through an accessor cv(f, a)
// (field f, corner a) that reads the brick's LDS node layers, so that no
// field is held in registers longer than it is used.
//
// Phase-field storage: FP64 fields hold phi, FP32 fields hold 1 + phi (so
// that rho keeps its relative accuracy near phi = -1 at large density ratios);
// the mixture laws are rho = ra s + rb, eta = ea s + eb in s = (1 + phi)/2.
// rm, em: rho-/rho+, eta-/eta+.
template <int DIM, typename T>
FormConst<T> form_const(const Phys& P, double rm, double em) {
  constexpr double wd = kWp<DIM>, w2d = kWp<2 * DIM>, g1 = 1.0 / (2.0 * march::kW);  // gamma / (2/h)
  const double st = DIM == 3 ? 1.0 / 12.0 : 1.0 / 6.0;
  FormConst<T> f;
  f.idt = T(1.0 / P.dt);
  f.kphi = const2<T>(st * P.Cn * P.Cn * 0.5);
  f.kmu = const2<T>(st / (2.0 * P.Pe * P.Cn));
  f.ra = T(1.0 - rm);
  f.rb = T(rm);
  f.rwa = T((1.0 - rm) * w2d);
  f.rwb = T(rm * w2d);
  // gamma^2 k, gamma^2 w^d gam/(2 Re) (grad eta~ of a transformed column, one
  // gamma its own and one of grad v) and gamma J / (2 Pe), without their 2/h
  f.kea = T((1.0 - em) / (2.0 * P.Re) * (g1 * g1 * w2d));
  f.keb = T(em / (2.0 * P.Re) * (g1 * g1 * w2d));
  f.cgp = T(P.gam / (2.0 * P.Re) * (wd * g1 * g1 * w2d));
  f.cJ = T(P.cJ * (wd * g1 * g1) / (2.0 * P.Pe));
  f.tau_c = T(4.0 / (P.dt * P.dt));
  f.va = T((1.0 - em) / P.Re);
  f.vb = T(em / P.Re);
  f.vc = T(P.C_I * DIM);
  return f;
}

// Newton Jacobian of the discrete Cahn-Hilliard system (Def. 6), fields
// x = [dphi, dmu] and coefficients [phi~ = (phi^{k+1} + phi^k)/2, u~]:
//   y_phi = M dphi / dt - 1/2 (grad q, u~ dphi) + K dmu / (2 Pe Cn)
//   y_mu  = 1/2 (q, psi''(phi~) dphi) + Cn^2/2 K dphi - 1/2 M dmu
// sum-factorised: values at the Gauss points by the two-point transforms,
// the constant-coefficient stiffness K in closed form (3D: the Q1 element
// matrix is (h/12)(5 I - 1 1^T + edge adjacency); 2D: (4 I - edge adjacency
// - 2 opposite corner)/6), the advection flux through the transposed
// gradient.  cv(f, a): f = 0 dphi, 1 dmu, 2 phi~, 3.. u~.
template <int DIM, typename T, class CV>
__device__ __forceinline__ void el_chj(const CV& cv, const FormConst<T>& K, int lev, T (*y)[1 << DIM]) {
  constexpr int NC = 1 << DIM, H = NC / 2;
  // the w^d of a transform and of its transpose folded into the weight
  const Const2<T> w = scaled(const2<T>(kWp<2 * DIM>), -(lev + 1) * DIM);
  constexpr Const2<T> wd = const2<T>(kWp<DIM>);
  // stiffness parts, corner form
  {
    T xp[NC], xm[NC];
#pragma unroll
    for (int a = 0; a < NC; ++a) {
      xp[a] = cv(0, a);
      xm[a] = cv(1, a);
    }
    const Const2<T> kphi = scaled(K.kphi, -lev * (DIM - 2)), kmu = scaled(K.kmu, -lev * (DIM - 2));
    T sp = T(0), sm = T(0);
#pragma unroll
    for (int a = 0; a < NC; ++a) {
      sp += xp[a];
      sm += xm[a];
    }
#pragma unroll
    for (int a = 0; a < NC; ++a) {
      T kp, km;
      if constexpr (DIM == 3) {
        kp = T(5) * xp[a] - sp + (xp[a ^ 1] + xp[a ^ 2] + xp[a ^ 4]);
        km = T(5) * xm[a] - sm + (xm[a ^ 1] + xm[a ^ 2] + xm[a ^ 4]);
      } else {
        kp = T(4) * xp[a] - (xp[a ^ 1] + xp[a ^ 2]) - T(2) * xp[a ^ 3];
        km = T(4) * xm[a] - (xm[a ^ 1] + xm[a ^ 2]) - T(2) * xm[a ^ 3];
      }
      y[0][a] = times(km, kmu);
      y[1][a] = times(kp, kphi);
    }
    // mass parts at the Gauss points (values scaled by w^-d)
    all_stages<DIM>(xp);
    all_stages<DIM>(xm);
    T pt[NC];
#pragma unroll
    for (int a = 0; a < NC; ++a) pt[a] = cv(2, a);
    all_stages<DIM>(pt);
    T fa[NC], fb[NC];
    const Const2<T> wi{w.hi * K.idt, w.lo * K.idt}, wh{w.hi * T(0.5), w.lo * T(0.5)};
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const T p = times(pt[q], wd);
      const T d2 = T(3) * p * p - T(1);
      fa[q] = times(xp[q], wi);
      fb[q] = times(d2 * xp[q] - xm[q], wh);
    }
    all_stages<DIM>(fa);
    all_stages<DIM>(fb);
#pragma unroll
    for (int a = 0; a < NC; ++a) {
      y[0][a] += fa[a];
      y[1][a] += fb[a];
    }
    // advection -1/2 (grad q, u~ dphi): flux F_d = -1/2 det J u~_d dphi at
    // each Gauss point, then the transposed gradient (constant along d)
    const Const2<T> wa = scaled(const2<T>(-0.5 * kWp<3 * DIM - 1>), -(lev + 1) * DIM + lev);
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      T u[NC];
#pragma unroll
      for (int a = 0; a < NC; ++a) u[a] = cv(3 + d, a);
      all_stages<DIM>(u);
      T g[H];
#pragma unroll
      for (int r = 0; r < H; ++r) {
        const int lo = insert0(r, d), hi = lo | (1 << d);
        g[r] = u[lo] * xp[lo] + u[hi] * xp[hi];
      }
      stage<H, 1>(g);
      if constexpr (H > 2) stage<H, 2>(g);
#pragma unroll
      for (int r = 0; r < H; ++r) {
        const int lo = insert0(r, d), hi = lo | (1 << d);
        const T v = times(g[r], wa);
        y[0][hi] += v;
        y[0][lo] -= v;
      }
    }
  }
}

// VMS velocity prediction (Def. 3, tau_m and R_m of Sec. 3.1), the same
// scalar operator for every component.  Per Gauss point, with
// b = u^/2 + J/(2 Pe rho~), g = grad eta~/(2 Re) and k = eta~/(2 Re):
//   R_lin(v) = rho~ (v/dt + b.grad v) - g.grad v,
//   Galerkin part  N_a rho~ (v/dt + b.grad v) + k grad N_a . grad v,
//   stabilisation  (b.grad N_a) tau_m R_lin(v).
// Sum-factorised: every field's values at the Gauss points come from the
// two-point transforms (w^-d times the value), its gradient along d from the
// differences along d carried through the transforms of the other
// directions (constant along d, so shared by the two Gauss points of a
// column).  In units of the transformed values a gradient is gamma times the
// transformed difference, gamma = (2/h)/(2 w), and the same factor stands in
// front of a gradient test function, so b and k are stored as gamma b and
// gamma^2 k and the weight det J w^2d goes into rho, k and grad eta~; the
// test functions are applied by the same transforms transposed.  The
// coefficients are formed once per Gauss point (the phase field clamped,
// tau_m, b scaled by 2/h, grad phi~ per column with the pull-back mask per
// point), then each component is transformed, combined and handed to
// out(f, y) in turn.  cv(f, a): f < DIM the velocity components, then phi~
// (phi in FP64, 1 + phi in FP32), mu~, u^.
template <int DIM, typename T, class CV, class OUT>
__device__ __forceinline__ void el_vp(const CV& cv, const FormConst<T>& K, int lev, const OUT& out) {
  constexpr int NC = 1 << DIM, H = NC / 2;
  // powers of two (2/h = 2^e1, det J = 2^-d e1) are applied with ldexp: exact,
  // and no per-level constants held in registers
  const int e1 = lev + 1;
  constexpr double g1 = 1.0 / (2.0 * march::kW);  // gamma / (2/h)
  constexpr Const2<T> iS = const2<T>(kWp<DIM>), hg = const2<T>(0.5 * g1);

  // ---- coefficients at the Gauss points
  T sc[NC], tau[NC], bs[DIM][NC], gp[DIM][H];
  unsigned inside = 0;
  {
    T v[NC];
#pragma unroll
    for (int a = 0; a < NC; ++a) v[a] = cv(DIM, a);
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
#pragma unroll
      for (int r = 0; r < H; ++r) {
        const int lo = insert0(r, d), hi = lo | (1 << d);
        gp[d][r] = v[hi] - v[lo];
      }
      stage<H, 1>(gp[d]);
      if constexpr (H > 2) stage<H, 2>(gp[d]);
#pragma unroll
      for (int r = 0; r < H; ++r) gp[d][r] = ldexp(gp[d][r] * K.cgp, 2 * e1);
    }
#pragma unroll
    for (int a = 0; a < NC; ++a) v[a] = phase_s<DIM>(v[a]);
    all_stages<DIM>(v);
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      sc[q] = march::sat(v[q]);
      if (v[q] > T(0) && v[q] < T(1)) inside |= 1u << q;
    }
  }
  asm volatile("" ::: "memory");
  {
    T J[DIM][H];
    {
      T m[NC];
#pragma unroll
      for (int a = 0; a < NC; ++a) m[a] = cv(DIM + 1, a);
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
#pragma unroll
        for (int r = 0; r < H; ++r) {
          const int lo = insert0(r, d), hi = lo | (1 << d);
          J[d][r] = m[hi] - m[lo];
        }
        stage<H, 1>(J[d]);
        if constexpr (H > 2) stage<H, 2>(J[d]);
#pragma unroll
        for (int r = 0; r < H; ++r) J[d][r] = ldexp(J[d][r] * K.cJ, e1);
      }
    }
    T irho[NC], uu[NC], uJ[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      irho[q] = rcp_t(fma_t(K.ra, sc[q], K.rb));
      uu[q] = uJ[q] = T(0);
    }
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      asm volatile("" ::: "memory");
      T u[NC];
#pragma unroll
      for (int a = 0; a < NC; ++a) u[a] = cv(DIM + 2 + d, a);
      all_stages<DIM>(u);
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const int r = (q & ((1 << d) - 1)) | ((q >> (d + 1)) << d);
        const T uh = times(u[q], iS);
        const T j2 = J[d][r];  // gamma J / (2 Pe) over 2/h
        uu[q] = fma_t(uh, uh, uu[q]);
        uJ[q] = fma_t(uh, j2, uJ[q]);
        bs[d][q] = ldexp(fma_t(j2, irho[q], times(uh, hg)), e1);
      }
    }
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const T r = fma_t(K.va, sc[q], K.vb) * irho[q];
      // u^.J / (Pe rho~) = 2 u^.(J / (2 Pe)) / rho~
      tau[q] = rsqrt_t(K.tau_c + ldexp(fma_t(T(2.0 / g1) * uJ[q], irho[q], uu[q]), 2 * e1) + ldexp(K.vc * r * r, 4 * e1));
    }
  }
  // ---- the components in turn (rho with the weight w^2d)
#pragma unroll
  for (int f = 0; f < DIM; ++f) {
    asm volatile("" ::: "memory");
    T v[NC], g[DIM][H], fs[DIM][H];
#pragma unroll
    for (int a = 0; a < NC; ++a) v[a] = cv(f, a);
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
#pragma unroll
      for (int r = 0; r < H; ++r) {
        const int lo = insert0(r, d), hi = lo | (1 << d);
        g[d][r] = v[hi] - v[lo];
        fs[d][r] = T(0);
      }
      stage<H, 1>(g[d]);
      if constexpr (H > 2) stage<H, 2>(g[d]);
    }
    all_stages<DIM>(v);
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const T rho = fma_t(K.rwa, sc[q], K.rwb);
      const T kg = ldexp(fma_t(K.kea, sc[q], K.keb), 2 * e1);
      T Gh = K.idt * v[q], gg = T(0);
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        const int r = (q & ((1 << d) - 1)) | ((q >> (d + 1)) << d);
        Gh = fma_t(bs[d][q], g[d][r], Gh);
        gg = fma_t(gp[d][r], g[d][r], gg);
      }
      const T A = rho * Gh;
      const T Tq = tau[q] * (((inside >> q) & 1u) ? A - gg : A);
      v[q] = A;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        const int r = (q & ((1 << d) - 1)) | ((q >> (d + 1)) << d);
        fs[d][r] = fma_t(kg, g[d][r], fma_t(bs[d][q], Tq, fs[d][r]));
      }
    }
    all_stages<DIM>(v);
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      stage<H, 1>(fs[d]);
      if constexpr (H > 2) stage<H, 2>(fs[d]);
#pragma unroll
      for (int r = 0; r < H; ++r) {
        const int lo = insert0(r, d), hi = lo | (1 << d);
        v[hi] += fs[d][r];
        v[lo] -= fs[d][r];
      }
    }
#pragma unroll
    for (int a = 0; a < NC; ++a) v[a] = ldexp(v[a], -e1 * DIM);  // det J
    out(f, v);
  }
}

template <typename T, bool MASK>
__device__ __forceinline__ T fetch(const T* v, const uint8_t* wall, int32_t i) {
  if constexpr (MASK) return wall[i] ? T(0) : v[i];
  return v[i];
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// The hardware deals workgroups round-robin to the 8 XCDs (block b runs on
// XCD b % 8), each with its own L2.  Bricks are numbered along the Morton
// curve, so handing XCD x the contiguous run of brick groups
// [start(x), start(x) + count(x)) keeps the node layers that neighbouring
// bricks share in one L2.  A bijection for any grid size.
__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t g) {
  constexpr uint32_t kXcd = 8;
  const uint32_t per = g / kXcd, rem = g % kXcd, x = b % kXcd;
  return x * per + (x < rem ? x : rem) + b / kXcd;
}

// per-level folded constants of a form (see op_const)
template <typename T>
struct OpConst {
  T A = 0, Bc = 0, Ms = 0, Am = 0, Bm = 0;
  double gs = 0, wdet = 0;  // right-hand sides, residual and energy: 2/h and det J = (h/2)^d
};
template <int DIM, typename T, int OP>
__device__ __forceinline__ OpConst<T> op_const(const BrickArgs<T>& a, int lev) {
  // rho = rho- + (rho+ - rho-) s and eta likewise, over rho+ and eta+
  const double ra = 1.0 - a.ratio, rb = a.ratio;
  OpConst<T> o;
  o.gs = ldexp(1.0, lev + 1);
  o.wdet = ldexp(1.0, -(lev + 1) * DIM);
  // mass: det J w^2d; stiffness: (h/2)^(d-2) / 4 w^2(d-1)
  const double mass = ldexp(kWp<2 * DIM>, -(lev + 1) * DIM);
  const double F = ldexp(kWp<2 * (DIM - 1)> / 4.0, -(lev + 1) * (DIM - 2));
  if constexpr (OP == K_PPS) o.Ms = T(a.shift * mass);
  if constexpr (OP == K_VPS) {
    // viscosity eta/(2 Re) on the stiffness (folded like the pressure
    // coefficient, without the reciprocal) and rho/dt on the mass
    o.A = T((1.0 - a.eta_ratio) / (2.0 * a.phys.Re) * F);
    o.Bc = T(a.eta_ratio / (2.0 * a.phys.Re) * F);
    o.Am = T(ra / a.phys.dt * mass);
    o.Bm = T(rb / a.phys.dt * mass);
  }
  if constexpr (OP == K_PP || OP == K_PPS) {
    // c~ = F / rho = 1 / (rho / F)
    const double f = ldexp(4.0 / kWp<2 * (DIM - 1)>, (lev + 1) * (DIM - 2));
    o.A = T(ra * f);
    o.Bc = T(rb * f);
  } else if constexpr (OP == K_MASS) {
    o.Bc = T(mass);
  } else if constexpr (OP == K_MASS_RHO) {
    o.A = T(ra * mass);
    o.Bc = T(rb * mass);
  }
  return o;
}

// One leaf's share of the exact diagonal of P^T K P for a scalar operator
// (a.diag_of: pressure with or without a mass shift, scalar momentum, mass,
// density mass): sum over its corner pairs (a, b) of P_ai P_bi K_ab for every
// independent node i.  The share goes through the corners' slots, which the
// combine adds with the squared constraint weights (1, 1/4, 1/16), so corner a
// takes K_aa, and the pairs with a hanging corner are written as follows.
//   * a independent and a parent of b (weight w): node a takes 2 w K_ab;
//   * both hanging with one common parent: it is a corner of the leaf (on a
//     2:1-balanced octree the parents outside the leaf belong to whole edges
//     or faces) and takes 2 w_a w_b K_ab;
//   * both hanging with two common parents: those are the ends of a split edge
//     of the leaf, whose midpoint m is a hanging corner with weights 1/2, so m
//     takes 2 w_a w_b K_ab / (1/2)^2.
// e: the corners' node entries (negative: hanging record).
template <int DIM, typename T>
__device__ __forceinline__ void leaf_diag(const BrickArgs<T>& a, int lev, const T* e, const T* ph, T* y) {
  constexpr int NC = 1 << DIM;
  const bool pp = a.diag_of == K_PP || a.diag_of == K_PPS, vps = a.diag_of == K_VPS;
  T c[NC], r[NC];
  if (pp) {
    const OpConst<T> o = op_const<DIM, T, K_PPS>(a, lev);
    elem_pp_coef<DIM, T, true>(ph, o.A, o.Bc, c);
#pragma unroll
    for (int i = 0; i < NC; ++i) r[i] = a.diag_of == K_PPS ? o.Ms : T(0);
  } else if (vps) {
    const OpConst<T> o = op_const<DIM, T, K_VPS>(a, lev);
    elem_pp_coef<DIM, T, false>(ph, o.A, o.Bc, c);
    elem_mass_coef<DIM, T, true>(ph, o.Am, o.Bm, r);
  } else {
#pragma unroll
    for (int i = 0; i < NC; ++i) c[i] = T(0);
    if (a.diag_of == K_MASS_RHO) {
      const OpConst<T> o = op_const<DIM, T, K_MASS_RHO>(a, lev);
      elem_mass_coef<DIM, T, true>(ph, o.A, o.Bc, r);
    } else {
      const T m = op_const<DIM, T, K_MASS>(a, lev).Bc;
#pragma unroll
      for (int i = 0; i < NC; ++i) r[i] = m;
    }
  }
  int32_t par[NC][4];
  bool hang = false;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int32_t n = (int32_t)e[i];
    y[i] = T(0);
    par[i][0] = n;
    par[i][1] = par[i][2] = par[i][3] = -1;
    if (n < 0) {
      hang = true;
#pragma unroll
      for (int k = 0; k < 4; ++k) par[i][k] = a.hang[4 * (int64_t)(-n - 1) + k];
    }
  }
  auto weight = [&](int i) { return par[i][1] < 0 ? T(1) : par[i][2] < 0 ? T(0.5) : T(0.25); };
#pragma unroll
  for (int b = 0; b < NC; ++b) {
    // column b of the leaf matrix
    T x[NC], k[NC], km[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) x[i] = T(i == b ? 1 : 0);
    elem_pp_apply<DIM, T>(x, c, k);
    elem_mass_apply<DIM, T>(x, r, km);
#pragma unroll
    for (int i = 0; i < NC; ++i) k[i] += km[i];
    y[b] += k[b];
    if (!hang) continue;
#pragma unroll
    for (int i = 0; i < b; ++i) {
      if (par[i][1] < 0 && par[b][1] < 0) continue;  // two independent corners
      const T w = T(2) * weight(i) * weight(b) * k[i];
      int32_t s0 = -1, s1 = -1;  // common parents
#pragma unroll
      for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (par[i][p] >= 0 && par[i][p] == par[b][q]) {
            s1 = s0;
            s0 = par[i][p];
          }
      if (s0 < 0) continue;
#pragma unroll
      for (int m = 0; m < NC; ++m) {
        const bool one = s1 < 0 && par[m][1] < 0 && par[m][0] == s0;
        const bool two = s1 >= 0 && par[m][1] >= 0 && par[m][2] < 0 &&
                         ((par[m][0] == s0 && par[m][1] == s1) || (par[m][0] == s1 && par[m][1] == s0));
        if (one) y[m] += w;
        if (two) y[m] += T(4) * w;
      }
    }
  }
}

// One leaf of the form OP (not the momentum form, which hands each component's
// results over in turn, see el_vp): corner values xc (inputs) and cc
// (coefficients), or the accessor cv(f, a) for the Cahn-Hilliard Jacobian, to
// corner results ye.
template <int DIM, typename T, int OP, class XC, class CC, class CV>
__device__ __forceinline__ void leaf_form(const BrickArgs<T>& a, const OpConst<T>& oc, int lev, const XC& xc,
                                          const CC& cc, const CV& cv, T (*ye)[1 << DIM]) {
  using TR = Traits<OP, DIM>;
  constexpr int NI = TR::NI, NC = 1 << DIM;
  if constexpr (OP == K_DIAG) {
    leaf_diag<DIM, T>(a, lev, xc[0], cc[0], ye[0]);
  } else if constexpr (OP == K_CH_JAC) {
    el_chj<DIM, T>(cv, a.fc, lev, ye);
  } else if constexpr (OP == K_PP || OP == K_PPS) {
    elem_pp<DIM, T>(xc[0], cc[0], oc.A, oc.Bc, ye[0]);
    if constexpr (OP == K_PPS) {
      T r[NC], ym[NC];
#pragma unroll
      for (int i = 0; i < NC; ++i) r[i] = oc.Ms;
      elem_mass_apply<DIM, T>(xc[0], r, ym);
#pragma unroll
      for (int i = 0; i < NC; ++i) ye[0][i] += ym[i];
    }
  } else if constexpr (OP == K_VPS) {
    elem_pp<DIM, T, false>(xc[0], cc[0], oc.A, oc.Bc, ye[0]);
    T r[NC], ym[NC];
    elem_mass_coef<DIM, T, true>(cc[0], oc.Am, oc.Bm, r);
    elem_mass_apply<DIM, T>(xc[0], r, ym);
#pragma unroll
    for (int i = 0; i < NC; ++i) ye[0][i] += ym[i];
  } else if constexpr (OP == K_MASS || OP == K_MASS_RHO) {
    T r[NC];
    elem_mass_coef<DIM, T, OP == K_MASS_RHO>(cc[0], oc.A, oc.Bc, r);
#pragma unroll
    for (int f = 0; f < NI; ++f) elem_mass_apply<DIM, T>(xc[f], r, ye[f]);
  } else if constexpr (OP == K_CH_RES) {
    el_ch_res<DIM>(xc, cc, a.phys, oc.gs, oc.wdet, ye);
  } else if constexpr (OP == K_VP_RHS) {
    el_vp_rhs<DIM>(cc, a.phys, oc.gs, oc.wdet, ye);
  } else if constexpr (OP == K_PP_RHS) {
    el_pp_rhs<DIM>(cc, a.phys, oc.gs, oc.wdet, ye);
  } else if constexpr (OP == K_VU_RHS) {
    el_vu_rhs<DIM>(cc, a.phys, oc.gs, oc.wdet, ye);
  } else {
    el_energy<DIM>(cc, a.phys, oc.gs, oc.wdet, ye);
  }
}

// Table meshes, every field of node entry e in two passes: first one load
// per field with no branch (a hanging node reads node 0 as a placeholder),
// so that all of them are in flight together; then, only in waves that
// hold a hanging node, its fields replaced by the mean of its parents
// (edge: (a + b) / 2, face: ((a + b) + (c + d)) / 4).
template <int DIM, typename T, int OP>
__device__ __forceinline__ void table_first(const BrickArgs<T>& a, int32_t e, T* v) {
  using TR = Traits<OP, DIM>;
  const int32_t i = e >= 0 ? e : 0;
#pragma unroll
  for (int f = 0; f < TR::NI + TR::NCF; ++f)
    v[f] = OP == K_DIAG && f == 0 ? T(e)
           : f < TR::NI           ? fetch<T, TR::MASK>(a.x + f * a.n, a.wall, i)
                                  : a.cf[f - TR::NI][i];
}
template <int DIM, typename T, int OP>
__device__ __forceinline__ void table_parents(const BrickArgs<T>& a, int32_t e, T* v) {
  using TR = Traits<OP, DIM>;
  const int32_t* hp = a.hang + 4 * (int64_t)(-e - 1);
  const int32_t p0 = hp[0], p1 = hp[1], p2 = hp[2], p3 = hp[3];
  const bool four = p2 >= 0;
  const int32_t q2 = four ? p2 : p0, q3 = four ? p3 : p1;
#pragma unroll
  for (int f = OP == K_DIAG ? 1 : 0; f < TR::NI + TR::NCF; ++f) {
    T v0, v1, v2, v3;
    if (f < TR::NI) {
      const T* src = a.x + f * a.n;
      v0 = fetch<T, TR::MASK>(src, a.wall, p0);
      v1 = fetch<T, TR::MASK>(src, a.wall, p1);
      v2 = fetch<T, TR::MASK>(src, a.wall, q2);
      v3 = fetch<T, TR::MASK>(src, a.wall, q3);
    } else {
      const T* src = a.cf[f - TR::NI];
      v0 = src[p0];
      v1 = src[p1];
      v2 = src[q2];
      v3 = src[q3];
    }
    const T s01 = v0 + v1;
    v[f] = four ? (s01 + (v2 + v3)) * T(0.25) : s01 * T(0.5);
  }
}

// One wavefront = BPB bricks; one lane = one leaf column of a brick, marching
// along the last axis.  WHOLE: every node of the brick is gathered into LDS
// up front (all loads in flight together); otherwise a three-layer LDS ring
// is refilled from registers two layers ahead.  STRUCT: uniform mesh with
// lexicographic node numbers, 32-bit offsets computed from the brick anchor.
// The layer march is unrolled for the small scalar forms (pressure, mass):
// ring slots, carries and node offsets become constants.
template <int DIM, int B, typename T, int OP, bool WHOLE>
struct BrickShm {
  using TR = Traits<OP, DIM>;
  static constexpr int NV = TR::NI + TR::NCF;
  static constexpr int LPB = DIM == 3 ? B * B : B;  // lanes (leaf columns) per brick
  static constexpr int BPB = 64 / LPB;              // bricks per wavefront
  static constexpr int NL = DIM == 3 ? (B + 1) * (B + 1) : (B + 1);  // nodes per layer
  static constexpr int NH = (1 << DIM) / 2;
  // heavy forms read corners from LDS on demand; a two-layer ring suffices
  // for them (the layer two ahead is stored after the barrier that ends the
  // reads of the layer it replaces) and leaves LDS for two waves per SIMD
  static constexpr bool HEAVY = OP == K_VP || OP == K_CH_JAC;
  static constexpr int RING = WHOLE ? B + 1 : (HEAVY ? 2 : 3);
  using Lay = T[RING][BPB][NV][NL];
  // per-corner-type leaf contributions, indexed by the node they land on
  // (zero where no leaf of the brick lands): a node sums NH entries
  using Acc = T[BPB][TR::NO][NH][NL];
  static constexpr size_t kBytes = sizeof(Lay) + sizeof(Acc);
};
// Pointer to the first of an LDS array's elements.  The bricks reach their LDS
// by pointers that say it is LDS: by plain references, kept in the closures of
// the body's lambdas, the compiler holds the reads of the layers back behind
// the stores of the contributions and spills more (velocity-update right-hand
// side at 8^3 40.4 us against 35.5, momentum apply 20.4 against 16.1).
template <class A>
using LdsPtr = __attribute__((address_space(3))) std::remove_extent_t<A>*;
// two objects: registers for a third wave of the Cahn-Hilliard Jacobian on
// table bricks
template <class SH>
struct TwoLds {
  __device__ __forceinline__ static auto lay() {
    __shared__ typename SH::Lay m;
    return (LdsPtr<typename SH::Lay>)m;
  }
  __device__ __forceinline__ static auto acc() {
    __shared__ typename SH::Acc m;
    return (LdsPtr<typename SH::Acc>)m;
  }
};
// one object of N bytes: for the momentum form on 8^3 bricks, which spills 8
// bytes a lane less so (437 us against 432 on the 6-9 octree), and for the
// kernels that run whichever class a block belongs to (two objects, each as
// large as the class that needs most of it, would cost the shifted pressure
// form a wave)
template <size_t N>
__device__ __forceinline__ auto lds_bytes() {
  using Bytes = unsigned char[N];
  __shared__ __align__(16) Bytes m;
  return (LdsPtr<Bytes>)m;
}
template <class SH, size_t N = SH::kBytes>
struct OneLds {
  __device__ __forceinline__ static auto lay() { return (LdsPtr<typename SH::Lay>)lds_bytes<N>(); }
  __device__ __forceinline__ static auto acc() {
    return (LdsPtr<typename SH::Acc>)(lds_bytes<N>() + sizeof(typename SH::Lay));
  }
};

template <int DIM, int B, typename T, int OP, bool WHOLE, bool STRUCT, class LDS>
__device__ __forceinline__ void brick_body(const BrickArgs<T>& a, uint32_t block, uint32_t grid) {
  using TR = Traits<OP, DIM>;
  using SH = BrickShm<DIM, B, T, OP, WHOLE>;
  constexpr int NI = TR::NI, NCF = TR::NCF, NO = TR::NO, NV = NI + NCF;
  constexpr int NIa = NI > 0 ? NI : 1, NCa = NCF > 0 ? NCF : 1;
  constexpr int LPB = SH::LPB, BPB = SH::BPB, NL = SH::NL;
  constexpr int KL = (NL + LPB - 1) / LPB;   // layer nodes handled per lane
  constexpr int NC = 1 << DIM, NH = NC / 2;
  constexpr bool HEAVY = SH::HEAVY;
  constexpr int RING = SH::RING;
  // the 3D pressure form keeps its lower layer transformed (march.h)
  constexpr bool MARCH = OP == K_PP && DIM == 3;
  auto* const lay = LDS::lay();
  auto* const accn = LDS::acc();
  if (a.done && *a.done) return;
  const int lane = threadIdx.x, bl = lane / LPB, ll = lane % LPB;
  const int64_t brick = (int64_t)xcd_block(block, grid) * BPB + bl;
  const bool active = brick < a.count;
  const int ix = ll % B, iy = DIM == 3 ? ll / B : 0;
  const int32_t* tab = a.table + (active ? brick : 0) * (int64_t)(NL * (B + 1));
  const int lev = active ? a.level[brick] : 0;
  int32_t base = 0;
  int32_t ax = 0, ay = 0, az = 0;
  if constexpr (STRUCT) {
    if (active) {
      ax = a.anchor[3 * brick];
      ay = a.anchor[3 * brick + 1];
      az = a.anchor[3 * brick + 2];
    }
    base = DIM == 3 ? ax + ay * (int32_t)a.sy + az * (int32_t)a.sz : ax + ay * (int32_t)a.sy;
  }
  // 8^3 bricks of a blocked node order whose numbers follow their 2x2x2
  // point blocks: node (jx, jy, z) is the base of its block plus its
  // lexicographic place in the block (the host checked this against the
  // table); the brick is one wavefront, so the choice is uniform.  Used by
  // the pressure and momentum forms only: in the others the extra registers
  // cost more (spills under the four-wave cap, a wave less for the CH
  // Jacobian) than the table loads they save
  constexpr bool AFF = !STRUCT && DIM == 3 && B == 8 && (OP == K_PP || OP == K_VP);
  int32_t ab[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  bool affine = false;
  if constexpr (AFF) {
    if (a.abase && active) {
      const int32_t* q = a.abase + brick * 8;
#pragma unroll
      for (int i = 0; i < 8; ++i) ab[i] = q[i];
      affine = ab[0] >= 0;
    }
  }
  auto affine_id = [&](int z, int p) -> int32_t {
    const int jx = p % (B + 1), jy = p / (B + 1);
    const bool zb = (z >> 3) != 0, yb = (jy >> 3) != 0, xb = (jx >> 3) != 0;
    const int32_t b0 = zb ? ab[4] : ab[0], b1 = zb ? ab[5] : ab[1], b2 = zb ? ab[6] : ab[2], b3 = zb ? ab[7] : ab[3];
    const int32_t bb = yb ? (xb ? b3 : b2) : (xb ? b1 : b0);
    return bb + (jx & 7) + 8 * (jy & 7) + 64 * (z & 7);
  };
  // index of layer-z node p (STRUCT) or its table entry
  auto entry = [&](int z, int p) -> int64_t {
    if constexpr (STRUCT) {
      const int jx = p % (B + 1), jy = DIM == 3 ? p / (B + 1) : 0;
      return DIM == 3 ? base + jx + jy * (int32_t)a.sy + z * (int32_t)a.sz : base + jx + z * (int32_t)a.sy;
    } else {
      if constexpr (AFF) {
        if (affine) return affine_id(z, p);
      }
      return tab[z * NL + p];
    }
  };
  auto on_wall = [&](int z, int p) -> bool {
    const int jx = p % (B + 1), jy = DIM == 3 ? p / (B + 1) : 0;
    const int cx = ax + jx, cy = DIM == 3 ? ay + jy : ay + z, cz = az + z;
    return cx == 0 || cx == a.side || cy == 0 || cy == a.side || (DIM == 3 && (cz == 0 || cz == a.side));
  };
  // structured meshes: field f of the node with index e at layer z, layer
  // position p (inputs read as zero on the walls when MASK)
  auto value = [&](int f, int64_t e, int z, int p) -> T {
    if (f < NI) {
      if constexpr (TR::MASK) {
        if (on_wall(z, p)) return T(0);
      }
      return (a.x + f * a.n)[(int32_t)e];
    }
    return a.cf[f - NI][(int32_t)e];
  };
  auto table_vals = [&](int32_t e, T* v) { table_first<DIM, T, OP>(a, e, v); };
  auto table_hang = [&](int32_t e, T* v) { table_parents<DIM, T, OP>(a, e, v); };
  const OpConst<T> oc = op_const<DIM, T, OP>(a, lev);

  // -------- layered pipeline state (entries three layers ahead, values two)
  int64_t ent[KL];
  T val[KL][NV];
  // table meshes read the node entries one layer ahead of the values;
  // structured meshes compute them where they are used
  auto load_entries = [&](int z) {
    if constexpr (!STRUCT) {
#pragma unroll
      for (int k = 0; k < KL; ++k) {
        const int p = ll + k * LPB;
        ent[k] = (active && z <= B && p < NL) ? entry(z, p) : 0;
      }
    }
  };
  auto gather_vals = [&](int z) {
    if constexpr (STRUCT) {
#pragma unroll
      for (int k = 0; k < KL; ++k) {
        const int p = ll + k * LPB;
        if (active && z <= B && p < NL) {
          const int64_t e = entry(z, p);
#pragma unroll
          for (int f = 0; f < NV; ++f) val[k][f] = value(f, e, z, p);
        }
      }
    } else {
#pragma unroll
      for (int k = 0; k < KL; ++k) {
        const int p = ll + k * LPB;
        if (active && z <= B && p < NL) table_vals((int32_t)ent[k], val[k]);
      }
#pragma unroll
      for (int k = 0; k < KL; ++k) {
        const int p = ll + k * LPB;
        if (active && z <= B && p < NL && ent[k] < 0) table_hang((int32_t)ent[k], val[k]);
      }
    }
  };
  auto store_vals = [&](int z) {
    if (!active || z > B) return;
    const int buf = z % RING;
#pragma unroll
    for (int k = 0; k < KL; ++k) {
      const int p = ll + k * LPB;
      if (p < NL)
#pragma unroll
        for (int f = 0; f < NV; ++f) lay[buf][bl][f][p] = val[k][f];
    }
  };

  double dot = 0.0;
  int64_t eo[KL];  // node indices of the layer being emitted (table meshes)
  auto load_emit_entries = [&](int z) {
    if constexpr (!STRUCT) {
#pragma unroll
      for (int k = 0; k < KL; ++k) {
        const int p = ll + k * LPB;
        eo[k] = (active && p < NL) ? entry(z, p) : 0;
      }
    }
  };
  auto emit_layer = [&](int z) {
    if (!active) return;
    const int buf = z % RING;
#pragma unroll
    for (int k = 0; k < KL; ++k) {
      const int p = ll + k * LPB;
      if (p >= NL) continue;
      const int jx = p % (B + 1), jy = DIM == 3 ? p / (B + 1) : 0;
      T v[NO];
#pragma unroll
      for (int f = 0; f < NO; ++f) {
        T t = accn[bl][f][0][p];
#pragma unroll
        for (int cl = 1; cl < NH; ++cl) t += accn[bl][f][cl][p];
        v[f] = t;
      }
      const bool interior = jx > 0 && jx < B && (DIM == 2 || (jy > 0 && jy < B)) && z > 0 && z < B;
      if (interior) {
        int64_t e;
        if constexpr (STRUCT) e = entry(z, p);
        else e = eo[k];
        if constexpr (OP == K_PP || OP == K_PPS || OP == K_VPS) {
          if (a.sm_r) v[0] = lay[buf][bl][0][p] + a.sm_w * a.sm_d[e] * (a.sm_r[e] - v[0]);
        }
#pragma unroll
        for (int f = 0; f < NO; ++f) {
          a.y[f * a.n + e] = v[f];
          if constexpr (NI == NO && !HEAVY) {
            if (a.partials) dot += (double)lay[buf][bl][f][p] * (double)v[f];
          }
        }
      } else {
        const int64_t sl = a.slot_base + brick * a.nbnd + brick_rank(DIM, B, jx, jy, z);
#pragma unroll
        for (int f = 0; f < NO; ++f) a.slots[f * a.n_slots + sl] = v[f];
      }
    }
  };

  T carry[NO][NH];
#pragma unroll
  for (int f = 0; f < NO; ++f)
#pragma unroll
    for (int c = 0; c < NH; ++c) carry[f][c] = T(0);

  if (active) {
#pragma unroll
    for (int k = 0; k < KL; ++k) {
      const int p = ll + k * LPB;
      if (p < NL)
#pragma unroll
        for (int f = 0; f < NO; ++f)
#pragma unroll
          for (int cl = 0; cl < NH; ++cl) accn[bl][f][cl][p] = T(0);
    }
  }
  if constexpr (WHOLE) {
    // every node of the brick: all loads issued before the first wait
    constexpr int NPB = NL * (B + 1);
    constexpr int KW = (NPB + LPB - 1) / LPB;
    if (active) {
      T w[KW][NV];
      if constexpr (STRUCT) {
#pragma unroll
        for (int k = 0; k < KW; ++k) {
          const int q = ll + k * LPB;
          if (q < NPB) {
            const int z = q / NL, p = q % NL;
            const int64_t e = entry(z, p);
#pragma unroll
            for (int f = 0; f < NV; ++f) w[k][f] = value(f, e, z, p);
          }
        }
      } else {
        int32_t ew[KW];
#pragma unroll
        for (int k = 0; k < KW; ++k) {
          const int q = ll + k * LPB;
          ew[k] = q < NPB ? tab[q] : 0;
        }
#pragma unroll
        for (int k = 0; k < KW; ++k)
          if (ll + k * LPB < NPB) table_vals(ew[k], w[k]);
#pragma unroll
        for (int k = 0; k < KW; ++k)
          if (ll + k * LPB < NPB && ew[k] < 0) table_hang(ew[k], w[k]);
      }
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        const int q = ll + k * LPB;
        if (q < NPB)
#pragma unroll
          for (int f = 0; f < NV; ++f) lay[q / NL][bl][f][q % NL] = w[k][f];
      }
    }
  } else {
    // prologue: layers 0 and 1 into LDS, layer 2 in flight, entries of layer 3
    load_entries(0);
    gather_vals(0);
    store_vals(0);
    load_entries(1);
    gather_vals(1);
    store_vals(1);
    load_entries(2);
    gather_vals(2);
    load_entries(3);
  }
  __syncthreads();
  // corner values of the upper node layer of one leaf layer are the lower
  // corners of the next: keep them in registers and read only the new layer
  T xc[NIa][NC], cc[NCa][NC];
  auto read_half = [&](int z, int half) {
#pragma unroll
    for (int c = 0; c < NH; ++c) {
      const int bx = c & 1, by = DIM == 3 ? (c >> 1) & 1 : 0;
      const int p = (ix + bx) + (DIM == 3 ? (iy + by) * (B + 1) : 0);
      const int buf = z % RING;
#pragma unroll
      for (int f = 0; f < NI; ++f) xc[f][c + half * NH] = lay[buf][bl][f][p];
#pragma unroll
      for (int f = 0; f < NCF; ++f) cc[f][c + half * NH] = lay[buf][bl][NI + f][p];
    }
  };
  march::PpMarch<T> M;
  march::PpCoef<T> pc{};
  if constexpr (MARCH) {
    pc = march::pp_coef3<T>(a.ratio, lev, march::pp_joint(a.ratio));
    if (active) {
      read_half(0, 1);
      M.start(xc[0] + NH, cc[0] + NH);
    }
  } else if constexpr (!HEAVY) {
    if (active) read_half(0, 1);
  }
  constexpr int kUnroll = (OP == K_PP || OP == K_PPS || OP == K_VPS || OP == K_MASS) ? B : 1;
#pragma unroll kUnroll
  for (int ez = 0; ez < B; ++ez) {
    load_emit_entries(ez);
    if (active) {
      T ye[NO][NC];
      if constexpr (MARCH) {
        read_half(ez + 1, 1);
        M.step(xc[0] + NH, cc[0] + NH, pc, ye[0], [] {});
      } else if constexpr (!HEAVY) {
#pragma unroll
        for (int c = 0; c < NH; ++c) {
#pragma unroll
          for (int f = 0; f < NI; ++f) xc[f][c] = xc[f][c + NH];
#pragma unroll
          for (int f = 0; f < NCF; ++f) cc[f][c] = cc[f][c + NH];
        }
        read_half(ez + 1, 1);
      }
      // corner a of field f (inputs first, then coefficients) from LDS
      auto cv = [&](int f, int ca) -> T {
        const int bx = ca & 1, by = DIM == 3 ? (ca >> 1) & 1 : 0, bz = (ca >> (DIM - 1)) & 1;
        const int p = (ix + bx) + (DIM == 3 ? (iy + by) * (B + 1) : 0);
        return lay[(ez + bz) % RING][bl][f][p];
      };
      if constexpr (OP == K_VP) {
        // each component's corner values go to the node accumulators as
        // soon as they are formed
        el_vp<DIM, T>(cv, a.fc, lev, [&](int f, const T* yf) {
#pragma unroll
          for (int c = 0; c < NH; ++c) {
            const int p = (ix + (c & 1)) + (DIM == 3 ? (iy + ((c >> 1) & 1)) * (B + 1) : 0);
            accn[bl][f][c][p] = yf[c] + carry[f][c];
            carry[f][c] = yf[c + NH];
          }
        });
      } else {
        // the right-hand sides are called here: through leaf_form the compiler
        // allocates their registers otherwise (pressure at 128^3 1,474 us,
        // here 1,412; velocity update on the 5-9 octree 3.50 ms, here 3.32)
        if constexpr (OP == K_VP_RHS) el_vp_rhs<DIM>(cc, a.phys, oc.gs, oc.wdet, ye);
        else if constexpr (OP == K_PP_RHS) el_pp_rhs<DIM>(cc, a.phys, oc.gs, oc.wdet, ye);
        else if constexpr (OP == K_VU_RHS) el_vu_rhs<DIM>(cc, a.phys, oc.gs, oc.wdet, ye);
        else if constexpr (!MARCH) leaf_form<DIM, T, OP>(a, oc, lev, xc, cc, cv, ye);
#pragma unroll
        for (int f = 0; f < NO; ++f)
#pragma unroll
          for (int c = 0; c < NH; ++c) {
            const int p = (ix + (c & 1)) + (DIM == 3 ? (iy + ((c >> 1) & 1)) * (B + 1) : 0);
            if constexpr (MARCH) {
              accn[bl][f][c][p] = ye[f][c];
            } else {
              accn[bl][f][c][p] = ye[f][c] + carry[f][c];
              carry[f][c] = ye[f][c + NH];
            }
          }
      }
    }
    __syncthreads();
    // values of layer ez + 2 (loads in flight since the previous layer) go to
    // LDS before this layer's outputs are stored: waiting for those loads
    // then does not also wait for the stores
    if constexpr (!WHOLE) store_vals(ez + 2);
    emit_layer(ez);
    if constexpr (!WHOLE) {
      gather_vals(ez + 3);
      load_entries(ez + 4);
    }
    __syncthreads();
  }
  load_emit_entries(B);
  if (active) {
    if constexpr (MARCH) M.finish(carry[0]);
#pragma unroll
    for (int f = 0; f < NO; ++f)
#pragma unroll
      for (int c = 0; c < NH; ++c) {
        const int p = (ix + (c & 1)) + (DIM == 3 ? (iy + ((c >> 1) & 1)) * (B + 1) : 0);
        accn[bl][f][c][p] = carry[f][c];
      }
  }
  __syncthreads();
  emit_layer(B);
  if (a.partials) {
    dot = wave_sum(dot);
    if (lane == 0) a.partials[block] = dot;
  }
}

// Uniform, lexicographically numbered 2D meshes: every form in one kernel,
// without shared-node slots and the combine pass.  These meshes are small
// (4,225 nodes at 64 x 64) and a form's time is its launches and one chain of
// dependent loads, so a second launch costs more than the leaves that two
// waves compute twice here.
//
// A wave walks 64 leaf columns up a chunk of `own` node rows.  A lane
// completes the nodes on its leaf's right side with the left-hand sums of the
// next lane; the wave's last column is computed by the next wave as well
// (64 columns give 63 nodes; the first wave also owns x = 0, the last the
// right wall), and a chunk starts one leaf row below its first node row.
constexpr int kTile2X = 63;
template <typename T, int OP>
__global__ __launch_bounds__(64) void k_tile2(BrickArgs<T> a, int tx, int own) {
  using TR = Traits<OP, 2>;
  constexpr int NI = TR::NI, NCF = TR::NCF, NO = TR::NO, NV = NI + NCF;
  constexpr int NIa = NI > 0 ? NI : 1, NCa = NCF > 0 ? NCF : 1;
  constexpr bool HEAVY = OP == K_VP || OP == K_CH_JAC;
  if (a.done && *a.done) return;
  const int lane = threadIdx.x, t = blockIdx.x % tx;
  const int S = a.side;
  const int64_t sy = S + 1;
  const int cx = kTile2X * t + lane, q = min(cx, S - 1);
  const bool leaf = cx < S;
  const bool owner = leaf && (lane < kTile2X || cx == S - 1);
  const int z0 = (int)(blockIdx.x / tx) * own, z1 = min(z0 + own, S + 1);
  const int zb = max(z0 - 1, 0), ze = min(z1, S);
  int lev = 0;
  while ((1 << lev) < S) ++lev;
  const OpConst<T> oc = op_const<2, T, OP>(a, lev);
  auto on_wall = [&](int x, int z) { return x == 0 || x == S || z == 0 || z == S; };
  // the two nodes of the lane's column in row z, wall nodes of a masked
  // input read as zero
  auto load = [&](int z, T (*v)[2]) {
    const int64_t i = z * sy + q;
#pragma unroll
    for (int f = 0; f < NV; ++f) {
      const T* src = f < NI ? a.x + f * a.n : a.cf[f < NI ? 0 : f - NI];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        v[f][c] = src[i + c];
        if (f < NI && TR::MASK && on_wall(q + c, z)) v[f][c] = T(0);
      }
    }
  };
  double dot = 0.0;
  auto put = [&](int x, int z, const T* v) {
    const int64_t i = z * sy + x;
#pragma unroll
    for (int f = 0; f < NO; ++f) {
      T w = v[f], xo = T(0);
      if constexpr (NI == NO) {
        if (TR::WALL == 1 || a.sm_r || a.partials) xo = (a.x + f * a.n)[i];
      }
      if (TR::WALL == 1 && on_wall(x, z)) w = xo;
      if (TR::WALL == 2 && on_wall(x, z)) w = T(0);
      if constexpr (OP == K_PP || OP == K_PPS || OP == K_VPS) {
        if (a.sm_r) w = xo + a.sm_w * a.sm_d[i] * (a.sm_r[i] - w);
      }
      (a.y + f * a.n)[i] = w;
      if constexpr (NI == NO && !HEAVY) {
        if (a.partials) dot += (double)xo * (double)w;
      }
    }
  };
  T carry[NO][2], r[NO][2];
  auto emit = [&](int z) {
    T v[NO], l[NO];
#pragma unroll
    for (int f = 0; f < NO; ++f) {
      l[f] = leaf ? r[f][0] : T(0);
      const T next = __shfl_down(l[f], 1, 64);
      v[f] = r[f][1] + (lane < 63 ? next : T(0));
    }
    if (owner) put(cx + 1, z, v);
    if (cx == 0) put(0, z, l);
  };
  T lo[NV][2], hi[NV][2];
  load(zb, lo);
  load(zb + 1, hi);
#pragma unroll
  for (int f = 0; f < NO; ++f) carry[f][0] = carry[f][1] = T(0);
  for (int z = zb; z < ze; ++z) {
    T xc[NIa][4], cc[NCa][4], ye[NO][4];
#pragma unroll
    for (int f = 0; f < NV; ++f)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        if (f < NI) {
          xc[f < NI ? f : 0][c] = lo[f][c];
          xc[f < NI ? f : 0][c + 2] = hi[f][c];
        } else {
          cc[f < NI ? 0 : f - NI][c] = lo[f][c];
          cc[f < NI ? 0 : f - NI][c + 2] = hi[f][c];
        }
        lo[f][c] = hi[f][c];
      }
    if (z + 1 < ze) load(z + 2, hi);
    auto cv = [&](int f, int ca) -> T { return f < NI ? xc[f < NI ? f : 0][ca] : cc[f < NI ? 0 : f - NI][ca]; };
    if constexpr (OP == K_VP) {
      el_vp<2, T>(cv, a.fc, lev, [&](int f, const T* yf) {
#pragma unroll
        for (int c = 0; c < 4; ++c) ye[f][c] = yf[c];
      });
    } else {
      leaf_form<2, T, OP>(a, oc, lev, xc, cc, cv, ye);
    }
#pragma unroll
    for (int f = 0; f < NO; ++f)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        r[f][c] = ye[f][c] + carry[f][c];
        carry[f][c] = ye[f][c + 2];
      }
    if (z >= z0) emit(z);
  }
  if (z1 == S + 1) {
#pragma unroll
    for (int f = 0; f < NO; ++f)
#pragma unroll
      for (int c = 0; c < 2; ++c) r[f][c] = carry[f][c];
    emit(S);
  }
  if (a.partials) {
    dot = wave_sum(dot);
    if (lane == 0) a.partials[blockIdx.x] = dot;
  }
}

template <int DIM, int B, typename T, int OP>
constexpr bool whole_fits() {
  using TR = Traits<OP, DIM>;
  constexpr int LPB = DIM == 3 ? B * B : B;
  constexpr int NL = DIM == 3 ? (B + 1) * (B + 1) : (B + 1);
  // deep bricks keep the three-layer ring (better occupancy, loads pipelined)
  return B <= 4 && (64 / LPB) * NL * (B + 1) * (TR::NI + TR::NCF) * (int)sizeof(T) <= 12 * 1024;
}
template <int DIM, int B, typename T, int OP>
using ShmOf = BrickShm<DIM, B, T, OP, whole_fits<DIM, B, T, OP>()>;

template <int DIM, int B, typename T, int OP, bool STRUCT>
__global__ __launch_bounds__(64) void k_brick(BrickArgs<T> a) {
  using SH = ShmOf<DIM, B, T, OP>;
  brick_body<DIM, B, T, OP, whole_fits<DIM, B, T, OP>(), STRUCT, TwoLds<SH>>(a, blockIdx.x, gridDim.x);
}
// the pressure forms (at most 128 VGPRs in FP64): capped at four waves per
// SIMD, which keeps the FP32 instances from trading their latency hiding for
// occupancy.  The mass form on uniform meshes (60 VGPRs) is bound by memory and
// runs uncapped: apply at 256^3 187 us FP64 and 135 FP32, against 224 and 162
// with the cap (equal at 128^3)
template <int DIM, int B, typename T, int OP, bool STRUCT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_brick_o4(BrickArgs<T> a) {
  using SH = ShmOf<DIM, B, T, OP>;
  brick_body<DIM, B, T, OP, whole_fits<DIM, B, T, OP>(), STRUCT, TwoLds<SH>>(a, blockIdx.x, gridDim.x);
}
// two FP64 3D forms on 8^3 bricks.  The Cahn-Hilliard Jacobian on structured
// bricks: its LDS admits three waves per SIMD, which at 128^3 leaves a third
// of the bricks to a second, sparse round; held to two waves it runs two full
// rounds (0.095 -> 0.090 ms; equal at 256^3; on adaptive meshes three are
// faster).  The momentum form: a chain of dependent FMAs and reciprocals
// bounds it, and left alone the compiler takes more than 256 registers and
// one wave per SIMD; held to two it spills 8 bytes a lane on structured
// bricks and 84 on table bricks and still gains, 192 -> 164 us at 128^3 and
// 461 -> 426 us on the 5-9 octree
template <int DIM, int B, typename T, int OP, bool STRUCT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_brick_o2(BrickArgs<T> a) {
  using SH = ShmOf<DIM, B, T, OP>;
  using LDS = std::conditional_t<OP == K_VP, OneLds<SH>, TwoLds<SH>>;
  brick_body<DIM, B, T, OP, whole_fits<DIM, B, T, OP>(), STRUCT, LDS>(a, blockIdx.x, gridDim.x);
}

// Single leaves (bricks of one) of a table mesh: one lane per leaf, its
// corners in registers, its results straight to its slots; no LDS.
template <int DIM, typename T, int OP>
__device__ __forceinline__ void single_body(const BrickArgs<T>& a, uint32_t block, uint32_t grid) {
  using TR = Traits<OP, DIM>;
  constexpr int NI = TR::NI, NCF = TR::NCF, NO = TR::NO, NV = NI + NCF;
  constexpr int NIa = NI > 0 ? NI : 1, NCa = NCF > 0 ? NCF : 1, NC = 1 << DIM;
  const int64_t leaf = (int64_t)xcd_block(block, grid) * 64 + threadIdx.x;
  // every node of a single leaf goes through the combine: no fused dot here
  if (a.partials && threadIdx.x == 0) a.partials[block] = 0.0;
  if (leaf >= a.count) return;
  const int lev = a.level[leaf];
  int32_t e[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) e[c] = a.table[leaf * NC + c];
  T v[NC][NV];
#pragma unroll
  for (int c = 0; c < NC; ++c) table_first<DIM, T, OP>(a, e[c], v[c]);
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (e[c] < 0) table_parents<DIM, T, OP>(a, e[c], v[c]);
  T xc[NIa][NC], cc[NCa][NC], ye[NO][NC];
#pragma unroll
  for (int f = 0; f < NV; ++f)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (f < NI) xc[f < NI ? f : 0][c] = v[c][f];
      else cc[f < NI ? 0 : f - NI][c] = v[c][f];
    }
  if constexpr (OP == K_PP && DIM == 3) {
    march::PpMarch<T> M;
    M.start(xc[0], cc[0]);
    M.step(xc[0] + 4, cc[0] + 4, march::pp_coef3<T>(a.ratio, lev, march::pp_joint(a.ratio)), ye[0], [] {});
    M.finish(ye[0] + 4);
  } else {
    auto cv = [&](int f, int ca) -> T { return f < NI ? xc[f < NI ? f : 0][ca] : cc[f < NI ? 0 : f - NI][ca]; };
    if constexpr (OP == K_VP) {
      el_vp<DIM, T>(cv, a.fc, lev, [&](int f, const T* yf) {
#pragma unroll
        for (int c = 0; c < NC; ++c) ye[f][c] = yf[c];
      });
    } else {
      leaf_form<DIM, T, OP>(a, op_const<DIM, T, OP>(a, lev), lev, xc, cc, cv, ye);
    }
  }
#pragma unroll
  for (int f = 0; f < NO; ++f)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int64_t sl = a.slot_base + leaf * a.nbnd + brick_rank(DIM, 1, c & 1, DIM == 3 ? (c >> 1) & 1 : 0, c >> (DIM - 1));
      a.slots[f * a.n_slots + sl] = ye[f][c];
    }
}

// Table meshes: every brick class in one launch, the largest bricks first.
// An octree around an interface has a few thousand waves of each class or
// less (levels 5-8: 1,248 of 4^3, 600 of 2^3 and 156 of single leaves for
// 1,024 SIMDs), so launched one after another each leaves most of the chip
// idle and its own tail exposed.  Each class starts at a multiple of eight
// blocks, which keeps its XCD order.  Four launches -> one: FP32 pressure
// apply at levels 5-9 82.8 -> 57.1 us, multigrid solve at levels 5-8 10.25 ->
// 7.97 ms, rising-bubble step at levels 5-8 212 -> 161 ms.
struct ClassArgs {
  const int32_t* table;
  const int32_t* abase;
  const int8_t* level;
  int64_t count, slot_base;
  int nbnd;
  uint32_t first, grid;  // its blocks
};
struct ClassTable {
  ClassArgs c[kBrickClasses];  // edge 8, 4, 2, 1
};
template <int DIM, typename T, int OP, bool EIGHT>
__device__ __forceinline__ void bricks_body(BrickArgs<T> a, const ClassTable& t) {
  constexpr size_t kShm = std::max({EIGHT ? ShmOf<DIM, 8, T, OP>::kBytes : 0, ShmOf<DIM, 4, T, OP>::kBytes,
                                    ShmOf<DIM, 2, T, OP>::kBytes});
  if (a.done && *a.done) return;
  const uint32_t b = blockIdx.x;
  auto take = [&](int k) {
    const ClassArgs& c = t.c[k];
    a.table = c.table;
    a.abase = c.abase;
    a.level = c.level;
    a.count = c.count;
    a.slot_base = c.slot_base;
    a.nbnd = c.nbnd;
    if (a.partials) a.partials += c.first;
    return b - c.first;
  };
  if (EIGHT && b < t.c[0].first + t.c[0].grid) {
    if constexpr (EIGHT) {
      const uint32_t i = take(0);
      brick_body<DIM, 8, T, OP, whole_fits<DIM, 8, T, OP>(), false,
                  OneLds<ShmOf<DIM, 8, T, OP>, kShm>>(a, i, t.c[0].grid);
    }
  } else if (b < t.c[1].first + t.c[1].grid) {
    const uint32_t i = take(1);
    brick_body<DIM, 4, T, OP, whole_fits<DIM, 4, T, OP>(), false,
                OneLds<ShmOf<DIM, 4, T, OP>, kShm>>(a, i, t.c[1].grid);
  } else if (b < t.c[2].first + t.c[2].grid) {
    const uint32_t i = take(2);
    brick_body<DIM, 2, T, OP, whole_fits<DIM, 2, T, OP>(), false,
                OneLds<ShmOf<DIM, 2, T, OP>, kShm>>(a, i, t.c[2].grid);
  } else {
    const uint32_t i = take(3);
    single_body<DIM, T, OP>(a, i, t.c[3].grid);
  }
}
template <int DIM, typename T, int OP, bool EIGHT>
__global__ __launch_bounds__(64) void k_bricks(BrickArgs<T> a, ClassTable t) {
  bricks_body<DIM, T, OP, EIGHT>(a, t);
}
// the scalar forms that fit 128 VGPRs without spills, as k_brick_o4
template <int DIM, typename T, int OP, bool EIGHT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_bricks_o4(BrickArgs<T> a,
                                                                                             ClassTable t) {
  bricks_body<DIM, T, OP, EIGHT>(a, t);
}

// Block-wide deterministic sum of one double (256 threads).
__device__ double block_sum256(double v, double* sh) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) r = (sh[0] + sh[1]) + (sh[2] + sh[3]);
  __syncthreads();
  return r;
}

template <typename T, int NO, int WALL, bool SQ>
__global__ __launch_bounds__(256) void k_combine(const int32_t* __restrict__ node, const int32_t* __restrict__ ptr,
                                                 const uint32_t* __restrict__ ent, int64_t nrows,
                                                 const T* __restrict__ slots, int64_t n_slots, T* __restrict__ y,
                                                 const T* __restrict__ x, int64_t n, const uint8_t* __restrict__ wall,
                                                 double* partials, const int* done, const T* __restrict__ sm_r,
                                                 const T* __restrict__ sm_d, T sm_w) {
  __shared__ double sh[4];
  if (done && *done) return;
  const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double dot = 0.0;
  if (row < nrows) {
    const int32_t i = node[row];
    const int32_t k0 = ptr[row], k1 = ptr[row + 1];
    // a row's entries and then its slots are loaded CH at a time, every load
    // of a group in flight together (a row holds 2 to 8 entries, more only
    // next to hanging nodes); the sum keeps the entry order
    constexpr int CH = 8;
    T v[NO];
#pragma unroll
    for (int f = 0; f < NO; ++f) v[f] = T(0);
    for (int32_t kb = k0; kb < k1; kb += CH) {
      uint32_t e[CH];
#pragma unroll
      for (int j = 0; j < CH; ++j) e[j] = kb + j < k1 ? ent[kb + j] : 0u;
#pragma unroll
      for (int f = 0; f < NO; ++f) {
        T sv[CH];
#pragma unroll
        for (int j = 0; j < CH; ++j) sv[j] = kb + j < k1 ? slots[f * n_slots + (e[j] & 0x3fffffffu)] : T(0);
#pragma unroll
        for (int j = 0; j < CH; ++j) {
          if (kb + j < k1) {
            const uint32_t code = e[j] >> 30;
            // SQ: squared weights (diagonals)
            v[f] += code == 0 ? sv[j] : (code == 1 ? sv[j] * T(SQ ? 0.25 : 0.5) : sv[j] * T(SQ ? 0.0625 : 0.25));
          }
        }
      }
    }
#pragma unroll
    for (int f = 0; f < NO; ++f) {
      T w = v[f];
      // wall rows: identity (WALL 1) or zero (WALL 2)
      if constexpr (WALL == 1) {
        if (wall[i]) w = x[f * n + i];
      } else if constexpr (WALL == 2) {
        if (wall[i]) w = T(0);
      }
      if (sm_r) w = x[i] + sm_w * sm_d[i] * (sm_r[i] - w);
      y[f * n + i] = w;
      if (partials) dot += (double)x[f * n + i] * (double)w;
    }
  }
  if (!partials) return;
  const double bs = block_sum256(dot, sh);
  if (threadIdx.x == 0) partials[blockIdx.x] = bs;
}

// One block sums the per-block partials of the fused x.y in a fixed order
// (1024 threads, four independent running sums each).
__global__ __launch_bounds__(1024) void k_sum_partials(const double* partials, int n, double* out, const int* done) {
  __shared__ double sh[16];
  if (done && *done) return;
  double v0 = 0.0, v1 = 0.0, v2 = 0.0, v3 = 0.0;
  int k = threadIdx.x;
  for (; k + 3 * 1024 < n; k += 4 * 1024) {
    v0 += partials[k];
    v1 += partials[k + 1024];
    v2 += partials[k + 2048];
    v3 += partials[k + 3072];
  }
  for (; k < n; k += 1024) v0 += partials[k];
  double v = wave_sum((v0 + v1) + (v2 + v3));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int i = 0; i < 16; ++i) t += sh[i];
    *out = t;
  }
}

// Wall rows of masked operators that no brick writes (all go through the
// combine, which handles them); nothing else is needed here.

// FP32 copy of coefficient fields; entries below `shifted` (the phase field
// of the momentum operator) are stored as 1 + value
__global__ void k_coef32(const double* src, float* dst, int64_t n, int64_t shifted) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = (float)(i < shifted ? 1.0 + src[i] : src[i]);
}

// Diagonal probing helpers.
// x = indicator of colour c in field `field` (every field when field < 0)
template <typename T>
__global__ void k_indicator(T* x, const uint8_t* color, int c, int64_t n, int nf, int field) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  T v = color[i] == c ? T(1) : T(0);
  for (int f = 0; f < nf; ++f) x[f * n + i] = (field < 0 || f == field) ? v : T(0);
}
template <typename T>
__global__ void k_take_diag(T* d, const T* y, const uint8_t* color, int c, int64_t n, int nf, int invert,
                            int field) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (color[i] != c) return;
  for (int f = 0; f < nf; ++f) {
    if (field >= 0 && f != field) continue;
    T v = y[f * n + i];
    d[f * n + i] = invert ? (v != T(0) ? T(1) / v : T(1)) : v;
  }
}
// one-pass diagonal: the same for every field, 1 on the walls of an operator
// with identity wall rows (wall != null), inverted on request
__global__ void k_diag_finish(double* d, int64_t n, int nf, const uint8_t* wall, int invert) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double v = wall && wall[i] ? 1.0 : d[i];
  if (invert) v = v != 0.0 ? 1.0 / v : 1.0;
  for (int f = 0; f < nf; ++f) d[f * n + i] = v;
}
__global__ void k_narrow(const double* a, float* b, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    b[i] = (float)a[i];
}
// column `field` of the nf x nf node blocks: blk[(g * nf + field) * n + i] = y_g,i
__global__ void k_take_block(double* blk, const double* y, const uint8_t* color, int c, int64_t n, int nf,
                             int field) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (color[i] != c) return;
  for (int g = 0; g < nf; ++g) blk[(g * nf + field) * n + i] = y[g * n + i];
}

// The uniform-mesh kernels' chunk length: node rows (2D) or layers (3D) a
// block completes.  A chunk costs one leaf row or layer more than it owns, so
// long chunks do less work and short ones fill the chip; `fill` blocks are
// enough (measured minimum of the chunk sweeps at 16 to 256 leaves per edge
// in 3D, where chunks below three layers only pay while the chip is not full).
int chunk_own(int64_t tiles, int side, int64_t fill, int least) {
  if (tiles * (side + 1) <= fill / 3) return 1;
  return (int)std::max<int64_t>(least, (tiles * (side + 1) + fill - 1) / fill);
}

int64_t tile3_columns(int side) {
  return (int64_t)((side + kTileX - 1) / kTileX) * ((side + kTileY - 1) / kTileY);
}
int tile3_own(int side) { return chunk_own(tile3_columns(side), side, 1536, 3); }
// the right-hand sides: every register of a SIMD, so one wave on each of the
// 1,024
template <int OP>
constexpr bool is_rhs() {
  return OP == K_VP_RHS || OP == K_PP_RHS || OP == K_VU_RHS;
}
// 2D: blocks of a right-hand side run in rounds of 1,024, so its chunks are
// those with the fewest rows to march in all rounds, the row below each chunk
// counted (against 6,144 blocks, the pressure's: 256^2 leaves 21.4 -> 16.4 us,
// 512^2 44.6 -> 31.2, 1024^2 110 -> 89, 8192^2 5.26 -> 4.80 ms; the bricks take
// 39.5, 41.1, 86 us and 5.23 ms)
template <int OP>
int tile2_own(int tiles, int side) {
  if (!is_rhs<OP>()) return chunk_own(tiles, side, 6144, 2);
  constexpr int kSlots = 1024, kRounds = 8;
  int best = 1;
  int64_t least = INT64_MAX;
  for (int r = 1; r <= kRounds; ++r) {
    const int chunks = std::min(std::max(1, r * kSlots / tiles), side + 1), own = (side + chunks) / chunks;
    const int64_t blocks = (int64_t)tiles * ((side + own) / own);
    const int64_t rows = (blocks + kSlots - 1) / kSlots * (own + 1);
    if (rows < least) {
      least = rows;
      best = own;
    }
  }
  return best;
}
// ... and on at most 32^2 leaves stays on the bricks: there a wave's two leaf
// rows take longer than one leaf of a brick and the combine (10.3 us against
// 8.4 at 8^2 and 10.4 against 9.4 at 32^2 for the pressure's, 10.4 against 14.0
// at 64^2)
template <int DIM, int OP>
bool rhs_on_bricks(int side) {
  return DIM == 2 && is_rhs<OP>() && side <= 32;
}
// 3D pressure operator on a uniform mesh: arguments of k_pp_tile
template <typename T>
TileArgs<T> tile3_args(const BrickArgs<T>& b, int level, int own) {
  TileArgs<T> t{};
  t.x = b.x;
  t.phi = b.cf[0];
  t.y = b.y;
  t.ratio = b.ratio;
  t.joint = march::pp_joint(b.ratio);
  t.level = level;
  t.sm_r = b.sm_r;
  t.sm_d = b.sm_d;
  t.sm_w = b.sm_w;
  t.partials = b.partials;
  t.done = b.done;
  tile_geometry(t, b.side, own);
  return t;
}

template <int DIM, int B, typename T, int OP, bool STRUCT>
void launch_one(int64_t grid, hipStream_t s, const BrickArgs<T>& a) {
  const dim3 g((unsigned)grid), blk(64);
  // the scalar momentum form (viscous stiffness and density mass together)
  // needs ~130 registers: capped at four waves it spilled (88 bytes per lane
  // on table bricks), uncapped it runs three without
  if constexpr (OP == K_PP || OP == K_PPS) k_brick_o4<DIM, B, T, OP, STRUCT><<<g, blk, 0, s>>>(a);
  else if constexpr (((OP == K_CH_JAC && STRUCT) || OP == K_VP) && DIM == 3 && B == 8 && sizeof(T) == 8)
    k_brick_o2<DIM, B, T, OP, STRUCT><<<g, blk, 0, s>>>(a);
  else k_brick<DIM, B, T, OP, STRUCT><<<g, blk, 0, s>>>(a);
}

// uniform meshes: one brick class, node numbers computed
template <int DIM, typename T, int OP>
void launch_structured(int B, int64_t grid, hipStream_t s, const BrickArgs<T>& a) {
  switch (B) {
    case 8: launch_one<DIM, 8, T, OP, true>(grid, s, a); break;
    case 4: launch_one<DIM, 4, T, OP, true>(grid, s, a); break;
    case 2: launch_one<DIM, 2, T, OP, true>(grid, s, a); break;
    default: launch_one<DIM, 1, T, OP, true>(grid, s, a); break;
  }
}

int64_t class_blocks(const DevBrickClass& bc, int dim) {
  const int bpb = 64 / (dim == 3 ? bc.B * bc.B : bc.B);
  return (bc.count + bpb - 1) / bpb;
}

// the forms of several fields keep their 8^3 bricks in a launch of their own:
// the small bricks' LDS (16 bricks of 2^3 in a wave) would take their waves
template <int OP>
constexpr bool eight_merged() {
  return OP == K_PP || OP == K_PPS || OP == K_VPS || OP == K_MASS || OP == K_DIAG;
}
// blocks that launch_bricks starts (the right-hand sides have no fused dot)
template <int DIM, int OP>
int64_t brick_blocks(const DevMesh& dm) {
  int64_t n = 0;
  for (const DevBrickClass& bc : dm.cls) {
    if (!bc.count) continue;
    const int64_t g = class_blocks(bc, DIM);
    n += dm.structured || (!eight_merged<OP>() && bc.B == 8) ? g : (g + 7) / 8 * 8;
  }
  return n;
}

template <int DIM, typename T, int OP>
int launch_bricks(const DevMesh& dm, BrickArgs<T> a, hipStream_t s, int& part_off) {
  constexpr bool EIGHT = eight_merged<OP>();
  // The 3D right-hand sides, of which the merged kernel holds two waves on a CU
  // (its LDS is that of sixteen 2^3 bricks): 4^3 bricks with a wave for every
  // SIMD run in a kernel of their own (1,827 us against 1,946 for the
  // prediction on the 5-9 octree; with fewer, one launch is faster: 105 us
  // against 139 at levels 4-7), and so do single leaves with no other class
  // beside them (pressure 41.4 us against 45.2 at levels 2-4).
  constexpr bool RHS3 = is_rhs<OP>() && DIM == 3;
  int classes = 0;
  for (const DevBrickClass& bc : dm.cls) classes += bc.count > 0;
  ClassTable t{};
  uint32_t end = 0;
  double* part = a.partials ? a.partials + part_off : nullptr;
  for (int k = 0; k < kBrickClasses; ++k) {
    const DevBrickClass& bc = dm.cls[k];
    const int64_t grid = bc.count ? class_blocks(bc, DIM) : 0;
    a.table = bc.table;
    a.abase = bc.abase;
    a.level = bc.level;
    a.count = bc.count;
    a.slot_base = bc.slot_base;
    a.nbnd = bc.nbnd;
    const bool alone =
        (!EIGHT && bc.B == 8) || (RHS3 && ((bc.B == 4 && grid >= 1024) || (bc.B == 1 && classes == 1)));
    if (dm.structured || alone) {
      if (!grid) continue;
      a.anchor = bc.anchor;
      a.partials = part;
      if constexpr (!EIGHT) {
        if (!dm.structured && bc.B == 8) launch_one<DIM, 8, T, OP, false>(grid, s, a);
      }
      if constexpr (RHS3) {
        if (!dm.structured && bc.B == 4) launch_one<DIM, 4, T, OP, false>(grid, s, a);
        if (!dm.structured && bc.B == 1) launch_one<DIM, 1, T, OP, false>(grid, s, a);
      }
      if constexpr (DIM == 3 ? !(OP == K_PP && sizeof(T) == 8) && OP != K_DIAG : is_rhs<OP>())
        if (dm.structured) launch_structured<DIM, T, OP>(bc.B, grid, s, a);
      CHNS_HIP(hipGetLastError());
      if (part) {
        part += grid;
        part_off += (int)grid;
      }
      continue;
    }
    const int at = bc.B == 8 ? 0 : bc.B == 4 ? 1 : bc.B == 2 ? 2 : 3;
    const uint32_t g = (uint32_t)((grid + 7) / 8 * 8);
    t.c[at] = {bc.table, bc.abase, bc.level, bc.count, bc.slot_base, bc.nbnd, 0, g};
  }
  for (int k = 0; k < kBrickClasses; ++k) {
    t.c[k].first = end;
    end += t.c[k].grid;
  }
  if (!end) return CHNS_OK;
  a.partials = part;
  const dim3 g(end), blk(64);
  if constexpr ((OP == K_PP && sizeof(T) == 4) || OP == K_PPS || OP == K_MASS) k_bricks_o4<DIM, T, OP, EIGHT><<<g, blk, 0, s>>>(a, t);
  else k_bricks<DIM, T, OP, EIGHT><<<g, blk, 0, s>>>(a, t);
  CHNS_HIP(hipGetLastError());
  if (part) part_off += (int)end;
  return CHNS_OK;
}

int64_t combine_blocks(const DevMesh& dm) { return (dm.n_comb + 255) / 256; }

Phys phys_of(const chns_params& p) {
  Phys f{};
  f.dt = p.dt;
  f.Pe = p.Pe;
  f.Cn = p.Cn;
  f.We = p.We;
  f.Re = p.Re;
  f.Fr = p.Fr;
  f.C_I = p.C_I;
  f.alpha = (p.rho_plus - p.rho_minus) / (2.0 * p.rho_plus);
  f.beta = (p.rho_plus + p.rho_minus) / (2.0 * p.rho_plus);
  f.gam = (p.eta_plus - p.eta_minus) / (2.0 * p.eta_plus);
  f.xi = (p.eta_plus + p.eta_minus) / (2.0 * p.eta_plus);
  f.cJ = (p.rho_minus - p.rho_plus) / (2.0 * p.rho_plus * p.Cn);
  f.gaxis = p.gravity_axis;
  return f;
}

const char* op_tag(int op, bool fp64) {
  static const char* tags[13][2] = {{"pp_brick_fp64", "pp_brick_fp32"},
                                    {"mass_brick_fp64", "mass_brick_fp32"},
                                    {"massrho_brick_fp64", "massrho_brick_fp32"},
                                    {"chres_brick_fp64", "chres_brick_fp32"},
                                    {"chjac_brick_fp64", "chjac_brick_fp32"},
                                    {"vp_brick_fp64", "vp_brick_fp32"},
                                    {"vprhs_brick_fp64", "vprhs_brick_fp32"},
                                    {"pprhs_brick_fp64", "pprhs_brick_fp32"},
                                    {"vurhs_brick_fp64", "vurhs_brick_fp32"},
                                    {"energy_brick_fp64", "energy_brick_fp32"},
                                    {"pps_brick_fp64", "pps_brick_fp32"},
                                    {"vps_brick_fp64", "vps_brick_fp32"},
                                    {"diag_brick_fp64", "diag_brick_fp32"}};
  return tags[op][fp64 ? 0 : 1];
}

// cf: the op's NCF coefficient fields (each n long, device)
template <int DIM, typename T, int OP>
int apply_t(Ctx& c, const LevelView& L, const T* x, T* y, const T* const* cf, hipStream_t s, const ApplyOut& o) {
  using TR = Traits<OP, DIM>;
  static_assert(TR::NCF <= kMaxCoef, "too many coefficient fields");
  const DevMesh& dm = *L.dm;
  if (o.fuse_dot && (TR::NI != TR::NO || OP == K_VP || OP == K_CH_JAC)) {
    set_error("fused dot needs as many inputs as outputs and a scalar-form operator");
    return CHNS_EINVAL;
  }
  if (o.sm_r && ((OP != K_PP && OP != K_PPS && OP != K_VPS) || o.fuse_dot || x == y)) {
    set_error("a fused smoothing sweep needs the pressure operator, no fused dot and y distinct from x");
    return CHNS_EINVAL;
  }
  BrickArgs<T> a{};
  a.n = dm.n;
  a.n_slots = dm.n_slots;
  a.x = x;
  for (int k = 0; k < TR::NCF; ++k) a.cf[k] = cf[k];
  a.y = y;
  a.slots = (T*)L.slots;
  a.hang = dm.hang_par;
  a.wall = dm.wall;
  a.phys = phys_of(c.prm);
  a.ratio = c.prm.rho_minus / c.prm.rho_plus;
  a.eta_ratio = c.prm.eta_minus / c.prm.eta_plus;
  a.done = o.done;
  a.sm_r = (const T*)o.sm_r;
  a.sm_d = (const T*)o.sm_dinv;
  a.sm_w = (T)o.sm_w;
  a.shift = c.pp_shift;
  if constexpr (OP == K_CH_JAC || OP == K_VP) a.fc = form_const<DIM, T>(a.phys, a.ratio, a.eta_ratio);
  a.diag_of = o.diag_of;
  a.sy = dm.side + 1;
  a.sz = (int64_t)(dm.side + 1) * (dm.side + 1);
  a.side = dm.side;
  int part_off = 0;
  const char* tag = op_tag(OP, sizeof(T) == 8);
  hipEvent_t ev;
  // uniform meshes in one kernel, no slots and no combine: every 2D form (the
  // right-hand sides from 64^2 leaves) and the 3D pressure operator in FP64.
  // In FP32 that operator keeps the bricks and their order of sums: it gives
  // the same bits as the brick path of an octree with the same leaves, so the
  // learned preconditioner's solves through the node grid and on the uniform
  // mesh take the same iterations (another order moves them by a few, either
  // way).  The price: 25 us at 128^3, where the FP64 kernel takes 23.
  constexpr bool TILE3 = DIM == 3 && OP == K_PP && sizeof(T) == 8;
  const bool whole = dm.structured && (DIM == 2 || TILE3) && OP != K_DIAG && !rhs_on_bricks<DIM, OP>(dm.side);
  const int tx2 = std::max(1, (dm.side - 1 + kTile2X - 1) / kTile2X);
  const int own = !whole ? 1 : DIM == 2 ? tile2_own<OP>(tx2, dm.side) : tile3_own(dm.side);
  const int64_t cb = whole ? 0 : combine_blocks(dm);
  const int64_t total = !whole ? brick_blocks<DIM, OP>(dm) + cb
                               : (DIM == 2 ? tx2 : tile3_columns(dm.side)) * (int64_t)((dm.side + own) / own);
  const bool fold = o.fuse_dot && o.fold && total <= kFoldPartials;
  if (o.fold) *o.fold = fold ? (int)total : 0;
  if (o.fuse_dot && total > kMaxPartials) {
    set_error("mesh needs more reduction partials than allocated");
    return CHNS_EINVAL;
  }
  double* const parts = o.fuse_dot ? c.partials + (fold ? o.fold_at : 0) : nullptr;
  a.partials = parts;
  if (whole) {
    c.prof_begin(tag, s, &ev);
    if constexpr (DIM == 2 && OP != K_DIAG) {
      k_tile2<T, OP><<<dim3((unsigned)total), dim3(64), 0, s>>>(a, tx2, own);
      part_off = (int)total;
    } else if constexpr (TILE3) {
      const TileArgs<T> t = tile3_args<T>(a, dm.max_level, own);
      if (t.sm_r) k_pp_tile<T, true><<<dim3((unsigned)total), dim3(256), 0, s>>>(t);
      else k_pp_tile<T, false><<<dim3((unsigned)total), dim3(256), 0, s>>>(t);
      part_off = (int)total;
    }
  }
  if (whole) {
    CHNS_HIP(hipGetLastError());
  } else {
    c.prof_begin(tag, s, &ev);
    int rc = launch_bricks<DIM, T, OP>(dm, a, s, part_off);
    if (rc) return rc;
  }
  c.prof_end(tag, s, ev);
  if (cb > 0) {
    c.prof_begin("combine", s, &ev);
    k_combine<T, TR::NO, TR::WALL, OP == K_DIAG><<<dim3((unsigned)cb), dim3(256), 0, s>>>(
        dm.comb_node, dm.comb_ptr, dm.comb_ent, dm.n_comb, (const T*)L.slots, dm.n_slots, y, x, dm.n, dm.wall,
        parts ? parts + part_off : nullptr, o.done, (const T*)o.sm_r, (const T*)o.sm_dinv, (T)o.sm_w);
    CHNS_HIP(hipGetLastError());
    c.prof_end("combine", s, ev);
  }
  if (o.fuse_dot && !fold) {
    k_sum_partials<<<1, 1024, 0, s>>>(parts, (int)total, &c.sc->pq, o.done);
    CHNS_HIP(hipGetLastError());
  }
  return CHNS_OK;
}

template <int OP, typename T>
int apply_d(Ctx& c, const LevelView& L, const T* x, T* y, const T* const* cf, hipStream_t s, const ApplyOut& o) {
  return L.dm->dim == 3 ? apply_t<3, T, OP>(c, L, x, y, cf, s, o) : apply_t<2, T, OP>(c, L, x, y, cf, s, o);
}

template <typename T>
int apply_dispatch(Ctx& c, const LevelView& L, int op, const T* x, T* y, const T* phi, hipStream_t s,
                   const ApplyOut& o) {
  const T* one[1] = {phi};
  switch (op) {
    case CHNS_OP_PRESSURE:
      if (c.pp_kind == 1) return apply_d<K_VPS, T>(c, L, x, y, one, s, o);
      if (c.pp_shift != 0.0) return apply_d<K_PPS, T>(c, L, x, y, one, s, o);
      return apply_d<K_PP, T>(c, L, x, y, one, s, o);
    case CHNS_OP_MASS:
      return apply_d<K_MASS, T>(c, L, x, y, one, s, o);
    case CHNS_OP_MASS_RHO:
      return apply_d<K_MASS_RHO, T>(c, L, x, y, one, s, o);
    case CHNS_OP_MOMENTUM_SCALAR:
      return apply_d<K_VPS, T>(c, L, x, y, one, s, o);
  }
  if constexpr (sizeof(T) == 8) {
    const int64_t n = L.dm->n;
    const double* cf[kMaxCoef] = {};
    if (op == CHNS_OP_MOMENTUM || op == CHNS_OP_CH_JACOBIAN) {
      const bool mom = op == CHNS_OP_MOMENTUM;
      const double* base = mom ? c.coef_mom : c.coef_chj;
      if (!base || !(mom ? c.coef_mom_set : c.coef_chj_set)) {
        set_error("chns_set_coefficients must be called for this operator first");
        return CHNS_ESTATE;
      }
      for (int k = 0; k < (mom ? 2 : 1) + L.dm->dim; ++k) cf[k] = base + k * n;
      return mom ? apply_d<K_VP, double>(c, L, x, y, cf, s, o) : apply_d<K_CH_JAC, double>(c, L, x, y, cf, s, o);
    }
  } else {
    if (op == CHNS_OP_MOMENTUM || op == CHNS_OP_CH_JACOBIAN) {
      const bool mom = op == CHNS_OP_MOMENTUM;
      const double* base = mom ? c.coef_mom : c.coef_chj;
      if (!base || !(mom ? c.coef_mom_set : c.coef_chj_set)) {
        set_error("chns_set_coefficients must be called for this operator first");
        return CHNS_ESTATE;
      }
      // FP32 copies of the coefficient fields, refreshed after every change
      // of the FP64 ones (the momentum phase field as 1 + phi)
      const int64_t n = L.dm->n;
      const int nf = (mom ? 2 : 1) + L.dm->dim;
      float*& c32 = mom ? c.coef_mom32 : c.coef_chj32;
      bool& ok = mom ? c.coef_mom32_ok : c.coef_chj32_ok;
      if (!c32 && !(c32 = (float*)c.dalloc(sizeof(float) * (size_t)nf * (size_t)n))) return CHNS_ENOMEM;
      if (!ok) {
        const int64_t tot = nf * n;
        k_coef32<<<(unsigned)std::min<int64_t>((tot + 255) / 256, 65535), 256, 0, s>>>(base, c32, tot,
                                                                                      mom ? n : 0);
        CHNS_HIP(hipGetLastError());
        ok = true;
      }
      const float* cf[kMaxCoef] = {};
      for (int k = 0; k < nf; ++k) cf[k] = c32 + k * n;
      return mom ? apply_d<K_VP, float>(c, L, x, y, cf, s, o) : apply_d<K_CH_JAC, float>(c, L, x, y, cf, s, o);
    }
  }
  set_error("operator not available");
  return CHNS_EINVAL;
}

}  // namespace

int op_fields(int op, int dim) {
  switch (op) {
    case CHNS_OP_PRESSURE:
    case CHNS_OP_MASS:
    case CHNS_OP_MOMENTUM_SCALAR:
      return 1;
    case CHNS_OP_MASS_RHO:
    case CHNS_OP_MOMENTUM:
      return dim;
    case CHNS_OP_CH_JACOBIAN:
      return 2;
  }
  return 0;
}

LevelView fine_view(Ctx& c) { return LevelView{&c.dm, c.phi64, c.phi32, c.slots}; }

// Device address of `scratch` on the current device, looked up once per
// device (with that device current) and kept for the process.
int scratch_address(void** out) {
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = -1;
  CHNS_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) {
    set_error("device index beyond the library's limit");
    return CHNS_EINVAL;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    CHNS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    addr[dev] = p;
  }
  *out = addr[dev];
  return CHNS_OK;
}

int launch_apply_noalloc(Ctx& c, int op, int prec, const void* x, void* y, hipStream_t s) {
  if (!c.scratch) {
    set_error("context has no scratch address");
    return CHNS_ESTATE;
  }
  const size_t es = prec == CHNS_FP64 ? sizeof(double) : sizeof(float);
  const int nf = op_fields(op, c.dm.dim);
  const size_t need = es * (size_t)nf * (size_t)(c.dm.n_slots > 0 ? c.dm.n_slots : 1);
  if (nf > 0 && need > kScratchBytes) {
    set_error("mesh needs " + std::to_string(need) + " bytes of slot scratch for this operator, more than the " +
              std::to_string(kScratchBytes) + " the allocation-free apply has");
    return CHNS_EINVAL;
  }
  LevelView L = fine_view(c);
  L.slots = c.scratch;
  ApplyOut o{};
  return launch_apply_lv(c, L, op, prec, x, y, s, o);
}

int launch_apply_lv(Ctx& c, const LevelView& L, int op, int prec, const void* x, void* y, hipStream_t s,
                    const ApplyOut& o) {
  if ((op == CHNS_OP_PRESSURE || op == CHNS_OP_MASS_RHO || op == CHNS_OP_MOMENTUM_SCALAR) && !c.phi_set) {
    set_error("set_phase_field must be called before this operator");
    return CHNS_ESTATE;
  }
  if ((op == CHNS_OP_MOMENTUM || op == CHNS_OP_CH_JACOBIAN) && L.dm != &c.dm) {
    set_error("the momentum and Cahn-Hilliard operators act on the fine mesh only");
    return CHNS_EINVAL;
  }
  if (prec == CHNS_FP64) return apply_dispatch<double>(c, L, op, (const double*)x, (double*)y, L.phi64, s, o);
  if (prec == CHNS_FP32) return apply_dispatch<float>(c, L, op, (const float*)x, (float*)y, L.phi32, s, o);
  set_error("prec must be CHNS_FP64 or CHNS_FP32");
  return CHNS_EINVAL;
}

int launch_apply(Ctx& c, int op, int prec, const void* x, void* y, hipStream_t s, const ApplyOut& o) {
  return launch_apply_lv(c, fine_view(c), op, prec, x, y, s, o);
}

static_assert((int)FORM_CH_RES == (int)K_CH_RES && (int)FORM_CH_JAC == (int)K_CH_JAC && (int)FORM_VP == (int)K_VP &&
                  (int)FORM_VP_RHS == (int)K_VP_RHS && (int)FORM_PP_RHS == (int)K_PP_RHS &&
                  (int)FORM_VU_RHS == (int)K_VU_RHS && (int)FORM_ENERGY == (int)K_ENERGY,
              "form numbering");

int launch_form(Ctx& c, int form, const double* x, const double* const* cf, double* y, hipStream_t s,
                const ApplyOut& o) {
  const LevelView L = fine_view(c);
  switch (form) {
    case FORM_CH_RES:
      return apply_d<K_CH_RES, double>(c, L, x, y, cf, s, o);
    case FORM_CH_JAC:
      return apply_d<K_CH_JAC, double>(c, L, x, y, cf, s, o);
    case FORM_VP:
      return apply_d<K_VP, double>(c, L, x, y, cf, s, o);
    case FORM_VP_RHS:
      return apply_d<K_VP_RHS, double>(c, L, x, y, cf, s, o);
    case FORM_PP_RHS:
      return apply_d<K_PP_RHS, double>(c, L, x, y, cf, s, o);
    case FORM_VU_RHS:
      return apply_d<K_VU_RHS, double>(c, L, x, y, cf, s, o);
    case FORM_ENERGY:
      return apply_d<K_ENERGY, double>(c, L, x, y, cf, s, o);
  }
  set_error("unknown form");
  return CHNS_EINVAL;
}

int launch_narrow(const double* a, float* b, int64_t n, hipStream_t s) {
  k_narrow<<<(unsigned)std::min<int64_t>((n + 255) / 256, 8192), 256, 0, s>>>(a, b, n);
  CHNS_HIP(hipGetLastError());
  return CHNS_OK;
}

// Exact diagonal of P^T K P.  The scalar operators on octrees in FP64: one
// pass over the leaves (K_DIAG).  Otherwise by probing: colour classes never
// share a leaf (directly or through constraint parents), so y = A 1_c has
// y_i = A_ii on colour c; eight colours on uniform meshes, but about twenty on
// octrees, where the pass replaces as many applies (35 us each with their
// helper kernels at levels 5-8).
int launch_diagonal_lv(Ctx& c, const LevelView& L, int op, int prec, void* d, bool invert, void* xi, void* yi,
                       hipStream_t s) {
  const int64_t n = L.dm->n;
  const int nf = op_fields(op, L.dm->dim);
  const unsigned g = (unsigned)((n + 255) / 256);
  ApplyOut o{};
  if (!L.dm->structured && prec == CHNS_FP64 &&
      (op == CHNS_OP_PRESSURE || op == CHNS_OP_MASS || op == CHNS_OP_MASS_RHO || op == CHNS_OP_MOMENTUM_SCALAR)) {
    if (op != CHNS_OP_MASS && !c.phi_set) {
      set_error("set_phase_field must be called before this operator");
      return CHNS_ESTATE;
    }
    o.diag_of = op == CHNS_OP_MASS       ? K_MASS
                : op == CHNS_OP_MASS_RHO ? K_MASS_RHO
                : op == CHNS_OP_MOMENTUM_SCALAR || c.pp_kind == 1
                    ? K_VPS
                    : (c.pp_shift != 0.0 ? K_PPS : K_PP);
    const double* cf[1] = {L.phi64};
    int rc = apply_d<K_DIAG, double>(c, L, L.phi64, (double*)d, cf, s, o);
    if (rc) return rc;
    k_diag_finish<<<g, 256, 0, s>>>((double*)d, n, nf, op == CHNS_OP_MASS_RHO ? L.dm->wall : nullptr, invert ? 1 : 0);
    CHNS_HIP(hipGetLastError());
    return CHNS_OK;
  }
  // fields of the Cahn-Hilliard Jacobian are coupled: probe them one at a time
  const bool coupled = op == CHNS_OP_CH_JACOBIAN;
  for (int col = 0; col < L.dm->n_colors; ++col) {
    for (int f = coupled ? 0 : -1; f < (coupled ? nf : 0); ++f) {
      if (prec == CHNS_FP64)
        k_indicator<double><<<g, 256, 0, s>>>((double*)xi, L.dm->color, col, n, nf, f);
      else
        k_indicator<float><<<g, 256, 0, s>>>((float*)xi, L.dm->color, col, n, nf, f);
      CHNS_HIP(hipGetLastError());
      int rc = launch_apply_lv(c, L, op, prec, xi, yi, s, o);
      if (rc) return rc;
      if (prec == CHNS_FP64)
        k_take_diag<double><<<g, 256, 0, s>>>((double*)d, (const double*)yi, L.dm->color, col, n, nf, invert, f);
      else
        k_take_diag<float><<<g, 256, 0, s>>>((float*)d, (const float*)yi, L.dm->color, col, n, nf, invert, f);
      CHNS_HIP(hipGetLastError());
    }
  }
  return CHNS_OK;
}

// nf x nf node blocks of an FP64 operator (the couplings between the fields
// of one node), by probing every field of every colour class
int launch_block_diagonal(Ctx& c, int op, double* blk, double* xi, double* yi, hipStream_t s) {
  const LevelView L = fine_view(c);
  const int64_t n = L.dm->n;
  const int nf = op_fields(op, L.dm->dim);
  const unsigned g = (unsigned)((n + 255) / 256);
  ApplyOut o{};
  for (int col = 0; col < L.dm->n_colors; ++col)
    for (int f = 0; f < nf; ++f) {
      k_indicator<double><<<g, 256, 0, s>>>(xi, L.dm->color, col, n, nf, f);
      CHNS_HIP(hipGetLastError());
      int rc = launch_apply_lv(c, L, op, CHNS_FP64, xi, yi, s, o);
      if (rc) return rc;
      k_take_block<<<g, 256, 0, s>>>(blk, yi, L.dm->color, col, n, nf, f);
      CHNS_HIP(hipGetLastError());
    }
  return CHNS_OK;
}

int launch_diagonal(Ctx& c, int op, int prec, void* d, bool invert, hipStream_t s) {
  const int64_t n = c.dm.n;
  size_t es = prec == CHNS_FP64 ? 8 : 4;
  for (int k = 6; k < 8; ++k) {
    if (prec == CHNS_FP64 && !c.w64[k]) c.w64[k] = (double*)c.dalloc(es * n * 3);
    if (prec == CHNS_FP32 && !c.w32[k]) c.w32[k] = (float*)c.dalloc(es * n * 3);
    if ((prec == CHNS_FP64 && !c.w64[k]) || (prec == CHNS_FP32 && !c.w32[k])) return CHNS_ENOMEM;
  }
  void* xi = prec == CHNS_FP64 ? (void*)c.w64[6] : (void*)c.w32[6];
  void* yi = prec == CHNS_FP64 ? (void*)c.w64[7] : (void*)c.w32[7];
  return launch_diagonal_lv(c, fine_view(c), op, prec, d, invert, xi, yi, s);
}

}  // namespace chns
