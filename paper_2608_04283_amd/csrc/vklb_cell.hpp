// Per-cell arithmetic of the weighted-upwind vector kinetic lattice Boltzmann
// step: physical fluxes, characteristic speeds, the sigmoid-weighted flux
// split and the weighted-upwind equilibrium. Host+device functions; the GPU
// kernels and the host-side cell check both include this header.
//
// The split is written as F+ = F/2 + D and F- = F/2 - D with
//   D = sum_j beta(lambda_j) phi_j r_j,  beta = alpha - 1/2 = tanh(k lambda / (2 Lambda)) / 2,
// which is the weighted splitting of Sec. 3.1 (alpha = 1/(1+exp(-k lambda/Lambda)))
// rearranged; D is evaluated per system in closed form, without forming
// the eigenvector matrix P or solving P Phi = F:
//   * linear advection: one wave;
//   * shallow water (Sec. 5.1): the two acoustic waves (the shear wave of the
//     2D system carries no flux);
//   * Euler (Sec. 5.2): the flux is homogeneous of degree one, so
//     D = P diag(beta_j lambda_j) P^-1 U, the Steger-Warming formula with each
//     eigenvalue scaled by its weight;
//   * ideal MHD with divergence cleaning (Sec. 5.3): the Jacobian is block
//     triangular, [[A7, C], [0, G]] with the (B_n, psi) pair in G. D on the
//     seven-wave block uses Roe-Balsara normalized primitive eigenvectors
//     (well defined at coinciding speeds); the coupling through C uses divided
//     differences of beta between each seven-wave speed and +-c_h; on the
//     cleaning pair D = beta(c_h) c_h (B_n, psi). In FP32, the eigenstructure
//     (speeds and normalization) of directions whose speeds nearly coincide is
//     evaluated in FP64.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

namespace vklb {

enum Kind { K_SW = 0, K_EULER = 1, K_MHD = 2, K_LINEAR = 3 };

// Physical and method parameters of one solve (read-only in kernels).
struct Phys {
  double g, gamma, ch_factor;
  double adv[2];
  double omega, c, k;
  int kinf;         // 1: discontinuous split (k = infinity)
  int alpha_local;  // 1: normalize the sigmoid by the cell's own max |lambda|
};

template <int KIND, int DIM>
struct SysInfo;
template <> struct SysInfo<K_SW, 1> { static constexpr int P = 2; };
template <> struct SysInfo<K_SW, 2> { static constexpr int P = 3; };
template <> struct SysInfo<K_EULER, 1> { static constexpr int P = 3; };
template <> struct SysInfo<K_EULER, 2> { static constexpr int P = 4; };
template <> struct SysInfo<K_MHD, 1> { static constexpr int P = 9; };
template <> struct SysInfo<K_MHD, 2> { static constexpr int P = 9; };
template <> struct SysInfo<K_LINEAR, 1> { static constexpr int P = 1; };
template <> struct SysInfo<K_LINEAR, 2> { static constexpr int P = 1; };

template <class S>
__host__ __device__ inline S sq(S a) { return a * a; }

// beta(lambda) = alpha(lambda) - 1/2 for the sigmoid of Sec. 3.1.
// Division, reciprocal and square root of the per-cell arithmetic. FP32
// device code uses the hardware reciprocal and square root (about 1 ulp),
// as plain operations the compiler cannot fuse differently in different
// places, so every inlined copy still rounds identically; FP64, and host
// code, use the correctly rounded operations.
template <class S>
__host__ __device__ inline S qrcp(S b) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (sizeof(S) == 4) return __builtin_amdgcn_rcpf(b);
#endif
  return S(1) / b;
}
template <class S>
__host__ __device__ inline S qdiv(S a, S b) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (sizeof(S) == 4) return a * __builtin_amdgcn_rcpf(b);
#endif
  return a / b;
}
template <class S>
__host__ __device__ inline S qsqrt(S x) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (sizeof(S) == 4) return __builtin_amdgcn_sqrtf(x);
#endif
  return sqrt(x);
}

// a / b where r = qrcp(b) serves several quotients of a cell. FP32 multiplies
// by r, as qdiv does. FP64 corrects that product by its remainder, which rounds
// as the division does (Markstein 1990: r is correctly rounded) in two fused
// operations a quotient; the product alone leaves the wave speeds up to 11 %
// further off (rms over random states, Mach < 5: Euler 0.655 roundings against
// 0.609, MHD's fast speed 8.86 against 7.98). Measured (us per step: product,
// this, a division each): 1D Euler of 1000 cells 3.19, 3.22, 3.34; 2D Euler
// 1024^2 23.3, 23.5, 24.3; MHD 512^2 33.0, 33.2, 33.6. (r overflows below
// b = 2^-1024, where the split's reciprocals do as well.)
template <class S>
__host__ __device__ inline S qover(S a, S b, S r) {
  const S q = a * r;
  if (sizeof(S) == 8) return fma(fma(-q, b, a), r, q);
  return q;
}

// Positive and finite: one class test on the device.
template <class S>
__host__ __device__ inline bool positive_finite(S x) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (sizeof(S) == 4) return __builtin_amdgcn_classf(x, 0x180);  // + subnormal, + normal
  else return __builtin_amdgcn_class(x, 0x180);
#endif
  return x > S(0) && isfinite(x);
}

// tanh for the weights. FP32 device code evaluates it from its exponential
// form, tanh z = sign(z) (1 - e^{-2|z|}) / (1 + e^{-2|z|}), with the hardware
// base-2 exponential and reciprocal: a few units in the last place (absolute
// error ~1e-7 near z = 0), far inside the FP32 path's tolerance, and an odd
// function exactly as tanh is. FP64 device code uses the same identity through
// expm1, tanh z = sign(z) (-m) / (2 + m) with m = e^{-2|z|} - 1: about two
// units in the last place at every z (no cancellation near 0), in 68 vector
// instructions where the library tanh takes 165. Host code calls tanh.
template <class S>
__host__ __device__ inline S wtanh(S z) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (sizeof(S) == 4) {
    const float t = __builtin_amdgcn_exp2f(-2.8853900817779268f * fabsf(z));  // e^{-2|z|}
    return copysignf((1.0f - t) * __builtin_amdgcn_rcpf(1.0f + t), z);
  } else {
    const double m = expm1(-2.0 * fabs(double(z)));
    return S(copysign(-m / (2.0 + m), double(z)));
  }
#endif
  return tanh(z);
}

template <class S>
__host__ __device__ inline S beta_w(S lam, S half_k_over_L, int kinf) {
  if (kinf) return lam >= S(0) ? S(0.5) : S(-0.5);
  return S(0.5) * wtanh(lam * half_k_over_L);
}

// beta of N speeds of one direction, none larger than lmax in magnitude. With
// the sigmoid normalized by the largest |lambda| and k <= 2 (Sec. 3.1, k = 2)
// every argument z = k lambda / (2 Lambda) lies in [-1, 1], where tanh(z) / 2 is
// an odd polynomial, z p(z^2): 9 vector operations a weight in FP32 (degree 6)
// and 18 in FP64 (degree 15), with no transcendental one among them, against
// 11 and about 85 of wtanh. The coefficients are the interpolant of
// tanh(sqrt w) / (2 sqrt w) at Chebyshev nodes of [0, 1.0414]; relative error
// 1.6e-7 and 2.2e-16 over |z| <= 1.02, rounding included (wtanh in FP32: 1.6e-6
// relative for |z| > 0.01, 6.5e-8 absolute against 5.9e-8 here). Larger
// arguments (k > 2, or a boundary state faster than the grid) take wtanh.
template <class S, int N>
__host__ __device__ inline void weights(const S (&lam)[N], S lmax, S hk, int kinf, S (&b)[N]) {
  if (!kinf && lmax * hk <= S(1.02)) {
    constexpr double c32[7] = {0.4999999701976776, -0.16666358709335327, 0.06661827117204666, -0.026692891493439674,
                               0.010071528144180775, -0.0030323248356580734, 0.0004960894584655762};
    constexpr double c64[16] = {0.5, -0.16666666666666183, 0.06666666666626553, -0.02698412697101095,
                                0.010934744042573333, -0.004431615413343778, 0.001796047850046346,
                                -0.0007278399231292868, 0.0002947479495034335, -0.00011889149097278873,
                                4.718446560211916e-05, -1.7825235404940583e-05, 6.004817950962269e-06,
                                -1.6264485337714894e-06, 3.023335014179045e-07, -2.7998503351044707e-08};
    constexpr int n = sizeof(S) == 4 ? 6 : 15;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const S z = lam[j] * hk, w = z * z;
      S p = S(sizeof(S) == 4 ? c32[6] : c64[15]);
#pragma unroll
      for (int i = n - 1; i >= 0; --i) p = p * w + S(sizeof(S) == 4 ? c32[i % 7] : c64[i]);
      b[j] = p * z;
    }
  } else {
#pragma unroll
    for (int j = 0; j < N; ++j) b[j] = beta_w(lam[j], hk, kinf);
  }
}

// k / (2 L): the weights' argument is lambda times this.
template <class S>
__host__ __device__ inline S half_k_over(const Phys& ph, S L) {
  return L > S(0) ? qdiv(S(0.5 * ph.k), L) : S(0);
}

// Divided difference (beta(a) - beta(b)) / (a - b) from the weights ba, bb
// already evaluated, with the derivative when the two speeds nearly coincide.
template <class S>
__host__ __device__ inline S beta_dd(S a, S ba, S b, S bb, S half_k_over_L, int kinf) {
  const S d = a - b;
  const S rel = sizeof(S) == 4 ? S(1e-3) : S(1e-6);
  if (fabs(d) > rel * (fabs(a) + fabs(b)) || kinf) return d != S(0) ? qdiv(ba - bb, d) : S(0);
  const S tm = wtanh(S(0.5) * (a + b) * half_k_over_L);
  return S(0.5) * half_k_over_L * (S(1) - tm * tm);
}

// ---------------------------------------------------------------------------
// Cell speeds: max |lambda| over directions and (MHD) the max fast speed.
// ---------------------------------------------------------------------------
template <int KIND, int DIM, class S>
struct Cell;

// ----------------------------- linear advection ----------------------------
template <int DIM, class S>
struct Cell<K_LINEAR, DIM, S> {
  static constexpr int P = 1;
  // Characteristic boundary of Sec. 3.3 (1D): out = g(a) dU with g(a) = a for
  // an outgoing wave (a > 0 at the right boundary, a < 0 at the left), else 0.
  __host__ __device__ static bool char_correction(const S* Ub, const S* dU, const Phys& ph, S, bool right, S* out) {
    (void)Ub;
    const S a = S(ph.adv[0]);
    out[0] = (right ? a > S(0) : a < S(0)) ? a * dU[0] : S(0);
    return true;
  }
  __host__ __device__ static void speeds(const S* U, const Phys& ph, S* lam, S* cfm) {
    S m = S(0);
    for (int d = 0; d < DIM; ++d) m = fmax(m, fabs(S(ph.adv[d])));
    *lam = m;
    *cfm = S(0);
  }
  __host__ __device__ static bool admissible(const S* U, const Phys&) { return isfinite(U[0]); }
  // F^(d) and D^(d); Lam normalizes the sigmoid (global max |lambda|), ch unused.
  __host__ __device__ static void split(int d, const S* U, const Phys& ph, S Lam, S, S* F, S* D) {
    S a = S(ph.adv[d]);
    const S hk = half_k_over(ph, ph.alpha_local ? S(fabs(a)) : Lam);
    S lam[1] = {a}, b[1];
    weights(lam, S(fabs(a)), hk, ph.kinf, b);
    F[0] = a * U[0];
    D[0] = b[0] * a * U[0];
  }
};

// ------------------------------- shallow water -----------------------------
template <int DIM, class S>
struct Cell<K_SW, DIM, S> {
  static constexpr int P = DIM + 1;
  // Characteristic boundary of Sec. 3.3 (1D): out = sum_j g(lambda_j) (l_j . dU) r_j
  // over u -+ c, with r = (1, u -+ c), l = (+-(u +- c), -+1) / (2c) and g the
  // speed for outgoing waves, 0 for incoming ones.
  __host__ __device__ static bool char_correction(const S* Ub, const S* dU, const Phys& ph, S, bool right, S* out) {
    const S h = Ub[0];
    const S u = qdiv(Ub[1], h);
    const S c = qsqrt(S(ph.g) * h);
    const S l1 = u - c, l2 = u + c;
    const S i2c = qrcp(S(2) * c);
    const S w1 = ((u + c) * dU[0] - dU[1]) * i2c;
    const S w2 = (dU[1] - (u - c) * dU[0]) * i2c;
    const S g1 = (right ? l1 > S(0) : l1 < S(0)) ? l1 : S(0);
    const S g2 = (right ? l2 > S(0) : l2 < S(0)) ? l2 : S(0);
    out[0] = g1 * w1 + g2 * w2;
    out[1] = g1 * w1 * l1 + g2 * w2 * l2;
    return isfinite(out[0]) && isfinite(out[1]);
  }
  __host__ __device__ static void speeds(const S* U, const Phys& ph, S* lam, S* cfm) {
    S h = U[0];
    S c = qsqrt(S(ph.g) * h);
    S m = S(0);
    for (int d = 0; d < DIM; ++d) m = fmax(m, fabs(qdiv(U[1 + d], h)) + c);
    *lam = m;
    *cfm = S(0);
  }
  __host__ __device__ static bool admissible(const S* U, const Phys&) {
    bool ok = U[0] > S(0);
    for (int i = 0; i < P; ++i) ok = ok && isfinite(U[i]);
    return ok;
  }
  __host__ __device__ static void split(int d, const S* U, const Phys& ph, S Lam, S, S* F, S* D) {
    const S h = U[0];
    const S g = S(ph.g);
    const S ud = qdiv(U[1 + d], h);
    const S c = qsqrt(g * h);
    F[0] = U[1 + d];
    for (int kk = 0; kk < DIM; ++kk) F[1 + kk] = U[1 + kk] * ud;
    F[1 + d] += S(0.5) * g * h * h;
    const S lm = ud - c, lp = ud + c;
    const S L = ph.alpha_local ? fmax(fabs(lm), fabs(lp)) : Lam;
    const S hk = L > S(0) ? qdiv(S(0.5 * ph.k), L) : S(0);
    // The weights' polynomial (weights) is used in 2D. In 1D FP32 its range
    // check costs what it saves on two weights (a 100-cell solve in one
    // workgroup: 1.39 us a step with it, 1.33 without). The 1D FP64 results
    // stay bit for bit: the dam break amplifies a rounding up to 10^8 times at
    // its rarefaction head, so any other rounding shows in them.
    S b[2];
    if (DIM == 2) {
      const S lam[2] = {lm, lp};
      weights(lam, S(fmax(fabs(lm), fabs(lp))), hk, ph.kinf, b);
    } else {
      b[0] = beta_w(lm, hk, ph.kinf);
      b[1] = beta_w(lp, hk, ph.kinf);
    }
    // coefficients of the two acoustic waves: phi = h (2 u_d -+ c) / 4
    const S wm = b[0] * h * (S(2) * ud - c) * S(0.25);
    const S wp = b[1] * h * (S(2) * ud + c) * S(0.25);
    D[0] = wm + wp;
    for (int kk = 0; kk < DIM; ++kk) D[1 + kk] = qdiv(U[1 + kk], h) * (wm + wp);
    D[1 + d] = lm * wm + lp * wp;
  }
};

// ----------------------------------- Euler ---------------------------------
template <int DIM, class S>
struct Cell<K_EULER, DIM, S> {
  static constexpr int P = DIM + 2;
  // Characteristic boundary of Sec. 3.3 (1D): out = sum_j g(lambda_j) (l_j . dU) r_j
  // over u - a, u, u + a with the textbook eigenvectors r = (1, u -+ a, H -+ ua),
  // (1, u, u^2/2) and left eigenvectors (b1 = (gamma-1)/a^2, b2 = b1 u^2/2)
  // l_1,3 = (b2 +- u/a, -(b1 u +- 1/a), b1)/2, l_2 = (1 - b2, b1 u, -b1);
  // g is the speed for outgoing waves, 0 for incoming ones.
  __host__ __device__ static bool char_correction(const S* Ub, const S* dU, const Phys& ph, S, bool right, S* out) {
    const S gamma = S(ph.gamma);
    const S rho = Ub[0];
    const S u = qdiv(Ub[1], rho);
    const S E = Ub[2];
    const S p = (gamma - S(1)) * (E - S(0.5) * rho * u * u);
    const S a = qsqrt(qdiv(gamma * p, rho));
    const S H = qdiv(E + p, rho);
    const S ia = qrcp(a);
    const S b1 = (gamma - S(1)) * ia * ia, b2 = S(0.5) * b1 * u * u;
    const S w1 = S(0.5) * ((b2 + u * ia) * dU[0] - (b1 * u + ia) * dU[1] + b1 * dU[2]);
    const S w2 = (S(1) - b2) * dU[0] + b1 * u * dU[1] - b1 * dU[2];
    const S w3 = S(0.5) * ((b2 - u * ia) * dU[0] - (b1 * u - ia) * dU[1] + b1 * dU[2]);
    const S lam[3] = {u - a, u, u + a};
    S g[3];
    for (int j = 0; j < 3; ++j) g[j] = (right ? lam[j] > S(0) : lam[j] < S(0)) ? lam[j] : S(0);
    const S c1 = g[0] * w1, c2 = g[1] * w2, c3 = g[2] * w3;
    out[0] = c1 + c2 + c3;
    out[1] = c1 * (u - a) + c2 * u + c3 * (u + a);
    out[2] = c1 * (H - u * a) + c2 * (S(0.5) * u * u) + c3 * (H + u * a);
    return isfinite(out[0]) && isfinite(out[1]) && isfinite(out[2]);
  }
  __host__ __device__ static S pressure(const S* U, S gamma) {
    S m2 = S(0);
    for (int kk = 0; kk < DIM; ++kk) m2 += U[1 + kk] * U[1 + kk];
    const S irho = qrcp(U[0]);
    if (sizeof(S) == 8) return (gamma - S(1)) * (U[DIM + 1] - S(0.5) * qover(m2, U[0], irho));
    return (gamma - S(1)) * (U[DIM + 1] - S(0.5) * m2 * irho);  // (the product fused: one rounding fewer)
  }
  __host__ __device__ static void speeds(const S* U, const Phys& ph, S* lam, S* cfm) {
    const S gamma = S(ph.gamma);
    const S irho = qrcp(U[0]);
    const S c = qsqrt(qover(gamma * pressure(U, gamma), U[0], irho));
    S m = S(0);
    for (int d = 0; d < DIM; ++d) m = fmax(m, fabs(qover(U[1 + d], U[0], irho)) + c);
    *lam = m;
    *cfm = S(0);
  }
  __host__ __device__ static bool admissible(const S* U, const Phys& ph) {
    // (an infinite or NaN momentum leaves p negative or NaN)
    return positive_finite(U[0]) && pressure(U, S(ph.gamma)) > S(0) && isfinite(U[DIM + 1]);
  }
  __host__ __device__ static void split(int d, const S* U, const Phys& ph, S Lam, S, S* F, S* D) {
    const S gamma = S(ph.gamma);
    const S rho = U[0];
    const S irho = qrcp(rho);
    S vel[DIM];
    S v2 = S(0);
    for (int kk = 0; kk < DIM; ++kk) { vel[kk] = U[1 + kk] * irho; v2 += vel[kk] * vel[kk]; }
    const S E = U[DIM + 1];
    const S p = (gamma - S(1)) * (E - S(0.5) * rho * v2);
    const S c = qsqrt(gamma * p * irho);
    const S ud = vel[d];
    F[0] = U[1 + d];
    for (int kk = 0; kk < DIM; ++kk) F[1 + kk] = U[1 + kk] * ud;
    F[1 + d] += p;
    F[DIM + 1] = (E + p) * ud;
    const S lam[3] = {ud - c, ud, ud + c};
    const S lmax = fabs(ud) + c;
    const S hk = half_k_over(ph, ph.alpha_local ? lmax : Lam);
    S b[3];
    if (sizeof(S) == 8 || DIM == 2) {
      weights(lam, lmax, hk, ph.kinf, b);
    } else {
      for (int j = 0; j < 3; ++j) b[j] = beta_w(lam[j], hk, ph.kinf);
    }
    const S mu1 = b[0] * lam[0], mu3 = b[2] * lam[2];
    const S H = (E + p) * irho;
    const S s = rho * qrcp(S(2) * gamma);
    const S ent = S(2) * (gamma - S(1)) * (b[1] * ud);
    const S sum = mu1 + mu3, dif = c * (mu3 - mu1);
    D[0] = s * (ent + sum);
    for (int kk = 0; kk < DIM; ++kk) D[1 + kk] = D[0] * vel[kk];
    D[1 + d] += s * dif;
    D[DIM + 1] = s * (ent * (S(0.5) * v2) + H * sum + ud * dif);
  }
};

// ------------------------- ideal MHD with GLM cleaning ----------------------
// Conserved order: rho, m_x, m_y, m_z, E, B_x, B_y, B_z, psi (3-vectors in 1D/2D).
template <int DIM, class S>
struct Cell<K_MHD, DIM, S> {
  static constexpr int P = 9;
  // Characteristic boundary of Sec. 3.3 (1D, normal x): out = g(A) dU with
  // g(lambda) = lambda for waves leaving through the boundary and 0 for the
  // others, over the nine waves of the GLM system: the seven MHD waves through
  // the primitive eigenvectors of the split below, the cleaning pair +-c_h on
  // (B_n, psi), and the pair's coupling into the seven-wave block through the
  // B_n column of the Jacobian, by divided differences of g (the Jacobian is
  // block triangular). Computed in FP64 in both precisions: it runs on two
  // cells per step.
  __host__ __device__ static bool char_correction(const S* Ub, const S* dU, const Phys& ph, S ch, bool right,
                                                  S* out) {
    double U[9], dv[9], o[9];
    for (int i = 0; i < 9; ++i) {
      U[i] = double(Ub[i]);
      dv[i] = double(dU[i]);
    }
    if (!char64(U, dv, ph, double(ch), right, o)) return false;
    bool ok = true;
    for (int i = 0; i < 9; ++i) {
      out[i] = S(o[i]);
      ok = ok && isfinite(out[i]);
    }
    return ok;
  }
  __host__ __device__ static bool char64(const double* Ug, const double* dv, const Phys& ph, double ch, bool right,
                                         double* out) {
    using C = Cell<K_MHD, DIM, double>;
    if (!(ch > 0.0)) return false;
    const double gamma = ph.gamma, gm1 = gamma - 1.0;
    const double rho = Ug[0], irho = 1.0 / rho;
    const double u = Ug[1] * irho, v = Ug[2] * irho, w = Ug[3] * irho;
    const double Bn = Ug[5], By = Ug[6], Bz = Ug[7];
    const double uu = u * u + v * v + w * w;
    const double p = gm1 * (Ug[4] - 0.5 * rho * uu - 0.5 * (Bn * Bn + By * By + Bz * Bz));
    typename C::template Eig<double> eg;
    C::template eigenstructure<double>(rho, p, Bn, By, Bz, gamma, eg);
    typename C::Waves W;
    W.rho = rho;
    W.sr = sqrt(rho);
    W.a2 = eg.a2;
    W.a = eg.a;
    W.cf = eg.cf;
    W.cs = eg.cs;
    const double ca = eg.ca;
    W.af = eg.af;
    W.as = eg.as;
    W.by = eg.by;
    W.bz = eg.bz;
    W.sgn = Bn >= 0.0 ? 1.0 : -1.0;
    const double lam[7] = {u - W.cf, u - ca, u - W.cs, u, u + W.cs, u + ca, u + W.cf};
    auto out_ = [right](double l) { return right ? l > 0.0 : l < 0.0; };
    auto g = [&](double l) { return out_(l) ? l : 0.0; };
    auto dd = [&](double a, double b) { return a != b ? (g(a) - g(b)) / (a - b) : (out_(a) ? 1.0 : 0.0); };
    // primitive images (B_n held fixed) of the seven-wave part of dU and of
    // the B_n column of the Jacobian
    double x[7], xC[7];
    x[0] = dv[0];
    x[1] = (dv[1] - u * dv[0]) * irho;
    x[2] = (dv[2] - v * dv[0]) * irho;
    x[3] = (dv[3] - w * dv[0]) * irho;
    x[4] = gm1 * (dv[4] + 0.5 * uu * dv[0] - (u * dv[1] + v * dv[2] + w * dv[3]) - By * dv[6] - Bz * dv[7]);
    x[5] = dv[6];
    x[6] = dv[7];
    xC[0] = 0.0;
    xC[1] = -gamma * Bn * irho;
    xC[2] = -By * irho;
    xC[3] = -Bz * irho;
    xC[4] = gm1 * (v * By + w * Bz);
    xC[5] = -v;
    xC[6] = -w;
    double c[7], cC[7], cD[7];
    C::project(W, x, c);
    C::project(W, xC, cC);
    // cleaning pair: eigenvalues +-c_h, eigenvectors (1, +-c_h) on (B_n, psi)
    const double qp = 0.5 * (dv[5] + dv[8] / ch), qm = 0.5 * (dv[5] - dv[8] / ch);
    for (int j = 0; j < 7; ++j) cD[j] = g(lam[j]) * c[j] + (dd(lam[j], ch) * qp + dd(lam[j], -ch) * qm) * cC[j];
    double y[7];
    C::combine(W, cD, y);
    out[0] = y[0];
    out[1] = u * y[0] + rho * y[1];
    out[2] = v * y[0] + rho * y[2];
    out[3] = w * y[0] + rho * y[3];
    out[4] = y[4] / gm1 + 0.5 * uu * y[0] + rho * (u * y[1] + v * y[2] + w * y[3]) + By * y[5] + Bz * y[6];
    out[6] = y[5];
    out[7] = y[6];
    out[5] = g(ch) * qp + g(-ch) * qm;
    out[8] = ch * (g(ch) * qp - g(-ch) * qm);
    return true;
  }

  __host__ __device__ static S pressure(const S* U, S gamma) {
    S m2 = U[1] * U[1] + U[2] * U[2] + U[3] * U[3];
    S B2 = U[5] * U[5] + U[6] * U[6] + U[7] * U[7];
    const S irho = qrcp(U[0]);
    if (sizeof(S) == 8) return (gamma - S(1)) * (U[4] - S(0.5) * qover(m2, U[0], irho) - S(0.5) * B2);
    return (gamma - S(1)) * (U[4] - S(0.5) * m2 * irho - S(0.5) * B2);  // (the product fused)
  }
  // fast speed along direction d
  __host__ __device__ static S fast(const S* U, S gamma, int d) {
    const S irho = qrcp(U[0]);
    const S a2 = qover(gamma * pressure(U, gamma), U[0], irho);
    const S bn2 = qover(U[5 + d] * U[5 + d], U[0], irho);
    const S bt2 = qover(U[5 + (d + 1) % 3] * U[5 + (d + 1) % 3] + U[5 + (d + 2) % 3] * U[5 + (d + 2) % 3], U[0], irho);
    const S disc = qsqrt(sq(a2 - bn2) + bt2 * (S(2) * a2 + S(2) * bn2 + bt2));
    return qsqrt(S(0.5) * (a2 + bn2 + bt2 + disc));
  }
  __host__ __device__ static void speeds(const S* U, const Phys& ph, S* lam, S* cfm) {
    const S gamma = S(ph.gamma);
    S m = S(0), cm = S(0);
    for (int d = 0; d < DIM; ++d) {
      const S cf = fast(U, gamma, d);
      m = fmax(m, fabs(qover(U[1 + d], U[0], qrcp(U[0]))) + cf);
      cm = fmax(cm, cf);
    }
    *lam = m;   // seven-wave max; the cleaning speed joins it globally
    *cfm = cm;
  }
  __host__ __device__ static bool admissible(const S* U, const Phys& ph) {
    // (an infinite or NaN momentum or field leaves p negative or NaN)
    return positive_finite(U[0]) && pressure(U, S(ph.gamma)) > S(0) && isfinite(U[4]) && isfinite(U[8]);
  }

  // Primitive-variable wave decomposition along the normal direction.
  struct Waves {
    S rho, sr, a, a2, cf, cs, af, as, by, bz, sgn;
  };

  // Coefficients (f-, a-, s-, e, s+, a+, f+) of a primitive 7-vector
  // x = (rho, u_n, u_t1, u_t2, p, B_t1, B_t2) in the right eigenvectors.
  __host__ __device__ static void project(const Waves& w, const S* x, S* c) {
    const S xvp = w.by * x[2] + w.bz * x[3];
    const S xvq = -w.bz * x[2] + w.by * x[3];
    const S xbp = w.by * x[5] + w.bz * x[6];
    const S xbq = -w.bz * x[5] + w.by * x[6];
    const S X = qdiv(x[4], w.rho * w.a2);
    const S Y = qdiv(xbp, w.a * w.sr);
    const S Fp = w.af * X + w.as * Y;
    const S Sp = w.as * X - w.af * Y;
    const S Z1 = x[1], Z2 = w.sgn * xvp;
    const S ia2 = qrcp(w.a2);
    const S Fm = (w.af * w.cf * Z1 - w.as * w.cs * Z2) * ia2;
    const S Sm = (w.as * w.cs * Z1 + w.af * w.cf * Z2) * ia2;
    const S Ap = qdiv(xbq, w.sr), Am = -w.sgn * xvq;
    c[0] = S(0.5) * (Fp - Fm);
    c[6] = S(0.5) * (Fp + Fm);
    c[2] = S(0.5) * (Sp - Sm);
    c[4] = S(0.5) * (Sp + Sm);
    c[1] = S(0.5) * (Ap - Am);
    c[5] = S(0.5) * (Ap + Am);
    c[3] = x[0] - x[4] * ia2;
  }
  // sum_j c_j r_j (primitive 7-vector) for the same eigenvectors.
  __host__ __device__ static void combine(const Waves& w, const S* c, S* y) {
    const S Fp = c[6] + c[0], Fm = c[6] - c[0];
    const S Sp = c[4] + c[2], Sm = c[4] - c[2];
    const S Ap = c[5] + c[1], Am = c[5] - c[1];
    const S pf = w.af * Fp + w.as * Sp;
    y[0] = c[3] + w.rho * pf;
    y[1] = w.af * w.cf * Fm + w.as * w.cs * Sm;
    const S vp = w.sgn * (-w.as * w.cs * Fm + w.af * w.cf * Sm);
    const S vq = -w.sgn * Am;
    y[2] = w.by * vp - w.bz * vq;
    y[3] = w.bz * vp + w.by * vq;
    y[4] = w.rho * w.a2 * pf;
    const S bp = w.a * w.sr * (w.as * Fp - w.af * Sp);
    const S bq = w.sr * Ap;
    y[5] = w.by * bp - w.bz * bq;
    y[6] = w.bz * bp + w.by * bq;
  }

  // Wave speeds and Roe-Balsara normalization of one direction, in precision
  // R: the squared sound, normal and transverse Alfven speeds give
  //   disc = c_f^2 - c_s^2, c_f^2 = (a^2 + b^2 + disc) / 2, c_s = a c_a / c_f,
  //   alpha_f^2 and alpha_s^2 = (disc +- (a^2 - b^2)) / (2 disc), the smaller one
  // from their product a^2 b_t^2 / disc^2, without cancellation. Returns
  // whether the direction is near the triple point, where the fast and slow
  // speeds nearly meet (disc small: transverse field -> 0 and a^2 -> b_n^2
  // together). The FP32 split then takes this structure from FP64. Near the
  // other coincidences (transverse field -> 0 alone, where the fast or slow
  // speed meets the Alfven speed, or normal field -> 0) the FP32 closed form
  // stays at FP32 rounding of the FP64 split at every distance; near the
  // triple point it loses up to ~1e-6 without FP64.
  template <class R>
  struct Eig {
    R a2, a, cf, cs, ca, af, as, by, bz, bt;  // bt = |B_t|
  };
  template <class R>
  __host__ __device__ static bool eigenstructure(R rho, R p, R Bn, R By, R Bz, R gamma, Eig<R>& e) {
    const R irho = qrcp(rho);
    const R a2 = gamma * p * irho;
    const R bn2 = Bn * Bn * irho;
    const R bt2r = By * By + Bz * Bz;
    const R bt2 = bt2r * irho;
    const R b2 = bn2 + bt2;
    const R disc2 = sq(a2 - bn2) + bt2 * (R(2) * a2 + R(2) * bn2 + bt2);
    const R disc = qsqrt(disc2);
    const R tot = a2 + b2;
    const R cf2 = R(0.5) * (tot + disc);
    e.a2 = a2;
    e.a = qsqrt(a2);
    e.cf = qsqrt(cf2);
    e.ca = qsqrt(bn2);
    e.cs = cf2 > R(0) ? qdiv(e.a * e.ca, e.cf) : R(0);
    e.af = R(1);
    e.as = R(0);
    if (disc > R(0)) {
      const R diff = a2 - b2;
      const R big = R(0.5) * (fabs(diff) + disc);
      const R id = qrcp(disc);
      const R nb = qsqrt(big * id), ns = qsqrt(qdiv(a2 * bt2, big) * id);
      e.af = fmin(R(1), diff >= R(0) ? nb : ns);
      e.as = fmin(R(1), diff >= R(0) ? ns : nb);
    }
    e.by = e.bz = R(0.70710678118654752440);
    e.bt = R(0);
    if (bt2r > R(0)) {
      e.bt = qsqrt(bt2r);
      const R ibt = qrcp(e.bt);
      e.by = By * ibt;
      e.bz = Bz * ibt;
    }
    return disc2 < R(1e-4) * tot * tot;
  }

  __host__ __device__ static void split(int d, const S* Ug, const Phys& ph, S Lam, S ch, S* Fg, S* Dg) {
    const S gamma = S(ph.gamma);
    const S gm1 = gamma - S(1);
    // local frame: n = d, t1 = the other in-plane axis, t2 = z
    const int n = d, t1 = 1 - d, t2 = 2;
    const S rho = Ug[0];
    const S irho = qrcp(rho);
    const S u = Ug[1 + n] * irho, v = Ug[1 + t1] * irho, w = Ug[1 + t2] * irho;
    const S E = Ug[4];
    const S Bn = Ug[5 + n], By = Ug[5 + t1], Bz = Ug[5 + t2];
    const S psi = Ug[8];
    const S uu = u * u + v * v + w * w;
    const S BB = Bn * Bn + By * By + Bz * Bz;
    const S uB = u * Bn + v * By + w * Bz;
    const S p = gm1 * (E - S(0.5) * rho * uu - S(0.5) * BB);
    const S pt = p + S(0.5) * BB;
    // flux in the local frame
    S F[9];
    F[0] = rho * u;
    F[1] = rho * u * u + pt - Bn * Bn;
    F[2] = rho * u * v - Bn * By;
    F[3] = rho * u * w - Bn * Bz;
    F[4] = (E + pt) * u - uB * Bn;
    F[5] = psi;
    F[6] = u * By - Bn * v;
    F[7] = u * Bz - Bn * w;
    F[8] = ch * ch * Bn;
    // wave speeds and Roe-Balsara normalization; in FP32 the directions near
    // the triple point get this eigenstructure in FP64
    Eig<S> e;
    if (eigenstructure<S>(rho, p, Bn, By, Bz, gamma, e) && sizeof(S) == 4) {
      Eig<double> f;
      eigenstructure<double>(double(rho), double(p), double(Bn), double(By), double(Bz), double(gamma), f);
      e = {S(f.a2), S(f.a), S(f.cf), S(f.cs), S(f.ca), S(f.af), S(f.as), S(f.by), S(f.bz), S(f.bt)};
    }
    const S sgn = Bn >= S(0) ? S(1) : S(-1);
    // speeds (f-, a-, s-, e, s+, a+, f+) and their weights
    const S lam[7] = {u - e.cf, u - e.ca, u - e.cs, u, u + e.cs, u + e.ca, u + e.cf};
    const S lmax = fabs(u) + e.cf;
    S hk = half_k_over(ph, Lam);
    S bcp = beta_w(ch, hk, ph.kinf);
    if (ph.alpha_local) {
      hk = half_k_over(ph, S(fmax(lmax, ch)));
      bcp = beta_w(ch, hk, ph.kinf);
    }
    S b[7];
    weights(lam, lmax, hk, ph.kinf, b);
    // Coefficients in the seven primitive eigenvectors of the flux (F) and of
    // the B_n column of the Jacobian (C). Both are taken in the frame of the
    // transverse field, t = (by, bz): their transverse momentum parts lie along
    // it (xvq = 0) and most of the flux cancels in its primitive image,
    //   x_F = (rho u, (p_t - B_n^2) / rho, -B_n B_t / rho, 0,
    //          u p + (gamma - 1) (u (B_n^2 - B_t^2) / 2 + B_n B_t v_t), u B_t - B_n v_t, -B_n v_q),
    //   x_C = (0, -gamma B_n / rho, -B_t / rho, 0, (gamma - 1) B_t v_t, -v_t, -v_q).
    const S vp = e.by * v + e.bz * w, vq = e.by * w - e.bz * v;
    // (FP64: 1 / a^2 in one rounding; its square leaves D up to 8 % further off
    // than the eigenvector route was, at low Mach numbers without a field)
    const S ia = qrcp(e.a), ia2 = sizeof(S) == 8 ? qrcp(e.a2) : ia * ia, sr = qsqrt(rho), isr = sr * irho;
    const S bt = e.bt, h2 = S(0.5) * ia2, h2r = h2 * irho, has = S(0.5) * ia * isr, hsr = S(0.5) * isr;
    const S afcf = e.af * e.cf, ascs = e.as * e.cs;
    struct Coef {
      S fm, fp, sm, sp, a, e;  // f-, f+, s-, s+, a- = a+, entropy
    };
    auto expand = [&](S x0, S x1, S xvp, S x4, S xbp, S xbq) {
      const S X = x4 * h2r, Y = xbp * has, Z1 = x1 * h2, Z2 = sgn * xvp * h2;  // halves of the coefficients' sums
      const S Fp = e.af * X + e.as * Y, Sp = e.as * X - e.af * Y;
      const S Fm = afcf * Z1 - ascs * Z2, Sm = ascs * Z1 + afcf * Z2;
      return Coef{Fp - Fm, Fp + Fm, Sp - Sm, Sp + Sm, xbq * hsr, x0 - x4 * ia2};
    };
    const S x4c = gm1 * (bt * vp), x4f = u * p + gm1 * (S(0.5) * u * (Bn * Bn - bt * bt)) + Bn * x4c;
    const Coef f = expand(F[0], (pt - Bn * Bn) * irho, -Bn * bt * irho, x4f, u * bt - Bn * vp, -Bn * vq);
    const Coef c = expand(S(0), -gamma * Bn * irho, -bt * irho, x4c, -vp, -vq);
    // s_j: divided differences of the weights between lambda_j and +-c_h, times
    // the cleaning pair's coefficients (psi +- c_h B_n) / 2. Over the common
    // denominator that is one reciprocal a wave; it is used where the speeds
    // are well apart from c_h (c_h is six times the largest fast speed).
    S s[7];
    if (lmax <= S(0.5) * ch) {
      const S c2 = ch * ch, c2B = c2 * Bn, bc = bcp * ch;
#pragma unroll
      for (int j = 0; j < 7; ++j)
        s[j] = (b[j] * (lam[j] * psi + c2B) - bc * (lam[j] * Bn + psi)) * qrcp(lam[j] * lam[j] - c2);
    } else {
      const S qp = S(0.5) * (psi + ch * Bn), qm = S(0.5) * (psi - ch * Bn);
      const S bcm = beta_w(-ch, hk, ph.kinf);
#pragma unroll
      for (int j = 0; j < 7; ++j)
        s[j] = beta_dd(lam[j], b[j], ch, bcp, hk, ph.kinf) * qp + beta_dd(lam[j], b[j], -ch, bcm, hk, ph.kinf) * qm;
    }
    // the weighted sum of the eigenvectors: a primitive vector y in the same frame
    const S d0 = b[0] * f.fm + s[0] * c.fm, d6 = b[6] * f.fp + s[6] * c.fp;
    const S d2 = b[2] * f.sm + s[2] * c.sm, d4 = b[4] * f.sp + s[4] * c.sp;
    const S Fp = d6 + d0, Fm = d6 - d0, Sp = d4 + d2, Sm = d4 - d2;
    const S Ap = (b[5] + b[1]) * f.a + (s[5] + s[1]) * c.a, Am = (b[5] - b[1]) * f.a + (s[5] - s[1]) * c.a;
    const S rpf = rho * (e.af * Fp + e.as * Sp);
    const S y0 = b[3] * f.e + s[3] * c.e + rpf;
    const S y1 = afcf * Fm + ascs * Sm;
    const S yvp = sgn * (afcf * Sm - ascs * Fm), yvq = -sgn * Am;
    const S ybp = e.a * sr * (e.as * Fp - e.af * Sp), ybq = sr * Ap;
    // back to conserved variables (B_n fixed in the seven-wave block)
    S D[9];
    D[0] = y0;
    D[1] = u * y0 + rho * y1;
    D[2] = v * y0 + rho * (e.by * yvp - e.bz * yvq);
    D[3] = w * y0 + rho * (e.bz * yvp + e.by * yvq);
    D[4] = qdiv(e.a2 * rpf, gm1) + S(0.5) * uu * y0 + rho * (u * y1 + vp * yvp + vq * yvq) + bt * ybp;
    D[6] = e.by * ybp - e.bz * ybq;
    D[7] = e.bz * ybp + e.by * ybq;
    const S eta = bcp * ch;
    D[5] = eta * Bn;
    D[8] = eta * psi;
    // scatter from the local frame
    const int perm[3] = {n, t1, t2};
    Fg[0] = F[0];
    Dg[0] = D[0];
    for (int kk = 0; kk < 3; ++kk) {
      Fg[1 + perm[kk]] = F[1 + kk];
      Dg[1 + perm[kk]] = D[1 + kk];
      Fg[5 + perm[kk]] = F[5 + kk];
      Dg[5 + perm[kk]] = D[5 + kk];
    }
    Fg[4] = F[4];
    Dg[4] = D[4];
    Fg[8] = F[8];
    Dg[8] = D[8];
  }
};

// ---------------------------------------------------------------------------
// Equilibrium populations from U and the per-direction (F, D).
// 1D order (+xi, 0, -xi); 2D order (+x, -x, 0, +y, -y) (Sec. 3.1, Sec. 3.4).
// With F+ = F/2 + D and F- = F/2 - D per direction:
//   moving populations  f = c U + F+/xi  (along +d)  and  f = c U - F-/xi  (along -d),
//   rest population     f = (1 - 2 D c) U - sum_d (F+ - F-)/xi   (D = lattice dimension).
// ---------------------------------------------------------------------------
template <int KIND, int DIM, class S>
struct Equilibrium {
  using C = Cell<KIND, DIM, S>;
  static constexpr int P = C::P;
  static constexpr int Q = DIM == 1 ? 3 : 5;
  // feq[q][v]
  __host__ __device__ static void eval(const S* U, const Phys& ph, S ixi, S Lam, S ch, S (*feq)[C::P]) {
    const S c = S(ph.c);
    if (DIM == 1) {
      S F[P], D[P];
      C::split(0, U, ph, Lam, ch, F, D);
      for (int v = 0; v < P; ++v) {
        const S Fp = S(0.5) * F[v] + D[v];
        const S Fm = S(0.5) * F[v] - D[v];
        feq[0][v] = c * U[v] + Fp * ixi;
        feq[1][v] = (S(1) - S(2) * c) * U[v] - (Fp - Fm) * ixi;
        feq[2][v] = c * U[v] - Fm * ixi;
      }
    } else {
      S F1[P], D1[P], F2[P], D2[P];
      C::split(0, U, ph, Lam, ch, F1, D1);
      C::split(1, U, ph, Lam, ch, F2, D2);
      for (int v = 0; v < P; ++v) {
        const S F1p = S(0.5) * F1[v] + D1[v], F1m = S(0.5) * F1[v] - D1[v];
        const S F2p = S(0.5) * F2[v] + D2[v], F2m = S(0.5) * F2[v] - D2[v];
        feq[0][v] = c * U[v] + F1p * ixi;
        feq[1][v] = c * U[v] - F1m * ixi;
        feq[2][v] = (S(1) - S(4) * c) * U[v] - (F1p + F2p - F1m - F2m) * ixi;
        feq[3][v] = c * U[v] + F2p * ixi;
        feq[4][v] = c * U[v] - F2m * ixi;
      }
    }
  }

  // 2D: the two equilibria moving along axis d (+d into fplus, -d into
  // fminus), needing only that direction's split; the same expressions as
  // eval, so the results are bitwise those of eval.
  __host__ __device__ static void eval_axis(const S* U, const Phys& ph, S ixi, S Lam, S ch, int d, S* fplus,
                                            S* fminus) {
    const S c = S(ph.c);
    S F[P], D[P];
    C::split(d, U, ph, Lam, ch, F, D);
    for (int v = 0; v < P; ++v) {
      const S Fp = S(0.5) * F[v] + D[v], Fm = S(0.5) * F[v] - D[v];
      fplus[v] = c * U[v] + Fp * ixi;
      fminus[v] = c * U[v] - Fm * ixi;
    }
  }

  // The same for solves that keep U (no stored population to agree with): f+-
  // as (c U + D / xi) +- F / (2 xi), four operations a value where the form
  // above takes six, and F+ - F- = 2 D, what the rest population gives up.
  __host__ __device__ static void eval_axis_net(const S* U, const Phys& ph, S ixi, S Lam, S ch, int d, S* fplus,
                                                S* fminus, S* net) {
    const S c = S(ph.c), hx = S(0.5) * ixi;
    S F[P], D[P];
    C::split(d, U, ph, Lam, ch, F, D);
    for (int v = 0; v < P; ++v) {
      const S h = hx * F[v];
      const S s = D[v] * ixi + c * U[v];
      fplus[v] = s + h;
      fminus[v] = s - h;
      net[v] = D[v] + D[v];
    }
  }
};

}  // namespace vklb
