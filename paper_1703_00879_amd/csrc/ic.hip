// Growth factors (FP64) and the Gaussian initial conditions.
//
// Growth (Secs. 3.1, 4.1, 4.2, App. B): per Fourier mode,
//   D1'' = kappa mu(k,a) D1,
//   D2'' = kappa mu D2 - kappa mu D1^2 [1 + 2 a^4 H^2 gamma_2(k, k/sqrt2, k/sqrt2, a)/(kappa mu)],
// primes d/dtau, kappa = 1.5 Omega_m a, with the Einstein-de Sitter growing-mode values at
// a_ini (D1 = 1, D1' = a^2 E, D2 = -3/7, D2' = -(6/7) a^2 E).  One thread integrates one
// integer |nu|^2 of the particle grid (k = 2 pi |nu| / L) in ln a with steps that end
// exactly on every a_i of the time grid (eighth-order extrapolation, see the growth tables
// below); the triangle solver takes classical fourth-order Runge-Kutta steps <= 1e-3.
//
// Initial field: counter-based SplitMix64 white noise (Steele, Lea & Flood 2014) with a
// Box-Muller transform, scaled in Fourier space by sqrt(N P_ini(k) / L^3), where P_ini is
// the Eisenstein-Hu no-wiggle spectrum normalised to sigma8 at z = 0 and divided by the
// square of the LCDM growth factor D1(a = 1) of the same ODE.

#include <algorithm>
#include <cmath>
#include <vector>

#include "internal.h"

namespace cola {

constexpr double kH0c = 1.0 / 2997.92458;   // H0/c in h/Mpc

struct GrowthDev {
  double om, fr0, rc, a_ini, kf;
  double sb, sm, sa;  // symmetron beta_*, m_*/H0, a_*
  double kb, kk0, kx0, kxn;   // k-Mouflage beta, K0, X(a) = kx0 a^kxn
  int km;                     // k-Mouflage exponent m
  int model;          // effective model for the growth (LCDM when growth_mode = 1)
  int kdep;           // table indexed by |nu|^2
  int n_steps;
  int64_t n_k;
};

__device__ __forceinline__ double dE(double a, double om) { return sqrt(om / (a * a * a) + 1.0 - om); }

// One classical fourth-order Runge-Kutta step of length h in ln a.
template <int NV, class Rhs>
__device__ __forceinline__ void rk4_step(double* y, double lna, double h, const Rhs& rhs) {
  double k1[NV], k2[NV], k3[NV], k4[NV], yt[NV];
  rhs(lna, y, k1);
  for (int c = 0; c < NV; ++c) yt[c] = y[c] + 0.5 * h * k1[c];
  rhs(lna + 0.5 * h, yt, k2);
  for (int c = 0; c < NV; ++c) yt[c] = y[c] + 0.5 * h * k2[c];
  rhs(lna + 0.5 * h, yt, k3);
  for (int c = 0; c < NV; ++c) yt[c] = y[c] + h * k3[c];
  rhs(lna + h, yt, k4);
  for (int c = 0; c < NV; ++c) y[c] += h / 6.0 * (k1[c] + 2.0 * k2[c] + 2.0 * k3[c] + k4[c]);
}

// RK4 in ln a from lna to le in equal steps <= 1e-3.
template <int NV, class Rhs>
__device__ __forceinline__ void rk4_segment(double* y, double& lna, double le, const Rhs& rhs) {
  const int nsub = (int)ceil((le - lna) / 1e-3);
  if (nsub <= 0) return;
  const double h = (le - lna) / nsub;
  for (int s = 0; s < nsub; ++s) {
    rk4_step<NV>(y, lna, h, rhs);
    lna = (s + 1 == nsub) ? le : lna + h;
  }
}

// RK4 from lna to l1 for a right-hand side that switches on at l_kink (the symmetron at
// a_*; -1e300 for the other models).  A step boundary falls exactly on l_kink.  Just after
// it the symmetron's gamma_2 term has a peak whose width in ln a scales as
// (k / (a_* m_*))^2, far below 1e-3 for the fundamental mode of a large box; the steps
// there start at 1e-10 and grow geometrically (h = 1e-10 + 0.02 (ln a - l_kink)) until
// they reach the 1e-3 of the rest of the integration.
template <int NV, class Rhs>
__device__ __forceinline__ void rk4_to(double* y, double& lna, double l1, double l_kink, const Rhs& rhs) {
  if (lna < l_kink && l_kink < l1) rk4_segment<NV>(y, lna, l_kink, rhs);
  if (lna >= l_kink) {
    while (lna < l1) {
      const double h = 1e-10 + 0.02 * (lna - l_kink);
      if (h >= 1e-3) break;
      if (h >= l1 - lna) {
        rk4_step<NV>(y, lna, l1 - lna, rhs);
        lna = l1;
      } else {
        rk4_step<NV>(y, lna, h, rhs);
        lna += h;
      }
    }
  }
  rk4_segment<NV>(y, lna, l1, rhs);
}

// RK4 from lna to l1 (as rk4_to) with a step boundary on every knot of a tabulated
// {m, beta} model in between: the splines' third derivatives jump there, which a step
// across a knot would integrate at lower order.
template <int NV, class Rhs>
__device__ __forceinline__ void rk4_to_knots(double* y, double& lna, double l1, double l_kink,
                                             const GrowthDev& g, const MBSpline& mb, const Rhs& rhs) {
  if (g.model == COLA_MBETA) {
    for (int j = 0; j < mb.n; ++j)
      if (mb.x[j] > lna && mb.x[j] < l1) rk4_to<NV>(y, lna, mb.x[j], l_kink, rhs);
  }
  rk4_to<NV>(y, lna, l1, l_kink, rhs);
}

__device__ __forceinline__ double growth_kink(const GrowthDev& g) {
  return g.model == COLA_SYMMETRON ? log(g.sa) : -1e300;
}

// mu(k, a) of the model (Secs. 5.1, 5.2, App. C)
__device__ __forceinline__ double growth_mu(const GrowthDev& g, const MBSpline& mb, double k, double a) {
  if (g.model == COLA_FR_HS1) {
    const double ol = 1.0 - g.om;
    const double X = g.om / (a * a * a) + 4.0 * ol, Y = g.om + 4.0 * ol;
    const double r = X / Y;
    const double a2m2 = a * a * kH0c * kH0c * Y * r * r * r / (2.0 * g.fr0);
    return 1.0 + k * k / (3.0 * (k * k + a2m2));
  }
  if (g.model == COLA_NDGP) {
    const double E = dE(a, g.om);
    const double oma = g.om / (a * a * a) / (E * E);
    return 1.0 + 1.0 / (3.0 * (1.0 + 2.0 * g.rc * E * (1.0 - 0.5 * oma)));
  }
  if (g.model == COLA_KMOUFLAGE) {   // App. B: 1 + 2 beta^2 / P_X(X(a)), P_X = 1 + m K0 X^(m-1)
    const double X = g.kx0 * pow(a, g.kxn);
    return 1.0 + 2.0 * g.kb * g.kb / (1.0 + g.km * g.kk0 * pow(X, (double)(g.km - 1)));
  }
  if (g.model == COLA_MBETA) {   // App. C: 1 + 2 beta^2 k^2/(k^2 + a^2 m^2), tabulated
    double b, m2, dm2;
    mb_eval(mb, a, b, m2, dm2);
    const double a2m2 = a * a * kH0c * kH0c * m2;
    return 1.0 + 2.0 * b * b * k * k / (k * k + a2m2);
  }
  if (g.model == COLA_SYMMETRON) {   // App. C: 1 + 2 beta^2 k^2/(k^2 + a^2 m^2)
    if (a <= g.sa) return 1.0;
    const double r = g.sa / a, s = 1.0 - r * r * r;
    const double a2m2 = a * a * kH0c * kH0c * g.sm * g.sm * s;
    return 1.0 + 2.0 * g.sb * g.sb * s * k * k / (k * k + a2m2);
  }
  return 1.0;
}

// 2 a^4 H^2 gamma_2^E(k, k1, k2, a) (Secs. 5.1, 5.2); c2 = cos^2 theta
__device__ __forceinline__ double gamma2E_term(const GrowthDev& g, const MBSpline& mb, double k, double k1,
                                               double k2, double c2, double a) {
  const double E = dE(a, g.om);
  const double a6 = (a * a * a) * (a * a * a);
  double g2 = 0.0;
  if (g.model == COLA_FR_HS1) {
    const double ol = 1.0 - g.om;
    const double X = g.om / (a * a * a) + 4.0 * ol, Y = g.om + 4.0 * ol;
    const double c0 = X * X * X / (2.0 * g.fr0 * Y * Y);
    const double ah = a * kH0c;
    const double P = k * k / (ah * ah) + c0, P1 = k1 * k1 / (ah * ah) + c0, P2 = k2 * k2 / (ah * ah) + c0;
    const double kah = k / (ah * E);
    g2 = -9.0 * g.om * g.om / (48.0 * a6 * g.fr0 * g.fr0) * kah * kah * (X * X * X * X * X) / (Y * Y * Y * Y)
         / (P * P1 * P2);
  } else if (g.model == COLA_NDGP) {
    const double oma = g.om / (a * a * a) / (E * E);
    const double beta = 1.0 + 2.0 * g.rc * E * (1.0 - 0.5 * oma);
    g2 = -(g.rc * g.rc * g.om * g.om) / (6.0 * E * E * beta * beta * beta * a6) * (1.0 - c2);
  } else if (g.model == COLA_MBETA) {
    // App. C with the tabulated beta, m^2/H0^2 and d(m^2/H0^2)/da
    double b, m2, dm2;
    mb_eval(mb, a, b, m2, dm2);
    const double ah = a * kH0c;
    const double P = k * k / (ah * ah) + m2, P1 = k1 * k1 / (ah * ah) + m2, P2 = k2 * k2 / (ah * ah) + m2;
    const double H = E * kH0c;
    g2 = m2 * dm2 * b * b * g.om / (2.0 * P * P1 * P2) * k * k / (a * a * a * a * H * H);
  } else if (g.model == COLA_SYMMETRON && a > g.sa) {
    // App. C: m^2 (dm^2/da) beta^2 Om / (2 H0^4 Pi Pi Pi) k^2/(a^4 H^2), Pi(q) = (q/(aH0))^2 + m^2/H0^2
    const double r = g.sa / a, s = 1.0 - r * r * r;
    const double m2 = g.sm * g.sm * s, dm2 = g.sm * g.sm * 3.0 * g.sa * g.sa * g.sa / (a * a * a * a);
    const double ah = a * kH0c;
    const double P = k * k / (ah * ah) + m2, P1 = k1 * k1 / (ah * ah) + m2, P2 = k2 * k2 / (ah * ah) + m2;
    const double H = E * kH0c;
    g2 = m2 * dm2 * g.sb * g.sb * s * g.om / (2.0 * P * P1 * P2) * k * k / (a * a * a * a * H * H);
  }
  return 2.0 * a * a * a * a * E * E * g2;
}

// mu(k, a) and 2 a^4 H^2 gamma_2(k, k/sqrt2, k/sqrt2, a) for the growth equations
__device__ __forceinline__ void growth_model(const GrowthDev& g, const MBSpline& mb, double k, double a,
                                             double& mu, double& g2term) {
  const double E = dE(a, g.om);
  if (g.model == COLA_FR_HS1) {
    const double ol = 1.0 - g.om;
    const double X = g.om / (a * a * a) + 4.0 * ol, Y = g.om + 4.0 * ol;
    const double r = X / Y;
    const double a2m2 = a * a * kH0c * kH0c * Y * r * r * r / (2.0 * g.fr0);
    const double k2 = k * k;
    mu = 1.0 + k2 / (3.0 * (k2 + a2m2));
    // gamma_2^E (Sec. 5.1) at k1 = k2 = k/sqrt2
    const double c0 = X * X * X / (2.0 * g.fr0 * Y * Y);
    const double ah = a * kH0c;
    const double Pk = k2 / (ah * ah) + c0;
    const double Ph = 0.5 * k2 / (ah * ah) + c0;
    const double kah = k / (ah * E);
    const double X5Y4 = (X * X * X * X * X) / (Y * Y * Y * Y);
    const double g2 = -9.0 * g.om * g.om / (48.0 * ((a * a * a) * (a * a * a)) * g.fr0 * g.fr0) * kah * kah * X5Y4
                      / (Pk * Ph * Ph);
    g2term = 2.0 * a * a * a * a * E * E * g2;
  } else if (g.model == COLA_NDGP) {
    const double oma = g.om / (a * a * a) / (E * E);
    const double beta = 1.0 + 2.0 * g.rc * E * (1.0 - 0.5 * oma);
    mu = 1.0 + 1.0 / (3.0 * beta);
    const double g2 = -(g.rc * g.rc * g.om * g.om) / (6.0 * E * E * beta * beta * beta * ((a * a * a) * (a * a * a)));
    g2term = 2.0 * a * a * a * a * E * E * g2;
  } else if (g.model == COLA_KMOUFLAGE) {   // gamma_2 = 0
    mu = growth_mu(g, mb, k, a);
    g2term = 0.0;
  } else if (g.model == COLA_SYMMETRON || g.model == COLA_MBETA) {
    mu = growth_mu(g, mb, k, a);
    g2term = gamma2E_term(g, mb, k, k * M_SQRT1_2, k * M_SQRT1_2, 0.0, a);
  } else {
    mu = 1.0;
    g2term = 0.0;
  }
}

// ------------------------------------------------------------------ growth tables
// y = (D1, D1', D2, D2') per |nu|^2, ' = d/dtau, integrated in ln a by Gragg-Bulirsch-Stoer
// steps of order 8: modified midpoint with 2, 4, 6 and 8 substeps over the same step,
// extrapolated in the substep squared.  Every sequence needs the right-hand side at
// rational points of the step only, and at a point the equations depend on the mode through
// k^2 alone:
//   mu = mu_0 + c_1 k^2/(k^2 + m),  gamma_2 term = s + G k^2/((k^2 + m)(k^2/2 + m)^2)
// with m = a^2 m^2 (no mode dependence where c_1 = G = 0).  So k_growth_nodes evaluates the
// model's functions of a once per point, for all modes, and k_growth_ode reads them from
// LDS: two reciprocals and about thirty FP64 operations per mode and point.
//
// What bounds it: up to about 10^5 modes (a wave or two per SIMD) the latency of one mode's
// chain of steps, so few, wide steps whose four sequences advance independently.  Measured
// on a whole table from z = 19: LCDM, 10 slices, 6.5 -> 0.08 ms (0.24 with the divisions of
// the mode terms, which one mode at k = 0 does not need), against
// fourth-order Runge-Kutta steps of 1e-3 that evaluated the model in full for every mode
// and stage.  Steps of 0.04 hold the largest relative error of any LCDM, nDGP or symmetron
// entry at 1e-13 (the Runge-Kutta steps: 4e-13, 9e-12 for the symmetron); it is truncation
// from 0.05 on, rounding below.  Models whose coefficients vary faster take the shorter steps
// of growth_step_bound().  f(R) modes keep the Runge-Kutta steps (further below).
constexpr double kGrowthStep = 0.04;     // longest step in ln a
constexpr double kGrowthFloor = 5e-4;    // no step bound is below this, half a Runge-Kutta step,
constexpr int kGrowthFine = 20000;       // nor below the range of ln a over this number
constexpr double kGradeFirst = 1e-10;    // after a_*: steps kGradeFirst + kGrade (ln a - ln a_*)
constexpr double kGrade = 0.1;           // (error 3e-13; 0.2 gives 7e-13, 0.3 1e-11)
constexpr int kGrowthNodes = 13;         // points of a step: 0 ... 7/8 of the sequences, and 1
constexpr int kGrowthChunk = 128;        // steps per k_growth_nodes launch (kernel arguments)
constexpr int kGrowthRound = 16;         // steps staged in LDS at a time

// Functions of a at one point, each times f = d tau / d ln a where it multiplies y:
// y_0' = f y_1, y_1' = q y_0 with q = A + B k^2 R, and the D2 source (q + g) y_0^2 with
// g = s + G k^2 R Q^2, R = 1/(k^2 + m), Q = 1/(k^2/2 + m).  kap: f kappa (LCDM's q).
// ext: the step length (point 0) and the slice written after the step, or -1 (point 12).
struct __align__(16) GrowthNode {
  double f, kap, A, B, m, s, G, ext;
};

// Consecutive steps: step j runs from l[j] to l[j + 1] in ln a.
struct GrowthSteps {
  int n, first;
  double l[kGrowthChunk + 1];
  int16_t out[kGrowthChunk];
};

__device__ __forceinline__ GrowthNode growth_node(const GrowthDev& g, const MBSpline& mb, double lna) {
  const double a = exp(lna);
  const double E = dE(a, g.om);
  const double f = 1.0 / (a * a * E), kap = 1.5 * g.om * a;
  const double ah = a * kH0c, ah2 = ah * ah, a3 = a * a * a;
  double mu0 = 1.0, c1 = 0.0, m = 1.0, s = 0.0, G = 0.0;
  if (g.model == COLA_FR_HS1) {
    const double ol = 1.0 - g.om;
    const double X = g.om / a3 + 4.0 * ol, Y = g.om + 4.0 * ol;
    const double r = X / Y;
    m = ah2 * Y * r * r * r / (2.0 * g.fr0);
    c1 = 1.0 / 3.0;
    // gamma_2^E (Sec. 5.1): the c_0 of its Pi(k) = k^2/(a H0)^2 + c_0 is m/(a H0)^2
    G = -18.0 * g.om * g.om * a / (48.0 * a3 * g.fr0 * g.fr0) * (X * X * X * X * X) / (Y * Y * Y * Y) * ah2 * ah2;
  } else if (g.model == COLA_NDGP) {
    const double oma = g.om / a3 / (E * E);
    const double beta = 1.0 + 2.0 * g.rc * E * (1.0 - 0.5 * oma);
    mu0 = 1.0 + 1.0 / (3.0 * beta);
    s = -(g.rc * g.rc * g.om * g.om) / (3.0 * beta * beta * beta * a * a);
  } else if (g.model == COLA_KMOUFLAGE) {   // gamma_2 = 0
    mu0 = growth_mu(g, mb, 0.0, a);
  } else if (g.model == COLA_MBETA || (g.model == COLA_SYMMETRON && a > g.sa)) {
    double b2, m2, dm2;   // beta^2, m^2/H0^2 and its derivative in a
    if (g.model == COLA_MBETA) {
      double b;
      mb_eval(mb, a, b, m2, dm2);
      b2 = b * b;
    } else {
      const double r = g.sa / a, sv = 1.0 - r * r * r;
      b2 = g.sb * g.sb * sv;
      m2 = g.sm * g.sm * sv;
      dm2 = g.sm * g.sm * 3.0 * g.sa * g.sa * g.sa / (a * a3);
    }
    m = ah2 * m2;
    c1 = 2.0 * b2;
    G = m2 * dm2 * b2 * g.om * ah2 * ah2 * ah2 / (kH0c * kH0c);
  }
  return GrowthNode{f, f * kap, f * kap * mu0, f * kap * c1, m, f * s, f * G, 0.0};
}

__global__ void __launch_bounds__(64)
k_growth_nodes(GrowthDev g, MBSpline mb, GrowthSteps st, GrowthNode* __restrict__ nodes) {
  constexpr double at[kGrowthNodes] = {0.0,     1.0 / 8, 1.0 / 6, 1.0 / 4, 1.0 / 3, 3.0 / 8, 1.0 / 2,
                                       5.0 / 8, 2.0 / 3, 3.0 / 4, 5.0 / 6, 7.0 / 8, 1.0};
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = e / kGrowthNodes, i = e % kGrowthNodes;
  if (j >= st.n) return;
  const double l0 = st.l[j], l1 = st.l[j + 1], h = l1 - l0;
  GrowthNode nd = growth_node(g, mb, i + 1 == kGrowthNodes ? l1 : l0 + at[i] * h);
  if (i == 0) nd.ext = h;
  if (i + 1 == kGrowthNodes) nd.ext = (double)st.out[j];
  nodes[(int64_t)(st.first + j) * kGrowthNodes + i] = nd;
}

// One mode's coefficients at a point; HALF (the COLA_READ_D2_HALF_K reading): y also
// carries (D1, D1') at k/sqrt2, whose q is qh, and the D2 source takes that D1 squared in
// place of D1(k)^2.
// KDEP: the table has an entry per mode; else k = 0, where the terms in R and Q vanish.
template <bool HALF, bool KDEP>
struct GrowthMode {
  double f, q, g, qh;
  __device__ __forceinline__ GrowthMode(const GrowthNode& n, double k2, bool ref) {
    if constexpr (!KDEP) {
      f = n.f;
      q = qh = ref ? n.kap : n.A;
      g = ref ? 0.0 : n.s;
      return;
    }
    const double R = 1.0 / (k2 + n.m), Q = 1.0 / (0.5 * k2 + n.m);
    f = n.f;
    q = ref ? n.kap : n.A + n.B * (k2 * R);
    g = ref ? 0.0 : n.s + n.G * (k2 * R) * (Q * Q);
    qh = HALF ? (ref ? n.kap : n.A + n.B * (0.5 * k2 * Q)) : 0.0;
  }
  // zm + h y'(z)
  __device__ __forceinline__ void midpoint(double* zm, double* z, double h) const {
    const double ds = HALF ? z[4] : z[0];
    const double d[4] = {f * z[1], q * z[0], f * z[3], q * z[2] - (q + g) * (ds * ds)};
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double t = zm[v] + h * d[v];
      zm[v] = z[v];
      z[v] = t;
    }
    if constexpr (HALF) {
      const double t4 = zm[4] + h * (f * z[5]), t5 = zm[5] + h * (qh * z[4]);
      zm[4] = z[4];
      zm[5] = z[5];
      z[4] = t4;
      z[5] = t5;
    }
  }
};

// one slice of the table from the state y at the point of `nd`
template <bool HALF, bool KDEP>
__device__ __forceinline__ void growth_store(const GrowthNode& nd, double k2, bool ref, const double* y,
                                             double* out) {
  const GrowthMode<HALF, KDEP> c(nd, k2, ref);
  const double ds = HALF ? y[4] : y[0];
  const double tau = 1.0 / c.f;   // D'' is per tau
  out[0] = y[0];
  out[1] = y[1];
  out[2] = c.q * tau * y[0];
  out[3] = y[2];
  out[4] = y[3];
  out[5] = (c.q * y[2] - (c.q + c.g) * (ds * ds)) * tau;
}

// Eisenstein & Hu (1998) no-wiggle spectrum in double precision: constants of k^ns T(k)^2.
struct SpecDev {
  double ns, th2, omh, alpha, kfac, s8;   // th2 = (T_CMB/2.7 K)^2, kfac = 0.43 s h (s in Mpc)
  __device__ __forceinline__ double power(double k) const {
    const double kk = kfac * k;
    const double k4 = (kk * kk) * (kk * kk);
    const double gam = omh * (alpha + (1.0 - alpha) / (1.0 + k4));
    const double q = k * th2 / gam;
    const double L0 = log(2.0 * 2.718281828459045235 + 1.8 * q);
    const double C0 = 14.2 + 731.0 / (1.0 + 62.5 * q);
    const double T = L0 / (L0 + C0 * q * q);
    return pow(k, ns) * T * T;
  }
};

// A with sigma8^2 = A int d ln k k^3/(2 pi^2) k^ns T^2 W(8 k)^2 over 1e-5 < k < 1e2 h/Mpc, by
// 16-point Gauss-Legendre panels: kSpecLow equal ones in ln k up to kSpecSplit, then kSpecHigh
// equal ones in k, whose 8 rad of the top-hat's phase each keeps the rule converged (relative
// difference from 4000 panels in ln k 1e-13, 1e-10 for n_s near -3).  One wave, a panel node per
// lane and turn.
constexpr int kSpecLow = 64, kSpecHigh = 96;
constexpr double kSpecSplit = 0.5;
__device__ __forceinline__ double sigma8_norm(const SpecDev& sp) {
  constexpr double gx[8] = {0.09501250983763745, 0.2816035507792589, 0.45801677765722737,
                            0.6178762444026438,  0.755404408355003,  0.8656312023878318,
                            0.9445750230732326,  0.9894009349916499};
  constexpr double gw[8] = {0.18945061045506859, 0.1826034150449236,  0.16915651939500262,
                            0.14959598881657676, 0.12462897125553403, 0.09515851168249259,
                            0.062253523938647706, 0.027152459411754037};
  const double l0 = log(1e-5), lm = log(kSpecSplit);
  double sum = 0.0;
  for (int e = (int)threadIdx.x; e < (kSpecLow + kSpecHigh) * 16; e += 64) {
    const int pnl = e >> 4, n = e & 7;
    double a, b;   // the panel in ln k
    if (pnl < kSpecLow) {
      a = l0 + pnl * ((lm - l0) / kSpecLow);
      b = l0 + (pnl + 1) * ((lm - l0) / kSpecLow);
    } else {
      const double dk = (1e2 - kSpecSplit) / kSpecHigh;
      a = log(kSpecSplit + (pnl - kSpecLow) * dk);
      b = log(kSpecSplit + (pnl - kSpecLow + 1) * dk);
    }
    const double x = (e & 8) ? gx[n] : -gx[n];
    const double k = exp(0.5 * (a + b) + 0.5 * (b - a) * x);
    const double y = 8.0 * k;
    const double W = y > 1e-4 ? 3.0 * (sin(y) - y * cos(y)) / (y * y * y) : 1.0 - y * y / 10.0;
    sum += 0.5 * (b - a) * gw[n] * (k * k * k * sp.power(k) * W * W);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  return sp.s8 * sp.s8 * (2.0 * M_PI * M_PI) / sum;
}

// Thread t integrates |nu|^2 = t (t == n_k: the LCDM reference of the initial spectrum, of
// which only the state at a = 1 is kept).  The substep points of the four sequences are
// visited in ascending order, so that each point's coefficients are formed once and used
// by every sequence that has a substep there.  The last work-group computes the spectrum's
// normalisation into ref_out[6] meanwhile: it is done well before the tables, and the host,
// whose own quadrature took 4-5 ms a run, only launches.
template <bool HALF, bool KDEP>
__global__ void __launch_bounds__(64)
k_growth_ode(GrowthDev g, SpecDev sp, const GrowthNode* __restrict__ nodes, int nsteps,
             double* __restrict__ table, double* __restrict__ ref_out) {
  if (blockIdx.x + 1 == gridDim.x) {
    const double A = sigma8_norm(sp);
    if (threadIdx.x == 0) ref_out[6] = A;
    return;
  }
  constexpr int NV = HALF ? 6 : 4, NS = 4;
  // extrapolation weights prod_{i != j} n_j^2/(n_j^2 - n_i^2) of n = 2, 4, 6, 8
  constexpr double wt[NS] = {-1.0 / 360.0, 16.0 / 45.0, -729.0 / 280.0, 1024.0 / 315.0};
  __shared__ GrowthNode nd[kGrowthRound * kGrowthNodes];
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const bool ref = t >= g.n_k, store = t < g.n_k;
  const double k2 = (ref || !g.kdep) ? 0.0 : g.kf * g.kf * (double)t;
  const double ai = g.a_ini;
  const double g0 = ai * ai * dE(ai, g.om);
  double y[NV];
  y[0] = 1.0;
  y[1] = g0;
  y[2] = -3.0 / 7.0;
  y[3] = -6.0 / 7.0 * g0;
  if constexpr (HALF) {
    y[4] = 1.0;
    y[5] = g0;
  }
  for (int s0 = 0; s0 < nsteps; s0 += kGrowthRound) {
    const int ns = nsteps - s0 < kGrowthRound ? nsteps - s0 : kGrowthRound;
    __syncthreads();   // the previous round's points have been read
    {
      constexpr int V = sizeof(GrowthNode) / sizeof(double2);
      const double2* src = reinterpret_cast<const double2*>(nodes + (int64_t)s0 * kGrowthNodes);
      double2* dst = reinterpret_cast<double2*>(nd);
      for (int e = threadIdx.x; e < ns * kGrowthNodes * V; e += blockDim.x) dst[e] = src[e];
    }
    __syncthreads();
    if (s0 == 0 && store) growth_store<HALF, KDEP>(nd[0], k2, ref, y, table + t * 6);
    for (int s = 0; s < ns; ++s) {
      const GrowthNode* p = nd + s * kGrowthNodes;
      const double H = p[0].ext;
      double zm[NS][NV], z[NS][NV];
#pragma unroll
      for (int j = 0; j < NS; ++j)
#pragma unroll
        for (int v = 0; v < NV; ++v) zm[j][v] = z[j][v] = y[v];
      // sequence j (2 j + 2 substeps) from point i to its next one; the first substep is an
      // Euler step of half the midpoint's length
      auto sub = [&](int i, int j, const GrowthMode<HALF, KDEP>& c) {
        const double h = H / (double)(2 * j + 2);
        c.midpoint(zm[j], z[j], i == 0 ? h : 2.0 * h);
      };
      // sequences with a substep at each point (bit j: 2 j + 2 substeps)
      constexpr int who[kGrowthNodes - 1] = {15, 8, 4, 2 | 8, 4, 8, 15, 8, 4, 2 | 8, 4, 8};
#pragma unroll
      for (int i = 0; i < kGrowthNodes - 1; ++i) {
        const GrowthMode<HALF, KDEP> c(p[i], k2, ref);
#pragma unroll
        for (int j = 0; j < NS; ++j)
          if ((who[i] >> j) & 1) sub(i, j, c);
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) y[v] = (wt[0] * z[0][v] + wt[1] * z[1][v]) + (wt[2] * z[2][v] + wt[3] * z[3][v]);
      const int out = (int)p[kGrowthNodes - 1].ext;   // uniform over the work-group
      if (out >= 0 && store) growth_store<HALF, KDEP>(p[kGrowthNodes - 1], k2, ref, y, table + ((int64_t)out * g.n_k + t) * 6);
    }
    if (t == g.n_k && s0 + ns == nsteps) growth_store<HALF, KDEP>(nd[ns * kGrowthNodes - 1], k2, ref, y, ref_out);
  }
}

// ------------------------------------------------------------------ growth tables of f(R) modes
// f(R) with its own growth has a table entry per mode and slice, up to 10^7 of them, each
// rounded to FP32 for the step's LPT coefficients.  They come from fourth-order Runge-Kutta
// steps <= 1e-3 in ln a, and keep those values to the last bit: an entry that rounds to
// another FP32 value changes every particle of a run, if only in its last digits.  What is
// shared is the model.  k_growth_fr_points evaluates the functions of a once per point;
// k_growth_fr takes 64 modes a work-group and works through the steps in chunks of
// kFrChunk as a pipeline of its waves,
//   waves 1-3  kappa mu and the gamma_2 term of every mode at the chunk's points,
//   wave 0     the Runge-Kutta steps of the chunk before,
// a lane a mode, with one barrier a chunk.  The step's own chain of 76 FP64 operations bounds
// small grids, the sum of the waves' operations large ones: 10.2 -> 0.55 ms for the 769
// modes of 32^3 particles, 18.6 -> 2.6 ms for the 110593 of 384^3 (before, one thread a
// mode evaluated the model in full at every stage).
constexpr int kFrChunk = 10;
constexpr int kFrPoints = 2 * kFrChunk + 2;   // start, (middle, end) a step, and the slice's a

// Functions of a that do not depend on the mode, in the groupings the mode's terms take them;
// r_hh and r_hE are the reciprocals of (a H0)^2 and a H0 E.
struct FrPoint {
  double f, kap, a2m2, c0, ahah, r_hh, ahE, r_hE, C0, X5Y4, G0, pad;
};
constexpr int kFrWords = sizeof(FrPoint) / sizeof(double2);

// One integration: slices i at a_i, each reached from the one before in nsub equal steps.
// Its points lie at off(i): the start, then (middle, end) of every step, then the slice's a.
struct FrPlan {
  double ai, l0;
  int n_steps;
  bool ref;   // the LCDM reference: one slice, at a = 1
  __device__ __forceinline__ FrPlan(const GrowthDev& g, bool is_ref)
      : ai(g.a_ini), l0(log(g.a_ini)), n_steps(g.n_steps), ref(is_ref) {}
  __device__ __forceinline__ int slices() const { return ref ? 1 : n_steps + 1; }
  __device__ __forceinline__ double a(int i) const { return ref ? 1.0 : ai + i * (1.0 - ai) / n_steps; }
  __device__ __forceinline__ double from(int i) const { return i == 0 ? l0 : log(a(i - 1)); }
  __device__ __forceinline__ int nsub(double lna, double le) const {
    const int n = (int)ceil((le - lna) / 1e-3);
    return n > 0 ? n : 0;
  }
  // a bound on the points of the slices before i (each needs 2 nsub + 2)
  __device__ __forceinline__ int64_t off(int i) const {
    return 2 * ((int64_t)((from(i) - l0) / 1e-3) + i) + 4 * (int64_t)i;
  }
};
// points of both integrations: the bound off() takes at the end, twice over a's range
static int64_t fr_points(const cola_params& p) {
  return 4 * (int64_t)(std::log1p(p.z_init) / 1e-3) + 6 * ((int64_t)p.n_steps + 4);
}
// The runs that take these steps.  Before ln a = -40 the gamma_2 term leaves the range of a double
// (it is not a number with either solver), so no usable run lies beyond the limit, which bounds
// the points (27 MB).
static bool fr_pipeline(const cola_params& p) {
  return p.model == COLA_FR_HS1 && p.growth_mode == 0 && !(p.readings & COLA_READ_D2_HALF_K) &&
         std::log1p(p.z_init) <= 64.0;
}
__device__ __forceinline__ int64_t fr_ref_base(const FrPlan& pl) {   // the reference's points follow
  return 2 * ((int64_t)((log(1.0) - pl.l0) / 1e-3)) + 6 * ((int64_t)pl.n_steps + 2);
}

__global__ void __launch_bounds__(256) k_growth_fr_points(GrowthDev g, FrPoint* __restrict__ pts) {
  const bool ref = blockIdx.x + 1 == gridDim.x;
  const FrPlan pl(g, ref);
  const int i = ref ? 0 : blockIdx.x;
  FrPoint* out = pts + (ref ? fr_ref_base(pl) : pl.off(i));
  const double lna0 = pl.from(i), le = log(pl.a(i));
  const int nsub = pl.nsub(lna0, le);
  const double h = (le - lna0) / nsub;
  for (int e = blockIdx.y * blockDim.x + threadIdx.x; e < 2 * nsub + 2; e += gridDim.y * blockDim.x) {
    const int j = e == 0 ? 0 : (e - 1) / 2;
    double l = lna0;   // ln a of step j, added up step by step as the integration does
#pragma unroll 16
    for (int at = 0; at < j; ++at) l += h;
    double x = l;
    if (e > 0) x = (e & 1) ? l + 0.5 * h : l + h;
    const double a = e == 2 * nsub + 1 ? pl.a(i) : exp(x);
    const double E = dE(a, g.om);
    FrPoint p;
    p.kap = 1.5 * g.om * a;
    p.f = 1.0 / (a * a * E);
    const double ol = 1.0 - g.om;
    const double X = g.om / (a * a * a) + 4.0 * ol, Y = g.om + 4.0 * ol;
    const double r = X / Y;
    p.a2m2 = a * a * kH0c * kH0c * Y * r * r * r / (2.0 * g.fr0);
    p.c0 = X * X * X / (2.0 * g.fr0 * Y * Y);
    const double ah = a * kH0c;
    p.ahah = ah * ah;
    p.r_hh = 1.0 / p.ahah;
    p.ahE = ah * E;
    p.r_hE = 1.0 / p.ahE;
    p.C0 = -9.0 * g.om * g.om / (48.0 * ((a * a * a) * (a * a * a)) * g.fr0 * g.fr0);
    p.X5Y4 = (X * X * X * X * X) / (Y * Y * Y * Y);
    p.G0 = 2.0 * a * a * a * a * E * E;
    p.pad = 0.0;
    out[e] = p;
  }
}

// x / d correctly rounded, from r = 1/d correctly rounded (Markstein's theorem: one corrected
// product; no overflow or underflow in the ranges of k, a H0 and E)
__device__ __forceinline__ double div_by(double x, double d, double r) {
  const double q = x * r;
  return fma(fma(-d, q, x), r, q);
}

__global__ void __launch_bounds__(256)
k_growth_fr(GrowthDev g, SpecDev sp, const FrPoint* __restrict__ pts, double* __restrict__ table,
            double* __restrict__ ref_out) {
  __shared__ __align__(16) FrPoint pt[3][kFrPoints];
  __shared__ double2 md[2][kFrPoints][64];   // (kappa mu, gamma_2 term) per mode
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (blockIdx.x + 1 == gridDim.x) {
    if (wave == 0) {
      const double A = sigma8_norm(sp);
      if (lane == 0) ref_out[6] = A;
    }
    return;
  }
  const bool ref = blockIdx.x + 2 == gridDim.x;
  const FrPlan pl(g, ref);
  const int64_t t = ref ? g.n_k : blockIdx.x * (int64_t)64 + lane;
  const double k = ref ? 0.0 : g.kf * sqrt((double)t), k2 = k * k;
  double y[4];
  {
    const double g0 = pl.ai * pl.ai * dE(pl.ai, g.om);
    y[0] = 1.0;
    y[1] = g0;
    y[2] = -3.0 / 7.0;
    y[3] = -6.0 / 7.0 * g0;
  }
  int turn = 0;   // chunks begun: chunk n is in pt[n % 3] and md[n % 2]
  // wave 0's work on a chunk of m steps (and its slice, if the chunk ends one)
  auto integrate = [&](int n, int m, double h, int slice) {
    const FrPoint* p = pt[n % 3];
    const double2(*v)[64] = md[n % 2];
    auto rhs = [&](double2 c, double f, const double* yy, double* dy) {
      const double ds = yy[0];
      dy[0] = yy[1] * f;
      dy[1] = c.x * yy[0] * f;
      dy[2] = yy[3] * f;
      dy[3] = (c.x * yy[2] - c.x * ds * ds - c.y * ds * ds) * f;
    };
    double2 ca = v[0][lane];
    double fa = p[0].f;
    for (int j = 0; j < m; ++j) {
      const double2 cb = v[2 * j + 1][lane], cc = v[2 * j + 2][lane];
      const double fb = p[2 * j + 1].f, fc = p[2 * j + 2].f;
      double k1[4], k2[4], k3[4], k4[4], yt[4];
      rhs(ca, fa, y, k1);
      for (int e = 0; e < 4; ++e) yt[e] = y[e] + 0.5 * h * k1[e];
      rhs(cb, fb, yt, k2);
      for (int e = 0; e < 4; ++e) yt[e] = y[e] + 0.5 * h * k2[e];
      rhs(cb, fb, yt, k3);
      for (int e = 0; e < 4; ++e) yt[e] = y[e] + h * k3[e];
      rhs(cc, fc, yt, k4);
      for (int e = 0; e < 4; ++e) y[e] += h / 6.0 * (k1[e] + 2.0 * k2[e] + 2.0 * k3[e] + k4[e]);
      ca = cc;
      fa = fc;
    }
    if (slice >= 0 && (ref ? lane == 0 : t < g.n_k)) {
      const double2 c = v[2 * m + 1][lane];
      const double ds = y[0];
      double* out = ref ? ref_out : table + ((int64_t)slice * g.n_k + t) * 6;
      out[0] = y[0];
      out[1] = y[1];
      out[2] = c.x * y[0];
      out[3] = y[2];
      out[4] = y[3];
      out[5] = c.x * y[2] - c.x * ds * ds - c.y * ds * ds;
    }
  };
  // points a chunk's first needs: start, then middle and end of its steps (and the slice's a)
  auto stage = [&](int n, const FrPoint* src, int np) {   // all threads but wave 0's
    const double2* s2 = reinterpret_cast<const double2*>(src);
    double2* d2 = reinterpret_cast<double2*>(pt[n % 3]);
    for (int e = threadIdx.x - 64; e < np * kFrWords; e += 192) d2[e] = s2[e];
  };
  // the chunk being formed and the one before it
  int m_prev = 0, slice_prev = -1;
  double h_prev = 0.0;
  bool have_prev = false;
  for (int i = 0; i < pl.slices(); ++i) {
    const FrPoint* base = pts + (ref ? fr_ref_base(pl) : pl.off(i));
    const double lna0 = pl.from(i), le = log(pl.a(i));
    const int nsub = pl.nsub(lna0, le);
    const double h = (le - lna0) / nsub;
    for (int s = 0; s == 0 || s < nsub; s += kFrChunk) {
      const int m = nsub - s < kFrChunk ? nsub - s : kFrChunk;
      const bool last = s + m == nsub;
      const int np = 2 * m + 1 + (last ? 1 : 0);
      if (wave > 0) stage(turn, base + 2 * s, np);   // pt[turn % 3] was last read two chunks ago
      __syncthreads();   // this chunk's points are staged; the chunk before is formed
      if (wave > 0) {
        for (int q = wave - 1; q < np; q += 3) {
          const FrPoint p = pt[turn % 3][q];
          double mu = 1.0, g2t = 0.0;
          if (!ref) {
            mu = 1.0 + k2 / (3.0 * (k2 + p.a2m2));
            const double kk = div_by(k2, p.ahah, p.r_hh);
            const double Pk = kk + p.c0;
            const double Ph = 0.5 * kk + p.c0;   // halving is exact
            const double kah = div_by(k, p.ahE, p.r_hE);
            const double g2 = p.C0 * kah * kah * p.X5Y4 / (Pk * Ph * Ph);
            g2t = p.G0 * g2;
          }
          md[turn % 2][q][lane] = make_double2(p.kap * mu, g2t);
        }
      } else if (have_prev) {
        integrate(turn - 1, m_prev, h_prev, slice_prev);
      }
      have_prev = true;
      m_prev = m;
      h_prev = h;
      slice_prev = last ? i : -1;
      ++turn;
    }
  }
  __syncthreads();   // the last chunk is formed
  if (wave == 0) integrate(turn - 1, m_prev, h_prev, slice_prev);
}

static SpecDev spec_dev(const cola_params& p) {
  SpecDev e;
  const double omh2 = p.omega_m * p.h * p.h, obh2 = p.omega_b * p.h * p.h;
  const double fb = p.omega_b / p.omega_m;
  const double sh = 44.5 * std::log(9.83 / omh2) / std::sqrt(1.0 + 10.0 * std::pow(obh2, 0.75));
  const double th = p.t_cmb / 2.7;
  e.ns = p.n_s;
  e.th2 = th * th;
  e.omh = p.omega_m * p.h;
  e.alpha = 1.0 - 0.328 * std::log(431.0 * omh2) * fb + 0.38 * std::log(22.3 * omh2) * fb * fb;
  e.kfac = 0.43 * sh * p.h;
  e.s8 = p.sigma8;
  return e;
}

// Range of ln a a run integrates over (at most that of a double, whose largest has ln 710).
static double growth_span(const cola_params& p) { return std::min(std::log1p(p.z_init), 710.0); }

static double growth_floor(const cola_params& p) {
  return std::max(kGrowthFloor, growth_span(p) / kGrowthFine);
}

// Longest step from l0 to l1 (no knot of a tabulated model between them).  The steps converge
// like a power series in the step over the distance to the nearest pole of the
// coefficients in the complex plane: at pi / s for a logistic term of log-slope s, such as
// k^2/(k^2 + m) with s = |d ln m / d ln a| at whatever k.  So a step takes 0.3 / s at
// most, and 0.2 / lambda, lambda^2 = 3/2 mu being the largest rate of the growth equation.  A
// spline piece is also cut in six: beta may rise from 0 to 1 within one.  Measured against
// steps of 1e-3 (z = 19): k-Mouflage with s = 42 and 84, 1e-8 and 2e-6 with steps of
// 0.04, 3e-13 now (Runge-Kutta steps of 1e-3: 2e-11 and 3e-11); tables of m^2 ~ a^-40 and a^-80,
// 6e-8 and 3e-5, now 3e-13 (3e-11 and 7e-10); beta from 0 to 1 over 0.05, 6e-10, now 3e-13 (4e-11).
// f(R) (s <= 7) and nDGP (s <= 3, mu <= 4/3) stay at kGrowthStep, and so does the symmetron
// for beta_* <= 2.8, whose slope the graded steps after a_* follow.
static double growth_step_bound(const cola_params& p, int model, const MBSpline& mb, double l0, double l1) {
  double slope = 0.0, mu = 1.0, piece = 1.0;   // piece: length of the spline piece
  if (model == COLA_KMOUFLAGE) {   // P_X - 1 ~ a^{n (m - 1)}
    slope = std::fabs(p.km_xn) * (p.km_m - 1);
    mu += 2.0 * p.km_beta * p.km_beta;
  } else if (model == COLA_SYMMETRON) {
    mu += 2.0 * p.sym_beta * p.sym_beta;
  } else if (model == COLA_MBETA) {   // m = a^2 m^2
    int j = 0;
    while (j + 2 < mb.n && mb.x[j + 1] <= l0) ++j;
    const double x0 = mb.x[j], x1 = mb.x[j + 1], h = x1 - x0, M0 = mb.Mm[j], M1 = mb.Mm[j + 1];
    auto at = [&](double x) {
      const double u = x1 - x, t = x - x0;
      slope = std::max(slope, std::fabs(2.0 + (mb.ym[j + 1] - mb.ym[j]) / h - M0 * u * u / (2.0 * h) +
                                        M1 * t * t / (2.0 * h) - h * (M1 - M0) / 6.0));
    };
    at(l0);
    at(l1);
    const double xe = x0 + h * M0 / (M0 - M1);   // where the slope is extreme
    if (xe > l0 && xe < l1) at(xe);
    const double b = std::max(std::fabs(mb.yb[j]), std::fabs(mb.yb[j + 1])) +
                     h * h / 8.0 * std::max(std::fabs(mb.Mb[j]), std::fabs(mb.Mb[j + 1]));
    mu += 2.0 * b * b;
    piece = h;
  }
  double bound = kGrowthStep;
  if (0.3 < bound * slope) bound = 0.3 / slope;
  if (0.2 < bound * std::sqrt(1.5 * mu)) bound = 0.2 / std::sqrt(1.5 * mu);
  if (piece < 6.0 * bound) bound = piece / 6.0;
  return std::max(bound, growth_floor(p));
}

// The steps of a run.  Boundaries in ln a: every a_i, the knots of a tabulated {m, beta}
// model (the splines' third derivatives jump there) and the symmetron's a_*.  Just after
// a_* the symmetron's gamma_2 term has a peak whose width in ln a scales as
// (k / (a_* m_*))^2, far below kGrowthStep for the fundamental mode of a large box, so the
// steps there start at kGradeFirst and grow by kGrade per step.
struct GrowthList {
  std::vector<double> l;      // boundaries: step j runs from l[j] to l[j + 1]
  std::vector<int16_t> out;   // the slice written after step j, or -1
};
static GrowthList growth_list(const cola_params& p, int model, const MBSpline& mb) {
  GrowthList g;
  double lna = std::log(1.0 / (1.0 + p.z_init));
  g.l.push_back(lna);
  auto step = [&](double l1, int out) {
    g.l.push_back(l1);
    g.out.push_back((int16_t)out);
  };
  // [l0, l1] in equal steps; the last one writes slice `out`
  auto uniform = [&](double l0, double l1, int out) {
    const double most = growth_step_bound(p, model, mb, l0, l1);
    const int n = (int)std::max(1.0, std::ceil(std::min(l1 - l0, 710.0) / most));   // a_ini may be 0
    const double h = (l1 - l0) / n;
    for (int j = 0; j < n; ++j) step(j + 1 == n ? l1 : l0 + (j + 1) * h, j + 1 == n ? out : -1);
  };
  const bool graded = model == COLA_SYMMETRON;
  const double kink = graded ? std::log(p.sym_astar) : 0.0;
  for (int i = 1; i <= p.n_steps; ++i) {
    const double l1 = std::log(a_of_step(p, i));
    if (model == COLA_MBETA)
      for (int j = 0; j < mb.n; ++j)
        if (mb.x[j] > lna && mb.x[j] < l1) {
          uniform(lna, mb.x[j], -1);
          lna = mb.x[j];
        }
    if (graded && lna < kink && kink < l1) {
      uniform(lna, kink, -1);
      lna = kink;
    }
    if (graded && lna >= kink) {
      const double most = growth_step_bound(p, model, mb, lna, l1);
      for (;;) {
        const double h = kGradeFirst + kGrade * (lna - kink);
        if (h >= most || h >= l1 - lna) break;
        step(lna + h, -1);
        lna += h;
      }
    }
    uniform(lna, l1, i);
    lna = l1;
  }
  return g;
}

// The points of f(R) modes, or of the longest list growth_list() can make: every piece between
// boundaries takes its length over the step bound, rounded up.
size_t growth_scratch_bytes(const cola_params& p) {
  if (fr_pipeline(p)) return (size_t)fr_points(p) * sizeof(FrPoint);
  const bool steep = p.growth_mode == 0 && (p.model == COLA_KMOUFLAGE || p.model == COLA_SYMMETRON ||
                                            p.model == COLA_MBETA);
  const double graded = std::log(kGrowthStep / kGradeFirst) / std::log1p(kGrade);
  const double steps = growth_span(p) / (steep ? growth_floor(p) : kGrowthStep) + p.n_steps +
                       COLA_MBETA_MAX_KNOTS + graded + 8;
  return (size_t)steps * kGrowthNodes * sizeof(GrowthNode);
}

void launch_growth_ode(const cola_params& p, const Layout& L, double* table, double* ref, void* scratch,
                       hipStream_t s) {
  ProfScope ps("growth_ode", s);
  GrowthDev g;
  g.om = p.omega_m;
  g.fr0 = p.fr0_abs;
  g.rc = p.rc_h0;
  g.a_ini = 1.0 / (1.0 + p.z_init);
  g.kf = 2.0 * M_PI / p.box;
  g.model = (p.growth_mode == 1) ? COLA_LCDM : p.model;
  g.sb = p.sym_beta;
  g.sm = p.sym_mass;
  g.sa = p.sym_astar;
  g.kb = p.km_beta;
  g.kk0 = p.km_k0;
  g.kx0 = p.km_x0;
  g.kxn = p.km_xn;
  g.km = p.km_m;
  g.kdep = L.kdep ? 1 : 0;
  g.n_steps = p.n_steps;
  g.n_k = L.n_k;
  const SpecDev sp = spec_dev(p);
  if (fr_pipeline(p)) {
    FrPoint* pts = static_cast<FrPoint*>(scratch);
    hipLaunchKernelGGL(k_growth_fr_points, dim3(p.n_steps + 2, 16), dim3(256), 0, s, g, pts);   // + reference
    const dim3 grid((unsigned)((L.n_k + 63) / 64) + 2), block(256);   // + reference, spectrum
    hipLaunchKernelGGL(k_growth_fr, grid, block, 0, s, g, sp, pts, table, ref);
    COLA_LAUNCH_CHECK();
    return;
  }
  const MBSpline mb = mb_spline(p);
  GrowthNode* nodes = static_cast<GrowthNode*>(scratch);
  const GrowthList list = growth_list(p, g.model, mb);
  const int nsteps = (int)list.out.size();
  if ((size_t)nsteps * kGrowthNodes * sizeof(GrowthNode) > L.scratch_bytes)
    throw Error{COLA_E_SIZE, "growth table steps exceed their scratch area"};
  for (int first = 0; first < nsteps; first += kGrowthChunk) {
    GrowthSteps st;
    st.n = std::min(kGrowthChunk, nsteps - first);
    st.first = first;
    std::copy_n(list.l.begin() + first, st.n + 1, st.l);
    std::copy_n(list.out.begin() + first, st.n, st.out);
    const int e = st.n * kGrowthNodes;
    hipLaunchKernelGGL(k_growth_nodes, dim3((e + 63) / 64), dim3(64), 0, s, g, mb, st, nodes);
    COLA_LAUNCH_CHECK();
  }
  const dim3 grid((unsigned)((L.n_k + 1 + 63) / 64) + 1), block(64);
  const bool half = (p.readings & COLA_READ_D2_HALF_K) != 0;
  auto* kernel = half ? (g.kdep ? k_growth_ode<true, true> : k_growth_ode<true, false>)
                      : (g.kdep ? k_growth_ode<false, true> : k_growth_ode<false, false>);
  hipLaunchKernelGGL(kernel, grid, block, 0, s, g, sp, nodes, nsteps, table, ref);
  COLA_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ per-step LPT coefficients
__global__ void k_lpt_coef(const double* __restrict__ table, int64_t slice0, int64_t slice1,
                           const StepDev* __restrict__ steps, const int* __restrict__ ctr,
                           int64_t n_k, float2* __restrict__ coef) {
  if (steps) {
    const StepDev& sd = step_entry(steps, ctr);
    slice0 = sd.slice0;
    slice1 = sd.slice1;
  }
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n_k;
       k += (int64_t)gridDim.x * blockDim.x) {
    const double* t0 = table + slice0 + 6 * k;
    const double* t1 = table + slice1 + 6 * k;
    coef[k] = make_float2((float)t0[2], (float)t0[5]);
    coef[n_k + k] = make_float2((float)(t1[0] - t0[0]), (float)(t1[3] - t0[3]));
  }
}

void launch_lpt_coef(const Layout& L, const double* table, int64_t slice0, int64_t slice1,
                     const StepDev* steps, const int* ctr, float2* coef, hipStream_t s) {
  ProfScope ps("lpt_coef", s);
  const unsigned g = (unsigned)std::min<int64_t>((L.n_k + 255) / 256, 4096);
  hipLaunchKernelGGL(k_lpt_coef, dim3(g), dim3(256), 0, s, table, slice0, slice1, steps, ctr,
                     L.n_k, coef);
  COLA_LAUNCH_CHECK();
}

__global__ void k_lpt_coef_ini(const double* __restrict__ table, int64_t n_k, float2* __restrict__ coef) {
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n_k;
       k += (int64_t)gridDim.x * blockDim.x)
    coef[k] = make_float2((float)table[6 * k], (float)table[6 * k + 3]);
}

void launch_lpt_coef_ini(const Layout& L, const double* table, float2* coef, hipStream_t s) {
  ProfScope ps("lpt_coef", s);
  const unsigned g = (unsigned)std::min<int64_t>((L.n_k + 255) / 256, 4096);
  hipLaunchKernelGGL(k_lpt_coef_ini, dim3(g), dim3(256), 0, s, table, L.n_k, coef);
  COLA_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ triangle growth
// Exact second-order growth of a Fourier triangle k = k1 + k2 (Sec. 4.2) beside the
// approximation the path uses, D2_hat(k)(1 - cos^2 theta), for checking it (Fig. 1):
//   D2'' = kappa mu(k) D2 - kappa mu(k) D1(k1) D1(k2)
//          [1 - (2 mu(k1) - mu(k))/mu(k) cos^2 theta + 2 a^4 H^2 gamma_2/(kappa mu(k))],
//   gamma_2 = gamma_2^E(k, k1, k2) + (3/2) Omega_m(a) [mu(k) - mu(k1)] k1.k2/k2^2  (Sec. 4),
// with D2 = -(3/7)(1 - cos^2 theta), D2' = -(6/7)(1 - cos^2 theta) a^2 E at a_ini; the
// terms that single out k1 are taken as printed.  Same integrator as k_growth_ode.

// y = (D1(k1), D1'(k1), D1(k2), D1'(k2), D1(k), D1'(k), D2, D2', D2_hat, D2_hat')
struct Triangle {
  double k, k1, k2, c, c2;
};

__device__ __forceinline__ void triangle_rhs(const GrowthDev& g, const MBSpline& mb, const Triangle& t,
                                             double lna, const double* y, double* dy) {
  const double a = exp(lna);
  const double E = dE(a, g.om);
  const double kap = 1.5 * g.om * a;
  const double f = 1.0 / (a * a * E);
  const double mu = growth_mu(g, mb, t.k, a), mu1 = growth_mu(g, mb, t.k1, a), mu2 = growth_mu(g, mb, t.k2, a);
  const double oma = g.om / (a * a * a) / (E * E);
  const double g2t = gamma2E_term(g, mb, t.k, t.k1, t.k2, t.c2, a)
                     + 2.0 * a * a * a * a * E * E * 1.5 * oma * (mu - mu1) * (t.k1 / t.k2) * t.c;
  const double src = 1.0 - (2.0 * mu1 - mu) / mu * t.c2 + g2t / (kap * mu);
  double muh, g2h;
  growth_model(g, mb, t.k, a, muh, g2h);   // the approximate equation at k
  dy[0] = y[1] * f;
  dy[1] = kap * mu1 * y[0] * f;
  dy[2] = y[3] * f;
  dy[3] = kap * mu2 * y[2] * f;
  dy[4] = y[5] * f;
  dy[5] = kap * mu * y[4] * f;
  dy[6] = y[7] * f;
  dy[7] = (kap * mu * y[6] - kap * mu * y[0] * y[2] * src) * f;
  dy[8] = y[9] * f;
  dy[9] = (kap * muh * y[8] - kap * muh * y[4] * y[4] - g2h * y[4] * y[4]) * f;
}

__global__ void __launch_bounds__(64) k_growth_triangle(GrowthDev g, MBSpline mb, int n, const double* __restrict__ tri, double a_end,
                                  double* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  Triangle t;
  t.k = tri[3 * i];
  t.k1 = tri[3 * i + 1];
  t.k2 = tri[3 * i + 2];
  const double tol = 1e-12 * (t.k1 + t.k2);
  if (!(t.k1 > 0.0 && t.k2 > 0.0 && t.k >= fabs(t.k1 - t.k2) - tol && t.k <= t.k1 + t.k2 + tol)) {
    out[2 * i] = out[2 * i + 1] = __builtin_nan("");
    return;
  }
  t.c = fmin(1.0, fmax(-1.0, (t.k * t.k - t.k1 * t.k1 - t.k2 * t.k2) / (2.0 * t.k1 * t.k2)));
  t.c2 = t.c * t.c;
  const double ai = g.a_ini;
  const double g0 = ai * ai * dE(ai, g.om);
  const double s2 = 1.0 - t.c2;
  double y[10] = {1.0, g0, 1.0, g0, 1.0, g0, -3.0 / 7.0 * s2, -6.0 / 7.0 * s2 * g0, -3.0 / 7.0,
                  -6.0 / 7.0 * g0};
  double lna = log(ai);
  rk4_to_knots<10>(y, lna, log(a_end), growth_kink(g), g, mb,
                   [&](double l, const double* yy, double* dy) { triangle_rhs(g, mb, t, l, yy, dy); });
  out[2 * i] = y[6];
  out[2 * i + 1] = y[8] * s2;
}

void launch_growth_triangles(const cola_params& p, int n, const double* tri, double a, double* out,
                             hipStream_t s) {
  ProfScope ps("growth_triangles", s);
  GrowthDev g{};
  g.om = p.omega_m;
  g.fr0 = p.fr0_abs;
  g.rc = p.rc_h0;
  g.a_ini = 1.0 / (1.0 + p.z_init);
  g.model = (p.growth_mode == 1) ? COLA_LCDM : p.model;
  g.sb = p.sym_beta;
  g.sm = p.sym_mass;
  g.sa = p.sym_astar;
  g.kb = p.km_beta;
  g.kk0 = p.km_k0;
  g.kx0 = p.km_x0;
  g.kxn = p.km_xn;
  g.km = p.km_m;
  const MBSpline mb = mb_spline(p);
  hipLaunchKernelGGL(k_growth_triangle, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, g, mb, n, tri,
                     a, out);
  COLA_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ white noise
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t k) {
  uint64_t z = seed + (k + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ float unit_open(uint64_t z) {   // ((z >> 11) + 1/2) 2^-53 in (0,1)
  return ((float)(z >> 11) + 0.5f) * 0x1p-53f;
}

// ------------------------------------------------------------------ initial amplitudes
struct EHDev {
  float ns, th2, omh, alpha, kfac;   // see SpecDev
};

__device__ __forceinline__ float eh_T(const EHDev& e, float k) {
  const float kk = e.kfac * k;
  const float k4 = (kk * kk) * (kk * kk);
  const float gam = e.omh * (e.alpha + (1.f - e.alpha) / (1.f + k4));
  const float q = k * e.th2 / gam;
  const float L0 = logf(2.f * 2.718281828459045f + 1.8f * q);
  const float C0 = 14.2f + 731.f / (1.f + 62.5f * q);
  return L0 / (L0 + C0 * q * q);
}

// What turns the white noise into phi1: phi1_k = amp[|nu|^2] W_k, amp = sqrt(N P_ini(k) / L^3) / k^2
// and 0 at k = 0.  One entry per |nu|^2, about 1.5 / n of the modes.
struct AmpTable {
  float* amp;
  int n;
  float kf, norm;
  EHDev eh;
  const double* ref;
};

// White noise, four cells of a row a thread; the blocks past the last x-plane fill the table of
// amplitudes, which saves a launch.  Bound by the hashes and the logarithm: 384^3 167 us, before
// (one cell and two 64-bit divisions a thread) 253.
__global__ void __launch_bounds__(256)
k_noise(uint64_t seed, int n, int rpitch, int64_t rplane, float* __restrict__ padded,
        float* __restrict__ flat, AmpTable t) {
  if (blockIdx.y == (unsigned)n) {
    const float d1 = (float)t.ref[0], A = (float)t.ref[6];   // sigma8 normalisation of k^ns T^2
    const float inv_d1sq = 1.f / (d1 * d1);
    for (int n2 = blockIdx.x * blockDim.x + threadIdx.x; n2 < t.n; n2 += gridDim.x * blockDim.x) {
      const float k2 = t.kf * t.kf * (float)n2;
      const float k = sqrtf(k2);
      const float T = eh_T(t.eh, k);
      const float P = A * powf(k, t.eh.ns) * T * T * inv_d1sq;
      t.amp[n2] = n2 > 0 ? sqrtf(t.norm * P) / k2 : 0.f;
    }
    return;
  }
  CellQuad c;
  if (!cell_quad(n, rpitch, rplane, c)) return;
  quad_t g;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint64_t j = (uint64_t)(c.e + i);
    const float u0 = unit_open(splitmix64(seed, 2 * j));
    const float u1 = unit_open(splitmix64(seed, 2 * j + 1));
    g[i] = sqrtf(-2.f * logf(u0)) * cospif(2.f * u1);
  }
  if (padded) *reinterpret_cast<quad_t*>(padded + c.pe) = g;
  if (flat) *reinterpret_cast<quad_t*>(flat + c.e) = g;
}

void launch_noise(const cola_params& p, int n, int pitch, int64_t plane, float* padded, float* flat,
                  hipStream_t s, float* amp, const double* ref) {
  ProfScope ps("noise", s);
  dim3 grid = quad_grid(n);
  AmpTable t{};
  if (amp) {
    const SpecDev d = spec_dev(p);
    const double N = (double)n * n * n;
    t.amp = amp;
    t.n = 3 * (n / 2) * (n / 2) + 1;
    t.kf = (float)(2.0 * M_PI / p.box);
    t.norm = (float)(N / (p.box * p.box * p.box));
    t.eh = EHDev{(float)d.ns, (float)d.th2, (float)d.omh, (float)d.alpha, (float)d.kfac};
    t.ref = ref;
    grid.y += 1;
  }
  hipLaunchKernelGGL(k_noise, grid, dim3(256), 0, s, p.seed, n, 2 * pitch, 2 * plane, padded, flat, t);
  COLA_LAUNCH_CHECK();
}

}  // namespace cola
