// Device code of the EIFE library: sine-transform axis passes, the fused
// reaction and diagonal phi stages, and the norm reductions (gfx950).
//
// A type-I sine transform of length n = N - 1 (Section 4: the matrices
// P_ij = sin(ij pi / N) diagonalise the 1D mass and stiffness matrices) is
// computed for two real lines at once: c = a + i b is extended oddly to
// length L = 2N (z_m = c_m, z_{2N-m} = -c_m, z_0 = z_N = 0), a complex FFT of
// length L gives Z_k = -2i (P a + i P b)_k, so the orthonormal transform
// S = sqrt(2/N) P is (S a)_k = -Im Z_k / sqrt(2N), (S b)_k = Re Z_k / sqrt(2N).
// This file holds what the passes share: butterflies, the diagonal stages, the
// reactions and the argument blocks; the passes themselves are in eife_fast.hpp,
// eife_fold.hpp, eife_long.hpp and, for any length, eife_mix.hpp.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace eife {

template <typename T>
struct Cx {
  T re, im;
};

template <typename T>
__device__ __forceinline__ Cx<T> cadd(Cx<T> a, Cx<T> b) { return {a.re + b.re, a.im + b.im}; }
template <typename T>
__device__ __forceinline__ Cx<T> csub(Cx<T> a, Cx<T> b) { return {a.re - b.re, a.im - b.im}; }
template <typename T>
__device__ __forceinline__ Cx<T> cmul(Cx<T> a, Cx<T> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
// multiply by -i
template <typename T>
__device__ __forceinline__ Cx<T> cmnegi(Cx<T> a) { return {a.im, -a.re}; }

template <typename T, int R>
struct Dft;

template <typename T>
struct Dft<T, 2> {
  static __device__ __forceinline__ void run(Cx<T>* v) {
    Cx<T> a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  }
};

template <typename T>
struct Dft<T, 3> {
  static __device__ __forceinline__ void run(Cx<T>* v) {
    const T c = T(0.86602540378443864676);  // sqrt(3)/2
    Cx<T> s = cadd(v[1], v[2]);
    Cx<T> d = csub(v[1], v[2]);
    Cx<T> m = {v[0].re - T(0.5) * s.re, v[0].im - T(0.5) * s.im};
    Cx<T> r = {c * d.im, -c * d.re};  // -i * c * d
    v[0] = cadd(v[0], s);
    v[1] = cadd(m, r);
    v[2] = csub(m, r);
  }
};

template <typename T>
struct Dft<T, 4> {
  static __device__ __forceinline__ void run(Cx<T>* v) {
    Cx<T> t0 = cadd(v[0], v[2]);
    Cx<T> t1 = csub(v[0], v[2]);
    Cx<T> t2 = cadd(v[1], v[3]);
    Cx<T> t3 = cmnegi(csub(v[1], v[3]));
    v[0] = cadd(t0, t2);
    v[2] = csub(t0, t2);
    v[1] = cadd(t1, t3);
    v[3] = csub(t1, t3);
  }
};

// Odd prime P: with a_r = v_r + v_{P-r}, b_r = v_r - v_{P-r} (r = 1 .. (P-1)/2)
// and theta = 2 pi r k / P,
//   X_k     = v_0 + sum_r a_r cos(theta) - i sum_r b_r sin(theta),
//   X_{P-k} = v_0 + sum_r a_r cos(theta) + i sum_r b_r sin(theta);
// cs[m-1], sn[m-1] hold cos and sin of 2 pi m / P for m = 1 .. (P-1)/2.
template <typename T, int P>
__device__ __forceinline__ void dft_odd_prime(Cx<T>* v, const T (&cs)[(P - 1) / 2], const T (&sn)[(P - 1) / 2]) {
  constexpr int Hh = (P - 1) / 2;
  Cx<T> a[Hh], b[Hh];
  Cx<T> sum = v[0];
#pragma unroll
  for (int r = 1; r <= Hh; ++r) {
    a[r - 1] = cadd(v[r], v[P - r]);
    b[r - 1] = csub(v[r], v[P - r]);
    sum = cadd(sum, a[r - 1]);
  }
  Cx<T> out[P];
  out[0] = sum;
#pragma unroll
  for (int k = 1; k <= Hh; ++k) {
    Cx<T> re = v[0], im = {T(0), T(0)};
#pragma unroll
    for (int r = 1; r <= Hh; ++r) {
      const int m = (r * k) % P;
      const int i = m <= Hh ? m : P - m;
      const T c = cs[i - 1];
      const T sg = m <= Hh ? sn[i - 1] : -sn[i - 1];
      re = Cx<T>{re.re + c * a[r - 1].re, re.im + c * a[r - 1].im};
      im = Cx<T>{im.re + sg * b[r - 1].re, im.im + sg * b[r - 1].im};
    }
    out[k] = Cx<T>{re.re + im.im, re.im - im.re};      // re - i im
    out[P - k] = Cx<T>{re.re - im.im, re.im + im.re};  // re + i im
  }
#pragma unroll
  for (int q = 0; q < P; ++q) v[q] = out[q];
}

template <typename T>
struct Dft<T, 5> {
  static __device__ __forceinline__ void run(Cx<T>* v) {
    const T cs[2] = {T(0.30901699437494742410), T(-0.80901699437494742410)};
    const T sn[2] = {T(0.95105651629515357212), T(0.58778525229247312917)};
    dft_odd_prime<T, 5>(v, cs, sn);
  }
};

template <typename T>
struct Dft<T, 7> {
  static __device__ __forceinline__ void run(Cx<T>* v) {
    const T cs[3] = {T(0.62348980185873353053), T(-0.22252093395631440429), T(-0.90096886790241912624)};
    const T sn[3] = {T(0.78183148246802980871), T(0.97492791218182360702), T(0.43388373911755812048)};
    dft_odd_prime<T, 7>(v, cs, sn);
  }
};

// Multiplies input q of a butterfly by w^q, q = 1 .. R - 1, w = tw[i] = exp(-2 pi i i / L)
// with (R - 1) i < L.  The powers 1, 2, 4 and 8 are loaded, the others at most three
// products of them: a chain of products from w alone multiplies the rounding error of
// its table value by q (FP32 240 x 150 x 100: error of four steps against 64 bits 4.4e-7
// with the chain, 2.8e-7 so, 2.7e-7 with every power loaded, 258 to 260 us a step; in the
// longest lines loads cost, 4000 intervals 88, 92 and 101 us a step).
template <typename T, int R>
__device__ __forceinline__ void twiddle_powers(Cx<T>* v, const Cx<T>* __restrict__ tw, int i) {
  Cx<T> p[R];
#pragma unroll
  for (int q = 1; q < R; ++q) {
    const int b = q >= 8 ? 8 : q >= 4 ? 4 : q >= 2 ? 2 : 1;
    p[q] = q == b ? tw[q * i] : cmul(p[b], p[q - b]);
  }
#pragma unroll
  for (int q = 1; q < R; ++q) v[q] = cmul(v[q], p[q]);
}

// ---------------------------------------------------------------------------
// Diagonal phi stage (Section 2.2, eqs. (2.13)-(2.14); Section 4, eq. (4.4)).
// For a spectral index with eigenvalue Lam = D (lam_x + lam_y + lam_z) and
// z = -tau Lam, the stage needs e^z, tau phi_1(z), tau phi_2(z) and
// c2 tau phi_1(c2 z).  They are built from per-axis double tables
//   M_a = e^{z_a} - 1,  Q_a = e^{z_a} - 1 - z_a,  Mc_a = e^{c2 z_a} - 1
// (z_a = -tau D lam_a) with the exact identities
//   e^{a+b} - 1       = M_a + M_b + M_a M_b
//   e^{a+b} - 1 - a - b = Q_a + Q_b + M_a M_b,
// in which, for z <= 0, every Q term and every product M_a M_b is >= 0, so
// no cancellation occurs anywhere in the spectrum.  Then
//   tau phi_1 = -M / Lam,  tau phi_2 = Q / (tau Lam^2),  c2 tau phi_1(c2 z) = -Mc / Lam.
struct AxisTab {
  const double* lam;  // lambda_k = lamB_k / lamA_k of the 1D pair (B, A) (padding: 1)
  const double* w;    // load weight h / lamA_k (lumped) or 1 (nodal); 0 on padding
  const double* M;    // expm1(-tau D lambda_k)
  const double* Q;    // expm1(-tau D lambda_k) + tau D lambda_k
  const double* Mc;   // expm1(-c2 tau D lambda_k)
  // three-stage scheme only (zero otherwise)
  const double* R;    // expm1(z) - z - z^2/2, z = -tau D lambda_k
  const double* Mc3;  // expm1(c3 z)
  const double* Qc3;  // expm1(c3 z) - c3 z
};

struct Sep {
  double lam, w, M, Q, Mc;
};

__device__ __forceinline__ Sep sep_load(const AxisTab& t, int k) {
  return Sep{t.lam[k], t.w[k], t.M[k], t.Q[k], t.Mc[k]};
}

__device__ __forceinline__ Sep sep_combine(const Sep& a, const Sep& b) {
  const double mm = a.M * b.M;
  return Sep{a.lam + b.lam, a.w * b.w, a.M + b.M + mm, a.Q + b.Q + mm, a.Mc + b.Mc + a.Mc * b.Mc};
}

enum DiagMode { DIAG_A = 1, DIAG_B = 2, DIAG_ETD1 = 3 };

// g: transformed (unweighted) reaction; h: spectral state (DIAG_A, DIAG_ETD1: u^;
// DIAG_B: E u^ + tau (phi_1 - phi_2/c2) G^_1).  Returns the value to inverse
// transform in *out and the new state in *nh.
template <int MODE>
__device__ __forceinline__ void diag_apply(const Sep& s, double D, double tau, double c2, double g, double h,
                                           double* out, double* nh) {
  const double G = g * s.w;
  if (s.lam == 0.0) {
    // the zero mode of a periodic grid (Lam = 0): e^0 = 1, phi_1(0) = 1, phi_2(0) = 1/2
    if (MODE == DIAG_ETD1) {
      *out = *nh = h + tau * G;
    } else if (MODE == DIAG_A) {
      *out = h + c2 * tau * G;
      *nh = h + tau * (1.0 - 0.5 / c2) * G;
    } else {
      *out = *nh = h + 0.5 * tau / c2 * G;
    }
    return;
  }
  const double rL = 1.0 / (D * s.lam);
  if (MODE == DIAG_ETD1) {
    const double un = h + s.M * h - s.M * rL * G;
    *out = un;
    *nh = un;
  } else if (MODE == DIAG_A) {
    *out = h + s.Mc * h - s.Mc * rL * G;
    const double a2 = s.Q * rL * rL / (tau * c2);
    *nh = h + s.M * h - (s.M * rL + a2) * G;
  } else {
    const double a2 = s.Q * rL * rL / (tau * c2);
    const double un = h + a2 * G;
    *out = un;
    *nh = un;
  }
}

struct Diag {
  AxisTab ax[3];
  double D, tau, c2;
  double c3;  // third node of the three-stage scheme
  void* X;    // its extra spectral state e^{c3 z} u^ + tau a31 G_1 (layout of H)
};

// The separable tables of the three-stage scheme (eq. (2.2), s = 3): besides
// e^z - 1 and e^z - 1 - z it needs R = e^z - 1 - z - z^2/2 (phi_3 = R / z^3) and
// the c3-scaled pair.  With e^a = 1 + a + Q_a, the product e^a e^b gives
//   R_{a+b} = R_a + R_b + a Q_b + b Q_a + Q_a Q_b.
struct Sep3 {
  double lam, w, M, Q, Mc, R, Mc3, Qc3;
};

__device__ __forceinline__ Sep3 sep3_load(const AxisTab& t, int k) {
  return Sep3{t.lam[k], t.w[k], t.M[k], t.Q[k], t.Mc[k], t.R[k], t.Mc3[k], t.Qc3[k]};
}

// tD = tau D, so that z = -tD lam
__device__ __forceinline__ Sep3 sep3_combine(const Sep3& a, const Sep3& b, double tD) {
  const double za = -tD * a.lam, zb = -tD * b.lam;
  return Sep3{a.lam + b.lam,
              a.w * b.w,
              a.M + b.M + a.M * b.M,
              a.Q + b.Q + a.M * b.M,
              a.Mc + b.Mc + a.Mc * b.Mc,
              a.R + b.R + za * b.Q + zb * a.Q + a.Q * b.Q,
              a.Mc3 + b.Mc3 + a.Mc3 * b.Mc3,
              a.Qc3 + b.Qc3 + a.Mc3 * b.Mc3};
}

// Column modes of the three-stage scheme (nodes 0, c2, c3; weights of eq. (2.2)
// from the Lagrange polynomials: b_i of all three nodes, a_3j of nodes 0, c2):
//   COL_S3_1: out = e^{c2 z} u^ + tau a21 G1,  X = e^{c3 z} u^ + tau a31 G1,
//             H = e^z u^ + tau b1 G1
//   COL_S3_2: out = X + tau a32 G2,  H += tau b2 G2
//   COL_S3_3: out = H + tau b3 G3 (the new u^), H = out
enum { COL_S3_1 = 5, COL_S3_2 = 6, COL_S3_3 = 7 };

// 1 / x in double from the hardware estimate and two Newton steps (x > 0 normal).
__device__ __forceinline__ double rcp64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// Step constants of the three-stage weights, formed once per thread.
struct S3K {
  double tau, c2, c3, D;
  double itau, itau2;        // 1 / tau, 1 / tau^2
  double kb1, kb2, kb3;      // 1 / (c2 c3), 1 / (c2 (c2 - c3)), 1 / (c3 (c3 - c2))
  double ka, ic3sq_tau;      // c3^2 / c2, 1 / (c3^2 tau)
};

__device__ __forceinline__ S3K s3k_make(const Diag& dg) {
  S3K k;
  k.tau = dg.tau;
  k.c2 = dg.c2;
  k.c3 = dg.c3;
  k.D = dg.D;
  k.itau = 1.0 / dg.tau;
  k.itau2 = k.itau * k.itau;
  k.kb1 = 1.0 / (dg.c2 * dg.c3);
  k.kb2 = 1.0 / (dg.c2 * (dg.c2 - dg.c3));
  k.kb3 = 1.0 / (dg.c3 * (dg.c3 - dg.c2));
  k.ka = dg.c3 * dg.c3 / dg.c2;
  k.ic3sq_tau = 1.0 / (dg.c3 * dg.c3 * dg.tau);
  return k;
}

template <int MODE>
__device__ __forceinline__ void diag3_apply(const Sep3& s, const S3K& k, double g, double h, double x, double* out,
                                            double* nh, double* nx) {
  const double G = g * s.w;
  // t_k = tau phi_k(z); a21 = tau a_21, a31 = tau a_31, a32 = tau a_32
  double t1, t2, t3, a21, a31, a32;
  if (s.lam == 0.0) {  // zero mode of a periodic grid: phi_k(0) = 1/k!
    t1 = k.tau;
    t2 = 0.5 * k.tau;
    t3 = k.tau / 6.0;
    a21 = k.c2 * k.tau;
    a32 = k.ka * 0.5 * k.tau;
    a31 = k.c3 * k.tau - a32;
  } else {
    const double rL = rcp64(k.D * s.lam);
    const double rL2 = rL * rL;
    t1 = -s.M * rL;
    t2 = s.Q * rL2 * k.itau;
    t3 = -s.R * rL2 * rL * k.itau2;
    // c2 tau phi_1(c2 z) = -Mc rL;  c3 tau phi_1(c3 z) = -Mc3 rL;  tau phi_2(c3 z) = Qc3 rL^2 / (c3^2 tau)
    a21 = -s.Mc * rL;
    a32 = k.ka * s.Qc3 * rL2 * k.ic3sq_tau;
    a31 = -s.Mc3 * rL - a32;
  }
  if (MODE == COL_S3_1) {
    *out = h + s.Mc * h + a21 * G;
    *nx = h + s.Mc3 * h + a31 * G;
    *nh = h + s.M * h + (2.0 * t3 - (k.c2 + k.c3) * t2 + k.c2 * k.c3 * t1) * k.kb1 * G;
  } else if (MODE == COL_S3_2) {
    *out = x + a32 * G;
    *nh = h + (2.0 * t3 - k.c3 * t2) * k.kb2 * G;
  } else {
    *out = *nh = h + (2.0 * t3 - k.c2 * t2) * k.kb3 * G;
  }
}



// Reaction parameters
struct Forcing {
  int kind;
  int d;
  double t;
  double c0, c1;
  double D;
  double a[3];
  double h[3];
  int n[3];  // interior nodes per axis (unused axes 1)
  // position-dependent forcings: sin(pi x_a) at the interior nodes of each axis
  // (device tables) and their time factor (e^-t for the manufactured problem,
  // e^(-pi^2 t) for Example 5.1), formed once per launch instead of per node
  const double* sinpi_ax[3];
  double et;
  // traveling wave: 1 / eps^2 and the boundary load's tables at the launch's time (ShellTab)
  double ieps2;
  const double* wave;
};

// sin(pi (a + (i + 1) h)) for i < n: the per-axis factors of the manufactured
// solution and of Example 5.1's forcing.
static __global__ void sinpi_table(double* __restrict__ out, int n, double a, double h) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = sinpi(a + (i + 1) * h);
}

enum FKind { FK_ZERO = 0, FK_AC = 1, FK_MMS = 2, FK_EX51 = 3, FK_CONST = 4, FK_AFFINE = 5, FK_FH = 6, FK_EX52 = 7 };

// Example 5.2's traveling wave g = (1 - tanh(xi)) / 2, xi = (x - s t) / (2 sqrt(2) eps),
// s = 3 / (sqrt(2) eps); returns g and stores dg/dt.
__device__ __forceinline__ double ex52_wave(double x, double t, double eps, double* g_t) {
  const double w = 2.0 * 1.4142135623730951 * eps;
  const double s = 3.0 / (1.4142135623730951 * eps);
  const double th = tanh((x - s * t) / w);
  *g_t = 0.5 * s / w * (1.0 - th * th);
  return 0.5 * (1.0 - th);
}

// Nonhomogeneous Dirichlet data as part of f (start of Section 4): with the
// boundary nodes carrying g(t), the Galerkin load of interior node i gains
// b_i = -sum over boundary neighbours j of (M_ij g_j' + D K1_ij g_j), formed here
// over prod(h), the scale of the lumped load f(u_i) prod(h), so that it adds to the
// reaction value.  Per axis the 1D entries over h are 2/3 (same node) and 1/6
// (neighbour) for the mass, 2/h^2 and -1/h^2 for the stiffness; nonzero only on the
// shell of nodes next to the boundary.
//
// The wave depends on x alone, so the sum over the neighbours separates: with A, B
// the 1D x entries and m, s the mass and stiffness sums over the row's (y, z)
// neighbours that lie on the boundary,
//   b_i = -(m P_i + s Q_i),  P = A g' + D B g,  Q = D A g   (at the x nodes i - 1 .. i + 1),
// plus, at the ends of a row, the x boundary node with the sums over the other
// (y, z) neighbours.  P and Q are tabulated per evaluation time (wave_tables), the
// four sums per row (ShellRow); forming the neighbours' waves at every shell
// node took most of the x pass and kept the traveling wave off the specialised row
// kernels, for want of registers (1024 x 64 x 64 FP64: 204 us a pass; with the
// tables 38.5 us, a pass without a load 37, and 4.7 us per 16 evaluation times for
// the tables).
constexpr int kWaveEvals = 16;  // evaluation times tabulated per launch
struct WaveTimes {
  double t[kWaveEvals];
};
// doubles of one evaluation's tables: P[n], Q[n], then the end terms
// (A g' + D B g, D A g) of the left and of the right x boundary node
__host__ __device__ constexpr int wave_stride(int n) { return 2 * n + 4; }

static __global__ void __launch_bounds__(256) wave_tables(double* __restrict__ out, WaveTimes tm, int n, double a,
                                                          double h, double D, double eps) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const double t = tm.t[blockIdx.y];
  double* tab = out + int64_t(blockIdx.y) * wave_stride(n);
  if (i < n) {
    double P = 0.0, Q = 0.0;
    for (int o = -1; o <= 1; ++o) {
      const double al = o ? 1.0 / 6.0 : 2.0 / 3.0, be = (o ? -1.0 : 2.0) / (h * h);
      double g_t;
      const double g = ex52_wave(a + (i + 1 + o) * h, t, eps, &g_t);
      P += al * g_t + D * be * g;
      Q += D * al * g;
    }
    tab[i] = P;
    tab[n + i] = Q;
  } else if (i < n + 2) {
    double g_t;
    const double g = ex52_wave(i == n ? a : a + (n + 1) * h, t, eps, &g_t);
    tab[2 * n + 2 * (i - n)] = g_t / 6.0 - D / (h * h) * g;
    tab[2 * n + 2 * (i - n) + 1] = D / 6.0 * g;
  }
}

// The (y, z) sums of one row: over the neighbours on the boundary (m, s) and over
// the others (mi, si).
struct ShellRow {
  double m, s, mi, si;
};

__device__ __forceinline__ ShellRow shell_row(const Forcing& F, int iy, int iz) {
  ShellRow r{0.0, 0.0, 0.0, 0.0};
  const double hy2 = 1.0 / (F.h[1] * F.h[1]), hz2 = 1.0 / (F.h[2] * F.h[2]);
  for (int oz = F.d > 2 ? -1 : 0; oz <= (F.d > 2 ? 1 : 0); ++oz)
    for (int oy = F.d > 1 ? -1 : 0; oy <= (F.d > 1 ? 1 : 0); ++oy) {
      const bool by = F.d > 1 && (iy + oy < 0 || iy + oy >= F.n[1]), bz = F.d > 2 && (iz + oz < 0 || iz + oz >= F.n[2]);
      const double ay = F.d > 1 ? (oy ? 1.0 / 6.0 : 2.0 / 3.0) : 1.0, az = F.d > 2 ? (oz ? 1.0 / 6.0 : 2.0 / 3.0) : 1.0;
      const double sy = F.d > 1 ? (oy ? -hy2 : 2.0 * hy2) : 0.0, sz = F.d > 2 ? (oz ? -hz2 : 2.0 * hz2) : 0.0;
      const double m = ay * az, s = sy * az + ay * sz;
      if (by || bz) {
        r.m += m;
        r.s += s;
      } else {
        r.mi += m;
        r.si += s;
      }
    }
  return r;
}

// Example 5.2's reaction at x index ix of a row: (u - u^3) / eps^2 plus the boundary load.
template <typename T>
__device__ __forceinline__ T reaction_wave(const Forcing& F, const ShellRow& r, T u, int ix) {
  const double ud = double(u);
  double v = (ud - ud * ud * ud) * F.ieps2;
  const int n = F.n[0];
  if (r.m != 0.0) v -= fma(r.m, F.wave[ix], r.s * F.wave[n + ix]);
  if (ix == 0) v -= fma(r.mi, F.wave[2 * n], r.si * F.wave[2 * n + 1]);
  if (ix == n - 1) v -= fma(r.mi, F.wave[2 * n + 2], r.si * F.wave[2 * n + 3]);
  return T(v);
}

// Per-instance data of a batched launch (instances of one size class share
// geometry and launch shape; blockIdx.y (row passes) or blockIdx.z (column
// passes) selects the instance).  A single grid launches with a null table.
template <typename T>
struct RowInst {
  T* W;          // work array
  T* H;          // spectral state
  int64_t uoff;  // offset of the instance in the caller's batched nodal array
  double D;      // diffusion coefficient (used by the manufactured forcing)
};

template <typename T>
struct ColInst {
  T* W;
  T* H;
  AxisTab ax[3];  // per-instance tables (phi tables depend on D)
  double D;
};

// Every kind but the traveling wave (reaction_wave).
template <typename T>
__device__ __forceinline__ T reaction(const Forcing& F, T u, int ix, int iy, int iz) {
  switch (F.kind) {
    case FK_AC:
      return u - u * u * u;
    case FK_ZERO:
      return T(0);
    case FK_CONST:
      return T(F.c0);
    case FK_AFFINE:
      return T(F.c0 + F.c1 * F.t);
    case FK_FH:  // Example 5.3: (theta/2) ln((1 - u)/(1 + u)) + theta_c u, theta = c0, theta_c = c1
      return T(0.5) * T(F.c0) * log((T(1) - u) / (T(1) + u)) + T(F.c1) * u;
    case FK_MMS: {
      double s = F.sinpi_ax[0][ix];
      if (F.d > 1) s *= F.sinpi_ax[1][iy];
      if (F.d > 2) s *= F.sinpi_ax[2][iz];
      const double e = F.et;  // e^-t
      const double PI2 = 9.8696044010893586188;
      const double g = (F.d * PI2 * F.D - 1.0) * e * s - e * e * s * s;
      const double ud = double(u);
      return T(ud * ud + g);
    }
    case FK_EX51: {
      const double PI2 = 9.8696044010893586188;
      const double s = F.sinpi_ax[0][ix] * F.sinpi_ax[1][iy];
      return T(-0.5 * PI2 * double(u) + 0.5 * PI2 * F.et * s);  // et = e^(-pi^2 t)
    }
    default:
      return T(0);
  }
}

// ---------------------------------------------------------------------------
// Row passes: lines along x (contiguous).
// ROW_FWD_PHYS (specialised kernels only): from the nodal values u, dst2 =
// S_x u and dst = S_x f(u) in one pass (the first reaction of a run).
// ROW_INV_CHG: ROW_INV_USER that also sums (u - u_n)^2 over each line pair
// (u_n in dst2, the user layout) into chg[pair] (specialised rows of one
// wavefront per pair only).
enum RowMode { ROW_PHYS = 0, ROW_FWD_USER = 1, ROW_INV_USER = 2, ROW_FWD_PHYS = 3, ROW_INV_CHG = 4 };

struct RowGeom {
  int n;         // line length (interior nodes along x)
  int nrows;     // number of rows (prod of the other axes)
  int ny;        // rows per z-slab (interior nodes along y)
  int64_t ld_src, ld_dst;  // row pitch of source / destination
  double* chg = nullptr;  // ROW_INV_CHG: per line pair sums of (u - u_n)^2
};

// Pointers of a row pass for one instance (batched launches) or the launch's own.
template <typename T, int MODE>
__device__ __forceinline__ void row_inst_ptrs(const RowInst<T>* insts, const T*& src, T*& dst, T*& dst2,
                                              Forcing& F) {
  if (!insts) return;
  const RowInst<T>& I = insts[blockIdx.y];
  F.D = I.D;
  if (MODE == ROW_FWD_USER || MODE == ROW_FWD_PHYS) {
    src = src + I.uoff;
    dst = I.W;
    dst2 = I.H;
  } else if (MODE == ROW_INV_USER) {
    src = I.W;
    dst = dst + I.uoff;
  } else {
    src = I.W;
    dst = I.W;
  }
}

// ---------------------------------------------------------------------------
// Column passes: lines along a strided axis.  A block handles pairs of adjacent
// x-columns of one "outer" index; element m of column c sits at
//   base + outer * ld_outer + m * ld_line + c.
// COL_PLAIN_INV: the inverse transform of periodic lines (COL_PLAIN is its own
// inverse on sine lines).
enum ColMode { COL_PLAIN = 0, COL_STAGE_A = 1, COL_STAGE_B = 2, COL_ETD1 = 3, COL_PLAIN_INV = 4 };

struct ColGeom {
  int n;            // line length
  int64_t ld_line;  // stride between consecutive elements of a line
  int64_t ld_outer; // stride between outer indices
  int last_is_z;    // 1: spectral index (kx, ky, kz) = (c, outer, m); 0: (c, m, 0)
  int ncols;        // real x-columns; columns ncols .. pitch-1 are padding, kept exactly zero
};

// Zero the padding half of a column pair (c = first column of the pair).
template <typename T>
__device__ __forceinline__ Cx<T> mask_pad(Cx<T> v, int c, int ncols) {
  if (c >= ncols) return Cx<T>{T(0), T(0)};
  if (c + 1 >= ncols) return Cx<T>{v.re, T(0)};
  return v;
}

// The separable tables of columns col, col + 1 combined with the non-line
// axis (z for y lines, y for z lines) at index ko.
__device__ __forceinline__ void sep3_pair(const Diag& dg, int col, bool last_is_z, int ko, Sep3* sxy) {
  const double tD = dg.tau * dg.D;
  const Sep3 so = last_is_z ? sep3_load(dg.ax[1], ko) : sep3_load(dg.ax[2], 0);
  sxy[0] = sep3_combine(sep3_load(dg.ax[0], col), so, tD);
  sxy[1] = sep3_combine(sep3_load(dg.ax[0], col + 1), so, tD);
}

// One spectral point pair (columns col, col + 1; sxy from sep3_pair) at line
// position m of a three-stage column pass: reads H (and X), writes H (and X),
// returns the two values to inverse transform.
template <typename T, int MODE>
__device__ __forceinline__ void stage3_pair(const Diag& dg, const S3K& k, const Sep3* sxy, bool last_is_z, int m,
                                            int col, int64_t off, T* H, T ga, T gb, int ncols, T* outv) {
  T* X = static_cast<T*>(dg.X);
  const Sep3 sl = sep3_load(last_is_z ? dg.ax[2] : dg.ax[1], m);
  const Cx<T> hv = *reinterpret_cast<const Cx<T>*>(H + off);
  Cx<T> xv{T(0), T(0)};
  if (MODE == COL_S3_2) xv = *reinterpret_cast<const Cx<T>*>(X + off);
  const T gin[2] = {ga, gb}, hin[2] = {hv.re, hv.im}, xin[2] = {xv.re, xv.im};
  T newh[2], newx[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const Sep3 sp = sep3_combine(sxy[q], sl, k.tau * k.D);
    double o, nh, nx = 0.0;
    diag3_apply<MODE>(sp, k, double(gin[q]), double(hin[q]), double(xin[q]), &o, &nh, &nx);
    outv[q] = T(o);
    newh[q] = T(nh);
    newx[q] = T(nx);
  }
  *reinterpret_cast<Cx<T>*>(H + off) = mask_pad(Cx<T>{newh[0], newh[1]}, col, ncols);
  if (MODE == COL_S3_1) *reinterpret_cast<Cx<T>*>(X + off) = mask_pad(Cx<T>{newx[0], newx[1]}, col, ncols);
}

// Block order of the generic column passes: the hardware hands linear block b
// (x fastest) to XCD b mod 8, so adjacent column pairs -- which share 128-byte
// lines -- would land on different XCDs and each XCD's L2 would fetch the whole
// line for a few bytes of it.  Logical block (b mod 8) * (nb / 8) + b / 8 gives
// every XCD a contiguous run of column pairs instead (a bijection; blocks past
// the last multiple of 8 keep their index).
__device__ __forceinline__ void xcd_block(int& bx, int& by) {
  const int nb = int(gridDim.x * gridDim.y);
  const int b = int(blockIdx.x + gridDim.x * blockIdx.y);
  const int q = nb / 8;
  const int l = b < 8 * q ? (b % 8) * q + b / 8 : b;
  bx = l % int(gridDim.x);
  by = l / int(gridDim.x);
}

// ---------------------------------------------------------------------------
// Periodic lines (the variant at the end of Section 4).  The 1D matrices are
// circulant, diagonalised by the real orthonormal Fourier basis; position r of
// a line holds the coefficient of the constant (r = 0), of sqrt(2/N) cos(2 pi k j/N)
// (r = k, 1 <= k < N/2), of sqrt(2/N) sin(2 pi k j/N) (r = N - k) and, for even
// N, of (-1)^j / sqrt(N) (r = N/2); its eigenvalues depend on cos(2 pi r/N)
// only.  Two real lines a, b are packed as c = a + i b of FFT length L = N.
// With Z = FFT(c) (unnormalised) and k < N - k:
//   a_k = (Z_k.re + Z_{N-k}.re) / sqrt(2N),      b_k = (Z_k.im + Z_{N-k}.im) / sqrt(2N),
//   a_{N-k} = (Z_{N-k}.im - Z_k.im) / sqrt(2N),  b_{N-k} = (Z_k.re - Z_{N-k}.re) / sqrt(2N),
// and a_r = Z_r.re / sqrt(N), b_r = Z_r.im / sqrt(N) for r = 0 and r = N/2.  The
// inverse rebuilds the Hermitian pair spectrum Z^ (Z^_k = a^_k + i b^_k) and,
// since c = conj(FFT(conj(Z^))) / sqrt(N), runs the same forward FFT.

// ---------------------------------------------------------------------------
// Norm reduction: per node, (M e)_i and (K_1 e)_i by the 3^d tensor stencil of
// the 1D matrices A = (h/6) tridiag(1,4,1), B = (1/h) tridiag(-1,2,-1)
// (Section 4, eq. (4.1)), accumulated in double.
struct NormGeom {
  int d;
  int n[3];
  int per[3];  // periodic axis: the stencil wraps around
  double ad[3], ao[3];  // A diagonal / off-diagonal
  double bd[3], bo[3];  // B diagonal / off-diagonal
  double cellvol;
  int pot;           // potential summed in accumulator 4: NORM_POT_DOUBLE_WELL or NORM_POT_FH
  double th, thc;    // Flory-Huggins theta, theta_c
};

enum { NORM_POT_DOUBLE_WELL = 0, NORM_POT_FH = 1 };

constexpr int kNormThreads = 256;
constexpr int kNormAcc = 5;  // eMe, eK1e, max|e|, uK1u, sum F(u_i)

template <typename T>
__device__ __forceinline__ double ld_err(const T* u, const T* ur, int64_t i) {
  double v = double(u[i]);
  if (ur) v -= double(ur[i]);
  return v;
}

template <typename T>
__global__ void __launch_bounds__(kNormThreads) norm_partial(const T* __restrict__ u, const T* __restrict__ ur,
                                                             NormGeom g, double* __restrict__ partials) {
  __shared__ double red[kNormAcc][kNormThreads];
  const int64_t total = int64_t(g.n[0]) * g.n[1] * g.n[2];
  double acc[kNormAcc] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const int64_t sx = 1, sy = g.n[0], sz = int64_t(g.n[0]) * g.n[1];
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < total;
       i += int64_t(gridDim.x) * blockDim.x) {
    const int ix = int(i % g.n[0]);
    const int iy = int((i / g.n[0]) % g.n[1]);
    const int iz = int(i / sz);
    double Me = 0.0, Ke = 0.0, Ku = 0.0;
    for (int oz = -1; oz <= 1; ++oz) {
      int jz = iz + oz;
      if (g.per[2]) jz = (jz + g.n[2]) % g.n[2];
      if (jz < 0 || jz >= g.n[2]) continue;
      const double az = oz ? g.ao[2] : g.ad[2];
      const double bz = oz ? g.bo[2] : g.bd[2];
      for (int oy = -1; oy <= 1; ++oy) {
        int jy = iy + oy;
        if (g.per[1]) jy = (jy + g.n[1]) % g.n[1];
        if (jy < 0 || jy >= g.n[1]) continue;
        const double ay = oy ? g.ao[1] : g.ad[1];
        const double by = oy ? g.bo[1] : g.bd[1];
        for (int ox = -1; ox <= 1; ++ox) {
          int jx = ix + ox;
          if (g.per[0]) jx = (jx + g.n[0]) % g.n[0];
          if (jx < 0 || jx >= g.n[0]) continue;
          const double axv = ox ? g.ao[0] : g.ad[0];
          const double bxv = ox ? g.bo[0] : g.bd[0];
          const int64_t j = jx * sx + jy * sy + jz * sz;
          const double ej = ld_err(u, ur, j);
          const double uj = double(u[j]);
          const double mw = axv * ay * az;
          const double kw = bxv * ay * az + axv * by * az + axv * ay * bz;
          Me += mw * ej;
          Ke += kw * ej;
          Ku += kw * uj;
        }
      }
    }
    const double ei = ld_err(u, ur, i);
    const double ui = double(u[i]);
    acc[0] += ei * Me;
    acc[1] += ei * Ke;
    acc[2] = fmax(acc[2], fabs(ei));
    acc[3] += ui * Ku;
    if (g.pot == NORM_POT_FH) {
      // F(u) = (theta/2)((1+u) ln(1+u) + (1-u) ln(1-u)) - (theta_c/2) u^2 (Example 5.3)
      acc[4] += 0.5 * g.th * ((1.0 + ui) * log1p(ui) + (1.0 - ui) * log1p(-ui)) - 0.5 * g.thc * ui * ui;
    } else {
      const double q = ui * ui - 1.0;
      acc[4] += 0.25 * q * q;
    }
  }
#pragma unroll
  for (int k = 0; k < kNormAcc; ++k) red[k][threadIdx.x] = acc[k];
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
#pragma unroll
      for (int k = 0; k < kNormAcc; ++k) {
        if (k == 2)
          red[k][threadIdx.x] = fmax(red[k][threadIdx.x], red[k][threadIdx.x + s]);
        else
          red[k][threadIdx.x] += red[k][threadIdx.x + s];
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < kNormAcc) partials[blockIdx.x * kNormAcc + threadIdx.x] = red[threadIdx.x][0];
}

// The same five sums for 3D grids, without LDS or barriers: a wavefront covers
// 64 consecutive x positions (it owns the middle 62; lanes 0 and 63 hold the
// neighbours x0 - 1 and x0 + 62) of kNwRows rows and marches over a chunk of z
// planes.  With P_A = A_y (x) A_x and P_B = A_y (x) B_x + B_y (x) A_x applied in
// the plane, M = A_z (x) P_A, K_1 = B_z (x) P_A + A_z (x) P_B and the symmetry of
// the z coupling,
//   e^T M e   = sum_z e_z . (ad_z P_A e_z + 2 ao_z P_A e_{z-1}),
//   e^T K_1 e = sum_z e_z . (bd_z P_A e_z + 2 bo_z P_A e_{z-1} + ad_z P_B e_z + 2 ao_z P_B e_{z-1}),
// so a chunk reads one plane before it (none after it) and a lane keeps only the
// previous plane's in-plane sums.  Per plane a lane loads its column of the rows
// y0 - 1 .. y0 + kNwRows (the next plane's while it computes this one), takes the
// x neighbours from the adjacent lanes (DPP shifts) and forms the in-plane sums
// separably.  Waves are ordered so that the blocks one XCD runs together own
// neighbouring rows of one z chunk: their shared halo rows come from that XCD's
// L2 (block b runs on XCD b mod 8).  Block partials as norm_partial; the grid is
// padded to a multiple of 8 blocks, waves without a task add nothing.
constexpr int kNwRows = 4;   // rows per wave
constexpr int kNwOwn = 62;   // x positions a wave owns
constexpr int kNwThreads = 256;

template <int CTRL>
__device__ __forceinline__ double dpp_double(double x) {
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = __builtin_amdgcn_update_dpp(0, int(b & 0xffffffff), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, int(b >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (long long)(unsigned(lo)) | ((long long)hi << 32));
}
__device__ __forceinline__ double from_lane_below(double x) { return dpp_double<0x138>(x); }  // lane l - 1
__device__ __forceinline__ double from_lane_above(double x) { return dpp_double<0x130>(x); }  // lane l + 1

// GEN = false: Dirichlet axes and the double-well potential only (fewer
// registers, three waves per SIMD); GEN = true: periodic axes and either potential.
template <typename T, bool GEN>
__global__ void __launch_bounds__(kNwThreads) norm_waves(const T* __restrict__ u, const T* __restrict__ ur,
                                                         NormGeom g, int zc, int nxw, int tiles_y, int ntasks,
                                                         double* __restrict__ partials) {
  constexpr int KY = kNwRows;
  __shared__ double red[kNormAcc][kNwThreads];
  double acc[kNormAcc] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const int lane = threadIdx.x & 63;
  const int nb = gridDim.x;
  const int blk = (blockIdx.x % 8) * (nb / 8) + blockIdx.x / 8;  // XCD-contiguous block order
  const int task = blk * (kNwThreads / 64) + (threadIdx.x >> 6);
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  if (task < ntasks) {
    const int xw = task % nxw;
    const int rest = task / nxw;
    const int ty = rest % tiles_y, zi = rest / tiles_y;
    int x = xw * kNwOwn + lane - 1;
    const bool own = lane >= 1 && lane <= kNwOwn && x < nx;
    if (GEN && g.per[0]) x = (x + nx) % nx;
    const bool xin = x >= 0 && x < nx;
    const int y0 = ty * KY;
    const int z0 = zi * zc, z1 = min(nz, z0 + zc);
    const int64_t sy = nx, sz = int64_t(nx) * ny;
    const double adx = g.ad[0], aox = g.ao[0], bdx = g.bd[0], box = g.bo[0];
    const double ady = g.ad[1], aoy = g.ao[1], bdy = g.bd[1], boy = g.bo[1];
    const double adz = g.ad[2], aoz2 = 2.0 * g.ao[2], bdz = g.bd[2], boz2 = 2.0 * g.bo[2];
    double pA[KY], pB[KY], qA[KY], qB[KY];  // previous plane: P_A e, P_B e, P_A u, P_B u
#pragma unroll
    for (int j = 0; j < KY; ++j) pA[j] = pB[j] = qA[j] = qB[j] = 0.0;
    // rows y0 - 1 .. y0 + KY of plane z at this lane's x (zero outside a Dirichlet boundary)
    auto load_plane = [&](int z, T (&cu)[KY + 2], T (&cr)[KY + 2]) {
      int zz = z;
      if (GEN && g.per[2]) zz = (zz + nz) % nz;
      const bool zin = zz >= 0 && zz < nz;
#pragma unroll
      for (int r = 0; r < KY + 2; ++r) {
        int yy = y0 - 1 + r;
        if (GEN && g.per[1]) yy = (yy + ny) % ny;
        const bool in = zin && yy >= 0 && yy < ny && xin;
        const int64_t j = x + yy * sy + int64_t(zz) * sz;
        cu[r] = in ? u[j] : T(0);
        cr[r] = (in && ur) ? ur[j] : T(0);
      }
    };
    T cu[KY + 2], cr[KY + 2];
    load_plane(z0 - 1, cu, cr);
    for (int z = z0 - 1; z < z1; ++z) {
      T nu[KY + 2], nr[KY + 2];
      if (z + 1 < z1) load_plane(z + 1, nu, nr);
      double sAe[KY + 2], sBe[KY + 2], sAu[KY + 2], sBu[KY + 2];
#pragma unroll
      for (int r = 0; r < KY + 2; ++r) {
        const double uv = double(cu[r]);
        const double ev = uv - double(cr[r]);
        const double en = from_lane_below(ev) + from_lane_above(ev);
        const double un = from_lane_below(uv) + from_lane_above(uv);
        sAe[r] = fma(aox, en, adx * ev);
        sBe[r] = fma(box, en, bdx * ev);
        sAu[r] = fma(aox, un, adx * uv);
        sBu[r] = fma(box, un, bdx * uv);
      }
#pragma unroll
      for (int j = 0; j < KY; ++j) {
        const double nAe = sAe[j] + sAe[j + 2], nAu = sAu[j] + sAu[j + 2];
        const double wAe = fma(aoy, nAe, ady * sAe[j + 1]);
        const double wBe = fma(aoy, sBe[j] + sBe[j + 2], fma(ady, sBe[j + 1], fma(boy, nAe, bdy * sAe[j + 1])));
        const double wAu = fma(aoy, nAu, ady * sAu[j + 1]);
        const double wBu = fma(aoy, sBu[j] + sBu[j + 2], fma(ady, sBu[j + 1], fma(boy, nAu, bdy * sAu[j + 1])));
        if (z >= z0 && own && y0 + j < ny) {
          const double ui = double(cu[j + 1]);
          const double ei = ui - double(cr[j + 1]);
          acc[0] = fma(ei, fma(adz, wAe, aoz2 * pA[j]), acc[0]);
          acc[1] = fma(ei, fma(bdz, wAe, fma(boz2, pA[j], fma(adz, wBe, aoz2 * pB[j]))), acc[1]);
          acc[2] = fmax(acc[2], fabs(ei));
          acc[3] = fma(ui, fma(bdz, wAu, fma(boz2, qA[j], fma(adz, wBu, aoz2 * qB[j]))), acc[3]);
          if (GEN && g.pot == NORM_POT_FH) {
            acc[4] += 0.5 * g.th * ((1.0 + ui) * log1p(ui) + (1.0 - ui) * log1p(-ui)) - 0.5 * g.thc * ui * ui;
          } else {
            const double q = ui * ui - 1.0;
            acc[4] = fma(0.25 * q, q, acc[4]);
          }
        }
        pA[j] = wAe;
        pB[j] = wBe;
        qA[j] = wAu;
        qB[j] = wBu;
      }
#pragma unroll
      for (int r = 0; r < KY + 2; ++r) {
        cu[r] = nu[r];
        cr[r] = nr[r];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < kNormAcc; ++k) red[k][threadIdx.x] = acc[k];
  __syncthreads();
  for (int h = kNwThreads / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) {
#pragma unroll
      for (int k = 0; k < kNormAcc; ++k) {
        if (k == 2)
          red[k][threadIdx.x] = fmax(red[k][threadIdx.x], red[k][threadIdx.x + h]);
        else
          red[k][threadIdx.x] += red[k][threadIdx.x + h];
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < kNormAcc) partials[int64_t(blockIdx.x) * kNormAcc + threadIdx.x] = red[threadIdx.x][0];
}

// Second level: 256 threads stride over the block partials, then a fixed-order
// tree in LDS (deterministic); accumulator 2 is a maximum, the others sums.
constexpr int kNormFinalThreads = 256;
static __global__ void __launch_bounds__(kNormFinalThreads) norm_final(const double* __restrict__ partials, int nblocks,
                                                                double* __restrict__ out5) {
  __shared__ double red[kNormAcc][kNormFinalThreads];
  const int t = threadIdx.x;
  double s[kNormAcc] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int b = t; b < nblocks; b += kNormFinalThreads)
#pragma unroll
    for (int k = 0; k < kNormAcc; ++k) {
      const double v = partials[b * kNormAcc + k];
      s[k] = (k == 2) ? fmax(s[k], v) : s[k] + v;
    }
#pragma unroll
  for (int k = 0; k < kNormAcc; ++k) red[k][t] = s[k];
  __syncthreads();
  for (int h = kNormFinalThreads / 2; h > 0; h >>= 1) {
    if (t < h)
#pragma unroll
      for (int k = 0; k < kNormAcc; ++k)
        red[k][t] = (k == 2) ? fmax(red[k][t], red[k][t + h]) : red[k][t] + red[k][t + h];
    __syncthreads();
  }
  if (t < kNormAcc) out5[t] = red[t][0];
}

// norm_final's reduction followed by the finishing arithmetic of eife_norms on
// the device: out4 = (||e||_0, ||e||_1, max|e|, energy) with ||e||_0^2 = e^T M e,
// ||e||_1^2 = e^T M e + e^T K_1 e and energy = (D/2) u^T K_1 u + cellvol sum F(u_i).
static __global__ void __launch_bounds__(kNormFinalThreads) norm_finish(const double* __restrict__ partials, int nblocks,
                                                                 double D, double cellvol, double* __restrict__ out4) {
  __shared__ double red[kNormAcc][kNormFinalThreads];
  const int t = threadIdx.x;
  double s[kNormAcc] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int b = t; b < nblocks; b += kNormFinalThreads)
#pragma unroll
    for (int k = 0; k < kNormAcc; ++k) {
      const double v = partials[b * kNormAcc + k];
      s[k] = (k == 2) ? fmax(s[k], v) : s[k] + v;
    }
#pragma unroll
  for (int k = 0; k < kNormAcc; ++k) red[k][t] = s[k];
  __syncthreads();
  for (int h = kNormFinalThreads / 2; h > 0; h >>= 1) {
    if (t < h)
#pragma unroll
      for (int k = 0; k < kNormAcc; ++k)
        red[k][t] = (k == 2) ? fmax(red[k][t], red[k][t + h]) : red[k][t] + red[k][t + h];
    __syncthreads();
  }
  if (t == 0) {
    out4[0] = sqrt(fmax(red[0][0], 0.0));
    out4[1] = sqrt(fmax(red[0][0] + red[1][0], 0.0));
    out4[2] = red[2][0];
    out4[3] = 0.5 * D * red[3][0] + cellvol * red[4][0];
  }
}

}  // namespace eife
