// Device-side integrals of a flat triangular cell with unit charge density
// (the cell integrals of eqs. (BEM2), (BEM3)):
//   IV(x) = int_C dS'/|x - r'|,   IE(x) = int_C (x - r')/|x - r'|^3 dS'.
// Closed form (divergence theorem on the flat cell): with edge unit tangents
// t_e, in-plane outward normals m_e = t_e x n, edge line integrals
// f_e = int_e dl'/|x - r'| and the signed solid angle Omega,
//   IE = sum_e m_e f_e + n Omega,   IV = sum_e (m_e . (p_e - x)) f_e - h Omega.
// Far from the cell the closed form cancels (its terms are O(D/R) for an
// O((D/R)^2) result), so distant cells use symmetric quadrature rules, whose
// truncation error at those distances is below the working precision.
#pragma once

#include <hip/hip_runtime.h>

namespace obem {

struct d3 {
  double x, y, z;
};
__device__ __forceinline__ d3 mk3(double x, double y, double z) { return d3{x, y, z}; }
__device__ __forceinline__ d3 operator-(d3 a, d3 b) { return d3{a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ d3 operator+(d3 a, d3 b) { return d3{a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ d3 operator*(d3 a, double s) { return d3{a.x * s, a.y * s, a.z * s}; }
__device__ __forceinline__ double dot3(d3 a, d3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ d3 cross3(d3 a, d3 b) {
  return d3{a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ __forceinline__ double norm3(d3 a) { return sqrt(dot3(a, a)); }

// FP64 reciprocal, quotient, square root and reciprocal square root from the
// hardware estimates (about 2^-24): Newton steps to full precision, without
// the range scaling of the library functions (the arguments here are sums and
// products of lengths, far from the ends of the exponent range).  sqrt_f64(0)
// is 0; the others are for positive arguments.
__device__ __forceinline__ double rcp_f64(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ double div_f64(double n, double x) {
  const double y = rcp_f64(x), q = n * y;
  return fma(fma(-x, q, n), y, q);
}
__device__ __forceinline__ double sqrt_f64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  g = fma(fma(-g, g, x), h, g);
  return x == 0.0 ? 0.0 : g;
}
// The square root and its reciprocal (x > 0).
__device__ __forceinline__ double sqrt_rcp_f64(double x, double &inv) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  g = fma(fma(-g, g, x), h, g);
  const double i = h + h;
  inv = fma(fma(-g, i, 1.0), i, i);
  return g;
}
// y (1 + e/2 + 3 e^2/8), e = 1 - x y^2: third order, one step from the
// estimate (two Newton steps took two operations more).
__device__ __forceinline__ double rsqrt_f64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * y), y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// a b + k for a constant k: k in a scalar register pair.  The compiler copies
// a polynomial's constants to vector registers instead (one more instruction
// per term, and the registers).
__device__ __forceinline__ double fma_k(double a, double b, double k) {
#ifdef __HIP_DEVICE_COMPILE__
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(k));
  return r;
#else
  return fma(a, b, k);
#endif
}
// (atanh(s) - s) / s^3 on s^2 = z <= 0.0297 and (WIDE) z <= 0.075, and
// (atan(t) - t) / t^3 on t^2 = u <= 1/16: minimax polynomials, relative error
// of the functions 5e-18, 3e-18 and 2e-17.
template <bool WIDE>
__device__ __forceinline__ double atanh_tail(double z) {
  double q;
  if (WIDE) {
    q = fma_k(z, 0.072060841267327696066, 0.055923049841696995365);
    q = fma_k(q, z, 0.066893222591322001645);
    q = fma_k(q, z, 0.076912886123458226635);
    q = fma_k(q, z, 0.09090935855713595118);
    q = fma_k(q, z, 0.11111110717632652524);
    q = fma_k(q, z, 0.14285714288605414739);
    q = fma_k(q, z, 0.19999999999991834572);
    return fma_k(q, z, 0.33333333333333337125);
  }
  q = fma_k(z, 0.073145028437917779823, 0.076653489385718816166);
  q = fma_k(q, z, 0.090914600915225965373);
  q = fma_k(q, z, 0.11111105352279153539);
  q = fma_k(q, z, 0.14285714314319351255);
  q = fma_k(q, z, 0.19999999999946780889);
  return fma_k(q, z, 0.33333333333333349485);
}
__device__ __forceinline__ double atan_tail(double u) {
  double q = fma_k(u, 0.04726845190252479579, -0.06554434847623053629);
  q = fma_k(q, u, 0.076865024041207992868);
  q = fma_k(q, u, -0.090907412155468317155);
  q = fma_k(q, u, 0.11111108462732517272);
  q = fma_k(q, u, -0.14285714265141588082);
  q = fma_k(q, u, 0.199999999999390121);
  return fma_k(q, u, -0.33333333333333303632);
}

// 1/sqrt(x) of a squared distance that may overflow (x > 0): 0 for an infinite
// one, where the estimate's product would be infinity times zero.
__device__ __forceinline__ double inv_sqrt_f64(double x) {
  const double r = rsqrt_f64(x);
  return x == (double)INFINITY ? 0.0 : r;
}

// Line integral of 1/|x - r'| along an edge of length L whose endpoints, seen
// from x, are Pm and Pp (lengths Rm, Rp): with S = Rm + Rp, a = S + L and
// b = S - L,
//   f = log(a / b),
// as e ln 2 + 2 atanh(s), s = (a 2^-e - b) / (a 2^-e + b), |s| <= 0.172, the
// atanh by a degree-15 polynomial: one polynomial for every target, where
// log1p of one of four quotients (by the position of the target's foot) ran up
// to four times in a wave.  s is formed from S and L, exact in the small
// difference far from the edge (e = 0: s = L / S).
// Close to the edge b cancels, and a / b is 1 + q with the quotient of terms
// of one sign instead (l = t . P, R0 = |t x P|; the mirrored one where lm + lp
// < 0):
//   q = L (S + lm + lp) / (S (Rm + lm))             for lm >= 0,
//       L (S + lm + lp) (Rm - lm) / (S R0^2)        for a foot inside the edge,
// s = (q 2^-e - (1 - 2^-e)) / (q 2^-e + (1 + 2^-e)).  Close is L > 0.45 S:
// there both forms round equally.  (With 0.667 and b from the edge's distance the
// field's error at 0.1 to 0.7 diameters was 12 to 18 % above that of log1p with
// the quotient everywhere; with 0.45 it is at most that at every distance, with
// 0.5 up to 1 % above it at 0.45 to 0.7 diameters.)
// On the edge itself q and f are infinite.
// C_out: C = 2 L / (a b), for the gradient, from a b / 2 = Rm Rp + Pm . Pp, or
// where x sees the edge under more than a right angle (its foot is inside, lm
// lp < 0), R0^2 (R0^2 + lm^2 + lp^2 + u) / u with u = Rm Rp - lm lp.
__device__ __forceinline__ double edge_f(d3 Pm, d3 Pp, double Rm, double Rp, d3 t, double L, double *C_out) {
  const double S = Rm + Rp;
  const bool close = L > 0.45 * S;
  double q = 0.0, B = S, ratio = (S + L) * __builtin_amdgcn_rcp(S - L);
  const double dp = C_out ? dot3(Pm, Pp) : 0.0;
  double cn = L, cd = fma(Rm, Rp, dp);
  if (close) {
    const d3 c = cross3(t, Pm);
    const double R2 = dot3(c, c);
    double lm = dot3(t, Pm), lp = lm + L, r1 = Rm;
    if (dp < 0.0) {
      const double u = fma(Rm, Rp, -(lm * lp));
      cn = L * u;
      cd = R2 * (R2 + fma(lm, lm, lp * lp) + u);
    }
    if (lp + lm < 0.0) {
      const double l = lm;
      lm = -lp;
      lp = -l;
      r1 = Rp;
    }
    const double n = L * (S + (lp + lm));
    B = S * (lm < 0.0 ? R2 : r1 + lm);
    q = div_f64(lm < 0.0 ? n * (r1 - lm) : n, B);
    ratio = 1.0 + q;
  }
  if (C_out) *C_out = div_f64(cn, cd);
  // e = round(log2(a / b)), from the estimate of the ratio
  const int e = __builtin_amdgcn_frexp_exp(ratio * 1.4142135623730951) - 1;
  const double k = __builtin_amdgcn_ldexp(1.0, -e);
  const double num = close ? fma(q, k, k - 1.0) : fma(-S, 1.0 - k, L * (1.0 + k));
  const double den = close ? fma(q, k, k + 1.0) : fma(S, 1.0 + k, -L * (1.0 - k));
  const double s = div_f64(num, den), z = s * s;
  const double s2 = s + s, tail = s2 * z * atanh_tail<false>(z);
  // e ln 2 in two parts, the first a product without rounding
  const double h = (double)e * 0x1.62e42fefap-1, f = h + s2;
  const double r = (h - f) + s2 + fma((double)e, 0x1.cf79abc9e3b39p-40, tail);
  return B == 0.0 ? (double)INFINITY : f + r;
}

// Large angles, rare: kept out of line, since the library's constants
// otherwise take registers of every wave of the kernel.
static __device__ __attribute__((noinline)) double wide_angle(double num, double den) { return 2.0 * atan2(num, den); }

// Solid angle 2 atan2(num, den): by atan_tail where |num| <= den / 4, which holds
// for every target farther than about a diameter; atan2 otherwise.
__device__ __forceinline__ double solid_angle(double num, double den) {
  if (fabs(num) <= 0.25 * den) {
    if (num == 0.0) return 0.0;
    const double z = div_f64(num, den), u = z * z;
    return 2.0 * fma(z * u, atan_tail(u), z);
  }
  return num != 0.0 ? wide_angle(num, den) : 0.0;
}

// The closed form's data of one cell, contiguous (cell-major): vertices,
// unit normal, twice the area (CR_*), then per edge e = a->b, b->c, c->a its
// length, unit tangent t_e and in-plane outward normal t_e x n, with pads to
// whole 16-byte loads.  One cell is then consecutive wide loads of a lane or
// scalar loads of a wave, instead of 34 loads from as many arrays.
enum CellRec { CR_V = 0, CR_N = 9, CR_2A = 12, CR_EDGE = 16, CR_EDGE_SIZE = 8, CR_COUNT = 40 };

// n (even) consecutive doubles at 16-byte aligned p.
template <int n>
__device__ __forceinline__ void load_doubles(const double *__restrict__ p, double *d) {
#pragma unroll
  for (int i = 0; i < n / 2; ++i) {
    const double2 t = reinterpret_cast<const double2 *>(p)[i];
    d[2 * i] = t.x;
    d[2 * i + 1] = t.y;
  }
}

// The vertices of a cell's record (CellRec) minus x, their distances, the
// normal, minus the height, and num / den of the solid angle's tangent.
struct CellSeen {
  d3 P[3], n;
  double R[3], mh, num, den;
};
__device__ __forceinline__ CellSeen cell_seen(const double *__restrict__ rec, d3 x) {
  CellSeen s;
  double d[14];
  load_doubles<14>(rec, d);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    s.P[k] = mk3(d[3 * k], d[3 * k + 1], d[3 * k + 2]) - x;
    s.R[k] = sqrt_f64(dot3(s.P[k], s.P[k]));
  }
  s.n = mk3(d[9], d[10], d[11]);
  s.mh = dot3(s.P[0], s.n);
  s.num = -d[12] * s.mh;
  s.den = fma(s.R[0] * s.R[1], s.R[2],
              fma(dot3(s.P[0], s.P[1]), s.R[2],
                  fma(dot3(s.P[0], s.P[2]), s.R[1], dot3(s.P[1], s.P[2]) * s.R[0])));
  return s;
}
// Next edge: rotates the vertices.
__device__ __forceinline__ void rotate3(CellSeen &s) {
  const d3 p = s.P[0];
  const double r = s.R[0];
  s.P[0] = s.P[1];
  s.R[0] = s.R[1];
  s.P[1] = s.P[2];
  s.R[1] = s.R[2];
  s.P[2] = p;
  s.R[2] = r;
}

// Closed form in FP64 of the cell with record rec at x.  A target exactly in
// the plane gets Omega = 0 (the principal value of the normal field).  Bound
// by FP64 operations; the edges run in a loop, each loading its own data,
// since unrolled they take over 200 registers and two waves per SIMD.
// Against 128-bit arithmetic the relative error of IE (root mean square of the
// 99 % smallest) is 6.0e-16 at 0.3-0.45 D, 8.2e-16 at 0.45-0.7 D, 2.4e-15 at
// 1.5-2.5 D and 4.1e-14 at 24-48 D (6.0e-16, 8.3e-16, 2.7e-15 and 4.8e-14 for
// log1p and atan2 of quotients without cancellation).
template <bool WANT_V>
__device__ __forceinline__ void cell_closed_form(const double *__restrict__ rec, d3 x, d3 &IE, double &IV) {
  CellSeen s = cell_seen(rec, x);
  const double Om = solid_angle(s.num, s.den);
  IE = s.n * Om;
  IV = s.mh * Om;
#pragma unroll 1
  for (int e = 0; e < 3; ++e) {
    double d[8];
    load_doubles<8>(rec + CR_EDGE + CR_EDGE_SIZE * e, d);
    const double f = edge_f(s.P[0], s.P[1], s.R[0], s.R[1], mk3(d[1], d[2], d[3]), d[0], nullptr);
    const d3 m = mk3(d[4], d[5], d[6]);
    IE = IE + m * f;
    if (WANT_V) IV = fma(dot3(m, s.P[0]), f, IV);
    rotate3(s);
  }
}

// The same for x at least kMidForm diameters D from the centroid: the
// vertices are within 2 D / 3 of it, so each edge has L / S < 0.273 (f = 2
// atanh(L / S), within the polynomial's range) and |num| < den / 4: no case
// is left to tell apart, and the four quotients share one reciprocal.
constexpr double kMidForm = 2.5;
template <bool WANT_V>
__device__ __forceinline__ void cell_mid_form(const double *__restrict__ rec, d3 x, d3 &IE, double &IV) {
  const CellSeen s = cell_seen(rec, x);
  const double S0 = s.R[0] + s.R[1], S1 = s.R[1] + s.R[2], S2 = s.R[2] + s.R[0];
  const double p01 = S0 * S1, p23 = S2 * s.den, r = rcp_f64(p01 * p23);
  const double r01 = r * p23, r23 = r * p01;
  auto quot = [](double n, double d, double rd) {
    const double q = n * rd;
    return fma(fma(-d, q, n), rd, q);
  };
  const double z = quot(s.num, s.den, r23 * S2), u = z * z;
  const double Om = 2.0 * fma(z * u, atan_tail(u), z);
  IE = s.n * Om;
  IV = s.mh * Om;
  const double S[3] = {S0, S1, S2}, iS[3] = {r01 * S1, r01 * S0, r23 * s.den};
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    double d[8];
    load_doubles<8>(rec + CR_EDGE + CR_EDGE_SIZE * e, d);
    const double t = quot(d[0], S[e], iS[e]), w = t * t, t2 = t + t;
    const double f = fma(t2 * w, atanh_tail<true>(w), t2);
    const d3 m = mk3(d[4], d[5], d[6]);
    IE = IE + m * f;
    if (WANT_V) IV = fma(dot3(m, s.P[e]), f, IV);
  }
}

// FP64 closed-form Jacobian of a unit-density cell contracted with w:
//   gtw = G^T w = sum_e (m_e . w) grad f_e + (n . w) grad Omega
// and ie_w = w . IE.  P[k] = vertex k minus the target.  With f = log(a / b)
// (edge_f) and C = 2 L / (a b),
//   grad f_e = C (Pm/Rm + Pp/Rp),   grad Omega = sum_e (t_e x Pm) C (1/Rm + 1/Rp),
// sums of terms of one sign in the far range: at 24-48 D the relative error
// against 128 bits is 2.9e-14 where differences of reciprocals had 9.7e-13, at
// 0.45-0.7 D 6.8e-16 and 9.1e-16.
__device__ __forceinline__ void cell_grad_closed(const double *__restrict__ rec, d3 x, d3 w, d3 &gtw, double &ie_w) {
  CellSeen s = cell_seen(rec, x);
  const double nw = dot3(s.n, w);
  ie_w = nw * solid_angle(s.num, s.den);
  gtw = mk3(0, 0, 0);
  d3 gO = mk3(0, 0, 0);
#pragma unroll 1
  for (int e = 0; e < 3; ++e) {
    double d[8];
    load_doubles<8>(rec + CR_EDGE + CR_EDGE_SIZE * e, d);
    const double L = d[0];
    const d3 t = mk3(d[1], d[2], d[3]);
    double C;
    const double f = edge_f(s.P[0], s.P[1], s.R[0], s.R[1], t, L, &C);
    const double im = rcp_f64(s.R[0]), ip = rcp_f64(s.R[1]);
    const double mw = dot3(mk3(d[4], d[5], d[6]), w);
    ie_w = fma(mw, f, ie_w);
    gtw = gtw + (s.P[0] * im + s.P[1] * ip) * (C * mw);
    gO = gO + cross3(t, s.P[0]) * (C * (im + ip));
    rotate3(s);
  }
  gtw = gtw + gO * nw;
}

// The same for x at least kMidForm diameters from the centroid (see
// cell_mid_form): with t = L / S, C = 2 t / (S (1 - t^2)); two reciprocals
// for the seven quotients.
__device__ __forceinline__ void cell_grad_mid(const double *__restrict__ rec, d3 x, d3 w, d3 &gtw, double &ie_w) {
  double d[14];
  load_doubles<14>(rec, d);
  d3 P[3];
  double R[3], iR[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    P[k] = mk3(d[3 * k], d[3 * k + 1], d[3 * k + 2]) - x;
    R[k] = sqrt_rcp_f64(dot3(P[k], P[k]), iR[k]);
  }
  const d3 n = mk3(d[9], d[10], d[11]);
  const double num = -d[12] * dot3(P[0], n);
  const double den = fma(R[0] * R[1], R[2],
                         fma(dot3(P[0], P[1]), R[2], fma(dot3(P[0], P[2]), R[1], dot3(P[1], P[2]) * R[0])));
  const double S0 = R[0] + R[1], S1 = R[1] + R[2], S2 = R[2] + R[0];
  const double p01 = S0 * S1, p23 = S2 * den, r = rcp_f64(p01 * p23);
  const double r01 = r * p23, r23 = r * p01;
  auto quot = [](double a, double b, double rb) {
    const double q = a * rb;
    return fma(fma(-b, q, a), rb, q);
  };
  const double z = quot(num, den, r23 * S2), zz = z * z;
  const double nw = dot3(n, w);
  ie_w = nw * (2.0 * fma(z * zz, atan_tail(zz), z));
  const double S[3] = {S0, S1, S2}, iS[3] = {r01 * S1, r01 * S0, r23 * den};
  double t[3], o[3];
  d3 et[3], em[3];
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    double c[8];
    load_doubles<8>(rec + CR_EDGE + CR_EDGE_SIZE * e, c);
    t[e] = quot(c[0], S[e], iS[e]);
    o[e] = fma(-t[e], t[e], 1.0);
    et[e] = mk3(c[1], c[2], c[3]);
    em[e] = mk3(c[4], c[5], c[6]);
  }
  const double o01 = o[0] * o[1], ro = rcp_f64(o01 * o[2]), rq = ro * o[2];
  const double io[3] = {rq * o[1], rq * o[0], ro * o01};
  gtw = mk3(0, 0, 0);
  d3 gO = mk3(0, 0, 0);
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const int e1 = (e + 1) % 3;
    const double t2 = t[e] + t[e], tt = t[e] * t[e];
    const double C = t2 * iS[e] * io[e];
    const double mw = dot3(em[e], w);
    ie_w = fma(mw, fma(t2 * tt, atanh_tail<true>(tt), t2), ie_w);
    gtw = gtw + (P[e] * iR[e] + P[e1] * iR[e1]) * (C * mw);
    gO = gO + cross3(et[e], P[e]) * (C * (iR[e] + iR[e1]));
  }
  gtw = gtw + gO * nw;
}

// Symmetric quadrature rules on the triangle, barycentric weights
// (Radon's 7-point degree-5 rule; the 3-point degree-2 rule at the edge
// midpoint-centroid points (2/3, 1/6, 1/6)).
// Near/far test of the mixed cell field (squared FP32 distance of values
// recentred on one target of the workgroup).  The far and near kernels of
// the field and of its adjoint all use this arithmetic on identically
// recentred operands, so each (target, cell) pair is taken by exactly one.
__device__ __forceinline__ float dist2f(float a0, float a1, float a2, float b0, float b1, float b2) {
  const float dx = a0 - b0, dy = a1 - b1, dz = a2 - b2;
  return fmaf(dx, dx, fmaf(dy, dy, dz * dz));
}

// Degree-4, 6-point symmetric rule on the triangle (Dunavant, Int. J.
// Numer. Methods Eng. 21 (1985) 1129): barycentric (b1, a1, a1) with weight
// w1 and (b2, a2, a2) with weight w2, each in its 3 permutations.
struct Rule6 {
  static constexpr double a1 = 0.445948490915965, b1 = 0.108103018168070, w1 = 0.223381589678011;
  static constexpr double a2 = 0.091576213509771, b2 = 0.816847572980459, w2 = 0.109951743655322;
};

// Degree-3, 4-point rule on the triangle (Strang and Fix, An Analysis of the
// Finite Element Method, 1973): the centroid with weight -27/48 and
// (3/5, 1/5, 1/5) in its 3 permutations with weight 25/48.
struct Rule4 {
  static constexpr double a = 0.2, b = 0.6, wc = -27.0 / 48.0, wp = 25.0 / 48.0;
};

struct Rule7 {
  // a = (6 - sqrt 15)/21, b = (6 + sqrt 15)/21
  static constexpr double a = 0.10128650732345633880;
  static constexpr double b = 0.47014206410511508977;
  static constexpr double w0 = 9.0 / 40.0;
  static constexpr double wa = 0.12593918054482715260;  // (155 - sqrt 15)/1200
  static constexpr double wb = 0.13239415278850618073;  // (155 + sqrt 15)/1200
};

}  // namespace obem
