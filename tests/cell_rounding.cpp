// Rounding errors of the FP64 cell integrals of csrc/cellmath.hpp, compiled for
// the host, against the plain form of the same integrals in double (edges as
// log1p of quotients of terms of one sign, the solid angle by atan2, gradients
// from the foot of the target on the edge's line), both measured with 128 bits.
// Prints per form and zone of distances (in diameters, from the centroid, the
// edges and the vertices) the root mean square of the 99 % smallest errors of
// field, potential and gradient: "<form> <lo> <hi> <quantity> <library> <plain>".
#include <quadmath.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

// The device's builtins on the host; its estimates are good to 2^-24.
static double hidden(double x) { return x * (1.0 + (drand48() - 0.5) * 0x1p-23); }
static double host_rcp(double x) { return hidden(1.0 / x); }
static double host_rsq(double x) { return hidden(1.0 / std::sqrt(x)); }
static int host_frexp_exp(double x) {
  int e = 0;
  std::frexp(x, &e);
  return e;
}
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_rcp host_rcp
#define __builtin_amdgcn_rsq host_rsq
#define __builtin_amdgcn_frexp_exp host_frexp_exp
#define __builtin_amdgcn_ldexp std::ldexp
struct alignas(16) double2 {
  double x, y;
};
using std::fabs;
using std::fma;
#include "cellmath.hpp"
using namespace obem;

typedef __float128 Q;
struct q3 {
  Q x, y, z;
};
static q3 wide(d3 a) { return {a.x, a.y, a.z}; }
static q3 operator-(q3 a, q3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
static q3 operator+(q3 a, q3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
static q3 operator*(q3 a, Q s) { return {a.x * s, a.y * s, a.z * s}; }
static Q dot(q3 a, q3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
static q3 cross(q3 a, q3 b) { return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x}; }

template <class V, class S>
struct Result {
  V E, G;
  S P;
};

static Result<q3, Q> exact(const d3 *v, d3 x, d3 w8) {
  const q3 u[3] = {wide(v[0]), wide(v[1]), wide(v[2])}, w = wide(w8);
  q3 P[3];
  Q R[3];
  for (int k = 0; k < 3; ++k) {
    P[k] = u[k] - wide(x);
    R[k] = sqrtq(dot(P[k], P[k]));
  }
  const q3 N = cross(u[1] - u[0], u[2] - u[0]);
  const Q ta = sqrtq(dot(N, N));
  const q3 n = N * (1 / ta);
  const Q h = -dot(P[0], n), den = R[0] * R[1] * R[2] + dot(P[0], P[1]) * R[2] + dot(P[0], P[2]) * R[1] + dot(P[1], P[2]) * R[0];
  const Q om = 2 * atan2q(ta * h, den);
  Result<q3, Q> r = {n * om, {0, 0, 0}, -h * om};
  q3 gO = {0, 0, 0};
  for (int e = 0; e < 3; ++e) {
    const int b = (e + 1) % 3;
    const q3 d = u[b] - u[e];
    const Q L = sqrtq(dot(d, d));
    const q3 t = d * (1 / L), m = cross(t, n), c = cross(t, P[e]);
    const Q lm = dot(t, P[e]), lp = lm + L, R2 = dot(c, c), p = lm * lp, mm = R[e] * R[b];
    const Q ab = 2 * (R2 + (p >= 0 ? mm + p : R2 * (R2 + lm * lm + lp * lp) / (mm - p))), a = R[e] + R[b] + L;
    const Q f = log1pq(2 * L * a / ab), C = 2 * L / ab, mw = dot(m, w);
    r.E = r.E + m * f;
    r.P += dot(m, P[e]) * f;
    r.G = r.G + (P[e] * (1 / R[e]) + P[b] * (1 / R[b])) * (C * mw);
    gO = gO + c * (C * (1 / R[e] + 1 / R[b]));
  }
  r.G = r.G + gO * dot(n, w);
  return r;
}

// A cell's record as the library makes it.
static void record(const d3 *v, double *rec) {
  const d3 N = cross3(v[1] - v[0], v[2] - v[0]);
  const double n2 = norm3(N);
  const d3 n = N * (1.0 / n2);
  for (int e = 0; e < 3; ++e) {
    d3 t = v[(e + 1) % 3] - v[e];
    double *re = rec + CR_EDGE + CR_EDGE_SIZE * e;
    re[0] = norm3(t);
    t = t * (1.0 / re[0]);
    const d3 m = cross3(t, n);
    const double d[6] = {t.x, t.y, t.z, m.x, m.y, m.z};
    for (int k = 0; k < 6; ++k) re[1 + k] = d[k];
    rec[3 * e] = v[e].x;
    rec[3 * e + 1] = v[e].y;
    rec[3 * e + 2] = v[e].z;
  }
  rec[CR_N] = n.x;
  rec[CR_N + 1] = n.y;
  rec[CR_N + 2] = n.z;
  rec[CR_2A] = n2;
}

static Result<d3, double> plain(const double *rec, d3 x, d3 w) {
  d3 P[3];
  double R[3];
  for (int k = 0; k < 3; ++k) {
    P[k] = mk3(rec[3 * k], rec[3 * k + 1], rec[3 * k + 2]) - x;
    R[k] = norm3(P[k]);
  }
  const d3 n = mk3(rec[CR_N], rec[CR_N + 1], rec[CR_N + 2]);
  const double h = -dot3(P[0], n), num = rec[CR_2A] * h;
  const double den = R[0] * R[1] * R[2] + dot3(P[0], P[1]) * R[2] + dot3(P[0], P[2]) * R[1] + dot3(P[1], P[2]) * R[0];
  const double om = num != 0.0 ? 2.0 * std::atan2(num, den) : 0.0;
  Result<d3, double> r = {n * om, mk3(0, 0, 0), -h * om};
  d3 gO = mk3(0, 0, 0);
  for (int e = 0; e < 3; ++e) {
    const int b = (e + 1) % 3;
    const double *re = rec + CR_EDGE + CR_EDGE_SIZE * e;
    const double L = re[0];
    const d3 t = mk3(re[1], re[2], re[3]), m = mk3(re[4], re[5], re[6]), c = cross3(t, P[e]);
    const double lm = dot3(t, P[e]), lp = lm + L, R2 = dot3(c, c), s = lp + lm, S = R[b] + R[e];
    double f, D;
    if (s >= 0.0)
      f = lm >= 0.0 ? std::log1p(L * (S + s) / (S * (R[e] + lm))) : std::log1p(L * (S + s) * (R[e] - lm) / (S * R2));
    else
      f = lp <= 0.0 ? std::log1p(L * (S - s) / (S * (R[b] - lp))) : std::log1p(L * (S - s) * (R[b] + lp) / (S * R2));
    if (lm >= 0.0)
      D = 1.0 / (R[e] * (R[e] + lm)) - 1.0 / (R[b] * (R[b] + lp));
    else if (lp <= 0.0)
      D = 1.0 / (R[b] * (R[b] - lp)) - 1.0 / (R[e] * (R[e] - lm));
    else
      D = (lp / R[b] - lm / R[e]) / R2;
    const double di = -L * s / (S * R[b] * R[e]);
    const d3 foot = t * lm - P[e];
    r.G = r.G + (foot * (-D) + t * (-di)) * dot3(m, w);
    gO = gO + cross3(t, foot) * (-D);
    r.E = r.E + m * f;
    r.P += dot3(m, P[e]) * f;
  }
  r.G = r.G + gO * dot3(n, w);
  return r;
}

static Result<d3, double> library(const double *rec, d3 x, d3 w, bool mid) {
  Result<d3, double> r;
  double u;
  if (mid) {
    cell_mid_form<true>(rec, x, r.E, r.P);
    cell_grad_mid(rec, x, w, r.G, u);
  } else {
    cell_closed_form<true>(rec, x, r.E, r.P);
    cell_grad_closed(rec, x, w, r.G, u);
  }
  return r;
}

static double normal() { return std::sqrt(-2.0 * std::log(1.0 - drand48())) * std::cos(6.283185307179586 * drand48()); }
static d3 normal3() { return mk3(normal(), normal(), normal()); }

static double trimmed_rms(std::vector<double> &e) {
  std::sort(e.begin(), e.end());
  const size_t n = e.size() * 99 / 100;
  double s = 0.0;
  for (size_t i = 0; i < n; ++i) s += e[i] * e[i];
  return std::sqrt(s / n);
}

int main(int argc, char **argv) {
  const int n = argc > 1 ? std::atoi(argv[1]) : 30000;
  srand48(argc > 2 ? std::atoi(argv[2]) : 1);
  const double zones[] = {0.01, 0.1, 0.18, 0.3, 0.45, 0.7, 1.0, 1.5, 2.5, 6.0, 24.0, 48.0};
  const int nz = (int)(sizeof zones / sizeof *zones) - 1;
  for (int z = 0; z < nz; ++z) {
    const bool far = zones[z] >= kMidForm;
    for (int mid = 0; mid <= (far ? 1 : 0); ++mid) {
      std::vector<double> err[2][3];
      for (int it = 0; it < n; ++it) {
        d3 v[3];
        double D = 0.0, ta;
        do {
          for (d3 &p : v) p = normal3() * 1e-5;
          D = 0.0;
          for (int k = 0; k < 3; ++k) D = std::max(D, norm3(v[(k + 1) % 3] - v[k]));
          ta = norm3(cross3(v[1] - v[0], v[2] - v[0]));
        } while (ta < 0.1 * D * D);
        const double t = drand48(), r = D * zones[z] * std::exp(drand48() * std::log(zones[z + 1] / zones[z]));
        const d3 centre = (v[0] + v[1] + v[2]) * (1.0 / 3.0);
        const d3 base = far || it % 3 == 0 ? centre : (it % 3 == 1 ? v[0] * t + v[1] * (1.0 - t) : v[0]);
        const d3 dir = normal3(), w = normal3(), x = base + dir * (r * (far ? 1.0 + 1e-9 : 1.0) / norm3(dir));
        alignas(16) double rec[CR_COUNT] = {};
        record(v, rec);
        const Result<q3, Q> ref = exact(v, x, w);
        const Result<d3, double> got[2] = {library(rec, x, w, mid != 0), plain(rec, x, w)};
        for (int k = 0; k < 2; ++k) {
          const q3 dE = wide(got[k].E) - ref.E, dG = wide(got[k].G) - ref.G;
          err[k][0].push_back((double)sqrtq(dot(dE, dE) / dot(ref.E, ref.E)));
          err[k][1].push_back((double)fabsq((got[k].P - ref.P) / ref.P));
          err[k][2].push_back((double)sqrtq(dot(dG, dG) / dot(ref.G, ref.G)));
        }
      }
      const char *what[] = {"field", "potential", "gradient"};
      for (int q = 0; q < 3; ++q)
        std::printf("%s %g %g %s %.4e %.4e\n", mid ? "mid" : "closed", zones[z], zones[z + 1], what[q],
                    trimmed_rms(err[0][q]), trimmed_rms(err[1][q]));
    }
  }
}
