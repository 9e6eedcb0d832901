// Influence of the point charges on the collocation equations (section
// 3.3.2, eqs. (potpart), (fldpart), (BEMpotpart), (BEMfldpart)): the charges'
// potential and field averaged over each cell,
//   Vbar_i = k_e/A_i sum_p q_p IV_i(x_p),   Ebar_i = -k_e/A_i sum_p q_p IE_i(x_p),
// change the left-hand side of the system before it is solved:
//   ed rows V_i - Vbar_i,   dd rows sigma_F,i - eps0 (eps_r2 - eps_r1) Ebar_i . n_i.
//
// It is the transpose of the cell field: the cells are taken in the mesh's
// Hilbert order of centroids (a workgroup's cells are spatially close and are
// recentred on the first centroid of their 256), the lanes hold charges,
// gridDim.y chunks of charges with per-chunk partial sums reduced in chunk
// order.  Precision regimes as in the field: mixed = FP32 7-point rule
// within 6 diameters, 6-point rule within 16, 4-point rule within 40, 3-point
// rule beyond (far kernel, charges ordered by charge sign, then Hilbert, so the
// charge comes out of the pair loop), FP64
// closed form within 3 diameters (near kernel, its own partial slots);
// FP64 = closed form within 48 diameters, FP64 7-point rule beyond.
#include <algorithm>
#include <cmath>

#include "cellmath.hpp"
#include "obem_internal.hpp"

namespace obem {

constexpr int kTI = 256;

// FP64 closed form of one cell at one charge: q IV and q IE.
__device__ __forceinline__ void infl_closed(const double *__restrict__ rec, int k, double px, double py, double pz,
                                            double q, double &sv, double &ex, double &ey, double &ez) {
  d3 IE;
  double IV;
  cell_closed_form<true>(rec + (size_t)k * CR_COUNT, mk3(px, py, pz), IE, IV);
  sv = fma(q, IV, sv);
  ex = fma(q, IE.x, ex);
  ey = fma(q, IE.y, ey);
  ez = fma(q, IE.z, ez);
}

// Far part of the mixed influence, charge-major: a workgroup owns 8 cells
// (consecutive in the mesh's Hilbert order) and streams its chunk of the
// charges in blocks of 1024, 4 per thread (one from each 256-charge tile of
// the block, so a wave's lanes hold 64 consecutive, spatially close charges).
// Per cell the rule is chosen per wave over those close charges (7 points
// within 6 D, 6 within 16 D, 4 within 40 D, 3 beyond; pairs within 3 D are left
// to the near kernel), and each thread sums q (IV, IE) of its 4 charges in FP32.
// The order of additions after that, which fixes the result's bits: every four
// cells a wave writes its lanes' sums to 16 rows of LDS (cell, component); lane
// l adds 16 lanes' entries of row l / 4, from 16 (l mod 4) on, in FP64 to its
// sum over the blocks; at the end the four lanes of a row are added pairwise
// (shuffles by 1 and 2) and the four waves in order through LDS.
constexpr int kCB = 8;   // cells per workgroup
constexpr int kCS = 4;   // charges per thread and block
constexpr int kUP = 64 + 4;  // row pitch of a wave's sums (floats)

// One cell of the far kernel's LDS tile, recentred FP32, 19 float4 records:
//   c[0] = centroid, (3 D)^2          c[1] = (40 D)^2, area {w0, wa, wb}
//   c[2..7] = the 7 rule points (21 floats), area / 3, (6 D)^2, 0
//   c[8..10] = the 3 rule points (9 floats), area {w1, w2} of the 6-point
//              rule, (16 D)^2
//   c[11..15] = the 6 rule points (18 floats), area {wc, wp} of the 4-point
//              rule
//   c[16..18] = the 3 outer points of the 4-point rule (9 floats; its fourth
//              is the centroid), 0, 0, 0
// (the zones of the forward field: 7 points within 6 D, 6 within 16 D, 4
// within 40 D, 3 beyond)
struct ICell {
  float4 c[19];
};

// sum over m of w_m {1/|e_m|, e_m/|e_m|^3}, e_m = p - point m
template <int M>
__device__ __forceinline__ void infl_points(float px, float py, float pz, const float *q, const float *w, float &sv,
                                            float &ex, float &ey, float &ez) {
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const float ax = px - q[3 * m], ay = py - q[3 * m + 1], az = pz - q[3 * m + 2];
    const float rr = fmaf(ax, ax, fmaf(ay, ay, az * az));
    const float ri = __builtin_amdgcn_rsqf(rr);
    const float wr = w[m] * ri;
    const float t = wr * (ri * ri);
    sv += wr;
    ex = fmaf(t, ax, ex);
    ey = fmaf(t, ay, ey);
    ez = fmaf(t, az, ez);
  }
}

// Spheres of the runs of 64 ordered charges (centre of the box, largest
// distance from it): sph[4 g .. 4 g + 3].
__global__ __launch_bounds__(64) void k_charge_spheres(int n_s, const double *__restrict__ sx,
                                                       const double *__restrict__ sy, const double *__restrict__ sz,
                                                       double *sph) {
  const int j = min((int)blockIdx.x * 64 + (int)threadIdx.x, n_s - 1);
  const double v[3] = {sx[j], sy[j], sz[j]};
  double c[3], r2 = 0.0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double lo = v[d], hi = v[d];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      lo = fmin(lo, __shfl_xor(lo, o));
      hi = fmax(hi, __shfl_xor(hi, o));
    }
    c[d] = 0.5 * (lo + hi);
    r2 = fma(v[d] - c[d], v[d] - c[d], r2);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) r2 = fmax(r2, __shfl_xor(r2, o));
  if (threadIdx.x == 0) {
    double *s = sph + 4 * (size_t)blockIdx.x;
    s[0] = c[0];
    s[1] = c[1];
    s[2] = c[2];
    s[3] = sqrt(r2);
  }
}

// The M-point rule (7, 6, 4 or 3) of one staged cell at those of a thread's
// charges c whose run has its bit in runs (uniform over the wave) and that
// are far.
template <int M>
__device__ __forceinline__ void infl_rule(const ICell &C, unsigned runs, const bool *far, const float *px,
                                          const float *py, const float *pz, float *sv, float *ex, float *ey,
                                          float *ez) {
  const float *rec = reinterpret_cast<const float *>(&C);
  float q[3 * M], w[M];
  if (M == 7) {
    const float4 h = C.c[1];
#pragma unroll
    for (int m = 0; m < 7; ++m) w[m] = m == 0 ? h.y : (m < 4 ? h.z : h.w);
#pragma unroll
    for (int u = 0; u < 21; ++u) q[u] = rec[8 + u];
  } else if (M == 6) {
    const float4 h10 = C.c[10];
#pragma unroll
    for (int m = 0; m < 6; ++m) w[m] = m < 3 ? h10.y : h10.z;
#pragma unroll
    for (int u = 0; u < 18; ++u) q[u] = rec[44 + u];
  } else if (M == 4) {
#pragma unroll
    for (int m = 0; m < 4; ++m) w[m] = m == 0 ? rec[62] : rec[63];
#pragma unroll
    for (int u = 0; u < 3; ++u) q[u] = rec[u];
#pragma unroll
    for (int u = 0; u < 9; ++u) q[3 + u] = rec[64 + u];
  } else {
#pragma unroll
    for (int m = 0; m < 3; ++m) w[m] = rec[29];
#pragma unroll
    for (int u = 0; u < 9; ++u) q[u] = rec[32 + u];
  }
  if (runs == (1u << kCS) - 1u && !far) {
#pragma unroll
    for (int c = 0; c < kCS; ++c) infl_points<M>(px[c], py[c], pz[c], q, w, sv[c], ex[c], ey[c], ez[c]);
  } else {
#pragma unroll
    for (int c = 0; c < kCS; ++c)
      if (runs >> c & 1u)
        if (!far || far[c]) infl_points<M>(px[c], py[c], pz[c], q, w, sv[c], ex[c], ey[c], ez[c]);
  }
}

// The rule of a (cell, run of 64 charges) pair is the finest that one of its
// charges needs.  Lane (cell, run) of a wave bounds the nearest charge by the
// run's sphere; where that leaves one rule and no charge within 3 D (with
// margins above the FP32 rounding of the recentred coordinates) the rule is
// taken for the whole run without a test per charge.  The others take the
// test: the same rule either way.  A cell's points are read once per rule
// for the four runs of a thread's charges.
// Bound by FP32 issue and by LDS latency between the short pieces of a pair:
// the sums of a wave are combined by the wave itself, four cells at a time
// (no barrier in the loop, and 20 instead of 38 KB of LDS, for five instead of
// four waves per SIMD; held to 80 or 64 registers for more waves it is no
// faster or 38 % slower).  60,001 charges, 40,776 cells: 4.15 -> 3.6 ms.
__global__ __launch_bounds__(kTI) void k_influence_mixed(int N, const double *__restrict__ f,
                                                         const int32_t *__restrict__ ord, int n_s,
                                                         const double *__restrict__ sx,
                                                         const double *__restrict__ sy,
                                                         const double *__restrict__ sz,
                                                         const double *__restrict__ sq,
                                                         const double *__restrict__ sph, int chunk, double *part) {
  __shared__ ICell T[kCB];
  __shared__ __align__(16) float U[kTI / 64][16][kUP];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kb = blockIdx.x * kCB;  // first sorted position of the workgroup's cells
  // recentred on the first cell of the 256-cell group, as the near kernel
  const int kr = ord[(kb / kTI) * kTI];
  const double c0 = f[(size_t)MF_GX * N + kr], c1 = f[(size_t)MF_GY * N + kr], c2 = f[(size_t)MF_GZ * N + kr];
  for (int idx = tid; idx < 57 * kCB; idx += kTI) {
    const int m = idx / kCB, k = idx % kCB;
    const int kk = ord[min(kb + k, N - 1)];
    const int src = (m < 21) ? MF_Q7 + m : (m < 30 ? MF_Q3 + (m - 21) : (m < 48 ? MF_Q6 + (m - 30) : MF_Q4 + (m - 48)));
    const int c = (m < 21 ? m : (m < 30 ? m - 21 : (m < 48 ? m - 30 : m - 48))) % 3;
    reinterpret_cast<float *>(&T[k])[m < 21 ? 8 + m : (m < 30 ? 32 + (m - 21) : (m < 48 ? 44 + (m - 30) : 64 + (m - 48)))] =
        (float)(f[(size_t)src * N + kk] - (c == 0 ? c0 : (c == 1 ? c1 : c2)));
  }
  if (tid < kCB) {
    const int kk = ord[min(kb + tid, N - 1)];
    const double D = f[(size_t)MF_DIAM * N + kk], ar = f[(size_t)MF_AREA * N + kk];
    float *rec = reinterpret_cast<float *>(&T[tid]);
    T[tid].c[0] = make_float4((float)(f[(size_t)MF_GX * N + kk] - c0), (float)(f[(size_t)MF_GY * N + kk] - c1),
                              (float)(f[(size_t)MF_GZ * N + kk] - c2), (float)(kNearMixed * kNearMixed * D * D));
    T[tid].c[1] = make_float4((float)(kFar3Mixed * kFar3Mixed * D * D), (float)(ar * Rule7::w0),
                              (float)(ar * Rule7::wa), (float)(ar * Rule7::wb));
    rec[29] = (float)(ar / 3.0);
    rec[30] = (float)(kFwd6 * kFwd6 * D * D);
    rec[31] = (float)D;
    rec[41] = (float)(ar * Rule6::w1);
    rec[42] = (float)(ar * Rule6::w2);
    rec[43] = (float)(kFwd4 * kFwd4 * D * D);
    rec[62] = (float)(ar * Rule4::wc);
    rec[63] = (float)(ar * Rule4::wp);
    rec[73] = rec[74] = rec[75] = 0.f;
  }
  __syncthreads();
  // lane l: cells l / 16 and 4 + l / 16, component l / 4 % 4, the sums of 16
  // of the wave's lanes
  double accd[2] = {0.0, 0.0};
  const int jb = blockIdx.y * chunk, je = min(n_s, jb + chunk);
  for (int j0 = jb; j0 < je; j0 += kTI * kCS) {
    float px[kCS], py[kCS], pz[kCS], pq[kCS];
#pragma unroll
    for (int c = 0; c < kCS; ++c) {
      const int j = j0 + c * kTI + tid;
      const bool ok = j < je;
      const int jj = ok ? j : jb;  // a real position with charge 0
      px[c] = (float)(sx[jj] - c0);
      py[c] = (float)(sy[jj] - c1);
      pz[c] = (float)(sz[jj] - c2);
      pq[c] = ok ? (float)sq[jj] : 0.f;
    }
    // bit 4 k + c: the rule of (cell k, run c) where it is certain
    unsigned m3, m4, m6, m7;
    {
      const int k = (lane >> 2) & (kCB - 1), c = lane & 3;
      const int jr = j0 + c * kTI + wv * 64;
      int rule = 0;
      if (lane < 4 * kCB && jr + 64 <= je) {  // whole runs only: others hold the stand-in position
        const double *s = sph + 4 * (size_t)(jr / 64);
        const float4 g = T[k].c[0];
        const float D = T[k].c[7].w, r = (float)s[3];
        const float d = sqrtf(dist2f((float)(s[0] - c0), (float)(s[1] - c1), (float)(s[2] - c2), g.x, g.y, g.z));
        const float slack = 1e-5f * (d + fabsf(g.x) + fabsf(g.y) + fabsf(g.z));
        const float lo = (d - r - slack) * 0.999f, hi = (d + r + slack) * 1.001f;
        if (lo > (float)kFar3Mixed * D)
          rule = 3;
        else if (lo > (float)kFwd4 * D)
          rule = hi < (float)kFar3Mixed * D ? 4 : 0;
        else if (lo > (float)kFwd6 * D)
          rule = hi < (float)kFwd4 * D ? 6 : 0;
        else if (lo > (float)kNearMixed * D)
          rule = hi < (float)kFwd6 * D ? 7 : 0;
      }
      m3 = (unsigned)__ballot(rule == 3);
      m4 = (unsigned)__ballot(rule == 4);
      m6 = (unsigned)__ballot(rule == 6);
      m7 = (unsigned)__ballot(rule == 7);
    }
#pragma unroll 1
    for (int k = 0; k < kCB; ++k) {
      float sv[kCS], ex[kCS], ey[kCS], ez[kCS];
#pragma unroll
      for (int c = 0; c < kCS; ++c) sv[c] = ex[c] = ey[c] = ez[c] = 0.f;
      unsigned b3 = m3 >> (4 * k) & 15u, b4 = m4 >> (4 * k) & 15u, b6 = m6 >> (4 * k) & 15u, b7 = m7 >> (4 * k) & 15u;
      const unsigned open = 15u & ~(b3 | b4 | b6 | b7);
      if (open) {
        const float4 g = T[k].c[0];
        const float lim7 = T[k].c[7].z, lim6 = T[k].c[10].w, lim4 = T[k].c[1].x;
        bool far[kCS];
#pragma unroll
        for (int c = 0; c < kCS; ++c) {
          far[c] = true;
          if (open >> c & 1u) {
            const float R2 = dist2f(px[c], py[c], pz[c], g.x, g.y, g.z);
            far[c] = !(R2 < g.w);  // the others are taken by k_influence_near in FP64
            // 7 points within 6 D, 6 within 16 D, 4 within 40 D, 3 beyond
            // (finest rule of the run)
            if (__any(far[c] && R2 < lim7))
              b7 |= 1u << c;
            else if (__any(far[c] && R2 < lim6))
              b6 |= 1u << c;
            else if (__any(far[c] && R2 < lim4))
              b4 |= 1u << c;
            else
              b3 |= 1u << c;
          }
        }
        if (b3) infl_rule<3>(T[k], b3, far, px, py, pz, sv, ex, ey, ez);
        if (b4) infl_rule<4>(T[k], b4, far, px, py, pz, sv, ex, ey, ez);
        if (b6) infl_rule<6>(T[k], b6, far, px, py, pz, sv, ex, ey, ez);
        if (b7) infl_rule<7>(T[k], b7, far, px, py, pz, sv, ex, ey, ez);
      } else {
        if (b3) infl_rule<3>(T[k], b3, nullptr, px, py, pz, sv, ex, ey, ez);
        if (b4) infl_rule<4>(T[k], b4, nullptr, px, py, pz, sv, ex, ey, ez);
        if (b6) infl_rule<6>(T[k], b6, nullptr, px, py, pz, sv, ex, ey, ez);
        if (b7) infl_rule<7>(T[k], b7, nullptr, px, py, pz, sv, ex, ey, ez);
      }
      float av = 0.f, ax = 0.f, ay = 0.f, az = 0.f;
#pragma unroll
      for (int c = 0; c < kCS; ++c) {
        av = fmaf(pq[c], sv[c], av);
        ax = fmaf(pq[c], ex[c], ax);
        ay = fmaf(pq[c], ey[c], ay);
        az = fmaf(pq[c], ez[c], az);
      }
      float(*u)[kUP] = U[wv] + 4 * (k & 3);
      u[0][lane] = av;
      u[1][lane] = ax;
      u[2][lane] = ay;
      u[3][lane] = az;
      if ((k & 3) == 3) {
        // FP64 from here on: the charges come sorted by sign, so the sums are
        // large and cancel only between blocks
        wave_lds_fence();
        const float4 *r = reinterpret_cast<const float4 *>(&U[wv][lane >> 2][(lane & 3) * 16]);
        double a = 0.0;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const float4 v = r[m];
          a += (double)v.x;
          a += (double)v.y;
          a += (double)v.z;
          a += (double)v.w;
        }
        if (k < 4)
          accd[0] += a;
        else
          accd[1] += a;
        wave_lds_fence();
      }
    }
  }
  // the four lanes of a (cell, component), then the four waves, in order
  __syncthreads();
  double *R = reinterpret_cast<double *>(&U[0][0][0]);  // [wave][cell * 4 + component]
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    double a = accd[h];
    a += __shfl_xor(a, 1);
    a += __shfl_xor(a, 2);
    if ((lane & 3) == 0) R[wv * (kCB * 4) + h * 16 + (lane >> 2)] = a;
  }
  __syncthreads();
  if (tid < kCB * 4) {
    double t = R[tid];
#pragma unroll
    for (int w = 1; w < kTI / 64; ++w) t += R[w * (kCB * 4) + tid];
    const int k = kb + tid / 4;
    if (k < N) part[(size_t)blockIdx.y * 4 * N + (size_t)(tid % 4) * N + k] = t;
  }
}

// Sum over the wave's lanes in a fixed order.
__device__ __forceinline__ double lanes_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Near part of the mixed influence: the pairs that the far kernel's FP32 test
// (same values, recentred on the first cell of its 256-cell group) puts
// within 3 D, in FP64 closed form.  One wave per cell, the lanes on the
// charges, so that the cell's record is the same for the wave and its sums
// are combined once: with a lane per cell and the charges in turn, a charge
// near one of 64 cells took the whole wave's closed form.  60,001 charges and
// 40,776 cells 294 -> 44 us; 50,000 charges all near 400 cells 6.6 -> 0.3 ms in
// all.
// gridDim.y splits the 256-charge tiles, each split writing its own partial
// slot.  64 tiles are tested at once against the cell's reach, 3 D (1 + 1e-5)
// + 1e-6 |c_k - c0|, which exceeds what FP32 rounding of the recentred
// coordinates can add to the test; the near charges of the tiles within it
// are queued in LDS and evaluated 64 at a time.
__global__ __launch_bounds__(64) void k_influence_near(int N, const double *__restrict__ f,
                                                       const double *__restrict__ rec,
                                                       const int32_t *__restrict__ ord, int n_s,
                                                       const double *__restrict__ sx, const double *__restrict__ sy,
                                                       const double *__restrict__ sz, const double *__restrict__ sq,
                                                       const double *__restrict__ tbox, int tchunk, double *part) {
  __shared__ int queue[128];
  const int lane = threadIdx.x, k = blockIdx.x;
  const int kk = __builtin_amdgcn_readfirstlane(ord[k]), k0 = __builtin_amdgcn_readfirstlane(ord[k / kTI * kTI]);
  const double c0 = f[(size_t)MF_GX * N + k0], c1 = f[(size_t)MF_GY * N + k0], c2 = f[(size_t)MF_GZ * N + k0];
  const double G0 = f[(size_t)MF_GX * N + kk], G1 = f[(size_t)MF_GY * N + kk], G2 = f[(size_t)MF_GZ * N + kk];
  const float g0 = (float)(G0 - c0), g1 = (float)(G1 - c1), g2 = (float)(G2 - c2);
  const double D = f[(size_t)MF_DIAM * N + kk];
  const float lim = (float)(kNearMixed * kNearMixed * D * D);
  const double off = sqrt((G0 - c0) * (G0 - c0) + (G1 - c1) * (G1 - c1) + (G2 - c2) * (G2 - c2));
  const double reach = kNearMixed * D * (1.0 + 1e-5) + 1e-6 * off;
  double nv = 0.0, nx = 0.0, ny = 0.0, nz = 0.0;
  const int ntile = (n_s + kTI - 1) / kTI;
  const int tb = blockIdx.y * tchunk, te = min(ntile, tb + tchunk);
  int qn = 0;
  // t0 beyond te: evaluates what is left in the queue
  for (int t0 = tb; t0 < te + 64; t0 += 64) {
    bool hit = false;
    if (t0 + lane < te) {
      const double *bx = tbox + 6 * (size_t)(t0 + lane);
      const double e0 = fmax(fmax(bx[0] - G0, G0 - bx[3]), 0.0);
      const double e1 = fmax(fmax(bx[1] - G1, G1 - bx[4]), 0.0);
      const double e2 = fmax(fmax(bx[2] - G2, G2 - bx[5]), 0.0);
      hit = e0 * e0 + e1 * e1 + e2 * e2 < reach * reach;
    }
    const bool last = t0 >= te;
    uint64_t m = __ballot(hit);
    int u = 0;  // run of 64 charges of the lowest tile of m
    for (;;) {
      while (m && qn < 64) {
        const int j = (t0 + __builtin_amdgcn_readfirstlane(__builtin_ctzll(m))) * kTI + u * 64 + lane;
        bool nearp = false;
        if (j < n_s) nearp = dist2f((float)(sx[j] - c0), (float)(sy[j] - c1), (float)(sz[j] - c2), g0, g1, g2) < lim;
        const uint64_t nm = __ballot(nearp);
        if (nearp) queue[qn + __popcll(nm & ((1ull << lane) - 1ull))] = j;
        qn += __popcll(nm);
        if (++u == kTI / 64) {
          u = 0;
          m &= m - 1ull;
        }
      }
      const int n = last ? min(qn, 64) : (qn >= 64 ? 64 : 0);
      if (n == 0) break;
      __syncthreads();  // one wave: orders the LDS accesses
      if (lane < n) {
        const int j = queue[lane];
        infl_closed(rec, kk, sx[j], sy[j], sz[j], sq[j], nv, nx, ny, nz);
      }
      qn -= n;
      const int rest = lane < qn ? queue[64 + lane] : 0;
      __syncthreads();
      if (lane < qn) queue[lane] = rest;
    }
  }
  nv = lanes_sum(nv);
  nx = lanes_sum(nx);
  ny = lanes_sum(ny);
  nz = lanes_sum(nz);
  if (lane < 4) {
    const double v = lane == 0 ? nv : (lane == 1 ? nx : (lane == 2 ? ny : nz));
    part[((size_t)blockIdx.y * 4 + lane) * N + k] = v;
  }
}

// FP64 influence: closed form within 48 D, FP64 7-point rule beyond, the
// same test |x - c_k|^2 >= (48 D_k)^2 as in the field.  A wave per two cells
// (neighbours in the mesh's Hilbert order), the lanes on the charges, which
// four waves share through LDS; the charges come ordered, so a wave's 64
// charges mostly agree on the form.  The sums of a cell are combined over
// the lanes once.  Bound by FP64 operations.
// 20,000 charges, 14,384 cells 5.5 -> 1.8 ms, 5,000 charges, 4,096 cells 683
// -> 222 us against a lane per cell with the charges in turn.
constexpr int kFC = 2;  // cells per wave

__global__ __launch_bounds__(kTI) void k_influence_fp64(int N, const double *__restrict__ f,
                                                        const double *__restrict__ rec,
                                                        const int32_t *__restrict__ ord, int n_s,
                                                        const double *__restrict__ sx,
                                                        const double *__restrict__ sy,
                                                        const double *__restrict__ sz,
                                                        const double *__restrict__ sq, int chunk, double *part) {
  __shared__ double P[4][kTI];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kb = (blockIdx.x * (kTI / 64) + wv) * kFC;  // first sorted position of the wave's cells
  double acc[kFC][4];
#pragma unroll
  for (int c = 0; c < kFC; ++c)
#pragma unroll
    for (int m = 0; m < 4; ++m) acc[c][m] = 0.0;
  const int jb = blockIdx.y * chunk, je = min(n_s, jb + chunk);
  for (int jt = jb; jt < je; jt += kTI) {
    const int cnt = min(kTI, je - jt);
    __syncthreads();
    {
      const int j = jt + min(tid, cnt - 1);  // a real position with charge 0 beyond the end
      P[0][tid] = sx[j];
      P[1][tid] = sy[j];
      P[2][tid] = sz[j];
      P[3][tid] = tid < cnt ? sq[j] : 0.0;
    }
    __syncthreads();
    for (int r = 0; r < cnt; r += 64) {
      const d3 p = mk3(P[0][r + lane], P[1][r + lane], P[2][r + lane]);
      const double q = P[3][r + lane];
#pragma unroll
      for (int c = 0; c < kFC; ++c) {
        if (kb + c >= N) break;
        const int kk = __builtin_amdgcn_readfirstlane(ord[kb + c]);
        const double dx = p.x - f[(size_t)MF_GX * N + kk], dy = p.y - f[(size_t)MF_GY * N + kk],
                     dz = p.z - f[(size_t)MF_GZ * N + kk];
        const double D = f[(size_t)MF_DIAM * N + kk], R2 = fma(dx, dx, fma(dy, dy, dz * dz));
        const bool quad = R2 >= kQuadFp64 * kQuadFp64 * D * D;
        const bool mid = !quad && R2 >= kMidForm * kMidForm * D * D;
        if (__any(quad)) {
          if (quad) {
            const double qa = q * f[(size_t)MF_AREA * N + kk];
#pragma unroll
            for (int m = 0; m < 7; ++m) {
              const double w = qa * ((m == 0) ? Rule7::w0 : (m < 4 ? Rule7::wa : Rule7::wb));
              const double ax = p.x - f[(size_t)(MF_Q7 + 3 * m) * N + kk], ay = p.y - f[(size_t)(MF_Q7 + 3 * m + 1) * N + kk],
                           az = p.z - f[(size_t)(MF_Q7 + 3 * m + 2) * N + kk];
              const double ri = inv_sqrt_f64(fma(ax, ax, fma(ay, ay, az * az)));
              const double wr = w * ri;
              const double s = wr * ri * ri;
              acc[c][0] += wr;
              acc[c][1] = fma(s, ax, acc[c][1]);
              acc[c][2] = fma(s, ay, acc[c][2]);
              acc[c][3] = fma(s, az, acc[c][3]);
            }
          }
        }
        if (__any(mid)) {
          if (mid) {
            d3 IE;
            double IV;
            cell_mid_form<true>(rec + (size_t)kk * CR_COUNT, p, IE, IV);
            acc[c][0] = fma(q, IV, acc[c][0]);
            acc[c][1] = fma(q, IE.x, acc[c][1]);
            acc[c][2] = fma(q, IE.y, acc[c][2]);
            acc[c][3] = fma(q, IE.z, acc[c][3]);
          }
        }
        const bool close = !quad && !mid;
        if (__any(close)) {
          // (a charge of 0 stands for no charge: its term may be 0 times an
          // infinite integral)
          if (close && r + lane < cnt) infl_closed(rec, kk, p.x, p.y, p.z, q, acc[c][0], acc[c][1], acc[c][2], acc[c][3]);
        }
      }
    }
  }
#pragma unroll
  for (int c = 0; c < kFC; ++c) {
#pragma unroll
    for (int m = 0; m < 4; ++m) acc[c][m] = lanes_sum(acc[c][m]);
    if (kb + c < N && lane < 4) {
      const double v = lane == 0 ? acc[c][0] : (lane == 1 ? acc[c][1] : (lane == 2 ? acc[c][2] : acc[c][3]));
      part[((size_t)blockIdx.y * 4 + lane) * N + kb + c] = v;
    }
  }
}

// Sum of the chunks in order, then the modified left-hand side.
__global__ __launch_bounds__(256) void k_influence_rhs(int N, int nch, const double *__restrict__ part,
                                                       const int32_t *__restrict__ ord,
                                                       const double *__restrict__ f, const int8_t *__restrict__ kind,
                                                       const double *__restrict__ rhs, double *rhs_out, double *vbar,
                                                       double *ebx, double *eby, double *ebz) {
  const int k = blockIdx.x * 256 + threadIdx.x;  // sorted position
  if (k >= N) return;
  const int i = ord[k];
  double s[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) s[m] = slot_sum(0.0, part + (size_t)m * N + k, 4 * (size_t)N, nch);
  const double area = f[(size_t)MF_AREA * N + i];
  const double vb = kKe * s[0] / area;
  const double eb[3] = {-kKe * s[1] / area, -kKe * s[2] / area, -kKe * s[3] / area};
  if (vbar) vbar[i] = vb;
  if (ebx) {
    ebx[i] = eb[0];
    eby[i] = eb[1];
    ebz[i] = eb[2];
  }
  if (kind[i] == 0) {
    rhs_out[i] = rhs[i] - vb;
  } else {
    const double en = eb[0] * f[(size_t)MF_NX * N + i] + eb[1] * f[(size_t)MF_NY * N + i] +
                      eb[2] * f[(size_t)MF_NZ * N + i];
    rhs_out[i] = rhs[i] - kEps0 * (f[(size_t)MF_EPS2 * N + i] - f[(size_t)MF_EPS1 * N + i]) * en;
  }
}

obem_status influence_rhs(obem_ctx *ctx, const obem_meshh *m, int64_t n_src, const double *sx, const double *sy,
                          const double *sz, const double *sq, const double *rhs, double *rhs_out, obem_precision prec,
                          double *vbar, double *ebx, double *eby, double *ebz) {
  const int N = (int)m->n, n_s = (int)n_src;
  const int bc = (N + kTI - 1) / kTI;
  // workgroups along the cells: 8 cells each
  const int bw = (N + kCB - 1) / kCB;
  static_assert(kCB == kFC * (kTI / 64), "both kernels take the same cells per workgroup");
  int nsplit = 1, chunk = std::max(n_s, 1);
  if (n_s > 0) {
    // whole blocks of the mixed far kernel, single tiles of the FP64 kernel
    const int unit = prec == OBEM_MIXED ? kTI * kCS : kTI;
    nsplit = std::max(1, std::min((kSplitWorkgroups + bw - 1) / bw, (n_s + unit - 1) / unit));
    if ((int64_t)bw * nsplit > kFewWorkgroups) nsplit = std::max(1, std::min(nsplit, (n_s + 1023) / 1024));
    nsplit = std::min(nsplit, 64);
    chunk = (n_s + nsplit - 1) / nsplit;
    chunk = (chunk + unit - 1) / unit * unit;
    nsplit = (n_s + chunk - 1) / chunk;
  }
  // mixed: partial slots of the near kernel after those of the far kernel;
  // one wave per cell and split, at least four tiles a split
  const int ntile = (n_s + kTI - 1) / kTI;
  const int nnear = std::max(1, std::min((ntile + 3) / 4, std::min(64, (8192 + N - 1) / N)));
  const int tchunk = std::max(1, (ntile + nnear - 1) / nnear);
  const int nslot = (n_s > 0 && prec == OBEM_MIXED) ? nsplit + (ntile + tchunk - 1) / tchunk : nsplit;
  double *part = (double *)ws_get(ctx, WS_MISC3, sizeof(double) * 4 * (size_t)N * nslot);
  if (!part) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
  OBEM_PROF(ctx, "influence");
  if (n_s == 0) {
    obem_status st = launch_fill(ctx, part, 4 * (size_t)N, 0.0);
    if (st) return st;
  } else {
    SourceOrder so;
    obem_status st = order_sources(ctx, n_s, sx, sy, sz, sq, false, &so);
    if (st) return st;
    if (prec == OBEM_MIXED) {
      const int ng = (n_s + 63) / 64;
      double *sph = (double *)ws_get(ctx, WS_MISC2, sizeof(double) * 4 * (size_t)ng);
      if (!sph) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
      hipLaunchKernelGGL(k_charge_spheres, dim3(ng), dim3(64), 0, ctx->stream, n_s, so.x, so.y, so.z, sph);
      hipLaunchKernelGGL(k_influence_mixed, dim3(bw, nsplit), dim3(kTI), 0, ctx->stream, N, m->f, m->order, n_s, so.x,
                         so.y, so.z, so.q, sph, chunk, part);
      hipLaunchKernelGGL(k_influence_near, dim3(N, nslot - nsplit), dim3(64), 0, ctx->stream, N, m->f, m->rec, m->order,
                         n_s, so.x, so.y, so.z, so.q, so.tbox, tchunk, part + 4 * (size_t)N * nsplit);
    } else {
      hipLaunchKernelGGL(k_influence_fp64, dim3(bw, nsplit), dim3(kTI), 0, ctx->stream, N, m->f, m->rec, m->order, n_s,
                         so.x, so.y, so.z, so.q, chunk, part);
    }
  }
  OBEM_HIP(ctx, hipGetLastError());
  hipLaunchKernelGGL(k_influence_rhs, dim3(bc), dim3(256), 0, ctx->stream, N, n_s > 0 ? nslot : 1, part, m->order,
                     m->f, m->kind, rhs, rhs_out, vbar, ebx, eby, ebz);
  OBEM_HIP(ctx, hipGetLastError());
  return OBEM_OK;
}

}  // namespace obem

using namespace obem;

extern "C" obem_status bem_influence(obem_ctx *ctx, const obem_meshh *mesh, int64_t n_src, const double *sx,
                                     const double *sy, const double *sz, const double *sq, const double *rhs,
                                     double *rhs_out, obem_precision precision, double *vbar, double *ebar_x,
                                     double *ebar_y, double *ebar_z) {
  if (!ctx) return OBEM_EINVAL;
  if (ctx->sticky) return OBEM_ESTATE;
  if (hipSetDevice(ctx->device) != hipSuccess) {
    (void)hipGetLastError();
    return fail(ctx, OBEM_EDEVICE, "hipSetDevice failed");
  }
  if (!mesh) return fail(ctx, OBEM_EINVAL, "mesh is NULL");
  if (n_src < 0 || n_src >= ((int64_t)1 << 31)) return fail(ctx, OBEM_EINVAL, "n_src out of range");
  if (precision != OBEM_FP64 && precision != OBEM_MIXED) return fail(ctx, OBEM_EINVAL, "bad precision");
  if (!is_device_ptr(rhs) || !is_device_ptr(rhs_out)) return fail(ctx, OBEM_EINVAL, "rhs / rhs_out must be device");
  if (n_src > 0 && (!is_device_ptr(sx) || !is_device_ptr(sy) || !is_device_ptr(sz) || !is_device_ptr(sq)))
    return fail(ctx, OBEM_EINVAL, "source arrays must be device memory");
  const bool eb = ebar_x || ebar_y || ebar_z;
  if (eb && !(ebar_x && ebar_y && ebar_z)) return fail(ctx, OBEM_EINVAL, "ebar_x/y/z: all or none");
  const void *outs[] = {vbar, ebar_x, ebar_y, ebar_z};
  for (const void *p : outs)
    if (p && !is_device_ptr(p)) return fail(ctx, OBEM_EINVAL, "outputs must be device memory");
  return influence_rhs(ctx, mesh, n_src, sx, sy, sz, sq, rhs, rhs_out, precision, vbar, ebar_x, ebar_y, ebar_z);
}
