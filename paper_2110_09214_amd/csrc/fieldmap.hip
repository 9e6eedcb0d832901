// Static field option (section 3.3.1): the cell field computed once on a
// uniform 3D grid and interpolated (trilinearly) at the particles; and the
// Shockley-Ramo current of eq. (ramo), whose weighting field comes either
// from the cells (dynamic option) or from such a map (static option).
#include <algorithm>
#include <cmath>

#include "obem_internal.hpp"

namespace obem {

// Points from which on the map is packed (map_pack), if they are also an
// eighth of the nodes or more.  With 304,448 nodes: 131,072 points 14 us as
// they are and 18 us packed, 262,144 25 and 25, 1,000,000 91 and 62, 2,000,000
// 176 and 108; with 978,912 nodes 262,144 points 49 and 33 us.
constexpr int64_t kPackPoints = 1 << 18;

// Node coordinates of the grid, SoA (x, y, z), index (k*ny + j)*nx + i.
__global__ __launch_bounds__(256) void k_grid_nodes(MapDev g, double *xs) {
  const int64_t M = (int64_t)g.nx * g.ny * g.nz;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= M) return;
  const int i = (int)(t % g.nx), j = (int)((t / g.nx) % g.ny), k = (int)(t / ((int64_t)g.nx * g.ny));
  // lo + h*i rounded twice (no contraction), so a node's coordinates do not
  // depend on the compiler's choice of fused multiply-add
  xs[t] = __dadd_rn(g.lo[0], __dmul_rn(g.h[0], (double)i));
  xs[M + t] = __dadd_rn(g.lo[1], __dmul_rn(g.h[1], (double)j));
  xs[2 * M + t] = __dadd_rn(g.lo[2], __dmul_rn(g.h[2], (double)k));
}

// The map's three arrays as one array of nodes.  A point's eight corners are
// then four runs of 48 bytes, 5 to 6 cache lines, instead of twelve runs of 16
// in as many lines; the reads of scattered points are bound by those lines.
__global__ __launch_bounds__(256) void k_map_pack(int64_t M, const double *__restrict__ ex,
                                                  const double *__restrict__ ey, const double *__restrict__ ez,
                                                  double *nodes) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= M) return;
  nodes[3 * t] = ex[t];
  nodes[3 * t + 1] = ey[t];
  nodes[3 * t + 2] = ez[t];
}

obem_status map_pack(obem_ctx *ctx, int64_t n, MapDev *g) {
  const int64_t M = (int64_t)g->nx * g->ny * g->nz;
  if (n < kPackPoints || n < M / 8) return OBEM_OK;
  // The plain map needs no workspace: a captured call takes it (it must not
  // allocate, and its graph may outlive the buffer), and so does a call that
  // cannot have the buffer.
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(ctx->stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) {
    (void)hipGetLastError();
    return OBEM_OK;
  }
  double *nodes = (double *)ws_get(ctx, WS_MAPNODES, sizeof(double) * 3 * (size_t)M);
  if (!nodes) return OBEM_OK;
  hipLaunchKernelGGL(k_map_pack, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, ctx->stream, M, g->ex, g->ey, g->ez,
                     nodes);
  OBEM_HIP(ctx, hipGetLastError());
  g->nodes = nodes;
  return OBEM_OK;
}

template <bool PACKED>
__global__ __launch_bounds__(256) void k_map_eval(MapDev g, int n, const double *__restrict__ x,
                                                  const double *__restrict__ y, const double *__restrict__ z,
                                                  double *Ex, double *Ey, double *Ez) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= n) return;
  double E[3];
  map_interp<PACKED>(g, x[t], y[t], z[t], E);
  Ex[t] = E[0];
  Ey[t] = E[1];
  Ez[t] = E[2];
}

// Per-particle q v . E_w and per-block sums by species (fixed-order tree).
// SRC 0: E_w from Ew (3 x n); 1 and 2: from the map (2: packed), without a
// trip of the field through memory.
template <int SRC>
__global__ __launch_bounds__(256) void k_ramo_terms(int n, const double *__restrict__ Ew, MapDev g,
                                                    const double *__restrict__ x, const double *__restrict__ y,
                                                    const double *__restrict__ z, const double *__restrict__ vx,
                                                    const double *__restrict__ vy, const double *__restrict__ vz,
                                                    const int8_t *__restrict__ sp, double *terms, double *part) {
  __shared__ double s[3][4];
  const int t = blockIdx.x * 256 + threadIdx.x;
  double c[3] = {0.0, 0.0, 0.0};
  if (t < n) {
    const int8_t k = sp[t];
    const double q = (k == 1) ? kQe : -kQe;
    double E[3];
    if (SRC == 0) {
      E[0] = Ew[t];
      E[1] = Ew[(size_t)n + t];
      E[2] = Ew[2 * (size_t)n + t];
    } else {
      map_interp<SRC == 2>(g, x[t], y[t], z[t], E);
    }
    const double term = q * (vx[t] * E[0] + vy[t] * E[1] + vz[t] * E[2]);
    if (terms) terms[t] = term;
    if (k >= 0 && k <= 2) c[k] = term;
  }
#pragma unroll
  for (int m = 0; m < 3; ++m) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c[m] += __shfl_xor(c[m], o);
    if ((threadIdx.x & 63) == 0) s[m][threadIdx.x >> 6] = c[m];
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const double *r = s[threadIdx.x];
    part[3 * (size_t)blockIdx.x + threadIdx.x] = ((r[0] + r[1]) + r[2]) + r[3];
  }
}

// Sum of the block sums in a fixed order (one workgroup per species; thread t
// takes blocks t, t + 256, ..., four loads in flight).
__global__ __launch_bounds__(256) void k_ramo_final(int nb, const double *__restrict__ part, double *out) {
  const int m = blockIdx.x;
  double acc = 0.0;
#pragma unroll 4
  for (int b = threadIdx.x; b < nb; b += 256) acc += part[3 * (size_t)b + m];
  __shared__ double s[4];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) out[m] = ((s[0] + s[1]) + s[2]) + s[3];
}

bool map_dev(const obem_field_map *m, MapDev *g) {
  if (!m || m->nx < 2 || m->ny < 2 || m->nz < 2) return false;
  if ((int64_t)m->nx * m->ny * m->nz >= kMaxCount) return false;
  for (int c = 0; c < 3; ++c)
    if (!(m->h[c] > 0.0) || !std::isfinite(m->h[c]) || !std::isfinite(m->lo[c])) return false;
  if (!is_device_ptr(m->ex) || !is_device_ptr(m->ey) || !is_device_ptr(m->ez)) return false;
  g->nx = m->nx;
  g->ny = m->ny;
  g->nz = m->nz;
  for (int c = 0; c < 3; ++c) {
    g->lo[c] = m->lo[c];
    g->h[c] = m->h[c];
  }
  g->ex = m->ex;
  g->ey = m->ey;
  g->ez = m->ez;
  g->nodes = nullptr;
  return true;
}

template <bool PACKED>
__global__ __launch_bounds__(256) void k_map_acc(MapDev g, int n, const double *__restrict__ xs, double *acc) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= n) return;
  double E[3];
  map_interp<PACKED>(g, xs[t], xs[(size_t)n + t], xs[2 * (size_t)n + t], E);
  acc[t] = E[0] / kKe;
  acc[(size_t)n + t] = E[1] / kKe;
  acc[2 * (size_t)n + t] = E[2] / kKe;
  acc[3 * (size_t)n + t] = 0.0;
}

obem_status launch_map_acc(obem_ctx *ctx, const MapDev &map, const TargetOrder &to, double *acc) {
  if (to.n == 0) return OBEM_OK;
  OBEM_PROF(ctx, "map");
  MapDev g = map;
  const obem_status st = map_pack(ctx, to.n, &g);
  if (st) return st;
  const dim3 grid((unsigned)((to.n + 255) / 256));
  if (g.nodes)
    hipLaunchKernelGGL(k_map_acc<true>, grid, dim3(256), 0, ctx->stream, g, to.n, to.xs, acc);
  else
    hipLaunchKernelGGL(k_map_acc<false>, grid, dim3(256), 0, ctx->stream, g, to.n, to.xs, acc);
  OBEM_HIP(ctx, hipGetLastError());
  return OBEM_OK;
}

}  // namespace obem

using namespace obem;

extern "C" {

obem_status field_map_build(obem_ctx *ctx, const obem_meshh *mesh, const double *sigma, const obem_field_map *map,
                            obem_precision precision) {
  CHECK_CTX(ctx);
  if (!mesh) return fail(ctx, OBEM_EINVAL, "mesh is NULL");
  REQ_DEV(ctx, sigma, "sigma");
  if (precision != OBEM_FP64 && precision != OBEM_MIXED) return fail(ctx, OBEM_EINVAL, "bad precision");
  MapDev g;
  if (!map_dev(map, &g)) return fail(ctx, OBEM_EINVAL, "bad field map (sizes >= 2, spacing > 0, device arrays)");
  const int64_t M = (int64_t)g.nx * g.ny * g.nz;
  double *xs = (double *)ws_get(ctx, WS_MAP, sizeof(double) * 3 * (size_t)M);
  double *acc = (double *)ws_get(ctx, WS_ACC, sizeof(double) * 4 * (size_t)M);
  if (!xs || !acc) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
  hipLaunchKernelGGL(k_grid_nodes, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, ctx->stream, g, xs);
  OBEM_HIP(ctx, hipGetLastError());
  TargetOrder to;
  obem_status st = order_targets(ctx, M, xs, xs + M, xs + 2 * M, &to);
  if (st) return st;
  Slots cells;
  st = launch_panel_field(ctx, mesh, sigma, to, precision, false, acc, &cells);
  if (st) return st;
  return launch_finish(ctx, to, cells, Slots{}, kKe, map->ex, map->ey, map->ez, nullptr);
}

obem_status field_map_eval(obem_ctx *ctx, const obem_field_map *map, int64_t n, const double *x, const double *y,
                           const double *z, double *Ex, double *Ey, double *Ez) {
  CHECK_CTX(ctx);
  MapDev g;
  if (!map_dev(map, &g)) return fail(ctx, OBEM_EINVAL, "bad field map (sizes >= 2, spacing > 0, device arrays)");
  if (n < 0 || n >= kMaxCount) return fail(ctx, OBEM_EINVAL, "n out of range");
  if (n == 0) return OBEM_OK;
  REQ_DEV(ctx, x, "x");
  REQ_DEV(ctx, y, "y");
  REQ_DEV(ctx, z, "z");
  REQ_DEV(ctx, Ex, "Ex");
  REQ_DEV(ctx, Ey, "Ey");
  REQ_DEV(ctx, Ez, "Ez");
  const obem_status st = map_pack(ctx, n, &g);
  if (st) return st;
  const dim3 grid((unsigned)((n + 255) / 256));
  if (g.nodes)
    hipLaunchKernelGGL(k_map_eval<true>, grid, dim3(256), 0, ctx->stream, g, (int)n, x, y, z, Ex, Ey, Ez);
  else
    hipLaunchKernelGGL(k_map_eval<false>, grid, dim3(256), 0, ctx->stream, g, (int)n, x, y, z, Ex, Ey, Ez);
  OBEM_HIP(ctx, hipGetLastError());
  return OBEM_OK;
}

obem_status induced_current(obem_ctx *ctx, const obem_meshh *mesh, const double *sigma_w, const obem_field_map *map,
                            int64_t n, const double *x, const double *y, const double *z, const double *vx,
                            const double *vy, const double *vz, const int8_t *species, obem_precision precision,
                            double *current, double *terms) {
  CHECK_CTX(ctx);
  if (n < 0 || n >= kMaxCount) return fail(ctx, OBEM_EINVAL, "n out of range");
  if ((map != nullptr) == (mesh != nullptr))
    return fail(ctx, OBEM_EINVAL, "give either mesh + sigma_w or a weighting-field map");
  MapDev g;
  if (map && !map_dev(map, &g)) return fail(ctx, OBEM_EINVAL, "bad field map");
  if (mesh) REQ_DEV(ctx, sigma_w, "sigma_w");
  if (precision != OBEM_FP64 && precision != OBEM_MIXED) return fail(ctx, OBEM_EINVAL, "bad precision");
  OPT_DEV(ctx, terms, "terms");
  if (n == 0) {
    if (current) current[0] = current[1] = current[2] = 0.0;
    return OBEM_OK;
  }
  const void *req[] = {x, y, z, vx, vy, vz, species};
  for (const void *p : req)
    if (!is_device_ptr(p)) return fail(ctx, OBEM_EINVAL, "particle arrays must be device memory");
  const int nb = (int)((n + 255) / 256);
  double *part = (double *)ws_get(ctx, WS_MISC1, sizeof(double) * (3 * (size_t)nb + 3));
  if (!part) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
#define RAMO(SRC, EW)                                                                                             \
  hipLaunchKernelGGL(k_ramo_terms<SRC>, dim3(nb), dim3(256), 0, ctx->stream, (int)n, EW, g, x, y, z, vx, vy, vz, \
                     species, terms, part)
  if (map) {
    const obem_status st = map_pack(ctx, n, &g);
    if (st) return st;
    if (g.nodes)
      RAMO(2, nullptr);
    else
      RAMO(1, nullptr);
  } else {
    double *Ew = (double *)ws_get(ctx, WS_MISC0, sizeof(double) * 3 * (size_t)n);
    double *acc = (double *)ws_get(ctx, WS_ACC, sizeof(double) * 4 * (size_t)n);
    if (!Ew || !acc) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
    TargetOrder to;
    obem_status st = order_targets(ctx, n, x, y, z, &to);
    if (st) return st;
    Slots cells;
    st = launch_panel_field(ctx, mesh, sigma_w, to, precision, false, acc, &cells);
    if (st) return st;
    st = launch_finish(ctx, to, cells, Slots{}, kKe, Ew, Ew + n, Ew + 2 * n, nullptr);
    if (st) return st;
    g = MapDev{};
    RAMO(0, Ew);
  }
#undef RAMO
  hipLaunchKernelGGL(k_ramo_final, dim3(3), dim3(256), 0, ctx->stream, nb, part, part + 3 * (size_t)nb);
  OBEM_HIP(ctx, hipGetLastError());
  if (current) {
    OBEM_HIP(ctx, hipMemcpyAsync(current, part + 3 * (size_t)nb, 3 * sizeof(double), hipMemcpyDeviceToHost,
                                 ctx->stream));
    OBEM_HIP(ctx, hipStreamSynchronize(ctx->stream));
  }
  return OBEM_OK;
}

}  // extern "C"
