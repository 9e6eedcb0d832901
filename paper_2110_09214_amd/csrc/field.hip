// Field evaluation kernels for gfx950: target ordering, cell (panel) field,
// pairwise point-charge field, fixed-order reduction and scatter.
//
// Layout: targets are reordered along a Hilbert curve so that the 256 targets
// of a workgroup are spatially compact; each workgroup recentres its targets
// and the staged source/cell data on its first target (FP64 difference, then
// FP32), which keeps FP32 differences relative to the pair distance instead
// of the absolute coordinates.  Sums are accumulated per tile in registers and
// carried across tiles with a compensated (Neumaier) FP32 sum in the mixed
// mode, plainly in FP64 in the FP64 mode.  No floating-point atomics: every
// reduction has a fixed order.
#include <hipcub/hipcub.hpp>

#include <type_traits>

#include "cellmath.hpp"
#include "obem_internal.hpp"
#include "paironce.hpp"

namespace obem {

constexpr int kThreads = 256;

// ---------------------------------------------------------------------------
// Target ordering
// ---------------------------------------------------------------------------
// Minimum (or maximum) over the wave's 64 lanes, valid in lane 63: within
// quads, eights and rows of 16, then rows 0 to 1 and 2 to 3, then 1 to 3.
template <bool MAX>
__device__ __forceinline__ double wave_extreme(double v) {
  auto op = [](double a, double b) { return MAX ? fmax(a, b) : fmin(a, b); };
  v = op(v, dpp_f64<0xB1, 0xf>(v, v));   // quad_perm 1 0 3 2
  v = op(v, dpp_f64<0x4E, 0xf>(v, v));   // quad_perm 2 3 0 1
  v = op(v, dpp_f64<0x141, 0xf>(v, v));  // row_half_mirror
  v = op(v, dpp_f64<0x140, 0xf>(v, v));  // row_mirror
  v = op(v, dpp_f64<0x142, 0xa>(v, v));  // row_bcast:15 into rows 1 and 3
  return op(v, dpp_f64<0x143, 0xc>(v, v));  // row_bcast:31 into rows 2 and 3
}

// Combines the waves' boxes b (lo xyz, hi xyz) of a workgroup of T threads;
// every thread gets the whole one.  red: 6 T / 64 doubles of LDS.
template <int T>
__device__ __forceinline__ void block_box(double b[6], double *red) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    b[c] = wave_extreme<false>(b[c]);
    b[3 + c] = wave_extreme<true>(b[3 + c]);
  }
  if ((threadIdx.x & 63) == 63)
#pragma unroll
    for (int c = 0; c < 6; ++c) red[6 * (threadIdx.x >> 6) + c] = b[c];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 6; ++c) b[c] = red[c];
#pragma unroll 4
  for (int w = 1; w < T / 64; ++w)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      b[c] = fmin(b[c], red[6 * w + c]);
      b[3 + c] = fmax(b[3 + c], red[6 * w + 3 + c]);
    }
}

__global__ __launch_bounds__(256) void k_bbox_partial(int n, const double *__restrict__ x,
                                                      const double *__restrict__ y,
                                                      const double *__restrict__ z, double *part) {
  __shared__ double red[24];
  double b[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const double v[3] = {x[i], y[i], z[i]};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      b[c] = fmin(b[c], v[c]);
      b[3 + c] = fmax(b[3 + c], v[c]);
    }
  }
  block_box<256>(b, red);
  if (threadIdx.x == 0)
#pragma unroll
    for (int c = 0; c < 6; ++c) part[blockIdx.x * 6 + c] = b[c];
}

__device__ __forceinline__ uint32_t spread3(uint32_t v) {
  v &= 0x3ffu;
  v = (v | (v << 16)) & 0x030000FFu;
  v = (v | (v << 8)) & 0x0300F00Fu;
  v = (v | (v << 4)) & 0x030C30C3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

// Index along the Hilbert curve of a cell (x0, x1, x2) of the 1024^3 grid,
// after J. Skilling's transpose form (AIP Conf. Proc. 707 (2004) 381): undo
// the excess work level by level, Gray-encode, then interleave the bits with
// x0 most significant.  Consecutive indices are neighbouring cells, so runs of
// consecutive points have tighter boxes than along the Morton curve (which
// jumps): at 4M cloud charges half as many 256-point tile pairs are near
// each other.
__device__ __forceinline__ uint32_t hilbert3(uint32_t x0, uint32_t x1, uint32_t x2) {
  uint32_t X[3] = {x0, x1, x2};
  for (uint32_t Q = 1u << 9; Q > 1u; Q >>= 1) {
    const uint32_t P = Q - 1u;
    if (X[0] & Q) X[0] ^= P;
#pragma unroll
    for (int i = 1; i < 3; ++i) {
      if (X[i] & Q) {
        X[0] ^= P;
      } else {
        const uint32_t t = (X[0] ^ X[i]) & P;
        X[0] ^= t;
        X[i] ^= t;
      }
    }
  }
  X[1] ^= X[0];
  X[2] ^= X[1];
  uint32_t t = 0u;
  for (uint32_t Q = 1u << 9; Q > 1u; Q >>= 1)
    if (X[2] & Q) t ^= Q - 1u;
  X[0] ^= t;
  X[1] ^= t;
  X[2] ^= t;
  return spread3(X[2]) | (spread3(X[1]) << 1) | (spread3(X[0]) << 2);
}

// Sorting key of point i: its class (species, or sign of the charge: -, +,
// other; 0 without either) above the 30 bits of its place along the curve in
// the box lo .. hi.  Points in (class, curve, caller) order are then one
// stable sort.
__device__ __forceinline__ uint32_t order_key(const OrderJob &J, int i, const double lo[3], const double hi[3]) {
  const double v[3] = {J.x[i], J.y[i], J.z[i]};
  uint32_t q[3];
  // one scale for the three axes, so that runs along the curve are compact
  // in space also in a flat or elongated point set
  const double span = fmax(fmax(hi[0] - lo[0], hi[1] - lo[1]), hi[2] - lo[2]);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    double t = span > 0.0 ? (v[c] - lo[c]) / span : 0.0;
    int qi = (int)(t * 1024.0);
    q[c] = (uint32_t)min(max(qi, 0), 1023);
  }
  uint32_t cls = 0;
  if (J.species)
    cls = (uint32_t)(J.species[i] & 3);
  else if (J.q)
    cls = J.q[i] < 0.0 ? 0u : (J.q[i] > 0.0 ? 1u : 2u);
  return (cls << 30) | hilbert3(q[0], q[1], q[2]);
}

// Keys of a large set; every workgroup reduces the nb partial boxes itself.
__global__ __launch_bounds__(256) void k_order_key(OrderJob J, int nb, const double *__restrict__ part, uint32_t *keys,
                                                   int32_t *idx) {
  __shared__ double red[24];
  double b[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  for (int k = threadIdx.x; k < nb; k += 256)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      b[c] = fmin(b[c], part[6 * k + c]);
      b[3 + c] = fmax(b[3 + c], part[6 * k + 3 + c]);
    }
  block_box<256>(b, red);
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= J.n) return;
  keys[i] = order_key(J, i, b, b + 3);
  idx[i] = i;
}

static inline int nblk(int64_t n, int t = 256) { return (int)((n + t - 1) / t); }

// Element i of the ordered copies: the point's coordinates (and charge), the
// inverse permutation.
__device__ __forceinline__ void order_gather(const OrderJob &J, int i, int j, double v[3]) {
  const size_t n = (size_t)J.n;
  v[0] = J.x[j];
  v[1] = J.y[j];
  v[2] = J.z[j];
  if (J.xs) {
    J.xs[i] = v[0];
    J.xs[n + i] = v[1];
    J.xs[2 * n + i] = v[2];
    if (J.q) J.xs[3 * n + i] = J.q[j];
  }
  if (J.inv) J.inv[j] = i;
}

// Box (lo xyz, hi xyz) of a 256-point tile held by four consecutive waves
// (thread tt of the tile); red: 24 doubles of LDS per tile.
__device__ __forceinline__ void tile_box(const double v[3], bool ok, int tt, double *red, double *box) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double lo = wave_extreme<false>(ok ? v[c] : INFINITY), hi = wave_extreme<true>(ok ? v[c] : -INFINITY);
    if ((tt & 63) == 63) {
      red[6 * (tt >> 6) + c] = lo;
      red[6 * (tt >> 6) + 3 + c] = hi;
    }
  }
  __syncthreads();
  if (tt < 6 && box) {
    double r = red[tt];
    for (int w = 1; w < 4; ++w) r = tt < 3 ? fmin(r, red[6 * w + tt]) : fmax(r, red[6 * w + tt]);
    box[tt] = r;
  }
}

struct OrderPair {
  OrderJob job[2];
};

// The copies of one or two orderings (gridDim.y) from their permutations.
__global__ __launch_bounds__(256) void k_order_gather(OrderPair jobs) {
  __shared__ double red[24];
  const OrderJob &J = jobs.job[blockIdx.y];
  if ((int)blockIdx.x * 256 >= J.n) return;  // workgroup-uniform
  const int i = blockIdx.x * 256 + threadIdx.x;
  double v[3] = {0.0, 0.0, 0.0};
  if (i < J.n) order_gather(J, i, J.perm[i], v);
  if (J.tbox) tile_box(v, i < J.n, threadIdx.x, red, J.tbox + 6 * (size_t)blockIdx.x);
}

// Bounding box of each 256-source tile of the source copy (lo xyz, hi xyz).
__global__ __launch_bounds__(256) void k_tile_boxes(int n, const double *__restrict__ src, double *box) {
  __shared__ double red[24];
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int k = min(i, n - 1);
  const double v[3] = {src[k], src[(size_t)n + k], src[2 * (size_t)n + k]};
  tile_box(v, true, threadIdx.x, red, box + 6 * (size_t)blockIdx.x);
}

void launch_tile_boxes(obem_ctx *ctx, int n, const double *src, double *box) {
  if (n > 0) hipLaunchKernelGGL(k_tile_boxes, dim3(nblk(n)), dim3(256), 0, ctx->stream, n, src, box);
}

// Up to 256 points, one workgroup a set and two of them side by side: box,
// keys, stable radix sort in LDS and copies in one launch instead of five to
// ten, each of which costs its latency (64 points 65 -> 6 us).
constexpr int kTinyOrder = 256;

__global__ __launch_bounds__(kTinyOrder) void k_order_tiny(OrderPair jobs) {
  using Sort = hipcub::BlockRadixSort<uint32_t, kTinyOrder, 1, int32_t>;
  __shared__ typename Sort::TempStorage tmp;
  __shared__ double red[6 * (kTinyOrder / 64)];
  const OrderJob &J = jobs.job[blockIdx.x];
  const int n = J.n, t = threadIdx.x;
  double box[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  if (t < n) {
    box[0] = box[3] = J.x[t];
    box[1] = box[4] = J.y[t];
    box[2] = box[5] = J.z[t];
  }
  block_box<kTinyOrder>(box, red);
  // padding keys sort behind every point (equal keys keep their order)
  uint32_t key[1] = {t < n ? order_key(J, t, box, box + 3) : 0xffffffffu};
  int32_t idx[1] = {t};
  Sort(tmp).Sort(key, idx, 0, (J.q || J.species) ? 32 : 30);
  double v[3] = {0.0, 0.0, 0.0};
  if (t < n) {
    J.perm[t] = idx[0];
    order_gather(J, t, idx[0], v);
  }
  __syncthreads();  // red is consumed
  if (J.tbox) tile_box(v, t < n, t, red, J.tbox);
}

// Small sets: a point's place is the number of keys before its own, counted
// against all of them.  n^2 comparisons are less than the passes of a sort
// while a launch of 16 points a workgroup does not fill the chip: every
// workgroup holds all keys, four a thread, and counts by ballots.
// Every workgroup of the keys' launch reduces the whole box itself.  A call
// with 4,096 charges in place of one workgroup's radix sort in LDS 212 -> 198
// us, against the launches of order_large with 4,097 charges 128 -> 111, with
// 8,000 130 -> 115, but with 16,000 134 -> 147 us.
constexpr int kSmallOrder = 8192;
constexpr int kRankPoints = 16;

__global__ __launch_bounds__(1024) void k_order_key_small(OrderPair jobs, uint32_t *k0, uint32_t *k1) {
  __shared__ double red[6 * 16];
  const OrderJob &J = jobs.job[blockIdx.y];
  const int n = J.n, t = threadIdx.x;
  if ((int)blockIdx.x * 1024 >= n) return;  // workgroup-uniform
  double box[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll 4
  for (int i = t; i < n; i += 1024) {
    const double v[3] = {J.x[i], J.y[i], J.z[i]};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      box[c] = fmin(box[c], v[c]);
      box[3 + c] = fmax(box[3 + c], v[c]);
    }
  }
  block_box<1024>(box, red);
  const int i = blockIdx.x * 1024 + t;
  if (i < n) (blockIdx.y ? k1 : k0)[i] = order_key(J, i, box, box + 3);
}

__global__ __launch_bounds__(1024) void k_order_rank(OrderPair jobs, const uint32_t *__restrict__ k0,
                                                     const uint32_t *__restrict__ k1) {
  __shared__ int cnt[16][kRankPoints];
  const OrderJob &J = jobs.job[blockIdx.y];
  const uint32_t *__restrict__ keys = blockIdx.y ? k1 : k0;
  const int n = J.n, t = threadIdx.x, first = blockIdx.x * kRankPoints;
  if (first >= n) return;  // workgroup-uniform
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  uint32_t own[kRankPoints];
  int c[kRankPoints];
#pragma unroll
  for (int p = 0; p < kRankPoints; ++p) {
    own[p] = keys[min(first + p, n - 1)];
    c[p] = 0;
  }
  for (int base = 0; base < n; base += 4096) {
    uint32_t k[4];
    const int j0 = base + 4 * t, w0 = base + 256 * wave;
#pragma unroll
    for (int u = 0; u < 4; ++u) k[u] = j0 + u < n ? keys[j0 + u] : 0xffffffffu;
    // equal keys keep their order: those of a wave's 256 points are all
    // before, all behind or around the workgroup's points
    auto count = [&](auto before) {
#pragma unroll
      for (int p = 0; p < kRankPoints; ++p)
#pragma unroll
        for (int u = 0; u < 4; ++u) c[p] += __popcll(__ballot(before(k[u], own[p], j0 + u < first + p)));
    };
    if (w0 + 256 <= first)
      count([](uint32_t a, uint32_t b, bool) { return a <= b; });
    else if (w0 > first)
      count([](uint32_t a, uint32_t b, bool) { return a < b; });
    else
      count([](uint32_t a, uint32_t b, bool l) { return a < b || (a == b && l); });
  }
  if ((t & 63) == 0)
#pragma unroll
    for (int p = 0; p < kRankPoints; ++p) cnt[wave][p] = c[p];
  __syncthreads();
  if (t < kRankPoints && first + t < n) {
    int r = 0;
    for (int w = 0; w < 16; ++w) r += cnt[w][t];
    J.perm[r] = first + t;
  }
}

// A large set: partial boxes, keys, one radix sort, copies.
static obem_status order_large(obem_ctx *ctx, const OrderJob &J) {
  const int n = J.n;
  const int nb = std::min(256, nblk(n, 1024));
  double *part = (double *)ws_get(ctx, WS_BBOX, sizeof(double) * 6 * nb);
  uint32_t *k0 = (uint32_t *)ws_get(ctx, WS_KEYS0, sizeof(uint32_t) * n);
  uint32_t *k1 = (uint32_t *)ws_get(ctx, WS_KEYS1, sizeof(uint32_t) * n);
  int32_t *i0 = (int32_t *)ws_get(ctx, WS_IDX0, sizeof(int32_t) * n);
  if (!part || !k0 || !k1 || !i0) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
  hipLaunchKernelGGL(k_bbox_partial, dim3(nb), dim3(256), 0, ctx->stream, n, J.x, J.y, J.z, part);
  hipLaunchKernelGGL(k_order_key, dim3(nblk(n)), dim3(256), 0, ctx->stream, J, nb, part, k0, i0);
  const int bits = (J.q || J.species) ? 32 : 30;
  size_t tmp_bytes = 0;
  OBEM_HIP(ctx, hipcub::DeviceRadixSort::SortPairs(nullptr, tmp_bytes, k0, k1, i0, J.perm, n, 0, bits, ctx->stream));
  void *tmp = ws_get(ctx, WS_SORT_TMP, tmp_bytes + 256);
  if (!tmp) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
  OBEM_HIP(ctx, hipcub::DeviceRadixSort::SortPairs(tmp, tmp_bytes, k0, k1, i0, J.perm, n, 0, bits, ctx->stream));
  if (J.xs || J.inv || J.tbox) {
    OrderPair one;
    one.job[0] = J;
    hipLaunchKernelGGL(k_order_gather, dim3(nblk(n), 1), dim3(256), 0, ctx->stream, one);
  }
  OBEM_HIP(ctx, hipGetLastError());
  return OBEM_OK;
}

obem_status order_points(obem_ctx *ctx, const OrderJob &a, const OrderJob &b) {
  OBEM_PROF(ctx, "order");
  OrderPair small;
  int ns = 0;
  for (const OrderJob *J : {&a, &b}) {
    if (J->n == 0) continue;
    if (J->n <= kSmallOrder) {
      small.job[ns++] = *J;
    } else {
      const obem_status st = order_large(ctx, *J);
      if (st) return st;
    }
  }
  if (ns) {
    const int m = std::max(small.job[0].n, small.job[1].n);
    if (m <= kTinyOrder) {
      hipLaunchKernelGGL(k_order_tiny, dim3(ns), dim3(kTinyOrder), 0, ctx->stream, small);
    } else {
      uint32_t *k0 = (uint32_t *)ws_get(ctx, WS_KEYS0, sizeof(uint32_t) * small.job[0].n);
      uint32_t *k1 = ns > 1 ? (uint32_t *)ws_get(ctx, WS_KEYS1, sizeof(uint32_t) * small.job[1].n) : nullptr;
      if (!k0 || (ns > 1 && !k1)) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
      hipLaunchKernelGGL(k_order_key_small, dim3(nblk(m, 1024), ns), dim3(1024), 0, ctx->stream, small, k0, k1);
      hipLaunchKernelGGL(k_order_rank, dim3(nblk(m, kRankPoints), ns), dim3(1024), 0, ctx->stream, small, k0, k1);
      hipLaunchKernelGGL(k_order_gather, dim3(nblk(m), ns), dim3(256), 0, ctx->stream, small);
    }
    OBEM_HIP(ctx, hipGetLastError());
  }
  return OBEM_OK;
}

// The jobs of a source copy and of a target order (workspace of ctx).
static obem_status source_job(obem_ctx *ctx, int n, const double *sx, const double *sy, const double *sz,
                              const double *sq, bool want_inv, OrderJob *J, SourceOrder *out) {
  const size_t nz = (size_t)n;
  out->n = n;
  if (n == 0) return OBEM_OK;
  int32_t *perm = (int32_t *)ws_get(ctx, WS_SRCPERM, sizeof(int32_t) * nz);
  double *src = (double *)ws_get(ctx, WS_SRC, sizeof(double) * 4 * nz + nz + 64);
  double *tbox = (double *)ws_get(ctx, WS_TBOX, sizeof(double) * 6 * (size_t)nblk(n));
  int32_t *inv = want_inv ? (int32_t *)ws_get(ctx, WS_SRCINV, sizeof(int32_t) * nz) : nullptr;
  if (!perm || !src || !tbox || (want_inv && !inv)) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
  J->n = n;
  J->x = sx;
  J->y = sy;
  J->z = sz;
  J->q = sq;
  J->perm = perm;
  J->xs = src;
  J->inv = inv;
  J->tbox = tbox;
  out->x = src;
  out->y = src + nz;
  out->z = src + 2 * nz;
  out->q = src + 3 * nz;
  out->tbox = tbox;
  out->inv = inv;
  out->perm = perm;
  return OBEM_OK;
}

static obem_status target_job(obem_ctx *ctx, int n, const double *tx, const double *ty, const double *tz, OrderJob *J,
                              TargetOrder *out) {
  out->n = n;
  if (n == 0) return OBEM_OK;
  int32_t *perm = (int32_t *)ws_get(ctx, WS_IDX1, sizeof(int32_t) * n);
  double *xs = (double *)ws_get(ctx, WS_TSORT, sizeof(double) * 3 * (size_t)n);
  if (!perm || !xs) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
  J->n = n;
  J->x = tx;
  J->y = ty;
  J->z = tz;
  J->perm = perm;
  J->xs = xs;
  out->perm = perm;
  out->xs = xs;
  return OBEM_OK;
}

obem_status order_sources(obem_ctx *ctx, int64_t n, const double *sx, const double *sy, const double *sz,
                          const double *sq, bool want_inv, SourceOrder *out) {
  OrderJob J;
  const obem_status st = source_job(ctx, (int)n, sx, sy, sz, sq, want_inv, &J, out);
  return st ? st : order_points(ctx, J, OrderJob{});
}

obem_status order_targets(obem_ctx *ctx, int64_t n, const double *tx, const double *ty, const double *tz,
                          TargetOrder *out) {
  OrderJob J;
  const obem_status st = target_job(ctx, (int)n, tx, ty, tz, &J, out);
  return st ? st : order_points(ctx, J, OrderJob{});
}

obem_status order_both(obem_ctx *ctx, int64_t n_src, const double *sx, const double *sy, const double *sz,
                       const double *sq, bool want_inv, SourceOrder *so, int64_t n_tgt, const double *tx,
                       const double *ty, const double *tz, TargetOrder *to) {
  OrderJob a, b;
  obem_status st = source_job(ctx, (int)n_src, sx, sy, sz, sq, want_inv, &a, so);
  if (!st) st = target_job(ctx, (int)n_tgt, tx, ty, tz, &b, to);
  return st ? st : order_points(ctx, a, b);
}

// ---------------------------------------------------------------------------
// Cell (panel) field
// ---------------------------------------------------------------------------
constexpr int kPT = 64;               // cells per LDS tile

// One cell of an LDS tile, recentred FP32, as 19 float4 records read whole
// (one address per cell, 128-bit LDS reads):
//   c[0] = centroid, (3 D)^2          c[1] = (40 D)^2, area sigma {w0, wa, wb}
//   c[2..7] = the 7 points of the degree-5 rule (21 floats), area sigma / 3,
//             (6 D)^2, D
//   c[8..10] = the 3 points of the degree-2 rule (9 floats), area sigma
//             {w1, w2} of the 6-point rule, (16 D)^2
//   c[11..15] = the 6 points of the degree-4 rule (18 floats), area sigma
//             {wc, wp} of the 4-point rule
//   c[16..18] = the 3 outer points of the degree-3 rule (9 floats; its
//             fourth point is the centroid), 0, 0, 0
struct PanelCell {
  float4 c[19];
};

// sum over the M rule points of w {e/|e|^3, 1/|e|}, e = target - point
template <int M, bool WANT_V>
__device__ __forceinline__ void panel_points(const float *q, const float *w, float r0, float r1, float r2,
                                             float &px, float &py, float &pz, float &pv) {
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const float ex = r0 - q[3 * m], ey = r1 - q[3 * m + 1], ez = r2 - q[3 * m + 2];
    const float rr = fmaf(ex, ex, fmaf(ey, ey, ez * ez));
    const float ri = __builtin_amdgcn_rsqf(rr);
    const float wr = w[m] * ri;
    const float s_ = wr * (ri * ri);
    px = fmaf(s_, ex, px);
    py = fmaf(s_, ey, py);
    pz = fmaf(s_, ez, pz);
    if (WANT_V) pv += wr;
  }
}

// n consecutive float4 records of a cell into registers
template <int N4>
__device__ __forceinline__ void load4(const float4 *c, float *q) {
#pragma unroll
  for (int u = 0; u < N4; ++u) {
    const float4 t = c[u];
    q[4 * u] = t.x;
    q[4 * u + 1] = t.y;
    q[4 * u + 2] = t.z;
    q[4 * u + 3] = t.w;
  }
}

__device__ __forceinline__ void neumaier(float &s, float &c, float v) {
  float t = s + v;
  if (fabsf(s) >= fabsf(v))
    c += (s - t) + v;
  else
    c += (v - t) + s;
  s = t;
}

// Target tile bx and split by of the cells into ranges of cchunk; split y writes
// its sums to part + 4 n_t y (part = acc when there is one split).
template <bool WANT_V>
__device__ __forceinline__ void panel_mixed(int bx, int by, int n_t, const double *__restrict__ xs, int N,
                                            const double *__restrict__ f, const double *__restrict__ sigma,
                                            int cchunk, double *part) {
  __shared__ PanelCell T[kPT];
  const int tid = threadIdx.x;
  const int i0 = bx * kThreads;
  const int i = i0 + tid;
  const bool active = i < n_t;
  const double c0 = xs[i0], c1 = xs[(size_t)n_t + i0], c2 = xs[2 * (size_t)n_t + i0];
  const double x0 = active ? xs[i] : c0;
  const double x1 = active ? xs[(size_t)n_t + i] : c1;
  const double x2 = active ? xs[2 * (size_t)n_t + i] : c2;
  const float r0 = (float)(x0 - c0), r1 = (float)(x1 - c1), r2 = (float)(x2 - c2);
  // the wave's sphere: centre of its targets' bounding box, radius the
  // largest distance from it (widened by 1e-4 for the rounding)
  float cw0, cw1, cw2, rw;
  {
    float lo0 = r0, lo1 = r1, lo2 = r2, hi0 = r0, hi1 = r1, hi2 = r2;
    for (int o = 32; o > 0; o >>= 1) {
      lo0 = fminf(lo0, __shfl_xor(lo0, o));
      lo1 = fminf(lo1, __shfl_xor(lo1, o));
      lo2 = fminf(lo2, __shfl_xor(lo2, o));
      hi0 = fmaxf(hi0, __shfl_xor(hi0, o));
      hi1 = fmaxf(hi1, __shfl_xor(hi1, o));
      hi2 = fmaxf(hi2, __shfl_xor(hi2, o));
    }
    cw0 = 0.5f * (lo0 + hi0);
    cw1 = 0.5f * (lo1 + hi1);
    cw2 = 0.5f * (lo2 + hi2);
    rw = sqrtf(dist2f(r0, r1, r2, cw0, cw1, cw2));
    for (int o = 32; o > 0; o >>= 1) rw = fmaxf(rw, __shfl_xor(rw, o));
    rw *= 1.0001f;
  }
  float hx = 0.f, hy = 0.f, hz = 0.f, hv = 0.f, lx = 0.f, ly = 0.f, lz = 0.f, lv = 0.f;
  const int kb = by * cchunk, ke = min(N, kb + cchunk);
  for (int k0 = kb; k0 < ke; k0 += kPT) {
    const int cnt = min(kPT, ke - k0);
    __syncthreads();
    // staging, coalesced along the cells: the 57 rule coordinates (7-, 3-, 6-
    // and 4-point rules, arrays MF_Q7 + m) of the 64 cells, wave w taking
    // rows m = w, w + 4, ... with lane k on cell k; a row's array, record
    // slot and coordinate are the same for the whole wave, and the wave's
    // loads are all issued before the first is used.  Then one thread per
    // cell for centroid, limits and weights.
    {
      const int k = tid & 63;
      const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
      const bool ok = k < cnt;
      const double *fk = f + (size_t)MF_Q7 * N + k0 + k;
      float *rec = reinterpret_cast<float *>(&T[k]);
      double v[15];
#pragma unroll
      for (int j = 0; j < 15; ++j) {
        const int m = w + 4 * j;
        v[j] = (m < 57 && ok) ? fk[(size_t)m * N] : 0.0;
      }
#pragma unroll
      for (int j = 0; j < 15; ++j) {
        const int m = w + 4 * j;
        if (m < 57) {
          const int c = m % 3;
          const double o = c == 0 ? c0 : (c == 1 ? c1 : c2);
          rec[m + (m < 21 ? 8 : (m < 30 ? 11 : (m < 48 ? 14 : 16)))] = ok ? (float)(v[j] - o) : 0.f;
        }
      }
    }
    if (tid < kPT) {
      const int k = tid;
      float4 g = make_float4(0.f, 0.f, 0.f, 0.f), h = g;
      float w3 = 0.f, lim7 = 0.f, lim6 = 0.f, w61 = 0.f, w62 = 0.f, w4c = 0.f, w4p = 0.f, dk = 0.f;
      if (k < cnt) {
        const int kk = k0 + k;
        const double D = f[(size_t)MF_DIAM * N + kk];
        const double as = f[(size_t)MF_AREA * N + kk] * sigma[kk];
        g = make_float4((float)(f[(size_t)MF_GX * N + kk] - c0), (float)(f[(size_t)MF_GY * N + kk] - c1),
                        (float)(f[(size_t)MF_GZ * N + kk] - c2), (float)(kNearMixed * kNearMixed * D * D));
        h = make_float4((float)(kFar3Mixed * kFar3Mixed * D * D), (float)(as * Rule7::w0), (float)(as * Rule7::wa),
                        (float)(as * Rule7::wb));
        w3 = (float)(as * (1.0 / 3.0));
        lim7 = (float)(kFwd6 * kFwd6 * D * D);
        lim6 = (float)(kFwd4 * kFwd4 * D * D);
        dk = (float)D;
        w61 = (float)(as * Rule6::w1);
        w62 = (float)(as * Rule6::w2);
        w4c = (float)(as * Rule4::wc);
        w4p = (float)(as * Rule4::wp);
      }
      float *rec = reinterpret_cast<float *>(&T[k]);
      T[k].c[0] = g;
      T[k].c[1] = h;
      rec[29] = w3;
      rec[30] = lim7;
      rec[31] = dk;
      rec[41] = w61;
      rec[42] = w62;
      rec[43] = lim6;
      rec[62] = w4c;
      rec[63] = w4p;
      rec[73] = rec[74] = rec[75] = 0.f;
    }
    __syncthreads();
    float px = 0.f, py = 0.f, pz = 0.f, pv = 0.f;
    // The rule of each cell for the whole wave, from one test per cell
    // against the wave's sphere: lane k tests cell k, and the ballots give
    // the cells some lane may see within 40 D (4 points or finer), 16 D (6
    // or finer), 6 D (7 points) and 3 D (the per-lane path, which leaves the
    // near pairs to k_panel_close).  Thresholds 1 % wide of the per-lane
    // ones, so that a cell not flagged near has no lane inside 3 D by the
    // per-lane test, and a coarser rule is never taken where a lane needs a
    // finer one.
    uint64_t m3, m4, m6, m7, mnear;
    {
      const int k = tid & 63;
      float t = 3.0e38f, Dk = 0.f;
      if (k < cnt) {
        const float4 g = T[k].c[0];
        Dk = T[k].c[7].w;
        t = sqrtf(dist2f(cw0, cw1, cw2, g.x, g.y, g.z)) - rw;
      }
      const uint64_t f4 = __ballot(t < (float)(kFar3Mixed * 1.01) * Dk);
      const uint64_t f6 = __ballot(t < (float)(kFwd4 * 1.01) * Dk);
      const uint64_t f7 = __ballot(t < (float)(kFwd6 * 1.01) * Dk);
      mnear = __ballot(t < (float)(kNearMixed * 1.01) * Dk);
      m3 = (cnt == 64 ? ~0ull : ((1ull << cnt) - 1ull)) & ~f4;
      m4 = f4 & ~f6;
      m6 = f6 & ~f7;
      m7 = f7 & ~mnear;
    }
    for (; m3; m3 &= m3 - 1ull) {
      const int k = __builtin_ctzll(m3);
      float q[12];
      load4<3>(&T[k].c[8], q);
      const float w3 = T[k].c[7].y;
      const float w[3] = {w3, w3, w3};
      panel_points<3, WANT_V>(q, w, r0, r1, r2, px, py, pz, pv);
    }
    for (; m4; m4 &= m4 - 1ull) {
      const int k = __builtin_ctzll(m4);
      float q[15];
      const float4 g = T[k].c[0];
      q[0] = g.x;
      q[1] = g.y;
      q[2] = g.z;
      load4<3>(&T[k].c[16], q + 3);
      const float4 h15 = T[k].c[15];
      const float w[4] = {h15.z, h15.w, h15.w, h15.w};
      panel_points<4, WANT_V>(q, w, r0, r1, r2, px, py, pz, pv);
    }
    for (; m6; m6 &= m6 - 1ull) {
      const int k = __builtin_ctzll(m6);
      float q[20];
      load4<5>(&T[k].c[11], q);
      const float4 h10 = T[k].c[10];
      const float w[6] = {h10.y, h10.y, h10.y, h10.z, h10.z, h10.z};
      panel_points<6, WANT_V>(q, w, r0, r1, r2, px, py, pz, pv);
    }
    for (; m7; m7 &= m7 - 1ull) {
      const int k = __builtin_ctzll(m7);
      float q[24];
      load4<6>(&T[k].c[2], q);
      const float4 h = T[k].c[1];
      const float w[7] = {h.y, h.z, h.z, h.z, h.w, h.w, h.w};
      panel_points<7, WANT_V>(q, w, r0, r1, r2, px, py, pz, pv);
    }
    for (; mnear; mnear &= mnear - 1ull) {
      const int k = __builtin_ctzll(mnear);
      const float4 g = T[k].c[0];
      const float R2 = dist2f(r0, r1, r2, g.x, g.y, g.z);
      const bool nearp = R2 < g.w;  // taken by k_panel_close in FP64
      const float4 h = T[k].c[1];
      const float4 h7 = T[k].c[7];    // {.., area sigma / 3, (6 D)^2, D}
      const float4 h10 = T[k].c[10];  // {.., w1, w2, (16 D)^2}
      // the rule by distance (7 points within 6 D, 6 within 16 D, 4 within
      // 40 D, 3 beyond), taken for the whole wave at the finest rule one of
      // its lanes needs
      const bool need7 = (!nearp) && (R2 < h7.z);
      const bool need6 = (!nearp) && (R2 < h10.w);
      const bool need4 = (!nearp) && (R2 < h.x);
      if (__any(need7)) {
        if (!nearp) {
          float q[24];
          load4<6>(&T[k].c[2], q);
          const float w[7] = {h.y, h.z, h.z, h.z, h.w, h.w, h.w};
          panel_points<7, WANT_V>(q, w, r0, r1, r2, px, py, pz, pv);
        }
      } else if (__any(need6)) {
        if (!nearp) {
          float q[20];
          load4<5>(&T[k].c[11], q);
          const float w[6] = {h10.y, h10.y, h10.y, h10.z, h10.z, h10.z};
          panel_points<6, WANT_V>(q, w, r0, r1, r2, px, py, pz, pv);
        }
      } else if (__any(need4)) {
        if (!nearp) {
          float q[15];
          q[0] = g.x;
          q[1] = g.y;
          q[2] = g.z;
          load4<3>(&T[k].c[16], q + 3);
          const float4 h15 = T[k].c[15];
          const float w[4] = {h15.z, h15.w, h15.w, h15.w};
          panel_points<4, WANT_V>(q, w, r0, r1, r2, px, py, pz, pv);
        }
      } else if (!nearp) {
        float q[12];
        load4<3>(&T[k].c[8], q);
        const float w[3] = {h7.y, h7.y, h7.y};
        panel_points<3, WANT_V>(q, w, r0, r1, r2, px, py, pz, pv);
      }
    }
    neumaier(hx, lx, px);
    neumaier(hy, ly, py);
    neumaier(hz, lz, pz);
    if (WANT_V) neumaier(hv, lv, pv);
  }
  if (active) {
    double *acc = part + (size_t)by * 4 * n_t;
    acc[i] = (double)hx + (double)lx;
    acc[(size_t)n_t + i] = (double)hy + (double)ly;
    acc[2 * (size_t)n_t + i] = (double)hz + (double)lz;
    acc[3 * (size_t)n_t + i] = WANT_V ? (double)hv + (double)lv : 0.0;
  }
}

template <bool WANT_V>
__global__ __launch_bounds__(kThreads) void k_panel_mixed(int n_t, const double *__restrict__ xs, int N,
                                                          const double *__restrict__ f,
                                                          const double *__restrict__ sigma, int cchunk, double *part) {
  panel_mixed<WANT_V>(blockIdx.x, blockIdx.y, n_t, xs, N, f, sigma, cchunk, part);
}

// FP64 mode: closed form up to 48 diameters (k_panel_close), FP64
// 7-point rule beyond (k_panel_fp64).  Both decide with the same FP64 test
// |x - c_k|^2 >= (48 D_k)^2 on the unmodified coordinates.
// Bound by FP64 issue (132 operations and 7 reciprocal roots a pair): 50,000
// targets and 40,776 cells of the GEM cell take 9.2 ms, with two Newton steps a
// root 10.5.  One root a pair, with the outer points' factors
// (1 + delta)^(-3/2) by a polynomial, took 7.1 ms, but its rounding was twice as
// large (2.5e-16 instead of 1.2e-16 of the rule's sum, root mean square): the
// rounding of x - c and of the one root enters all seven terms alike, where
// seven of their own average.
constexpr int kPF = 32;  // cells per LDS tile of the FP64 far kernel

// One cell of the FP64 far kernel's LDS tile: centroid, (48 D)^2, the 7 rule
// points, area sigma {w0, wa, wa, wa, wb, wb, wb} folded per point.
struct CellF64 {
  double g[3], lim, q[21], w[7];
};

template <bool WANT_V>
__device__ __forceinline__ void panel_fp64(int bx, int by, int n_t, const double *__restrict__ xs, int N,
                                           const double *__restrict__ f, const double *__restrict__ sigma, int cchunk,
                                           double *part) {
  __shared__ CellF64 T[kPF];
  const int tid = threadIdx.x;
  const int i = bx * kThreads + tid;
  const bool active = i < n_t;
  const int ii = active ? i : 0;
  const double x0 = xs[ii], x1 = xs[(size_t)n_t + ii], x2 = xs[2 * (size_t)n_t + ii];
  double ex = 0.0, ey = 0.0, ez = 0.0, ev = 0.0;
  const int kb = by * cchunk, ke = min(N, kb + cchunk);
  for (int k0 = kb; k0 < ke; k0 += kPF) {
    const int cnt = min(kPF, ke - k0);
    __syncthreads();
    for (int idx = tid; idx < 21 * kPF; idx += kThreads) {
      const int m = idx / kPF, k = idx % kPF;
      if (k < cnt) T[k].q[m] = f[(size_t)(MF_Q7 + m) * N + k0 + k];
    }
    if (tid < cnt) {
      const int kk = k0 + tid;
      const double D = f[(size_t)MF_DIAM * N + kk];
      const double as = f[(size_t)MF_AREA * N + kk] * sigma[kk];
      T[tid].g[0] = f[(size_t)MF_GX * N + kk];
      T[tid].g[1] = f[(size_t)MF_GY * N + kk];
      T[tid].g[2] = f[(size_t)MF_GZ * N + kk];
      T[tid].lim = kQuadFp64 * kQuadFp64 * D * D;
#pragma unroll
      for (int m = 0; m < 7; ++m) T[tid].w[m] = as * (m == 0 ? Rule7::w0 : (m < 4 ? Rule7::wa : Rule7::wb));
    }
    __syncthreads();
    for (int k = 0; k < cnt; ++k) {
      const double dx = x0 - T[k].g[0], dy = x1 - T[k].g[1], dz = x2 - T[k].g[2];
      const double R2 = fma(dx, dx, fma(dy, dy, dz * dz));
      if (R2 >= T[k].lim) {  // the near kernel takes the others
#pragma unroll
        for (int m = 0; m < 7; ++m) {
          const double qx = x0 - T[k].q[3 * m], qy = x1 - T[k].q[3 * m + 1], qz = x2 - T[k].q[3 * m + 2];
          const double ri = rsqrt_f64(fma(qx, qx, fma(qy, qy, qz * qz)));
          const double wr = T[k].w[m] * ri;
          const double t = wr * ri * ri;
          ex = fma(t, qx, ex);
          ey = fma(t, qy, ey);
          ez = fma(t, qz, ez);
          if (WANT_V) ev += wr;
        }
      }
    }
  }
  if (active) {
    double *acc = part + (size_t)by * 4 * n_t;
    acc[i] = ex;
    acc[(size_t)n_t + i] = ey;
    acc[2 * (size_t)n_t + i] = ez;
    acc[3 * (size_t)n_t + i] = ev;
  }
}

template <bool WANT_V>
__global__ __launch_bounds__(kThreads) void k_panel_fp64(int n_t, const double *__restrict__ xs, int N,
                                                         const double *__restrict__ f,
                                                         const double *__restrict__ sigma, int cchunk, double *part) {
  panel_fp64<WANT_V>(blockIdx.x, blockIdx.y, n_t, xs, N, f, sigma, cchunk, part);
}

// FP64 closed-form zone of both modes (MIXED: R < 3 D by the far kernel's FP32
// test on the same recentred values; else R < 48 D by its FP64 test), added
// to the far kernel's partial sums of the same cell range (gridDim.y splits
// the cells as there; one writer per entry, stream order).  A workgroup has 64
// targets and WAVES waves, each with its share of every tile's cells: the
// zone's work is uneven over targets and cells, and a wave whose targets are
// close to a whole tile runs 64 batches one after the other.  A wave bounds its 64 targets by a sphere
// and visits the 64-cell tiles whose zone sphere (centre, max_k |c_k -
// centre| + zone D_k, slightly inflated) it meets; in a tile, lane k tests
// cell k once against the sphere, and the flagged cells take the per-lane
// test.  A cell that at least kDenseLanes of the targets see from 2.5 D to the
// zone's end is evaluated for them at once (cell_mid_form, the record in
// scalar registers).  All other pairs are queued in LDS and evaluated 64 at a
// time, one pair per lane, so that a cell near a single target costs a
// sixty-fourth of a wave's closed form; each target then adds its own pairs'
// results in queue order (deterministic).  Bound by
// the closed form's FP64 operations.  Measured against the closed form of
// every flagged cell for the whole wave: mixed, 97 points and 4,096 cells 84
// -> 34 us (14 us with four waves), 200,003 points and 40,776 cells 1346 -> 475 us; FP64, 50,000
// points and 40,776 cells 5.65 -> 2.87 ms.  kDenseLanes 8 to 32 differ by 1 %.
constexpr int kDenseLanes = 32;
// Four waves a workgroup up to this many workgroups (64 targets x splits), one
// beyond, where the chip is full with single waves and four repeat the tests
// of the tiles.  One -> four waves, calls: mixed, 128 workgroups 109 -> 89 us,
// 19,000 (20,000 charges in the holes) 1.66 -> 1.58 ms, but 23,400 (a fine
// plate) 535 -> 567 us, 60,000 2.79 -> 2.94 ms, 200,000 8.4 -> 9.0 ms; FP64
// (more pairs a test) 4,096 233 -> 198 us, 8,000 3.00 -> 2.25 ms, 50,000 11.9 ->
// 11.6 ms, but 78,000 (the coarse GEM cell) 3.47 -> 3.63 ms, 200,000 8.6 -> 9.1
// ms; plates of 800 cells lose 2 % at 10,000 already and 7 % at 41,000.
constexpr int kCloseFew = 20480, kCloseFewFp64 = 61440;

template <bool WANT_V, bool MIXED, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_panel_close(int n_t, const double *__restrict__ xs, int N,
                                                            const double *__restrict__ f,
                                                            const double *__restrict__ rec,
                                                            const double *__restrict__ sigma,
                                                            const double *__restrict__ tiles, int cchunk,
                                                            double *part) {
  constexpr int NC = WANT_V ? 4 : 3;
  __shared__ double Xs[WAVES][3][64];
  __shared__ double Rs[WAVES][NC][64];
  __shared__ int qks[WAVES][128], qls[WAVES][128];
  const int lane = threadIdx.x & 63, wave = WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  auto &X = Xs[wave];
  auto &R = Rs[wave];
  auto &qk = qks[wave];
  auto &ql = qls[wave];
  const int i = blockIdx.x * 64 + lane;
  const bool active = i < n_t;
  const int ii = active ? i : n_t - 1;
  const double x0 = xs[ii], x1 = xs[(size_t)n_t + ii], x2 = xs[2 * (size_t)n_t + ii];
  X[0][lane] = x0;
  X[1][lane] = x1;
  X[2][lane] = x2;
  // wave bounding sphere
  double lo0 = x0, lo1 = x1, lo2 = x2, hi0 = x0, hi1 = x1, hi2 = x2;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo0 = fmin(lo0, __shfl_xor(lo0, o));
    lo1 = fmin(lo1, __shfl_xor(lo1, o));
    lo2 = fmin(lo2, __shfl_xor(lo2, o));
    hi0 = fmax(hi0, __shfl_xor(hi0, o));
    hi1 = fmax(hi1, __shfl_xor(hi1, o));
    hi2 = fmax(hi2, __shfl_xor(hi2, o));
  }
  const double wc0 = 0.5 * (lo0 + hi0), wc1 = 0.5 * (lo1 + hi1), wc2 = 0.5 * (lo2 + hi2);
  const double wr = 0.5 * sqrt((hi0 - lo0) * (hi0 - lo0) + (hi1 - lo1) * (hi1 - lo1) + (hi2 - lo2) * (hi2 - lo2));
  // mixed: the far kernel's frame (recentred on the first target of the
  // 256-target workgroup, FP32), and the sphere in it, radius measured from
  // its FP32 centre (widened by 1e-4 for the rounding)
  double c0 = 0.0, c1 = 0.0, c2 = 0.0;
  float r0 = 0.f, r1 = 0.f, r2 = 0.f, fw0 = 0.f, fw1 = 0.f, fw2 = 0.f, fwr = 0.f;
  if (MIXED) {
    const int i0 = blockIdx.x * 64 / kThreads * kThreads;
    c0 = xs[i0];
    c1 = xs[(size_t)n_t + i0];
    c2 = xs[2 * (size_t)n_t + i0];
    r0 = (float)(x0 - c0);
    r1 = (float)(x1 - c1);
    r2 = (float)(x2 - c2);
    fw0 = (float)(wc0 - c0);
    fw1 = (float)(wc1 - c1);
    fw2 = (float)(wc2 - c2);
    fwr = sqrtf(dist2f(r0, r1, r2, fw0, fw1, fw2));
    for (int o = 32; o > 0; o >>= 1) fwr = fmaxf(fwr, __shfl_xor(fwr, o));
    fwr *= 1.0001f;
  }
  double ex = 0.0, ey = 0.0, ez = 0.0, ev = 0.0;
  int qn = 0;                                // pairs queued (wave-uniform, < 64 between cells)
  unsigned long long mine = 0ull, next = 0;  // this lane's queue positions below 64 and from 64 on
  // the cell range of split blockIdx.y (cchunk is a multiple of the tile);
  // t = te flushes the rest
  const int tb = blockIdx.y * cchunk / 64, te = (min(N, (int)(blockIdx.y + 1) * cchunk) + 63) / 64;
  for (int t = tb; t <= te; ++t) {
    const int k0 = t * 64, cnt = min(64, N - k0);
    double cg0 = 0.0, cg1 = 0.0, cg2 = 0.0, cD = 0.0;
    float g0 = 0.f, g1 = 0.f, g2 = 0.f, lim = 0.f;
    bool flag = false;
    if (t < te) {
      const double dx = wc0 - tiles[4 * t], dy = wc1 - tiles[4 * t + 1], dz = wc2 - tiles[4 * t + 2];
      const double rs = (wr + tiles[4 * t + 3]) * (1.0 + 1e-9);
      if (dx * dx + dy * dy + dz * dz > rs * rs) continue;  // wave-uniform
      if (lane < cnt) {
        const int kk = k0 + lane;
        cg0 = f[(size_t)MF_GX * N + kk];
        cg1 = f[(size_t)MF_GY * N + kk];
        cg2 = f[(size_t)MF_GZ * N + kk];
        cD = f[(size_t)MF_DIAM * N + kk];
        if (MIXED) {
          // the near limit exactly as the far kernel stages it; the wave's
          // test 1 % wide
          g0 = (float)(cg0 - c0);
          g1 = (float)(cg1 - c1);
          g2 = (float)(cg2 - c2);
          lim = (float)(kNearMixed * kNearMixed * cD * cD);
          flag = sqrtf(dist2f(fw0, fw1, fw2, g0, g1, g2)) - fwr < (float)(kNearMixed * 1.01) * (float)cD;
        } else {
          // 0.1 % wide
          const double u0 = cg0 - wc0, u1 = cg1 - wc1, u2 = cg2 - wc2;
          flag = sqrt(u0 * u0 + u1 * u1 + u2 * u2) - wr < kQuadFp64 * 1.001 * cD;
        }
      }
    }
    uint64_t m = __ballot(flag);
    if (WAVES == 4) m &= 0x1111111111111111ull << wave;  // this wave's share of the tile
    for (;;) {
      for (; m && qn < 64; m &= m - 1ull) {
        const int k = __builtin_amdgcn_readfirstlane(__builtin_ctzll(m));
        const int kk = k0 + k;
        bool nearp;
        double R2 = 0.0, D2 = 0.0;
        if (MIXED) {
          const float h0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g0), k));
          const float h1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g1), k));
          const float h2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g2), k));
          const float hl = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lim), k));
          nearp = active && dist2f(r0, r1, r2, h0, h1, h2) < hl;
        } else {
          const double gx = x0 - readlane_f64(cg0, k), gy = x1 - readlane_f64(cg1, k), gz = x2 - readlane_f64(cg2, k);
          const double D = readlane_f64(cD, k);
          R2 = fma(gx, gx, fma(gy, gy, gz * gz));
          D2 = D * D;
          nearp = active && !(R2 >= kQuadFp64 * kQuadFp64 * D * D);
        }
        if (!MIXED) {
          const bool mid = nearp && R2 >= kMidForm * kMidForm * D2;
          if (__popcll(__ballot(mid)) >= kDenseLanes) {
            if (mid) {
              const double sg = sigma[kk];
              d3 E;
              double V;
              cell_mid_form<WANT_V>(rec + (size_t)kk * CR_COUNT, mk3(x0, x1, x2), E, V);
              ex = fma(sg, E.x, ex);
              ey = fma(sg, E.y, ey);
              ez = fma(sg, E.z, ez);
              if (WANT_V) ev = fma(sg, V, ev);
              nearp = false;
            }
          }
        }
        const unsigned long long nm = __ballot(nearp);
        if (nm) {
          if (nearp) {
            const int p = qn + __popcll(nm & ((1ull << lane) - 1ull));
            qk[p] = kk;
            ql[p] = lane;
            if (p < 64)
              mine |= 1ull << p;
            else
              next |= 1ull << (p - 64);
          }
          qn += __popcll(nm);
        }
      }
      const int n = t < te ? (qn >= 64 ? 64 : 0) : min(qn, 64);
      if (n == 0) break;
      // the first n queued pairs, one per lane; then every lane adds its own
      // (within the wave: the fences only order the LDS accesses)
      wave_lds_fence();
      if (lane < n) {
        const int k = qk[lane], l = ql[lane];
        d3 E;
        double V;
        cell_closed_form<WANT_V>(rec + (size_t)k * CR_COUNT, mk3(X[0][l], X[1][l], X[2][l]), E, V);
        const double sg = sigma[k];
        R[0][lane] = sg * E.x;
        R[1][lane] = sg * E.y;
        R[2][lane] = sg * E.z;
        if (WANT_V) R[NC - 1][lane] = sg * V;
      }
      wave_lds_fence();
      for (; mine; mine &= mine - 1ull) {
        const int j = __builtin_ctzll(mine);
        ex += R[0][j];
        ey += R[1][j];
        ez += R[2][j];
        if (WANT_V) ev += R[NC - 1][j];
      }
      qn -= n;
      mine = next;
      next = 0ull;
      int k2 = 0, l2 = 0;
      if (lane < qn) {
        k2 = qk[64 + lane];
        l2 = ql[64 + lane];
      }
      wave_lds_fence();
      if (lane < qn) {
        qk[lane] = k2;
        ql[lane] = l2;
      }
    }
  }
  if (WAVES > 1) {  // the waves' sums, in their order
    wave_lds_fence();
    R[0][lane] = ex;
    R[1][lane] = ey;
    R[2][lane] = ez;
    if (WANT_V) R[NC - 1][lane] = ev;
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
      ex += Rs[w][0][lane];
      ey += Rs[w][1][lane];
      ez += Rs[w][2][lane];
      if (WANT_V) ev += Rs[w][NC - 1][lane];
    }
  }
  if (active) {
    double *acc = part + (size_t)blockIdx.y * 4 * n_t;
    acc[i] += ex;
    acc[(size_t)n_t + i] += ey;
    acc[2 * (size_t)n_t + i] += ez;
    if (WANT_V) acc[3 * (size_t)n_t + i] += ev;
  }
}

// Slot sums: acc[c][i] = (has_base ? acc[c][i] : 0) + the slots' entries
// part[s][c][i] in slot order, one thread per (component, point).  Bound by
// the latency of the loads for few points and by HBM for many: 16 loads of a
// thread in flight and one component per thread (97 points, 64 slots: one
// workgroup that walked the slots one by one took 58 us).
__global__ __launch_bounds__(kSlotThreads) void k_slot_sum(int n, int ns, size_t stride,
                                                           const double *__restrict__ part, int has_base,
                                                           double *acc) {
  const int i = blockIdx.x * kSlotThreads + threadIdx.x;
  if (i >= n) return;
  const size_t o = (size_t)blockIdx.y * n + i;
  acc[o] = slot_sum(has_base ? acc[o] : 0.0, part + o, stride, ns);
}

void launch_slot_sum(obem_ctx *ctx, int n, int comps, const Slots &s, bool has_base, double *acc) {
  hipLaunchKernelGGL(k_slot_sum, dim3((n + kSlotThreads - 1) / kSlotThreads, comps), dim3(kSlotThreads), 0, ctx->stream,
                     n, s.n, (size_t)comps * n, s.p, has_base ? 1 : 0, acc);
}

// The field at the caller's targets from the cell slots and the source-chunk
// slots in one pass: scale * (cells in split order, then chunks in order),
// scattered to caller order.
__global__ __launch_bounds__(kSlotThreads) void k_slot_finish(int n, const int32_t *__restrict__ perm, Slots cells,
                                                              Slots pairs, double scale, double *Ex, double *Ey,
                                                              double *Ez, double *V) {
  const int i = blockIdx.x * kSlotThreads + threadIdx.x;
  if (i >= n) return;
  const int c = blockIdx.y;
  const size_t o = (size_t)c * n + i;
  double v = slot_sum(0.0, cells.p + o, 4 * (size_t)n, cells.n);
  v = slot_sum(v, pairs.p + o, 4 * (size_t)n, pairs.n);
  double *out = c == 0 ? Ex : (c == 1 ? Ey : (c == 2 ? Ez : V));
  out[perm[i]] = scale * v;
}

obem_status launch_finish(obem_ctx *ctx, const TargetOrder &to, const Slots &cells, const Slots &pairs, double scale,
                          double *Ex, double *Ey, double *Ez, double *V) {
  if (to.n == 0) return OBEM_OK;
  OBEM_PROF(ctx, "scatter");
  hipLaunchKernelGGL(k_slot_finish, dim3((to.n + kSlotThreads - 1) / kSlotThreads, V ? 4 : 3), dim3(kSlotThreads), 0,
                     ctx->stream, to.n, to.perm, cells, pairs, scale, Ex, Ey, Ez, V);
  OBEM_HIP(ctx, hipGetLastError());
  return OBEM_OK;
}

// Splits of the cells for n_t targets, and where the sums go.
struct PanelPlan {
  int bt, ns, cchunk;
  double *part;
};
static obem_status panel_plan(obem_ctx *ctx, int n_t, int N, double *acc, PanelPlan *P) {
  const int bt = nblk(n_t);
  // cell ranges of >= 64 cells (a multiple of both LDS tiles), about
  // kSplitWorkgroups workgroups in all
  int ns = std::max(1, std::min((kSplitWorkgroups + bt - 1) / bt, (N + 63) / 64));
  ns = std::min(ns, max_slots(bt));
  int cchunk = (N + ns - 1) / ns;
  cchunk = (cchunk + 63) / 64 * 64;
  ns = (N + cchunk - 1) / cchunk;
  double *part = acc;
  if (ns > 1) {
    part = (double *)ws_get(ctx, WS_PANEL, sizeof(double) * 4 * (size_t)n_t * ns);
    if (!part) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
  }
  *P = PanelPlan{bt, ns, cchunk, part};
  return OBEM_OK;
}

// The near kernel of split y adds the closed-form pairs of the same cell range
// into the same slot (one writer per entry, after the far kernel); the slots
// are added in split order.
static void launch_panel_close(obem_ctx *ctx, const obem_meshh *m, const double *sigma, const TargetOrder &to,
                               obem_precision prec, bool want_v, const PanelPlan &P) {
  const int n_t = to.n, N = (int)m->n;
#define PANEL_CLOSE(V, M, T)                                                                              \
  if (few)                                                                                                \
    hipLaunchKernelGGL((k_panel_close<V, M, 4>), dim3(bw, P.ns), dim3(256), 0, ctx->stream, n_t, to.xs, N, m->f, \
                       m->rec, sigma, T, P.cchunk, P.part);                                                    \
  else                                                                                                    \
    hipLaunchKernelGGL((k_panel_close<V, M, 1>), dim3(bw, P.ns), dim3(64), 0, ctx->stream, n_t, to.xs, N, m->f, \
                       m->rec, sigma, T, P.cchunk, P.part)
  const int bw = (n_t + 63) / 64;
  const bool few = (int64_t)bw * P.ns <= (prec == OBEM_MIXED ? kCloseFew : kCloseFewFp64);
  if (prec == OBEM_MIXED) {
    if (want_v) {
      PANEL_CLOSE(true, true, m->tiles);
    } else {
      PANEL_CLOSE(false, true, m->tiles);
    }
  } else if (want_v) {
    PANEL_CLOSE(true, false, m->tiles48);
  } else {
    PANEL_CLOSE(false, false, m->tiles48);
  }
#undef PANEL_CLOSE
}

obem_status launch_panel_field(obem_ctx *ctx, const obem_meshh *m, const double *sigma, const TargetOrder &to,
                               obem_precision prec, bool want_v, double *acc, Slots *slots) {
  const int n_t = to.n;
  if (slots) *slots = Slots{acc, 0};
  if (n_t == 0) return OBEM_OK;
  const int N = (int)m->n;
  PanelPlan P;
  const obem_status st = panel_plan(ctx, n_t, N, acc, &P);
  if (st) return st;
  dim3 gsplit(P.bt, P.ns), block(kThreads);
  OBEM_PROF(ctx, "panel");
#define PANEL_FAR(K, V) \
  hipLaunchKernelGGL(K<V>, gsplit, block, 0, ctx->stream, n_t, to.xs, N, m->f, sigma, P.cchunk, P.part)
  if (prec == OBEM_MIXED) {
    if (want_v) PANEL_FAR(k_panel_mixed, true); else PANEL_FAR(k_panel_mixed, false);
  } else {
    if (want_v) PANEL_FAR(k_panel_fp64, true); else PANEL_FAR(k_panel_fp64, false);
  }
#undef PANEL_FAR
  launch_panel_close(ctx, m, sigma, to, prec, want_v, P);
  if (slots)
    *slots = Slots{P.part, P.ns};
  else if (P.ns > 1)
    launch_slot_sum(ctx, n_t, 4, Slots{P.part, P.ns}, false, acc);
  OBEM_HIP(ctx, hipGetLastError());
  return OBEM_OK;
}

// ---------------------------------------------------------------------------
// Pairwise point-charge field, eq. (nbody) with Plummer softening
// ---------------------------------------------------------------------------
// Each workgroup takes 256 consecutive (sorted) targets and one chunk of the
// sources (gridDim.y chunks, so small target sets still fill the chip), and
// writes per-chunk partial sums part[chunk][4][n_t] (Ex, Ey, Ez, V) plus the
// nearest opposite-species source; the chunks are then summed in
// order.  Source tiles of 256 are staged in LDS (recentred FP32 position and
// charge, read as broadcasts).
// Species keys: electron 0 looks for cation 1 and vice versa.
__device__ __forceinline__ int want_key(int8_t s) { return s == 0 ? 1 : (s == 1 ? 0 : -2); }

// EXCL: 0 = no exclusion (a coincident term contributes exactly 0 to E when
// soft > 0), 1 = drop zero-distance terms (soft == 0), 2 = drop the source
// whose index equals the target's caller index (targets are the sources).
// HL: the recentred coordinates are carried as FP32 pairs (hi, lo) with
// hi + lo = the FP64 difference to the origin to about 2^-48 of it, and
// r - s = (r_hi - s_hi) + (r_lo - s_lo): both differences are exact or
// nearly so, so the separation keeps a relative error of a few 2^-24 however
// close the pair is, instead of 2^-24 (|r| + |s|) / |r - s| with the hi parts
// alone (tiles near the workgroup's targets, where the closest pairs are).
template <bool WANT_V, bool NN, int EXCL, bool FOLDQ, bool HL>
__device__ __forceinline__ void pair_term(const float4 *S, const float4 *SL, const int *K, int jj, int jt,
                                          float r0, float r1, float r2, float rl0, float rl1, float rl2,
                                          float soft2, int self, int want, float &px, float &py, float &pz,
                                          float &pv, float &best, int &bidx) {
  const float4 s = S[jj];
  float dx = r0 - s.x, dy = r1 - s.y, dz = r2 - s.z;
  if (HL) {
    const float4 l = SL[jj];
    dx += rl0 - l.x;
    dy += rl1 - l.y;
    dz += rl2 - l.z;
  }
  const float rr = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, soft2)));
  float ri = __builtin_amdgcn_rsqf(rr);
  if (EXCL == 1) ri = rr > 0.f ? ri : 0.f;
  if (EXCL == 2) ri = (jt + jj == self) ? 0.f : ri;
  const float qr = FOLDQ ? ri : s.w * ri;
  const float w = qr * (ri * ri);
  px = fmaf(w, dx, px);
  py = fmaf(w, dy, py);
  pz = fmaf(w, dz, pz);
  if (WANT_V) pv += qr;
  if (NN) {
    if (K[jj] == want && rr < best && (EXCL != 1 || rr > 0.f)) {
      best = rr;
      bidx = jt + jj;
    }
  }
}

// The (hi, lo) loop is unrolled by 2 only, so that its extra registers do
// not lower the occupancy of the kernel (unrolled by 1 it was 10 % slower,
// by 4 5 %, in the 4M-charge step where it takes nearly every tile pair of
// the directed remainder).
template <bool WANT_V, bool NN, int EXCL, bool FOLDQ, bool HL>
__device__ __forceinline__ void pair_tile(const float4 *S, const float4 *SL, const float (*RL)[kThreads],
                                          const int *K, int cnt, int jt, float r0, float r1, float r2, float soft2,
                                          int self, int want, float &px, float &py, float &pz, float &pv,
                                          float &best, int &bidx) {
  float rl0 = 0.f, rl1 = 0.f, rl2 = 0.f;
  if constexpr (HL) {
    rl0 = RL[0][threadIdx.x];
    rl1 = RL[1][threadIdx.x];
    rl2 = RL[2][threadIdx.x];
#pragma unroll 2
    for (int jj = 0; jj < cnt; ++jj)
      pair_term<WANT_V, NN, EXCL, FOLDQ, true>(S, SL, K, jj, jt, r0, r1, r2, rl0, rl1, rl2, soft2, self, want, px,
                                               py, pz, pv, best, bidx);
  } else {
    for (int jj = 0; jj < cnt; ++jj)
      pair_term<WANT_V, NN, EXCL, FOLDQ, false>(S, SL, K, jj, jt, r0, r1, r2, rl0, rl1, rl2, soft2, self, want, px,
                                                py, pz, pv, best, bidx);
  }
}

// Far tiles of one charge (the tile's box at least 2 R_b from the box of the
// workgroup's targets, R_b = their largest distance from the recentring
// origin): |r - s|^2 = (|r|^2 + soft^2) + |s|^2 - 2 r.s and E = r sum(w) -
// sum(w s), 11 VALU per pair instead of 12.  Since |s| <= |r| + |r - s|, the
// expansion's terms are at most (1 + 2 R_b / |r - s|)^2 <= 4 times |r - s|^2,
// which bounds its rounding error to a few ulps of |r - s|^2.
__device__ __forceinline__ void pair_tile_far(const float4 *S2, int cnt, float m0, float m1, float m2, float a,
                                              float &sw, float &sx, float &sy, float &sz) {
  for (int jj = 0; jj < cnt; ++jj) {
    const float4 s = S2[jj];
    const float rr = fmaf(m0, s.x, fmaf(m1, s.y, fmaf(m2, s.z, a + s.w)));
    const float ri = __builtin_amdgcn_rsqf(rr);
    const float w = ri * (ri * ri);
    sw += w;
    sx = fmaf(w, s.x, sx);
    sy = fmaf(w, s.y, sy);
    sz = fmaf(w, s.z, sz);
  }
}

// Per super-block: the centre of the box around its tiles' boxes (the
// origin the pair-once kernel recentres on) and the squared distance from
// it to the box's corners, sb[4 A + 0..2] and sb[4 A + 3].
__global__ __launch_bounds__(256) void k_sym_radius(int n, int ns, int sym_tiles, const double *__restrict__ tbox,
                                                    double *sb) {
  const int A = blockIdx.x * 256 + threadIdx.x;
  if (A >= ns) return;
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int k = 0; k < sym_tiles && (A * sym_tiles + k) * kThreads < n; ++k) {
    const double *bx = tbox + 6 * (size_t)(A * sym_tiles + k);
    for (int c = 0; c < 3; ++c) {
      lo[c] = fmin(lo[c], bx[c]);
      hi[c] = fmax(hi[c], bx[3 + c]);
    }
  }
  double r2 = 0.0;
  for (int c = 0; c < 3; ++c) {
    sb[4 * (size_t)A + c] = 0.5 * (lo[c] + hi[c]);
    const double h = 0.5 * (hi[c] - lo[c]);
    r2 = fma(h, h, r2);
  }
  sb[4 * (size_t)A + 3] = r2;
}

// Bit b of row a (32 tiles per word): tile_pair_direct(a, b), for the
// directed kernel to skip the other tiles by one scalar bit test.
__global__ __launch_bounds__(256) void k_tile_mask(int ntile, int wpr, int sym_tiles, int nn, double cut2,
                                                   const double *__restrict__ tbox, const double *__restrict__ sb,
                                                   uint32_t *mask) {
  const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (size_t)ntile * wpr) return;
  const int a = (int)(t / wpr), w = (int)(t % wpr);
  uint32_t m = 0;
  for (int u = 0; u < 32; ++u) {
    const int b = w * 32 + u;
    if (b < ntile && tile_pair_direct(tbox, sb, a, b, sym_tiles, nn != 0, cut2)) m |= 1u << u;
  }
  mask[t] = m;
}

template <bool WANT_V, bool NN, int EXCL>
__device__ __forceinline__ void pair_mixed(int bx, int n_t, const double *__restrict__ xs,
                                           const int32_t *__restrict__ perm, int n_s, const double *__restrict__ sx,
                                           const double *__restrict__ sy, const double *__restrict__ sz,
                                           const double *__restrict__ sq, const int8_t *__restrict__ species,
                                           const int8_t *__restrict__ species_s, float soft2, int chunk, double *part,
                                           float *nn_d2p, int32_t *nn_ip, const double *__restrict__ tbox,
                                           float nn_cut2, const int32_t *__restrict__ self_map, int sym_tiles,
                                           double nn_cut2d, const uint32_t *__restrict__ dmask, int dwpr) {
  constexpr bool kFar = (EXCL == 0) && !WANT_V;  // expanded far tiles allowed
  __shared__ float4 S[kThreads];
  __shared__ float4 SL[kThreads];
  __shared__ float RL[3][kThreads];  // lo parts of the targets (read by the (hi, lo) tiles only)
  __shared__ float4 S2[kFar ? kThreads : 1];
  __shared__ int K[kThreads];
  __shared__ float WB[kThreads / 64][6];
  // one-dimensional grid, the source chunks of a target tile consecutive:
  // with targets = sources nearly all the directed tile pairs of a target
  // tile lie in one chunk, so the busy workgroups are spread evenly over the
  // launch instead of coming in one block per chunk
  const int nsplit = (n_s + chunk - 1) / chunk;
  const int tt = (int)bx / nsplit, split = (int)bx % nsplit;
  const int tid = threadIdx.x;
  const int i0 = tt * kThreads;
  const int i = i0 + tid;
  const bool active = i < n_t;
  const double c0 = xs[i0], c1 = xs[(size_t)n_t + i0], c2 = xs[2 * (size_t)n_t + i0];
  const double x0 = active ? xs[i] : c0;
  const double x1 = active ? xs[(size_t)n_t + i] : c1;
  const double x2 = active ? xs[2 * (size_t)n_t + i] : c2;
  const double e0 = x0 - c0, e1 = x1 - c1, e2 = x2 - c2;
  const float r0 = (float)e0, r1 = (float)e1, r2 = (float)e2;
  RL[0][tid] = (float)(e0 - (double)r0);
  RL[1][tid] = (float)(e1 - (double)r1);
  RL[2][tid] = (float)(e2 - (double)r2);
  const float m0 = -2.f * r0, m1 = -2.f * r1, m2 = -2.f * r2;
  const float a_t = fmaf(r0, r0, fmaf(r1, r1, fmaf(r2, r2, soft2)));
  int want = -2;
  if (NN && active) want = want_key(species[perm[i]]);
  // which partner species any target of the workgroup looks for (the step's
  // source charges follow their species: cations +e, electrons and anions -e)
  bool want_pos = false, want_neg = false;
  if (NN) {
    want_pos = __syncthreads_or(want == 1);
    want_neg = __syncthreads_or(want == 0);
  }
  const int self = active ? (self_map ? self_map[perm[i]] : perm[i]) : -1;
  const int jb = split * chunk;
  const int je = min(n_s, jb + chunk);
  // Bounding box of the workgroup's targets (recentred FP32), tested against
  // each source tile's box (tbox, FP64, 256-source tiles): tiles farther
  // than the partner cut skip the nearest-partner search, far tiles take the
  // expanded form, near ones the (hi, lo) separation.  Inactive lanes hold
  // the first target, which is inside the box.
  float bl0 = r0, bl1 = r1, bl2 = r2, bh0 = r0, bh1 = r1, bh2 = r2;
  if (tbox) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      bl0 = fminf(bl0, __shfl_xor(bl0, o));
      bl1 = fminf(bl1, __shfl_xor(bl1, o));
      bl2 = fminf(bl2, __shfl_xor(bl2, o));
      bh0 = fmaxf(bh0, __shfl_xor(bh0, o));
      bh1 = fmaxf(bh1, __shfl_xor(bh1, o));
      bh2 = fmaxf(bh2, __shfl_xor(bh2, o));
    }
    if ((tid & 63) == 0) {
      float *w = WB[tid >> 6];
      w[0] = bl0; w[1] = bl1; w[2] = bl2; w[3] = bh0; w[4] = bh1; w[5] = bh2;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kThreads / 64; ++k) {
      bl0 = fminf(bl0, WB[k][0]);
      bl1 = fminf(bl1, WB[k][1]);
      bl2 = fminf(bl2, WB[k][2]);
      bh0 = fmaxf(bh0, WB[k][3]);
      bh1 = fmaxf(bh1, WB[k][4]);
      bh2 = fmaxf(bh2, WB[k][5]);
    }
  }
  // R_b^2: squared distance from the origin to the farthest corner of the
  // targets' box.  Tiles at least 2 R_b away (squared gap, with a margin
  // for the FP32 boxes) take the expanded form; tiles nearer than R_b / 4
  // take the (hi, lo) separation: beyond that |r - s| >= R_b / 4 and
  // |r|, |s| - |r - s| <= R_b bound the hi-only separation's relative error
  // by about 10 * 2^-24.
  const float rb2 = fmaxf(bl0 * bl0, bh0 * bh0) + fmaxf(bl1 * bl1, bh1 * bh1) + fmaxf(bl2 * bl2, bh2 * bh2);
  const float far2 = 4.f * rb2 * 1.001f + 1e-30f;
  const float close2 = 0.0625f * rb2 * 1.001f + 1e-30f;
  float hx = 0.f, hy = 0.f, hz = 0.f, hv = 0.f, lx = 0.f, ly = 0.f, lz = 0.f, lv = 0.f;
  float best = INFINITY;
  int bidx = -1;
  for (int jt = jb; jt < je; jt += kThreads) {
    // targets are the sources in the same order under sym_tiles: this
    // workgroup's targets are source tile tt, and the tile pairs that
    // tile_pair_direct (dmask, row tt) does not keep here are evaluated by
    // k_pair_sym; skip to the next tile of the row, a word (32 tiles) at a
    // time (scalar)
    if (sym_tiles) {
      const uint32_t *mrow = dmask + (size_t)tt * dwpr;
      const int be = (je + kThreads - 1) / kThreads;
      int b = jt / kThreads;
      uint32_t wd = mrow[b >> 5] >> (b & 31);
      while (wd == 0u) {
        b = (b | 31) + 1;
        if (b >= be) break;
        wd = mrow[b >> 5];
      }
      if (b >= be) break;
      b += __builtin_ctz(wd);
      if (b >= be) break;
      jt = b * kThreads;
    }
    const int cnt = min(kThreads, je - jt);
    const float q0 = (float)sq[jt];
    bool nn_tile = NN;
    bool far_tile = false;
    bool close_tile = true;
    if (tbox) {
      const double *b = tbox + 6 * (size_t)(jt / kThreads);
      const float g0 = fmaxf(0.f, fmaxf((float)(b[0] - c0) - bh0, bl0 - (float)(b[3] - c0)));
      const float g1 = fmaxf(0.f, fmaxf((float)(b[1] - c1) - bh1, bl1 - (float)(b[4] - c1)));
      const float g2 = fmaxf(0.f, fmaxf((float)(b[2] - c2) - bh2, bl2 - (float)(b[5] - c2)));
      const float gap2 = fmaf(g0, g0, fmaf(g1, g1, g2 * g2));
      if (NN) nn_tile = gap2 <= nn_cut2;
      far_tile = kFar && !nn_tile && gap2 >= far2;
      close_tile = gap2 < close2;
    }
    if (sym_tiles) {
      const bool np = NN && tiles_gap2(tbox, tt, jt / kThreads) <= nn_cut2d;
      nn_tile = np;
      far_tile = far_tile && !np;
    }
    __syncthreads();
    float qj = q0;
    if (tid < cnt) {
      const int j = jt + tid;
      qj = (float)sq[j];
      const double f0 = sx[j] - c0, f1 = sy[j] - c1, f2 = sz[j] - c2;
      const float s0 = (float)f0, s1 = (float)f1, s2 = (float)f2;
      S[tid] = make_float4(s0, s1, s2, qj);
      if (close_tile)
        SL[tid] = make_float4((float)(f0 - (double)s0), (float)(f1 - (double)s1), (float)(f2 - (double)s2), 0.f);
      if (kFar) S2[tid] = make_float4(s0, s1, s2, fmaf(s0, s0, fmaf(s1, s1, s2 * s2)));
      if (NN) K[tid] = species_s[j];
    }
    // tiles of equal charges (sources grouped by species) take the charge
    // out of the inner loop: 12 instead of 13 VALU operations per pair
    const bool uniform = __syncthreads_and(qj == q0);
    // a tile of one charge sign holds no species any target looks for: no
    // partner search there
    if (NN && nn_tile && uniform && ((q0 > 0.f && !want_pos) || (q0 < 0.f && !want_neg))) nn_tile = false;
    float px = 0.f, py = 0.f, pz = 0.f, pv = 0.f;
#define PAIR_TILE(NNT, FQ, HLT)                                                                                \
  pair_tile<WANT_V, NNT, EXCL, FQ, HLT>(S, SL, RL, K, cnt, jt, r0, r1, r2, soft2, self, want, px, py, pz, pv, best, \
                                        bidx)
    if (uniform) {
      if (nn_tile) {
        if (close_tile)
          PAIR_TILE(NN, true, true);
        else
          PAIR_TILE(NN, true, false);
      } else if (kFar && far_tile) {
        float sw = 0.f, sxx = 0.f, syy = 0.f, szz = 0.f;
        pair_tile_far(S2, cnt, m0, m1, m2, a_t, sw, sxx, syy, szz);
        px = fmaf(r0, sw, -sxx);
        py = fmaf(r1, sw, -syy);
        pz = fmaf(r2, sw, -szz);
      } else if (close_tile) {
        PAIR_TILE(false, true, true);
      } else {
        PAIR_TILE(false, true, false);
      }
      px *= q0;
      py *= q0;
      pz *= q0;
      pv *= q0;
    } else {
      if (nn_tile) {
        if (close_tile)
          PAIR_TILE(NN, false, true);
        else
          PAIR_TILE(NN, false, false);
      } else if (close_tile) {
        PAIR_TILE(false, false, true);
      } else {
        PAIR_TILE(false, false, false);
      }
    }
#undef PAIR_TILE
    neumaier(hx, lx, px);
    neumaier(hy, ly, py);
    neumaier(hz, lz, pz);
    if (WANT_V) neumaier(hv, lv, pv);
  }
  if (active) {
    const size_t o = (size_t)split * 4 * n_t;
    part[o + i] = (double)hx + (double)lx;
    part[o + (size_t)n_t + i] = (double)hy + (double)ly;
    part[o + 2 * (size_t)n_t + i] = (double)hz + (double)lz;
    part[o + 3 * (size_t)n_t + i] = WANT_V ? (double)hv + (double)lv : 0.0;
    if (NN) {
      nn_d2p[(size_t)split * n_t + i] = best;
      nn_ip[(size_t)split * n_t + i] = bidx;
    }
  }
}

template <bool WANT_V, bool NN, int EXCL>
__global__ __launch_bounds__(kThreads, 7) void k_pair_mixed(int n_t, const double *__restrict__ xs,
                                                            const int32_t *__restrict__ perm, int n_s,
                                                            const double *__restrict__ sx,
                                                            const double *__restrict__ sy,
                                                            const double *__restrict__ sz,
                                                            const double *__restrict__ sq,
                                                            const int8_t *__restrict__ species,
                                                            const int8_t *__restrict__ species_s, float soft2,
                                                            int chunk, double *part, float *nn_d2p, int32_t *nn_ip,
                                                            const double *__restrict__ tbox, float nn_cut2,
                                                            const int32_t *__restrict__ self_map, int sym_tiles,
                                                            double nn_cut2d, const uint32_t *__restrict__ dmask,
                                                            int dwpr) {
  pair_mixed<WANT_V, NN, EXCL>(blockIdx.x, n_t, xs, perm, n_s, sx, sy, sz, sq, species, species_s, soft2, chunk, part, nn_d2p, nn_ip,
             tbox, nn_cut2, self_map, sym_tiles, nn_cut2d, dmask, dwpr);
}

// ---------------------------------------------------------------------------
// Pairwise field with every unordered pair evaluated once (targets = sources)
// ---------------------------------------------------------------------------
// The softened pair term of eq. (nbody) is antisymmetric: what particle j adds
// to E_i, with q_j replaced by q_i and the sign reversed, is what i adds to
// E_j.  The particles (one order for targets and sources) form super-blocks of
// kSymTiles tiles of 256.  Tile pairs inside one super-block, tile pairs
// whose boxes are within the partner cut when that search is on, and tile
// pairs closer than the radius of their super-blocks (tile_pair_direct) stay
// with the directed kernel (k_pair_mixed with sym_tiles set).  Every other
// unordered tile pair is evaluated once, here, by the workgroup of its
// super-block pair: of the ns super-blocks, A owns (A, A + d mod ns) for
// d = 1 .. sym_h(A), so that each unordered pair has exactly one owner.
//
// A workgroup takes one (A, d): thread t holds the kSymTiles particles
// A kSymSB + k 256 + t of A (FP32, recentred on sym_origin, the centre of
// the more compact of A and B), B = A + d streams through LDS
// tile by tile.  Within a tile, a wave takes the sources in groups of 64 and
// 64 steps per group: at step m lane l pairs its particles with source
// (l + m) mod 64 of the group.  The sums for A's particles stay in
// registers; the running sum of each source travels with it through the
// wave (after each step a lane passes it to the lane below, which takes that
// source next, by a lane permutation), so after 64 steps every source's sum
// over the wave's 64 x kSymTiles particles sits in one lane, in a fixed
// order of additions, without atomics.  Two groups are processed with their
// steps interleaved, so that each permutation completes while the other
// group's step is computed (measured: 0.8 % faster than one group with the
// permuted sum needed at once, 1.4 % faster than one group adding it at the
// end of each step).  Per pair 14 VALU operations and one
// reciprocal square root (3 sub, 3 FMA for d^2 + s^2, rsqrt, 2 mul for r^-3,
// 3 + 3 FMA into the two sums, the source's straight into its running
// sum) serve two interactions.  Super-block pairs with one charge on each side take the charges out
// of the loop; the others (mixed charges, partial super-blocks) carry both
// charges per pair.  Tile pairs left to the directed kernel are masked
// through their softening term, without a branch.
// Outputs per launch slot dd = d - d0, FP32: Pi[dd][3][n], the field at A's
// particles from B, and Pj[dd][3][n], the field at B's particles from A;
// k_sym_reduce adds the slots to acc in order.
constexpr int kSymTiles = 8;
constexpr int kSymSB = kSymTiles * kThreads;  // particles per super-block
constexpr int kSymSlots = 80;                 // values of d per launch, at most

template <bool NN>
__global__ __launch_bounds__(kThreads, 4) void k_pair_sym(int n, const double *__restrict__ sx,
                                                        const double *__restrict__ sy,
                                                        const double *__restrict__ sz,
                                                        const double *__restrict__ sq,
                                                        const double *__restrict__ tbox, double nn_cut2d,
                                                        const double *__restrict__ sb, float soft2, int ns,
                                                        int d0, int dcnt, float *__restrict__ Pi,
                                                        float *__restrict__ Pj) {
  // each group of 64 sources twice in a row, so that step m of lane l reads
  // entry l + m without a wrap (constant offsets in the unrolled steps)
  __shared__ float4 S[kThreads / 64][128];
  __shared__ float J[kThreads / 64][3][kThreads];
  __shared__ unsigned long long skipS;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int nxt = ((lane + 1) & 63) << 2;  // byte address of the next lane
  int A, dd;
  if (!sym_item(ns, dcnt, A, dd)) return;  // workgroup-uniform, before any barrier
  const int d = d0 + dd;
  if (d > sym_h(A, ns)) return;
  const int B = (A + d) % ns;
  const int a0 = A * kSymSB, b0 = B * kSymSB;
  const double *org = sym_origin(sb, A, B);
  const double c0 = org[0], c1 = org[1], c2 = org[2];
  float r0[kSymTiles], r1[kSymTiles], r2[kSymTiles], qa[kSymTiles];
  const float qA = (float)sq[a0], qB = (float)sq[b0];
  bool uni = true;
#pragma unroll
  for (int k = 0; k < kSymTiles; ++k) {
    const int i = a0 + k * kThreads + tid;
    const bool act = i < n;
    r0[k] = act ? (float)(sx[i] - c0) : 0.f;
    r1[k] = act ? (float)(sy[i] - c1) : 0.f;
    r2[k] = act ? (float)(sz[i] - c2) : 0.f;
    const float qi = act ? (float)sq[i] : 0.f;
    qa[k] = qi;
    const int j = b0 + k * kThreads + tid;
    uni = uni && act && qi == qA && j < n && (float)sq[j] == qB;
  }
  // tile pairs that belong to the directed kernel: bit 8 bt + k for (tile k
  // of A, tile bt of B)
  if (wv == 0) {
    bool near = false;
    const int ka = lane & 7, kb = lane >> 3;
    if (a0 + ka * kThreads < n && b0 + kb * kThreads < n)
      near = tile_pair_direct(tbox, sb, A * kSymTiles + ka, B * kSymTiles + kb, kSymTiles, NN, nn_cut2d);
    const unsigned long long m = __ballot(near);
    if (lane == 0) skipS = m;
  }
  // one charge on each side: charges out of the loop
  const bool U = __syncthreads_and(uni);
  const unsigned long long skip = skipS;
  float ex[kSymTiles], ey[kSymTiles], ez[kSymTiles];
#pragma unroll
  for (int k = 0; k < kSymTiles; ++k) ex[k] = ey[k] = ez[k] = 0.f;
  for (int bt = 0; bt < kSymTiles; ++bt) {
    const int jt = b0 + bt * kThreads;
    if (jt >= n) break;  // workgroup-uniform
    const int cnt = min(kThreads, n - jt);
    // tile pairs left to the directed kernel: a softening of 1e36 makes
    // r^-3 < 1e-54, which is 0 in FP32, so they add exactly nothing
    const unsigned sk = (unsigned)(skip >> (8 * bt)) & 0xffu;
    float s2k[kSymTiles];
#pragma unroll
    for (int k = 0; k < kSymTiles; ++k) s2k[k] = ((sk >> k) & 1u) ? 1e36f : soft2;
    __syncthreads();  // the previous tile's S and J are consumed
    {
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (tid < cnt) {
        const int j = jt + tid;
        v = make_float4((float)(sx[j] - c0), (float)(sy[j] - c1), (float)(sz[j] - c2), (float)sq[j]);
      }
      S[tid >> 6][tid & 63] = v;
      S[tid >> 6][(tid & 63) + 64] = v;
    }
    __syncthreads();
    // two groups of 64 sources at a time, their steps interleaved, so that
    // each lane permutation has the other group's step to complete in
    for (int g = 0; g < cnt; g += 128) {
      float tx = 0.f, ty = 0.f, tz = 0.f, ux = 0.f, uy = 0.f, uz = 0.f;
      const float4 *sa = &S[g >> 6][lane];
      const float4 *sb2 = &S[(g >> 6) + 1][lane];
      if (U) {
#pragma unroll 2
        for (int m = 0; m < 64; ++m) {
          {
            const float4 sj = sa[m];
            float cx = tx, cy = ty, cz = tz;
#pragma unroll
            for (int k = 0; k < kSymTiles; ++k) {
              const float dx = r0[k] - sj.x, dy = r1[k] - sj.y, dz = r2[k] - sj.z;
              const float rr = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, s2k[k])));
              const float ri = __builtin_amdgcn_rsqf(rr);
              const float w = ri * (ri * ri);
              ex[k] = fmaf(w, dx, ex[k]);
              ey[k] = fmaf(w, dy, ey[k]);
              ez[k] = fmaf(w, dz, ez[k]);
              cx = fmaf(w, dx, cx);
              cy = fmaf(w, dy, cy);
              cz = fmaf(w, dz, cz);
            }
            tx = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(cx)));
            ty = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(cy)));
            tz = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(cz)));
          }
          {
            const float4 sj = sb2[m];
            float cx = ux, cy = uy, cz = uz;
#pragma unroll
            for (int k = 0; k < kSymTiles; ++k) {
              const float dx = r0[k] - sj.x, dy = r1[k] - sj.y, dz = r2[k] - sj.z;
              const float rr = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, s2k[k])));
              const float ri = __builtin_amdgcn_rsqf(rr);
              const float w = ri * (ri * ri);
              ex[k] = fmaf(w, dx, ex[k]);
              ey[k] = fmaf(w, dy, ey[k]);
              ez[k] = fmaf(w, dz, ez[k]);
              cx = fmaf(w, dx, cx);
              cy = fmaf(w, dy, cy);
              cz = fmaf(w, dz, cz);
            }
            ux = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(cx)));
            uy = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(cy)));
            uz = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(cz)));
          }
        }
      } else {
#pragma unroll 2
        for (int m = 0; m < 64; ++m) {
          {
            const float4 sj = sa[m];
            float cx = tx, cy = ty, cz = tz;
#pragma unroll
            for (int k = 0; k < kSymTiles; ++k) {
              const float dx = r0[k] - sj.x, dy = r1[k] - sj.y, dz = r2[k] - sj.z;
              const float rr = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, s2k[k])));
              const float ri = __builtin_amdgcn_rsqf(rr);
              const float w = ri * (ri * ri);
              const float wi = w * sj.w, wj = w * qa[k];
              ex[k] = fmaf(wi, dx, ex[k]);
              ey[k] = fmaf(wi, dy, ey[k]);
              ez[k] = fmaf(wi, dz, ez[k]);
              cx = fmaf(wj, dx, cx);
              cy = fmaf(wj, dy, cy);
              cz = fmaf(wj, dz, cz);
            }
            tx = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(cx)));
            ty = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(cy)));
            tz = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(cz)));
          }
          {
            const float4 sj = sb2[m];
            float cx = ux, cy = uy, cz = uz;
#pragma unroll
            for (int k = 0; k < kSymTiles; ++k) {
              const float dx = r0[k] - sj.x, dy = r1[k] - sj.y, dz = r2[k] - sj.z;
              const float rr = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, s2k[k])));
              const float ri = __builtin_amdgcn_rsqf(rr);
              const float w = ri * (ri * ri);
              const float wi = w * sj.w, wj = w * qa[k];
              ex[k] = fmaf(wi, dx, ex[k]);
              ey[k] = fmaf(wi, dy, ey[k]);
              ez[k] = fmaf(wi, dz, ez[k]);
              cx = fmaf(wj, dx, cx);
              cy = fmaf(wj, dy, cy);
              cz = fmaf(wj, dz, cz);
            }
            ux = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(cx)));
            uy = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(cy)));
            uz = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(cz)));
          }
        }
      }
      const int jl = g + lane;
      J[wv][0][jl] = tx;
      J[wv][1][jl] = ty;
      J[wv][2][jl] = tz;
      J[wv][0][jl + 64] = ux;
      J[wv][1][jl + 64] = uy;
      J[wv][2][jl + 64] = uz;
    }
    __syncthreads();
    // field at the tile's sources from A: E_j = -sum_i q_i w (r_i - s_j),
    // the four waves' rows added in order
    if (tid < cnt) {
      const float fj = U ? -qA : -1.f;
      const size_t o = (size_t)dd * 3 * n + jt + tid;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float v = ((J[0][c][tid] + J[1][c][tid]) + J[2][c][tid]) + J[3][c][tid];
        Pj[o + (size_t)c * n] = fj * v;
      }
    }
  }
  const float fi = U ? qB : 1.f;
#pragma unroll
  for (int k = 0; k < kSymTiles; ++k) {
    const int i = a0 + k * kThreads + tid;
    if (i < n) {
      const size_t o = (size_t)dd * 3 * n + i;
      Pi[o] = fi * ex[k];
      Pi[o + (size_t)n] = fi * ey[k];
      Pi[o + 2 * (size_t)n] = fi * ez[k];
    }
  }
}

// The pair-once evaluation of few super-block pairs.  A workgroup of
// k_pair_sym is one long serial chain (2048 steps of 8 pairs a wave), so a
// launch of W workgroups takes about 600 us for any W up to 256, with the
// chip idle beside it.  Here each item (A, d) is cut in two roles: the sums
// for A's particles (a workgroup holds kSplitA of A's tiles and streams all
// of B) and the sums for B's (a workgroup streams kSplitB of B's tiles past
// all of A); one tile each measured 3 to 15 % faster than two.  Every pair is evaluated twice, 24 instead of 15 VALU
// operations, but the item is spread over 8 / kSplitA + 8 / kSplitB
// workgroups.  Each sum takes the same terms in the same order as in
// k_pair_sym, so the slots are the same bit for bit.
constexpr int kSplitA = 1;
constexpr int kSplitB = 1;
constexpr int kSplitParts = kSymTiles / kSplitA + kSymTiles / kSplitB;

// One group of 64 sources and one step of k_pair_sym's inner loop for KA
// tiles of A: into A's sums e (SUM_A) or the source's running sum c.
template <int KA, bool SUM_A, bool U>
__device__ __forceinline__ void sym_step(const float4 sj, const float (&r0)[KA], const float (&r1)[KA],
                                         const float (&r2)[KA], const float (&qa)[KA], const float (&s2k)[KA],
                                         float (&ex)[KA], float (&ey)[KA], float (&ez)[KA], float &cx, float &cy,
                                         float &cz) {
#pragma unroll
  for (int k = 0; k < KA; ++k) {
    const float dx = r0[k] - sj.x, dy = r1[k] - sj.y, dz = r2[k] - sj.z;
    const float rr = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, s2k[k])));
    const float ri = __builtin_amdgcn_rsqf(rr);
    const float w = ri * (ri * ri);
    if (SUM_A) {
      const float wi = U ? w : w * sj.w;
      ex[k] = fmaf(wi, dx, ex[k]);
      ey[k] = fmaf(wi, dy, ey[k]);
      ez[k] = fmaf(wi, dz, ez[k]);
    } else {
      const float wj = U ? w : w * qa[k];
      cx = fmaf(wj, dx, cx);
      cy = fmaf(wj, dy, cy);
      cz = fmaf(wj, dz, cz);
    }
  }
}

// A workgroup's share: tiles ka .. ka + KA - 1 of A against tiles bt0 .. bt0 +
// NB - 1 of B, one of the two sums.
template <int KA, int NB, bool SUM_A, bool NN>
__device__ __forceinline__ void sym_part(int n, const double *__restrict__ sx, const double *__restrict__ sy,
                                         const double *__restrict__ sz, const double *__restrict__ sq,
                                         const double *__restrict__ tbox, double nn_cut2d,
                                         const double *__restrict__ sb, float soft2, int A, int B, int dd, int ka,
                                         int bt0, float *__restrict__ Pi, float *__restrict__ Pj,
                                         float4 (*S)[128], float (*J)[3][kThreads]) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int nxt = ((lane + 1) & 63) << 2;
  const int a0 = A * kSymSB, b0 = B * kSymSB;
  const double *org = sym_origin(sb, A, B);
  const double c0 = org[0], c1 = org[1], c2 = org[2];
  float r0[KA], r1[KA], r2[KA], qa[KA], ex[KA], ey[KA], ez[KA];
  const float qA = (float)sq[a0], qB = (float)sq[b0];
#pragma unroll
  for (int k = 0; k < KA; ++k) {
    const int i = a0 + (ka + k) * kThreads + tid;
    const bool act = i < n;
    r0[k] = act ? (float)(sx[i] - c0) : 0.f;
    r1[k] = act ? (float)(sy[i] - c1) : 0.f;
    r2[k] = act ? (float)(sz[i] - c2) : 0.f;
    qa[k] = act ? (float)sq[i] : 0.f;
    ex[k] = ey[k] = ez[k] = 0.f;
  }
  // one charge on each side of the whole item
  bool uni = true;
#pragma unroll
  for (int k = 0; k < kSymTiles; ++k) {
    const int i = a0 + k * kThreads + tid, j = b0 + k * kThreads + tid;
    uni = uni && i < n && (float)sq[min(i, n - 1)] == qA && j < n && (float)sq[min(j, n - 1)] == qB;
  }
  const bool U = __syncthreads_and(uni);
  for (int bt = bt0; bt < bt0 + NB; ++bt) {
    const int jt = b0 + bt * kThreads;
    if (jt >= n) break;  // workgroup-uniform
    const int cnt = min(kThreads, n - jt);
    float s2k[KA];
#pragma unroll
    for (int k = 0; k < KA; ++k) {
      const bool direct = a0 + (ka + k) * kThreads < n &&
                          tile_pair_direct(tbox, sb, A * kSymTiles + ka + k, B * kSymTiles + bt, kSymTiles, NN, nn_cut2d);
      s2k[k] = direct ? 1e36f : soft2;
    }
    __syncthreads();  // the previous tile's S and J are consumed
    {
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (tid < cnt) {
        const int j = jt + tid;
        v = make_float4((float)(sx[j] - c0), (float)(sy[j] - c1), (float)(sz[j] - c2), (float)sq[j]);
      }
      S[tid >> 6][tid & 63] = v;
      S[tid >> 6][(tid & 63) + 64] = v;
    }
    __syncthreads();
    for (int g = 0; g < cnt; g += 128) {
      float tx = 0.f, ty = 0.f, tz = 0.f, ux = 0.f, uy = 0.f, uz = 0.f;
      const float4 *sa = &S[g >> 6][lane];
      const float4 *sb2 = &S[(g >> 6) + 1][lane];
      auto steps = [&](auto Uc) {
        constexpr bool UC = decltype(Uc)::value;
#pragma unroll 4
        for (int m = 0; m < 64; ++m) {
          sym_step<KA, SUM_A, UC>(sa[m], r0, r1, r2, qa, s2k, ex, ey, ez, tx, ty, tz);
          if (!SUM_A) {
            tx = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(tx)));
            ty = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(ty)));
            tz = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(tz)));
          }
          sym_step<KA, SUM_A, UC>(sb2[m], r0, r1, r2, qa, s2k, ex, ey, ez, ux, uy, uz);
          if (!SUM_A) {
            ux = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(ux)));
            uy = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(uy)));
            uz = __int_as_float(__builtin_amdgcn_ds_bpermute(nxt, __float_as_int(uz)));
          }
        }
      };
      if (U)
        steps(std::true_type());
      else
        steps(std::false_type());
      if (!SUM_A) {
        const int jl = g + lane;
        J[wv][0][jl] = tx;
        J[wv][1][jl] = ty;
        J[wv][2][jl] = tz;
        J[wv][0][jl + 64] = ux;
        J[wv][1][jl + 64] = uy;
        J[wv][2][jl + 64] = uz;
      }
    }
    if (!SUM_A) {
      __syncthreads();
      if (tid < cnt) {
        const float fj = U ? -qA : -1.f;
        const size_t o = (size_t)dd * 3 * n + jt + tid;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const float v = ((J[0][c][tid] + J[1][c][tid]) + J[2][c][tid]) + J[3][c][tid];
          Pj[o + (size_t)c * n] = fj * v;
        }
      }
    }
  }
  if (SUM_A) {
    const float fi = U ? qB : 1.f;
#pragma unroll
    for (int k = 0; k < KA; ++k) {
      const int i = a0 + (ka + k) * kThreads + tid;
      if (i < n) {
        const size_t o = (size_t)dd * 3 * n + i;
        Pi[o] = fi * ex[k];
        Pi[o + (size_t)n] = fi * ey[k];
        Pi[o + 2 * (size_t)n] = fi * ez[k];
      }
    }
  }
}

template <bool NN>
__global__ __launch_bounds__(kThreads, 4) void k_pair_sym_split(int n, const double *__restrict__ sx,
                                                              const double *__restrict__ sy,
                                                              const double *__restrict__ sz,
                                                              const double *__restrict__ sq,
                                                              const double *__restrict__ tbox, double nn_cut2d,
                                                              const double *__restrict__ sb, float soft2, int ns,
                                                              int d0, int dcnt, float *__restrict__ Pi,
                                                              float *__restrict__ Pj) {
  __shared__ float4 S[kThreads / 64][128];
  __shared__ float J[kThreads / 64][3][kThreads];
  const int item = (int)blockIdx.x / kSplitParts, part = (int)blockIdx.x % kSplitParts;
  const int A = item / dcnt, dd = item % dcnt, d = d0 + dd;
  if (d > sym_h(A, ns)) return;  // workgroup-uniform, before any barrier
  const int B = (A + d) % ns;
  constexpr int nA = kSymTiles / kSplitA;
  if (part < nA)
    sym_part<kSplitA, kSymTiles, true, NN>(n, sx, sy, sz, sq, tbox, nn_cut2d, sb, soft2, A, B, dd, part * kSplitA, 0, Pi,
                                           Pj, S, J);
  else
    sym_part<kSymTiles, kSplitB, false, NN>(n, sx, sy, sz, sq, tbox, nn_cut2d, sb, soft2, A, B, dd, 0,
                                            (part - nA) * kSplitB, Pi, Pj, S, J);
}

// Whether a launch of ns dcnt items takes the cut form: an item in parts adds
// 2.6 us to the launch, a launch of whole items takes about 600 us up to a
// quarter of the resident workgroups, so the line lies at 7/32 of them (224
// of 1024).  Whole calls with 7,568 cells: 5,001 charges 880 -> 360 us, 20,001
// 1237 -> 810 us, 40,001 (200 items) 1643 -> 1549 us; at 47,001 (253 items) the
// parts took 1821 us against 1790.
static bool sym_in_parts(int ns, int dcnt, int resident) { return (int64_t)ns * dcnt <= (int64_t)resident * 7 / 32; }

// acc[c][p] += the launch's slots that hold a field at p, in slot order: the
// slot of d as the owner of (A, A + d) and the slot of d as the partner of
// (A - d, A).
__global__ __launch_bounds__(256) void k_sym_reduce(int n, int sbsz, int ns, int d0, int dcnt,
                                                    const float *__restrict__ Pi, const float *__restrict__ Pj,
                                                    double *acc) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= n) return;
  const int A = p / sbsz;
  const int hA = sym_h(A, ns);
  // the three components side by side, so that six loads per slot are in
  // flight (each component keeps its order of additions)
  double s0 = acc[p], s1 = acc[(size_t)n + p], s2 = acc[2 * (size_t)n + p];
#pragma unroll 4
  for (int dd = 0; dd < dcnt; ++dd) {
    const int d = d0 + dd;
    const size_t o = (size_t)dd * 3 * n + p;
    if (d <= hA) {
      s0 += (double)Pi[o];
      s1 += (double)Pi[o + (size_t)n];
      s2 += (double)Pi[o + 2 * (size_t)n];
    }
    if (d <= sym_h((A - d + ns) % ns, ns)) {
      s0 += (double)Pj[o];
      s1 += (double)Pj[o + (size_t)n];
      s2 += (double)Pj[o + 2 * (size_t)n];
    }
  }
  acc[p] = s0;
  acc[(size_t)n + p] = s1;
  acc[2 * (size_t)n + p] = s2;
}

template <bool WANT_V, bool NN, int EXCL>
__device__ __forceinline__ void pair_fp64(int bx, int by, int n_t, const double *__restrict__ xs,
                                          const int32_t *__restrict__ perm, int n_s, const double *__restrict__ sx,
                                          const double *__restrict__ sy, const double *__restrict__ sz,
                                          const double *__restrict__ sq, const int8_t *__restrict__ species,
                                          const int8_t *__restrict__ species_s, double soft2, int chunk, double *part,
                                          double *nn_d2p, int32_t *nn_ip, const int32_t *__restrict__ self_map) {
  __shared__ double4 S[kThreads];
  __shared__ int K[kThreads];
  const int tid = threadIdx.x;
  const int i = bx * kThreads + tid;
  const bool active = i < n_t;
  const int ii = active ? i : 0;
  const double x0 = xs[ii], x1 = xs[(size_t)n_t + ii], x2 = xs[2 * (size_t)n_t + ii];
  int want = -2;
  if (NN && active) want = want_key(species[perm[i]]);
  const int self = active ? (self_map ? self_map[perm[i]] : perm[i]) : -1;
  const int jb = by * chunk;
  const int je = min(n_s, jb + chunk);
  double ex = 0.0, ey = 0.0, ez = 0.0, ev = 0.0;
  double best = INFINITY;
  int bidx = -1;
  for (int jt = jb; jt < je; jt += kThreads) {
    const int cnt = min(kThreads, je - jt);
    __syncthreads();
    if (tid < cnt) {
      const int j = jt + tid;
      S[tid] = make_double4(sx[j], sy[j], sz[j], sq[j]);
      if (NN) K[tid] = species_s[j];
    }
    __syncthreads();
    for (int jj = 0; jj < cnt; ++jj) {
      const double4 s = S[jj];
      const double dx = x0 - s.x, dy = x1 - s.y, dz = x2 - s.z;
      const double dd = fma(dx, dx, fma(dy, dy, dz * dz));
      const double rr = dd + soft2;
      double ri = inv_sqrt_f64(rr);
      if (EXCL == 1) ri = rr > 0.0 ? ri : 0.0;
      if (EXCL == 2) ri = (jt + jj == self) ? 0.0 : ri;
      const double qr = s.w * ri;
      const double w = qr * ri * ri;
      ex = fma(w, dx, ex);
      ey = fma(w, dy, ey);
      ez = fma(w, dz, ez);
      if (WANT_V) ev += qr;
      if (NN) {
        if (K[jj] == want && dd < best && (EXCL != 1 || rr > 0.0)) {
          best = dd;
          bidx = jt + jj;
        }
      }
    }
  }
  if (active) {
    const size_t o = (size_t)by * 4 * n_t;
    part[o + i] = ex;
    part[o + (size_t)n_t + i] = ey;
    part[o + 2 * (size_t)n_t + i] = ez;
    part[o + 3 * (size_t)n_t + i] = ev;
    if (NN) {
      nn_d2p[(size_t)by * n_t + i] = best;
      nn_ip[(size_t)by * n_t + i] = bidx;
    }
  }
}

template <bool WANT_V, bool NN, int EXCL>
__global__ __launch_bounds__(kThreads) void k_pair_fp64(int n_t, const double *__restrict__ xs,
                                                        const int32_t *__restrict__ perm, int n_s,
                                                        const double *__restrict__ sx, const double *__restrict__ sy,
                                                        const double *__restrict__ sz, const double *__restrict__ sq,
                                                        const int8_t *__restrict__ species,
                                                        const int8_t *__restrict__ species_s, double soft2, int chunk,
                                                        double *part, double *nn_d2p, int32_t *nn_ip,
                                                        const int32_t *__restrict__ self_map) {
  pair_fp64<WANT_V, NN, EXCL>(blockIdx.x, blockIdx.y, n_t, xs, perm, n_s, sx, sy, sz, sq, species, species_s, soft2, chunk, part,
            nn_d2p, nn_ip, self_map);
}

// Nearest partner over the source chunks: smallest distance, ties to the
// earlier chunk (lower source index).
template <typename DT>
__global__ __launch_bounds__(kSlotThreads) void k_nn_reduce(int n_t, int nsplit, const DT *__restrict__ nn_d2p,
                                                            const int32_t *__restrict__ nn_ip, double *nn_d2,
                                                            int32_t *nn_idx) {
  const int i = blockIdx.x * kSlotThreads + threadIdx.x;
  if (i >= n_t) return;
  DT best = INFINITY;
  int kb = -1;
#pragma unroll 8
  for (int k = 0; k < nsplit; ++k) {
    const DT d = nn_d2p[(size_t)k * n_t + i];
    if (d < best) {
      best = d;
      kb = k;
    }
  }
  nn_d2[i] = (double)best;
  nn_idx[i] = kb < 0 ? -1 : nn_ip[(size_t)kb * n_t + i];
}

// Terms of the tile pairs kept by the directed kernel (mask bits weighted
// by the two tiles' particle counts), added to *work; profiling only.
__global__ __launch_bounds__(256) void k_mask_work(int ntile, int wpr, int n, const uint32_t *__restrict__ mask,
                                                   unsigned long long *work) {
  const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
  unsigned long long w = 0;
  if (t < (size_t)ntile * wpr) {
    const int a = (int)(t / wpr), wd = (int)(t % wpr);
    const unsigned long long ca = (unsigned long long)min(kThreads, n - a * kThreads);
    uint32_t m = mask[t];
    while (m) {
      const int u = __builtin_ctz(m);
      m &= m - 1;
      const int b = wd * 32 + u;
      w += ca * (unsigned long long)min(kThreads, n - b * kThreads);
    }
  }
  if (w) atomicAdd(work, w);
}

template <bool WANT_V, bool NN, int CZ>
static void launch_pair_t(obem_ctx *ctx, dim3 grid, int n_t, const double *xs, const int32_t *perm, int n_s,
                          const double *sx, const double *sy, const double *sz, const double *sq,
                          const int8_t *sp, const int8_t *sps, double soft, obem_precision prec, int chunk,
                          double *part, void *nnd, int32_t *nni, const double *tbox, float nn_cut2,
                          const int32_t *self_map, int sym_tiles, double nn_cut2d, const uint32_t *dmask,
                          int dwpr) {
  if (prec == OBEM_MIXED)
    hipLaunchKernelGGL((k_pair_mixed<WANT_V, NN, CZ>), dim3(grid.x * grid.y), dim3(kThreads), 0, ctx->stream, n_t,
                       xs, perm, n_s,
                       sx, sy, sz, sq, sp, sps, (float)(soft * soft), chunk, part, (float *)nnd, nni, tbox, nn_cut2,
                       self_map, sym_tiles, nn_cut2d, dmask, dwpr);
  else
    hipLaunchKernelGGL((k_pair_fp64<WANT_V, NN, CZ>), grid, dim3(kThreads), 0, ctx->stream, n_t, xs, perm, n_s,
                       sx, sy, sz, sq, sp, sps, soft * soft, chunk, part, (double *)nnd, nni, self_map);
}

// Workgroups of k_pair_sym<nn> resident at once on the context's device.
static int sym_resident(obem_ctx *ctx, bool nn) {
  int &cache = nn ? ctx->sym_resident_nn : ctx->sym_resident;
  if (cache <= 0)
    cache = resident_workgroups(nn ? reinterpret_cast<const void *>(&k_pair_sym<true>)
                                   : reinterpret_cast<const void *>(&k_pair_sym<false>),
                                kThreads, ctx->device);
  return cache;
}

// Splits of the sources for n_t targets, and where the sums go.
struct PairPlan {
  int nsplit, chunk;
  double *part;
};
static obem_status pair_plan(obem_ctx *ctx, int n_t, int n_s, PairPlan *P) {
  const int bt = nblk(n_t);
  // about 128k workgroups (64 rounds of the 2048 resident ones), so that the
  // last workgroups to start are short and the chip drains quickly at the
  // end; chunks of at least one tile, of two where these fill the chip
  int nsplit = (kSplitWorkgroups + bt - 1) / bt;
  nsplit = std::max(1, std::min(nsplit, (n_s + kThreads - 1) / kThreads));
  if ((int64_t)bt * nsplit > kFewWorkgroups) nsplit = std::max(1, std::min(nsplit, (n_s + 511) / 512));
  nsplit = std::min(nsplit, max_slots(bt));
  int chunk = (n_s + nsplit - 1) / nsplit;
  chunk = (chunk + kThreads - 1) / kThreads * kThreads;
  nsplit = (n_s + chunk - 1) / chunk;
  double *part = (double *)ws_get(ctx, WS_PART, sizeof(double) * 4 * (size_t)n_t * nsplit);
  if (!part) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
  *P = PairPlan{nsplit, chunk, part};
  return OBEM_OK;
}

// soft == 0: drop zero-distance terms (1: the self term and coincident
// points); soft > 0 with targets = sources: only the potential needs the self
// term removed (2; its field term is exactly 0).
static int excluded(double soft, bool tgt_is_src, bool want_v) {
  if (!(soft > 0.0)) return 1;
  return tgt_is_src && want_v ? 2 : 0;
}

// Cells beyond the close zone and charges in one launch: workgroups below nc
// take a target tile and a range of cells, the others a target tile and a
// range of charges, each as its own kernel does.
template <bool FP64, bool WANT_V, int EXCL>
__global__ __launch_bounds__(kThreads) void k_cells_and_charges(
    int nc, int bt, int n_t, const double *__restrict__ xs, int N, const double *__restrict__ f,
    const double *__restrict__ sigma, int cchunk, double *cpart,
    const int32_t *__restrict__ perm, int n_s, const double *__restrict__ sx, const double *__restrict__ sy,
    const double *__restrict__ sz, const double *__restrict__ sq, double soft2, int chunk, double *ppart,
    const double *__restrict__ tbox, float cut2, double cut2d, const int32_t *__restrict__ self_map) {
  const int b = blockIdx.x, p = b - nc;
  if (FP64) {
    if (b < nc)
      panel_fp64<WANT_V>(b % bt, b / bt, n_t, xs, N, f, sigma, cchunk, cpart);
    else
      pair_fp64<WANT_V, false, EXCL>(p % bt, p / bt, n_t, xs, perm, n_s, sx, sy, sz, sq, nullptr, nullptr, soft2,
                                     chunk, ppart, nullptr, nullptr, self_map);
  } else {
    if (b < nc)
      panel_mixed<WANT_V>(b % bt, b / bt, n_t, xs, N, f, sigma, cchunk, cpart);
    else
      pair_mixed<WANT_V, false, EXCL>(p, n_t, xs, perm, n_s, sx, sy, sz, sq, nullptr, nullptr, (float)soft2, chunk,
                                      ppart, nullptr, nullptr, tbox, cut2, self_map, 0, cut2d, nullptr, 0);
  }
}

obem_status launch_pair_field(obem_ctx *ctx, int64_t n_src, const double *sx, const double *sy, const double *sz,
                              const double *sq, const TargetOrder &to, double soft, obem_precision prec,
                              bool tgt_is_src, bool want_v, const int8_t *species, const int8_t *species_s,
                              double *acc, int32_t *nn_idx, double *nn_d2, const double *tbox, double nn_cut,
                              const int32_t *self_map, bool once, Slots *slots) {
  const int n_t = to.n;
  const int n_s = (int)n_src;
  if (slots) *slots = Slots{acc, 0};
  if (n_t == 0 || n_s == 0) return OBEM_OK;
  if (once && slots) return fail(ctx, OBEM_EINVAL, "the pair-once evaluation adds its sums itself");
  if (once && !(tgt_is_src && n_s == n_t && tbox && pair_once_applies(n_t, prec, soft, want_v)))
    return fail(ctx, OBEM_EINVAL, "pair-once evaluation needs targets = sources in one order");
  const int bt = nblk(n_t);
  PairPlan P;
  obem_status pst = pair_plan(ctx, n_t, n_s, &P);
  if (pst) return pst;
  const int nsplit = P.nsplit, chunk = P.chunk;
  double *part = P.part;
  const bool nn = nn_idx != nullptr;
  void *nnd = nullptr;
  int32_t *nni = nullptr;
  if (nn) {
    nnd = ws_get(ctx, WS_NN, sizeof(double) * (size_t)n_t * nsplit);
    nni = (int32_t *)ws_get(ctx, WS_MISC7, sizeof(int32_t) * (size_t)n_t * nsplit);
    if (!nnd || !nni) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
  }
  const int excl = excluded(soft, tgt_is_src, want_v);
  dim3 grid(bt, nsplit);
  // cut with a margin for the FP32 box coordinates (a larger cut only costs time)
  const double nn_cut2d = tbox ? std::pow(nn_cut * (1.0 + 1e-4) + 1e-9, 2) : INFINITY;
  const float nn_cut2 = (float)nn_cut2d;
  const int sym_tiles = once ? kSymTiles : 0;
  const int ns = (n_t + kSymSB - 1) / kSymSB;
  double *sb = nullptr;
  uint32_t *dmask = nullptr;
  int dwpr = 0;
  if (once) {
    obem_status st = pair_once_setup(ctx, n_t, kSymTiles, tbox, nn, nn_cut2d, &sb, &dmask, &dwpr);
    if (st) return st;
    if (ctx->prof && ctx->work_dev) {
      const int ntile = nblk(n_t);
      const size_t nw = (size_t)ntile * dwpr;
      hipLaunchKernelGGL(k_mask_work, dim3((unsigned)((nw + 255) / 256)), dim3(256), 0, ctx->stream, ntile, dwpr,
                         n_t, dmask, ctx->work_dev);
      ctx->work_once_n2 += (int64_t)n_t * n_t;
    }
  } else if (ctx->prof) {
    ctx->work_directed += (int64_t)n_t * n_s;
  }
  {
  OBEM_PROF(ctx, "pair");
#define PAIR_CASE(V, N, Z)                                                                                   \
  if (want_v == V && nn == N && excl == Z)                                                                   \
    launch_pair_t<V, N, Z>(ctx, grid, n_t, to.xs, to.perm, n_s, sx, sy, sz, sq, species, species_s, soft, prec, \
                           chunk, part, nnd, nni, tbox, nn_cut2, self_map, sym_tiles, nn_cut2d, dmask, dwpr);
  PAIR_CASE(false, false, 0)
  PAIR_CASE(false, false, 1)
  PAIR_CASE(false, false, 2)
  PAIR_CASE(false, true, 0)
  PAIR_CASE(false, true, 1)
  PAIR_CASE(false, true, 2)
  PAIR_CASE(true, false, 0)
  PAIR_CASE(true, false, 1)
  PAIR_CASE(true, false, 2)
  PAIR_CASE(true, true, 0)
  PAIR_CASE(true, true, 1)
  PAIR_CASE(true, true, 2)
#undef PAIR_CASE
  }
  OBEM_HIP(ctx, hipGetLastError());
  // the accumulator already holds the cell field when the panel kernel ran
  {
    OBEM_PROF(ctx, "pair_reduce");
    if (slots)
      *slots = Slots{part, nsplit};
    else
      launch_slot_sum(ctx, n_t, 4, Slots{part, nsplit}, true, acc);
    const dim3 gn((n_t + kSlotThreads - 1) / kSlotThreads);
    if (nn && prec == OBEM_MIXED)
      hipLaunchKernelGGL(k_nn_reduce<float>, gn, dim3(kSlotThreads), 0, ctx->stream, n_t, nsplit, (const float *)nnd,
                         nni, nn_d2, nn_idx);
    else if (nn)
      hipLaunchKernelGGL(k_nn_reduce<double>, gn, dim3(kSlotThreads), 0, ctx->stream, n_t, nsplit, (const double *)nnd,
                         nni, nn_d2, nn_idx);
  }
  OBEM_HIP(ctx, hipGetLastError());
  if (once) {
    // the tile pairs between super-blocks, each evaluated once, in launches
    // of up to kSymSlots values of d (bounded partial buffers)
    const int hmax = ns / 2;
    if (hmax > 0) {
      OBEM_PROF(ctx, "pair_once");
      const float soft2 = (float)(soft * soft);
      obem_status st = run_pair_once(ctx, n_t, kSymSB, ns, sym_resident(ctx, nn), kSymSlots, acc,
                                     [&](int d0, int dcnt, float *pi, float *pj) {
#define SYM(K, G)                                                                                                     \
  hipLaunchKernelGGL(K, dim3(G), dim3(kThreads), 0, ctx->stream, n_t, sx, sy, sz, sq, tbox, nn_cut2d, sb, soft2, ns,   \
                     d0, dcnt, pi, pj)
                                       if (sym_in_parts(ns, dcnt, sym_resident(ctx, nn))) {
                                         const unsigned g = (unsigned)ns * dcnt * kSplitParts;
                                         if (nn)
                                           SYM(k_pair_sym_split<true>, g);
                                         else
                                           SYM(k_pair_sym_split<false>, g);
                                       } else {
                                         if (nn)
                                           SYM(k_pair_sym<true>, sym_grid(ns, dcnt));
                                         else
                                           SYM(k_pair_sym<false>, sym_grid(ns, dcnt));
                                       }
#undef SYM
                                     });
      if (st) return st;
    }
  }
  return OBEM_OK;
}

// Side by side where the two launches together have at most this many
// workgroups (target tiles x splits): alone, each leaves part of the chip idle
// or ends with a part of it idle.  Apart -> side by side, calls: 97 points,
// 4,096 cells and 1,000 charges (68 workgroups) 88 -> 68 us, 4,096 charges
// between plates in FP64 209 -> 200 us, 20,011 points, 40,776 cells and 200,003
// charges (10,112) 2.55 -> 2.42 ms.  Beyond the line mixed precision gains 1 % at
// 25,000 workgroups and loses 0.4 % at 100,000 (both kernels take the larger
// register count); FP64, 16,384 charges, gains 4 % on both sides of it (20,000
// points 5.50 -> 5.28 ms, 30,000 7.95 -> 7.67) and 2 % at 30,000 workgroups.
constexpr int64_t kSideBySide = 12288;

bool side_by_side(const obem_ctx *ctx, int64_t n_t, int64_t N, int64_t n_s) {
  const int bt = nblk(n_t), slots = max_slots(bt);
  const int64_t w = std::min<int64_t>(slots, (N + 63) / 64) + std::min<int64_t>(slots, (n_s + kThreads - 1) / kThreads);
  return !ctx->prof && bt * w <= kSideBySide;  // profiles time the two apart
}

obem_status launch_cells_and_charges(obem_ctx *ctx, const obem_meshh *m, const double *sigma, const SourceOrder &so,
                                     const TargetOrder &to, double soft, obem_precision prec, bool tgt_is_src,
                                     bool want_v, double *acc, Slots *cells, Slots *charges) {
  const int n_t = to.n, N = (int)m->n, n_s = (int)so.n;
  PanelPlan C;
  PairPlan P;
  obem_status st = panel_plan(ctx, n_t, N, acc, &C);
  if (!st) st = pair_plan(ctx, n_t, n_s, &P);
  if (st) return st;
  const int excl = excluded(soft, tgt_is_src, want_v);
  // no partner search: the cut of its tiles is that of launch_pair_field at 0
  const double cut2d = so.tbox ? 1e-18 : INFINITY;
  const int nc = C.bt * C.ns, np = C.bt * P.nsplit;
  const double soft2 = prec == OBEM_MIXED ? (double)(float)(soft * soft) : soft * soft;
#define BOTH(F, V, Z)                                                                                               \
  if ((prec == OBEM_FP64) == F && want_v == V && excl == Z)                                                         \
  hipLaunchKernelGGL((k_cells_and_charges<F, V, Z>), dim3(nc + np), dim3(kThreads), 0, ctx->stream, nc, C.bt, n_t,  \
                     to.xs, N, m->f, sigma, C.cchunk, C.part, to.perm, n_s, so.x, so.y, so.z, so.q, soft2,  \
                     P.chunk, P.part, so.tbox, (float)cut2d, cut2d, tgt_is_src ? so.inv : nullptr)
  BOTH(false, false, 0);
  BOTH(false, false, 1);
  BOTH(false, true, 0);
  BOTH(false, true, 1);
  BOTH(false, true, 2);
  BOTH(true, false, 0);
  BOTH(true, false, 1);
  BOTH(true, true, 0);
  BOTH(true, true, 1);
  BOTH(true, true, 2);
#undef BOTH
  launch_panel_close(ctx, m, sigma, to, prec, want_v, C);
  *cells = Slots{C.part, C.ns};
  *charges = Slots{P.part, P.nsplit};
  OBEM_HIP(ctx, hipGetLastError());
  return OBEM_OK;
}

// Up to 2^24 particles: the tile-pair mask takes at most 512 MB and the
// double-buffered partial slots 32 GB; larger sets keep the directed
// evaluation.
obem_status pair_once_setup(obem_ctx *ctx, int n, int sym_tiles, const double *tbox, bool nn, double cut2d,
                            double **sb, uint32_t **dmask, int *dwpr) {
  const int ns = (n + sym_tiles * kThreads - 1) / (sym_tiles * kThreads);
  const int ntile = nblk(n);
  *dwpr = (ntile + 31) / 32;
  *sb = (double *)ws_get(ctx, WS_SYMR, sizeof(double) * 4 * (size_t)ns);
  *dmask = (uint32_t *)ws_get(ctx, WS_SYMM, sizeof(uint32_t) * (size_t)ntile * *dwpr);
  if (!*sb || !*dmask) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
  hipLaunchKernelGGL(k_sym_radius, dim3((ns + 255) / 256), dim3(256), 0, ctx->stream, n, ns, sym_tiles, tbox, *sb);
  const size_t nw = (size_t)ntile * *dwpr;
  hipLaunchKernelGGL(k_tile_mask, dim3((unsigned)((nw + 255) / 256)), dim3(256), 0, ctx->stream, ntile, *dwpr,
                     sym_tiles, nn ? 1 : 0, cut2d, tbox, *sb, *dmask);
  OBEM_HIP(ctx, hipGetLastError());
  return OBEM_OK;
}

obem_status run_pair_once(obem_ctx *ctx, int n, int sbsz, int ns, int resident, int max_slots, double *acc,
                          const std::function<void(int, int, float *, float *)> &launch) {
  const int hmax = ns / 2;
  if (hmax <= 0) return OBEM_OK;
  // with more than one launch the slots are double-buffered: launch L's
  // slots are added to acc on the second stream while launch L + 1
  // evaluates into the other half (the additions stay in launch order, on
  // one stream, so the result does not depend on the overlap)
  const bool dbl = launch_slots(ns, hmax, resident, max_slots) < hmax;
  const size_t half = 3 * (size_t)std::min(max_slots, hmax) * n;
  float *Pi = (float *)ws_get(ctx, WS_SYMI, sizeof(float) * half * (dbl ? 2 : 1));
  float *Pj = (float *)ws_get(ctx, WS_SYMJ, sizeof(float) * half * (dbl ? 2 : 1));
  if (!Pi || !Pj) return fail(ctx, OBEM_ENOMEM, "workspace allocation failed");
  if (dbl) {
    obem_status st = aux_stream(ctx);
    if (st) return st;
  }
  int launch_no = 0;
  for (int d0 = 1, dcnt = 0; d0 <= hmax; d0 += dcnt, ++launch_no) {
    // equal workgroups run in rounds: at 32 values of d and 1954
    // super-blocks the last round of a launch held 64 of 1024
    dcnt = launch_slots(ns, hmax - d0 + 1, resident, max_slots);
    const int b = dbl ? (launch_no & 1) : 0;
    float *pi = Pi + b * half, *pj = Pj + b * half;
    if (dbl && launch_no >= 2) OBEM_HIP(ctx, hipStreamWaitEvent(ctx->stream, ctx->ev_free[b], 0));
    launch(d0, dcnt, pi, pj);
    OBEM_HIP(ctx, hipGetLastError());
    hipStream_t rs = ctx->stream;
    if (dbl) {
      OBEM_HIP(ctx, hipEventRecord(ctx->ev_slots[b], ctx->stream));
      OBEM_HIP(ctx, hipStreamWaitEvent(ctx->aux, ctx->ev_slots[b], 0));
      rs = ctx->aux;
    }
    hipLaunchKernelGGL(k_sym_reduce, dim3(nblk(n)), dim3(256), 0, rs, n, sbsz, ns, d0, dcnt, pi, pj, acc);
    OBEM_HIP(ctx, hipGetLastError());
    if (dbl) OBEM_HIP(ctx, hipEventRecord(ctx->ev_free[b], ctx->aux));
  }
  if (dbl) {
    OBEM_HIP(ctx, hipEventRecord(ctx->ev_join, ctx->aux));
    OBEM_HIP(ctx, hipStreamWaitEvent(ctx->stream, ctx->ev_join, 0));
  }
  return OBEM_OK;
}

bool pair_once_applies(int64_t n, obem_precision prec, double soft, bool want_v) {
  return prec == OBEM_MIXED && soft > 0.0 && !want_v && n > 2 * (int64_t)kSymSB && n <= ((int64_t)1 << 24);
}

// ---------------------------------------------------------------------------
// Scatter back to caller order, scaling by k_e
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_scatter(int n, const int32_t *__restrict__ perm, const double *__restrict__ acc,
                                                 double scale, double *Ex, double *Ey, double *Ez, double *V) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int j = perm[i];
  Ex[j] = scale * acc[i];
  Ey[j] = scale * acc[(size_t)n + i];
  Ez[j] = scale * acc[2 * (size_t)n + i];
  if (V) V[j] = scale * acc[3 * (size_t)n + i];
}

__global__ __launch_bounds__(256) void k_fill(size_t n, double *p, double v) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = v;
}

obem_status launch_scatter(obem_ctx *ctx, const TargetOrder &to, const double *acc, double scale, double *Ex,
                           double *Ey, double *Ez, double *V) {
  if (to.n == 0) return OBEM_OK;
  OBEM_PROF(ctx, "scatter");
  hipLaunchKernelGGL(k_scatter, dim3(nblk(to.n)), dim3(256), 0, ctx->stream, to.n, to.perm, acc, scale, Ex, Ey,
                     Ez, V);
  OBEM_HIP(ctx, hipGetLastError());
  return OBEM_OK;
}

obem_status launch_fill(obem_ctx *ctx, double *p, size_t n, double v) {
  if (n == 0) return OBEM_OK;
  hipLaunchKernelGGL(k_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, ctx->stream, n, p, v);
  OBEM_HIP(ctx, hipGetLastError());
  return OBEM_OK;
}

}  // namespace obem
