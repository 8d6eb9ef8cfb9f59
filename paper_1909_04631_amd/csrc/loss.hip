// Differentiable form: the S-BKI concentrations (Eq. (7)-(8) of Gan et al.,
// arXiv 1909.04631) at arbitrary labelled query points, the mean negative log
// predictive probability of their labels, and its adjoint with respect to the
// kernel length-scale l, the kernel scale sigma0 and every coordinate.
//
//   alpha_h^k = alpha0 + sum_t sigma0 f(r_ht) [y_t = k],  r = |x_t - x_h| / l < 1
//   loss      = -(1/H) sum_h log(alpha_h^{y_h} / S_h),     S_h = sum_k alpha_h^k
//   G_hk      = dloss/dalpha_hk = -(1/H)([k = y_h] / alpha_hk - 1/S_h)
//   dloss/dl      = sum over pairs  G_{h,y_t} sigma0 f'(r) (-r/l)
//   dloss/dsigma0 = sum_h sum_k G_hk (alpha_hk - alpha0) / sigma0      (closed form)
//   dloss/dx_t    = sum_h G_{h,y_t} sigma0 (f'(r)/r) (x_t - x_h) / l^2, dloss/dx_h = -(same)
//
// Rows and queries are bucketed in cells slightly larger than l, so a point's
// support lies in its own cell and the 26 around it.  Kernel weights are
// recomputed in the backward pass; nothing per pair is stored.  A query is
// owned by one wavefront, whose lanes take its rows, a training row by one lane;
// every sum is taken in a fixed order (deterministic, no floating-point atomics).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>

#include "smki_gather.h"
#include "smki_loss_layout.h"
#include "../../include/smki.h"

namespace {

// f'(r)/r = s^4 P(s), s = 1 - r: P is a relative degree-10 fit on s in [0, 1]
// (error 1.5e-8) of [f'(1 - s)/s^4]/(1 - s), the series f'(1 - s) = sum_{n>=2}
// (-1)^(n+1) (2n-2) (2 pi)^(2n) s^(2n) / (3 (2n)!) divided by s^4 r;
// kernel_poly.py derives it.  Highest degree first.
__constant__ float kG[11] = {0.826695529413764f,  0.8883087167660566f, -18.68107694361095f,
                             33.6151725453642f,   12.821709617420272f, -46.914955742370914f,
                             -50.511732012322824f, 70.73862871627226f, 70.64347982896255f,
                             -43.2927725732048f,  -43.292930014879026f};

struct LossArgs {
  BucketGeom g;
  const float4* pts;     // sorted records of the set being walked (label bits in .w)
  const int32_t* dense;
  const int32_t* prefix;
  const int32_t* sidx;   // sorted position -> original row (queries: training rows + query)
  int32_t planes, plane; // label planes of the sorted set, and the one that is walked
  float l, l2, inv_l, sigma0, alpha0;
  float coef[SMKI_POLY_N];  // sigma0 * Q (per-class form: Q, the class's sigma0 applied apart)
  int32_t K;
  int64_t H;
  const float4* cls;        // per-class form: [K] (l^2, 1/l, sigma0, l) of each class's kernel;
                            // l, l2 and inv_l above then hold the largest l (the search cut)
};

__device__ __forceinline__ float kernel_weight(const float* c, float s) {
  const float u = s * s;
  float q = c[0];
#pragma unroll
  for (int i = 1; i < SMKI_POLY_N; ++i) q = fmaf(q, u, c[i]);
  return (u * u) * (s * q);
}

__device__ __forceinline__ float dfdr_over_r(float s) {
  float p = kG[0];
#pragma unroll
  for (int i = 1; i < 11; ++i) p = fmaf(p, s, kG[i]);
  const float s2 = s * s;
  return (s2 * s2) * p;
}

// The cell of a coordinate, and how far (in cells, squared) the cells below and
// above it are: less a margin for the rounding of the cell index, which grows
// with it.  A cell edge is a little over l, so a cell at a squared distance of 1
// or more holds no row in the support: of the 27 cells around a point that
// leaves 21 on average.
struct Axis {
  int c;
  float lo2, hi2;
};
__device__ __forceinline__ Axis axis_of(float x, double inv_h, float h) {
  Axis a;
  const float f = floorf(quot_rn(x, inv_h, h));
  a.c = (int)f;
  const float u = (float)((double)x * inv_h - (double)f);   // in [0, 1], up to rounding
  const float m = 1e-3f + fabsf(f) * 0x1p-20f;
  const float lo = fmaxf(u - m, 0.0f), hi = fmaxf(1.0f - u - m, 0.0f);
  a.lo2 = lo * lo;
  a.hi2 = hi * hi;
  return a;
}
__device__ __forceinline__ float axis_dist2(const Axis& a, int o) {
  return o < 0 ? a.lo2 : (o > 0 ? a.hi2 : 0.0f);
}

// Header of a call (kHdr bytes): bounding-box copies (min x, y, z, max x, y, z,
// two unused), then the error word.
constexpr int kBoxCopies = 8;
constexpr size_t kErrOff = 480;
__global__ void __launch_bounds__(64) k_loss_header(int32_t* __restrict__ bbox,
                                                    uint32_t* __restrict__ err) {
  const int c = threadIdx.x & 7;
  bbox[threadIdx.x] = c < 3 ? INT32_MAX : (c < 6 ? INT32_MIN : 0);
  if (threadIdx.x < 4) err[threadIdx.x] = 0;
}

// Validation of both sets and the box of their cells.  Workgroups [0, gt) take
// the training rows, the rest the queries, in grid strides; a workgroup reduces
// its box and then updates one copy of it.  (One atomic per row on one box, as
// before, was bound by the atomics on six addresses: 3.2e6 rows 3.4 ms; the grid
// is capped so that each copy meets about a hundred updates.)
__global__ void __launch_bounds__(256) k_validate(const float* __restrict__ txyz,
                                                  const int32_t* __restrict__ tlab, int64_t nt,
                                                  int32_t gt, const float* __restrict__ qxyz,
                                                  const int32_t* __restrict__ qlab, int64_t nq,
                                                  int32_t K, float h, int32_t* __restrict__ bbox,
                                                  uint32_t* __restrict__ err) {
  const bool train = (int32_t)blockIdx.x < gt;
  const float* __restrict__ xyz = train ? txyz : qxyz;
  const int32_t* __restrict__ lab = train ? tlab : qlab;
  const int64_t n = train ? nt : nq;
  const int64_t b = train ? blockIdx.x : blockIdx.x - gt;
  const int64_t stride = (int64_t)(train ? gt : (int32_t)gridDim.x - gt) * blockDim.x;
  const double inv_h = 1.0 / (double)h;
  int32_t box[6] = {INT32_MAX, INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN, INT32_MIN};
  uint32_t e = 0;
  constexpr int U = 4;   // rows in flight per thread
  for (int64_t i0 = b * blockDim.x + threadIdx.x; i0 < n; i0 += U * stride) {
    float v[U][3];
    int32_t y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = min(i0 + u * stride, n - 1);   // (past the end: the last row again)
      v[u][0] = xyz[3 * i];
      v[u][1] = xyz[3 * i + 1];
      v[u][2] = xyz[3 * i + 2];
      y[u] = lab[i];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (y[u] < 0 || y[u] >= K) e |= DEVERR_LABEL;
      const bool fin = isfinite(v[u][0]) && isfinite(v[u][1]) && isfinite(v[u][2]);
      if (!fin) e |= DEVERR_NONFINITE;
      float c[3];
      bool in = fin;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        c[a] = floorf(quot_rn(v[u][a], inv_h, h));
        in = in && c[a] >= -(float)SMKI_COORD_LIM && c[a] < (float)SMKI_COORD_LIM;
      }
      if (fin && !in) e |= DEVERR_RANGE;
      if (in) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          box[a] = min(box[a], (int32_t)c[a]);
          box[3 + a] = max(box[3 + a], (int32_t)c[a]);
        }
      }
    }
  }
  if (e) atomicOr(err, e);
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int o = SMKI_WAVE / 2; o > 0; o >>= 1) {
      box[a] = min(box[a], __shfl_xor(box[a], o, SMKI_WAVE));
      box[3 + a] = max(box[3 + a], __shfl_xor(box[3 + a], o, SMKI_WAVE));
    }
  __shared__ int32_t part[256 / SMKI_WAVE][6];
  if ((threadIdx.x & (SMKI_WAVE - 1)) == 0)
    for (int a = 0; a < 6; ++a) part[threadIdx.x / SMKI_WAVE][a] = box[a];
  __syncthreads();
  if (threadIdx.x < 6) {
    const int a = threadIdx.x;
    int32_t v = part[0][a];
    for (int w = 1; w < 256 / SMKI_WAVE; ++w) v = a < 3 ? min(v, part[w][a]) : max(v, part[w][a]);
    int32_t* box_out = bbox + (blockIdx.x % kBoxCopies) * 8 + a;
    if (a < 3 && v != INT32_MAX) atomicMin(box_out, v);
    if (a >= 3 && v != INT32_MIN) atomicMax(box_out, v);
  }
}

// ---------------------------------------------------------------------------
// Query side: one wavefront per query, lanes over the rows around it.  A query
// meets 10^2 to 10^4 rows and every row is one 16-byte record, so what bounds
// these kernels is the latency of dependent loads: one lane per query, as
// before, walked them one after the other with a read-modify-write of global
// memory for each (room scene, 380 queries: 4.4 ms forward, now 0.02; LiDAR
// scan, 2.4e4 queries: 1.8 ms).
//
// The 27 cells are nine columns along z, each one run of sorted rows per block
// that it crosses: lanes 0..17 look the runs up together.  Lane i then takes
// rows i, i + 64, ... of the runs' concatenation.
// ---------------------------------------------------------------------------
constexpr int kRuns = 32;   // at most 18 used; a power of two for the search
struct RunTable {
  float4 at[kRuns];       // the point relative to the run's block centre; .w: first row minus
                          // the rows of the runs before it (as bits)
  int32_t incl[kRuns];    // rows up to and including the run; INT32_MAX past the last run
};

// Fills the table for point (x, y, z) (all 64 lanes); returns the rows in all runs.
__device__ __forceinline__ int32_t find_runs(const LossArgs& a, float x, float y, float z,
                                             RunTable& t) {
  const BucketGeom& g = a.g;
  const int lane = threadIdx.x;
  const double inv_h = 1.0 / (double)g.res;
  const Axis ax = axis_of(x, inv_h, g.res), ay = axis_of(y, inv_h, g.res),
             az = axis_of(z, inv_h, g.res);
  const int cx = ax.c, cy = ay.c, cz = az.c;
  const int col = lane >> 1, part = lane & 1;
  // the column's cells along z that the support reaches
  const float r2 = 1.0f - axis_dist2(ax, col / 3 - 1) - axis_dist2(ay, col % 3 - 1);
  const int zlo = az.lo2 < r2 ? cz - 1 : cz, zhi = az.hi2 < r2 ? cz + 1 : cz;
  const int vx = cx + col / 3 - 1, vy = cy + col % 3 - 1;
  const int bx = vx >> LLOG2B, by = vy >> LLOG2B, b0 = zlo >> LLOG2B, b1 = zhi >> LLOG2B;
  const int bz = part ? b1 : b0;
  const int z0 = part ? b1 * LB : zlo, z1 = part || b0 == b1 ? zhi : b0 * LB + LB - 1;
  const int px = bx - g.blo[0], py = by - g.blo[1], pz = bz - g.blo[2];
  int32_t first = 0, n = 0;
  if (lane < 18 && r2 > 0.0f && !(part && b0 == b1) && px >= 0 && py >= 0 && pz >= 0 && px < g.nb[0] &&
      py < g.nb[1] && pz < g.nb[2]) {
    const int32_t slot = a.dense[(((int64_t)px * g.nb[1] + py) * g.nb[2] + pz) * a.planes + a.plane];
    if (slot >= 0) {
      const int32_t c0 = ((vx - bx * LB) * LB + (vy - by * LB)) * LB - bz * LB;
      const int32_t* P = a.prefix + (int64_t)slot * (LB * LB * LB + 1);
      first = P[c0 + z0];
      n = P[c0 + z1 + 1] - first;
    }
  }
  int32_t inc = n;
#pragma unroll
  for (int o = 1; o < 32; o <<= 1) {
    const int32_t v = __shfl_up(inc, o, SMKI_WAVE);
    if (lane >= o) inc += v;
  }
  const uint64_t some = __ballot(n > 0);
  __syncthreads();   // (the previous point's table is no longer read)
  if (lane < kRuns && lane >= __popcll(some)) t.incl[lane] = INT32_MAX;
  if (n > 0) {
    const int k = __popcll(some & ((1ull << lane) - 1ull));
    const double h = (double)g.res;
    t.incl[k] = inc;
    // the point relative to the exact centre of block (bx, by, bz)
    t.at[k] = make_float4((float)((double)x - ((double)(bx * LB) + 0.5 * LB) * h),
                          (float)((double)y - ((double)(by * LB) + 0.5 * LB) * h),
                          (float)((double)z - ((double)(bz * LB) + 0.5 * LB) * h),
                          __int_as_float(first - (inc - n)));
  }
  __syncthreads();
  return __builtin_amdgcn_readlane(inc, 17);
}

// Visits the rows of the table, 64 at a time: fn(in, record, dx, dy, dz, d2) is
// called by every lane, in = this lane holds a row within the search cut.  The
// searches and loads of kAhead sets of 64 go out together: one set at a time,
// each waited for its chain of five LDS reads and a load (1.4 us a set where a
// query meets thousands of rows and few wavefronts run).
constexpr int kAhead = 4;
template <typename Fn>
__device__ __forceinline__ void for_rows(const LossArgs& a, const RunTable& t, int32_t total, Fn fn) {
  for (int32_t b = 0; b < total; b += kAhead * SMKI_WAVE) {
    int k[kAhead];
    float4 p[kAhead], q[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) k[u] = 0;
    // the run of row i: the first whose inclusive count exceeds it
#pragma unroll
    for (int st = kRuns / 2; st > 0; st >>= 1)
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
        if (t.incl[k[u] + st - 1] <= b + u * SMKI_WAVE + (int32_t)threadIdx.x) k[u] += st;
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int32_t i = b + u * SMKI_WAVE + (int32_t)threadIdx.x;
      p[u] = q[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (i < total) {
        q[u] = t.at[k[u]];
        p[u] = a.pts[__float_as_int(q[u].w) + i];
      }
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (b + u * SMKI_WAVE >= total) break;   // (uniform)
      const bool live = b + u * SMKI_WAVE + (int32_t)threadIdx.x < total;
      const float dx = p[u].x - q[u].x, dy = p[u].y - q[u].y, dz = p[u].z - q[u].z;
      const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
      fn(live && d2 < a.l2, p[u], dx, dy, dz, d2);
    }
  }
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = SMKI_WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, SMKI_WAVE);
  return v;
}

// Sums per class in LDS, spread over COLS columns: lanes l, l + COLS, ... share
// column l % COLS and take turns (a barrier of the one-wavefront workgroup
// between them), so each sum has one order.
template <typename T, int COLS>
__device__ __forceinline__ void class_add(T* bins, bool in, int32_t c, T v) {
  const int lane = threadIdx.x;
  if constexpr (COLS == SMKI_WAVE) {
    if (in) bins[c * COLS + lane] += v;
  } else {
#pragma unroll
    for (int r = 0; r < SMKI_WAVE / COLS; ++r) {
      if (in && lane / COLS == r) bins[c * COLS + lane % COLS] += v;
      __syncthreads();
    }
  }
}

// Sum of class c's columns in double (callers' lanes hold consecutive classes:
// the rotated order keeps their reads in different banks).
template <typename T, int COLS>
__device__ __forceinline__ double class_total(const T* bins, int32_t c) {
  double s = 0.0;
  for (int j = 0; j < COLS; ++j) s += (double)bins[c * COLS + ((j + c) & (COLS - 1))];
  return s;
}

// alpha at each query, in query order, and the query's term of the loss,
// log(alpha[h][y_h] / S_h).  PC: per-class kernels.
template <bool PC, int COLS>
__global__ void __launch_bounds__(SMKI_WAVE) k_alpha_q(LossArgs a, const float* __restrict__ qxyz,
                                                       const int32_t* __restrict__ qlab,
                                                       float* __restrict__ alpha_q,
                                                       double* __restrict__ term) {
  __shared__ RunTable t;
  extern __shared__ float bins[];   // [K][COLS]
  const int lane = threadIdx.x;
  for (int64_t h = blockIdx.x; h < a.H; h += gridDim.x) {
    for (int i = lane; i < a.K * COLS; i += SMKI_WAVE) bins[i] = 0.0f;
    const int32_t total = find_runs(a, qxyz[3 * h], qxyz[3 * h + 1], qxyz[3 * h + 2], t);
    for_rows(a, t, total, [&](bool in, const float4& p, float, float, float, float d2) {
      const int32_t y = __float_as_int(p.w);
      float v;
      if constexpr (PC) {
        const float4 c = a.cls[in ? y : 0];
        in = in && d2 < c.x;
        const float s = fmaxf(fmaf(-__builtin_sqrtf(d2), c.y, 1.0f), 0.0f);
        v = c.z * kernel_weight(a.coef, s);
      } else {
        const float s = fmaxf(fmaf(-__builtin_sqrtf(d2), a.inv_l, 1.0f), 0.0f);
        v = kernel_weight(a.coef, s);
      }
      class_add<float, COLS>(bins, in, y, v);
    });
    __syncthreads();
    const int32_t yh = qlab[h];
    double S = 0.0, ay = 0.0;
    for (int32_t k = lane; k < a.K; k += SMKI_WAVE) {
      const float v = (float)((double)a.alpha0 + class_total<float, COLS>(bins, k));
      alpha_q[h * a.K + k] = v;
      S += (double)v;
      if (k == yh) ay = (double)v;
    }
    S = wave_sum(S);
    ay = wave_sum(ay);   // (one lane holds it)
    if (lane == 0) term[h] = log(ay / S);
    __syncthreads();
  }
}

// Query-side adjoint: dloss/dx_h, (1/S_h, 1/alpha_y) for the training side, and
// the query's shares of the scalar gradients: dl_part[h] and, in closed form,
//   sum_k G_hk (alpha_hk - alpha0) / sigma0 = -(g/(H sigma0)) (K alpha0/S - alpha0/alpha_y),
// or (PC) dl[h][k] and ds[h][k] per class.
template <bool PC, int COLS>
__global__ void __launch_bounds__(SMKI_WAVE) k_query_grad(
    LossArgs a, int64_t n_train, const int32_t* __restrict__ n_near,
    const float* __restrict__ qxyz, const int32_t* __restrict__ qlab,
    const float* __restrict__ alpha_q, const float* __restrict__ gscale,
    float2* __restrict__ inv, float* __restrict__ grad_q, double* __restrict__ dl_part,
    double* __restrict__ dsig, double* __restrict__ dl, double* __restrict__ ds) {
  __shared__ RunTable t;
  extern __shared__ double dbins[];   // PC: [2][K][COLS]
  const int lane = threadIdx.x;
  const float gH = gscale[0] / (float)a.H;
  // queries in sorted order where the set holds them (n_near non-null: they
  // follow its training rows): the wavefronts in flight share rows
  const int64_t q0 = n_near ? *n_near : 0;
  for (int64_t j = blockIdx.x; j < a.H; j += gridDim.x) {
    const int64_t h = n_near ? a.sidx[q0 + j] - n_train : j;
    const int32_t yh = qlab[h];
    double S = 0.0;
    for (int32_t k = lane; k < a.K; k += SMKI_WAVE) S += (double)alpha_q[h * a.K + k];
    S = wave_sum(S);
    const double ay = (double)alpha_q[h * a.K + yh];
    const float is = (float)(1.0 / S), ia = (float)(1.0 / ay);
    double* DL = dbins;
    double* DS = dbins + (PC ? a.K * COLS : 0);
    if constexpr (PC)
      for (int i = lane; i < 2 * a.K * COLS; i += SMKI_WAVE) dbins[i] = 0.0;
    const int32_t total = find_runs(a, qxyz[3 * h], qxyz[3 * h + 1], qxyz[3 * h + 2], t);
    float gx = 0.f, gy = 0.f, gz = 0.f;
    double dlh = 0.0;
    for_rows(a, t, total, [&](bool in, const float4& p, float dx, float dy, float dz, float d2) {
      const int32_t yt = __float_as_int(p.w);
      float inv_l = a.inv_l, s0 = a.sigma0;
      if constexpr (PC) {
        const float4 c = a.cls[in ? yt : 0];
        in = in && d2 < c.x;
        inv_l = c.y;
        s0 = c.z;
      }
      const float G = -gH * ((yt == yh ? ia : 0.0f) - is);
      const float r = __builtin_sqrtf(d2) * inv_l;
      const float s = fmaxf(1.0f - r, 0.0f);
      const float gr = s0 * dfdr_over_r(s);                // sigma0 f'(r)/r
      if (in) {
        const float c = G * gr * (inv_l * inv_l);          // coefficient of (x_t - x_h)
        gx -= c * dx;
        gy -= c * dy;
        gz -= c * dz;
      }
      const double vl = (double)(-G * gr * r * r * inv_l);   // G sigma0 f'(r) (-r/l)
      if constexpr (PC) {
        class_add<double, COLS>(DL, in, yt, vl);
        class_add<double, COLS>(DS, in, yt, (double)(G * kernel_weight(a.coef, s)));
      } else if (in) {
        dlh += vl;
      }
    });
    gx = wave_sum(gx);
    gy = wave_sum(gy);
    gz = wave_sum(gz);
    if constexpr (PC) {
      __syncthreads();
      for (int32_t k = lane; k < a.K; k += SMKI_WAVE) {
        dl[h * a.K + k] = class_total<double, COLS>(DL, k);
        ds[h * a.K + k] = class_total<double, COLS>(DS, k);
      }
      __syncthreads();
    } else {
      dlh = wave_sum(dlh);
    }
    if (lane == 0) {
      inv[j] = make_float2(is, ia);
      if (grad_q) {
        grad_q[3 * h] = gx;
        grad_q[3 * h + 1] = gy;
        grad_q[3 * h + 2] = gz;
      }
      if constexpr (!PC) {
        const double g = (double)gscale[0];
        dl_part[h] = dlh;
        dsig[h] = -(g / ((double)a.H * (double)a.sigma0)) *
                  ((double)a.K * a.alpha0 / S - (double)a.alpha0 / ay);
      }
    }
  }
}

// Training-side adjoint: dloss/dx_t of the rows near a query, one lane per row in
// sorted order, walking the sorted queries around it: the rows of a wavefront
// lie in a few cells, so that they read the same cell tables and queries.  (One
// lane per row of the caller's order, with 27 table look-ups for each of the
// 3.1e6 rows, took 385 us; most rows have no query near and are zeroed when the
// near ones are picked.)  PC: per-class kernels,
//   dloss/dl_k      = sum over pairs with y_t = k  G_{h,k} sigma0_k f'(r) (-r/l_k)
//   dloss/dsigma0_k = sum over pairs with y_t = k  G_{h,k} f(r)
// (summed per query by k_query_grad, then per class in a fixed order).
template <bool PC>
__global__ void __launch_bounds__(256) k_train_grad(LossArgs a, const float* __restrict__ txyz,
                                                    const int32_t* __restrict__ tlab,
                                                    const int32_t* __restrict__ n_near,
                                                    const float2* __restrict__ inv,
                                                    const float* __restrict__ gscale,
                                                    float* __restrict__ grad_t) {
  const BucketGeom& g = a.g;
  const int32_t q0 = *n_near;   // the first query in sorted order
  const float gH = gscale[0] / (float)a.H;
  const double h = (double)g.res, inv_h = 1.0 / h;
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < q0;
       j += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = a.sidx[j];
    const float x = txyz[3 * t], y = txyz[3 * t + 1], z = txyz[3 * t + 2];
    const int32_t yt = tlab[t];
    float inv_l = a.inv_l, s0 = a.sigma0, l2 = a.l2;
    if constexpr (PC) {
      const float4 c = a.cls[yt];
      l2 = fminf(l2, c.x);
      inv_l = c.y;
      s0 = c.z;
    }
    const float il2 = inv_l * inv_l;
    const Axis ax = axis_of(x, inv_h, g.res), ay = axis_of(y, inv_h, g.res),
               az = axis_of(z, inv_h, g.res);
    const int cx = ax.c, cy = ay.c, cz = az.c;
    float gx = 0.f, gy = 0.f, gz = 0.f;
    for (int ox = -1; ox <= 1; ++ox) {
      // the runs of three columns, two blocks each: all look-ups in flight together
      const int vx = cx + ox, bx = vx >> LLOG2B, px = bx - g.blo[0];
      int32_t slot[6], S[6], E[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const int oy = k / 2 - 1, vy = cy + oy;
        const float r2 = 1.0f - axis_dist2(ax, ox) - axis_dist2(ay, oy);
        const int b0 = (az.lo2 < r2 ? cz - 1 : cz) >> LLOG2B, b1 = (az.hi2 < r2 ? cz + 1 : cz) >> LLOG2B;
        const int py = (vy >> LLOG2B) - g.blo[1], pz = (k & 1 ? b1 : b0) - g.blo[2];
        const bool in = r2 > 0.0f && px >= 0 && py >= 0 && pz >= 0 && px < g.nb[0] && py < g.nb[1] &&
                        pz < g.nb[2] && !((k & 1) && b0 == b1);
        slot[k] = in ? a.dense[(((int64_t)px * g.nb[1] + py) * g.nb[2] + pz) * a.planes + a.plane] : -1;
      }
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const int oy = k / 2 - 1, vy = cy + oy;
        const float r2 = 1.0f - axis_dist2(ax, ox) - axis_dist2(ay, oy);
        const int zlo = az.lo2 < r2 ? cz - 1 : cz, zhi = az.hi2 < r2 ? cz + 1 : cz;
        const int z0 = (k & 1 ? zhi : zlo) & ~(LB - 1);   // the block's first cell
        const int32_t c0 = ((vx - bx * LB) * LB + (vy & (LB - 1))) * LB;
        const int32_t* P = a.prefix + (int64_t)max(slot[k], 0) * (LB * LB * LB + 1) + c0;
        S[k] = P[max(zlo - z0, 0)];
        E[k] = slot[k] >= 0 ? P[min(zhi - z0, LB - 1) + 1] : S[k];
      }
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        if (S[k] >= E[k]) continue;
        const int oy = k / 2 - 1, by = (cy + oy) >> LLOG2B;
        const float r2 = 1.0f - axis_dist2(ax, ox) - axis_dist2(ay, oy);
        const int bz = ((k & 1) ? (az.hi2 < r2 ? cz + 1 : cz) : (az.lo2 < r2 ? cz - 1 : cz)) >> LLOG2B;
        // the row relative to the exact centre of block (bx, by, bz)
        const float tx = (float)((double)x - ((double)(bx * LB) + 0.5 * LB) * h);
        const float ty = (float)((double)y - ((double)(by * LB) + 0.5 * LB) * h);
        const float tz = (float)((double)z - ((double)(bz * LB) + 0.5 * LB) * h);
        for (int32_t i = S[k]; i < E[k]; ++i) {
          const float4 p = a.pts[i];   // a query record; (dx, dy, dz) = x_h - x_t
          const float dx = p.x - tx, dy = p.y - ty, dz = p.z - tz;
          const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
          if (!(d2 < l2)) continue;
          const float2 iv = inv[i - q0];
          const float G = -gH * ((yt == __float_as_int(p.w) ? iv.y : 0.0f) - iv.x);
          const float s = fmaxf(fmaf(-__builtin_sqrtf(d2), inv_l, 1.0f), 0.0f);
          const float c = G * s0 * dfdr_over_r(s) * il2;
          gx -= c * dx;
          gy -= c * dy;
          gz -= c * dz;
        }
      }
    }
    grad_t[3 * t] = gx;
    grad_t[3 * t + 1] = gy;
    grad_t[3 * t + 2] = gz;
  }
}

// Sums over queries in a fixed order (one workgroup each): thread t adds entries
// t, t + 1024, ..., then a tree over the threads.
constexpr int kSumThreads = 1024;
constexpr int64_t kFoldRows = 8192;
__device__ __forceinline__ double block_sum(double s) {
  __shared__ double part[kSumThreads];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int o = kSumThreads / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) part[threadIdx.x] += part[threadIdx.x + o];
    __syncthreads();
  }
  return part[0];
}

// loss = -(1/H) sum_h term[h]
__global__ void __launch_bounds__(kSumThreads) k_loss_value(const double* __restrict__ term,
                                                            int64_t H, float* __restrict__ loss) {
  double s = 0.0;
  for (int64_t h = threadIdx.x; h < H; h += kSumThreads) s += term[h];
  s = block_sum(s);
  if (threadIdx.x == 0) *loss = (float)(-s / (double)H);
}

// The first part of k_colsum2's sums for many queries, in place and in its order: thread
// (t, k) adds entries t, t + 1024, ... of class k into v[t][k], so that k_colsum2 has
// 1,024 entries left.  Lanes take consecutive entries of a row (a workgroup per class
// reads 8 bytes of each line that it loads: 3e5 queries of 255 classes 1,825 us for
// both, now 248 + 7).
__global__ void __launch_bounds__(256) k_colsum_fold(double* __restrict__ v0, bool use0,
                                                     double* __restrict__ v1, bool use1, int64_t H,
                                                     int32_t K) {
  const int64_t n = (int64_t)kSumThreads * K, i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= 2 * n || !(i < n ? use0 : use1)) return;
  double* v = (i < n ? v0 : v1) + (i < n ? i : i - n);   // (fewer than H rows: H > kSumThreads)
  double s = 0.0;
#pragma unroll 8
  for (int64_t e = 0; e * kSumThreads + (i < n ? i : i - n) / K < H; ++e) s += v[e * n];
  *v = s;
}

// out[k] = sum_h v[h][k], one workgroup per class: workgroups [0, K) sum v0, the
// next K sum v1 (a null output is skipped)
__global__ void __launch_bounds__(kSumThreads) k_colsum2(const double* __restrict__ v0,
                                                         float* __restrict__ out0,
                                                         const double* __restrict__ v1,
                                                         float* __restrict__ out1, int64_t H,
                                                         int32_t K) {
  const bool second = (int32_t)blockIdx.x >= K;
  const double* v = second ? v1 : v0;
  float* out = second ? out1 : out0;
  if (!out) return;   // (the whole workgroup)
  const int32_t k = (int32_t)blockIdx.x - (second ? K : 0);
  double s = 0.0;
  for (int64_t h = threadIdx.x; h < H; h += kSumThreads) s += v[h * K + k];
  s = block_sum(s);
  if (threadIdx.x == 0) out[k] = (float)s;
}

// The sums of [H][K] v0 and v1 over the queries (v0 and v1 may be overwritten).  Up to
// kFoldRows queries one launch (a backward of 5,000 queries of 20 classes 219 us, 231 with
// a second launch; of 10,000 240 and 223), above a fold first.
void launch_colsum2(double* v0, float* out0, double* v1, float* out1, int64_t H, int32_t K,
                    hipStream_t st) {
  if (K > 1 && H > kFoldRows) {
    hipLaunchKernelGGL(k_colsum_fold, dim3((unsigned)(2 * kSumThreads / 256 * K)), dim3(256), 0, st,
                       v0, out0 != nullptr, v1, out1 != nullptr, H, K);
    H = kSumThreads;
  }
  hipLaunchKernelGGL(k_colsum2, dim3(2 * K), dim3(kSumThreads), 0, st, (const double*)v0, out0,
                     (const double*)v1, out1, H, K);
}

inline unsigned nblk(int64_t n, int t) { return (unsigned)ceil_div_i64(n > 0 ? n : 1, t); }

smki_status err_status(uint32_t e) {
  if (e & (DEVERR_LABEL | DEVERR_NONFINITE)) return SMKI_E_BAD_INPUT;
  if (e & DEVERR_RANGE) return SMKI_E_RANGE;
  return SMKI_E_DEVICE;
}

constexpr int kValidateGrid = 1024;   // workgroups per set in the validation

constexpr unsigned kTrainGrid = 8192;   // workgroups of the training-side kernel (they stride)
constexpr int64_t kQueryGrid = 1 << 20;   // workgroups of the query-side kernels (they stride)

// The query-side kernels; few classes take a column per lane (float) or 16
// columns (double), many take fewer columns, so that the sums stay within 33 KB.
void launch_alpha_q(bool pc, const LossArgs& a, const float* qxyz, const int32_t* qlab, float* A,
                    double* term, hipStream_t st) {
  const dim3 grid((unsigned)std::min<int64_t>(a.H, kQueryGrid)), block(SMKI_WAVE);
  const bool few = a.K <= 64;
  const unsigned lds = (unsigned)(sizeof(float) * a.K * (few ? 64 : 16));
  if (pc && few)
    hipLaunchKernelGGL((k_alpha_q<true, 64>), grid, block, lds, st, a, qxyz, qlab, A, term);
  else if (pc)
    hipLaunchKernelGGL((k_alpha_q<true, 16>), grid, block, lds, st, a, qxyz, qlab, A, term);
  else if (few)
    hipLaunchKernelGGL((k_alpha_q<false, 64>), grid, block, lds, st, a, qxyz, qlab, A, term);
  else
    hipLaunchKernelGGL((k_alpha_q<false, 16>), grid, block, lds, st, a, qxyz, qlab, A, term);
}

void launch_query_grad(bool pc, const LossArgs& a, const float* qxyz, const int32_t* qlab,
                       const float* alpha_q, const float* gscale, const LossBufs& b, int64_t n_train,
                       bool sorted, float* grad_q, hipStream_t st) {
  const int32_t* nn = sorted ? b.n_near : nullptr;
  const dim3 grid((unsigned)std::min<int64_t>(a.H, kQueryGrid)), block(SMKI_WAVE);
  if (!pc) {
    hipLaunchKernelGGL((k_query_grad<false, 16>), grid, block, 0, st, a, n_train, nn, qxyz, qlab,
                       alpha_q, gscale, b.inv, grad_q, b.dl, b.dsig, b.dlk, b.dsk);
    return;
  }
  const bool few = a.K <= 64;
  const unsigned lds = (unsigned)(2 * sizeof(double) * a.K * (few ? 16 : 8));
  if (few)
    hipLaunchKernelGGL((k_query_grad<true, 16>), grid, block, lds, st, a, n_train, nn, qxyz, qlab,
                       alpha_q, gscale, b.inv, grad_q, b.dl, b.dsig, b.dlk, b.dsk);
  else
    hipLaunchKernelGGL((k_query_grad<true, 8>), grid, block, lds, st, a, n_train, nn, qxyz, qlab,
                       alpha_q, gscale, b.inv, grad_q, b.dl, b.dsig, b.dlk, b.dsk);
}

char* align_up(char* p) { return (char*)(((uintptr_t)p + kAl - 1) / kAl * kAl); }

// Validate both sets and size the grid (synchronous); then carve the body from
// the caller's workspace or a fresh allocation, and bucket the training rows
// near a query (and the queries if both_sets; grad_train, nullable, is zeroed at
// the rows left out).
// h_cls (nullable): per-class kernel table, copied into the header before the
// synchronisation (so the host array may go out of scope after the call).
smki_status prepare(const float* txyz, const int32_t* tlab, int64_t nt, const float* qxyz,
                    const int32_t* qlab, int64_t nq, float l, int32_t K, bool both_sets,
                    float* grad_train, char* ws, size_t ws_bytes, char** own, LossBufs& b, BucketGeom& g,
                    hipStream_t st, const float4* h_cls = nullptr) {
  const float h = (float)((double)l * (1.0 + 1.0 / 1024.0));
  char* hdr = ws ? align_up(ws) : nullptr;
  if (ws && ws_bytes < kHdr + kAl) return SMKI_E_CAPACITY;
  if (!ws) {
    SMKI_HIP_TRY(hipMallocAsync((void**)own, kHdr, st));
    hdr = *own;
  }
  b.bbox = (int32_t*)hdr;
  b.err = (uint32_t*)(hdr + kErrOff);
  b.dn = (int64_t*)(hdr + kCountOff);
  b.n_near = (int32_t*)(hdr + kCountOff + sizeof(int64_t));
  b.cls = (float4*)(hdr + 512);
  if (h_cls)
    SMKI_HIP_TRY(hipMemcpyAsync(b.cls, h_cls, sizeof(float4) * K, hipMemcpyHostToDevice, st));
  const int32_t gt = (int32_t)std::min<int64_t>(nt > 0 ? nblk(nt, 256) : 0, kValidateGrid),
                gq = (int32_t)std::min<int64_t>(nblk(nq, 256), kValidateGrid);
  hipLaunchKernelGGL(k_loss_header, dim3(1), dim3(64), 0, st, b.bbox, b.err);
  hipLaunchKernelGGL(k_validate, dim3(gt + gq), dim3(256), 0, st, txyz, tlab, nt, gt, qxyz, qlab,
                     nq, K, h, b.bbox, b.err);
  SMKI_HIP_TRY(hipGetLastError());
  char hh[512];   // the boxes and the error word, in one copy
  SMKI_HIP_TRY(hipMemcpyAsync(hh, hdr, sizeof(hh), hipMemcpyDeviceToHost, st));
  SMKI_HIP_TRY(stream_wait(st));
  uint32_t e = 0;
  memcpy(&e, hh + kErrOff, sizeof(e));
  if (e) return err_status(e);
  int32_t hb[8] = {INT32_MAX, INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN, INT32_MIN, 0, 0};
  for (int c = 0; c < kBoxCopies; ++c) {
    int32_t box[8];
    memcpy(box, hh + c * sizeof(box), sizeof(box));
    for (int a = 0; a < 3; ++a) {
      hb[a] = std::min(hb[a], box[a]);
      hb[3 + a] = std::max(hb[3 + a], box[3 + a]);
    }
  }
  g = BucketGeom{};
  g.planes = both_sets ? 2 : 1;
  g.res = h;
  g.B = LB;
  g.log2B = LLOG2B;
  g.n_blocks = 1;
  for (int a = 0; a < 3; ++a) {
    const int32_t lo = (hb[a] - 1) >> LLOG2B, hi = (hb[3 + a] + 1) >> LLOG2B;
    g.blo[a] = lo;
    g.nb[a] = hi - lo + 1;
    g.n_blocks *= g.nb[a];
  }
  if (g.n_blocks > kMaxLossBlocks) return SMKI_E_CAPACITY;
  int bits = 0;
  while (bits < 62 && (int64_t(1) << bits) < g.n_blocks * g.planes) ++bits;
  g.key_bits = std::max(1, bits + 3 * LLOG2B);
  const size_t body = body_bytes(nt, nq, K, g.n_blocks);
  const size_t with_near = carve_body(nullptr, b, nt, nq, K, g.n_blocks, true);
  char* bbase = nullptr;
  bool near = true;
  if (ws) {
    bbase = align_up(hdr + kHdr);
    if ((size_t)(bbase - ws) + body > ws_bytes) return SMKI_E_CAPACITY;
    near = (size_t)(bbase - ws) + with_near <= ws_bytes;
  } else {
    char* p = nullptr;
    SMKI_HIP_TRY(hipMallocAsync((void**)&p, with_near, st));
    own[1] = p;
    bbase = align_up(p);
  }
  carve_body(bbase, b, nt, nq, K, g.n_blocks, near);
  SMKI_HIP_TRY(bucket_near(txyz, tlab, nt, qxyz, qlab, nq, both_sets, g, b.ps, b.scr, b.near,
                           grad_train, b.dn, b.n_near, b.err, st));
  return SMKI_OK;
}

void release(char** own, hipStream_t st) {
  for (int i = 0; i < 2; ++i)
    if (own[i]) (void)hipFreeAsync(own[i], st);
}

LossArgs make_args(const BucketGeom& g, const LossBufs& b, int32_t plane, float l, float sigma0,
                   float alpha0, int32_t K, int64_t H) {
  LossArgs a{};
  a.g = g;
  a.pts = b.ps.pts;
  a.dense = b.ps.dense;
  a.prefix = b.ps.prefix;
  a.sidx = (const int32_t*)b.scr.idx;
  a.planes = g.planes;
  a.plane = plane;
  a.l = l;
  a.l2 = l * l;
  a.inv_l = 1.0f / l;
  a.sigma0 = sigma0;
  a.alpha0 = alpha0;
  for (int i = 0; i < SMKI_POLY_N; ++i) a.coef[i] = (float)(kSmkiQ[i] * (double)sigma0);
  a.K = K;
  a.H = H;
  return a;
}

bool bad_params(int64_t nt, int64_t nq, float l, float sigma0, float alpha0, int32_t K) {
  return nt < 0 || nq <= 0 || !(std::isfinite(l) && l > 0) || !(std::isfinite(sigma0) && sigma0 > 0) ||
         !(std::isfinite(alpha0) && alpha0 > 0) || K < 2 || K > 255 ||
         nt > (int64_t)INT32_MAX / 2 || nq > (int64_t)INT32_MAX / 2;
}

}  // namespace

extern "C" size_t smki_loss_workspace_bytes(int64_t n_train, int64_t n_query, int32_t K) {
  return kHdr + 2 * kAl + body_bytes(std::max<int64_t>(n_train, 0), std::max<int64_t>(n_query, 1),
                                     std::max(K, 1), kMaxLossBlocks);
}

extern "C" smki_status smki_loss_forward(const float* txyz, const int32_t* tlab, int64_t nt,
                                         const float* qxyz, const int32_t* qlab, int64_t nq,
                                         float l, float sigma0, float alpha0, int32_t K,
                                         void* hip_stream, void* workspace, size_t ws_bytes,
                                         float* loss, float* alpha_q) {
  if (bad_params(nt, nq, l, sigma0, alpha0, K) || !qxyz || !qlab || !loss ||
      (nt > 0 && (!txyz || !tlab)))
    return SMKI_E_INVALID_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  char* own[2] = {nullptr, nullptr};
  LossBufs b{};
  BucketGeom g{};
  smki_status rc = prepare(txyz, tlab, nt, qxyz, qlab, nq, l, K, false, nullptr, (char*)workspace,
                           ws_bytes, own, b, g, st);
  if (rc == SMKI_OK) {
    const LossArgs a = make_args(g, b, 0, l, sigma0, alpha0, K, nq);
    float* A = alpha_q ? alpha_q : b.alpha_q;
    launch_alpha_q(false, a, qxyz, qlab, A, b.dl, st);
    hipLaunchKernelGGL(k_loss_value, dim3(1), dim3(kSumThreads), 0, st, (const double*)b.dl, nq,
                       loss);
    if (hipGetLastError() != hipSuccess) rc = SMKI_E_DEVICE;
  }
  release(own, st);
  return rc;
}

extern "C" smki_status smki_loss_backward(const float* txyz, const int32_t* tlab, int64_t nt,
                                          const float* qxyz, const int32_t* qlab, int64_t nq,
                                          float l, float sigma0, float alpha0, int32_t K,
                                          void* hip_stream, void* workspace, size_t ws_bytes,
                                          const float* alpha_q, const float* grad_loss,
                                          float* grad_l, float* grad_sigma0, float* grad_train,
                                          float* grad_query) {
  if (bad_params(nt, nq, l, sigma0, alpha0, K) || !qxyz || !qlab || !alpha_q || !grad_loss ||
      (nt > 0 && (!txyz || !tlab)))
    return SMKI_E_INVALID_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  char* own[2] = {nullptr, nullptr};
  LossBufs b{};
  BucketGeom g{};
  smki_status rc = prepare(txyz, tlab, nt, qxyz, qlab, nq, l, K, grad_train != nullptr,
                           grad_train, (char*)workspace, ws_bytes, own, b, g, st);
  if (rc == SMKI_OK) {
    const LossArgs aq = make_args(g, b, 0, l, sigma0, alpha0, K, nq);
    launch_query_grad(false, aq, qxyz, qlab, alpha_q, grad_loss, b, nt, grad_train != nullptr,
                      grad_query, st);
    if (grad_l || grad_sigma0)
      launch_colsum2(b.dl, grad_l, b.dsig, grad_sigma0, nq, 1, st);
    if (grad_train && nt > 0) {
      const LossArgs at = make_args(g, b, 1, l, sigma0, alpha0, K, nq);
      hipLaunchKernelGGL(k_train_grad<false>, dim3(std::min(nblk(nt, 256), kTrainGrid)), dim3(256),
                         0, st, at, txyz, tlab, (const int32_t*)b.n_near, (const float2*)b.inv,
                         grad_loss, grad_train);
    }
    if (hipGetLastError() != hipSuccess) rc = SMKI_E_DEVICE;
  }
  release(own, st);
  return rc;
}

// ---------------------------------------------------------------------------
// per-class kernels (l_k, sigma0_k per class)
// ---------------------------------------------------------------------------
namespace {

// Host table of the class kernels and the largest l; false if a value is invalid.
bool class_table(const float* l, const float* sigma0, int32_t K, float4* t, float* lmax) {
  if (!l || !sigma0 || K < 2 || K > 255) return false;
  *lmax = 0.0f;
  for (int32_t k = 0; k < K; ++k) {
    if (!(std::isfinite(l[k]) && l[k] > 0) || !(std::isfinite(sigma0[k]) && sigma0[k] > 0))
      return false;
    t[k] = make_float4(l[k] * l[k], 1.0f / l[k], sigma0[k], l[k]);
    *lmax = std::max(*lmax, l[k]);
  }
  return true;
}

LossArgs make_args_pc(const BucketGeom& g, const LossBufs& b, int32_t plane, float lmax,
                      const float4* cls, float alpha0, int32_t K, int64_t H) {
  LossArgs a = make_args(g, b, plane, lmax, 1.0f, alpha0, K, H);   // coef = Q: sigma0_k applied per row
  a.cls = cls;
  return a;
}

}  // namespace

extern "C" smki_status smki_loss_forward_classes(const float* txyz, const int32_t* tlab,
                                                 int64_t nt, const float* qxyz,
                                                 const int32_t* qlab, int64_t nq, const float* l,
                                                 const float* sigma0, float alpha0, int32_t K,
                                                 void* hip_stream, void* workspace,
                                                 size_t ws_bytes, float* loss, float* alpha_q) {
  float4 tab[256];
  float lmax = 0.0f;
  if (!class_table(l, sigma0, K, tab, &lmax) || bad_params(nt, nq, lmax, 1.0f, alpha0, K) ||
      !qxyz || !qlab || !loss || (nt > 0 && (!txyz || !tlab)))
    return SMKI_E_INVALID_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  char* own[2] = {nullptr, nullptr};
  LossBufs b{};
  BucketGeom g{};
  smki_status rc = prepare(txyz, tlab, nt, qxyz, qlab, nq, lmax, K, false, nullptr, (char*)workspace,
                           ws_bytes, own, b, g, st, tab);
  if (rc == SMKI_OK) {
    const LossArgs a = make_args_pc(g, b, 0, lmax, b.cls, alpha0, K, nq);
    float* A = alpha_q ? alpha_q : b.alpha_q;
    launch_alpha_q(true, a, qxyz, qlab, A, b.dl, st);
    hipLaunchKernelGGL(k_loss_value, dim3(1), dim3(kSumThreads), 0, st, (const double*)b.dl, nq,
                       loss);
    if (hipGetLastError() != hipSuccess) rc = SMKI_E_DEVICE;
  }
  release(own, st);
  return rc;
}

extern "C" smki_status smki_loss_backward_classes(
    const float* txyz, const int32_t* tlab, int64_t nt, const float* qxyz, const int32_t* qlab,
    int64_t nq, const float* l, const float* sigma0, float alpha0, int32_t K, void* hip_stream,
    void* workspace, size_t ws_bytes, const float* alpha_q, const float* grad_loss, float* grad_l,
    float* grad_sigma0, float* grad_train, float* grad_query) {
  float4 tab[256];
  float lmax = 0.0f;
  if (!class_table(l, sigma0, K, tab, &lmax) || bad_params(nt, nq, lmax, 1.0f, alpha0, K) ||
      !qxyz || !qlab || !alpha_q || !grad_loss || (nt > 0 && (!txyz || !tlab)))
    return SMKI_E_INVALID_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  char* own[2] = {nullptr, nullptr};
  LossBufs b{};
  BucketGeom g{};
  smki_status rc = prepare(txyz, tlab, nt, qxyz, qlab, nq, lmax, K, grad_train != nullptr,
                           grad_train, (char*)workspace, ws_bytes, own, b, g, st, tab);
  if (rc == SMKI_OK) {
    const LossArgs aq = make_args_pc(g, b, 0, lmax, b.cls, alpha0, K, nq);
    launch_query_grad(true, aq, qxyz, qlab, alpha_q, grad_loss, b, nt, grad_train != nullptr,
                      grad_query, st);
    if (grad_l || grad_sigma0)
      launch_colsum2(b.dlk, grad_l, b.dsk, grad_sigma0, nq, K, st);
    if (grad_train && nt > 0) {
      const LossArgs at = make_args_pc(g, b, 1, lmax, b.cls, alpha0, K, nq);
      hipLaunchKernelGGL(k_train_grad<true>, dim3(std::min(nblk(nt, 256), kTrainGrid)), dim3(256),
                         0, st, at, txyz, tlab, (const int32_t*)b.n_near, (const float2*)b.inv,
                         grad_loss, grad_train);
    }
    if (hipGetLastError() != hipSuccess) rc = SMKI_E_DEVICE;
  }
  release(own, st);
  return rc;
}

// ---------------------------------------------------------------------------
// the predictive loss without any allocation: a fixed device array as workspace
// ---------------------------------------------------------------------------
namespace {

// Workspace of smki_loss_forward_noalloc.  Each device the library runs on
// holds its own copy until the process ends.  Host code never passes this
// name to a kernel or a copy: it stands in for the array on the host side;
// the device address comes from hipGetSymbolAddress (static_scratch below).
constexpr size_t kStaticScratchBytes = SMKI_LOSS_NOALLOC_BYTES;
static __device__ __align__(256) char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char* g_scratch_ptr[kMaxDevices] = {};

// Device address of the current device's copy of `scratch`, looked up once per
// device (with that device current) and kept.
smki_status static_scratch(char** out) {
  int dev = -1;
  SMKI_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return SMKI_E_DEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    SMKI_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return SMKI_E_DEVICE;
    g_scratch_ptr[dev] = (char*)p;
  }
  *out = g_scratch_ptr[dev];
  return SMKI_OK;
}

}  // namespace

extern "C" smki_status smki_loss_forward_noalloc(const float* txyz, const int32_t* tlab,
                                                 int64_t nt, const float* qxyz,
                                                 const int32_t* qlab, int64_t nq, float l,
                                                 float sigma0, float alpha0, int32_t K,
                                                 void* hip_stream, float* loss, float* alpha_q) {
  if (bad_params(nt, nq, l, sigma0, alpha0, K) || !qxyz || !qlab || !loss ||
      (nt > 0 && (!txyz || !tlab)))
    return SMKI_E_INVALID_ARG;
  // the buffers that do not depend on the grid must fit before anything runs;
  // the grid-dependent tables are checked once the grid is known
  if (kHdr + 2 * kAl + body_bytes(nt, nq, K, 1) > kStaticScratchBytes)
    return SMKI_E_CAPACITY;
  char* ws = nullptr;
  const smki_status rc = static_scratch(&ws);
  if (rc != SMKI_OK) return rc;
  return smki_loss_forward(txyz, tlab, nt, qxyz, qlab, nq, l, sigma0, alpha0, K, hip_stream, ws,
                           kStaticScratchBytes, loss, alpha_q);
}
