// Training-set construction and spatial bucketing.
//
// Rows of the training set (Sec. III and IV of Gan et al., arXiv 1909.04631):
// every labelled hit, plus free-space points interpolated along its beam and
// labelled with the free class.  The free-sample positions and the voxel index
// of every row follow a binary32 contract (each operation rounded once, no
// fused multiply-add), so that cell keys are bit-reproducible.
//
// Bucketing: rows are keyed by (map block, voxel inside the block) over a dense
// grid of the blocks that the scan's bounding box covers, radix sorted, and
// stored as float4 records (x, y, z relative to the exact centre of the row's
// own block; label bits).  A per-block prefix table of B^3 + 1 entries maps
// any voxel range inside a block to a contiguous row range.
#include "smki_bucket.h"
#include "smki_plan.h"

#pragma clang fp contract(off)

// Correctly rounded binary32 division and square root: the double-precision
// result rounded once to binary32 is the correctly rounded binary32 result
// (53 >= 2*24 + 2, so the double rounding is innocuous).
__device__ __forceinline__ float div_rn(float a, float b) { return (float)((double)a / (double)b); }
__device__ __forceinline__ float sqrt_rn(float a) { return (float)sqrt((double)a); }

// ---------------------------------------------------------------------------
// binary32 beam arithmetic (reading of the paper's free-space sampling):
//   v = p - o ; L = sqrt((vx*vx + vy*vy) + vz*vz) ; n = ceil(L/s) - 1 ;
//   q_j = o + (((float)j * s) / L) * v
// ---------------------------------------------------------------------------
__device__ __forceinline__ float beam_len(float px, float py, float pz, float ox, float oy,
                                          float oz, float* vx, float* vy, float* vz) {
  *vx = px - ox;
  *vy = py - oy;
  *vz = pz - oz;
  const float xx = *vx * *vx, yy = *vy * *vy, zz = *vz * *vz;
  const float a = xx + yy;
  const float L2 = a + zz;
  return sqrt_rn(L2);
}

__device__ __forceinline__ int voxel_index(float x, double inv_res, float res, int32_t* out) {
  const float f = floorf(quot_rn(x, inv_res, res));
  if (!(f >= -(float)SMKI_COORD_LIM && f < (float)SMKI_COORD_LIM)) return 0;
  *out = (int32_t)f;
  return 1;
}

__device__ __forceinline__ bool finite3(float x, float y, float z) {
  return isfinite(x) && isfinite(y) && isfinite(z);
}

// Which scan a hit belongs to (scan_off has S+1 entries, S >= 1).
__device__ __forceinline__ int32_t scan_of(const int64_t* scan_off, int32_t S, int64_t i) {
  int32_t lo = 0, hi = S - 1;
  while (lo < hi) {
    int32_t mid = (lo + hi + 1) >> 1;
    if (scan_off[mid] <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Scan offsets in LDS (up to kScanLds scans; else they stay in global memory).
constexpr int kScanLds = 512;
__device__ __forceinline__ const int64_t* stage_scans(const int64_t* __restrict__ scan_off, int32_t S,
                                                      int64_t* lds) {
  if (S > kScanLds) return scan_off;
  for (int32_t s = threadIdx.x; s <= S; s += blockDim.x) lds[s] = scan_off[s];
  __syncthreads();
  return lds;
}

// Per hit: validation, hit rows (kept: 1 for a labelled hit; for soft weights
// the number of classes with a positive weight), number of free samples of a
// kept hit, voxel bounding box.  probs (nullable) replaces label: [n][K]
// weights, each finite and >= 0; all zero drops the hit and its beam.
// Threads stride over the hits in a capped grid, so that the box copies meet few
// atomics (a workgroup per 256 hits of 4.5e6: 159 us, now 40).
__global__ void __launch_bounds__(256) k_count(
    const float* __restrict__ xyz, const int32_t* __restrict__ label,
    const float* __restrict__ probs, int64_t n, const int64_t* __restrict__ scan_off,
    const float* __restrict__ origins, int32_t S, float res, float step, int32_t K,
    int64_t* __restrict__ nfree, int32_t* __restrict__ kept, int32_t* __restrict__ bbox,
    uint32_t* __restrict__ err) {
  __shared__ int64_t so[kScanLds + 1];
  const int64_t* soff = stage_scans(scan_off, S, so);
  const double inv_res = 1.0 / (double)res, inv_step = 1.0 / (double)step;
  int32_t lo[3] = {INT32_MAX, INT32_MAX, INT32_MAX};
  int32_t hi[3] = {INT32_MIN, INT32_MIN, INT32_MIN};
  uint32_t err_all = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float px = xyz[3 * i], py = xyz[3 * i + 1], pz = xyz[3 * i + 2];
    uint32_t e = 0;
    int64_t c = 0;
    int32_t k = 0;
    if (probs) {
      for (int32_t j = 0; j < K; ++j) {
        const float w = probs[i * K + j];
        if (!(isfinite(w) && w >= 0.0f)) e |= DEVERR_LABEL;
        k += w > 0.0f ? 1 : 0;
      }
    } else {
      const int32_t y = label[i];
      if (y < -1 || y >= K) e |= DEVERR_LABEL;
      k = y != -1 ? 1 : 0;
    }
    if (!finite3(px, py, pz)) e |= DEVERR_NONFINITE;
    if (e == 0 && k > 0) {
      int32_t v[3];
      if (!voxel_index(px, inv_res, res, &v[0]) || !voxel_index(py, inv_res, res, &v[1]) ||
          !voxel_index(pz, inv_res, res, &v[2])) {
        e |= DEVERR_RANGE;
      } else {
        for (int a = 0; a < 3; ++a) { lo[a] = min(lo[a], v[a]); hi[a] = max(hi[a], v[a]); }
      }
      if (step > 0.0f) {
        const int32_t s = scan_of(soff, S, i);
        const float ox = origins[3 * s], oy = origins[3 * s + 1], oz = origins[3 * s + 2];
        float vx, vy, vz;
        const float L = beam_len(px, py, pz, ox, oy, oz, &vx, &vy, &vz);
        if (L > 0.0f) {
          const float cf = ceilf(quot_rn(L, inv_step, step));
          if (!(cf - 1.0f <= (float)SMKI_MAX_SAMPLES_PER_RAY)) e |= DEVERR_RAY;
          else c = (int64_t)cf - 1;
        }
        if (c > 0) {
          int32_t vo[3];
          if (voxel_index(ox, inv_res, res, &vo[0]) && voxel_index(oy, inv_res, res, &vo[1]) &&
              voxel_index(oz, inv_res, res, &vo[2])) {
            for (int a = 0; a < 3; ++a) { lo[a] = min(lo[a], vo[a]); hi[a] = max(hi[a], vo[a]); }
          } else {
            e |= DEVERR_RANGE;
          }
        }
      }
    }
    nfree[i] = e ? 0 : c;
    kept[i] = e ? 0 : k;
    err_all |= e;
  }
  if (err_all) atomicOr(err, err_all);
  // workgroup reduction of the bounding box, then one atomic per workgroup
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int o = SMKI_WAVE / 2; o > 0; o >>= 1) {
      lo[a] = min(lo[a], __shfl_xor(lo[a], o, SMKI_WAVE));
      hi[a] = max(hi[a], __shfl_xor(hi[a], o, SMKI_WAVE));
    }
  __shared__ int32_t part[256 / SMKI_WAVE][6];
  if ((threadIdx.x & (SMKI_WAVE - 1)) == 0)
    for (int a = 0; a < 3; ++a) {
      part[threadIdx.x / SMKI_WAVE][a] = lo[a];
      part[threadIdx.x / SMKI_WAVE][3 + a] = hi[a];
    }
  __syncthreads();
  if (threadIdx.x < 6) {   // spread over copies: workgroups rarely contend on one address
    const int a = threadIdx.x;
    int32_t v = part[0][a];
    for (int w = 1; w < 256 / SMKI_WAVE; ++w) v = a < 3 ? min(v, part[w][a]) : max(v, part[w][a]);
    int32_t* bb = bbox + (blockIdx.x % SMKI_BBOX_COPIES) * 8 + a;
    if (a < 3 && v != INT32_MAX) atomicMin(bb, v);
    if (a >= 3 && v != INT32_MIN) atomicMax(bb, v);
  }
}

__device__ __forceinline__ void block_of(const BucketGeom& g, const int32_t v[3], int32_t b[3],
                                         int32_t l[3]) {
  for (int a = 0; a < 3; ++a) {
    b[a] = v[a] >> g.log2B;             // floor division (arithmetic shift)
    l[a] = v[a] - b[a] * g.B;
  }
}

// Key of a row: (label plane, block of the grid, voxel inside the block), so a
// sort groups rows by class first (planes = K for the map, 1 otherwise), then
// by block, then by voxel with z fastest.
template <typename KeyT>
__device__ __forceinline__ KeyT make_key(const BucketGeom& g, int32_t plane, const int32_t b[3],
                                         const int32_t l[3]) {
  const int64_t lin = (int64_t)plane * g.n_blocks +
                      ((int64_t)(b[0] - g.blo[0]) * g.nb[1] + (b[1] - g.blo[1])) * g.nb[2] +
                      (b[2] - g.blo[2]);
  const int64_t loc = ((int64_t)l[0] << (2 * g.log2B)) | ((int64_t)l[1] << g.log2B) | l[2];
  return (KeyT)(((uint64_t)lin << (3 * g.log2B)) | (uint64_t)loc);
}

// Record of a row: coordinates relative to the exact centre ((b + 1/2) B res) of
// its own block, computed in double and rounded once; label bits in .w.
__device__ __forceinline__ float4 make_record(const BucketGeom& g, float x, float y, float z,
                                              const int32_t b[3], int32_t label) {
  const double r = (double)g.res, hb = 0.5 * (double)g.B;
  float4 o;
  o.x = (float)((double)x - ((double)(b[0] * g.B) + hb) * r);
  o.y = (float)((double)y - ((double)(b[1] * g.B) + hb) * r);
  o.z = (float)((double)z - ((double)(b[2] * g.B) + hb) * r);
  o.w = __int_as_float(label);
  return o;
}

// Record of a map row: |u| per axis, u = x - (v + 1/2) res the row relative to
// the centre of its voxel (double, rounded once), and in .w the row's cell
// within its block and the octant of u:  (cell << 3) | (ux < 0) | (uy < 0) << 1
// | (uz < 0) << 2.  The class is the row's plane in the key, not stored here.
__device__ __forceinline__ float4 make_map_record(const BucketGeom& g, float x, float y, float z,
                                                  const int32_t v[3], const int32_t l[3]) {
  const double r = (double)g.res;
  const double ux = (double)x - ((double)v[0] + 0.5) * r;
  const double uy = (double)y - ((double)v[1] + 0.5) * r;
  const double uz = (double)z - ((double)v[2] + 0.5) * r;
  const int32_t cell = (l[0] << (2 * g.log2B)) | (l[1] << g.log2B) | l[2];
  const int32_t oct = (ux < 0.0 ? 1 : 0) | (uy < 0.0 ? 2 : 0) | (uz < 0.0 ? 4 : 0);
  float4 o;
  o.x = (float)fabs(ux);
  o.y = (float)fabs(uy);
  o.z = (float)fabs(uz);
  o.w = __int_as_float((cell << 3) | oct);
  return o;
}

__device__ __forceinline__ bool in_grid(const BucketGeom& g, const int32_t b[3]) {
  return b[0] >= g.blo[0] && b[0] < g.blo[0] + g.nb[0] && b[1] >= g.blo[1] &&
         b[1] < g.blo[1] + g.nb[1] && b[2] >= g.blo[2] && b[2] < g.blo[2] + g.nb[2];
}

// Kept hits -> (key, index) and records (unsorted), at rows kpos[i]...  With
// soft weights (probs non-null) a hit gives one row per class of positive
// weight, in class order, and wt[row] = that weight.  Also, for the free-sample
// kernel (workgroups of wg samples): wgbeam[b] = the beam that holds free
// sample b wg (each such sample lies in exactly one beam's range).
// dcnt (device, nullable): row counts [total, hits, free samples] of the
// insert, read here instead of nf (a capacity then).
template <typename KeyT>
__global__ void k_hit_keys(const float* __restrict__ xyz, const int32_t* __restrict__ label,
                           const float* __restrict__ probs, int32_t K, int64_t n,
                           const int32_t* __restrict__ kept, const int32_t* __restrict__ kpos,
                           const int64_t* __restrict__ off, int64_t nf_cap, int32_t wg,
                           const int64_t* __restrict__ dcnt,
                           int32_t* __restrict__ wgbeam, BucketGeom g, KeyT* __restrict__ keys,
                           float4* __restrict__ rec,
                           float* __restrict__ wt, uint32_t* __restrict__ err) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t nf = dcnt ? dcnt[2] : nf_cap;
  if (nf > 0) {
    // (clamped: a captured insert may hold fewer samples than its beams ask for)
    const int64_t a0 = min(off[i], nf), a1 = min(i + 1 < n ? off[i + 1] : nf, nf);
    for (int64_t b = (a0 + wg - 1) / wg; b * wg < a1; ++b) wgbeam[b] = (int32_t)i;
  }
  if (!kept[i]) return;
  const float px = xyz[3 * i], py = xyz[3 * i + 1], pz = xyz[3 * i + 2];
  int32_t v[3], b[3], l[3];
  const double inv_res = 1.0 / (double)g.res;
  voxel_index(px, inv_res, g.res, &v[0]);
  voxel_index(py, inv_res, g.res, &v[1]);
  voxel_index(pz, inv_res, g.res, &v[2]);
  block_of(g, v, b, l);
  int32_t w = kpos[i];
  const int32_t rows = kept[i];
  if (!in_grid(g, b)) {
    atomicOr(err, DEVERR_RANGE);
    for (int32_t r = 0; r < rows; ++r, ++w) {
      keys[w] = (KeyT)0; rec[w] = make_float4(0, 0, 0, 0);
      if (wt) wt[w] = 0.0f;
    }
    return;
  }
  const float4 r4 = make_map_record(g, px, py, pz, v, l);
  if (!probs) {
    keys[w] = make_key<KeyT>(g, label[i], b, l);
    rec[w] = r4;
    return;
  }
  for (int32_t k = 0; k < K; ++k) {
    const float p = probs[i * K + k];
    if (!(p > 0.0f)) continue;
    keys[w] = make_key<KeyT>(g, k, b, l);
    rec[w] = r4;
    wt[w] = p;
    ++w;
  }
}

// Samples per thread of the free-sample kernel (256 threads a workgroup): four
// share a beam's set-up, one where four would leave CUs without a workgroup (nf: the
// capacity of a captured insert).
static inline int32_t free_per(int64_t nf) { return nf <= (int64_t(1) << 18) ? 1 : 4; }

// Free sample f -> its beam (largest i with off[i] <= f), its position, key and
// record.  The beams of a workgroup's samples lie between the beam of its first
// sample and the beam of the next workgroup's first sample (wgbeam, written by
// k_hit_keys).  What the samples of a beam share (its offset, its vector and
// length, its origin's scan, the reciprocal of the length) is computed once per
// beam and workgroup, into LDS, where up to MAXB beams fit; else by every sample.
// Writes 24 bytes a sample; the divisions in double by every sample bound it
// (1.6e8 samples: 1,777 us, now 1,059; 3.9e6: 29 us, now 27).
struct Beam {
  float vx, vy, vz, L;
  float ox, oy, oz;
  double inv_l;
};
__device__ __forceinline__ Beam beam_of(const float* __restrict__ xyz, int64_t i,
                                        const float* __restrict__ origins, int32_t s) {
  Beam b;
  b.ox = origins[3 * s];
  b.oy = origins[3 * s + 1];
  b.oz = origins[3 * s + 2];
  b.L = beam_len(xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2], b.ox, b.oy, b.oz, &b.vx, &b.vy, &b.vz);
  b.inv_l = 1.0 / (double)b.L;
  return b;
}

template <typename KeyT>
__global__ void __launch_bounds__(256) k_free_keys(
    const float* __restrict__ xyz, int64_t n, const int64_t* __restrict__ off, int64_t nf_cap,
    int32_t per, const int64_t* __restrict__ dcnt, const int64_t* __restrict__ scan_off,
    const float* __restrict__ origins, int32_t S, float step, int32_t free_class, BucketGeom g,
    int64_t out_base_h, KeyT* __restrict__ keys, float4* __restrict__ rec, float* __restrict__ wrow,
    const int32_t* __restrict__ wgbeam, uint32_t* __restrict__ err) {
  constexpr int MAXB = 256;
  __shared__ int64_t soff[MAXB];
  __shared__ Beam beam[MAXB];
  const int64_t nf = dcnt ? dcnt[2] : nf_cap;             // (launch sized for nf_cap)
  const int64_t out_base = dcnt ? dcnt[1] : out_base_h;   // free samples follow the hits
  const int64_t nwg = (nf + 256 * per - 1) / (256 * per);
  if ((int64_t)blockIdx.x >= nwg) return;   // (the whole workgroup)
  const int64_t b0 = wgbeam[blockIdx.x];
  const int64_t b1 = (int64_t)blockIdx.x + 1 < nwg ? wgbeam[blockIdx.x + 1] : n - 1;
  const bool staged = b1 - b0 < MAXB;   // (the same range for the whole workgroup)
  if (staged) {
    if (threadIdx.x <= b1 - b0) {
      const int64_t i = b0 + threadIdx.x;
      soff[threadIdx.x] = off[i];
      // (a dropped hit holds no sample: its beam may be anything)
      beam[threadIdx.x] = beam_of(xyz, i, origins, scan_of(scan_off, S, i));
    }
    __syncthreads();
  }
  const double inv_res = 1.0 / (double)g.res;
  for (int u = 0; u < per; ++u) {
    const int64_t f = ((int64_t)blockIdx.x * per + u) * 256 + threadIdx.x;
    if (f >= nf) break;
    Beam b;
    int64_t o;
    if (staged) {
      int32_t a = 0, c = (int32_t)(b1 - b0);
      while (a < c) {
        const int32_t mid = (a + c + 1) >> 1;
        if (soff[mid] <= f) a = mid; else c = mid - 1;
      }
      b = beam[a];
      o = soff[a];
    } else {
      int64_t lo = b0, hi = b1;
      while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (off[mid] <= f) lo = mid; else hi = mid - 1;
      }
      b = beam_of(xyz, lo, origins, scan_of(scan_off, S, lo));
      o = off[lo];
    }
    const int64_t j = f - o + 1;
    const float t = (float)j * step;
    const float wt = quot_rn(t, b.inv_l, b.L);
    const float mx = wt * b.vx, my = wt * b.vy, mz = wt * b.vz;
    const float qx = b.ox + mx, qy = b.oy + my, qz = b.oz + mz;
    const int64_t w = out_base + f;
    int32_t v[3] = {0, 0, 0}, bl[3], l[3];
    bool ok = voxel_index(qx, inv_res, g.res, &v[0]) && voxel_index(qy, inv_res, g.res, &v[1]) &&
              voxel_index(qz, inv_res, g.res, &v[2]);
    block_of(g, v, bl, l);
    ok = ok && in_grid(g, bl);
    if (!ok) atomicOr(err, DEVERR_RANGE);
    keys[w] = ok ? make_key<KeyT>(g, free_class, bl, l) : (KeyT)0;
    rec[w] = ok ? make_map_record(g, qx, qy, qz, v, l) : make_float4(0, 0, 0, 0);
    if (wrow) wrow[w] = ok ? 1.0f : 0.0f;
  }
}

// Rows without labels (the bucketing entry point): keys and records.
template <typename KeyT>
__global__ void k_row_keys(const float* __restrict__ xyz, int64_t n, BucketGeom g,
                           KeyT* __restrict__ keys, uint32_t* __restrict__ idx, float4* __restrict__ rec,
                           uint32_t* __restrict__ err) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float px = xyz[3 * i], py = xyz[3 * i + 1], pz = xyz[3 * i + 2];
  int32_t v[3], b[3], l[3];
  const double inv_res = 1.0 / (double)g.res;
  if (!finite3(px, py, pz) || !voxel_index(px, inv_res, g.res, &v[0]) ||
      !voxel_index(py, inv_res, g.res, &v[1]) || !voxel_index(pz, inv_res, g.res, &v[2])) {
    atomicOr(err, DEVERR_RANGE);
    keys[i] = (KeyT)0; idx[i] = (uint32_t)i; rec[i] = make_float4(0, 0, 0, 0);
    return;
  }
  block_of(g, v, b, l);
  if (!in_grid(g, b)) { atomicOr(err, DEVERR_RANGE); keys[i] = (KeyT)0; idx[i] = (uint32_t)i; rec[i] = make_float4(0, 0, 0, 0); return; }
  keys[i] = make_key<KeyT>(g, 0, b, l);
  idx[i] = (uint32_t)i;
  rec[i] = make_record(g, px, py, pz, b, 0);
}

// Sorted records: out[i] = rec[idx[i]] (and the weights alike when present).
__global__ void k_permute_rec(const float4* __restrict__ rec, const float* __restrict__ wt,
                              const uint32_t* __restrict__ idx, int64_t n,
                              float4* __restrict__ out, float* __restrict__ wout) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t j = idx[i];
  out[i] = rec[j];
  if (wt) wout[i] = wt[j];
}

// Slots: the runs of sorted rows that share (plane, block) = key >> log2B3.
// A row heads a slot when its block differs from the previous row's.  Tiles of
// 256 RD rows (one workgroup; wavefront w takes its 64 RD consecutive rows, 64 per
// round) first mark their heads, one bit per row, and count them; after the scan
// of the counts they give their heads consecutive slot numbers in row order.
// The second pass reads the bits and the heads' keys only (reading every key and
// its predecessor twice took 492 us of the 1.7e8 rows of a town, now 234).
// Few rows take tiles of four rounds, which run one after the other, instead of
// sixteen (26,000 rows: 16 us, now 7).
constexpr int HT_THREADS = 256;
constexpr int kHeadRounds = 16, kHeadSmallRounds = 4;
constexpr int64_t kHeadSmallN = int64_t(1) << 18;

template <typename KeyT, int RD>
__global__ void __launch_bounds__(HT_THREADS) k_head_counts(const KeyT* __restrict__ keys,
                                                            int64_t ncap,
                                                            const int64_t* __restrict__ dn,
                                                            int shift,
                                                            unsigned long long* __restrict__ heads,
                                                            int32_t* __restrict__ tcount) {
  const int64_t n = eff_n(ncap, dn);   // (rows past the count head nothing)
  __shared__ int32_t wc[HT_THREADS / SMKI_WAVE];
  const int lane = threadIdx.x & (SMKI_WAVE - 1), w = threadIdx.x / SMKI_WAVE;
  const int64_t first = ((int64_t)blockIdx.x * (HT_THREADS / SMKI_WAVE) + w) * (RD * SMKI_WAVE);
  KeyT k[RD];
#pragma unroll
  for (int r = 0; r < RD; ++r) {
    const int64_t i = first + r * SMKI_WAVE + lane;
    k[r] = i < n ? keys[i] : (KeyT)0;
  }
  // the block before the wavefront's rows, then the last of each round (row 0
  // heads a slot whatever came before)
  uint64_t prev = first > 0 && first < n ? (uint64_t)(keys[first - 1] >> shift) : 0ull;
  int32_t c = 0;
#pragma unroll
  for (int r = 0; r < RD; ++r) {
    const int64_t i = first + r * SMKI_WAVE + lane;
    const uint64_t b = (uint64_t)(k[r] >> shift);
    const uint64_t up = __shfl_up(b, 1, SMKI_WAVE);
    const bool head = i < n && (i == 0 || b != (lane == 0 ? prev : up));
    prev = __shfl(b, SMKI_WAVE - 1, SMKI_WAVE);
    const uint64_t m = __ballot(head);
    if (lane == 0 && i < ncap) heads[i / SMKI_WAVE] = m;
    c += (int32_t)__popcll(m);
  }
  if (lane == 0) wc[w] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t t = 0;
    for (int q = 0; q < HT_THREADS / SMKI_WAVE; ++q) t += wc[q];
    tcount[blockIdx.x] = t;
  }
}

// After the scan of the tile counts (tstart, total in *d_nslots): the first
// row of every slot, the dense grid -> slot index and each slot's grid
// position.  The dense table is block-major: entry (block * planes + plane),
// so the classes of one block share a cache line.
template <typename KeyT, int RD>
__global__ void __launch_bounds__(HT_THREADS) k_slot_heads(
    const KeyT* __restrict__ keys, int64_t ncap, const int64_t* __restrict__ dn, int log2B3,
    int64_t n_blocks, int32_t planes, const unsigned long long* __restrict__ heads,
    const int32_t* __restrict__ tstart, int32_t* __restrict__ dense, int32_t* __restrict__ slot_lin,
    int32_t* __restrict__ head, const int32_t* __restrict__ d_nslots, int32_t cap_slots) {
  // (slots past cap_slots are not stored: a captured insert whose rows make
  // more slots than it was sized for is failed by its capacity check)
  const int64_t n = eff_n(ncap, dn);
  __shared__ int32_t wc[HT_THREADS / SMKI_WAVE];
  const int lane = threadIdx.x & (SMKI_WAVE - 1), w = threadIdx.x / SMKI_WAVE;
  const int64_t first = ((int64_t)blockIdx.x * (HT_THREADS / SMKI_WAVE) + w) * (RD * SMKI_WAVE);
  if (blockIdx.x == 0 && threadIdx.x == 0 && *d_nslots <= cap_slots) head[*d_nslots] = (int32_t)n;
  // lane r holds the bits of round r
  const uint64_t mine = lane < RD && first + lane * SMKI_WAVE < n ? heads[first / SMKI_WAVE + lane] : 0ull;
  int32_t c = (int32_t)__popcll(mine);
#pragma unroll
  for (int o = SMKI_WAVE / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, SMKI_WAVE);
  if (lane == 0) wc[w] = c;
  __syncthreads();
  int32_t slot = tstart[blockIdx.x];
  for (int q = 0; q < w; ++q) slot += wc[q];
#pragma unroll
  for (int r = 0; r < RD; ++r) {
    const uint64_t m = __shfl(mine, r, SMKI_WAVE);
    if ((m >> lane) & 1ull) {
      const int64_t i = first + r * SMKI_WAVE + lane;
      // plane * n_blocks + block, below 2^30
      const uint32_t blk = (uint32_t)((uint64_t)keys[i] >> log2B3), nb = (uint32_t)n_blocks;
      const int32_t sl = slot + (int32_t)__popcll(m & ((1ull << lane) - 1ull));
      if (sl < cap_slots) {
        dense[(int64_t)(blk % nb) * planes + blk / nb] = sl;
        slot_lin[sl] = (int32_t)blk;
        head[sl] = (int32_t)i;
      }
    }
    slot += (int32_t)__popcll(m);
  }
}

// Cell table of every slot: prefix[slot][c] = first row of cell c, [B3] = the
// slot's end.  One wavefront per slot (they stride over the slots), lane c
// searching the slot's sorted keys for cell c: log2(rows) dependent loads, which
// the other wavefronts hide.  (A histogram of the rows in LDS and its scan, by a
// workgroup per slot with four barriers, took 79 us for 3.2e6 rows.)
template <typename KeyT, int LOG2B3>
__global__ void __launch_bounds__(256) k_slot_prefix(const KeyT* __restrict__ keys,
                                                     const int32_t* __restrict__ head,
                                                     const int32_t* __restrict__ d_nslots,
                                                     int32_t* __restrict__ prefix) {
  constexpr int B3 = 1 << LOG2B3;
  const int32_t ns = *d_nslots, lane = threadIdx.x & (SMKI_WAVE - 1);
  const int32_t nw = gridDim.x * (256 / SMKI_WAVE);
  for (int32_t s = blockIdx.x * (256 / SMKI_WAVE) + threadIdx.x / SMKI_WAVE; s < ns; s += nw) {
    const int32_t r0 = head[s], r1 = head[s + 1];
    int32_t* P = prefix + (int64_t)s * (B3 + 1);
    for (int32_t c = lane; c <= B3; c += SMKI_WAVE) {
      int32_t lo = r0, hi = r1;   // the first row whose cell is at least c
      while (lo < hi) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if ((int32_t)((uint64_t)keys[mid] & (uint64_t)(B3 - 1)) < c) lo = mid + 1; else hi = mid;
      }
      P[c] = lo;
    }
  }
}

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// ---------------------------------------------------------------------------
// host-side launchers
// ---------------------------------------------------------------------------
static inline unsigned nblk(int64_t n, int t) { return (unsigned)ceil_div_i64(n > 0 ? n : 1, t); }

constexpr unsigned kCountGrid = 2048;   // workgroups of the hit validation (they stride)

hipError_t launch_count(const float* xyz, const int32_t* label, const float* probs, int64_t n,
                        const int64_t* scan_off, const float* origins, int32_t S, float res,
                        float step, int32_t K, int64_t* nfree, int32_t* kept, int32_t* bbox,
                        uint32_t* err, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_count, dim3(std::min(nblk(n, 256), kCountGrid)), dim3(256), 0, st, xyz, label, probs, n,
                     scan_off, origins, S, res, step, K, nfree, kept, bbox, err);
  return hipGetLastError();
}

// Three ranges in one launch: z0[0, n0) = 0, z1[0, n1) = 0, f[0, nf) = fv.
__global__ void k_clear3(int32_t* __restrict__ z0, int64_t n0, int32_t* __restrict__ z1, int64_t n1,
                         int32_t* __restrict__ f, int64_t nf, int32_t fv) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n0 + n1 + nf; i += stride) {
    if (i < n0)
      z0[i] = 0;
    else if (i < n0 + n1)
      z1[i - n0] = 0;
    else
      f[i - n0 - n1] = fv;
  }
}

hipError_t launch_clear3(int32_t* z0, int64_t n0, int32_t* z1, int64_t n1, int32_t* f, int64_t nf,
                         int32_t fv, hipStream_t st) {
  const int64_t n = n0 + n1 + nf;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_clear3, dim3((unsigned)std::min<int64_t>(nblk(n, 256), 4096)), dim3(256), 0,
                     st, z0, n0, z1, n1, f, nf, fv);
  return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3(nblk(n, 256)), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

// Keys, sort, records and block tables of one point set.
template <typename KeyT>
// idx_iota: idx was not written (row i's value is i): the first radix pass
// takes the indices itself.
// dn (device, nullable): the row count; ps.n is then the capacity.
static hipError_t finish_set(PointSet& ps, KeyT* keys, uint32_t* idx, KeyT* akeys, uint32_t* aidx,
                             float4* rec_unsorted, const BucketGeom& g, int key_bits,
                             BucketScratch& scr, hipStream_t st, bool idx_iota = false,
                             const int64_t* dn = nullptr, int32_t cap_slots = INT32_MAX) {
  const int64_t n = ps.n;
  if (n <= 0) return hipSuccess;
  hipError_t e;
  if (idx_iota && n == 1 && !dn) {   // no radix pass: the single index by hand
    e = hipMemsetAsync(idx, 0, sizeof(uint32_t), st);
    if (e != hipSuccess) return e;
  }
  // the last radix pass gathers the records (and weights) into sorted order,
  // if the set keeps sorted records; else they are read through the permutation
  const SortPayload pl{rec_unsorted, ps.pts, scr.wt, ps.wts};
  const SortPayload* plp = ((n > 1 || dn) && ps.pts) ? &pl : nullptr;
  if (sizeof(KeyT) == 4)
    e = radix_sort_u32((uint32_t*)keys, idx, (uint32_t*)akeys, aidx, n, key_bits, scr.sort_tmp,
                       scr.sort_tmp_bytes, st, plp, idx_iota, dn);
  else
    e = radix_sort_u64((uint64_t*)keys, idx, (uint64_t*)akeys, aidx, n, key_bits, scr.sort_tmp,
                       scr.sort_tmp_bytes, st, plp, idx_iota, dn);
  if (e != hipSuccess) return e;
  if (!plp && ps.pts)
    hipLaunchKernelGGL(k_permute_rec, dim3(nblk(n, 256)), dim3(256), 0, st, rec_unsorted,
                       (const float*)scr.wt, idx, n, ps.pts, ps.wts);
  ps.perm = idx;
  const int log2B3 = 3 * g.log2B;
  // slot heads: their bits and per-tile counts (both in scr.flag), the scan of
  // the counts (scr.slot_excl), numbering
  const bool few = n <= kHeadSmallN;
  const int64_t ntiles =
      ceil_div_i64(n, HT_THREADS * (few ? kHeadSmallRounds : kHeadRounds));
  unsigned long long* heads = (unsigned long long*)(scr.flag + (ntiles + 1) / 2 * 2);
  const dim3 grid((unsigned)ntiles), block(HT_THREADS);
  if (few)
    hipLaunchKernelGGL((k_head_counts<KeyT, kHeadSmallRounds>), grid, block, 0, st, keys, n, dn,
                       log2B3, heads, scr.flag);
  else
    hipLaunchKernelGGL((k_head_counts<KeyT, kHeadRounds>), grid, block, 0, st, keys, n, dn, log2B3,
                       heads, scr.flag);
  e = scan_excl_i32(scr.flag, scr.slot_excl, ntiles, ps.d_nslots, scr.scan_tmp, st);
  if (e != hipSuccess) return e;
  if (few)
    hipLaunchKernelGGL((k_slot_heads<KeyT, kHeadSmallRounds>), grid, block, 0, st, keys, n, dn,
                       log2B3, g.n_blocks, g.planes, (const unsigned long long*)heads, scr.slot_excl,
                       ps.dense, ps.slot_lin, ps.head, ps.d_nslots, cap_slots);
  else
    hipLaunchKernelGGL((k_slot_heads<KeyT, kHeadRounds>), grid, block, 0, st, keys, n, dn, log2B3,
                       g.n_blocks, g.planes, (const unsigned long long*)heads, scr.slot_excl,
                       ps.dense, ps.slot_lin, ps.head, ps.d_nslots, cap_slots);
  if (!ps.prefix) return hipGetLastError();
  // (cell tables: the differentiable form's, blocks of 4^3 cells and 32-bit keys)
  if constexpr (sizeof(KeyT) == 4) {
    if (log2B3 != 6) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_slot_prefix<KeyT, 6>), dim3((unsigned)std::min<int64_t>(nblk(n, 4), 4096)),
                       dim3(256), 0, st, keys, ps.head, ps.d_nslots, ps.prefix);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}

template <typename KeyT>
static hipError_t bucket_scan_t(const float* xyz, const int32_t* label, const float* probs,
                                int32_t K, int64_t n, const int32_t* kept, const int32_t* kpos,
                                int64_t nk, const int64_t* off, int64_t nf, int32_t* wgbeam,
                                const int64_t* scan_off, const float* origins, int32_t S,
                                float step, int32_t free_class, const BucketGeom& g, PointSet& ps,
                                BucketScratch& scr, uint32_t* err, hipStream_t st,
                                const int64_t* dcnt, int32_t cap_slots) {
  if (nk > 0 || dcnt)
    hipLaunchKernelGGL(k_hit_keys<KeyT>, dim3(nblk(n, 256)), dim3(256), 0, st, xyz, label, probs,
                       K, n, kept, kpos, off, nf, 256 * free_per(nf), dcnt, wgbeam, g, (KeyT*)scr.keys, scr.rec,
                       scr.wt, err);
  if (nf > 0)
    hipLaunchKernelGGL(k_free_keys<KeyT>, dim3(nblk(nf, 256 * free_per(nf))), dim3(256), 0,
                       st, xyz, n, off, nf, free_per(nf), dcnt, scan_off, origins, S, step, free_class, g, nk,
                       (KeyT*)scr.keys, scr.rec, scr.wt, (const int32_t*)wgbeam, err);
  return finish_set<KeyT>(ps, (KeyT*)scr.keys, scr.idx, (KeyT*)scr.akeys, scr.aidx, scr.rec, g,
                          g.key_bits, scr, st, true, dcnt, cap_slots);
}

// All training rows of an insert in one sorted set: kept hits at [0, nk), free
// samples after them; keys carry the class plane, so each (class, block) is a
// contiguous range.  wgbeam: scratch of free_sample_workgroups(nf) entries.
hipError_t bucket_scan(const float* xyz, const int32_t* label, const float* probs, int32_t K,
                       int64_t n, const int32_t* kept, const int32_t* kpos, int64_t nk,
                       const int64_t* off, int64_t nf, int32_t* wgbeam, const int64_t* scan_off,
                       const float* origins, int32_t S, float step, int32_t free_class,
                       const BucketGeom& g, PointSet& ps, BucketScratch& scr, uint32_t* err,
                       hipStream_t st, const int64_t* dcnt, int32_t cap_slots) {
  if (ps.n <= 0) return hipSuccess;
  if (g.key_bits <= 32)
    return bucket_scan_t<uint32_t>(xyz, label, probs, K, n, kept, kpos, nk, off, nf, wgbeam,
                                   scan_off, origins, S, step, free_class, g, ps, scr, err, st,
                                   dcnt, cap_slots);
  return bucket_scan_t<uint64_t>(xyz, label, probs, K, n, kept, kpos, nk, off, nf, wgbeam,
                                 scan_off, origins, S, step, free_class, g, ps, scr, err, st,
                                 dcnt, cap_slots);
}

int64_t free_sample_workgroups(int64_t nf) { return nf > 0 ? ceil_div_i64(nf, 256 * free_per(nf)) : 1; }

// ---------------------------------------------------------------------------
// rows and queries of the differentiable form
// ---------------------------------------------------------------------------
// The cells within one cell of a query, as one bit per cell (64 cells a block):
// eight threads per query, one for each of the at most 2 x 2 x 2 blocks (the grid
// strides over the queries).
__global__ void __launch_bounds__(256) k_mark_near(const float* __restrict__ qxyz, int64_t nq,
                                                   BucketGeom g,
                                                   unsigned long long* __restrict__ near) {
  const double inv_res = 1.0 / (double)g.res;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; (t >> 3) < nq;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = t >> 3;
    int32_t b[3];
    uint32_t m[3];   // the cells [v - 1, v + 1] of each axis that lie in block b
    bool own = true;   // (no second block along an axis: the first one's thread marks it)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      // (validated before: the voxel index is in range)
      const int32_t v = (int32_t)floorf(quot_rn(qxyz[3 * i + a], inv_res, g.res));
      const int32_t b0 = (v - 1) >> 2, b1 = (v + 1) >> 2;
      const bool second = (t >> a) & 1;
      own = own && !(second && b0 == b1);
      b[a] = second ? b1 : b0;
      const int32_t lo = max(v - 1 - b[a] * 4, 0), hi = min(v + 1 - b[a] * 4, 3);
      m[a] = ((1u << (hi - lo + 1)) - 1u) << lo;
    }
    if (!own || !in_grid(g, b)) continue;
    unsigned long long m2 = 0, m3 = 0;   // bits of one x layer, of the block
#pragma unroll
    for (int y = 0; y < 4; ++y)
      if ((m[1] >> y) & 1) m2 |= (unsigned long long)m[2] << (4 * y);
#pragma unroll
    for (int x = 0; x < 4; ++x)
      if ((m[0] >> x) & 1) m3 |= m2 << (16 * x);
    unsigned long long* w =
        near + ((int64_t)(b[0] - g.blo[0]) * g.nb[1] + (b[1] - g.blo[1])) * g.nb[2] + (b[2] - g.blo[2]);
    if ((*w & m3) != m3) atomicOr(w, m3);
  }
}

// The cell of a row: block, cell in the block and (with near) whether a query
// lies within one cell of it; rows outside the grid are errors and not near.
__device__ __forceinline__ bool row_cell(const BucketGeom& g, double inv_res, float x, float y,
                                         float z, const unsigned long long* __restrict__ near,
                                         int32_t b[3], int32_t l[3], uint32_t* __restrict__ err) {
  const float f[3] = {floorf(quot_rn(x, inv_res, g.res)), floorf(quot_rn(y, inv_res, g.res)),
                      floorf(quot_rn(z, inv_res, g.res))};
  int32_t v[3];
  bool ok = true;
  for (int a = 0; a < 3; ++a) {
    ok = ok && f[a] >= -(float)SMKI_COORD_LIM && f[a] < (float)SMKI_COORD_LIM;
    v[a] = ok ? (int32_t)f[a] : 0;
  }
  block_of(g, v, b, l);
  if (!ok || !in_grid(g, b)) {
    atomicOr(err, DEVERR_RANGE);
    return false;
  }
  if (!near) return true;
  const int64_t w = ((int64_t)(b[0] - g.blo[0]) * g.nb[1] + (b[1] - g.blo[1])) * g.nb[2] + (b[2] - g.blo[2]);
  return (near[w] >> ((l[0] * 4 + l[1]) * 4 + l[2])) & 1ull;
}

// Tiles of the two passes over the rows: NT rows, four per thread, loaded before
// any is used (sixteen left 25,000 rows to seven workgroups).
constexpr int NR = 4;
constexpr int NS = NR * SMKI_WAVE;       // rows per wavefront
constexpr int NT = HT_THREADS * NR;      // rows per tile

// Rows near a query: one bit per row (mask), their count per tile, and the
// gradient of every other row (zero: it is in no query's support).
__global__ void __launch_bounds__(HT_THREADS) k_near_count(
    const float* __restrict__ xyz, int64_t n, BucketGeom g,
    const unsigned long long* __restrict__ near, unsigned long long* __restrict__ mask,
    int32_t* __restrict__ tcount, float* __restrict__ grad, uint32_t* __restrict__ err) {
  __shared__ int32_t wc[HT_THREADS / SMKI_WAVE];
  const int lane = threadIdx.x & (SMKI_WAVE - 1), w = threadIdx.x / SMKI_WAVE;
  const int64_t base = (int64_t)blockIdx.x * NT + (int64_t)w * NS;
  const double inv_res = 1.0 / (double)g.res;
  int32_t c = 0;
  float v[NR][3];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int64_t i = min(base + r * SMKI_WAVE + lane, n - 1);
    v[r][0] = xyz[3 * i];
    v[r][1] = xyz[3 * i + 1];
    v[r][2] = xyz[3 * i + 2];
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int64_t i = base + r * SMKI_WAVE + lane;
    bool is = false;
    if (i < n) {
      int32_t b[3], l[3];
      is = row_cell(g, inv_res, v[r][0], v[r][1], v[r][2], near, b, l, err);
      if (grad && !is) grad[3 * i] = grad[3 * i + 1] = grad[3 * i + 2] = 0.0f;
    }
    const uint64_t m = __ballot(is);
    if (lane == 0 && i < n) mask[i / SMKI_WAVE] = m;
    c += (int32_t)__popcll(m);
  }
  if (lane == 0) wc[w] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t t = 0;
    for (int q = 0; q < HT_THREADS / SMKI_WAVE; ++q) t += wc[q];
    tcount[blockIdx.x] = t;
  }
}

// Keys and indices of the rows near a query, in row order (tstart: the scan of
// the tile counts, *n_near its total), and their records, at their indices; then (workgroups from gt on) the
// queries, plane 1 of the keys, with indices n + h.  dn receives the rows written.
template <typename KeyT>
__global__ void __launch_bounds__(HT_THREADS) k_near_keys(
    const float* __restrict__ xyz, const int32_t* __restrict__ label, int64_t n, int32_t gt,
    const float* __restrict__ qxyz, const int32_t* __restrict__ qlab, int64_t nq, BucketGeom g,
    const unsigned long long* __restrict__ mask, const int32_t* __restrict__ tstart,
    const int32_t* __restrict__ n_near, int64_t* __restrict__ dn, KeyT* __restrict__ keys,
    uint32_t* __restrict__ idx, float4* __restrict__ rec, uint32_t* __restrict__ err) {
  const double inv_res = 1.0 / (double)g.res;
  int32_t b[3], l[3];
  if (blockIdx.x == 0 && threadIdx.x == 0) *dn = (int64_t)*n_near + nq;
  if ((int32_t)blockIdx.x >= gt) {
    const int64_t h = (int64_t)(blockIdx.x - gt) * blockDim.x + threadIdx.x;
    if (h >= nq) return;
    const float x = qxyz[3 * h], y = qxyz[3 * h + 1], z = qxyz[3 * h + 2];
    const int64_t pos = (int64_t)*n_near + h;
    const bool ok = row_cell(g, inv_res, x, y, z, nullptr, b, l, err);
    keys[pos] = ok ? make_key<KeyT>(g, 1, b, l) : (KeyT)0;
    idx[pos] = (uint32_t)(n + h);
    rec[n + h] = ok ? make_record(g, x, y, z, b, qlab[h]) : make_float4(0, 0, 0, 0);
    return;
  }
  __shared__ int32_t wc[HT_THREADS / SMKI_WAVE];
  const int lane = threadIdx.x & (SMKI_WAVE - 1), w = threadIdx.x / SMKI_WAVE;
  const int64_t base = (int64_t)blockIdx.x * NT + (int64_t)w * NS;
  // lane r holds round r's mask
  const int64_t word = base / SMKI_WAVE + lane;
  const uint64_t mine = lane < NR && word * SMKI_WAVE < n ? mask[word] : 0ull;
  int32_t c = (int32_t)__popcll(mine);
#pragma unroll
  for (int o = SMKI_WAVE / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, SMKI_WAVE);
  if (lane == 0) wc[w] = c;
  __syncthreads();
  int32_t run = tstart[blockIdx.x];
  for (int q = 0; q < w; ++q) run += wc[q];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const uint64_t m = __shfl(mine, r, SMKI_WAVE);
    if ((m >> lane) & 1ull) {
      const int64_t i = base + r * SMKI_WAVE + lane;
      const float x = xyz[3 * i], y = xyz[3 * i + 1], z = xyz[3 * i + 2];
      row_cell(g, inv_res, x, y, z, nullptr, b, l, err);
      const int32_t pos = run + (int32_t)__popcll(m & ((1ull << lane) - 1ull));
      keys[pos] = make_key<KeyT>(g, 0, b, l);
      idx[pos] = (uint32_t)i;
      rec[i] = make_record(g, x, y, z, b, label[i]);   // (the sort gathers records by index)
    }
    run += (int32_t)__popcll(m);
  }
}

hipError_t bucket_near(const float* txyz, const int32_t* tlab, int64_t nt, const float* qxyz,
                       const int32_t* qlab, int64_t nq, bool both, const BucketGeom& g, PointSet& ps,
                       BucketScratch& scr, unsigned long long* near, float* grad_far, int64_t* dn,
                       int32_t* n_near, uint32_t* err, hipStream_t st) {
  if (g.key_bits > 32 || g.log2B != 2 || g.planes != (both ? 2 : 1)) return hipErrorInvalidValue;
  hipError_t e = launch_clear3(ps.d_nslots, 1, (int32_t*)near, near ? 2 * g.n_blocks : 0, ps.dense,
                               g.n_blocks * g.planes, -1, st);
  if (e != hipSuccess) return e;
  const int64_t n_sorted_q = both ? nq : 0;
  ps.n = nt + n_sorted_q;
  if (ps.n <= 0) return hipSuccess;
  if (near && nt > 0)
    hipLaunchKernelGGL(k_mark_near, dim3(near_mark_grid(nq)), dim3(256), 0, st, qxyz, nq, g, near);
  const int64_t tiles = ceil_div_i64(nt, NT);
  int32_t* tcount = scr.flag;
  int32_t* tstart = scr.flag + tiles;
  unsigned long long* mask = (unsigned long long*)scr.slot_excl;
  if (nt > 0)
    hipLaunchKernelGGL(k_near_count, dim3((unsigned)tiles), dim3(HT_THREADS), 0, st, txyz, nt, g,
                       (const unsigned long long*)near, mask, tcount, grad_far, err);
  e = scan_excl_i32(tcount, tstart, tiles, n_near, scr.scan_tmp, st);   // (no rows: total 0)
  if (e != hipSuccess) return e;
  const int64_t gq = both ? ceil_div_i64(nq, HT_THREADS) : 0;
  hipLaunchKernelGGL(k_near_keys<uint32_t>, dim3((unsigned)(tiles + gq)), dim3(HT_THREADS), 0, st,
                     txyz, tlab, nt, (int32_t)tiles, qxyz, qlab, n_sorted_q, g,
                     (const unsigned long long*)mask, (const int32_t*)tstart,
                     (const int32_t*)n_near, dn, (uint32_t*)scr.keys, scr.idx, scr.rec, err);
  return finish_set<uint32_t>(ps, (uint32_t*)scr.keys, scr.idx, (uint32_t*)scr.akeys, scr.aidx,
                              scr.rec, g, g.key_bits, scr, st, false, dn);
}

// ---------------------------------------------------------------------------
// cell table of a sorted row set (the bucketing entry point)
// ---------------------------------------------------------------------------
template <typename KeyT>
__global__ void k_cell_flags(const KeyT* __restrict__ keys, int64_t n, int32_t* __restrict__ flag) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) flag[i] = (i == 0 || keys[i] != keys[i - 1]) ? 1 : 0;
}

template <typename KeyT>
__global__ void k_cell_starts(const KeyT* __restrict__ keys, int64_t n, BucketGeom g,
                              const int32_t* __restrict__ flag, const int32_t* __restrict__ cpos,
                              uint64_t* __restrict__ cell_keys, int32_t* __restrict__ cell_start) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n || !flag[i]) return;
  const int l3 = 3 * g.log2B;
  const uint64_t key = (uint64_t)keys[i];
  int64_t lin = (int64_t)(key >> l3);
  const int32_t loc = (int32_t)(key & ((1ull << l3) - 1));
  const int32_t pz = (int32_t)(lin % g.nb[2]);
  lin /= g.nb[2];
  const int32_t py = (int32_t)(lin % g.nb[1]);
  const int32_t px = (int32_t)(lin / g.nb[1]);
  const int32_t B = g.B;
  const int32_t vx = (px + g.blo[0]) * B + (loc >> (2 * g.log2B));
  const int32_t vy = (py + g.blo[1]) * B + ((loc >> g.log2B) & (B - 1));
  const int32_t vz = (pz + g.blo[2]) * B + (loc & (B - 1));
  const int32_t c = cpos[i];
  cell_start[c] = (int32_t)i;
  cell_keys[c] = ((uint64_t)(int64_t)(vx + SMKI_COORD_LIM) << 42) |
                 ((uint64_t)(int64_t)(vy + SMKI_COORD_LIM) << 21) |
                 (uint64_t)(int64_t)(vz + SMKI_COORD_LIM);
}

__global__ void k_cell_counts(const int32_t* __restrict__ cell_start, int64_t ncells, int64_t n,
                              int32_t* __restrict__ cell_count) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncells) return;
  const int64_t e = (c + 1 < ncells) ? cell_start[c + 1] : n;
  cell_count[c] = (int32_t)(e - cell_start[c]);
}

__global__ void k_copy_order(const uint32_t* __restrict__ idx, int64_t n, int32_t* __restrict__ o) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) o[i] = (int32_t)idx[i];
}

// Sort rows by key (keys/idx filled by k_row_keys into scr), then count cells.
hipError_t bucket_cells_sort(const float* xyz, int64_t n, const BucketGeom& g, BucketScratch& scr,
                             uint32_t* err, int32_t* d_ncells, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipError_t e;
  if (g.key_bits <= 32) {
    hipLaunchKernelGGL(k_row_keys<uint32_t>, dim3(nblk(n, 256)), dim3(256), 0, st, xyz,
                       n, g, (uint32_t*)scr.keys, scr.idx, scr.rec, err);
    e = radix_sort_u32((uint32_t*)scr.keys, scr.idx, (uint32_t*)scr.akeys, scr.aidx, n, g.key_bits,
                       scr.sort_tmp, scr.sort_tmp_bytes, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cell_flags<uint32_t>, dim3(nblk(n, 256)), dim3(256), 0, st,
                       (const uint32_t*)scr.keys, n, scr.flag);
  } else {
    hipLaunchKernelGGL(k_row_keys<uint64_t>, dim3(nblk(n, 256)), dim3(256), 0, st, xyz,
                       n, g, (uint64_t*)scr.keys, scr.idx, scr.rec, err);
    e = radix_sort_u64((uint64_t*)scr.keys, scr.idx, (uint64_t*)scr.akeys, scr.aidx, n, g.key_bits,
                       scr.sort_tmp, scr.sort_tmp_bytes, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cell_flags<uint64_t>, dim3(nblk(n, 256)), dim3(256), 0, st,
                       (const uint64_t*)scr.keys, n, scr.flag);
  }
  return scan_excl_i32(scr.flag, scr.slot_excl, n, d_ncells, scr.scan_tmp, st);
}

hipError_t bucket_cells_table(int64_t n, int64_t ncells, const BucketGeom& g, BucketScratch& scr,
                              uint64_t* cell_keys, int32_t* cell_start, int32_t* cell_count,
                              int32_t* order, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (g.key_bits <= 32)
    hipLaunchKernelGGL(k_cell_starts<uint32_t>, dim3(nblk(n, 256)), dim3(256), 0, st,
                       (const uint32_t*)scr.keys, n, g, scr.flag, scr.slot_excl, cell_keys,
                       cell_start);
  else
    hipLaunchKernelGGL(k_cell_starts<uint64_t>, dim3(nblk(n, 256)), dim3(256), 0, st,
                       (const uint64_t*)scr.keys, n, g, scr.flag, scr.slot_excl, cell_keys,
                       cell_start);
  hipLaunchKernelGGL(k_cell_counts, dim3(nblk(ncells, 256)), dim3(256), 0, st, cell_start, ncells,
                     n, cell_count);
  if (order)
    hipLaunchKernelGGL(k_copy_order, dim3(nblk(n, 256)), dim3(256), 0, st, scr.idx, n, order);
  return hipGetLastError();
}

__global__ void k_free_xyz(const float* __restrict__ xyz, int64_t n, const int64_t* __restrict__ off,
                           int64_t nf, const float* __restrict__ origin, float step,
                           float* __restrict__ out, int64_t* __restrict__ parent) {
  const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= nf) return;
  int64_t lo = 0, hi = n - 1;
  while (lo < hi) {
    int64_t mid = (lo + hi + 1) >> 1;
    if (off[mid] <= f) lo = mid; else hi = mid - 1;
  }
  const int64_t i = lo;
  const int64_t j = f - off[i] + 1;
  float vx, vy, vz;
  const float L = beam_len(xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2], origin[0], origin[1],
                           origin[2], &vx, &vy, &vz);
  const float t = (float)j * step;
  const float w = div_rn(t, L);
  const float mx = w * vx, my = w * vy, mz = w * vz;
  out[3 * f] = origin[0] + mx;
  out[3 * f + 1] = origin[1] + my;
  out[3 * f + 2] = origin[2] + mz;
  if (parent) parent[f] = i;
}

hipError_t launch_free_xyz(const float* xyz, int64_t n, const int64_t* off, int64_t nf,
                           const float* origin_dev, float step, float* out, int64_t* parent,
                           hipStream_t st) {
  if (nf <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_free_xyz, dim3(nblk(nf, 256)), dim3(256), 0, st, xyz, n, off, nf,
                     origin_dev, step, out, parent);
  return hipGetLastError();
}
