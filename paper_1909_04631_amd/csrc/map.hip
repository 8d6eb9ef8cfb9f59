// Persistent map: block hash, readout (Eq. 3-4), export / import.
#include "smki_gather.h"

namespace {

inline unsigned nblk(int64_t n, int t) { return (unsigned)ceil_div_i64(n > 0 ? n : 1, t); }

__device__ __forceinline__ int32_t hash_find(const MapDev& m, uint64_t key) {
  uint64_t h = smki_mix64(key) & (uint64_t)(m.hcap - 1);
  for (int64_t probe = 0; probe < m.hcap; ++probe) {
    const uint64_t k = m.hkeys[h];
    const int32_t v = m.hvals[h];   // (loaded with the key, not after it)
    if (k == key) return v;
    if (k == ~0ull) return -1;
    h = (h + 1) & (uint64_t)(m.hcap - 1);
  }
  return -1;
}

__global__ void k_hash_clear(uint64_t* keys, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) keys[i] = ~0ull;
}

// Readout of Eq. (3)-(4): mean alpha/S, variance mean(1-mean)/(S+1), label =
// argmax (lowest index on ties), occupancy = 1 - mean of the free class.
// SEG consecutive lanes serve one query, lane kl holding classes kl, kl + SEG,
// ... (at most 8; SEG >= K / 8): every lane finds the query's block and loads
// its classes' alpha (all loads in flight together), and the segment reduces
// the sum, the free class's alpha and the argmax with shuffles.  Few lanes per
// query keep the number of wavefronts, each waiting on the same chain of
// dependent loads, small.  The workgroup's alpha then lie in LDS and its rows of
// alpha, mean and var, which are contiguous, are written by consecutive threads
// (from the lanes that hold the classes, each store instruction touched sixteen
// rows in pieces of 16 bytes: 1e6 voxels of 20 classes 278 us, now 143,
// 720 MB of it read in 128-byte lines: the hash, the class-slot rows, the alphas).
// kmagic = ceil(2^32 / K): e / K for e < 2^16.
template <int SEG>
__global__ void __launch_bounds__(256) k_query(MapDev m, const int32_t* __restrict__ ijk,
                                               int64_t M, float* __restrict__ alpha,
                                               float* __restrict__ mean, float* __restrict__ var,
                                               int32_t* __restrict__ label,
                                               float* __restrict__ p_occ, int32_t free_class,
                                               uint32_t kmagic) {
  constexpr int MAXC = 8;   // classes per lane
  constexpr int NQ = 256 / SEG;   // queries per workgroup
  __shared__ float sa[NQ * SEG * MAXC];   // [query][K]
  __shared__ double sS[NQ], sI[NQ], sI1[NQ];   // S, 1/S, 1/(S + 1)
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = t / SEG;
  const int kl = (int)(t % SEG);
  const bool live = i < M;   // whole segments are live or not; shuffles stay inside a segment
  const int32_t K = m.K, B = m.B, B3 = B * B * B;
  int32_t slot = -1, v = 0;
  if (live) {
    const int32_t vx = ijk[3 * i], vy = ijk[3 * i + 1], vz = ijk[3 * i + 2];
    const int32_t bx = vx >> m.log2B, by = vy >> m.log2B, bz = vz >> m.log2B;
    if (vx >= -(1 << 20) && vx < (1 << 20) && vy >= -(1 << 20) && vy < (1 << 20) &&
        vz >= -(1 << 20) && vz < (1 << 20))
      slot = hash_find(m, smki_block_key(bx, by, bz));
    v = ((vx - bx * B) * B + (vy - by * B)) * B + (vz - bz * B);
  }
  // this lane's classes kl, kl + SEG, ...; classes without a class block hold alpha0
  // (all class-slot loads, then all alpha loads: each set in flight together)
  int32_t cb[MAXC];
#pragma unroll
  for (int j = 0; j < MAXC; ++j) {
    const int k = kl + j * SEG;
    cb[j] = (live && k < K && slot >= 0) ? m.cslot[(int64_t)slot * K + k] : -1;
  }
  float a[MAXC];
#pragma unroll
  for (int j = 0; j < MAXC; ++j) a[j] = cb[j] >= 0 ? m.calpha[(int64_t)cb[j] * B3 + v] : m.alpha0;
  double S = 0.0, af = 0.0;
  float bestv = -1.0f;
  int32_t best = 0;
#pragma unroll
  for (int j = 0; j < MAXC; ++j) {
    const int k = kl + j * SEG;
    if (live && k < K) {
      S += (double)a[j];
      if (k == free_class) af = (double)a[j];
      if (a[j] > bestv) {
        bestv = a[j];
        best = k;
      }
    }
  }
  // moments in double: 1 - mean cancels when one class dominates
#pragma unroll
  for (int o = 1; o < SEG; o <<= 1) {
    S += __shfl_xor(S, o, SEG);
    af += __shfl_xor(af, o, SEG);
    const float ov = __shfl_xor(bestv, o, SEG);
    const int32_t ok = __shfl_xor(best, o, SEG);
    if (ov > bestv || (ov == bestv && ok < best)) {
      bestv = ov;
      best = ok;
    }
  }
  const int ql = threadIdx.x / SEG;   // the query inside the workgroup
  const bool rows = alpha || mean || var;   // (the whole launch)
  if (live) {
    if (rows) {
#pragma unroll
      for (int j = 0; j < MAXC; ++j) {
        const int k = kl + j * SEG;
        if (k < K) sa[ql * K + k] = a[j];
      }
    }
    if (kl == 0) {
      const double inv_s = 1.0 / S;
      sS[ql] = S;
      sI[ql] = inv_s;
      sI1[ql] = 1.0 / (S + 1.0);
      if (label) label[i] = best;
      if (p_occ) p_occ[i] = (float)((S - af) * inv_s);
    }
  }
  if (!rows) return;   // (label and occupancy alone, 3e5 voxels of 255 classes: 124 us with the rows staged, now 104)
  __syncthreads();
  const int64_t q0 = (int64_t)blockIdx.x * NQ;
  const int n = (int)min((int64_t)NQ, M - q0) * K;
  for (int e = threadIdx.x; e < n; e += 256) {
    const float v = sa[e];
    const int64_t o = q0 * K + e;
    if (alpha) __builtin_nontemporal_store(v, &alpha[o]);
    if (!mean && !var) continue;
    const int q = (int)(((uint64_t)e * kmagic) >> 32);
    const double inv_s = sI[q];
    const double x = (double)v * inv_s;
    if (mean) __builtin_nontemporal_store((float)x, &mean[o]);
    if (var)
      __builtin_nontemporal_store((float)(x * ((sS[q] - (double)v) * inv_s) * sI1[q]), &var[o]);
  }
}

__global__ void k_hash_insert_slots(MapDev m, int64_t slot0, int64_t n, uint32_t* err) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int32_t slot = (int32_t)(slot0 + i);
  const uint64_t key = m.bkeys[slot];
  uint64_t h = smki_mix64(key) & (uint64_t)(m.hcap - 1);
  for (int64_t probe = 0; probe < m.hcap; ++probe) {
    const unsigned long long old =
        atomicCAS((unsigned long long*)&m.hkeys[h], ~0ull, (unsigned long long)key);
    if (old == ~0ull || old == key) {
      m.hvals[h] = slot;
      return;
    }
    h = (h + 1) & (uint64_t)(m.hcap - 1);
  }
  atomicOr(err, DEVERR_HASH);
}

// Export and import move dense [K][B^3] blocks, so the caller's array bounds them.
// V consecutive voxels per access: 4 (a float4) where B^3 and the caller's array
// allow it, else 1; four accesses per thread in flight.  6,007 blocks of 20 x 512
// (246 MB): export 167 us, now 57; import's two passes 100 + 49 us, now 46 + 22.
template <int V>
struct VecOf;
template <>
struct VecOf<1> { using T = float; };
template <>
struct VecOf<4> { using T = float4; };

// class block index -> (block, class): 32-bit arithmetic where it fits
__device__ __forceinline__ void split_bk(int64_t bk, int32_t K, int64_t* b, int32_t* k) {
  if (bk < (int64_t(1) << 32)) {
    const uint32_t q = (uint32_t)bk / (uint32_t)K;
    *b = q;
    *k = (int32_t)((uint32_t)bk - q * (uint32_t)K);
  } else {
    *b = bk / K;
    *k = (int32_t)(bk % K);
  }
}

// out block b <- pool slot order[b], dense [K][B^3] (alpha0 where a class has no class block)
template <int V>
__global__ void __launch_bounds__(256) k_gather_blocks(MapDev m, const uint32_t* __restrict__ order,
                                                       int64_t n, float* __restrict__ out) {
  using T = typename VecOf<V>::T;
  constexpr int U = 4;
  const int shift = 3 * m.log2B - (V == 4 ? 2 : 0);   // accesses per class block: 2^shift
  const int64_t total = (n * m.K) << shift;
  const int64_t base = (int64_t)blockIdx.x * (256 * U) + threadIdx.x;
  int32_t cb[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t i = min(base + u * 256, total - 1);
    int64_t b;
    int32_t k;
    split_bk(i >> shift, m.K, &b, &k);
    cb[u] = m.cslot[(int64_t)order[b] * m.K + k];
  }
  T v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t i = min(base + u * 256, total - 1);
    if constexpr (V == 4)
      v[u] = make_float4(m.alpha0, m.alpha0, m.alpha0, m.alpha0);
    else
      v[u] = m.alpha0;
    if (cb[u] >= 0) v[u] = ((const T*)m.calpha)[((int64_t)cb[u] << shift) + (i & ((int64_t(1) << shift) - 1))];
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (base + u * 256 < total) ((T*)out)[base + u * 256] = v[u];
}

// import: flag[b][k] = 1 if any voxel of class k in input block b differs from
// alpha0; one wavefront per class block
template <int V>
__global__ void __launch_bounds__(256) k_import_flags(MapDev m, const float* __restrict__ alpha,
                                                      int64_t nbk, int32_t* __restrict__ flag) {
  using T = typename VecOf<V>::T;
  constexpr int U = 4;
  const int lane = threadIdx.x & (SMKI_WAVE - 1);
  const int64_t bk = (int64_t)blockIdx.x * (256 / SMKI_WAVE) + threadIdx.x / SMKI_WAVE;
  if (bk >= nbk) return;
  const int per = (1 << (3 * m.log2B)) / V;
  const T* p = (const T*)alpha + bk * per;
  bool any = false;
  for (int i0 = 0; i0 < per && !__ballot(any); i0 += U * SMKI_WAVE) {
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = p[min(i0 + u * SMKI_WAVE + lane, per - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (V == 4)
        any = any || v[u].x != m.alpha0 || v[u].y != m.alpha0 || v[u].z != m.alpha0 || v[u].w != m.alpha0;
      else
        any = any || v[u] != m.alpha0;
    }
  }
  const bool set = __ballot(any) != 0;
  if (lane == 0) flag[bk] = set ? 1 : 0;
}

// import: (block b, class k) flagged -> class block c0 + pos[b][k]; others alpha0
// (no block); one wavefront per class block
template <int V>
__global__ void __launch_bounds__(256) k_import_copy(MapDev m, const float* __restrict__ alpha,
                                                     int64_t nbk, const int32_t* __restrict__ flag,
                                                     const int32_t* __restrict__ pos, int64_t c0) {
  using T = typename VecOf<V>::T;
  const int lane = threadIdx.x & (SMKI_WAVE - 1);
  const int64_t bk = (int64_t)blockIdx.x * (256 / SMKI_WAVE) + threadIdx.x / SMKI_WAVE;
  if (bk >= nbk) return;
  const int32_t cb = flag[bk] ? (int32_t)(c0 + pos[bk]) : -1;
  if (lane == 0) m.cslot[bk] = cb;
  if (cb < 0) return;
  const int per = (1 << (3 * m.log2B)) / V;
  const T* p = (const T*)alpha + bk * per;
  T* q = (T*)m.calpha + (int64_t)cb * per;
#pragma unroll 4
  for (int i = lane; i < per; i += SMKI_WAVE) q[i] = p[i];
}

// Blocks of an import that appear twice: their keys go into a table of hcap
// entries (a power of two, at least twice n, every word ~0 before); a key that
// is already there is a duplicate.  (A sort of the 63-bit keys took 21 launches.)
__global__ void k_find_dups(const uint64_t* __restrict__ keys, int64_t n,
                            unsigned long long* __restrict__ table, int64_t hcap,
                            uint32_t* __restrict__ err) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const unsigned long long key = keys[i];
  uint64_t h = smki_mix64(key) & (uint64_t)(hcap - 1);
  for (int64_t probe = 0; probe < hcap; ++probe) {
    const unsigned long long old = atomicCAS(&table[h], ~0ull, key);
    if (old == ~0ull) return;
    if (old == key) {
      atomicOr(err, DEVERR_DUP);
      return;
    }
    h = (h + 1) & (uint64_t)(hcap - 1);
  }
}

// Sort keys of the map's blocks relative to a box that holds them (lowest block
// lo, bits[] bits per axis), in the order of the full keys, and their indices.
__global__ void k_box_keys(const uint64_t* __restrict__ bkeys, int64_t n, int3 lo, int3 bits,
                           uint32_t* __restrict__ keys, uint32_t* __restrict__ idx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint64_t k = bkeys[i];
  const uint32_t x = (uint32_t)((int32_t)((k >> 42) & 0x1FFFFF) - (1 << 20) - lo.x);
  const uint32_t y = (uint32_t)((int32_t)((k >> 21) & 0x1FFFFF) - (1 << 20) - lo.y);
  const uint32_t z = (uint32_t)((int32_t)(k & 0x1FFFFF) - (1 << 20) - lo.z);
  keys[i] = (((x << bits.y) | y) << bits.z) | z;
  idx[i] = (uint32_t)i;
}

// block coordinates of pool slots order[0, n)
__global__ void k_keys_to_ijk(const uint64_t* __restrict__ bkeys, const uint32_t* __restrict__ order,
                              int64_t n, int32_t* ijk) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint64_t k = bkeys[order[i]];
  ijk[3 * i] = (int32_t)((k >> 42) & 0x1FFFFF) - (1 << 20);
  ijk[3 * i + 1] = (int32_t)((k >> 21) & 0x1FFFFF) - (1 << 20);
  ijk[3 * i + 2] = (int32_t)(k & 0x1FFFFF) - (1 << 20);
}

__global__ void k_ijk_to_keys(const int32_t* __restrict__ ijk, int64_t n, int32_t log2B,
                              uint64_t* keys, uint32_t* err, int32_t* __restrict__ box) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int32_t b[3] = {INT32_MAX, INT32_MAX, INT32_MAX}, hi[3] = {INT32_MIN, INT32_MIN, INT32_MIN};
  if (i < n) {
    const int32_t lim = (1 << 20) >> log2B;   // the block's voxels stay in [-2^20, 2^20)
    bool ok = true;
    for (int a = 0; a < 3; ++a) {
      b[a] = hi[a] = ijk[3 * i + a];
      ok = ok && b[a] >= -lim && b[a] < lim;
    }
    if (!ok) atomicOr(err, DEVERR_RANGE);
    keys[i] = ok ? smki_block_key(b[0], b[1], b[2]) : 0;
  }
  // the box of the blocks (one atomic per wavefront and side)
#pragma unroll
  for (int a = 0; a < 3; ++a) {
#pragma unroll
    for (int o = SMKI_WAVE / 2; o > 0; o >>= 1) {
      b[a] = min(b[a], __shfl_xor(b[a], o, SMKI_WAVE));
      hi[a] = max(hi[a], __shfl_xor(hi[a], o, SMKI_WAVE));
    }
    if ((threadIdx.x & (SMKI_WAVE - 1)) == 0) {
      atomicMin(&box[a], b[a]);
      atomicMax(&box[3 + a], hi[a]);
    }
  }
}

__global__ void k_iota(uint32_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = (uint32_t)i;
}

// ---------------------------------------------------------------------------
// captured inserts: device-side counts and checks (single small workgroups)
// ---------------------------------------------------------------------------
__global__ void k_batch_start(const int64_t* __restrict__ hdr, int64_t* __restrict__ counts,
                              unsigned long long* __restrict__ stats) {
  if (threadIdx.x == 0 && hdr[0]) {
    counts[0] = hdr[1];
    counts[1] = hdr[2];
  }
  for (int i = threadIdx.x; i < 4 * SMKI_STAT_COPIES; i += blockDim.x) stats[i] = 0ull;
}

__global__ void k_batch_rows(const int64_t* __restrict__ sc, int64_t cap_rows,
                             int64_t* __restrict__ pc, uint32_t* __restrict__ err) {
  const int64_t nf = sc[0];
  const int64_t nk = (int64_t)((const int32_t*)(sc + 1))[0];
  int64_t nt = nk + nf;
  if (nt > cap_rows) {
    atomicOr(err, DEVERR_CAPACITY);
    nt = cap_rows;   // (hit rows never exceed cap_rows: it is at least the hits)
  }
  pc[0] = nt;
  pc[1] = nk;
  pc[2] = nt - nk;
}

__global__ void k_batch_units(const int32_t* __restrict__ si, int64_t cap_slots,
                              int64_t cap_units, uint32_t* __restrict__ err) {
  if (si[0] > cap_slots || si[2] > cap_units) atomicOr(err, DEVERR_CAPACITY);
}

__global__ void k_batch_alloc_check(const int32_t* __restrict__ cnt,
                                    const int64_t* __restrict__ counts, int64_t pool_cap,
                                    int64_t cpool_cap, int64_t hcap, uint32_t* __restrict__ err) {
  const int64_t nb = counts[0] + cnt[0], nc = counts[1] + cnt[1];
  if (nb > pool_cap || nc > cpool_cap || 2 * nb > hcap) atomicOr(err, DEVERR_CAPACITY);
}

__global__ void k_batch_commit(const int32_t* __restrict__ cnt, int64_t* __restrict__ counts,
                               const uint32_t* __restrict__ err, uint32_t* __restrict__ map_err,
                               const int64_t* __restrict__ pc, const int32_t* __restrict__ si,
                               int64_t* __restrict__ out) {
  const uint32_t e = *err;
  if (e == 0) {
    counts[0] += cnt[0];
    counts[1] += cnt[1];
  } else {
    atomicOr(map_err, e);
  }
  out[0] = e;
  out[1] = e ? 0 : cnt[0];
  out[2] = e ? 0 : cnt[1];
  out[3] = pc[0];
  out[4] = pc[1];
  out[5] = pc[2];
  out[6] = si[0];
  out[7] = si[1];
  out[8] = si[2];
}

// An ordinary insert's new block counts, added on the device to the counts the
// host held before it (the host reads them back at its next synchronisation),
// and copied to out (read back with the insert counters).  The allocation
// kernel does the same when it runs; this serves an insert with no targets.
__global__ void k_commit_counts(const int32_t* __restrict__ cnt, int64_t* __restrict__ counts,
                                int64_t n_blocks, int64_t n_cblocks, int32_t* __restrict__ out) {
  counts[0] = n_blocks + cnt[0];
  counts[1] = n_cblocks + cnt[1];
  out[0] = cnt[0];
  out[1] = cnt[1];
}

}  // namespace

hipError_t launch_commit_counts(const int32_t* cnt, int64_t* counts, int64_t n_blocks,
                                int64_t n_cblocks, int32_t* out, hipStream_t st) {
  hipLaunchKernelGGL(k_commit_counts, dim3(1), dim3(1), 0, st, cnt, counts, n_blocks, n_cblocks,
                     out);
  return hipGetLastError();
}

hipError_t launch_batch_start(const int64_t* hdr, int64_t* counts, unsigned long long* stats,
                              hipStream_t st) {
  hipLaunchKernelGGL(k_batch_start, dim3(1), dim3(256), 0, st, hdr, counts, stats);
  return hipGetLastError();
}

hipError_t launch_batch_rows(const int64_t* sc, int64_t cap_rows, int64_t* pc, uint32_t* err,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_batch_rows, dim3(1), dim3(1), 0, st, sc, cap_rows, pc, err);
  return hipGetLastError();
}

hipError_t launch_batch_units(const int32_t* si, int64_t cap_slots, int64_t cap_units,
                              uint32_t* err, hipStream_t st) {
  hipLaunchKernelGGL(k_batch_units, dim3(1), dim3(1), 0, st, si, cap_slots, cap_units, err);
  return hipGetLastError();
}

hipError_t launch_batch_alloc_check(const int32_t* cnt, const int64_t* counts, int64_t pool_cap,
                                    int64_t cpool_cap, int64_t hcap, uint32_t* err,
                                    hipStream_t st) {
  hipLaunchKernelGGL(k_batch_alloc_check, dim3(1), dim3(1), 0, st, cnt, counts, pool_cap,
                     cpool_cap, hcap, err);
  return hipGetLastError();
}

hipError_t launch_batch_commit(const int32_t* cnt, int64_t* counts, const uint32_t* err,
                               uint32_t* map_err, const int64_t* pc, const int32_t* si,
                               int64_t* out, hipStream_t st) {
  hipLaunchKernelGGL(k_batch_commit, dim3(1), dim3(1), 0, st, cnt, counts, err, map_err, pc, si,
                     out);
  return hipGetLastError();
}

hipError_t launch_query(const MapDev& m, const int32_t* ijk, int64_t M, float* alpha, float* mean,
                        float* var, int32_t* label, float* p_occ, int32_t free_class,
                        hipStream_t st) {
  if (M <= 0) return hipSuccess;
  // K <= 255: at most 8 classes per lane
  const int seg = m.K <= 32 ? 4 : m.K <= 64 ? 8 : m.K <= 128 ? 16 : 32;
  const unsigned grid = nblk(M * seg, 256);
  const uint32_t kmagic = (uint32_t)(((uint64_t(1) << 32) + m.K - 1) / m.K);
  switch (seg) {
    case 4:
      hipLaunchKernelGGL(k_query<4>, dim3(grid), dim3(256), 0, st, m, ijk, M, alpha, mean, var,
                         label, p_occ, free_class, kmagic);
      break;
    case 8:
      hipLaunchKernelGGL(k_query<8>, dim3(grid), dim3(256), 0, st, m, ijk, M, alpha, mean, var,
                         label, p_occ, free_class, kmagic);
      break;
    case 16:
      hipLaunchKernelGGL(k_query<16>, dim3(grid), dim3(256), 0, st, m, ijk, M, alpha, mean, var,
                         label, p_occ, free_class, kmagic);
      break;
    default:
      hipLaunchKernelGGL(k_query<32>, dim3(grid), dim3(256), 0, st, m, ijk, M, alpha, mean, var,
                         label, p_occ, free_class, kmagic);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_hash_clear(const MapDev& m, hipStream_t st) {
  hipLaunchKernelGGL(k_hash_clear, dim3(nblk(m.hcap, 256)), dim3(256), 0, st, m.hkeys, m.hcap);
  return hipGetLastError();
}

hipError_t launch_hash_insert_slots(const MapDev& m, int64_t slot0, int64_t n, uint32_t* err,
                                    hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_hash_insert_slots, dim3(nblk(n, 256)), dim3(256), 0, st, m, slot0, n, err);
  return hipGetLastError();
}

// float4 accesses: whole class blocks of a multiple of four voxels, an aligned array
static bool vec4_ok(const MapDev& m, const void* p) { return m.B >= 2 && ((uintptr_t)p & 15) == 0; }

hipError_t launch_gather_blocks(const MapDev& m, const uint32_t* order, int64_t n,
                                float* alpha_out, hipStream_t st) {
  const int64_t tot = n * (int64_t)m.K * m.B * m.B * m.B;
  if (tot <= 0) return hipSuccess;
  if (vec4_ok(m, alpha_out))
    hipLaunchKernelGGL(k_gather_blocks<4>, dim3(nblk(tot / 4, 1024)), dim3(256), 0, st, m, order, n,
                       alpha_out);
  else
    hipLaunchKernelGGL(k_gather_blocks<1>, dim3(nblk(tot, 1024)), dim3(256), 0, st, m, order, n,
                       alpha_out);
  return hipGetLastError();
}

hipError_t launch_import_flags(const MapDev& m, const float* alpha, int64_t n, int32_t* flag,
                               hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t nbk = n * m.K;
  const dim3 grid(nblk(nbk, 256 / SMKI_WAVE)), block(256);
  if (vec4_ok(m, alpha))
    hipLaunchKernelGGL(k_import_flags<4>, grid, block, 0, st, m, alpha, nbk, flag);
  else
    hipLaunchKernelGGL(k_import_flags<1>, grid, block, 0, st, m, alpha, nbk, flag);
  return hipGetLastError();
}

hipError_t launch_import_copy(const MapDev& m, const float* alpha, int64_t n, const int32_t* flag,
                              const int32_t* pos, int64_t c0, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t nbk = n * m.K;
  const dim3 grid(nblk(nbk, 256 / SMKI_WAVE)), block(256);
  if (vec4_ok(m, alpha))
    hipLaunchKernelGGL(k_import_copy<4>, grid, block, 0, st, m, alpha, nbk, flag, pos, c0);
  else
    hipLaunchKernelGGL(k_import_copy<1>, grid, block, 0, st, m, alpha, nbk, flag, pos, c0);
  return hipGetLastError();
}

hipError_t launch_find_dups(const uint64_t* keys, int64_t n, uint64_t* table, int64_t hcap,
                            uint32_t* err, hipStream_t st) {
  if (n <= 1) return hipSuccess;
  hipLaunchKernelGGL(k_hash_clear, dim3(nblk(hcap, 256)), dim3(256), 0, st, table, hcap);
  hipLaunchKernelGGL(k_find_dups, dim3(nblk(n, 256)), dim3(256), 0, st, keys, n,
                     (unsigned long long*)table, hcap, err);
  return hipGetLastError();
}

hipError_t launch_box_keys(const uint64_t* bkeys, int64_t n, const int32_t lo[3],
                           const int32_t bits[3], uint32_t* keys, uint32_t* idx, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_box_keys, dim3(nblk(n, 256)), dim3(256), 0, st, bkeys, n,
                     make_int3(lo[0], lo[1], lo[2]), make_int3(bits[0], bits[1], bits[2]), keys, idx);
  return hipGetLastError();
}

hipError_t launch_block_keys_to_ijk(const uint64_t* bkeys, const uint32_t* order, int64_t n,
                                    int32_t* ijk, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_keys_to_ijk, dim3(nblk(n, 256)), dim3(256), 0, st, bkeys, order, n, ijk);
  return hipGetLastError();
}

hipError_t launch_ijk_to_block_keys(const int32_t* ijk, int64_t n, int32_t log2B, uint64_t* keys,
                                    uint32_t* err, int32_t* box, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_ijk_to_keys, dim3(nblk(n, 256)), dim3(256), 0, st, ijk, n, log2B, keys,
                     err, box);
  return hipGetLastError();
}

hipError_t launch_iota_u32(uint32_t* p, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_iota, dim3(nblk(n, 256)), dim3(256), 0, st, p, n);
  return hipGetLastError();
}
