// Workspace of the differentiable form: its header and the buffers carved after it
// (host; the layout alone, without a kernel).
#pragma once
#include <algorithm>

#include "smki_bucket.h"
#include "smki_plan.h"

constexpr int LB = 4;       // cells per block edge of the loss grid
constexpr int LLOG2B = 2;
constexpr int64_t kMaxLossBlocks = int64_t(1) << 22;

constexpr size_t kAl = 256;
struct Carve {
  char* base;
  size_t used;
  template <typename T>
  T* take(size_t n) {
    size_t off = (used + kAl - 1) / kAl * kAl;
    used = off + (n > 0 ? n : 1) * sizeof(T);
    return base ? (T*)(base + off) : nullptr;
  }
};

struct LossBufs {
  PointSet ps;
  BucketScratch scr;
  unsigned long long* near;   // [n_blocks] cells near a query; nullptr: no room for it
  int32_t* bbox;
  uint32_t* err;
  int64_t* dn;        // rows of the sorted set
  int32_t* n_near;    // its training rows
  float* alpha_q;
  float2* inv;   // (1/S, 1/alpha_y) of the queries in sorted order
  double* dsig;
  double* dl;
  double* dlk;   // [H][K] per-class form
  double* dsk;   // [H][K]
  float4* cls;   // [K] per-class form: class kernels (in the header)
};

// Header of a call (first 512 bytes: the bounding-box copies, the row counts of
// the sorted set, the error word) and the per-class kernel table (up to 255
// float4), ahead of the carved buffers
constexpr size_t kHdr = 512 + 256 * sizeof(float4);
constexpr size_t kCountOff = 256;

// Bytes that a workspace has to offer after the header for a grid of nblocks
// blocks (what the calls accept: two row sets with 64-bit keys, each with tables
// of its own).
inline size_t body_bytes(int64_t nt, int64_t nq, int32_t K, int64_t nblocks) {
  Carve c{nullptr, 0};
  c.take<float>((size_t)nq * K);
  c.take<float>(nq);
  c.take<float>(nq);
  c.take<double>(nq);
  c.take<double>(nq);
  c.take<double>((size_t)nq * K);
  c.take<double>((size_t)nq * K);
  for (int64_t n : {nt, nq}) {
    const int64_t slots = std::min<int64_t>(n, nblocks);
    c.take<float4>(n);
    c.take<int32_t>(nblocks);
    c.take<int32_t>(slots);
    c.take<int32_t>(slots * (LB * LB * LB + 1));
    c.take<int32_t>(1);
    c.take<uint64_t>(n);
    c.take<uint64_t>(n);
    c.take<uint32_t>(n);
    c.take<uint32_t>(n);
    c.take<float4>(n);
    c.take<int32_t>(n);
    c.take<int32_t>(n);
    c.take<int32_t>(n + 1);
    c.take<char>(sizeof(uint32_t) * 512 * (ceil_div_i64(std::max<int64_t>(n, 1), 4096) + 1) + 256);
    c.take<char>(scan_tmp_bytes(n));
  }
  return c.used + kAl;
}

// Buffers after the header (nullptr base: size only): one set of nt + nq rows
// with 32-bit keys, which never takes more than body_bytes without the bits of
// the cells near a query; near: with them.
inline size_t carve_body(char* base, LossBufs& b, int64_t nt, int64_t nq, int32_t K, int64_t nblocks,
                  bool near) {
  Carve c{base, 0};
  const int64_t n = nt + nq;
  const int64_t slots = std::min<int64_t>(nt, nblocks) + std::min<int64_t>(nq, nblocks);
  b.alpha_q = c.take<float>((size_t)nq * K);
  b.inv = c.take<float2>(nq);
  b.dsig = c.take<double>(nq);
  b.dl = c.take<double>(nq);
  b.dlk = c.take<double>((size_t)nq * K);
  b.dsk = c.take<double>((size_t)nq * K);
  b.ps.wts = nullptr;   // every training row of the loss weighs 1
  b.scr.wt = nullptr;
  b.ps.pts = c.take<float4>(n);
  b.ps.dense = c.take<int32_t>(2 * nblocks);
  b.ps.slot_lin = c.take<int32_t>(slots);
  b.ps.prefix = c.take<int32_t>(slots * (LB * LB * LB + 1));
  b.ps.d_nslots = c.take<int32_t>(1);
  b.scr.keys = c.take<uint32_t>(n);
  b.scr.akeys = c.take<uint32_t>(n);
  b.scr.idx = c.take<uint32_t>(n);
  b.scr.aidx = c.take<uint32_t>(n);
  b.scr.rec = c.take<float4>(n);
  b.scr.flag = c.take<int32_t>(n);
  b.scr.slot_excl = c.take<int32_t>(n);
  b.ps.head = c.take<int32_t>(n + 1);
  // (without grad_train only the nt training rows are sorted)
  b.scr.sort_tmp_bytes = radix_tmp_bytes(n);
  b.scr.sort_tmp = c.take<char>(b.scr.sort_tmp_bytes);
  b.scr.scan_tmp = c.take<char>(scan_tmp_bytes(n));
  b.near = near ? c.take<unsigned long long>(nblocks) : nullptr;
  return c.used + kAl;
}
