// Cross-family vocabularies: the decision step for drafter rows in their own
// vocabulary (Sec. 6.4, App. D), reached through the map vmap[x] = drafter id of
// verifier token x.
//
// What bounds a mapped row is its gathers: a random 2-byte read from a row of
// drafter logits moves a 128-byte line.  So a drafter row is cut into tiles of
// XTile::kN logits, a tile of a and b is read once, contiguously, into LDS as
// (a, b) pairs, and the random half of every access is an LDS read.  The shared
// tokens that map into a tile form the tile's list, in ascending verifier order,
// so t is read nearly in order as well.  The lists are rebuilt from the map for
// every call (two short kernels), since the caller's map may change.
//
// A call is a sequence of kernels on the caller's stream, without waits between
// workgroups: list count, list fill, statistics (one workgroup per row and
// tile), decide, pass 2 (row and tile, rows with a task only), pick; with early
// exit the statistics of the first rows and a verdict come first.
//
// Tiles of 64 KiB with 512 threads put two workgroups on a CU, so that one
// streams its tile in while the other reduces; XCD-grouped block numbers keep
// the tiles of a row on one XCD, whose L2 then holds the row of t that all of
// them read.  Measured on B = 128, K = 6, V = 151936, Vd = 128256, 109566
// shared, bf16: 32 KiB tiles 1430 us, 64 KiB 330 us, 128 KiB (one workgroup per
// CU, with or without the next tile prefetched in registers) 347-357 us, 321 us
// with one batch's gathers of t in flight while the batch before is reduced,
// 311 us now; element-wise gathers from global memory, with a and b in drafter
// order and t through the inverse map, took 1070 us.  What is left is bound by
// the address unit: in the statistics, two thirds of the call, it is 65% busy and
// the VALU 53%, with 90 M cache accesses, about 50 per 64-lane gather of t.

#ifndef ASYMSPEC_XVOCAB_H_
#define ASYMSPEC_XVOCAB_H_

#include <cstddef>

#include "device.h"
#include "resolve.h"

namespace asym {

// Verifier tokens are grouped in units of 2^ulog consecutive ones, by which the
// lists are indexed: the smallest unit that leaves at most kXUnits of them.  The
// weight sums of pass 2 are kept per (row, tile, sub-block of 2^slog tokens): the
// unit, or down to 1024 tokens as long as all of them take no more than kXSumBytes,
// so that the pick, which scans one sub-block, has less to scan.  Beyond that a row's
// sums take no more of the workspace than the pass-2 records of a plain call (T * U
// * 4 bytes against 320 a chunk): sub-blocks of 512 tokens at any size took 316 MB
// at B = 512, K = 8, V = Vd = 256000 fp32; a pick over units of 4096 instead of 1024
// takes 26 us instead of 13 at B = 2.
constexpr int kXUnitLog = 10, kXUnitLogMax = 16;
constexpr int kXUnits = 79, kXSubs = kThreads;
constexpr size_t kXSumBytes = 8u << 20;
constexpr int x_unit_log(int V) {
  int l = kXUnitLog;
  while (((V - 1) >> l) + 1 > kXUnits && l < kXUnitLogMax) ++l;
  return l;
}
constexpr int x_sub_log(int U, int ulog, size_t row_tiles) {
  int l = ulog;
  while (l > kXUnitLog && (U << (ulog - l + 1)) <= kXSubs &&
         row_tiles * (size_t)(U << (ulog - l + 1)) * 4 <= kXSumBytes) --l;
  return l;
}
static_assert(((4194297 - 1) >> x_unit_log(4194297)) + 1 <= kXUnits, "the longest row has too many units");
constexpr int kXBatch = 8;            // entries per thread and step

constexpr int x_log2(int n) { return n <= 1 ? 0 : 1 + x_log2(n / 2); }
template <int DT> struct XTileBase {
  static constexpr int kBytes = 65536;
  static constexpr int kThr = 512;
  static constexpr int kWv = kThr / 64;
  static constexpr int kN = kBytes / (DT == ASYMSPEC_BF16 ? 4 : 8);   // drafter ids per tile
  using Entry = XEntry<x_log2(kN)>;
  static constexpr int kSpan = (int)Entry::kSpan;
  static_assert(kSpan % (1 << kXUnitLogMax) == 0, "a span of tokens ends with a unit");
  static constexpr int kVec = kN / (DT == ASYMSPEC_BF16 ? 8 : 4) / kThr;   // staged vectors per thread and stream
};
template <int DT> struct XTile;
template <> struct XTile<ASYMSPEC_BF16> : XTileBase<ASYMSPEC_BF16> {
  typedef uint32_t Pair;
  DEV static float a(Pair p) { return __uint_as_float(p << 16); }
  DEV static float b(Pair p) { return __uint_as_float(p & 0xFFFF0000u); }
  DEV static Pair make(uint32_t wa, uint32_t wb) { return (wa >> 16) | (wb & 0xFFFF0000u); }
  DEV static Pair masked() { return kBf16NegInf * 0x10001u; }
};
template <> struct XTile<ASYMSPEC_FP32> : XTileBase<ASYMSPEC_FP32> {
  typedef uint64_t Pair;
  DEV static float a(Pair p) { return __uint_as_float((uint32_t)p); }
  DEV static float b(Pair p) { return __uint_as_float((uint32_t)(p >> 32)); }
  DEV static Pair make(uint32_t wa, uint32_t wb) { return (uint64_t)wa | ((uint64_t)wb << 32); }
  DEV static Pair masked() { return (uint64_t)kF32NegInf * 0x100000001ull; }
};

struct XArgs {
  uint32_t* list;     // entries of every tile, tile after tile
  int32_t* cnt;       // [U][T] entries per unit and tile
  int32_t* idx;       // [T][U + 1] first entry of tile tl in unit u; [U] the tile's end
  float* sums;        // [rows][T][nsub] pass-2 weight sums
  float* jpart;       // [rows][T] pass-2 divergence partials
  int32_t* work;      // [1 + rows] number of rows with a pass-2 task, then those rows
  int T, U, nsub;
  int ulog, slog;     // 2^ulog tokens per unit, 2^slog per sub-block
  int tlog;           // 2^tlog >= T
  int r0, r1;         // rows of each request this launch covers
  unsigned b0;        // first of its blocks (a launch holds fewer than 2^32 threads)
};

// ------------------------------------------------------------------- lists
// One workgroup per unit, each wave a run of consecutive tokens of it.  The work
// per token does not grow with the number of tiles: lanes with the same tile find
// each other with one ballot per bit of the tile's number.  B = 2, K = 4, V = 256000,
// Vd = 250000 fp32 (31 tiles): count 3.8 and fill 7.1 us, where 250 workgroups that
// looped over the tiles and summed all counts took 6.0 and 21.2.
constexpr int kXMaxT = 256;                 // tiles of a row (a row has at most 256 chunks)
constexpr int kXListThr = 1024, kXListWv = kXListThr / 64;
constexpr int kXK = 4;                      // tokens per lane at once

// The wave's first token of unit u, and its steps of 64 tokens.
DEV int xv_first(const XArgs& X, int u, int w) { return (u << X.ulog) + w * ((1 << X.ulog) / kXListWv); }
DEV int xv_steps(const XArgs& X) { return (1 << X.ulog) / kXListThr; }

// This lane's drafter ids at steps [k0, k0 + kXK) of the wave (-1: none).
DEV void xv_ids(const KArgs& A, const XArgs& X, int x0, int k0, int lane, int (&j)[kXK]) {
  #pragma unroll
  for (int k = 0; k < kXK; ++k) {
    const int x = x0 + (k0 + k) * 64 + lane;
    j[k] = k0 + k < xv_steps(X) ? map_id(A.vmap, A.V, A.Vd, x) : -1;
  }
}
// Entries per tile among the wave's tokens, into its row n of LDS (zeros before).
template <int DT>
DEV void xv_wave_counts(const KArgs& A, const XArgs& X, int x0, int lane, int* n) {
  for (int k0 = 0; k0 < xv_steps(X); k0 += kXK) {
    int j[kXK];
    xv_ids(A, X, x0, k0, lane, j);
    #pragma unroll
    for (int k = 0; k < kXK; ++k)
      if (j[k] >= 0) __hip_atomic_fetch_add(n + j[k] / XTile<DT>::kN, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// count: the unit's entries per tile.  (Also clears the pass-2 work list.)
template <int DT>
__global__ __launch_bounds__(kXListThr) void xv_count_kernel(KArgs A, XArgs X) {
  __shared__ int n[kXListWv][kXMaxT];
  const int u = (int)blockIdx.x, tid = (int)threadIdx.x, lane = lane_id(), w = wave_id();
  if (u == 0 && tid == 0) X.work[0] = 0;
  for (int i = tid; i < kXListWv * kXMaxT; i += kXListThr) (&n[0][0])[i] = 0;
  __syncthreads();
  xv_wave_counts<DT>(A, X, xv_first(X, u, w), lane, n[w]);
  __syncthreads();
  if (tid < X.T) {
    int c = 0;
    #pragma unroll
    for (int q = 0; q < kXListWv; ++q) c += n[q][tid];
    X.cnt[u * X.T + tid] = c;
  }
}

// fill: where the unit's entries of every tile start (after the tiles before,
// and after the units before in the tile), then the entries in token order.
template <int DT>
__global__ __launch_bounds__(kXListThr) void xv_fill_kernel(KArgs A, XArgs X) {
  __shared__ int n[kXListWv][kXMaxT], all[kXMaxT], before[kXMaxT];
  const int u = (int)blockIdx.x, tid = (int)threadIdx.x, lane = lane_id(), w = wave_id();
  for (int i = tid; i < kXListWv * kXMaxT; i += kXListThr) (&n[0][0])[i] = 0;
  if (tid < kXMaxT) all[tid] = before[tid] = 0;
  __syncthreads();
  const int x0 = xv_first(X, u, w);
  xv_wave_counts<DT>(A, X, x0, lane, n[w]);
  #pragma unroll 4
  for (int i = tid; i < X.U << X.tlog; i += kXListThr) {
    const int t = i & ((1 << X.tlog) - 1), q = i >> X.tlog;
    const int c = t < X.T ? X.cnt[q * X.T + t] : 0;
    if (c != 0) {
      __hip_atomic_fetch_add(all + t, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (q < u) __hip_atomic_fetch_add(before + t, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
  __syncthreads();
  if (w == 0) {
    // lane l: tiles 4l .. 4l + 3, after the tiles before
    constexpr int kPer = kXMaxT / 64;
    int own = 0;
    #pragma unroll
    for (int e = 0; e < kPer; ++e) own += all[lane * kPer + e];
    int incl = own;
    #pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    int start = incl - own;
    #pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const int t = lane * kPer + e, len = all[t];
      before[t] += start;
      if (t < X.T) {
        X.idx[t * (X.U + 1) + u] = before[t];
        if (u == 0) X.idx[t * (X.U + 1) + X.U] = start + len;
      }
      start += len;
    }
  }
  __syncthreads();
  if (tid < X.T) {
    // the waves' runs in order
    int at = before[tid];
    #pragma unroll
    for (int q = 0; q < kXListWv; ++q) {
      const int c = n[q][tid];
      n[q][tid] = at;
      at += c;
    }
  }
  __syncthreads();
  const unsigned long long lt = (1ull << lane) - 1ull;
  for (int k0 = 0; k0 < xv_steps(X); k0 += kXK) {
    int j[kXK];
    xv_ids(A, X, x0, k0, lane, j);
    #pragma unroll
    for (int k = 0; k < kXK; ++k) {
      const bool in = j[k] >= 0;
      const int t = in ? j[k] / XTile<DT>::kN : 0;
      // the lanes with an entry in the same tile
      unsigned long long m = __ballot(in);
      for (int b = 0; b < X.tlog; ++b) {
        const bool bit = ((t >> b) & 1) != 0;
        const unsigned long long s = __ballot(bit);
        m &= bit ? s : ~s;
      }
      const int at = in ? n[w][t] : 0;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // every lane has read its place
      if (in) {
        const uint32_t x = (uint32_t)(x0 + (k0 + k) * 64 + lane);
        X.list[at + __popcll(m & lt)] = XTile<DT>::Entry::make(x, (uint32_t)(j[k] - t * XTile<DT>::kN));
        if ((m & lt) == 0) n[w][t] = at + __popcll(m);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  }
}

// -------------------------------------------------------------------- tile
template <int DT>
struct alignas(16) XSmem {
  using XT = XTile<DT>;
  // a row may start one element after a 4-byte boundary: the tile holds the
  // elements from that boundary on
  union {
    typename XT::Pair pair[XT::kN + 16];
    // after the tile's last use: every thread's reference and sum per slot
    struct { float R[kSlots][XT::kThr], s[kSlots][XT::kThr], W[XT::kThr]; } red;
  };
  int q[64];
  float wj[XT::kWv], wmarg[XT::kWv];
  int warg[XT::kWv], wneq[XT::kWv];
};
// the tile is written 16 bytes at a time
static_assert(alignof(XSmem<ASYMSPEC_BF16>) >= sizeof(u4) && offsetof(XSmem<ASYMSPEC_BF16>, pair) == 0 &&
              alignof(XSmem<ASYMSPEC_FP32>) >= sizeof(u4) && offsetof(XSmem<ASYMSPEC_FP32>, pair) == 0, "tile alignment");

// Drafter ids [j0, j0 + n) of a row on their way into LDS: 16-byte loads from
// the 4-byte boundary at or before the first (a and b are 4-byte aligned),
// each thread's share held in registers; the few elements the whole vectors
// leave (the array's last partial vector, the vector that a shifted start
// adds) are read one by one when the tile is written.
template <int DT>
struct XStage {
  using XT = XTile<DT>;
  __amdgpu_buffer_rsrc_t ra, rb;
  unsigned long long el0;   // array index of slot 0
  int lead;                 // slot of id j0 (0 or 1)
  int nslot, nreg;          // slots in use, vectors read as vectors
  u4 va[XT::kVec], vb[XT::kVec];

  DEV void load(const KArgs& A, int row, int tile) {
    constexpr int VE = Elem<DT>::VE, ES = 16 / VE;
    const int j0 = tile * XT::kN, n = min(XT::kN, A.Vd - j0);
    const unsigned long long n_el = (unsigned long long)A.B * (A.K + 1) * (unsigned long long)A.Vd;
    const unsigned long long e0 = (unsigned long long)row * A.Vd + (unsigned long long)j0;
    const unsigned long long byte0 = (e0 * ES) & ~3ull;
    el0 = byte0 / ES;
    lead = (int)(e0 - el0);
    nslot = lead + n;
    const unsigned long long full = (n_el * ES - byte0) / 16;
    nreg = min((nslot + VE - 1) / VE, XT::kVec * XT::kThr);
    nreg = full < (unsigned long long)nreg ? (int)full : nreg;
    ra = make_rsrc((const char*)A.a + byte0, (unsigned long long)nreg * 16);
    rb = make_rsrc((const char*)A.b + byte0, (unsigned long long)nreg * 16);
    #pragma unroll
    for (int k = 0; k < XT::kVec; ++k) {
      // past the resource: zeros, no access
      const uint32_t off = ((uint32_t)threadIdx.x + (uint32_t)(k * XT::kThr)) * 16u;
      va[k] = buf_load_nt(ra, off);
      vb[k] = buf_load_nt(rb, off);
    }
  }
  DEV void store(const KArgs& A, typename XT::Pair* pair) {
    constexpr int VE = Elem<DT>::VE;
    #pragma unroll
    for (int k = 0; k < XT::kVec; ++k) {
      const int v = (int)threadIdx.x + k * XT::kThr;
      if (v >= nreg) break;
      u4* dst = reinterpret_cast<u4*>(pair + v * VE);
      if (DT == ASYMSPEC_BF16) {
        u4 lo, hi;
        #pragma unroll
        for (int e = 0; e < 2; ++e) {
          lo[2 * e] = (va[k][e] & 0xFFFFu) | (vb[k][e] << 16);
          lo[2 * e + 1] = (va[k][e] >> 16) | (vb[k][e] & 0xFFFF0000u);
          hi[2 * e] = (va[k][2 + e] & 0xFFFFu) | (vb[k][2 + e] << 16);
          hi[2 * e + 1] = (va[k][2 + e] >> 16) | (vb[k][2 + e] & 0xFFFF0000u);
        }
        dst[0] = lo;
        dst[1] = hi;
      } else {
        dst[0] = u4{va[k][0], vb[k][0], va[k][1], vb[k][1]};
        dst[1] = u4{va[k][2], vb[k][2], va[k][3], vb[k][3]};
      }
    }
    const int s = nreg * VE + (int)threadIdx.x;
    if (threadIdx.x < 16 && s < nslot) {
      const long long idx = (long long)(el0 + (unsigned long long)s);
      pair[s] = XT::make(__float_as_uint(Elem<DT>::load_one(A.a, idx)), __float_as_uint(Elem<DT>::load_one(A.b, idx)));
    }
  }
};

// One tile of one row: its list, the row of t, and where the tokens' spans
// change.  Both are read through buffer resources, which return zeros past
// the list's end without a branch (entry 0 names token 0 and the tile's first
// slot: both exist).
struct XItem {
  int row, req, i, tile, n, lead, nhi;
  int q1;   // list position from which tokens are at kSpan or above
  __amdgpu_buffer_rsrc_t list, t;
};

template <int DT>
DEV XItem xv_item(const KArgs& A, const XArgs& X, int row, int tile) {
  constexpr int ES = 16 / Elem<DT>::VE;
  XItem it;
  it.row = row;
  it.req = row / (A.K + 1);
  it.i = row - it.req * (A.K + 1);
  it.tile = tile;
  const int32_t* ix = X.idx + (size_t)tile * (X.U + 1);
  const int first = ix[0];
  it.n = ix[X.U] - first;
  it.list = make_rsrc(X.list + first, (unsigned long long)it.n * 4);
  it.t = make_rsrc((const char*)A.t + (unsigned long long)row * A.V * ES, (unsigned long long)A.V * ES);
  it.nhi = (A.V - 1) / XTile<DT>::kSpan;
  it.lead = 0;
  it.q1 = 0x7FFFFFFF;
  return it;
}

// Thread h fills the list position from which tokens are at h spans or above
// (q1 by xv_bounds_in once they are in).
template <int DT>
DEV void xv_bounds(const XArgs& X, const XItem& it, XSmem<DT>& sm) {
  const int h = (int)threadIdx.x;
  if (h <= it.nhi && h < 64) {
    const int32_t* ix = X.idx + (size_t)it.tile * (X.U + 1);
    sm.q[h] = ix[h * (XTile<DT>::kSpan >> X.ulog)] - ix[0];
  }
}

template <int DT>
DEV void xv_bounds_in(XItem& it, const XSmem<DT>& sm) {
  if (it.nhi >= 1) it.q1 = __builtin_amdgcn_readfirstlane(sm.q[1]);
}

// Verifier tokens of the entries en[e] at list positions p0 + e * kStride.
template <int DT, int kStride>
DEV void xv_tokens(const XItem& it, const XSmem<DT>& sm, const uint32_t (&en)[kXBatch], int p0, int (&x)[kXBatch]) {
  constexpr int kHi = XTile<DT>::kSpan;
  #pragma unroll
  for (int e = 0; e < kXBatch; ++e) x[e] = (int)XTile<DT>::Entry::token(en[e]);
  if (it.nhi >= 1) {
    #pragma unroll
    for (int e = 0; e < kXBatch; ++e) x[e] += p0 + e * kStride >= it.q1 ? kHi : 0;
  }
  for (int h = 2; h <= it.nhi; ++h) {
    const int q = __builtin_amdgcn_readfirstlane(sm.q[h]);
    #pragma unroll
    for (int e = 0; e < kXBatch; ++e) x[e] += p0 + e * kStride >= q ? kHi : 0;
  }
}

// Entry at list position p.
DEV uint32_t xv_entry(const XItem& it, int p) {
  return __builtin_amdgcn_raw_buffer_load_b32(it.list, p * 4, 0, 0);
}
// t at token x.
template <int DT>
DEV float xv_t(const XItem& it, int x) {
  if (DT == ASYMSPEC_BF16)
    return __uint_as_float((uint32_t)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(it.t, x * 2, 0, 0) << 16);
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(it.t, x * 4, 0, 0));
}
template <int DT>
DEV typename XTile<DT>::Pair xv_pair(const XItem& it, const XSmem<DT>& sm, uint32_t e) {
  return sm.pair[XTile<DT>::Entry::id(e) + it.lead];
}

// Tokens and t of the entries en[e] at positions p0 + e * kThr.
template <int DT>
DEV void xv_load_t(const XItem& it, const XSmem<DT>& sm, const uint32_t (&en)[kXBatch], int p0, int (&x)[kXBatch],
                   float (&xt)[kXBatch]) {
  using XT = XTile<DT>;
  xv_tokens<DT, XT::kThr>(it, sm, en, p0, x);
  #pragma unroll
  for (int e = 0; e < kXBatch; ++e) xt[e] = xv_t<DT>(it, x[e]);
}
// Their a and b (ab), everything masked past the list's end; whether any pair
// differs in this lane.
template <int DT>
DEV bool xv_load_ab(const XItem& it, const XSmem<DT>& sm, const uint32_t (&en)[kXBatch], int p0, bool ab,
                    float (&xt)[kXBatch], float (&xa)[kXBatch], float (&xb)[kXBatch]) {
  using XT = XTile<DT>;
  typename XT::Pair pr[kXBatch];
  #pragma unroll
  for (int e = 0; e < kXBatch; ++e) pr[e] = ab ? xv_pair<DT>(it, sm, en[e]) : XT::masked();
  // (uniform: the batch's last wave-wide position)
  if (__builtin_expect(__any(p0 + (kXBatch - 1) * XT::kThr >= it.n), 0)) {
    #pragma unroll
    for (int e = 0; e < kXBatch; ++e)
      if (p0 + e * XT::kThr >= it.n) {
        xt[e] = -INFINITY;
        pr[e] = XT::masked();
      }
  }
  uint32_t ne = 0;
  #pragma unroll
  for (int e = 0; e < kXBatch; ++e) {
    xa[e] = XT::a(pr[e]);
    xb[e] = XT::b(pr[e]);
    ne |= __float_as_uint(xa[e]) ^ __float_as_uint(xb[e]);
  }
  return ne != 0u;
}

template <int THR>
DEV void xv_entries(const XItem& it, int p0, uint32_t (&en)[kXBatch]) {
  #pragma unroll
  for (int e = 0; e < kXBatch; ++e) en[e] = xv_entry(it, p0 + e * THR);
}

// -------------------------------------------------------------- statistics
// One workgroup per (row, tile); the record of tile `tile` of the row, as the
// decide reads it (A.S = X.T records per row).
template <int DT, int DM>
__global__ __launch_bounds__(XTile<DT>::kThr) __attribute__((amdgpu_waves_per_eu(4)))
void xv_stats_kernel(KArgs A, XArgs X) {
  using XT = XTile<DT>;
  __shared__ XSmem<DT> sm;
  const int lane = (int)threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // consecutive blocks go to the 8 XCDs in turn: the tiles of a row take
  // blocks 8 apart, so they run on one XCD at about the same time
  const unsigned blk = X.b0 + blockIdx.x;
  const int nr = X.r1 - X.r0, s = (int)(blk >> 3);
  const int lr = s / X.T * 8 + (int)(blk & 7u), tile = s % X.T;
  if (lr >= A.B * nr) return;
  XItem it = xv_item<DT>(A, X, lr / nr * (A.K + 1) + X.r0 + lr % nr, tile);
  if (X.r0 > 0) {
    // early exit: rows after the first group, unneeded after a sure rejection
    const uint64_t v = ld_tag(dec_hdr(A, it.req) + H_VERDICT);
    if (tag_ok(v, A.epoch) && pay(v) == kVerdictSkip) return;
  }
  const bool draft = it.i < A.K, fused = draft || A.fuse_bonus != 0;
  uint32_t en[kXBatch];
  xv_entries<XT::kThr>(it, (int)threadIdx.x, en);   // the first entries come in beside the tile
  {
    XStage<DT> stg;
    if (fused) {
      stg.load(A, it.row, tile);
      it.lead = stg.lead;
    }
    xv_bounds<DT>(X, it, sm);
    if (fused) stg.store(A, sm.pair);
  }
  __syncthreads();
  xv_bounds_in<DT>(it, sm);
  const float tau = sload_f32(A.tau, it.req);
  const bool samp = tau > 0.0f;
  const float c = samp ? kL2E / tau : kL2E;
  const bool sum_t = draft ? !samp : !fused, sum_at = draft && samp && tau != 1.0f;
  const bool arg = !samp, kl = draft && A.gate_mode == ASYMSPEC_GATE_KL;
  Acc qT, qA, qB, qF, qAT;
  const float ct = draft ? kL2E : c;
  acc_init(qT, ct); acc_init(qA, kL2E); acc_init(qB, kL2E); acc_init(qF, c); acc_init(qAT, c);
  float W = 0.0f;
  uint64_t neq = 0;
  bool bsame = true;   // a and b equal so far in every lane: b's sum is a's
  // one batch's gathers of t are in flight while the batch before is reduced
  // (a wave whose first position is past the end is done; the wave stays whole)
  int x[kXBatch];
  float xt[kXBatch];
  const int p_first = (int)threadIdx.x;
  xv_load_t<DT>(it, sm, en, p_first, x, xt);
  for (int k = 0; p_first - lane + k * kXBatch * XT::kThr < it.n; ++k) {
    const int p0 = p_first + k * kXBatch * XT::kThr;
    float xa[kXBatch], xb[kXBatch], tn[kXBatch];
    const uint64_t nm = __ballot(xv_load_ab<DT>(it, sm, en, p0, fused, xt, xa, xb));
    xv_entries<XT::kThr>(it, p0 + kXBatch * XT::kThr, en);
    xv_load_t<DT>(it, sm, en, p0 + kXBatch * XT::kThr, x, tn);
    neq |= nm;
    if (sum_t) {
      if (arg && !draft) acc_vec<kXBatch, false, true>(qT, xt, ct, k);
      else acc_vec_lazy<kXBatch, false>(qT, xt, ct);
    }
    if (fused) {
      float xf[kXBatch];
      #pragma unroll
      for (int e = 0; e < kXBatch; ++e) xf[e] = fuse<DM>(xt[e], xa[e], xb[e], A.beta);
      if (arg) acc_vec<kXBatch, true, true>(qF, xf, c, k);
      else acc_vec_lazy<kXBatch, true>(qF, xf, c);
    }
    if (draft) {
      if (!(bsame && nm == 0)) {
        if (bsame) { qB = qA; bsame = false; }
        acc_vec_lazy<kXBatch, false>(qB, xb, kL2E);
      }
      if (kl) {
        float dab[kXBatch];
        #pragma unroll
        for (int e = 0; e < kXBatch; ++e) dab[e] = __fsub_rn(xa[e], xb[e]);
        acc_vec_w<kXBatch, false>(qA, W, xa, dab, kL2E);
      } else {
        acc_vec_lazy<kXBatch, false>(qA, xa, kL2E);
      }
      if (sum_at) acc_vec_lazy<kXBatch, false>(qAT, xa, c);
    }
    #pragma unroll
    for (int e = 0; e < kXBatch; ++e) xt[e] = tn[e];
  }
  if (bsame) qB = qA;
  int cand = 0x7FFFFFFF;
  float mw = kFloorM;
  if (arg) {
    const Acc& qa = fused ? qF : qT;
    mw = wave_max(qa.m);
    if (qa.m == mw && mw > kFloorM) {
      // the batch where this thread first reached the maximum, once more
      float xa[kXBatch], xb[kXBatch];
      const int p0 = qa.pos * kXBatch * XT::kThr + (int)threadIdx.x;
      xv_entries<XT::kThr>(it, p0, en);
      xv_load_t<DT>(it, sm, en, p0, x, xt);
      xv_load_ab<DT>(it, sm, en, p0, fused, xt, xa, xb);
      #pragma unroll
      for (int e = kXBatch - 1; e >= 0; --e) {
        const float v = fused ? fuse<DM>(xt[e], xa[e], xb[e], A.beta) : xt[e];
        cand = v == mw ? x[e] : cand;
      }
    }
    cand = wave_min_i(cand);
  }
  if (lane == 0) { sm.warg[w] = cand; sm.wneq[w] = neq != 0 ? 1 : 0; sm.wmarg[w] = mw; }
  __syncthreads();
  // every thread's slots into LDS; wave s then combines slot s, lane by lane
  // over the waves and then over its lanes (one wave's reductions per slot
  // rather than every wave's over every slot)
  {
    const int tid = (int)threadIdx.x;
    auto put = [&](int slot, const Acc& q, bool used) {
      sm.red.R[slot][tid] = used ? q.R : kFloorM;
      sm.red.s[slot][tid] = used ? q.s : 0.0f;
    };
    put(sT, qT, sum_t);
    put(sA, qA, draft);
    put(sB, qB, draft);
    put(sF, qF, fused);
    put(sAT, qAT, sum_at);
    sm.red.W[tid] = W;
  }
  __syncthreads();
  uint64_t* rec = A.rec1 + ((size_t)it.row * A.S + tile) * kR1;
  static_assert(XT::kWv > kSlots, "one wave per slot and one for the rest");
  if (w < kSlots) {
    float R = kFloorM, S = 0.0f, Wl = 0.0f;
    #pragma unroll
    for (int i = 0; i < XT::kWv; ++i) R = fmaxf(R, sm.red.R[w][i * 64 + lane]);
    R = wave_max(R);
    #pragma unroll
    for (int i = 0; i < XT::kWv; ++i) {
      const float sc = __builtin_amdgcn_exp2f(sm.red.R[w][i * 64 + lane] - R);
      S += sm.red.s[w][i * 64 + lane] * sc;
      if (kl && w == sA) Wl += sm.red.W[i * 64 + lane] * sc;
    }
    S = wave_sum(S);
    if (w == sA) Wl = wave_sum(Wl);
    if (lane == 0) {
      st_tag(rec + R1_R + w, __float_as_uint(R), A.epoch);
      st_tag(rec + R1_S + w, __float_as_uint(S), A.epoch);
      if (w == sA) st_tag(rec + R1_W, __float_as_uint(Wl), A.epoch);
    }
  } else if (w == kSlots && lane == 0) {
    float Mall = kFloorM;
    for (int i = 0; i < XT::kWv; ++i) Mall = fmaxf(Mall, sm.wmarg[i]);
    int argx = 0x7FFFFFFF, nq = 0;
    for (int i = 0; i < XT::kWv; ++i) {
      if (sm.wmarg[i] == Mall) argx = min(argx, sm.warg[i]);
      nq |= sm.wneq[i];
    }
    st_tag(rec + R1_ARG, (uint32_t)argx, A.epoch);
    st_tag(rec + R1_NEQ, (uint32_t)nq, A.epoch);
    st_tag(rec + R1_MARG, __float_as_uint(Mall), A.epoch);
  }
}

// ------------------------------------------------------------------ decide
// ... and the rows that pass 2 must look at, into the work list (in any order:
// each row's sums are its own).
template <int DT>
__global__ __launch_bounds__(kThreads) void xv_decide_kernel(KArgs A, XArgs X, int verdict) {
  __shared__ Smem sm;
  const int req = (int)blockIdx.x;
  decide_item<DT, true>(A, req, sm, verdict != 0);
  if (verdict != 0 || wave_id() != 0 || sm.req[R_FAIL] != 0u || sm.req[R_FIN] != 0u) return;
  const int lane = lane_id();
  const bool task = lane <= A.K && sm.rows[lane][D_TASK] != 0u;
  const unsigned long long m = __ballot(task);
  int at = 0;
  if (lane == 0 && m != 0)
    at = __hip_atomic_fetch_add(X.work, __popcll(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  at = __builtin_amdgcn_readfirstlane(at);
  if (task) X.work[1 + at + __popcll(m & ((1ull << lane) - 1ull))] = req * (A.K + 1) + lane;
}

// ------------------------------------------------------------------ pass 2
// One workgroup per (listed row, tile), a fixed grid walking the work list:
// the divergence partial and the weight sums of the row's sub-blocks over the
// tile's tokens.  A wave takes a run of whole units and walks their entries 64
// at a time; a sub-block's sum is closed when the tokens leave it, so it has
// one order.
template <int DT, int DM>
__global__ __launch_bounds__(XTile<DT>::kThr) __attribute__((amdgpu_waves_per_eu(4)))
void xv_pass2_kernel(KArgs A, XArgs X) {
  using XT = XTile<DT>;
  __shared__ XSmem<DT> sm;
  // as in the statistics, the tiles of a row on one XCD (the grid is a
  // multiple of 8): every tile reads nearly every line of the row of t
  const int nlist = X.work[0], nwork = (nlist + 7) / 8 * 8 * X.T;
  const int lane = (int)threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  XStage<DT> stg;
  for (int q0 = (int)blockIdx.x; q0 < nwork; q0 += (int)gridDim.x) {
    const int s = q0 >> 3, lr = (s / X.T) * 8 + (q0 & 7), tile = s % X.T;
    if (lr >= nlist) continue;
    XItem it = xv_item<DT>(A, X, X.work[1 + lr], tile);
    const int32_t* ix = X.idx + (size_t)tile * (X.U + 1);
    const int u0 = (int)((long long)X.U * w / XT::kWv), u1 = (int)((long long)X.U * (w + 1) / XT::kWv);
    const int pa = ix[u0] - ix[0], pe = ix[u1] - ix[0];
    uint32_t en[kXBatch];
    #pragma unroll
    for (int k = 0; k < kXBatch; ++k) en[k] = xv_entry(it, pa + k * 64 + lane);
    const uint64_t* blk = dec_row(A, it.req, it.i);
    uint32_t cst[D_JSB + 1];
    #pragma unroll
    for (int k = 0; k <= D_JSB; ++k) cst[k] = pay(blk[k]);
    const uint32_t task = cst[D_TASK];
    const bool dj = (task & kTaskJsd) != 0u, dr = (task & kTaskRes) != 0u, db = (task & kTaskBonus) != 0u;
    const ResidConst rk = resid_const(A, cst);
    const JsdConst jk = jsd_const(cst);
    if (dj || dr) stg.load(A, it.row, tile);
    __syncthreads();   // the item before is done with the tile
    if (dj || dr) {
      stg.store(A, sm.pair);
      it.lead = stg.lead;
    }
    xv_bounds<DT>(X, it, sm);
    __syncthreads();
    xv_bounds_in<DT>(it, sm);
    float* sums = X.sums + ((size_t)it.row * X.T + tile) * X.nsub;
    int cur = u0 << (X.ulog - X.slog);
    const int send = u1 << (X.ulog - X.slog);
    JsdAcc accj{0.0f, 0.0f};
    float acc = 0.0f;
    for (int p0 = pa; p0 < pe; p0 += 64 * kXBatch) {
      float xt[kXBatch];
      int x[kXBatch];
      typename XT::Pair pr[kXBatch];
      xv_tokens<DT, 64>(it, sm, en, p0 + lane, x);
      #pragma unroll
      for (int k = 0; k < kXBatch; ++k) {
        xt[k] = dr || db ? xv_t<DT>(it, x[k]) : 0.0f;
        pr[k] = dj || dr ? xv_pair<DT>(it, sm, en[k]) : XT::masked();
      }
      #pragma unroll
      for (int k = 0; k < kXBatch; ++k) en[k] = xv_entry(it, p0 + (kXBatch + k) * 64 + lane);
      #pragma unroll
      for (int k = 0; k < kXBatch; ++k) {
        const bool in = p0 + k * 64 + lane < pe;
        if (p0 + k * 64 >= pe) break;
        const float xa = XT::a(pr[k]), xb = XT::b(pr[k]);
        // (masked: no mass in either view)
        if (dj) jsd_add<true>(accj, in ? xa : -INFINITY, in ? xb : -INFINITY, jk);
        if (dr || db) {
          float v = dr ? resid_elem<DM>(xt[k], xa, xb, rk) : bonus_elem(xt[k], rk.c, rk.Rf);
          v = in ? v : 0.0f;
          // lanes past the end follow the last token
          const int sub = in ? x[k] >> X.slog : 0x7FFFFFFF;
          // (uniform) the last sub-block among the step's tokens
          const int last = __builtin_amdgcn_readlane(sub, min(63, pe - 1 - (p0 + k * 64)));
          while (cur < last) {
            const float total = wave_sum(acc + (sub == cur ? v : 0.0f));
            if (lane == 0) sums[cur] = plain_sum(total);
            acc = 0.0f;
            ++cur;
          }
          acc += sub == cur ? v : 0.0f;
        }
      }
    }
    if (dr || db) {
      for (; cur < send; ++cur) {
        const float total = wave_sum(acc);
        if (lane == 0) sums[cur] = plain_sum(total);
        acc = 0.0f;
      }
    }
    if (dj) {
      const float wj = wave_sum(jsd_sum(accj, jk));
      if (lane == 0) sm.wj[w] = wj;
      __syncthreads();
      if (threadIdx.x == 0) {
        float v = 0.0f;
        for (int q = 0; q < XT::kWv; ++q) v += sm.wj[q];
        X.jpart[(size_t)it.row * X.T + tile] = plain_sum(v);
      }
    }
  }
}

// -------------------------------------------------------------------- pick
template <int DT, int DM>
__global__ __launch_bounds__(kThreads) void xv_pick_kernel(KArgs A, XArgs X) {
  __shared__ Smem sm;
  const XPass2 src{X.sums, X.jpart, X.T, X.nsub, X.slog};
  pick_item<DT, DM, true>(A, (int)blockIdx.x, sm, src);
}

}  // namespace asym

#endif  // ASYMSPEC_XVOCAB_H_
