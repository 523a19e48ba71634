// Full-vocabulary fused log-probabilities (optional output): every element's
// log-probability under the distribution its row defines,
//   rows i < K   log softmax(f_i / tau), f_i = t_i + beta delta_i (Eq. 1-2),
//   row K        log softmax(t_K / tau) (Alg. 1 bonus row), or of f_K when the
//                bonus row is fused,
// at tau = 1 for greedy requests.  A token whose fused logit is not a number
// (a = b = -inf) gets -inf, as everywhere else.
//
// The statistics items write them (full_norm, full_store): an item keeps the
// emission logits of its chunk in registers, publishes its record, waits for
// the records of the row's other chunks, and writes the chunk from the
// registers, so that the logits are read from HBM once.  Bound by the mixed
// read and write rate: B = 128, K = 6, V = 151936 bf16 moves 1284 MB in 277 us
// (4.6 TB/s; a plain copy reaches 4.8), where a second kernel that read the
// rows again (2.02 GB in all) took 399.

#ifndef ASYMSPEC_FULL_H_
#define ASYMSPEC_FULL_H_

#include "device.h"

namespace asym {

typedef float f4v __attribute__((ext_vector_type(4)));

// One output element: (x c - L2) ln 2, in double (c = log2(e) / tau).
DEV float full_elem(float x, double c, double l2) {
  const float r = (float)(((double)x * c - l2) * kLn2);
  return r != r ? -INFINITY : r;
}

// Writes vector rel (counted from the row's first vector), of emission logits
// x; elements of a boundary vector that belong to the neighbouring row are
// left to that row.
template <int DT>
DEV void full_put(const KArgs& A, float* out, const RowGeo& g, long long rel, const float* x, double c, double l2) {
  constexpr int VE = Elem<DT>::VE;
  const long long f0 = (g.vbeg + rel) * VE;   // flat index of the vector's first element
  float r[VE];
  #pragma unroll
  for (int e = 0; e < VE; ++e) r[e] = full_elem(x[e], c, l2);
  if (f0 >= g.e0 && f0 + VE <= g.e0 + A.V) {
    #pragma unroll
    for (int q = 0; q < VE / 4; ++q) {
      const f4v w = {r[4 * q], r[4 * q + 1], r[4 * q + 2], r[4 * q + 3]};
      __builtin_nontemporal_store(w, reinterpret_cast<f4v*>(out + f0) + q);
    }
  } else {
    #pragma unroll
    for (int e = 0; e < VE; ++e)
      if (f0 + e >= g.e0 && f0 + e < g.e0 + A.V) out[f0 + e] = r[e];
  }
}
template <int DT>
DEV void full_store(const KArgs& A, const RowGeo& g, int rel, const float* x, double c, double l2) {
  full_put<DT>(A, A.full, g, rel, x, c, l2);
}

// Bound of an item's wait for the other items of its row, in ticks of the 100 MHz
// clock (0.5 ms; a whole call of B = 128, K = 6, V = 151936 takes 0.28): an item
// that runs late only costs a second read of its request.
constexpr uint64_t kFullTicks = 50000;
// Polls of one lane within that bound; over at once when another item of the
// call has already run late.
struct FullPoll {
  uint64_t t0;
  int n;
  DEV FullPoll() : t0(__builtin_amdgcn_s_memrealtime()), n(0) {}
  DEV bool again(const KArgs& A) {
    const int reps = 1 << (n < kPollMaxShift ? n : kPollMaxShift);
    for (int i = 0; i < reps; ++i) __builtin_amdgcn_s_sleep(2);
    ++n;
    if (tag_ok(ld_tag(full_late(A)), A.epoch)) return false;
    const uint64_t most = A.poll_ticks < kFullTicks ? A.poll_ticks : kFullTicks;
    return __builtin_amdgcn_s_memrealtime() - t0 <= most;
  }
};
// The fp32 value in the tagged slot at p; ok is cleared when it came too late.
DEV float full_wait(const uint64_t* p, const KArgs& A, FullPoll& pl, bool& ok) {
  uint64_t v = ld_tag(p);
  while (ok && !tag_ok(v, A.epoch)) {
    ok = pl.again(A);
    v = ld_tag(p);
  }
  return payf(v);
}

// The log2 normaliser of row g's emission distribution (slot `slot`) from the
// records of all its chunks: wave 0 waits for them.  False, in every thread,
// when they came too late: the chunk is then left to full_rest_kernel, which
// runs behind this kernel and writes the marked requests' rows (H_FULL).
//
// The items of a row wait for each other, also for later ones.  They are
// neighbours in the list, each XCD starts its share of the workgroups in list
// order and holds more of them (at least 64) than the at most 33 that a row of up
// to 256 chunks puts there, so in a launch that has the chip to itself the items
// of the oldest unfinished row are always started.  Beside another launch they
// need not be: two calls on two streams can each hold the slots that the other's
// oldest row needs.  So the wait is short, counts as no error, and the first item
// to run late stops every other one of its call from waiting.
template <int SLOT>
DEV bool full_norm(const KArgs& A, const RowGeo& g, Smem& sm, double& l2) {
  const int lane = lane_id();
  if (wave_id() == 0) {
    const uint64_t* base = A.rec1 + (size_t)g.row * A.S * kR1;
    float R = kFloorM;
    double sum = 0.0;
    bool ok = true;
    FullPoll pl;
    // first every record's reference, then the sums against the largest
    for (int ch = lane; ch < A.S; ch += 64) R = fmaxf(R, full_wait(base + (size_t)ch * kR1 + R1_R + SLOT, A, pl, ok));
    R = wave_max(R);
    for (int ch = lane; ch < A.S; ch += 64) {
      const float r = payf(ld_tag(base + (size_t)ch * kR1 + R1_R + SLOT));
      sum += (double)(full_wait(base + (size_t)ch * kR1 + R1_S + SLOT, A, pl, ok) * __builtin_amdgcn_exp2f(r - R));
    }
    sum = wave_sum_d(sum);
    const bool in = __all(ok);
    if (lane == 0) {
      sm.dd[0] = (double)R + log2_dbl(sum);
      sm.flags[0] = in ? 1 : 0;
      if (!in) {
        st_tag(dec_hdr(A, g.req) + H_FULL, 1u, A.epoch);
        st_tag(full_late(A), 1u, A.epoch);
      }
    }
  }
  __syncthreads();
  l2 = sm.dd[0];
  return sm.flags[0] != 0;
}

// Chunk m of row g read (again) and written.  nb: b differs from a somewhere in
// the row.  kXv: a cross-family call, a and b gathered through the map.
template <int DT, int DM, bool kXv>
DEV void full_chunk(const KArgs& A, float* out, const RowGeo& g, int m, bool fused, bool nb, double c, double l2) {
  constexpr int VE = Elem<DT>::VE;
  constexpr int kPerThread = kChunkVec / kThreads;
  const __amdgpu_buffer_rsrc_t rt = row_rsrc(A, A.t, g);
  const __amdgpu_buffer_rsrc_t ra = row_rsrc(A, kXv ? A.t : A.a, g);
  const __amdgpu_buffer_rsrc_t rb = row_rsrc(A, kXv ? A.t : A.b, g);
  const long long v0 = (long long)m * kChunkVec;
  const long long c0 = g.vbeg + v0;
  const bool tail = has_tail(A, c0, c0 + kChunkVec);
  const int tid = (int)threadIdx.x;
  #pragma unroll 2
  for (int k = 0; k < kPerThread; ++k) {
    const long long rel = v0 + tid + (long long)k * kThreads;
    const long long vi = g.vbeg + rel;
    if (vi >= g.vend) break;
    const uint32_t off = (uint32_t)(rel * 16);
    u4 vt = buf_load_nt(rt, off), va = vt, vb = vt;
    if (kXv) {
      fix_vec<DT>(A, g, A.t, vi, vt);
      map_vecs<DT>(A, g, vi, vt, va, vb, fused);
    } else if (fused) {
      va = buf_load_nt(ra, off);
      vb = nb ? buf_load_nt(rb, off) : va;
    }
    if (tail && !kXv) {
      fix_vec<DT>(A, g, A.t, vi, vt);
      if (fused) {
        fix_vec<DT>(A, g, A.a, vi, va);
        if (nb) fix_vec<DT>(A, g, A.b, vi, vb);
        else vb = va;
      }
    }
    float x[VE];
    #pragma unroll
    for (int e = 0; e < VE; ++e) {
      const float xt = Elem<DT>::get(vt, e);
      x[e] = fused ? fuse<DM>(xt, Elem<DT>::get(va, e), Elem<DT>::get(vb, e), A.beta) : xt;
    }
    full_put<DT>(A, out, g, rel, x, c, l2);
  }
}

}  // namespace asym

#endif  // ASYMSPEC_FULL_H_
