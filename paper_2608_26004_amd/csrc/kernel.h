// The decision kernel: one workgroup per work item of the launch's list.

#ifndef ASYMSPEC_KERNEL_H_
#define ASYMSPEC_KERNEL_H_

#include "device.h"
#include "resolve.h"
#include "schedule.h"
#include "stats.h"

namespace asym {

template <int DT, bool kB1, int DM, bool kKL, bool kFull>
DEV void stats_chunk(const KArgs& A, int req, int i, int m, Smem& sm) {
  const int row = req * (A.K + 1) + i;
  const float tau = sload_f32(A.tau, req);
  if (i == A.K) {
    if (A.fuse_bonus) {
      if (tau > 0.0f) stats_item<DT, kSampleBonusF, kB1, DM, false, kFull>(A, row, m, sm);
      else stats_item<DT, kGreedyBonusF, kB1, DM, false, kFull>(A, row, m, sm);
    } else if (tau > 0.0f) {
      stats_item<DT, kSampleBonus, kB1, DM, false, kFull>(A, row, m, sm);
    } else {
      stats_item<DT, kGreedyBonus, kB1, DM, false, kFull>(A, row, m, sm);
    }
  } else if (!(tau > 0.0f)) {
    stats_item<DT, kGreedyDraft, kB1, DM, kKL, kFull>(A, row, m, sm);
  } else if (tau == 1.0f) {
    stats_item<DT, kSampleDraft1, kB1, DM, kKL, kFull>(A, row, m, sm);
  } else {
    stats_item<DT, kSampleDraftT, kB1, DM, kKL, kFull>(A, row, m, sm);
  }
}

template <int DT, bool kB1, int DM, bool kKL, bool kFull>
DEV void stats_dispatch(const KArgs& A, int req, int sub, Smem& sm) {
  const int i = sub / A.S, m = sub - i * A.S;
  stats_chunk<DT, kB1, DM, kKL, kFull>(A, req, i, m, sm);
}

#ifndef ASYMSPEC_WAVES
#define ASYMSPEC_WAVES 4
#endif
#ifndef ASYMSPEC_WAVES_FULL
#define ASYMSPEC_WAVES_FULL 3
#endif

// One workgroup per item.  An item waits only for items earlier in the list
// (lower workgroup index; the kFull instances excepted), and each XCD starts its share of the workgroups in
// index order, so the lowest waiting workgroup always waits on items that are
// running or queued behind workgroups that never wait: the list drains
// whether or not every workgroup fits on the chip at once.  The waits are
// bounded besides (Poll), and a timeout is counted in the workspace.  A
// statistics item of a kFull instance also waits for the later items of its row,
// within a short bound of its own; when that runs out it leaves its rows to the
// kernel behind this one and ends, so these launches drain as well (full.h).
// kKL: calls with the KL gate, whose draft rows also sum the divergence
// beside the A slot (a kernel of its own, so that the extra registers of
// those items do not weigh on the other gates' kernels).
// kFull: calls with the full log-probability rows, whose statistics items keep
// their chunk's emission logits (64 registers a thread in bf16, so three
// workgroups per CU) and write them once the row's records are in.
template <int DT, bool kB1, int DM, bool kKL, bool kFull>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kFull ? ASYMSPEC_WAVES_FULL : ASYMSPEC_WAVES)))
void fuse_verify_kernel(KArgs A) {
  __shared__ Smem sm;
#ifdef ASYMSPEC_TRACE
  const uint64_t t_start = __builtin_amdgcn_s_memrealtime();
  if (threadIdx.x == 0) sm.t_mark[0] = sm.t_mark[1] = t_start;
#endif
  const Item it = sched_item(A.sc, A.K, A.S, (int)blockIdx.x);
  int type = it.type;
  if (type == kItemStats2) {
    // early exit: the rows after the first group are read unless the
    // verdict found a sure rejection among the first rows
    type = load_verdict(A, it.req, sm) == kVerdictSkip ? kItemNone : kItemStats;
  }
  // one call site per item kind keeps a single inlined copy of each
  switch (type) {
    case kItemStats: stats_dispatch<DT, kB1, DM, kKL, kFull>(A, it.req, it.sub, sm); break;
    case kItemVerdict:
    case kItemDecide: decide_item<DT>(A, it.req, sm, type == kItemVerdict); break;
    case kItemPass2: pass2_item<DT, DM>(A, it.req, it.sub, sm); break;
    case kItemPick: pick_item<DT, DM>(A, it.req, sm); break;
    default: break;
  }
#ifdef ASYMSPEC_TRACE
  // timeline of the launch (a build option for measurement): per item its
  // start and end on the 100 MHz clock, kind and request, and for statistics
  // items when the first streaming load went out and when the stream ended
  if (threadIdx.x == 0 && A.trace != nullptr && blockIdx.x < A.trace_items) {
    uint64_t* tr = A.trace + (size_t)blockIdx.x * 4;
    tr[0] = t_start;
    tr[1] = __builtin_amdgcn_s_memrealtime();
    tr[2] = (uint64_t)(uint32_t)it.type | ((uint64_t)(uint32_t)it.req << 8) | ((uint64_t)(uint32_t)it.sub << 40);
    tr[3] = (sm.t_mark[0] - t_start) | ((sm.t_mark[1] - t_start) << 32);
  }
#endif
}

}  // namespace asym

#endif  // ASYMSPEC_KERNEL_H_
