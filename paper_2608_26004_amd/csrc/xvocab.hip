// The kernels of a cross-family call for storage type ASYMSPEC_PART_DT (set by
// the build), and their launches.

#include <hip/hip_runtime.h>

#include <algorithm>

#include "asymspec.h"
#include "xvocab.h"
#include "xvocab_host.h"

namespace asym {

template <>
size_t xv_layout<ASYMSPEC_PART_DT>(int B, int K, int V, int Vd, XLayout& L) {
  constexpr int kN = XTile<ASYMSPEC_PART_DT>::kN;
  L.T = (Vd + kN - 1) / kN;
  L.ulog = x_unit_log(V);
  L.U = ((V - 1) >> L.ulog) + 1;
  const size_t rows = (size_t)B * (K + 1);
  L.slog = x_sub_log(L.U, L.ulog, rows * L.T);
  L.nsub = L.U << (L.ulog - L.slog);
  size_t off = 0;
  auto take = [&](size_t n) { const size_t at = off; off = (off + n + 255) / 256 * 256; return at; };
  L.off_list = take((size_t)V * 4);
  L.off_cnt = take((size_t)L.T * L.U * 4);
  L.off_idx = take((size_t)L.T * (L.U + 1) * 4);
  L.off_sums = take(rows * L.T * L.nsub * 4);
  L.off_jpart = take(rows * L.T * 4);
  L.off_work = take((rows + 1) * 4);
  return off;
}

template <int DT, int DM>
static hipError_t launch(KArgs A, const XLayout& L, char* base, int ee_rows, int n_cu, hipStream_t st) {
  XArgs X;
  X.list = (uint32_t*)(base + L.off_list);
  X.cnt = (int32_t*)(base + L.off_cnt);
  X.idx = (int32_t*)(base + L.off_idx);
  X.sums = (float*)(base + L.off_sums);
  X.jpart = (float*)(base + L.off_jpart);
  X.work = (int32_t*)(base + L.off_work);
  X.T = L.T; X.U = L.U; X.nsub = L.nsub; X.ulog = L.ulog; X.slog = L.slog;
  X.tlog = 0;
  while ((1 << X.tlog) < X.T) ++X.tlog;
  const int nrow = A.K + 1;
  A.S = X.T;                   // records per row
  A.full_poll = 1;
  A.sc.ee = (ee_rows >= 1 && ee_rows < nrow) ? 1 : 0;
  A.sc.G = A.sc.ee ? ee_rows : nrow;
  constexpr int kThr = XTile<DT>::kThr;
  // the statistics of rows [r0, r1) of every request: one workgroup per (row,
  // tile), in launches of fewer than 2^32 threads, the most HIP takes (a multiple
  // of 8 blocks each, so that a row's tiles stay on one XCD)
  constexpr long long kMost = ((1LL << 32) / kThr - 1) / 8 * 8;
  auto blocks = [&](int r0, int r1) { return ((long long)A.B * (r1 - r0) + 7) / 8 * 8 * X.T; };
  auto stats = [&](int r0, int r1) {
    X.r0 = r0;
    X.r1 = r1;
    for (long long b0 = 0, n = blocks(r0, r1); b0 < n; b0 += kMost) {
      X.b0 = (unsigned)b0;
      hipLaunchKernelGGL((xv_stats_kernel<DT, DM>), dim3((unsigned)std::min(kMost, n - b0)), dim3(kThr), 0, st, A, X);
    }
  };
  hipLaunchKernelGGL((xv_count_kernel<DT>), dim3(L.U), dim3(kXListThr), 0, st, A, X);
  hipLaunchKernelGGL((xv_fill_kernel<DT>), dim3(L.U), dim3(kXListThr), 0, st, A, X);
  stats(0, A.sc.G);
  if (A.sc.ee) {
    hipLaunchKernelGGL((xv_decide_kernel<DT>), dim3(A.B), dim3(kThreads), 0, st, A, X, 1);
    stats(A.sc.G, nrow);
  }
  hipLaunchKernelGGL((xv_decide_kernel<DT>), dim3(A.B), dim3(kThreads), 0, st, A, X, 0);
  // pass 2: what the chip holds at once (two workgroups per CU), a multiple of 8
  const long long g2 = std::min(blocks(0, nrow), (long long)std::max(8, 2 * n_cu / 8 * 8));
  hipLaunchKernelGGL((xv_pass2_kernel<DT, DM>), dim3((unsigned)g2), dim3(kThr), 0, st, A, X);
  hipLaunchKernelGGL((xv_pick_kernel<DT, DM>), dim3(A.B), dim3(kThreads), 0, st, A, X);
  return hipGetLastError();
}

template <>
hipError_t xv_launch<ASYMSPEC_PART_DT>(const KArgs& A, const XLayout& L, char* base, int ee_rows, int n_cu,
                                       hipStream_t st) {
  constexpr int DT = ASYMSPEC_PART_DT;
  if (A.delta_mode == kDeltaA) return launch<DT, kDeltaA>(A, L, base, ee_rows, n_cu, st);
  if (A.delta_mode == kDeltaTB) return launch<DT, kDeltaTB>(A, L, base, ee_rows, n_cu, st);
  return launch<DT, kDeltaAB>(A, L, base, ee_rows, n_cu, st);
}

}  // namespace asym
