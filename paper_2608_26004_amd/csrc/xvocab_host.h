// Host interface of the cross-family kernels (xvocab.hip, one object per
// storage type).

#ifndef ASYMSPEC_XVOCAB_HOST_H_
#define ASYMSPEC_XVOCAB_HOST_H_

#include <hip/hip_runtime.h>

#include "device.h"

namespace asym {

// Places of a cross-family call's own arrays within its part of the workspace.
struct XLayout {
  int T, U, nsub;   // drafter tiles; list units and pass-2 sub-blocks per row
  int ulog, slog;   // of 2^ulog and 2^slog verifier tokens
  size_t off_list, off_cnt, off_idx, off_sums, off_jpart, off_work;
};

// Fills L and returns the bytes of that part.
template <int DT>
size_t xv_layout(int B, int K, int V, int Vd, XLayout& L);

// Enqueues the whole step (the full rows excepted) on st.  base: this call's
// part of the workspace; ee_rows: rows read before the verdict, 0 for all.
template <int DT>
hipError_t xv_launch(const KArgs& A, const XLayout& L, char* base, int ee_rows, int n_cu, hipStream_t st);

template <> size_t xv_layout<ASYMSPEC_BF16>(int, int, int, int, XLayout&);
template <> size_t xv_layout<ASYMSPEC_FP32>(int, int, int, int, XLayout&);
template <> hipError_t xv_launch<ASYMSPEC_BF16>(const KArgs&, const XLayout&, char*, int, int, hipStream_t);
template <> hipError_t xv_launch<ASYMSPEC_FP32>(const KArgs&, const XLayout&, char*, int, int, hipStream_t);

}  // namespace asym

#endif  // ASYMSPEC_XVOCAB_HOST_H_
