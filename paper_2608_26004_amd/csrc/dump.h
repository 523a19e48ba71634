// Full log-probability rows by a second kernel on the same stream, after the
// decision: every row is streamed once more and written with the normaliser
// that the decide items published (the kernel boundary orders them).  For the
// calls whose statistics items do not write them (full.h): cross-family calls
// and the KL gate, whose instances have no registers left to keep a chunk.
//
// One workgroup per (row, chunk); thread j takes vectors j, j + 256, ... of
// the chunk, so each load and store instruction of a wave covers contiguous
// memory.

#ifndef ASYMSPEC_DUMP_H_
#define ASYMSPEC_DUMP_H_

#include "device.h"
#include "full.h"
#include "schedule.h"

namespace asym {

template <int DT, int DM>
__global__ __launch_bounds__(kThreads) void dump_kernel(KArgs A, float* out) {
  const int S = A.S, nrow = A.K + 1;
  // through a vocabulary map, the workgroups one XCD runs take consecutive
  // chunks of the same rows (each chunk gathers from the whole drafter row)
  const int b = A.vmap != nullptr ? xcd_grouped((int)blockIdx.x, (int)gridDim.x) : (int)blockIdx.x;
  const int row = b / S;
  const int m = b - row * S;
  const int req = row / nrow, i = row - req * nrow;
  const uint64_t* blk = dec_row(A, req, i);
  const double c = (double)payf(blk[D_C]);
  const double l2 = payd(blk[D_L2E_LO], blk[D_L2E_HI]);
  const bool fused = i < A.K || A.fuse_bonus != 0;
  // b is a bitwise copy of a on a row whose views never differ
  const bool nb = (pay(blk[D_STATUS]) & kStNeq) != 0u;
  if (A.vmap != nullptr) full_chunk<DT, DM, true>(A, out, row_span<DT>(A, row), m, fused, nb, c, l2);
  else full_chunk<DT, DM, false>(A, out, row_span<DT>(A, row), m, fused, nb, c, l2);
}

// Behind a decision kernel whose statistics items write the full rows: the rows
// of the requests that some item left (H_FULL), all of them, read again.  A fixed
// grid that ends at one word when nothing is left, as in nearly every call.
template <int DT, int DM>
__global__ __launch_bounds__(kThreads) void full_rest_kernel(KArgs A) {
  if (!tag_ok(*full_late(A), A.epoch)) return;
  const int S = A.S, nrow = A.K + 1;
  const long long nblk = (long long)A.B * nrow * S;
  for (long long b = blockIdx.x; b < nblk; b += gridDim.x) {
    const int row = (int)(b / S), m = (int)(b - (long long)row * S);
    const int req = row / nrow, i = row - req * nrow;
    const uint64_t* hdr = dec_hdr(A, req);
    // (a request whose decision failed is marked invalid and has no normalisers)
    if (!tag_ok(hdr[H_FULL], A.epoch) || !tag_ok(hdr[H_STATE], A.epoch) || pay(hdr[H_STATE]) == kStateFailed) continue;
    const uint64_t* blk = dec_row(A, req, i);
    const bool fused = i < A.K || A.fuse_bonus != 0;
    full_chunk<DT, DM, false>(A, A.full, row_span<DT>(A, row), m, fused, (pay(blk[D_STATUS]) & kStNeq) != 0u,
                              (double)payf(blk[D_C]), payd(blk[D_L2E_LO], blk[D_L2E_HI]));
  }
}

}  // namespace asym

#endif  // ASYMSPEC_DUMP_H_
