// One instance of the decision kernel: storage type ASYMSPEC_PART_DT, source
// of delta ASYMSPEC_PART_DM, variant ASYMSPEC_PART_VAR (set by the build).

#include <hip/hip_runtime.h>

#include "asymspec.h"
#include "kernel.h"
#include "kernels.h"

namespace asym {

template <>
const void* fuse_verify_ptr<ASYMSPEC_PART_DT, ASYMSPEC_PART_DM, ASYMSPEC_PART_VAR>() {
  constexpr bool kB1 = ASYMSPEC_PART_VAR == kVarBeta1, kKL = ASYMSPEC_PART_VAR == kVarKL;
  constexpr bool kFull = ASYMSPEC_PART_VAR == kVarFull;
  return (const void*)fuse_verify_kernel<ASYMSPEC_PART_DT, kB1, ASYMSPEC_PART_DM, kKL, kFull>;
}

}  // namespace asym
