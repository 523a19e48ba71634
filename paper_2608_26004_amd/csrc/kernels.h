// Addresses of the decision kernel's instances.  Each instance is compiled on
// its own (kernels.hip, once per combination), so that the build runs them in
// parallel.

#ifndef ASYMSPEC_KERNELS_H_
#define ASYMSPEC_KERNELS_H_

namespace asym {

enum { kVarBeta1 = 0, kVarBeta = 1, kVarKL = 2, kVarFull = 3 };

template <int DT, int DM, int VAR>
const void* fuse_verify_ptr();

// every specialisation, defined in its own object
#define ASYM_VARS(DT, DM)                              \
  template <> const void* fuse_verify_ptr<DT, DM, 0>(); \
  template <> const void* fuse_verify_ptr<DT, DM, 1>(); \
  template <> const void* fuse_verify_ptr<DT, DM, 2>(); \
  template <> const void* fuse_verify_ptr<DT, DM, 3>();
ASYM_VARS(0, 0) ASYM_VARS(0, 1) ASYM_VARS(0, 2)
ASYM_VARS(1, 0) ASYM_VARS(1, 1) ASYM_VARS(1, 2)
#undef ASYM_VARS

}  // namespace asym

#endif  // ASYMSPEC_KERNELS_H_
