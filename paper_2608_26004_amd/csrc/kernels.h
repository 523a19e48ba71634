// Addresses of the decision kernel's instances.  Each instance is compiled on
// its own (kernels.hip, once per combination), so that the build runs them in
// parallel.

#ifndef ASYMSPEC_KERNELS_H_
#define ASYMSPEC_KERNELS_H_

namespace asym {

enum { kVarBeta1 = 0, kVarBeta = 1, kVarKL = 2, kVarFull = 3 };

template <int DT, int DM, int VAR>
const void* fuse_verify_ptr();

}  // namespace asym

#endif  // ASYMSPEC_KERNELS_H_
