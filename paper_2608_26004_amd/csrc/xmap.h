// Where the logits of a mapped verifier token lie (cross-family vocabularies).
//
// Plain C++ (no HIP types) so that a host-only test can check every place
// against the arrays that a call brings.

#ifndef ASYMSPEC_XMAP_H_
#define ASYMSPEC_XMAP_H_

#include <cstdint>

#ifndef ASYM_HD
#define ASYM_HD
#endif

namespace asym {

// Drafter id of verifier token x, or -1 when it has no shared counterpart (or
// x lies outside the vocabulary).
ASYM_HD inline int map_id(const int32_t* vmap, int V, int Vd, long long x) {
  if (x < 0 || x >= V) return -1;
  const int j = vmap[x];
  return (j >= 0 && j < Vd) ? j : -1;
}

// Flat places of the logits of verifier token x of row `row`: t in [rows][V],
// and ab in the drafter's [rows][Vd], or -1 with ab = false: a plain bonus row
// reads the verifier alone, and a call without drafts may bring no a and b at
// all.  A token that is not shared (in = false) has the places of token 0 and
// drafter id 0, which exist, so that a kernel may load without a branch.
struct XPlace { bool in; long long t, ab; };
ASYM_HD inline XPlace map_place(const int32_t* vmap, long long row, int V, int Vd, long long x, bool ab) {
  const int j = map_id(vmap, V, Vd, x);
  const bool in = j >= 0;
  return XPlace{in, row * V + (in ? x : 0), ab ? row * Vd + (in ? j : 0) : -1};
}

}  // namespace asym

#endif  // ASYMSPEC_XMAP_H_
