// Epochs, and the untagged words that share a workspace with tagged slots.
//
// A tagged slot counts as written when its high word is the call's epoch.
// Cross-family calls also keep plain 32-bit words (list entries and indices,
// weight sums, divergence partials) in the workspace, which a later call of
// another shape or kind may read as the high words of its slots.  So every epoch
// has bits 31 and 30 set and no plain word has both.
//
// Plain C++ (no HIP types) so that a host-only test can check both sides.

#ifndef ASYMSPEC_TAGS_H_
#define ASYMSPEC_TAGS_H_

#include <cstdint>

#ifndef ASYM_HD
#define ASYM_HD
#endif

namespace asym {

constexpr uint32_t kEpochBits = 0xC0000000u;

// Epoch of the n-th call.
ASYM_HD inline uint32_t epoch_of(uint32_t n) { return n | kEpochBits; }

// A sum of terms that are not negative, as a plain word: rounding residues
// below zero, -0 and values that are not a number become +0.
ASYM_HD inline float plain_sum(float v) { return v > 0.0f ? v : 0.0f; }

// Entry of a drafter tile's token list: the drafter id within the tile (low
// JBITS bits) and the verifier token modulo kSpan, whose quotient follows from
// the entry's place in the list.  kSpan is three quarters of what the bits
// hold, which keeps both top bits from being set.  (One bit less for the token
// would keep bit 31 clear, but then a vocabulary of 151936 tokens has a quotient
// in bf16: 326 us against 315 at B = 128, K = 6, Vd = 128256.)
template <int JBITS>
struct XEntry {
  static constexpr uint32_t kSpan = 3u << (30 - JBITS);
  ASYM_HD static uint32_t make(uint32_t x, uint32_t j) { return ((x % kSpan) << JBITS) | j; }
  ASYM_HD static uint32_t token(uint32_t e) { return e >> JBITS; }
  ASYM_HD static uint32_t id(uint32_t e) { return e & ((1u << JBITS) - 1u); }
};

}  // namespace asym

#endif  // ASYMSPEC_TAGS_H_
