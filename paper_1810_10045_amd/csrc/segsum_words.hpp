// The words by which waves of one Seg-Sum launch tell each other that a piece
// of a cut segment is in memory: one per chunk and column tile, in a workspace
// that is never cleared. Plain C++ over the memory operations of Mem (the
// device's agent-scope atomics in segsum_kernels.hpp), so that a host test can
// run every interleaving of them.
//
// A word: a tag that is new for every call, a flag (the chunk's own piece of a
// head is there) and a count (pieces that are there of the segment that starts
// in the chunk, at most 16). What an earlier call left carries another tag, and
// of other data one word in 2^56 carries this call's.
//
// A wave claims every word that it will add to, before its walk: it loads the
// word and, where the tag is another's, tries once to exchange what it loaded
// for this call's tag over zeros. Nothing but such an exchange ever changes a
// word of another tag, so a failed one means that another wave of the call has
// put the tag there: after it, won or lost, the word is this call's for as long
// as the call runs, and additions need no look at the tag. (Adding first and
// looking at the tag of the sum is wrong: the flag added to a stale word whose
// flag is set carries into the tag, and the tag before this call's becomes this
// call's over a stale count.)
#pragma once

#include <stdint.h>

namespace lmz {

constexpr int kTagShift = 8;
constexpr uint64_t kTagMask = (uint64_t(1) << (64 - kTagShift)) - 1;
constexpr uint64_t kPieceFlag = uint64_t(1) << (kTagShift - 1);
constexpr uint64_t kCountMask = kPieceFlag - 1;

constexpr bool word_is(uint64_t word, uint64_t tag) { return (word >> kTagShift) == tag; }
constexpr uint32_t word_count(uint64_t word) { return static_cast<uint32_t>(word & kCountMask); }

// Claim word w, of which `seen` has been loaded.
template <class Mem>
constexpr void word_claim(Mem mem, uint64_t* w, uint64_t seen, uint64_t tag) {
  if (!word_is(seen, tag)) mem.exchange_if(w, seen, tag << kTagShift);
}

// Add to a claimed word: the word after the addition.
template <class Mem>
constexpr uint64_t word_add(Mem mem, uint64_t* w, uint64_t x) {
  return mem.add(w, x) + x;
}

}  // namespace lmz
