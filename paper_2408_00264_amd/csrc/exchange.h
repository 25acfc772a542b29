// How the workgroups that share a result meet: each of S of them leaves its part in memory, and each finishes one share of the whole.
//
// One word per result: arrivals (bits 0 .. 7), members that left without finishing their share (bits 8 .. 23, S <= 16), and a count of
// finished meetings above, which tells a meeting from the next in the same word.  Zero before the first; the last arrival readies it for
// the next launch, so a launch that is replayed (a captured graph) finds it as the first did.
//
// Nobody waits without an end.  A member that has looked `polls` times without seeing all others leaves its share behind by setting
// its bit -- only while arrivals are missing, in one step with that test -- and the last arrival, whose own step returns the bits,
// finishes those shares as well.  So it makes no difference to the results whether all members run at once (another launch may hold
// the compute units that some of them need), only to the time.
#pragma once

// Returns the shares that the caller has to finish, bit i for member i's.  Word: add(v) and load() return the word (add: before it),
// store(v), swap(from, to): true if it held `from`.
template <class Word>
__device__ __forceinline__ unsigned meet(Word word, unsigned S, unsigned member, int polls) {
  const unsigned before = word.add(1u), own = 1u << member;
  if ((before & 255u) == S - 1u) {
    word.store((before & 0xff000000u) + 0x1000000u);   // (nobody writes it any more: all have arrived, and so nobody leaves)
    return own | (before >> 8 & 0xffffu);
  }
  auto all_here = [&](unsigned w) { return (w & 255u) == S || (w ^ before) >> 24 != 0u; };
  for (int i = 0; i < polls; ++i)
    if (all_here(word.load())) return own;
  for (;;) {   // (a swap fails only where another member arrived or left since: fewer than 2 S times)
    const unsigned w = word.load();
    if (all_here(w)) return own;
    if (word.swap(w, w | own << 8)) return 0u;
  }
}
