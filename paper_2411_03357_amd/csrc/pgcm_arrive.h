// How the workgroups of a chunk add up their shares of its tag, and, where different ones come to hold its
// words, their verdicts: the steps of a lane, for the kernels and, with another Memory, for the CPU.
// Memory has the operations on the slots, each atomic and relaxed:
//   uint64_t fetch_xor(uint64_t* at, uint64_t v), uint32_t fetch_add(uint32_t* at, uint32_t v), clear(T* at).
#pragma once
#include <stdint.h>

#include "pgcm_types.h"

#ifdef __HIPCC__
#define PGCM_STEP __host__ __device__ __forceinline__
#else
#define PGCM_STEP inline
#endif

namespace pgcm {

// Adds `word` to an accumulator that `of` workgroups add to, the caller's as number `member`, and counts it
// in, by the same atomic: the lower half holds the words added so far, the upper half a bit for each
// workgroup that has added its own.  True if that completes it: `word` is the whole sum, and the
// accumulator is left zero.
template <class Memory>
PGCM_STEP bool add_and_arrive(uint64_t* at, uint32_t member, uint32_t of, uint32_t& word) {
    const uint64_t own = (uint64_t)(1u << member) << 32 | word;
    const uint64_t now = own ^ Memory::fetch_xor(at, own);
    word = (uint32_t)now;
    const bool whole = (uint32_t)(now >> 32) == 0xFFFFFFFFu >> (32 - of);
    if (whole) Memory::clear(at);
    return whole;
}

// Word `lane` of the share of workgroup g of n, more than kArriveSet, whose slots begin at `slots`: first added
// up in sets.
template <class Memory>
PGCM_STEP bool add_in_set(ArriveSlot* slots, uint32_t g, uint32_t n, uint32_t lane, uint32_t& word) {
    const uint32_t first = g / kArriveSet * kArriveSet;
    return add_and_arrive<Memory>(&slots[first].of_set[lane], g - first,
                                  n - first < kArriveSet ? n - first : kArriveSet, word);
}
// ... and then, by who completed a set's word, or of fewer workgroups at once, for the chunk: as this number
// of so many.
struct ChunkMember {
    uint32_t number, of;
};
PGCM_STEP ChunkMember set_of_chunk(uint32_t g, uint32_t n) {
    return ChunkMember{g / kArriveSet, (n + kArriveSet - 1) / kArriveSet};
}
template <class Memory>
PGCM_STEP bool add_in_chunk(ArriveSlot* slots, ChunkMember m, uint32_t lane, uint32_t& word) {
    return add_and_arrive<Memory>(&slots->of_chunk[lane], m.number, m.of, word);
}

// Decrypting, where different workgroups completed the four words: one that completed `words` of them, and
// found a difference or not, counts them.  In the second slot, which a chunk of several workgroups has: the
// words compared, and above them the workgroups that found a difference.
template <class Memory>
PGCM_STEP uint32_t count_verdict(ArriveSlot* slots, uint32_t words, bool differs) {
    const uint32_t own = words + (differs ? 256u : 0u);
    return own + Memory::fetch_add(reinterpret_cast<uint32_t*>(slots[1].of_chunk), own);
}
// Of what that returned: are all words compared?  Then the caller ends the chunk, with this verdict, and clears
// the count.
PGCM_STEP bool verdict_whole(uint32_t count) { return count % 256 == 4; }
PGCM_STEP bool verdict_differs(uint32_t count) { return count >= 256; }
template <class Memory>
PGCM_STEP void clear_verdict(ArriveSlot* slots) {
    Memory::clear(reinterpret_cast<uint32_t*>(slots[1].of_chunk));
}

}  // namespace pgcm
