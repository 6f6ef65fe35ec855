// The claim word of the device-driven solve: how a published superstep's tile
// list is handed out in pieces.  Host code too: the protocol is stepped
// through on the CPU by a test.
#pragma once

#include <stdint.h>

namespace pmf {

// The word is {count | superstep tag | batch, next}.  The high half describes
// the superstep and only its publisher writes it; a claim adds an amount to
// the low half and is answered with the word as it was.  The tag is the number
// of supersteps the instance has left in the launch (at most 65536), so that
// no two supersteps of a launch have the same high half.
constexpr int kClCountBits = 10, kClCountMax = (1 << kClCountBits) - 1;
constexpr int kClTags = 1 << (28 - kClCountBits);
constexpr int kClBatchMax = 16;
constexpr uint32_t claim_hi(int count, int tag, int batch) {
    return (uint32_t)count | ((uint32_t)(tag & (kClTags - 1)) << kClCountBits) | ((uint32_t)(batch - 1) << 28);
}
constexpr int claim_count(uint32_t hi) { return (int)(hi & (uint32_t)kClCountMax); }
constexpr int claim_batch(uint32_t hi) { return (int)(hi >> 28) + 1; }

// Entries [first, first + n) of the list of the superstep `hi`; n = 0: none were
// left.  last: the list's last entry is among them.
struct Claim {
    uint32_t hi;
    int first, n;
    bool last;
};

// What a claim that added `added` and was answered with `old` has got: as many
// entries as it added, whatever the batch of the superstep it got them from.
// The amount is that of an earlier look at the word, and another superstep
// with another batch may have been published in between; only if every claim
// takes what it added do the claims of a superstep cover its list once.
constexpr Claim claim_take(uint64_t old, int added) {
    const uint32_t hi = (uint32_t)(old >> 32), next = (uint32_t)old;
    const uint32_t count = (uint32_t)claim_count(hi);
    if (next >= count) return Claim{hi, 0, 0, false};
    const uint32_t left = count - next;
    return Claim{hi, (int)next, (int)((uint32_t)added < left ? (uint32_t)added : left), (uint32_t)added >= left};
}

}  // namespace pmf
