// The words through which the workgroups of the one-launch score + decision + compaction kernel (rules NONE and THRESHOLD) hand each other
// the chunks' decisions, and what a reader takes from them; and the keys of rule TOPK. Plain C++ for the host and the device: the kernels use
// these functions, and host programs (publish_check.cpp) step the same exchanges with a word missing.
//
// Two 64-bit words per chunk of 64 rows, zero at the start, each valid on its own (one relaxed device-scope access each):
//   word 0 = kept mask bits 0..31 | kept count << 32 | READY      word 1 = kept mask bits 32..63 | READY
// A reader whose bounded wait ends without READY fails the call; publishers publish without having waited.
#pragma once

#include "staging_addr.h"

namespace dash {

constexpr unsigned long long kPubReady = 1ull << 62;

DASH_HD unsigned long long pub_word0(unsigned long long mask, int count) {
    return (mask & 0xFFFFFFFFull) | ((unsigned long long)count << 32) | kPubReady;
}
DASH_HD unsigned long long pub_word1(unsigned long long mask) { return (mask >> 32) | kPubReady; }
DASH_HD bool pub_ready(unsigned long long w) { return (w & kPubReady) != 0; }
DASH_HD unsigned long long pub_mask(unsigned long long w0, unsigned long long w1) {
    return (w0 & 0xFFFFFFFFull) | ((w1 & 0xFFFFFFFFull) << 32);
}
DASH_HD int pub_count(unsigned long long w0) { return (int)((w0 >> 32) & 0x7Full); }

// Rule TOPK (topk_compact_kernel): one 32-bit word per row, its score's key, zero at the start. No key is 0, so a word is its own READY
// flag. Keys u of a thread are rows u * stride + tid; a key whose word is still 0 when it has been asked for kKeyAsks times (a trip to
// memory each: tens of microseconds in all, several times what the whole launch takes) is made from its row's norm pairs, which the launch before has written. So nothing
// depends on when, or whether, the word's writer gets onto the chip: the XCDs take their workgroups each at its own pace, and beside
// calls on other streams a writer may start long after those that ask for its words.
// ask(row): the row's word; own(row): its key from the pairs; rest(): between two rounds of asking.
#if defined(__clang__)
#define DASH_UNROLL _Pragma("unroll")
#else
#define DASH_UNROLL
#endif
constexpr int kKeyAsks = 64;
template <int B, class Ask, class Own, class Rest>
DASH_HD void take_keys(uint32_t (&key)[B], int tid, int stride, int n, Ask ask, Own own, Rest rest) {
    DASH_UNROLL
    for (int u = 0; u < B; ++u) key[u] = 0u;
    for (int asks = 1;; ++asks) {  // all of a thread's words at once, and those that had not arrived again together
        DASH_UNROLL
        for (int u = 0; u < B; ++u)
            if (u * stride + tid < n && key[u] == 0u) key[u] = ask(u * stride + tid);
        bool all = true;
        DASH_UNROLL
        for (int u = 0; u < B; ++u) all = all && (key[u] != 0u || u * stride + tid >= n);
        if (all) return;
        if (asks == kKeyAsks) break;
        rest();
    }
    DASH_UNROLL
    for (int u = 0; u < B; ++u)
        if (u * stride + tid < n && key[u] == 0u) key[u] = own(u * stride + tid);
}

}  // namespace dash
