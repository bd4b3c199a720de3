// The words through which the workgroups of the one-launch score + decision + compaction kernel (rules NONE and THRESHOLD) hand each other
// the chunks' decisions, and what a reader takes from them. Plain C++ for the host and the device: the kernel uses these functions, and
// a host program (staging_check.cpp) steps the same exchange with a key missing.
//
// Two 64-bit words per chunk of 64 rows, zero at the start, each valid on its own (one relaxed device-scope access each):
//   word 0 = kept mask bits 0..31 | kept count << 32 | FAILED | READY      word 1 = kept mask bits 32..63 | FAILED | READY
// FAILED: the publisher gave up and its mask means nothing (those of NONE and THRESHOLD wait for nothing and never do).
#pragma once

#include "staging_addr.h"

namespace dash {

constexpr unsigned long long kPubReady = 1ull << 62, kPubFailed = 1ull << 61;

DASH_HD unsigned long long pub_word0(unsigned long long mask, int count, bool failed) {
    return failed ? kPubReady | kPubFailed : (mask & 0xFFFFFFFFull) | ((unsigned long long)count << 32) | kPubReady;
}
DASH_HD unsigned long long pub_word1(unsigned long long mask, bool failed) {
    return failed ? kPubReady | kPubFailed : (mask >> 32) | kPubReady;
}
// A word that never became READY (the bounded wait ended), or that says FAILED: the reader fails as well.
DASH_HD bool pub_bad(unsigned long long w) { return (w & (kPubReady | kPubFailed)) != kPubReady; }
DASH_HD unsigned long long pub_mask(unsigned long long w0, unsigned long long w1) {
    return (w0 & 0xFFFFFFFFull) | ((w1 & 0xFFFFFFFFull) << 32);
}
DASH_HD int pub_count(unsigned long long w0) { return (int)((w0 >> 32) & 0x7Full); }

}  // namespace dash
