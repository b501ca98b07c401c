// Arrival words of a launch whose last workgroup merges: tag of the launch in the upper 48 bits, arrivals below.
//
// A workspace may hold any bytes, and a launch of one kernel has nobody before it who could clear its words: a word that does not
// carry the launch's own tag counts as no arrivals yet.  What a workspace holds is mostly small integers (index lists, counters) and
// floats, so that tags that count up from 1 would be met there: they are spread over all 48 bits, from a start that differs from
// process to process.
#pragma once

#include <atomic>
#include <chrono>
#include <stdint.h>

namespace antkv {

constexpr int kArrivalBits = 16;                                   // a launch has fewer than 2^16 workgroups per word
constexpr uint64_t kArrivalMask = (1ull << kArrivalBits) - 1;
constexpr uint64_t kTagMask = ~0ull >> kArrivalBits;

// one-to-one on 48-bit numbers: every step can be undone (the factors, from the digits of sqrt 2 and e, are odd)
constexpr uint64_t spread48(uint64_t x)
{
    x &= kTagMask;
    x ^= x >> 23;
    x = x * 0x6A09E667F3BDull & kTagMask;
    x ^= x >> 21;
    x = x * 0xB7E151628AEDull & kTagMask;
    return x ^ x >> 25;
}

// the word is not one of this launch's, or a replay of the same launch finds all `most` arrivals of the last time
constexpr bool arrivals_are_stale(uint64_t word, uint64_t tag, uint32_t most) { return (word ^ tag) >= most; }

// no two of a process are the same (short of 2^48); the arrival bits are 0
inline uint64_t next_launch_tag() noexcept
{
    static std::atomic<uint64_t> counter{spread48((uint64_t)std::chrono::system_clock::now().time_since_epoch().count() ^
                                                  (uint64_t)(uintptr_t)&spread48)};
    return spread48(counter.fetch_add(1, std::memory_order_relaxed)) << kArrivalBits;
}

}  // namespace antkv
