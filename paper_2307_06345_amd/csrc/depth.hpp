// How deep a split sort's top digits go: which keys are sampled and what their
// pairs say, in plain C++ (constexpr functions run on the device and on the host).
#pragma once

#include <cstdint>

namespace cs {

// The split sort's three top digits leave buckets of one 27-bit prefix. Where
// many keys share theirs with hundreds of others (a cluster's core), the bucket
// kernel and the low passes over listed buckets cost more than one more digit
// pass below the top ones, after which the buckets are those of one 36-bit
// prefix. The size of the bucket that a key finds itself in, on average over
// the keys, tells: n times the share of pairs of keys with one prefix, less the
// pairs that the next digit does not part either (heaps of equal keys gain
// nothing by it).
constexpr uint32_t kDeepSample = 2048;
// Mean bucket from which the extra digit pays. Sorts of Plummer keys, three top
// digits against four: 2^18 keys (mean 6.5) 101 / 109 us, 2^20 (23) 154 / 136,
// 2^22 (89) 255 / 207, 2^24 (354) 742 / 581, 2^27 (2828) 6149 / 3985; uniform
// 2^24 (1.1) 468 / 568. In proportion it pays from 12 on; the estimate at 2^20 lies
// between 17 and 31.
constexpr uint32_t kDeepBucket = 12;
constexpr uint32_t kDeepPairs = 4;  // fewer pairs in the sample may be chance
constexpr uint32_t kDeepMinKeys = 1u << 20;  // shorter sorts gain less than the extra launch costs where it is left out

// Place of the i-th sampled key: in one of kDeepShares equal shares of the keys,
// anywhere in it. Samples of one share pair as those of all keys do, so the
// buckets of keys that come in order are seen as well as those of scattered ones
// (a share each would hide them: two samples hardly meet in a bucket), and a
// wave's reads stay on a few pages (anywhere in 2^24 keys: 5 us more).
constexpr uint32_t kDeepShares = 64;
constexpr uint64_t depth_place(uint32_t i, uint64_t n) {
    uint32_t h = i + 0x9e3779b9u;  // the number's bits mixed: two rounds of a shift and an odd multiplier
    h = (h ^ (h >> 16)) * 0x7feb352du;
    h = (h ^ (h >> 15)) * 0x846ca68bu;
    h ^= h >> 16;
    const uint64_t share = i / (kDeepSample / kDeepShares);
    const uint64_t from = n * share / kDeepShares, to = n * (share + 1) / kDeepShares;
    return from + ((h * (to - from)) >> 32);
}

// Of a sampled key: its prefix (and 1, so that no word is 0), the digit below it
// and room for a count in the low bits.
constexpr uint64_t depth_word(uint64_t key) { return ((key >> 36) + 1) << 32 | ((key >> 27) & 511u) << 8; }
constexpr uint64_t kDepthCount = 15;  // bits of the count, and the most that is counted
constexpr bool depth_one_prefix(uint64_t a, uint64_t b) { return a >> 32 == b >> 32; }
constexpr bool depth_one_digit(uint64_t a, uint64_t b) { return (a & ~kDepthCount) == (b & ~kDepthCount); }

// pairs: pairs of sampled keys with one prefix; with_first: those with the first
// key of their prefix, of which `together` share its next digit too.
constexpr bool depth_pays(uint64_t pairs, uint64_t with_first, uint64_t together, uint64_t n) {
    const uint64_t parted = with_first ? pairs * (with_first - together) / with_first : 0;
    return parted >= kDeepPairs && 2 * parted * n >= static_cast<uint64_t>(kDeepBucket) * kDeepSample * kDeepSample;
}

}  // namespace cs
