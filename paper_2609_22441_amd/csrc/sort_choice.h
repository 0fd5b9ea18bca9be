// Which kernels sort a call: the automatic choice of the affinity-record sort (CC_SORT_AUTO), from the
// call's sizes alone. Host code without HIP, so that tests can ask it which kernels a call takes.
//
// Times below are in us, 16-byte rows and 24-bit ids unless a width is named, as a / b: the method in
// question against the one the call takes otherwise (merge below kSortRadixMinRecords, else radix).
#pragma once

#include <stdint.h>

namespace ccj {

// Sort methods (the values of CC_SORT_AUTO, CC_SORT_MERGE, CC_SORT_RADIX), the call size from which
// the automatic choice prefers radix to merge, and the three methods of part_sort_kernels.hip,
// which only the automatic choice takes.
constexpr int32_t kSortAuto = 0;
constexpr int32_t kSortMerge = 1;
constexpr int32_t kSortRadix = 2;
constexpr int64_t kSortRadixMinRecords = (int64_t)1 << 20;
constexpr int32_t kSortRank = 3;       // ranks by comparison, one launch
constexpr int32_t kSortPart = 4;       // partition, one launch
constexpr int32_t kSortSplit = 5;      // partition of long lists, split by part beforehand: two

// Ranks by comparison: calls with few enough compares, total * ceil(longest / 512), in viewers of
// kRankMinMean records or more on average. They take 8.5 to 9 us up to 5,000 records in one viewer
// (partition: 11 for viewers of one part, 20 for longer ones), 12 us at 100,000 units of work and
// 28 at 200,000 (4 x 5,000, where the partition takes 20); viewers of one part 9 us at 19,200 units
// and 12.6 at 128,000 (64 x 1,000, partition 11.4).
constexpr int64_t kRankWorkShort = 40000;         // viewers of one part
constexpr int64_t kRankWorkLong = 130000;
constexpr int64_t kRankTotal = 10240;             // 1 x 10,000: 18.5 us, partition 23
constexpr int64_t kRankMinMean = 128;

// Records per part in calls of up to kPartSmallTotal records (the chip is not full, so short parts
// end sooner: 1 x 20,000 27 us against 30 with 2,048) and in larger ones (fewer reads of the key
// lists: 30 x 20,000 44 us against 57 with 1,024, 45 with 2,048).
constexpr int32_t kPartSmall = 1024;
constexpr int32_t kPartLarge = 1280;
constexpr int64_t kPartSmallTotal = (int64_t)1 << 18;
constexpr int64_t kPartMaxRecords = (int64_t)1 << 20;    // per viewer, exclusive (32-bit sample)
constexpr int32_t kPartMaxViewers = 1 << 21;     // one workgroup each: the grid stays launchable

// Partition: calls whose key reads, about total * longest / part, stay below those of a few passes
// over the call: 64 x 5,000 records of 64 bytes 29 / 53, 230 x 5,000 58 / 85, 300 x 8,000 100 / 131,
// 1,000 x 5,000 202 / 205. Past the line 2,000 x 5,000 392 / 385 and 2,700 x 5,000 549 / 506 (10 us
// more of a gap where the caller names the key span), 900 x 8,000 of 64 bytes 371 / 357, 2 x 180,000
// 111 / 99, 1 x 262,000 112 / 91. Viewers of one part each read their keys once, whatever their
// number: 60,000 x 1,000 1,374 / 3,354.
constexpr int64_t kPartMaxWork = 5 * ((int64_t)1 << 32);     // total * longest
constexpr int64_t kPartMaxWorkWhole = (int64_t)1 << 36;      // ... of viewers of one part

// In calls that radix would take instead, viewers of fewer records than this on average: a workgroup
// of the partition takes 14.6 ns per viewer, one of radix (several viewers each) 10 to 13. 1,200,000
// x 8 17,460 / 12,306, 600,000 x 16 8,757 / 7,915, 600,000 x 24 8,831 / 10,540.
constexpr int64_t kPartMinMean = 20;

// Two launches, the first of which puts long viewers' records in order of their parts: taken where
// viewers have at most kSplitMax records (256 parts, of whose number two go to the ends) and by the
// caller's bound (their mean, without one) may have more than kSplitMin. 1 x 160,000 27 / 84,
// 130 x 8,500 52 / 107, 3,000 x 8,500 958 / 1,116, 40 x 130,000 175 / 225, 100 x 160,000 547 / 569;
// against the partition in one launch: 64 x 5,000 33 / 30, 30 x 10,000 31 / 31, 100 x 10,000 60 / 66.
constexpr int32_t kPartSplit = 640;              // records per part
constexpr int64_t kSplitMin = 8192;
constexpr int64_t kSplitMax = (256 - 2) * (int64_t)kPartSplit;

// A call without a bound on its viewers (max_keys = 0) may hold one viewer of nearly all its records.
// One launch would then read that list once per part: 1,000 viewers of 20 records and one of 130,000
// 90 / 90, of 300,000 158 / 116, of 500,000 257 / 126. Past the partition's limit with `total` for the
// longest list, and up to kSplitTotal records, such a call takes the two launches, which read each list
// twice however long; a viewer of more than kSplitMax records is cut into 256 longer parts. One of
// 165,000 among the 1,000 39 / 97, of 300,000 64 / 116, of 500,000 80 / 126 (62-bit keys, 128-byte rows
// 126 / 172), alone 65 / 108; 64 x 5,000 30 / 56 (25 with a bound, in one launch), 64 viewers of 100 to
// 30,000 32 / 92, 300 x 1,700 18 / 56. The same for a bound above kSplitMax. Lists of at most kTinyMean
// records on average keep the one launch, where the merge's time per viewer covers a long one: 20,000 x
// 10 286 / 888, 8,000 viewers of 4 with one of 500,000 466 / 466.
constexpr int64_t kSplitTotal = (int64_t)1 << 19;
constexpr int64_t kTinyMean = 64;

// The method of a call of total records (1 to 2^32 - 1) in n_viewers viewers (at least 1), none
// longer than max_keys if that is positive.
inline int32_t sort_choice(int64_t total, int64_t n_viewers, int64_t max_keys) {
    const int64_t limit = max_keys > 0 && max_keys < total ? max_keys : total;
    const int64_t compares = total * ((limit + 511) / 512);
    if (total >= n_viewers * kRankMinMean &&
        (limit <= kPartSmall ? compares <= kRankWorkShort
                             : compares <= kRankWorkLong || total <= kRankTotal))
        return kSortRank;
    if (n_viewers <= kPartMaxViewers) {
        if ((max_keys > 0 ? limit : total / n_viewers) > kSplitMin && limit <= kSplitMax)
            return kSortSplit;
        const bool short_lists = total >= kSortRadixMinRecords && total < n_viewers * kPartMinMean;
        if (!short_lists && limit <= (limit <= kPartLarge ? kPartMaxWorkWhole : kPartMaxWork) / total)
            return kSortPart;
        if (total <= kSplitTotal)
            return total <= n_viewers * kTinyMean ? kSortPart : kSortSplit;
    }
    return total >= kSortRadixMinRecords ? kSortRadix : kSortMerge;
}

}  // namespace ccj
