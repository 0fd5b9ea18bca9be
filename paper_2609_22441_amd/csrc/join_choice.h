// Rules of a join launch on its sizes. Host code without HIP, so that tests can ask them. Times are in
// us, warm launches in a row, 128-byte doc and 32-byte edge rows unless others are named.
#pragma once

#include <stdint.h>

namespace ccj {

// Fences that a segment of any size may have (the rest of its budget grows with its candidates).
// kFencesShort, one round of staging loads, leaves windows of few keys: 17,187 candidates in shares
// of 67, two lookups into 68,767 keys: 17.1 with them, 22.2 with kFencesLeast; 100 viewers of 90
// candidates and 20,000 keys 9.4 and 10.0. But every fence of a long list is a line of its own, read for
// few candidates: where the lists average more than four default tables (long_lists) and the viewers'
// fences are more than kFenceBytes of lines (3 of the 4 MiB of L2 of every XCD), the smaller table is
// faster: 100 viewers of 60,000 keys with 10 candidates 10.0 against 15.7, with 90 10.6 against 16.2;
// 64 with 550 13.4 against 15.8. (32 viewers, 15 MiB of lines: 9.9 and 10.1; two lookups 12.0 and 11.6.)
constexpr int32_t kFencesShort = 4096;
constexpr int32_t kFencesLeast = 512;
constexpr int64_t kFenceBytes = (int64_t)24 << 20;

inline int32_t least_fences(int64_t total_keys, int64_t viewers, bool long_lists) {
    const int64_t lines = total_keys / viewers / 16 + 1;      // of 16 keys, in a list
    const int64_t bytes = viewers * 128 * (lines < kFencesShort ? lines : kFencesShort);
    return long_lists && bytes > kFenceBytes ? kFencesLeast : kFencesShort;
}

// Number of ranges near n, at most `most`, that is a multiple of the viewers; 0 where there is none. A
// range that holds the end of one viewer and the start of the next goes through two segments one after
// the other, each with its own fences and first sub-tile. With equal viewers a multiple of them avoids
// it: 16 viewers of 160 candidates and 10,000 keys 12.0 -> 8.3, 3 of 250 11.8 -> 8.3, 16 of 1,000 and
// 20,000 keys 13.5 -> 9.7, 100 of 10 and 60,000 keys 65.4 -> 10.0. More ranges than asked for cost little
// (a few candidates less for each); fewer are taken down to 15 of 16 only, for ragged viewers gain nothing
// from them (150 of 1,000 on average: 17.6 on 512 ranges, 19.0 on 450). Above that line ragged ones stay
// within 2% mostly, and pay 6 at most: 20 of up to 5,000 12.5 -> 13.2 on 240 ranges, 12.6 -> 12.6 with other
// sizes; equal ones of 3,125 12.4 -> 10.4. (The kernel could look whether the viewers are equal, but that
// costs every such launch 0.4.)
inline int64_t ranges_of_viewers(int64_t n, int64_t viewers, int64_t most) {
    const int64_t up = (n + viewers - 1) / viewers * viewers, down = n / viewers * viewers;
    if (up <= most)
        return up;
    return 16 * down >= 15 * n ? down : 0;
}

// Whether output rows of run-time widths are copied without the pipeline and its streaming stores: rows of
// two or three chunks with gaps between them, which end inside a line that the next row begins in, of
// outputs that L2 can put together. Rows of 16 + 16 bytes at 80, 10,000 candidates 5.0 us, 5.7 with the
// pipeline; 50,000 6.5 and 7.1. Longer rows or larger outputs keep it (48 + 16 bytes at 80, 2,000
// candidates 5.6, 5.9 without; 16 + 16 at 80, 15 MiB 15 and 17).
constexpr int64_t kPlainWidth = 48;
constexpr int64_t kPlainBytes = (int64_t)8 << 20;

inline bool plain_copy(int64_t rows, int64_t stride, int64_t width) {
    return stride != width && width <= kPlainWidth && rows * stride <= kPlainBytes;
}

}  // namespace ccj
