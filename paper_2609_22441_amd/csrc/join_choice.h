// Rules of a join launch on its sizes. Host code without HIP, so that tests can ask them. Times are in
// us, warm launches in a row, 128-byte doc and 32-byte edge rows unless others are named.
#pragma once

#include <stdint.h>

namespace ccj {

// Fences that a segment of any size may have (the rest of its budget grows with its candidates).
// kFencesShort, one round of staging loads, leaves windows of few keys: 17,187 candidates in shares
// of 67, two lookups into 68,767 keys: 17.1 with them, 22.2 with kFencesLeast; 100 viewers of 90
// candidates and 20,000 keys 9.4 and 10.0. But every fence of a long list is a line of its own, which the
// viewer's segments read for few candidates: where lists are longer than the largest table's windows
// of eight keys reach (long_lists) and the viewers' fences are more lines than kFenceBytes, 4 MiB per
// XCD below what the L2s hold, the smaller table is faster: 100 viewers of 60,000 keys with 10
// candidates 10.0 against 15.7, with 90 10.6 against 16.2; 64 with 550 13.4 against 15.8. (32 viewers,
// 15 MiB of lines: 9.9 and 10.1; two lookups 12.0 and 11.6.)
constexpr int32_t kFencesShort = 4096;
constexpr int32_t kFencesLeast = 512;
constexpr int64_t kFenceBytes = (int64_t)24 << 20;

inline int32_t least_fences(int64_t total_keys, int64_t viewers, bool long_lists) {
    const int64_t lines = total_keys / viewers / 16 + 1;      // of 16 keys, in a list
    const int64_t bytes = viewers * 128 * (lines < kFencesShort ? lines : kFencesShort);
    return long_lists && bytes > kFenceBytes ? kFencesLeast : kFencesShort;
}

}  // namespace ccj
