// Whether an ingestion batch updates the map in a launch of its own, after the one that writes its
// rows: a rule on the batch's sizes. Host code without HIP, so that tests can ask it.
#pragma once

#include <stdint.h>

namespace ccj {

// The update's random writes between the row writes save a launch (300,000 records of 128 bytes: 62 us
// in one, 72 in two and a rollback), but cost more than that once the rows are many bytes. Whole batches
// of stored ids, us in one launch / two: 1,000,000 records of 256 bytes 213 / 225, of 512 321 / 311, of
// 1,024 527 / 491; 2,000,000 of 128 301 / 319, of 256 423 / 407, of 512 647 / 581; 300,000 of 2,048
// 281 / 280. Short rows: 10M of 128 1,065 / 867.
constexpr int64_t kCommitApartFrom = 1 << 21;                  // records
constexpr int64_t kCommitApartBytes = 3 * ((int64_t)1 << 27);  // of rows

inline bool commit_apart(int64_t n_records, int64_t row_bytes) {
    return n_records >= kCommitApartFrom || n_records * row_bytes >= kCommitApartBytes;
}

}  // namespace ccj
