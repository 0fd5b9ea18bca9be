// Alg. 1 Step 1 in one or two launches (Connected Content Retriever §3.1): the affinity-record sort
// for calls whose lists are not very long. A launch that depends on the one before costs 3 to 5 us
// here however small it is, and the merge method takes 4 to 10 of them; both methods below need one,
// and the partition of long lists two (split_kernel). 64-byte rows, 24-bit ids: one viewer of 5,000
// records 46.9 -> 8.3 us (ranks by comparison), 64 x 5,000 56 -> 30 us (partition: the dependent
// steps of a part set the time).
//
// The partition method needs no plan, no histogram over the call and no pass over global memory
// that a later launch waits for. A viewer of n records is cut into G parts of about `part` records
// in key order, one workgroup each, and every workgroup finds its part by itself:
//   1. sample: the same pseudo-random positions of the viewer's input in every workgroup (one
//      per stratum of n / S records), put in (key, position) order; its records of rank g S / G
//      and (g + 1) S / G bound part g. No two records are equal in that order, so repeated keys
//      split like any others.
//   2. select: the workgroup reads every key of the viewer (8 n bytes, from L2 after the first
//      part's read), counts the records below its part, which is where its output starts, and
//      keeps the records of its part in LDS, in input order.
//   3. sort: a stable least-significant-digit radix sort of the part in LDS (digits of at most 8
//      bits over the span of the part's own keys; equal keys keep their input order).
//   4. emit: keys and feature rows to the part's contiguous output.
// What bounds a part is the length of its dependent chain (about 3 us of sample, 1 us per 4,096
// keys selected, 2 us per digit, 3 to 5 us of rows), so a part is as short as the redundant key
// reads allow. 512 threads and kCap = 4096 leave two workgroups per CU: 1,024 threads were 30%
// slower from 64 x 5,000 records on (one workgroup per CU), and no faster below.
//
// A part that the sample judged wrong by more than kCap / part (or that malformed offsets made
// so) does not fit in LDS: its records are then sorted by the same digit passes in chunks,
// through the two element arrays of the workspace, by the one workgroup. Slower, never wrong.
// (Parts of split calls are sorted in pieces first, see overlong_part.) The sample has kPerPart
// records per part: a part of more than kCap / kPartLarge = 3.2 times its share is a 2e-6 event in
// key orders that know nothing of the sample.
#include "join_internal.h"
#include "sort_choice.h"
#include "sort_device.h"

namespace ccj {
namespace {

constexpr int kPartThreads = 512;
constexpr int kPartWaves = kPartThreads / 64;
constexpr int kEpt = 8;                        // records per thread of a part in LDS
constexpr int kCap = kEpt * kPartThreads;      // records a part sorts in LDS (4096)
constexpr int kBits = 8;                       // widest digit
constexpr int kRadix = 1 << kBits;
constexpr int kSampleMin = 64;
constexpr int kPerPart = 10;                   // sample records per part
constexpr int kSampleCount = 256;              // samples up to this size are ranked by counting
static_assert(kSplitTotal < kPartMaxRecords && kPartLarge < kPartMaxRecords &&
                  kPartMaxWork <= (kPartMaxRecords - 1) * (kPartMaxRecords - 1),
              "every viewer of a call that the automatic choice sends here can be sorted");

// Tables of a workgroup whose part may hold E records per thread.
template <int E>
struct PartTables {
    static constexpr int kEpt = E;
    static constexpr int kCap = E * kPartThreads;
    uint64_t key[kCap];              // key - smallest key (select: the key itself)
    uint32_t pos[kCap];              // position in the viewer
    uint16_t cnt[kPartWaves][kRadix];    // per wavefront: running count, then the first sorted index
                                     // of the wavefront's records of that digit value
    uint32_t start[kRadix];          // first sorted index of each digit value
    uint32_t adj[kRadix];            // big_part: a chunk's sorted index to the part's
    uint32_t run[2][kPartWaves];         // select: records of the part per wavefront (two turns)
    uint32_t below[kPartWaves];          // ... and records below it
    int64_t lo[kPartWaves], hi[kPartWaves];  // key range per wavefront
    int64_t bound_key[2];
    uint32_t bound_pos[2];
};

// Element of the chunked passes through the workspace.
struct Elem {
    uint64_t key;
    uint64_t pos;
};

__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// threadIdx.x, opaque to the compiler: what is derived from it stays local to a step, where it
// would otherwise be kept in registers from one step of the kernel to the next.
__device__ __forceinline__ int thread_index() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// The wavefront's index in the workgroup, as a scalar.
__device__ __forceinline__ int wave_index() {
    return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
}

// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ uint32_t uniform(uint32_t x) {
    return __builtin_amdgcn_readfirstlane((int)x);
}
__device__ __forceinline__ int64_t uniform(int64_t x) {
    return (int64_t)(((uint64_t)uniform((uint32_t)((uint64_t)x >> 32)) << 32) | uniform((uint32_t)x));
}

__device__ __forceinline__ int lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// x of the lane that DPP control CTRL names (rows masked out and lanes without a source get x).
template <int CTRL, int ROWS>
__device__ __forceinline__ int64_t dpp64(int64_t x) {
    const int lo = (int)(uint32_t)x, hi = (int)(uint32_t)((uint64_t)x >> 32);
    const int a = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xF, false);
    const int b = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xF, false);
    return (int64_t)(((uint64_t)(uint32_t)b << 32) | (uint32_t)a);
}

// DPP steps of a wavefront reduction or scan: shifts by 1, 2, 4 and 8 lanes within rows of 16,
// then lane 15 of a row to the next row, then lane 31 to the upper half. Lane 63 ends with all.
constexpr int kShr1 = 0x111, kShr2 = 0x112, kShr4 = 0x114, kShr8 = 0x118;
constexpr int kBcast15 = 0x142, kBcast31 = 0x143;

template <int CTRL, int ROWS>
__device__ __forceinline__ void range_step(int64_t &lo, int64_t &hi) {
    lo = min(lo, dpp64<CTRL, ROWS>(lo));
    hi = max(hi, dpp64<CTRL, ROWS>(hi));
}

// Smallest lo and largest hi over the workgroup. Has one barrier.
template <typename SH>
__device__ __forceinline__ void key_range(SH &sh, int64_t &lo, int64_t &hi) {
    const int lane = thread_index() & 63, w = wave_index();
    range_step<kShr1, 0xF>(lo, hi);
    range_step<kShr2, 0xF>(lo, hi);
    range_step<kShr4, 0xF>(lo, hi);
    range_step<kShr8, 0xF>(lo, hi);
    range_step<kBcast15, 0xA>(lo, hi);
    range_step<kBcast31, 0xC>(lo, hi);
    if (lane == 63) {
        sh.lo[w] = lo;
        sh.hi[w] = hi;
    }
    lds_sync();
    lo = sh.lo[0];
    hi = sh.hi[0];
#pragma unroll
    for (int k = 1; k < kPartWaves; ++k) {
        lo = min(lo, sh.lo[k]);
        hi = max(hi, sh.hi[k]);
    }
}

template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t sum_step(uint32_t x) {
    return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
}

// Inclusive prefix sum over the wavefront.
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
    x = sum_step<kShr1, 0xF>(x);
    x = sum_step<kShr2, 0xF>(x);
    x = sum_step<kShr4, 0xF>(x);
    x = sum_step<kShr8, 0xF>(x);
    x = sum_step<kBcast15, 0xA>(x);
    return sum_step<kBcast31, 0xC>(x);
}

// The digits of a span of kbits bits: passes of D bits.
struct Digits {
    int passes, D;
    uint32_t mask;
};

__device__ __forceinline__ Digits digits_of(uint64_t span) {
    const int kbits = span ? 64 - __clzll(span) : 0;
    const int passes = (kbits + kBits - 1) / kBits;
    const int D = passes ? (kbits + passes - 1) / passes : 0;
    return Digits{passes, D, (1u << D) - 1};
}

// Ranks R rounds of 64 records per wavefront by digit: rd[m] = (records of the same digit before
// this one in the wavefront) << 8 | digit, and the wavefront's digit counts in sh.cnt[w]. The
// lanes that share a digit are found with one ballot per digit bit.
template <typename SH, typename K, int E>
__device__ __forceinline__ void rank_rounds(SH &sh, const K (&key)[E], int R,
                                            int first, int n, int shift, uint32_t mask,
                                            uint32_t (&rd)[E]) {
    const int lane = thread_index() & 63, w = wave_index();
    __builtin_memset(&sh.cnt[w][lane * (kRadix / 64)], 0, kRadix / 64 * sizeof(uint16_t));
#pragma unroll
    for (int m = 0; m < E; ++m) {
        if (m < R) {                                     // uniform
            // The lanes of a round read what lanes of earlier rounds wrote: the wavefront's LDS
            // accesses complete in order, the fence keeps the compiler to that order.
            wave_lds_order();
            const bool valid = first + m * 64 + lane < n;
            const uint32_t d = (uint32_t)(key[m] >> shift) & mask;
            const uint64_t all = __ballot(valid);
            uint32_t plo = (uint32_t)all, phi = (uint32_t)(all >> 32);
#pragma unroll
            for (int b = 0; b < kBits; ++b) {
                const uint32_t s = (uint32_t)((int32_t)(d << (31 - b)) >> 31);   // bit b, 0 or ~0
                const uint64_t bal = __ballot(s != 0);
                plo &= ~((uint32_t)bal ^ s);
                phi &= ~((uint32_t)(bal >> 32) ^ s);
            }
            const uint64_t peers = (uint64_t)plo | ((uint64_t)phi << 32);
            const int before = lanes_below(peers);
            const uint32_t c = sh.cnt[w][d];
            wave_lds_order();
            if (valid && before == 0)
                sh.cnt[w][d] = (uint16_t)(c + (uint32_t)__popcll(peers));
            // Pinned, so that no mask or partial count stays alive until the scatter.
            uint32_t x = ((c + (uint32_t)before) << 8) | d;
            asm volatile("" : "+v"(x));
            rd[m] = x;
        }
    }
}

// Between two barriers after rank_rounds: the wavefronts' counts become the first sorted index of
// each wavefront's records of each digit value, and sh.start that of each digit value. Wavefront
// 0 does it alone, four digit values per lane as 16-bit fields of one word (no field exceeds
// kCap): one barrier and one round of LDS reads less than a scan over all threads.
template <typename SH>
__device__ __forceinline__ void digit_offsets(SH &sh) {
    if (wave_index() != 0)
        return;
    const int lane = thread_index() & 63;
    uint64_t c[kPartWaves];
#pragma unroll
    for (int k = 0; k < kPartWaves; ++k)
        __builtin_memcpy(&c[k], &sh.cnt[k][lane * 4], 8);
    uint64_t tot = 0;
#pragma unroll
    for (int k = 0; k < kPartWaves; ++k)
        tot += c[k];
    const uint32_t t0 = (uint32_t)tot & 0xFFFFu, t1 = t0 + ((uint32_t)tot >> 16);
    const uint32_t t2 = t1 + ((uint32_t)(tot >> 32) & 0xFFFFu), t3 = t2 + (uint32_t)(tot >> 48);
    const uint32_t s0 = wave_scan(t3) - t3, s1 = s0 + t0, s2 = s0 + t1, s3 = s0 + t2;
    uint64_t at = (uint64_t)(s0 | (s1 << 16)) | ((uint64_t)(s2 | (s3 << 16)) << 32);
    sh.start[lane * 4] = s0;
    sh.start[lane * 4 + 1] = s1;
    sh.start[lane * 4 + 2] = s2;
    sh.start[lane * 4 + 3] = s3;
#pragma unroll
    for (int k = 0; k < kPartWaves; ++k) {
        __builtin_memcpy(&sh.cnt[k][lane * 4], &at, 8);
        at += c[k];
    }
}
static_assert(kRadix == 4 * 64, "four digit values per lane");

// Records first + m * 64 + lane of a tile of n, m < R: the order (wavefront, round, lane).
struct Rounds {
    int n, R, first;
    __device__ explicit Rounds(int n_) : n(n_), R((n_ + kPartThreads - 1) / kPartThreads) {
        first = wave_index() * R * 64;
    }
    __device__ int at(int m) const { return first + m * 64 + (thread_index() & 63); }
};

// Sorts n <= kCap records stably by key: key and pos hold them in the order of Rounds (records
// past n repeat the last one). Leaves the sorted offsets from the smallest key (returned) and
// positions in sh.key / sh.pos, with a barrier behind them. Called with a barrier behind the last
// use of sh.
template <typename SH>
__device__ __forceinline__ int64_t sort_lds(SH &sh, const Rounds &rs,
                                            uint64_t (&key)[SH::kEpt], uint32_t (&pos)[SH::kEpt]) {
    constexpr int kEpt = SH::kEpt;
    int64_t lo = INT64_MAX, hi = INT64_MIN;
#pragma unroll
    for (int m = 0; m < kEpt; ++m) {
        if (m < rs.R) {                                  // uniform
            lo = min(lo, (int64_t)key[m]);
            hi = max(hi, (int64_t)key[m]);
        }
    }
    key_range(sh, lo, hi);
    const Digits dg = digits_of((uint64_t)hi - (uint64_t)lo);
#pragma unroll
    for (int m = 0; m < kEpt; ++m) {
        if (m < rs.R)
            key[m] -= (uint64_t)lo;
    }
    const int w = wave_index();
    // Equal keys (no digit to sort by) take one pass of one value, which leaves them in order.
    for (int p = 0;; ++p) {
        uint32_t rd[kEpt];
        rank_rounds(sh, key, rs.R, rs.first, rs.n, p * dg.D, dg.mask, rd);
        lds_sync();
        digit_offsets(sh);
        lds_sync();
#pragma unroll
        for (int m = 0; m < kEpt; ++m) {
            if (m < rs.R && rs.at(m) < rs.n) {
                const uint32_t to = sh.cnt[w][rd[m] & 0xFFu] + (rd[m] >> 8);
                sh.key[to] = key[m];
                sh.pos[to] = pos[m];
            }
        }
        lds_sync();
        if (p + 1 >= dg.passes)
            return lo;
#pragma unroll
        for (int m = 0; m < kEpt; ++m) {
            if (m < rs.R) {
                const int i = min(rs.at(m), rs.n - 1);
                key[m] = sh.key[i];
                pos[m] = sh.pos[i];
            }
        }
    }
}

// Part g of G of the viewer with records [kb, kb + n).
struct Part {
    int64_t kb;
    uint32_t n;
    uint32_t g, G;
};

// Split calls: records per thread of a part in LDS (31 KB and at most 64 registers: four workgroups
// per CU, so that some copy rows while others sort; 32 x 100,000 records of 128 bytes, parts of 640:
// 184 us, with 6 per thread, three workgroups and parts of 1,024: 198) and of a chunk.
constexpr int kSplitEpt = 4;
constexpr uint32_t kSplitCap = kSplitEpt * kPartThreads;
constexpr int kChunkEpt = 6;
constexpr uint32_t kChunk = kChunkEpt * kPartThreads;
static_assert(kSplitCap <= kChunk && kChunk <= kCap, "row(), 16-bit counts");

// The records of the viewers that split_kernel goes through, chunk by chunk: each chunk's records
// by part, in input order within a part, and per chunk the first one of every part.
struct Split {
    int64_t *key;               // [total]
    uint32_t *pos;              // [total] position in the viewer
    uint16_t *start;            // rows of kRadix entries, see row()
    uint32_t firsts;            // rows before those of the viewers' first chunks
    // Row of chunk g of the viewer that starts at kb. Chunks behind a viewer's first one are
    // numbered by the multiple of kChunk that they start nearest to, first chunks by the first
    // multiple of kSplitCap inside the viewer, which has more records than that.
    __device__ int64_t row(int64_t kb, uint32_t g) const {
        return g == 0 ? (int64_t)firsts + (uint32_t)kb / kSplitCap + 1
                      : (int64_t)((uint32_t)kb / kChunk) + g;
    }
};

__device__ __forceinline__ uint32_t parts_of(int64_t kb, int64_t ke, uint32_t part) {
    // One more than the multiples of `part` strictly inside (offsets are below 2^32).
    return ke - kb <= part ? 1 : 1 + (uint32_t)(ke - 1) / part - (uint32_t)kb / part;
}

__device__ __forceinline__ uint32_t part_begin(uint32_t n, uint32_t g, uint32_t G) {
    return (uint32_t)((uint64_t)n * g / G);
}

// A viewer's sample: S records, record i anywhere in the i-th stratum (Knuth's multiplicative
// hash of i), so that no regular pattern of the input falls in step with it.
struct Sample {
    uint32_t S, step;                                    // stratum width, 12 fractional bits
    __device__ explicit Sample(const Part &pt, uint32_t per = kPerPart, uint32_t most = kCap) {
        S = pt.G > most / per ? most : max((uint32_t)kSampleMin, pt.G * per);
        S = min(S, pt.n);                                // n > part: at least a record per part
        step = (pt.n << 12) / S;
    }
    __device__ uint32_t pos(uint32_t i) const {
        const uint32_t a = (i * step) >> 12, b = ((i + 1) * step) >> 12;
        return a + __umulhi(i * 2654435761u, b - a);
    }
};
static_assert(kPartMaxRecords <= (int64_t)1 << 20 && kCap <= 1 << 12, "i * step fits 32 bits");

// Bound `side` of part g (0: at or above it, 1: below it) is the sample record of this rank; the
// first and the last part have none on their outer side.
__device__ __forceinline__ uint32_t bound_rank(const Part &pt, uint32_t side, uint32_t S) {
    return min((pt.g + side) * S / pt.G, S - 1);
}

template <typename SH>
__device__ __forceinline__ void open_bounds(SH &sh, const Part &pt) {
    if (thread_index() == 0) {
        // Below, and above, every record (positions are below 2^32 - 1).
        if (pt.g == 0) {
            sh.bound_key[0] = INT64_MIN;
            sh.bound_pos[0] = 0;
        }
        if (pt.g + 1 == pt.G) {
            sh.bound_key[1] = INT64_MAX;
            sh.bound_pos[1] = ~0u;
        }
    }
}

// Bounds from a sample of at most kSampleCount records, whose ranks are counted: thread (h, i)
// compares record i with share h of the sample. Positions grow with the sample index, so equal
// keys order by index. Ends with a barrier.
template <typename SH>
__device__ __forceinline__ void count_bounds(SH &sh, const int64_t *__restrict__ keys,
                                             const Part &pt, const Sample &sm) {
    constexpr int kShares = kPartThreads / kSampleCount;
    const int tid = thread_index(), i = tid & (kSampleCount - 1), h = tid / kSampleCount;
    const int S = (int)sm.S;
    const uint32_t p = sm.pos(min(i, S - 1));
    const int64_t x = keys[pt.kb + p];
    if (h == 0)
        sh.key[i] = (uint64_t)x;                         // records past S repeat the last one
    lds_sync();
    const int share = (S + kShares - 1) / kShares, j0 = h * share, j1 = min(S, j0 + share);
    uint32_t rank = 0;
    if ((wave_index() & (kSampleCount / 64 - 1)) * 64 < S) { // uniform per wavefront
#pragma unroll 8
        for (int j = j0; j < j1; ++j) {
            const int64_t y = (int64_t)sh.key[j];
            rank += (y < x || (y == x && j < i)) ? 1 : 0;
        }
    }
    sh.pos[tid] = rank;
    open_bounds(sh, pt);
    lds_sync();
    if (h == 0 && i < S) {
#pragma unroll
        for (int q = 1; q < kShares; ++q)
            rank += sh.pos[q * kSampleCount + i];
        if (pt.g > 0 && rank == bound_rank(pt, 0, S)) {
            sh.bound_key[0] = x;
            sh.bound_pos[0] = p;
        }
        if (pt.g + 1 < pt.G && rank == bound_rank(pt, 1, S)) {
            sh.bound_key[1] = x;
            sh.bound_pos[1] = p;
        }
    }
    lds_sync();
}

// Bounds from the sorted sample. Ends with a barrier.
template <typename SH>
__device__ __forceinline__ void pick_bounds(SH &sh, const Part &pt, uint32_t S,
                                            int64_t kmin) {
    const int tid = thread_index();
    if (tid < 2 && (tid == 0 ? pt.g > 0 : pt.g + 1 < pt.G)) {
        const uint32_t r = bound_rank(pt, tid, S);
        sh.bound_key[tid] = (int64_t)(sh.key[r] + (uint64_t)kmin);
        sh.bound_pos[tid] = sh.pos[r];
    }
    open_bounds(sh, pt);
    lds_sync();
}

// (key, position) bounds: records at or above (k0, p0) and below (k1, p1).
struct Bounds {
    int64_t k0, k1;
    uint32_t p0, p1;
};

constexpr int kScan = 8;                       // rounds of 64 keys read together
constexpr uint32_t kTurn = kScan * kPartThreads;   // keys of the viewer per turn of the workgroup

// The wavefront's keys of the turn that starts at t0: records first + u * 64 + lane, from
// clamped positions; returns first.
__device__ __forceinline__ uint32_t read_keys(const int64_t *__restrict__ keys, const Part &pt,
                                              uint32_t t0, int64_t (&k)[kScan]) {
    const uint32_t first = t0 + wave_index() * (kScan * 64);
    const uint32_t i = first + (thread_index() & 63);
#pragma unroll
    for (int u = 0; u < kScan; ++u)
        k[u] = keys[pt.kb + min(i + u * 64, pt.n - 1)];
    return first;
}

// Goes through the viewer in turns of kTurn keys, input order being (turn, wavefront, round,
// lane), and calls put(place, key, position) for every record of the part, place its index among
// them in input order. The next turn's keys are read meanwhile; k holds the first turn's. Returns
// the number of records of the part, below the number of records below it. Ends with a barrier.
template <typename SH, typename F>
__device__ __forceinline__ uint32_t scan_viewer(SH &sh, const int64_t *__restrict__ keys,
                                                const Part &pt, const Bounds &bd,
                                                int64_t (&k)[kScan], uint32_t &below, F put) {
    const int lane = thread_index() & 63, w = wave_index();
    uint32_t m = 0, under = 0;
    for (uint32_t t0 = 0, turn = 0; t0 < pt.n; t0 += kTurn, turn ^= 1) {
        int64_t next[kScan];
        read_keys(keys, pt, t0 + kTurn, next);
        const uint32_t first = t0 + w * (kScan * 64), i = first + lane;
        uint64_t mask[kScan];
        uint32_t c = 0;
        // By key alone; a turn with keys equal to a bound (one record each, unless keys repeat)
        // or past the viewer's end settles them by position.
        uint64_t rest = __ballot(i + (kScan - 1) * 64 >= pt.n);
#pragma unroll
        for (int u = 0; u < kScan; ++u) {
            const uint64_t lt0 = __ballot(k[u] < bd.k0), lt1 = __ballot(k[u] < bd.k1);
            rest |= __ballot(k[u] == bd.k0) | __ballot(k[u] == bd.k1);
            under += __popcll(lt0);
            mask[u] = lt1 & ~lt0;
            c += __popcll(mask[u]);
        }
        if (rest) {                                      // uniform per wavefront
            c = 0;
#pragma unroll
            for (int u = 0; u < kScan; ++u) {
                const uint32_t p = i + u * 64;
                const uint64_t lt0 = __ballot(k[u] < bd.k0), lt1 = __ballot(k[u] < bd.k1);
                const uint64_t ok = __ballot(p < pt.n);
                const uint64_t lt = ok & (lt0 | (__ballot(k[u] == bd.k0) & __ballot(p < bd.p0)));
                const uint64_t in = lt1 | (__ballot(k[u] == bd.k1) & __ballot(p < bd.p1));
                under += __popcll(lt) - __popcll(lt0);
                mask[u] = ok & in & ~lt;
                c += __popcll(mask[u]);
            }
        }
        if (lane == 0)
            sh.run[turn][w] = c;
        lds_sync();
        uint32_t at = m;
#pragma unroll
        for (int q = 0; q < kPartWaves; ++q) {
            const uint32_t r = sh.run[turn][q];
            at += q < w ? r : 0;
            m += r;
        }
        if (c) {                                         // uniform per wavefront
#pragma unroll
            for (int u = 0; u < kScan; ++u) {
                if ((mask[u] >> lane) & 1)
                    put(at + lanes_below(mask[u]), k[u], i + u * 64);
                at += __popcll(mask[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < kScan; ++u)
            k[u] = next[u];
    }
    if (lane == 0)
        sh.below[w] = under;
    lds_sync();
    below = 0;
#pragma unroll
    for (int q = 0; q < kPartWaves; ++q)
        below += sh.below[q];
    return m;
}

// The part's records in global memory: sorted keys, then rows, to output positions from `to` on.
// Sorted records [0, m) come from sh.key / sh.pos.
template <typename SH>
__device__ __forceinline__ void emit(const SH &sh, const Part &pt, uint64_t kmin, int m,
                                     int64_t to, const SortOut &o) {
    for (int i = threadIdx.x; i < m; i += kPartThreads)
        __builtin_nontemporal_store((int64_t)(sh.key[i] + kmin), o.keys_out + to + i);
    copy_rows<4, kPartThreads>(m, o, [&](int rec, int64_t &from, int64_t &dst) {
        from = pt.kb + sh.pos[rec];
        dst = to + rec;
    });
}

constexpr int kChunks = 256;                   // of one viewer, at most
static_assert(kSplitTotal <= (int64_t)(kChunks - 2) * kChunk && kChunks <= kRadix, "four per lane");

// Chunks that a lane looks at: two, or four for viewers of more than 128.
__device__ __forceinline__ int chunks_per_lane(const Part &pt) {
    return parts_of(pt.kb, pt.kb + pt.n, kChunk) > kChunks / 2 ? kChunks / 64 : kChunks / 128;
}

// By one wavefront, PER chunks per lane. (PER is a constant, so that all entries are read together.)
template <int PER, typename SH>
__device__ __forceinline__ void look_at_chunks(SH &sh, const Part &pt, const Split &sp) {
    const int lane = thread_index() & 63;
    const uint32_t C = parts_of(pt.kb, pt.kb + pt.n, kChunk);
    uint32_t len[PER], at[PER], sum = 0, under = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t q = PER * lane + j, c = min(q, C - 1);
        const uint32_t c0 = part_begin(pt.n, c, C), cn = part_begin(pt.n, c + 1, C) - c0;
        const uint16_t *row = sp.start + sp.row(pt.kb, c) * kRadix;
        const uint32_t s = min((uint32_t)row[pt.g], cn);
        const uint32_t e = pt.g + 1 < kRadix ? row[pt.g + 1] : cn;
        at[j] = c0 + s;
        len[j] = q < C ? max(s, min(e, cn)) - s : 0;
        sum += len[j];
        under += q < C ? s : 0;
    }
    const uint32_t end = wave_scan(sum);
    uint32_t b = end - sum;
    under = wave_scan(under);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        sh.adj[PER * lane + j] = b;
        sh.start[PER * lane + j] = at[j] - b;            // modulo 2^32
        b += len[j];
    }
    if (lane == 63) {
        sh.run[0][0] = end;
        sh.below[0] = under;
    }
}

// Where split_kernel left the records of the part: sh.adj[c] those in the chunks before chunk c,
// sh.start[c] + i the place of the part's record i, if it is in chunk c. Returns their number, below
// the number of records below the part (what every chunk holds of earlier parts). Entries are
// clamped to their chunk, whatever malformed offsets made of them. Ends with a barrier.
template <typename SH>
__device__ __forceinline__ uint32_t find_records(SH &sh, const Part &pt, const Split &sp,
                                                 uint32_t &below) {
    if (wave_index() == 0) {
        if (chunks_per_lane(pt) == kChunks / 128)        // uniform
            look_at_chunks<kChunks / 128>(sh, pt, sp);
        else
            look_at_chunks<kChunks / 64>(sh, pt, sp);
    }
    lds_sync();
    below = sh.below[0];
    return sh.run[0][0];
}

template <typename SH>
__device__ __forceinline__ int64_t split_record(const SH &sh, const Part &pt,
                                                const Split &sp, uint32_t i, uint32_t &p) {
    // The last chunk that starts at or before record i.
    uint32_t c = 0;
    if (chunks_per_lane(pt) > kChunks / 128)             // uniform
        c = sh.adj[kChunks / 2] <= i ? kChunks / 2 : 0;
#pragma unroll
    for (uint32_t half = kChunks / 4; half > 0; half >>= 1)
        c += sh.adj[c + half] <= i ? half : 0;
    const uint32_t at = min(sh.start[c] + i, pt.n - 1);
    p = min(sp.pos[pt.kb + at], pt.n - 1);
    return sp.key[pt.kb + at];
}

// The records of a part of m > kCap, in input order, to a[0, m); lo and hi their key range. Called by the
// whole workgroup; a is the part's own slice of the workspace. Has a barrier behind the range.
template <typename SH>
__device__ __forceinline__ void gather_part(SH &sh, const int64_t *__restrict__ keys,
                                            const Part &pt, const Bounds &bd, uint32_t m, Elem *a,
                                            int64_t &lo, int64_t &hi) {
    const int tid = thread_index(), lane = tid & 63, w = wave_index();
    lo = INT64_MAX;
    hi = INT64_MIN;
    uint32_t found = 0;
    for (uint32_t p0 = 0; p0 < pt.n; p0 += kPartThreads) {
        const uint32_t p = p0 + tid;
        const int64_t k = keys[pt.kb + min(p, pt.n - 1)];
        const bool in = p < pt.n && (k > bd.k0 || (k == bd.k0 && p >= bd.p0)) &&
                        (k < bd.k1 || (k == bd.k1 && p < bd.p1));
        const uint64_t mask = __ballot(in);
        if (lane == 0)
            sh.run[0][w] = __popcll(mask);
        lds_sync();
        uint32_t at = found + lanes_below(mask);
#pragma unroll 1
        for (int q = 0; q < kPartWaves; ++q) {
            at += q < w ? sh.run[0][q] : 0;
            found += sh.run[0][q];
        }
        if (in) {
            lo = min(lo, k);
            hi = max(hi, k);
            if (at < m)
                a[at] = Elem{(uint64_t)k, p};
        }
        lds_sync();                                      // run is written again
    }
    key_range(sh, lo, hi);
}

// The same where split_kernel has put the part's records together.
template <typename SH>
__device__ __forceinline__ void gather_part(SH &sh, const Part &pt, const Split &sp, uint32_t m,
                                            Elem *a, int64_t &lo, int64_t &hi) {
    lo = INT64_MAX;
    hi = INT64_MIN;
    for (uint32_t i = thread_index(); i < m; i += kPartThreads) {
        uint32_t p;
        const int64_t k = split_record(sh, pt, sp, i, p);
        lo = min(lo, k);
        hi = max(hi, k);
        a[i] = Elem{(uint64_t)k, p};
    }
    key_range(sh, lo, hi);
}

// A part of m > kCap records, by digit passes through the workspace's element arrays: one stable pass
// per digit between a (where the records are, in input order) and b, each a count of the digits and a
// scatter of chunks of kPartThreads. Called by the whole workgroup; a and b are the part's own slices.
// Written for few registers: it shares the kernel with the path above.
template <typename SH>
__device__ __forceinline__ void big_part(SH &sh, const Part &pt, uint32_t m, int64_t lo, int64_t hi,
                                         Elem *a, Elem *b, int64_t to, const SortOut &o) {
    const int tid = thread_index(), w = wave_index();
    const Digits dg = digits_of((uint64_t)hi - (uint64_t)lo);
    __syncthreads();                                     // the stores, before their readers
#pragma unroll 1
    for (int p = 0; p < dg.passes; ++p) {
        const int shift = p * dg.D;
        if (tid < kRadix)
            sh.start[tid] = 0;
        lds_sync();
#pragma unroll 1
        for (uint32_t i = tid; i < m; i += kPartThreads)
            atomicAdd(&sh.start[(uint32_t)((a[i].key - (uint64_t)lo) >> shift) & dg.mask], 1u);
        lds_sync();
        uint32_t run = 0;                                // records before this digit's next one
        if (tid < kRadix) {
#pragma unroll 1
            for (int d = 0; d < tid; ++d)
                run += sh.start[d];
        }
        lds_sync();
#pragma unroll 1
        for (uint32_t c0 = 0; c0 < m; c0 += kPartThreads) {
            const int n = (int)min<uint32_t>(kPartThreads, m - c0);
            const Elem e = a[c0 + min(tid, n - 1)];
            const uint64_t key[1] = {e.key - (uint64_t)lo};
            uint32_t rd[1];
            rank_rounds(sh, key, 1, w * 64, n, shift, dg.mask, rd);
            lds_sync();
            digit_offsets(sh);
            lds_sync();
            if (tid < kRadix) {
                const uint32_t at = sh.start[tid];
                sh.adj[tid] = run - at;
                run += (tid + 1 < kRadix ? sh.start[tid + 1] : (uint32_t)n) - at;
            }
            lds_sync();
            const uint32_t d = rd[0] & 0xFFu, dst = sh.adj[d] + sh.cnt[w][d] + (rd[0] >> 8);
            if (tid < n && dst < m)
                b[dst] = e;
            lds_sync();
        }
        __syncthreads();                                 // the pass's stores, before its readers
        Elem *t = a;
        a = b;
        b = t;
    }
    for (uint32_t i = tid; i < m; i += kPartThreads)
        o.keys_out[to + i] = (int64_t)a[i].key;
    const int64_t chunks = (int64_t)m * o.row_chunks;
#pragma unroll 4
    for (int64_t c = tid; c < chunks; c += kPartThreads) {
        const uint32_t i = (uint32_t)((uint64_t)c / (uint32_t)o.row_chunks);
        // Viewers that overlap (malformed offsets) share slices of a and b and may leave places of
        // them unwritten: whatever those hold names a record of this viewer.
        const int64_t from = pt.kb + (int64_t)min<uint64_t>(a[i].pos, pt.n - 1);
        o.rows_out[to * o.row_chunks + c] =
            o.rows_in[from * o.row_chunks + (c - (int64_t)i * o.row_chunks)];
    }
}

template <typename SH>
__device__ __forceinline__ void sort_part(SH &sh, const int64_t *__restrict__ keys,
                                          const Part &pt, Elem *buf0, Elem *buf1,
                                          const SortOut &o) {
    constexpr int kEpt = SH::kEpt, kCap = SH::kCap;
    // Up to two rounds through one copy of the LDS sort: the sample, unless its ranks are counted
    // or the viewer is one part; then the part. The first turn's keys are on their way meanwhile.
    const Sample sm(pt);
    int64_t k0[kScan];
    const bool whole = pt.G == 1, counted = sm.S <= kSampleCount;
    if (!whole) {
        read_keys(keys, pt, 0, k0);
        if (counted)
            count_bounds(sh, keys, pt, sm);
    }
    int64_t kmin = 0;
    uint32_t m = 0, below = 0;
    for (int phase = whole || counted ? 1 : 0; phase < 2; ++phase) {
        uint64_t key[kEpt];
        uint32_t pos[kEpt];
        if (phase == 0 || whole) {
            m = phase == 0 ? sm.S : pt.n;
            const Rounds rs((int)m);
#pragma unroll
            for (int r = 0; r < kEpt; ++r) {
                if (r < rs.R) {                          // uniform
                    const uint32_t i = min((uint32_t)rs.at(r), m - 1);
                    pos[r] = phase == 0 ? sm.pos(i) : i;
                    key[r] = (uint64_t)keys[pt.kb + pos[r]];
                }
            }
        } else {
            if (!counted)
                pick_bounds(sh, pt, sm.S, kmin);
            const Bounds bd{sh.bound_key[0], sh.bound_key[1], sh.bound_pos[0], sh.bound_pos[1]};
            m = scan_viewer(sh, keys, pt, bd, k0, below, [&](uint32_t at, int64_t k, uint32_t p) {
                if (at < kCap) {
                    sh.key[at] = (uint64_t)k;
                    sh.pos[at] = p;
                }
            });
            if (m == 0)
                return;
            if (m > kCap)
                break;
            const Rounds rs((int)m);
#pragma unroll
            for (int r = 0; r < kEpt; ++r) {
                if (r < rs.R) {
                    const int i = min(rs.at(r), (int)m - 1);
                    key[r] = sh.key[i];
                    pos[r] = sh.pos[i];
                }
            }
        }
        kmin = sort_lds(sh, Rounds((int)m), key, pos);
    }
    const int64_t to = pt.kb + below;
    if (m <= kCap) {
        emit(sh, pt, (uint64_t)kmin, (int)m, to, o);
    } else {
        const Bounds bd{sh.bound_key[0], sh.bound_key[1], sh.bound_pos[0], sh.bound_pos[1]};
        int64_t lo, hi;
        gather_part(sh, keys, pt, bd, m, buf0 + to, lo, hi);
        big_part(sh, pt, m, lo, hi, buf0 + to, buf1 + to, to, o);
    }
}

// ---- overlong parts of split calls, a piece at a time -----------------------------------------
//
// A part of up to kPieces times what LDS holds is cut once more, by a histogram of its records over
// 256 equal shares of its key span: runs of shares that fit are picked from its records (in input order,
// at a[0, m)) and sorted in LDS one after the other. 1 x 100,000 records with one part of 2,300: 25 us
// without it, 41 in pieces, 71 by digit passes; rows of 128 bytes 33, 54 and 92. One of 300,000 among
// 1,000 short lists (parts of 1,170, some overlong), 62-bit keys, rows of 128 bytes: 96 against 189.
constexpr uint32_t kPieces = 4;

// (Bounded whatever an overlapping viewer, from malformed offsets, has left in its place.)
__device__ __forceinline__ uint32_t share_of(uint64_t key, int64_t lo, int shift) {
    const uint64_t s = (key - (uint64_t)lo) >> shift;
    return s < kRadix ? (uint32_t)s : kRadix - 1;
}

// sh.adj[b] becomes the number of records in shares 0 to b, `shift` the width of a share. False where a
// share alone does not fit. Called after gather_part; ends with a barrier, behind which a can be read.
template <typename SH>
__device__ __forceinline__ bool count_shares(SH &sh, const Elem *a, uint32_t m, int64_t lo, int64_t hi,
                                             int &shift) {
    const int tid = thread_index(), lane = tid & 63;
    const uint64_t span = (uint64_t)hi - (uint64_t)lo;
    shift = (int)uniform((uint32_t)max(0, (span ? 64 - __clzll(span) : 0) - kBits));
    if (tid < kRadix)
        sh.start[tid] = 0;
    lds_sync();
    for (uint32_t i = tid; i < m; i += kPartThreads)     // its own records of gather_part
        atomicAdd(&sh.start[share_of(a[i].key, lo, shift)], 1u);
    lds_sync();
    if (wave_index() == 0) {
        uint32_t c[4], sum = 0, most = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c[j] = sh.start[lane * 4 + j];
            sum += c[j];
            most = max(most, c[j]);
        }
        uint32_t at = wave_scan(sum) - sum;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            sh.adj[lane * 4 + j] = at += c[j];
        const uint64_t over = __ballot(most > (uint32_t)SH::kCap);
        if (lane == 0)
            sh.below[0] = over != 0;
    }
    __syncthreads();
    return sh.below[0] == 0;
}

// The records behind the first `done` of the part, as many whole shares as fit in LDS: to sh.key and
// sh.pos in input order. Returns their number. Called with a barrier behind the last use of sh.key;
// ends with one.
template <typename SH>
__device__ __forceinline__ uint32_t pick_shares(SH &sh, const Elem *a, uint32_t m, int64_t lo,
                                                int shift, uint32_t done) {
    const int tid = thread_index(), lane = tid & 63, w = wave_index();
    uint32_t b0 = 0, b1 = 0;                             // shares [b0, b1)
#pragma unroll
    for (uint32_t half = kRadix / 2; half > 0; half >>= 1) {
        b0 += sh.adj[b0 + half - 1] <= done ? half : 0;
        b1 += sh.adj[b1 + half - 1] <= done + SH::kCap ? half : 0;
    }
    b1 += sh.adj[b1] <= done + SH::kCap ? 1 : 0;         // the last share too
    const uint32_t count = sh.adj[b1 - 1] - done;
    uint32_t found = 0;
    for (uint32_t p0 = 0, turn = 0; p0 < m; p0 += kPartThreads, turn ^= 1) {
        const uint32_t p = p0 + tid;
        const Elem e = a[min(p, m - 1)];
        const uint32_t s = share_of(e.key, lo, shift);
        const bool in = p < m && s >= b0 && s < b1;
        const uint64_t mask = __ballot(in);
        if (lane == 0)
            sh.run[turn][w] = __popcll(mask);
        lds_sync();
        uint32_t at = found + lanes_below(mask);
#pragma unroll 1
        for (int q = 0; q < kPartWaves; ++q) {
            at += q < w ? sh.run[turn][q] : 0;
            found += sh.run[turn][q];
        }
        if (in && at < (uint32_t)SH::kCap) {
            sh.key[at] = e.key;
            sh.pos[at] = (uint32_t)e.pos;
        }
    }
    lds_sync();
    return count;
}

// A part of m > kCap records: in pieces, or by digit passes where these do not do.
template <typename SH>
__device__ __forceinline__ void overlong_part(SH &sh, const Part &pt, const Split &sp, uint32_t m,
                                              Elem *a, Elem *b, int64_t to, const SortOut &o) {
    constexpr int kEpt = SH::kEpt;
    int64_t lo, hi;
    int shift;
    gather_part(sh, pt, sp, m, a, lo, hi);
    if (m > kPieces * (uint32_t)SH::kCap || !count_shares(sh, a, m, lo, hi, shift)) {
        big_part(sh, pt, m, lo, hi, a, b, to, o);
        return;
    }
#pragma unroll 1
    for (uint32_t done = 0; done < m;) {                 // uniform
        const uint32_t count = uniform(pick_shares(sh, a, m, uniform(lo), shift, done));
        uint64_t key[kEpt];
        uint32_t pos[kEpt];
        const Rounds rs((int)count);
#pragma unroll
        for (int r = 0; r < kEpt; ++r) {
            if (r < rs.R) {                              // uniform
                const uint32_t i = min((uint32_t)rs.at(r), count - 1);
                key[r] = sh.key[i];
                // What an overlapping viewer (malformed offsets) left here may lie past n.
                pos[r] = min(sh.pos[i], pt.n - 1);
            }
        }
        lds_sync();                                      // sh.key is written again
        const uint64_t kmin = (uint64_t)sort_lds(sh, rs, key, pos);
        for (uint32_t i = thread_index(); i < count; i += kPartThreads)
            o.keys_out[to + done + i] = (int64_t)(sh.key[i] + kmin);
        const int64_t chunks = (int64_t)count * o.row_chunks;
        const int64_t first = (to + done) * o.row_chunks;
#pragma unroll 4
        for (int64_t c = thread_index(); c < chunks; c += kPartThreads) {
            const uint32_t i = (uint32_t)((uint64_t)c / (uint32_t)o.row_chunks);
            const int64_t from = pt.kb + sh.pos[i];
            o.rows_out[first + c] =
                o.rows_in[from * o.row_chunks + (c - (int64_t)i * o.row_chunks)];
        }
        done += count;
        lds_sync();                                      // sh.key is written again
    }
}

// A part whose records split_kernel has put together, or a viewer that was not split (at most SH::kCap
// records, one part).
template <typename SH>
__device__ __forceinline__ void sort_split_part(SH &sh, const int64_t *__restrict__ keys,
                                                const Part &pt, const Split &sp, Elem *buf0,
                                                Elem *buf1, const SortOut &o) {
    constexpr int kEpt = SH::kEpt;
    constexpr uint32_t kCap = SH::kCap;
    const bool whole = pt.n <= kSplitCap;
    uint32_t below = 0, m = pt.n;
    if (!whole)
        m = uniform(find_records(sh, pt, sp, below));
    if (m == 0)
        return;
    const int64_t to = uniform(pt.kb + below);
    if (m > kCap) {
        overlong_part(sh, pt, sp, m, buf0 + to, buf1 + to, to, o);
        return;
    }
    uint64_t key[kEpt];
    uint32_t pos[kEpt];
    const Rounds rs((int)m);
#pragma unroll
    for (int r = 0; r < kEpt; ++r) {
        if (r < rs.R) {                                  // uniform
            const uint32_t i = min((uint32_t)rs.at(r), m - 1);
            pos[r] = i;
            key[r] = (uint64_t)(whole ? keys[pt.kb + i] : split_record(sh, pt, sp, i, pos[r]));
        }
    }
    lds_sync();                                          // sh.adj and sh.start are written again
    const int64_t kmin = sort_lds(sh, rs, key, pos);
    emit(sh, pt, (uint64_t)kmin, (int)m, to, o);
}

// Records [base, base + n) go to the output unchanged (keys and rows, in input order).
__device__ __forceinline__ void copy_slice(const int64_t *__restrict__ keys, int64_t base, int64_t n,
                                           const SortOut &o) {
    for (int64_t i = threadIdx.x; i < n; i += kPartThreads)
        o.keys_out[base + i] = keys[base + i];
    const int64_t c0 = base * o.row_chunks, c1 = (base + n) * o.row_chunks;
    for (int64_t c = c0 + threadIdx.x; c < c1; c += kPartThreads)
        o.rows_out[c] = o.rows_in[c];
}

// Work items: one per viewer (its part 0), then one per multiple of `part` in [part, total). The
// multiple a * part that falls strictly inside a viewer is one more part of it, so a viewer's
// parts are numbered by the multiples it covers and no scan over the viewers is needed. A viewer of
// more than `most` parts is cut into `most`, its items taken together in even runs. False for items
// without records or inside a run (and where offsets break the rules).
__device__ __forceinline__ bool part_of(const int64_t *off, int32_t B, int64_t total, int32_t part,
                                        int64_t whole, uint32_t most, Part &pt, int64_t &n) {
    const int64_t it = blockIdx.x;
    int64_t v, a = 0;
    if (it < B) {
        v = it;
    } else {
        a = it - B + 1;
        v = owner<kPartThreads>(off, B, a * part);
    }
    int64_t ke;
    segment(off, total, v, pt.kb, ke);
    n = ke - pt.kb;
    const int64_t g = it < B ? 0 : a - (uint32_t)pt.kb / (uint32_t)part;
    if (n <= 0)
        return false;
    pt.G = n <= whole ? 1 : parts_of(pt.kb, ke, part);
    if (g < 0 || g >= pt.G || (it >= B && g == 0))
        return false;
    pt.n = (uint32_t)n;
    pt.g = (uint32_t)g;
    if (pt.G > most && n < kPartMaxRecords) {
        const uint32_t run = pt.g * most / pt.G;         // both below 2^12: see the limit of n
        if (pt.g > 0 && run == (pt.g - 1) * most / pt.G)
            return false;
        pt.g = run;
        pt.G = most;
    }
    return true;
}

// SPLIT: split_kernel has gone through the viewers of more than kSplitCap records; shorter ones are
// one part.
template <bool SPLIT>
__global__ __launch_bounds__(kPartThreads, SPLIT ? 8 : 4) void part_sort_kernel(
    const int64_t *__restrict__ keys, const int64_t *off, int32_t B, int32_t part, Split sp,
    Elem *buf0, Elem *buf1, SortOut o) {
    __shared__ PartTables<SPLIT ? kSplitEpt : kEpt> sh;
    Part pt;
    int64_t n;
    if (!part_of(off, B, o.total, part, SPLIT ? kSplitCap : part, SPLIT ? kRadix : ~0u, pt, n))
        return;
    if (n > o.limit || n >= kPartMaxRecords) {        // larger than the caller's bound
        const int64_t b0 = pt.kb + n * pt.g / pt.G, b1 = pt.kb + n * (pt.g + 1) / pt.G;
        copy_slice(keys, b0, b1 - b0, o);
        return;
    }
    if constexpr (SPLIT)
        sort_split_part(sh, keys, Part{uniform(pt.kb), uniform(pt.n), uniform(pt.g), uniform(pt.G)}, sp,
                        buf0, buf1, o);
    else
        sort_part(sh, keys, pt, buf0, buf1, o);
}

// ---- long viewers: records by part beforehand --------------------------------------------------
//
// Step 2 above reads a viewer once per part, which for long viewers costs more than all else, and
// the radix method's nine launches keep the rows waiting for six passes over the keys. Here
// every workgroup takes one chunk of at most kChunk records of a viewer of more than kSplitCap, finds the
// bounds of all the viewer's parts from the same sample, and writes the chunk's keys and positions
// ordered by part (stably, one digit pass in LDS) with the first index of every part. Nothing is
// counted over chunks: a part's workgroup in the next launch adds up the chunks' entries. Two
// launches against radix (or the scan above): 32 x 100,000 records of 128 bytes 262 -> 224 us, 64
// viewers of 100 to 30,000 of 64 bytes 42.6 -> 33, 1 x 100,000 58.6 -> 27.7.
//
// The bounds come from a histogram of the sample over kBins equal shares of its key span, a part
// starting as far into the share that holds its first sample record as that record is among the
// share's: any bounds will do that every chunk finds alike and that ascend. Where a share holds more
// than kShareMost sample records (keys that crowd or repeat), the sample is sorted instead, and the
// bounds are its records by key and position.
// A part of more than kSplitCap records, 3.2 times its share, is rare in key orders that know nothing
// of the sample, the rarer the more sample records a part has: kPerSplit of them up to 170 parts
// (108,000 records), fewer in longer viewers, whose sample is full, 8 at the longest. Per part (the
// share of a part is close to a gamma variate): 2e-7 at 12, 1.3e-6 at 200 parts, 4.4e-6 at 225, 1.4e-5
// at 255, which is one viewer of kSplitMax records in 280. (One is sorted in pieces, below.) Half of the
// keys in a tenth of the span, parts that start at their share's edge: the largest of 47,000 parts had
// 2,027 records; as far into it as above, 1,714 of 63,000. Viewers of more than kSplitMax records have
// longer parts, the longest 2,048 on average.
//
// Bound by its dependent steps and the instructions of the ranking: 3.2M records 37.9 us with four
// workgroups per CU, where 38 MB in and out alone take 12. Sorting the sample by 16 key bits instead
// of the histogram: 53 us; records straight from registers to their places, without LDS: 49.
constexpr int kBinBits = 13;
constexpr int kBins = 1 << kBinBits;
constexpr uint32_t kShareMost = 8;
constexpr uint32_t kPerSplit = 12;                       // sample records per part
// A bound is its share's lower edge plus less than a share, which in the last share that holds a sample
// record could pass the largest key and wrap. It does not: a bound's record has S / G records of
// the sample or more from itself on, so one that is not the last share's first would make it hold
// more than kShareMost, and the sample is then sorted.
static_assert(kPerSplit >= kShareMost && kSplitCap / kRadix >= kShareMost, "S / G >= kShareMost");

struct SplitShared {
    union {
        PartTables<kSplitEpt> p;
        int64_t out_key[kChunk];                         // over p.key and p.pos
        uint32_t out_pos[kChunk];
    };
    int64_t key[kRadix];                                 // lower bounds of parts 1, 2, ...
    uint32_t pos[kRadix];
};
static_assert(kChunk * sizeof(int64_t) <= offsetof(PartTables<kSplitEpt>, cnt), "p.cnt is in use");
static_assert(sizeof(PartTables<kSplitEpt>::key) >= kBins * 2, "16-bit counts of the shares");
static_assert(kBins == 16 * kPartThreads, "16 shares per thread");

// Bounds of the parts from the sample. Ends with a barrier.
__device__ __forceinline__ void sample_bounds(SplitShared &ss, const int64_t *__restrict__ keys,
                                              const Part &pt) {
    constexpr int E = kSplitEpt;
    PartTables<E> &sh = ss.p;
    const int tid = thread_index(), lane = tid & 63, w = wave_index();
    const Sample sm(pt, kPerSplit, kSplitCap);
    const Rounds sr((int)sm.S);
    uint64_t key[E];
    uint32_t pos[E];
    int64_t lo = INT64_MAX, hi = INT64_MIN;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        if (r < sr.R) {                                  // uniform
            pos[r] = sm.pos(min((uint32_t)sr.at(r), sm.S - 1));
            key[r] = (uint64_t)keys[pt.kb + pos[r]];
            lo = min(lo, (int64_t)key[r]);
            hi = max(hi, (int64_t)key[r]);
        }
    }
    uint32_t *bins = reinterpret_cast<uint32_t *>(sh.key);   // two 16-bit counts per word
    uint4 *mine = reinterpret_cast<uint4 *>(bins) + tid * 2;
    mine[0] = mine[1] = uint4{0, 0, 0, 0};
    key_range(sh, lo, hi);                               // has a barrier
    const uint64_t span = (uint64_t)hi - (uint64_t)lo;
    const int shift = max(0, (span ? 64 - __clzll(span) : 0) - kBinBits);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        if (r < sr.R && sr.at(r) < sr.n) {
            const uint32_t b = (uint32_t)((key[r] - (uint64_t)lo) >> shift);
            atomicAdd(&bins[b >> 1], 1u << (16 * (b & 1)));
        }
    }
    lds_sync();
    uint32_t sum = 0, most = 0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint4 x = mine[q];
        const uint32_t f[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            sum += (f[j] & 0xFFFFu) + (f[j] >> 16);
            most = max(most, max(f[j] & 0xFFFFu, f[j] >> 16));
        }
    }
    uint32_t before = wave_scan(sum);
    if (lane == 63)
        sh.run[0][w] = before;
    before -= sum;
    if (!__syncthreads_or(most > kShareMost)) {
#pragma unroll
        for (int q = 0; q < kPartWaves; ++q)
            before += q < w ? sh.run[0][q] : 0;
        sh.pos[tid] = before;                            // sample records before the thread's shares
        lds_sync();
        for (uint32_t b = tid + 1; b < pt.G; b += kPartThreads) {
            const uint32_t r = min(b * sm.S / pt.G, sm.S - 1);
            uint32_t t = 0;
#pragma unroll
            for (uint32_t half = kPartThreads / 2; half > 0; half >>= 1)
                t += sh.pos[t + half] <= r ? half : 0;
            uint32_t c = sh.pos[t], at = t * 16, first = c, in = 1;
            for (int j = 0; j < 16; ++j) {               // the share that holds record r
                const uint32_t x = (bins[t * 8 + j / 2] >> (16 * (j & 1))) & 0xFFFFu;
                if (c <= r) {
                    at = t * 16 + j;
                    first = c;
                    in = max(x, 1u);
                }
                c += x;
            }
            const double part = (double)(r - first) / (double)in;
            const uint64_t off = (uint64_t)(part * (double)((uint64_t)1 << shift));
            ss.key[b - 1] = (int64_t)(((uint64_t)at << shift) + off + (uint64_t)lo);
            ss.pos[b - 1] = 0;
        }
    } else {
        const int64_t kmin = sort_lds(sh, sr, key, pos);
        for (uint32_t b = tid + 1; b < pt.G; b += kPartThreads) {
            const uint32_t r = min(b * sm.S / pt.G, sm.S - 1);
            ss.key[b - 1] = (int64_t)(sh.key[r] + (uint64_t)kmin);
            ss.pos[b - 1] = sh.pos[r];
        }
    }
    lds_sync();
}

__global__ __launch_bounds__(kPartThreads, 8) void split_kernel(
    const int64_t *__restrict__ keys, const int64_t *off, int32_t B, Split sp, SortOut o) {
    constexpr int E = kChunkEpt;
    __shared__ SplitShared ss;
    PartTables<kSplitEpt> &sh = ss.p;
    Part ck;                                             // the chunk
    int64_t n64;
    if (!part_of(off, B, o.total, kChunk, kChunk, ~0u, ck, n64) || n64 <= kSplitCap || n64 > o.limit ||
        n64 >= kPartMaxRecords)
        return;
    const int tid = thread_index(), w = wave_index();
    const Part pt{ck.kb, ck.n, 0, min(parts_of(ck.kb, ck.kb + n64, kPartSplit), (uint32_t)kRadix)};
    const uint32_t c0 = part_begin(ck.n, ck.g, ck.G);
    const int n = (int)(part_begin(ck.n, ck.g + 1, ck.G) - c0);
    const Rounds rs(n);
    int64_t k[E];
#pragma unroll
    for (int r = 0; r < E; ++r)
        k[r] = keys[ck.kb + c0 + min(rs.at(r), n - 1)];
    sample_bounds(ss, keys, pt);
    // Part of each record: the bounds at or below it. By key alone first; where a bound's key is
    // the record's own, by position as well.
    const uint32_t nb = pt.G - 1;                        // >= 1
    uint32_t at[E];
#pragma unroll
    for (int r = 0; r < E; ++r)
        at[r] = 0;
    for (uint32_t len = nb; len > 1;) {                  // uniform
        const uint32_t half = len >> 1;
#pragma unroll
        for (int r = 0; r < E; ++r)
            at[r] += ss.key[at[r] + half - 1] <= k[r] ? half : 0;
        len -= half;
    }
#pragma unroll
    for (int r = 0; r < E; ++r) {
        at[r] += ss.key[at[r]] <= k[r] ? 1 : 0;
        const bool tie = at[r] > 0 && ss.key[at[r] - 1] == k[r];
        if (__ballot(tie)) {                             // uniform per wavefront
            const uint32_t p = c0 + rs.at(r);
            uint32_t a = 0;
            for (uint32_t l = nb; l > 0;) {
                const uint32_t half = l > 1 ? l >> 1 : 1, i = a + half - 1;
                const int64_t y = ss.key[i];
                a += y < k[r] || (y == k[r] && ss.pos[i] <= p) ? half : 0;
                l = l > 1 ? l - half : 0;
            }
            at[r] = a;
        }
    }
    uint32_t rd[E];
    rank_rounds(sh, at, rs.R, rs.first, n, 0, kRadix - 1, rd);
    lds_sync();
    digit_offsets(sh);
    lds_sync();
    // Through LDS, keys and then positions, so that both are written in order.
    const int64_t base = ck.kb + c0;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        if (r < rs.R && rs.at(r) < n) {
            rd[r] = sh.cnt[w][rd[r] & 0xFFu] + (rd[r] >> 8);
            ss.out_key[rd[r]] = k[r];
        }
    }
    lds_sync();
    for (int i = tid; i < n; i += kPartThreads)
        sp.key[base + i] = ss.out_key[i];
    lds_sync();
#pragma unroll
    for (int r = 0; r < E; ++r)
        if (r < rs.R && rs.at(r) < n)
            ss.out_pos[rd[r]] = c0 + rs.at(r);
    lds_sync();
    for (int i = tid; i < n; i += kPartThreads)
        sp.pos[base + i] = ss.out_pos[i];
    if (tid < kRadix)
        sp.start[sp.row(ck.kb, ck.g) * kRadix + tid] = (uint16_t)sh.start[tid];
}

// ---- ranks by comparison: the smallest calls --------------------------------------------------
//
// A record's place is the number of records of its viewer that order before it. A workgroup takes
// `per` consecutive records, holds the viewer's whole key list in registers (kRankEpt keys per
// lane at a time) and counts for one record after the other: a compare per 64 keys, whose lane
// mask the scalar unit counts. Quadratic in the list, but the compares of a short list cost less
// than one dependent step of any other method, and nothing but the key load comes before them.
// The rows are read meanwhile. The cost is the instructions issued, about 14 + 3 R per record and
// wavefront that holds R rounds of the list: a list of up to 512 keys is therefore held whole by
// every wavefront, each with records of its own, and longer ones by groups of 2, 4, 8 or 16.
constexpr int kRankThreads = 1024;
constexpr int kRankWaves = kRankThreads / 64;
constexpr int kRankEpt = 8;
constexpr int kRankGrid = 256;                 // workgroups, of at most kRankMaxPer records each
constexpr int kRankMaxPer = 256;

// Groups of 1 << rank_group(n) wavefronts hold a list of n keys.
__host__ __device__ inline int rank_group(int64_t n) {
    int gs = 0;
    while ((kRankWaves >> gs) > 1 && n > (int64_t)(kRankEpt * 64) << gs)
        ++gs;
    return gs;
}

struct RankShared {
    uint32_t diff[kRankWaves];
    uint32_t cnt[kRankWaves][64];
    uint32_t rank[kRankMaxPer];
};

__device__ __forceinline__ uint64_t lane_value(uint64_t x, int lane) {
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)x, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// cnt of lane t < c += keys k[r], r < R, of the wavefront that order before the record whose key
// lane t holds in x. PACKED: k and x hold (key, position) in one word each. Otherwise k[r]'s
// position is pos + r * 64 and lane t's record's is p + t.
template <int R, bool PACKED>
__device__ __forceinline__ void count_before(const uint64_t (&k)[kRankEpt], uint64_t x, int c,
                                             uint32_t pos, uint32_t p, uint32_t &cnt) {
    const int lane = threadIdx.x & 63;
    for (int t = 0; t < c; ++t) {
        const uint64_t y = lane_value(x, t);
        uint32_t n = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            n += __popcll(__ballot(k[r] < y));
            if (!PACKED)
                n += __popcll(__ballot(k[r] == y) & __ballot(pos + r * 64 < p + t));
        }
        cnt += lane == t ? n : 0;
    }
}

template <bool PACKED>
__device__ __forceinline__ void count_before(int R, const uint64_t (&k)[kRankEpt], uint64_t x, int c,
                                             uint32_t pos, uint32_t p, uint32_t &cnt) {
    switch (R) {                                         // uniform
    case 1: count_before<1, PACKED>(k, x, c, pos, p, cnt); break;
    case 2: count_before<2, PACKED>(k, x, c, pos, p, cnt); break;
    case 3: count_before<3, PACKED>(k, x, c, pos, p, cnt); break;
    case 4: count_before<4, PACKED>(k, x, c, pos, p, cnt); break;
    case 5: count_before<5, PACKED>(k, x, c, pos, p, cnt); break;
    case 6: count_before<6, PACKED>(k, x, c, pos, p, cnt); break;
    case 7: count_before<7, PACKED>(k, x, c, pos, p, cnt); break;
    default: count_before<8, PACKED>(k, x, c, pos, p, cnt); break;
    }
}

// Records [p, p + c) of the viewer with records [kb, kb + n), p relative to kb.
__device__ __forceinline__ void rank_records(RankShared &sh, const int64_t *__restrict__ keys,
                                             int64_t kb, uint32_t n, uint32_t p, int c,
                                             const SortOut &o) {
    constexpr uint64_t kFlip = (uint64_t)1 << 63;        // signed order as unsigned order
    const int tid = threadIdx.x, lane = tid & 63, w = wave_index();
    const int64_t *gk = keys + kb;
    // Groups of 1 << gs wavefronts hold the list; group `grp` ranks records [t0, t0 + mine).
    const int gs = rank_group(n);
    const int in = w & ((1 << gs) - 1), grp = w >> gs;
    const int share = (c + (kRankWaves >> gs) - 1) / (kRankWaves >> gs);
    const int t0 = grp * share, mine = max(0, min(share, c - t0));
    const uint32_t mp = p + min(t0 + lane, c - 1);       // the record whose rank the lane gets
    const uint64_t key = (uint64_t)gk[mp] ^ kFlip;
    const uint64_t ref = (uint64_t)gk[p] ^ kFlip;
    const int64_t out_key = gk[p + min(tid, c - 1)];
    // The first row chunk of the thread, on its way while the ranks are counted.
    const int chunks = c * o.row_chunks;
    const chunk_t *rows = o.rows_in + (kb + p) * o.row_chunks;
    const chunk_t first = rows[min(tid, chunks - 1)];
    const int bits = 32 - __clz(n);                      // positions are below 2^bits
    const uint32_t turn = (uint32_t)(kRankEpt * 64) << gs;
    uint32_t cnt = 0;
    for (uint32_t c0 = 0; c0 < n; c0 += turn) {          // uniform
        const int R = (int)((min(n - c0, turn) + (64u << gs) - 1) >> (6 + gs));
        const uint32_t pos = c0 + in * R * 64 + lane;    // (wavefront, round, lane)
        uint64_t k[kRankEpt];
#pragma unroll
        for (int r = 0; r < kRankEpt; ++r)
            if (r < R)                                   // uniform
                k[r] = (uint64_t)gk[min(pos + r * 64, n - 1)] ^ kFlip;
        uint64_t diff = key ^ ref;
#pragma unroll
        for (int r = 0; r < kRankEpt; ++r)
            if (r < R)
                diff |= k[r] ^ ref;
        // Bits in which keys differ, over the workgroup: below them, room for the position?
        uint32_t any = (uint32_t)(diff >> 32);
#pragma unroll
        for (int d = 32; d > 0; d >>= 1)
            any |= __shfl_xor(any, d);
        lds_sync();                                      // the last turn's readers are done
        if (lane == 0)
            sh.diff[w] = any;
        lds_sync();
#pragma unroll
        for (int q = 0; q < kRankWaves; ++q)
            any |= sh.diff[q];
        any = __builtin_amdgcn_readfirstlane(any);
        const bool packed = __clz(any | 1) >= bits;      // uniform: the top bits are alike
#pragma unroll
        for (int r = 0; r < kRankEpt; ++r) {
            // Past the end: above every packed record; or the largest key, at a position past
            // every record's.
            if (r < R)
                k[r] = pos + r * 64 >= n ? ~(uint64_t)0
                                         : (packed ? (k[r] << bits) | (pos + r * 64) : k[r]);
        }
        if (packed)
            count_before<true>(R, k, (key << bits) | mp, mine, pos, p + t0, cnt);
        else
            count_before<false>(R, k, key, mine, pos, p + t0, cnt);
    }
    sh.cnt[w][lane] = cnt;
    lds_sync();
    if (tid < c) {
        const int g = tid / share, t = tid - g * share;
        uint32_t rank = 0;
        for (int q = 0; q < 1 << gs; ++q)
            rank += sh.cnt[(g << gs) + q][t];
        sh.rank[tid] = rank;
        o.keys_out[kb + rank] = out_key;
    }
    lds_sync();
    for (int g = tid; g < chunks; g += kRankThreads) {
        const int rec = g / o.row_chunks;
        o.rows_out[(kb + sh.rank[rec]) * o.row_chunks + (g - rec * o.row_chunks)] =
            g < kRankThreads ? first : rows[g];
    }
}

// Workgroup b takes the records [b * per, (b + 1) * per) of the call, viewer by viewer.
__global__ __launch_bounds__(kRankThreads) void rank_sort_kernel(const int64_t *__restrict__ keys,
                                                                 const int64_t *off, int32_t B,
                                                                 int32_t per, SortOut o) {
    __shared__ RankShared sh;
    int64_t p = (int64_t)blockIdx.x * per;
    const int64_t end = min(p + per, o.total);
    while (p < end) {                                    // uniform
        const int64_t v = owner<kRankThreads>(off, B, p);
        int64_t kb, ke;
        segment(off, o.total, v, kb, ke);
        if (p < kb || p >= ke)
            break;                                       // offsets that break the rules
        const int64_t e = min(end, ke);
        if (ke - kb > o.limit) {                         // larger than the caller's bound
            for (int64_t i = p + threadIdx.x; i < e; i += kRankThreads)
                o.keys_out[i] = keys[i];
            for (int64_t g = p * o.row_chunks + threadIdx.x; g < e * o.row_chunks; g += kRankThreads)
                o.rows_out[g] = o.rows_in[g];
        } else {
            rank_records(sh, keys, kb, (uint32_t)(ke - kb), (uint32_t)(p - kb), (int)(e - p), o);
        }
        lds_sync();                                      // sh is reused
        p = e;
    }
}

}  // namespace

hipError_t launch_part_sort(int32_t n_viewers, const int64_t *key_offsets, const int64_t *keys_in,
                            const void *rows_in, int32_t row_bytes, int64_t total, int64_t limit,
                            int64_t *keys_out, void *rows_out, void *buf0, void *buf1,
                            void *chunks, int32_t method, hipStream_t stream) {
    const SortOut o{limit, total, static_cast<const chunk_t *>(rows_in), row_bytes / 16, keys_out,
                    static_cast<chunk_t *>(rows_out), nullptr};
    if (method == kSortRank) {
        int32_t per = (int32_t)((total + kRankGrid - 1) / kRankGrid);
        // A group of wavefronts ranks at most 64 records (one lane each).
        const int32_t most = min(kRankMaxPer, 64 * (kRankWaves >> rank_group(limit)));
        if (per > most)
            per = most;
        hipLaunchKernelGGL(rank_sort_kernel, dim3((unsigned)((total + per - 1) / per)),
                           dim3(kRankThreads), 0, stream, keys_in, key_offsets, n_viewers, per, o);
        return hipGetLastError();
    }
    Elem *b0 = static_cast<Elem *>(buf0), *b1 = static_cast<Elem *>(buf1);
    if (method == kSortSplit) {
        Split sp{static_cast<int64_t *>(chunks), nullptr, nullptr, (uint32_t)(total / kChunk) + 1};
        sp.pos = reinterpret_cast<uint32_t *>(sp.key + total);
        sp.start = reinterpret_cast<uint16_t *>(sp.pos + total);
        hipLaunchKernelGGL(split_kernel, dim3((unsigned)(n_viewers + (total - 1) / kChunk)),
                           dim3(kPartThreads), 0, stream, keys_in, key_offsets, n_viewers, sp, o);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL(part_sort_kernel<true>,
                           dim3((unsigned)(n_viewers + (total - 1) / kPartSplit)),
                           dim3(kPartThreads), 0, stream, keys_in, key_offsets, n_viewers,
                           kPartSplit, sp, b0, b1, o);
        return hipGetLastError();
    }
    const int32_t part = total <= kPartSmallTotal ? kPartSmall : kPartLarge;
    hipLaunchKernelGGL(part_sort_kernel<false>, dim3((unsigned)(n_viewers + (total - 1) / part)),
                       dim3(kPartThreads), 0, stream, keys_in, key_offsets, n_viewers, part, Split{},
                       b0, b1, o);
    return hipGetLastError();
}

}  // namespace ccj
