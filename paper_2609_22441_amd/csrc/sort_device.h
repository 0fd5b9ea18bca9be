// Device helpers shared by the sort kernels (sort_kernels.hip, part_sort_kernels.hip).
#pragma once

#include <stdint.h>

#include <hip/hip_runtime.h>

namespace ccj {
namespace {

constexpr int kThreads = 512;                     // threads per workgroup
constexpr int kWaves = kThreads / 64;

typedef unsigned int chunk_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ int64_t clampk(int64_t v, int64_t hi) {
    return v < 0 ? 0 : (v > hi ? hi : v);
}

// Segment [kb, ke) of viewer v, offsets clamped to [0, total] and made non-decreasing.
__device__ __forceinline__ void segment(const int64_t *off, int64_t total, int64_t v, int64_t &kb,
                                        int64_t &ke) {
    kb = clampk(off[v], total);
    ke = max(kb, clampk(off[v + 1], total));
}

// Largest v in [0, B) with tile_off[v] <= t (tile_off non-decreasing, tile_off[0] = 0), found by
// the whole workgroup of THREADS (call it uniformly). Each round every thread probes one of THREADS
// evenly spaced viewers; the probes at or below t are a prefix, and its length narrows the range
// THREADS-fold. Up to THREADS viewers take one round of independent loads instead of a chain
// of ~log2(B) dependent ones.
template <int THREADS = kThreads>
__device__ __forceinline__ int64_t owner(const int64_t *tile_off, int64_t B, int64_t t) {
    int64_t lo = 0, hi = B - 1;                   // tile_off[lo] <= t; the answer is in [lo, hi]
    while (lo < hi) {
        const int64_t step = (hi - lo + THREADS) / THREADS;
        const int64_t v = lo + (int64_t)threadIdx.x * step;
        // Probe lo holds by the invariant; offsets that break the rules could deny it, and the
        // floor of 1 keeps every later probe in [0, B) all the same.
        const int c = max(1, __syncthreads_count(v <= hi && tile_off[v] <= t));
        const int64_t nlo = lo + (int64_t)(c - 1) * step;
        hi = min(hi, nlo + step - 1);
        lo = nlo;
    }
    return lo;
}

struct SortOut {
    int64_t limit;          // viewers with more records are copied through in input order
    int64_t total;
    const chunk_t *rows_in;
    int32_t row_chunks;
    int64_t *keys_out;
    chunk_t *rows_out;
    uint32_t *perm;         // [total]: input position of the record at each output position
};

// Copy the feature rows of n sorted records: record i's row goes from flat input position
// src(i) to flat output position dst(i), skipped where dst(i) < 0. 16-byte chunks in batches of U
// per thread, two batches in flight: the loads of the next batch are issued before the stores
// of the current one (vector-memory completions are counted in issue order, stores included, so
// a load issued after a store could only be waited for together with it). The sorted rows are
// not read again by this call: non-temporal stores keep them from evicting the lines of rows
// still to be gathered.
template <int U, int THREADS = kThreads, typename Map>
__device__ __forceinline__ void copy_rows(int n, const SortOut &o, Map map) {
    const int row_chunks = o.row_chunks;
    const int n_chunks = n * row_chunks;
    // Chunk g of the thread's sequence (g = threadIdx.x + j * THREADS) is chunk q of record
    // rec; both advance by THREADS chunks without a division.
    const int drec = THREADS / row_chunks, dq = THREADS - drec * row_chunks;
    int rec = threadIdx.x / row_chunks, q = threadIdx.x - rec * row_chunks;
    auto load = [&](int g0, chunk_t (&c)[U], int64_t (&to)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int g = g0 + u * THREADS;
            to[u] = -1;
            if (g < n_chunks) {
                int64_t src, dst;
                map(rec, src, dst);
                if (dst >= 0) {
                    c[u] = o.rows_in[src * row_chunks + q];
                    to[u] = dst * row_chunks + q;
                }
            }
            rec += drec;
            q += dq;
            if (q >= row_chunks) {
                q -= row_chunks;
                ++rec;
            }
        }
    };
    auto store = [&](const chunk_t (&c)[U], const int64_t (&to)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (to[u] >= 0)
                __builtin_nontemporal_store(c[u], o.rows_out + to[u]);
    };
    chunk_t ca[U], cb[U];
    int64_t ta[U], tb[U];
    load(threadIdx.x, ca, ta);
    for (int g0 = threadIdx.x; g0 < n_chunks; g0 += 2 * U * THREADS) {
        load(g0 + U * THREADS, cb, tb);
        store(ca, ta);
        load(g0 + 2 * U * THREADS, ca, ta);
        store(cb, tb);
    }
}

}  // namespace
}  // namespace ccj
