// Weight-ordered loop for graphs without locality (declarations; see
// gr_order.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace gr {

// In-arcs ordered by weight (one device allocation, `base`): rows as the
// graph's in-arcs (ro_in), every run of kOrderChunk arcs of a row sorted.
// The two lightest arcs of each vertex and the weight of the third stand in
// arrays of their own; vertices of more than kOrderChunk arcs have none there
// (weight INF, tail kOrderNone) and are listed chunk by chunk instead.
constexpr int32_t kOrderChunk = 1024;
constexpr uint32_t kOrderNone = 0xFFFFFFFFu;
// Arcs per queue entry of a push.  The loop's arc indices are 32-bit and step
// past the end of a row by up to that many.
constexpr int32_t kOrderRun = 256;
constexpr bool order_indexes(int32_t m) { return m > 0 && m <= INT32_MAX - kOrderRun; }
struct OrderSet {
    void *base = nullptr;
    size_t bytes = 0;
    uint2 *arc = nullptr;      // [m] (tail, weight bits)
    uint2 *a0 = nullptr, *a1 = nullptr;  // [n] each: the two lightest arcs (tail, weight bits)
    uint32_t *w2 = nullptr;    // [n]
    uint4 *chunk = nullptr;    // the long rows' chunks: (vertex, first arc, end, lightest weight)
    int32_t nchunks = 0;
};
// ro_in / adj_in: the graph's in-arcs; h_ro_in: the offsets on the host; limit:
// bytes that the layout may take (past them hipErrorOutOfMemory).
hipError_t order_build(OrderSet *out, int32_t n, int32_t m, const int32_t *ro_in, const uint2 *adj_in,
                       const int32_t *h_ro_in, int wt, size_t limit, hipStream_t st);

// One query of a launch.
struct OrderJob {
    const int32_t *ro;      // out-arcs (push)
    const uint2 *adj;
    const int32_t *ro_in;   // in-arcs, by weight
    const uint2 *arc;
    const uint2 *a0, *a1;
    const uint32_t *w2;
    const uint4 *chunk;
    uint32_t *dist;         // the query's output, n values
    uint64_t *bits;         // workspace: 2 bitmaps of nword words, of what a push put on the next frontier
    uint2 *queue;           // workspace: 2 x kOrderRegions x cap frontier entries, by round parity
    unsigned long long *ctl;  // workspace: kOrderCtlWords
    int32_t n, m, nchunks, src, nword, cap;
};
constexpr int kOrderRegions = 16;
constexpr int kOrderRegionWords = 32;  // a region's counters fill a 256-byte line
constexpr int kOrderState = 3 * kOrderRegions * kOrderRegionWords;
constexpr int kOrderCtlWords = kOrderState + 32;
constexpr int kOrderMaxJobs = 64;
// Statistics words per query in stat (pinned host memory): 1 at the end, else 0
// until the last launch of a call of order_rounds stores 2 (first + rounds); rounds; pull rounds; frontier vertices; arcs pushed; arcs pulled.
constexpr int kOrderStatWords = 6;

// Batched queries on one graph: up to kBatchLanes sources, one per wave lane,
// with the distances vertex-major (64 words per vertex).
struct OrderBatch {
    OrderJob g;               // the graph (dist, bits and src unused)
    uint32_t *D;              // workspace: n x 64
    int32_t k;
    unsigned long long *mask;  // workspace: 3 x n, the sources whose frontier holds a vertex, by round mod 3
    uint32_t *mu;             // workspace: 3 x kOrderRegions x 64 complements of each source's mu
};
constexpr int kOrderBatchStatWords = 6;  // as above, rounds, pull rounds, frontier vertices, arcs read, (arc, source) pairs decided

size_t order_batch_bytes(int32_t n);
void order_batch_carve(OrderBatch *b, void *ws);
hipError_t order_batch_begin(const OrderBatch &b, const int32_t *srcs, int wt, hipStream_t st);
hipError_t order_batch_rounds(const OrderBatch &b, int wt, int64_t first, int32_t rounds, int num_cu,
                              unsigned long long *stat, hipStream_t st);

size_t order_ws_bytes(int32_t n);
// Fills j's workspace pointers from ws.
void order_carve(OrderJob *j, void *ws);
// The job table (device memory, kOrderMaxJobs entries) and every query's first frontier.
hipError_t order_begin(const OrderJob *jobs, int32_t k, int wt, OrderJob *table, hipStream_t st);
// `rounds` rounds of every query (those that are done return at once), from
// round `first` on.
hipError_t order_rounds(const OrderJob *jobs, int32_t k, int wt, const OrderJob *table, int64_t first, int32_t rounds,
                        unsigned long long *stat, hipStream_t st);

}  // namespace gr
