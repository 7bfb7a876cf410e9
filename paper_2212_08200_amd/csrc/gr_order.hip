// Weight-ordered loop (the paper's push / pull operators, Section III-C, with
// the pull's arcs ordered by weight).
//
// On graphs without locality a push relaxes every arc of the frontier, three
// to five times over the query (R-MAT 20: 166 M relaxations for 31 M arcs),
// each a random access and some a memory-side atomic.  Nearly all are lost: the
// hubs' distances lie within a few light weights of each other, so a vertex is
// improved through its lightest arcs or not at all.  Here a round pulls: with mu
// the smallest distance that the round before improved, an arc (u, v, w) can
// only improve v if mu (+) w < dist[v], so v's arcs are read in order of weight
// until that fails -- one or two arcs per vertex and round (R-MAT 20: 15 M arcs
// read in 19 rounds).  (+) is monotone in both operands, so what is not read
// could not have improved v: mu (+) w <= dist[u] (+) w for every u that the
// round before improved, and a u improved earlier was read then or was ruled
// out then.  Whether a tail is on the frontier is not asked: a pull keeps no
// bitmap, and a distance lowered earlier in the same round counts at once
// (against testing the tails' bits first, R-MAT 22: 929-1253 -> 817-1082 us,
// 31-48 -> 25-42 M arcs; 20: 621-724 -> 583-669; uniform of 200,000 vertices:
// 537-566 -> 475-501; 15: 203-232 -> 193-219).
//
// Bound by the chain of dependent loads in a round (its counters, a vertex, its
// tails, its row, the tails again: 17-20 us at 200,000 to 1 M vertices, 6 us at
// 32 K) and, on graphs past the caches, by memory: R-MAT 22 moves 247 MB per
// launch of 60 us on average, 4.1 TB/s where a copy reaches 4.7 (62% of the L2s'
// requests miss).  Measured against the push-only rounds: R-MAT 15, 432 -> 190
// us; 20 (binary32), 1925 -> 570; 22, 3421 -> 820.
//
// A pull round reads every vertex's distance and lightest weight (streamed),
// so small frontiers are pushed instead, from a queue of (vertex, run of 256
// arcs) entries: a round pushes while its frontier is small (kOrderBias) and
// the queue held it.  A pull writes no queue, so pulls follow, until their
// frontier is small again: then they keep one, and a push may follow
// (kBackArcs).
//
// One launch is one round of every query in it; the launches of a query are
// enqueued ahead, each reads the state that the round before left, and those
// past the end return at once.  State: three slots of counters rotated over the
// rounds, each in kOrderRegions regions on 256-byte lines of their own (memory-
// side atomics to one line are serialised: a block adds to region blockIdx mod
// kOrderRegions), summed by every block at its start; two bitmaps of what a
// push put on the next frontier (one written, one cleared).
#include "gr_order.h"

#include <algorithm>
#include <vector>

#include "gr_device.h"

namespace gr {

namespace {

// A first pull reads each vertex's arcs until one comes from the frontier,
// about m / E of them (E: the frontier's arcs), so n m / E in all, against E
// for a push: pull when kOrderBias E^2 >= n m.  (A scale-22 R-MAT query whose
// 9 M-arc frontier pulled under E >= m / 24 read 31 M arcs and took 1570 us,
// 1050 with this rule; a bias of 1 or 16 measures the same on other queries.)
constexpr double kOrderBias = 4.0;
// After pulls.  A pull streams every vertex (n) and reads the arcs of the
// vertices not reached yet in vain (R, as many as the pull before read), so a
// query with a second wave of growth, or a long tail, pushes again: when the
// frontier's arcs E satisfy kBackArcs E + kBackFixed <= n + kBackRead R.  That
// needs a queue from the pull before, which it keeps where a push could follow
// (n + kBackRead R >= kBackFixed) and its own frontier was at most n /
// kBackShare vertices.  Two R-MAT 17 graphs joined by a path of 300: 58.5 ms
// when all rounds after the first pull pulled, 3.6 so (7.2 in pushes alone);
// R-MAT 14 and a path of 1,000: 168 -> 8.2 (13.8); uniform of 300,000 vertices
// with unreachable parts 0.73 -> 0.62.  kBackFixed is what keeping a queue and
// a push's longer chain cost (with half of it R-MAT 18 with two arcs per
// vertex took 0.25 ms against 0.235; with kBackArcs 4 instead of 16 against
// kBackRead 1 the same); kBackShare 4 and 64 measure within 5%.
constexpr unsigned long long kBackArcs = 16, kBackFixed = 1ull << 20, kBackRead = 4, kBackShare = 16;
constexpr int kOrderVerts = 512;     // vertices per block of a pull, two per thread
// Lines of a row's arcs that a pull reads at once after the first: rows are
// bound by the chain of line, tails' distances and best (a bipartite graph of
// 2,000 and 200,000 vertices whose rows have 500 arcs 1.52 ms with one, 1.25
// with two, 1.01 with four, in pushes 0.95; R-MAT 15 3% less with four).
constexpr int kPullWide = 4;
constexpr int kPushRun = kOrderRun;  // arcs per queue entry

// Counters of a region, as words: frontier vertices, their arcs, the complement
// of mu (a maximum: a cleared word is neutral), queue entries, flags, and the
// arcs that the round before read.
constexpr int kRgF = 0, kRgE = 1, kRgMu = 2, kRgCnt = 3, kRgFlags = 4, kRgRead = 5;
// Over: the queue does not hold the frontier; Pulled: the round before pulled.
constexpr unsigned long long kFlagOver = 1ull, kFlagPulled = 2ull;
// Batches: the frontier's masks are set; those of the frontier before were.
constexpr unsigned long long kFlagMarked = 4ull, kFlagWasMarked = 8ull;
// State words after the slots (block 0 of each launch keeps them).
constexpr int kStDone = 0, kStPulls = 2, kStF = 3, kStPushed = 4, kStPulledArcs = 5;

template <typename T>
using gptr = T __attribute__((address_space(1))) *;
template <typename T>
__device__ __forceinline__ gptr<T> to_global(T *p) {
    return (gptr<T>)p;
}
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct OrderArgs {
    const OrderJob *job;
    int64_t round;
    unsigned long long *stat;
    unsigned long long tag;  // stored if the query goes on, and not 0
};

__device__ __forceinline__ uint32_t ld_dev(gptr<uint32_t> p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Across a wave with DPP moves (a permute keeps a register per distance for the
// whole kernel, 15 spills in k_order).
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp(unsigned long long x) {
    return (unsigned long long)dpp<CTRL>((uint32_t)(x >> 32)) << 32 | dpp<CTRL>((uint32_t)x);
}
// The first lane's value, as a scalar.
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ unsigned long long uniform(unsigned long long x) {
    return (unsigned long long)uniform((uint32_t)(x >> 32)) << 32 | uniform((uint32_t)x);
}
// f over every run of 16 lanes, in each of them.
template <typename T, typename F>
__device__ __forceinline__ T over_row(T x, F f) {
    x = f(x, dpp<0xB1>(x));   // quad_perm 1,0,3,2
    x = f(x, dpp<0x4E>(x));   // quad_perm 2,3,0,1
    x = f(x, dpp<0x141>(x));  // row_half_mirror
    return f(x, dpp<0x140>(x));  // row_mirror
}
// Inclusive running sum.
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
#define DPPADD(ctrl, rows) x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, rows, 0xF, false)
    DPPADD(0x111, 0xF);  // row_shr 1, 2, 4, 8
    DPPADD(0x112, 0xF);
    DPPADD(0x114, 0xF);
    DPPADD(0x118, 0xF);
    DPPADD(0x142, 0xA);  // row_bcast 15 into the odd rows
    DPPADD(0x143, 0xC);  // row_bcast 31 into the upper half
#undef DPPADD
    return x;
}

// Totals of a slot (every lane of every wave gets them).  A launch's chain starts
// with them: 64 bits only where the sum needs them.
struct Totals {
    unsigned long long E;
    uint32_t F, flags, read, mu;
};
__device__ __forceinline__ Totals read_slot(gptr<const unsigned long long> s) {
    static_assert(kOrderRegions == 16, "a region per lane of a row");
    gptr<const unsigned long long> r = s + (threadIdx.x % kOrderRegions) * kOrderRegionWords;
    const unsigned long long E = r[kRgE];
    const uint32_t F = (uint32_t)r[kRgF], o = (uint32_t)r[kRgFlags], d = (uint32_t)r[kRgRead], mu = ~(uint32_t)r[kRgMu];
    const auto sum = [](auto x, auto y) { return x + y; };
    Totals T;
    T.F = uniform(over_row(F, sum));
    T.E = uniform(over_row(E, sum));
    T.flags = uniform(over_row(o, [](uint32_t x, uint32_t y) { return x | y; }));
    T.read = uniform(over_row(d, sum));
    T.mu = uniform(over_row(mu, [](uint32_t x, uint32_t y) { return min(x, y); }));
    return T;
}

constexpr int kBeginJobs = 16;
struct BeginArgs {
    OrderJob job[kBeginJobs];
    OrderJob *table;
    uint32_t inf;
};

__global__ __launch_bounds__(256) void k_order_begin(BeginArgs a) {
    const OrderJob j = a.job[blockIdx.y];
    const int32_t t = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
    for (int64_t i = t; i < j.n; i += step) j.dist[i] = i == j.src ? 0u : a.inf;
    for (int64_t i = t; i < 2 * (int64_t)j.nword; i += step) j.bits[i] = 0ull;
    const int32_t deg = j.ro[j.src + 1] - j.ro[j.src], runs = (deg + kPushRun - 1) / kPushRun;
    // round 0's counters (region 0); mu = 0, complemented
    const bool fits = runs <= j.cap;
    for (int32_t i = t; i < kOrderCtlWords; i += step)
        j.ctl[i] = i == kRgF ? (deg > 0 ? 1ull : 0ull)
                   : i == kRgE ? (unsigned long long)deg
                   : i == kRgMu ? 0xFFFFFFFFull
                   : i == kRgCnt ? (unsigned long long)(fits ? runs : 0)
                   : i == kRgFlags ? (fits ? 0ull : kFlagOver)
                                  : 0ull;
    if (fits)
        for (int32_t i = t; i < runs; i += step) j.queue[i] = make_uint2((uint32_t)j.src, (uint32_t)i);
    if (t == 0) a.table[blockIdx.y] = j;
}

// Puts up to K vertices per lane on the next frontier: their runs go to the
// region's list, in one atomic per wave.  count: whether the vertices are
// counted too.
template <int K, int RUN>
__device__ __forceinline__ void enqueue(gptr<const int32_t> ro, int32_t cap, gptr<unsigned long long> region,
                                        gptr<u32x2> next_queue, const uint32_t (&v)[K], const bool (&on)[K],
                                        bool count) {
    const int lane = threadIdx.x & 63;
    uint32_t runs = 0, low = 0, high = 0, deg[K];
    uint32_t news = 0;  // (a vertex without out-arcs is on no frontier)
#pragma unroll
    for (int k = 0; k < K; ++k) {
        deg[k] = on[k] ? (uint32_t)(ro[v[k] + 1] - ro[v[k]]) : 0u;
        runs += (deg[k] + RUN - 1) / RUN;
        low += deg[k] & 0xFFFFu;
        high += deg[k] >> 16;
        news += (uint32_t)__popcll(__ballot(deg[k] > 0u));
    }
    if (news == 0u) return;
    const uint32_t before = wave_scan(runs);
    const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)before, 63);
    const unsigned long long sum =
        ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)wave_scan(high), 63) << 16) +
        (uint32_t)__builtin_amdgcn_readlane((int)wave_scan(low), 63);
    unsigned long long base = 0;
    if (lane == 0) {
        base = __hip_atomic_fetch_add(region + kRgCnt, (unsigned long long)all, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
        if (count)
            (void)__hip_atomic_fetch_add(region + kRgF, (unsigned long long)news, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
        (void)__hip_atomic_fetch_add(region + kRgE, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    base = (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(base >> 32)) << 32 |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
    if (base + all > (unsigned long long)cap) {  // the next round pulls
        if (lane == 0)
            (void)__hip_atomic_fetch_or(region + kRgFlags, kFlagOver, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    uint32_t at = (uint32_t)base + before - runs;
#pragma unroll
    for (int k = 0; k < K; ++k)
        for (uint32_t r = 0; r * RUN < deg[k]; ++r) next_queue[at++] = u32x2{v[k], r};
}

constexpr int kPushArcs = kPushRun / 64;  // arcs per lane of an entry
constexpr int kPackArcs = 2;              // of a pass over several entries

// One push pass of a wave: K arcs per lane, each (if ok) offering its
// tail's distance du (+) its weight.
template <int WT, int K>
__device__ __forceinline__ void push_pass(const OrderJob &J, gptr<uint32_t> dist, gptr<unsigned long long> next_bits,
                                          gptr<u32x2> next_queue, gptr<unsigned long long> region,
                                          const u32x2 (&a)[K], const uint32_t (&du)[K],
                                          const bool (&ok)[K], uint32_t &lowest) {
    uint32_t cur[K], nd[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        nd[k] = plus<WT>(du[k], a[k].y);
        cur[k] = dist[a[k].x];
    }
    uint32_t old[K], v[K];
    bool win[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        win[k] = ok[k] && nd[k] < cur[k];
        if (win[k])
            old[k] = __hip_atomic_fetch_min(dist + a[k].x, nd[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    unsigned long long was[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        win[k] = win[k] && nd[k] < old[k];
        if (win[k]) {
            lowest = min(lowest, nd[k]);
            was[k] = __hip_atomic_fetch_or(next_bits + (a[k].x >> 6), 1ull << (a[k].x & 63), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // vertices new on the next frontier
#pragma unroll
    for (int k = 0; k < K; ++k) {
        v[k] = a[k].x;
        win[k] = win[k] && !(was[k] >> (a[k].x & 63) & 1ull);
    }
    enqueue<K, kPushRun>(to_global(J.ro), J.cap, region, next_queue, v, win, true);
}

// An entry of the queue: a wave takes its arcs in one pass.
template <int WT>
__device__ __forceinline__ void push_entry(const OrderJob &J, gptr<uint32_t> dist, gptr<unsigned long long> next_bits,
                                           gptr<u32x2> next_queue, gptr<unsigned long long> region, u32x2 ent,
                                           uint32_t &lowest) {
    const int lane = threadIdx.x & 63;
    gptr<const int32_t> ro = to_global(J.ro);
    gptr<const u32x2> adj = reinterpret_cast<gptr<const u32x2>>(to_global(J.adj));
    const int32_t e0 = ro[ent.x] + (int32_t)ent.y * kPushRun, e1 = min(ro[ent.x + 1], e0 + kPushRun);
    const uint32_t d = ld_dev(dist + ent.x);
    u32x2 a[kPushArcs];
    uint32_t du[kPushArcs];
    bool ok[kPushArcs];
#pragma unroll
    for (int k = 0; k < kPushArcs; ++k) {
        a[k] = adj[min(e0 + k * 64 + lane, e1 - 1)];
        du[k] = d;
        ok[k] = e0 + k * 64 + lane < e1;
    }
    push_pass<WT, kPushArcs>(J, dist, next_bits, next_queue, region, a, du, ok, lowest);
}

// Several entries at once (one per lane, has: this lane's): their arcs end to
// end, 128 to a pass, each lane finding its arcs' entries among the running
// sums.  For rounds of more entries than waves, whose entries are mostly short:
// bound by the chain of dependent loads per entry, a wave taking them one by
// one ran 60 of 64 lanes idle (mesh 1024^2 with a hub of 80 arcs: 31.4 -> 10.1
// ms, the session's rounds 13.1; a random tree of a million vertices 1.68 ->
// 0.81, 1.26).  Two arcs per lane: four take the registers of two waves.
template <int WT>
__device__ __forceinline__ void push_entries(const OrderJob &J, gptr<uint32_t> dist,
                                             gptr<unsigned long long> next_bits, gptr<u32x2> next_queue,
                                             gptr<unsigned long long> region, u32x2 ent, bool has, uint32_t &lowest) {
    const int lane = threadIdx.x & 63;
    gptr<const int32_t> ro = to_global(J.ro);
    gptr<const u32x2> adj = reinterpret_cast<gptr<const u32x2>>(to_global(J.adj));
    int32_t e0 = 0, len = 0;
    uint32_t d = 0;
    if (has) {
        e0 = ro[ent.x] + (int32_t)ent.y * kPushRun;
        len = min(ro[ent.x + 1] - e0, kPushRun);
        d = ld_dev(dist + ent.x);
    }
    const int32_t upto = (int32_t)wave_scan((uint32_t)len);
    const int32_t all = __builtin_amdgcn_readlane(upto, 63);
    const int32_t first = e0 - (upto - len);  // its arc x of all is first + x
    for (int32_t x0 = 0; x0 < all; x0 += 64 * kPackArcs) {
        u32x2 a[kPackArcs];
        uint32_t du[kPackArcs];
        bool ok[kPackArcs];
#pragma unroll
        for (int k = 0; k < kPackArcs; ++k) {
            const int32_t x = min(x0 + k * 64 + lane, all - 1);
            int p = 0;  // entries that end at or before arc x
#pragma unroll
            for (int b = 32; b > 0; b >>= 1) p += __shfl(upto, p + b - 1, 64) <= x ? b : 0;
            a[k] = adj[__shfl(first, p, 64) + x];
            du[k] = (uint32_t)__shfl((int)d, p, 64);
            ok[k] = x0 + k * 64 + lane < all;
        }
        push_pass<WT, kPackArcs>(J, dist, next_bits, next_queue, region, a, du, ok, lowest);
    }
}

// A row's arcs [e, e1) in order of weight by G lanes, U x G of them: lowers low
// (the lanes' common best) and returns whether the arcs after them may lower it
// further.
template <int WT, int G, int U>
__device__ __forceinline__ bool pull_arcs(gptr<const u32x2> arc, gptr<const uint32_t> dist, uint32_t mu, int32_t e,
                                          int32_t e1, uint32_t &low, uint32_t &nread) {
    const int lane = threadIdx.x & 63, my = e + (lane & (G - 1));
    u32x2 a[U];
    bool in[U];
    uint32_t d[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = arc[min(my + u * G, e1 - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        in[u] = my + u * G < e1 && plus<WT>(mu, a[u].y) < low;
        if (in[u]) d[u] = dist[a[u].x];
    }
    uint32_t c = low;
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (in[u]) {
            ++nread;
            c = min(c, plus<WT>(d[u], a[u].y));
        }
    c = min(c, dpp<0xB1>(c));  // the lanes of the group are active together
    c = min(c, dpp<0x4E>(c));
    c = min(c, dpp<0x141>(c));
    if constexpr (G == 16) c = min(c, dpp<0x140>(c));
    low = c;
    return __ballot(in[U - 1] && plus<WT>(mu, a[U - 1].y) < low) >> ((lane & (64 - G)) + G - 1) & 1ull;
}

// AHEAD: the third weight and the row's bounds are loaded with the tails'
// distances, for every vertex whose second arc may help, instead of one after
// the other for those that go on: two trips less per round, against loads for
// nothing where few vertices go on (R-MAT 13 185 -> 191 us, 15 195 -> 199, 18
// 220 -> 225, 19 264 -> 266, 20 binary32 613 -> 586, 22 1058 -> 1020; uniform of
// half a million vertices 950 -> 885, of a million 1350 -> 1307).  How many go
// on is not known beforehand; the line lies where the R-MAT graphs, of which the
// fewest do, begin to gain.  Uniform graphs would from half a million on.
constexpr int32_t kOrderAhead = 3 << 18;  // vertices from which on

// WT: 0 uint32, 1 binary32, 2 unit steps.  Blocks [0, vblocks) of a pull take
// kOrderVerts vertices each, the others the long rows' chunks.
template <int WT, bool AHEAD>
__global__ __launch_bounds__(256, 8) void k_order(OrderArgs g) {
    const OrderJob &J = g.job[blockIdx.y];
    const int t = threadIdx.x, lane = t & 63;
    gptr<unsigned long long> ctl = to_global(J.ctl);
    const int32_t n = J.n;
    const int s0 = (int)(g.round % 3), s1 = (int)((g.round + 1) % 3), s2 = (int)((g.round + 2) % 3);
    constexpr int slot_words = kOrderRegions * kOrderRegionWords;
    const Totals T = read_slot(ctl + s0 * slot_words);
    const bool pulled = (T.flags & (uint32_t)kFlagPulled) != 0u;
    const bool pull = (T.flags & (uint32_t)kFlagOver) != 0u ||
                      (pulled ? kBackArcs * T.E + kBackFixed > (unsigned long long)n + kBackRead * T.read
                              : kOrderBias * (double)T.E * (double)T.E >= (double)n * (double)J.m);
    const bool keep = pull && pulled && (unsigned long long)T.F * kBackShare <= (unsigned long long)n &&
                      (unsigned long long)n + kBackRead * T.read >= kBackFixed;
    // the slot of the round after next
    if (blockIdx.x == 0)
        for (int i = t; i < slot_words; i += 256) ctl[s2 * slot_words + i] = 0ull;
    gptr<unsigned long long> region = ctl + s1 * slot_words + (blockIdx.x % kOrderRegions) * kOrderRegionWords;
    if (blockIdx.x == 0 && t == 0) {
        gptr<unsigned long long> state = ctl + kOrderState;
        for (int i = 0; i < kOrderRegions; ++i)
            state[kStPulledArcs] += ctl[s0 * slot_words + i * kOrderRegionWords + kRgRead];
        if (T.F == 0u) {
            if (state[kStDone] == 0ull) {
                state[kStDone] = 1ull;
                unsigned long long *st = g.stat + (size_t)blockIdx.y * kOrderStatWords;
                const unsigned long long v[kOrderStatWords] = {1ull, (unsigned long long)g.round, state[kStPulls],
                                                               state[kStF], state[kStPushed], state[kStPulledArcs]};
#pragma unroll
                for (int i = 1; i < kOrderStatWords; ++i)
                    __hip_atomic_store(st + i, v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                __hip_atomic_store(st, v[0], __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);  // (the host polls it)
            }
        } else {
            if (g.tag != 0ull)
                __hip_atomic_store(g.stat + (size_t)blockIdx.y * kOrderStatWords, g.tag, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_SYSTEM);
            state[kStF] += T.F;
            if (pull) {
                (void)__hip_atomic_fetch_or(region + kRgFlags, kFlagPulled | (keep ? 0ull : kFlagOver), __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
                state[kStPulls] += 1ull;
            } else {
                state[kStPushed] += T.E;
            }
        }
    }
    if (T.F == 0u) return;
    gptr<uint32_t> dist = to_global(J.dist);
    __shared__ uint32_t sLow, sCnt, sArcs, sRead;
    if (t == 0) {
        sLow = 0xFFFFFFFFu;
        sCnt = sArcs = sRead = 0u;
    }
    __syncthreads();  // (a block of chunks alone meets no other barrier before it adds to them)
    uint32_t lowest = 0xFFFFFFFFu, nread = 0, nnew = 0;
    const int32_t vblocks = (n + kOrderVerts - 1) / kOrderVerts;
    gptr<unsigned long long> bits = reinterpret_cast<gptr<unsigned long long>>(to_global(J.bits));
    gptr<u32x2> queue = reinterpret_cast<gptr<u32x2>>(to_global(J.queue));
    gptr<u32x2> to = queue + ((size_t)((g.round + 1) & 1) * kOrderRegions + blockIdx.x % kOrderRegions) * J.cap;
    if (!pulled)  // what a push marked of this frontier (pulls mark nothing)
        for (int32_t i = blockIdx.x * 256 + t; i < J.nword; i += gridDim.x * 256)
            bits[(size_t)(g.round & 1) * J.nword + i] = 0ull;
    if (!pull) {
        gptr<unsigned long long> next_bits = bits + (size_t)((g.round + 1) & 1) * J.nword;
        gptr<const u32x2> from = queue + (size_t)(g.round & 1) * kOrderRegions * J.cap;
        // entry i of the regions' lists laid end to end
        uint32_t mine = lane < kOrderRegions ? (uint32_t)ctl[s0 * slot_words + lane * kOrderRegionWords + kRgCnt] : 0u;
        const uint32_t upto = wave_scan(mine);
        const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
        const uint32_t waves = gridDim.x * 4u, wave = blockIdx.x * 4u + (uint32_t)(t >> 6);
        if (all <= waves) {
            if (wave < all) {
                const int rg = (int)__popcll(__ballot(upto <= wave));
                const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)upto, rg);
                const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)mine, rg);
                const u32x2 ent = from[(size_t)rg * J.cap + (wave - (end - cnt))];
                push_entry<WT>(J, dist, next_bits, to, region, ent, lowest);
            }
        } else {
            const uint32_t per = min((all + waves - 1) / waves, 64u);  // entries that a wave takes at once
            for (uint32_t i0 = wave * per; i0 < all; i0 += waves * per) {
                const uint32_t i = min(i0 + (uint32_t)lane, all - 1);
                uint32_t rg = 0, start = 0;
#pragma unroll
                for (int r = 0; r < kOrderRegions; ++r) {
                    const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)upto, r);
                    if (end <= i) {
                        rg = (uint32_t)r + 1u;
                        start = end;
                    }
                }
                const bool has = (uint32_t)lane < per && i0 + (uint32_t)lane < all;
                const u32x2 ent = from[(size_t)rg * J.cap + (i - start)];
                push_entries<WT>(J, dist, next_bits, to, region, ent, has, lowest);
            }
        }
        __syncthreads();
    } else {
        gptr<const u32x2> arc = reinterpret_cast<gptr<const u32x2>>(to_global(J.arc));
        const uint32_t mu = T.mu;
        const auto step = [](uint32_t d, uint32_t w) { return plus<WT>(d, w); };
        __shared__ uint32_t sList[kOrderVerts], sWas[kOrderVerts], sBest[kOrderVerts];
        __shared__ int2 sRow[AHEAD ? kOrderVerts : 1];
        // keep: the vertices that a pass improved, a bit each, for the queue
        __shared__ uint32_t sWon[kOrderVerts / 32];
        for (int32_t vb = blockIdx.x; vb < vblocks; vb += gridDim.x) {
            if (t == 0) sCnt = 0u;
            __syncthreads();
            // the two lightest arcs: every load of a vertex is issued at once,
            // then the tails' distances
            constexpr int V = kOrderVerts / 256;
            uint32_t b[V], best[V], d0[V], d1[V], w2[V];
            int32_t r0[V], r1[V];
            u32x2 a0[V], a1[V];
            bool in0[V], in1[V];
#pragma unroll
            for (int k = 0; k < V; ++k) {
                const int32_t v = min(vb * kOrderVerts + k * 256 + t, n - 1);
                b[k] = dist[v];
                a0[k] = reinterpret_cast<gptr<const u32x2>>(to_global(J.a0))[v];
                a1[k] = reinterpret_cast<gptr<const u32x2>>(to_global(J.a1))[v];
            }
#pragma unroll
            for (int k = 0; k < V; ++k) {
                const bool ok = vb * kOrderVerts + k * 256 + t < n;
                // (absent arcs: weight INF, and no tail)
                in0[k] = ok && a0[k].x != kOrderNone && step(mu, a0[k].y) < b[k];
                in1[k] = in0[k] && a1[k].x != kOrderNone && step(mu, a1[k].y) < b[k];
                if (in0[k]) d0[k] = dist[a0[k].x];
                if (in1[k]) d1[k] = dist[a1[k].x];
                if constexpr (AHEAD) {
                    const int32_t v = vb * kOrderVerts + k * 256 + t;
                    if (in1[k]) {
                        w2[k] = to_global(J.w2)[v];
                        r0[k] = to_global(J.ro_in)[v];
                        r1[k] = to_global(J.ro_in)[v + 1];
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < V; ++k) {
                nread += (in0[k] ? 1u : 0u) + (in1[k] ? 1u : 0u);
                best[k] = b[k];
                if (in0[k]) best[k] = min(best[k], step(d0[k], a0[k].y));
                if (in1[k]) best[k] = min(best[k], step(d1[k], a1[k].y));
                // the others, below, for the vertices they may still improve
                bool row = in1[k] && step(mu, a1[k].y) < best[k];
                const int i = k * 256 + t;
                const int32_t v = vb * kOrderVerts + i;
                if constexpr (AHEAD) row = row && step(mu, w2[k]) < best[k];
                else if (row) row = step(mu, to_global(J.w2)[v]) < best[k];
                const unsigned long long m = __ballot(row);
                if (m != 0ull) {
                    uint32_t at = 0;
                    if (lane == 0) at = atomicAdd(&sCnt, (uint32_t)__popcll(m));
                    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                    if (row) {
                        sList[at] = (uint32_t)i;
                        sWas[at] = b[k];
                        sBest[at] = best[k];
                        if constexpr (AHEAD) sRow[at] = make_int2(r0[k], r1[k]);
                    }
                }
                const bool won = !row && best[k] < b[k];
                if (won) {
                    dist[v] = best[k];
                    lowest = min(lowest, best[k]);
                    ++nnew;
                }
                if (keep) {
                    const unsigned long long w = __ballot(won);
                    if ((lane & 31) == 0) sWon[(k * 256 + t) / 32] = (uint32_t)(w >> lane);
                }
            }
            __syncthreads();
            // eight lanes per vertex: a line of eight arcs, then several at a time
            const uint32_t cnt = sCnt;
            gptr<const int32_t> ro = to_global(J.ro_in);
            for (uint32_t k = (uint32_t)t >> 3; k < cnt; k += 32u) {
                const int32_t v = vb * kOrderVerts + (int32_t)sList[k];
                uint32_t low = sBest[k];
                int32_t e0, e1;
                if constexpr (AHEAD) {
                    e0 = sRow[k].x + 2;
                    e1 = sRow[k].y;
                } else {
                    e0 = ro[v] + 2;
                    e1 = ro[v + 1];
                }
                bool more = e0 < e1 && pull_arcs<WT, 8, 1>(arc, dist, mu, e0, e1, low, nread);
                for (int32_t e = e0 + 8; more && e < e1; e += 8 * kPullWide)
                    more = pull_arcs<WT, 8, kPullWide>(arc, dist, mu, e, e1, low, nread);
                // (only this block writes dist[v])
                if ((t & 7) == 0 && low < sWas[k]) {
                    dist[v] = low;
                    lowest = min(lowest, low);
                    ++nnew;
                    if (keep) atomicOr(&sWon[sList[k] / 32], 1u << (sList[k] % 32));
                }
            }
            __syncthreads();
            if (keep) {
                uint32_t v[V];
                bool on[V];
#pragma unroll
                for (int k = 0; k < V; ++k) {
                    v[k] = (uint32_t)(vb * kOrderVerts + k * 256 + t);
                    on[k] = sWon[(k * 256 + t) / 32] >> (t % 32) & 1u;
                }
                enqueue<V, kPushRun>(to_global(J.ro), J.cap, region, to, v, on, false);
            }
        }
        if (keep) {  // (now of the vertices that chunks improve, some of them several times)
            if (t == 0) sCnt = 0u;
            __syncthreads();
        }
        // long rows: 16 lanes per chunk
        const int32_t cfirst = ((int32_t)gridDim.x > vblocks ? (int32_t)blockIdx.x - vblocks : (int32_t)blockIdx.x);
        const int32_t cstep = ((int32_t)gridDim.x > vblocks ? (int32_t)gridDim.x - vblocks : (int32_t)gridDim.x) * 16;
        for (int32_t c = cfirst * 16 + (t >> 4); cfirst >= 0 && c < J.nchunks; c += cstep) {
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const u32x4 ch = reinterpret_cast<gptr<const u32x4>>(to_global(J.chunk))[c];
            const uint32_t b0 = ld_dev(dist + ch.x);
            uint32_t low = b0;
            if (!(step(mu, ch.w) < low)) continue;  // its lightest arc
            const int32_t e0 = (int32_t)ch.y, e1 = (int32_t)ch.z;
            bool more = pull_arcs<WT, 16, 1>(arc, dist, mu, e0, e1, low, nread);
            for (int32_t e = e0 + 16; more && e < e1; e += 16 * kPullWide)
                more = pull_arcs<WT, 16, kPullWide>(arc, dist, mu, e, e1, low, nread);
            if ((t & 15) == 0 && low < b0 &&
                low < __hip_atomic_fetch_min(dist + ch.x, low, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                lowest = min(lowest, low);
                ++nnew;
                if (keep) {
                    const uint32_t at = atomicAdd(&sCnt, 1u);
                    if (at < (uint32_t)kOrderVerts) sList[at] = ch.x;
                }
            }
        }
        if (keep) {
            __syncthreads();
            const uint32_t cnt = min(sCnt, (uint32_t)kOrderVerts);
            if (t == 0 && cnt < sCnt)
                (void)__hip_atomic_fetch_or(region + kRgFlags, kFlagOver, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (uint32_t i = (uint32_t)t; __ballot(i < cnt) != 0ull; i += 256u) {
                const bool on[1] = {i < cnt};
                const uint32_t v[1] = {on[0] ? sList[i] : 0u};
                enqueue<1, kPushRun>(to_global(J.ro), J.cap, region, to, v, on, false);
            }
        }
    }
    if (lowest != 0xFFFFFFFFu) atomicMin(&sLow, lowest);
    if (nnew) atomicAdd(&sArcs, nnew);
    if (nread) atomicAdd(&sRead, nread);
    __syncthreads();
    if (t == 0) {
        if (sLow != 0xFFFFFFFFu)
            (void)__hip_atomic_fetch_max(region + kRgMu, (unsigned long long)(uint32_t)~sLow, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
        if (sArcs)
            (void)__hip_atomic_fetch_add(region + kRgF, (unsigned long long)sArcs, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
        if (sRead)
            (void)__hip_atomic_fetch_add(region + kRgRead, (unsigned long long)sRead, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ---- batched queries -----------------------------------------------------------

// The same rounds for up to 64 sources of one graph, a source per lane and the
// distances vertex-major, so that an arc costs one 256-byte row: a pull reads a
// vertex's arcs while they can still improve any of its lanes.  Bound by those
// rows (64 sources on R-MAT 22: 2.2 GB per launch of 505 us, 4.4 TB/s; 69% of
// the L2s' requests miss) and where these stay in the caches by the instructions
// per arc, hence scalar loads of the graph, a saturating add and one comparison
// per arc, and rows read through a scalar base.  A pull doesn't ask whether a tail is on the frontier: the
// row's newer distances help the lanes along, 17 M arcs read instead of 38 M.
// 64 sources on a scale-20 R-MAT graph of 31 M arcs: 1.90 ms, of which 0.16
// transposes the output (the queue-driven push rounds of the session kernels
// took 10.8 ms); 0.65 ms at scale 15 (1.42).
struct OrderBatchArgs {
    OrderBatch b;
    int64_t round;
    unsigned long long *stat;
    unsigned long long tag;  // as in OrderArgs
};
constexpr int kRgPairs = 6;   // region: (arc, source) pairs of the frontier
constexpr int kStPairs = 6;   // state: their total
constexpr int kBatchVerts = 4;   // vertices in flight per wave
constexpr int kBatchArcs = 4;   // arcs of a row in flight (2000 us for the 64 queries below, 2066 with 8)
constexpr int kBatchRun = 64;   // arcs per queue entry
constexpr int kBatchKeep = 512;  // vertices that a block of a pull can put on the queue
// Pushes again as above, where a pull costs a row per vertex: when kBatchBack E
// <= n + R (1, 4 and 16 measure the same).  16 sources: two R-MAT 17 graphs
// joined by a path of 300 135 -> 10 ms (the session kernels 11.7), R-MAT 14
// and a path of 1,000 202 -> 13.0 (23.4), R-MAT 20 with a tail of 3,000 200 ->
// 47 (74); R-MAT 20 1.60 -> 1.52.
constexpr unsigned long long kBatchBack = 4;
static_assert(kBatchRun <= kOrderRun && kBatchArcs <= kOrderRun, "steps past a row's end");

struct BatchBeginArgs {
    OrderBatch b;
    int32_t src[kBatchLanes];
};

// (lanes without a source hold 0: nothing improves them)
__global__ __launch_bounds__(256) void k_order_batch_clear(OrderBatch b, uint32_t inf) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;  // (a multiple of 16)
    const int l = (int)(t % (kBatchLanes / 4)) * 4;
    const int k = b.k;
    const u32x4 x = u32x4{l < k ? inf : 0u, l + 1 < k ? inf : 0u, l + 2 < k ? inf : 0u, l + 3 < k ? inf : 0u};
    for (int64_t i = t; i < (int64_t)b.g.n * (kBatchLanes / 4); i += step) reinterpret_cast<u32x4 *>(b.D)[i] = x;
    for (int64_t i = t; i < 3 * (int64_t)b.g.n; i += step) b.mask[i] = 0ull;
    for (int64_t i = t; i < 3 * kOrderRegions * 64; i += step) b.mu[i] = 0u;
    for (int64_t i = t; i < kOrderCtlWords; i += step) b.g.ctl[i] = 0ull;
}

// One wave, a source per lane (repeated sources share an entry).
__global__ __launch_bounds__(64) void k_order_batch_begin(BatchBeginArgs a) {
    const int lane = threadIdx.x;
    unsigned long long *ctl = a.b.g.ctl;
    const bool mine = lane < a.b.k;
    const int32_t s = a.src[mine ? lane : 0];
    const int32_t deg = a.b.g.ro[s + 1] - a.b.g.ro[s];
    bool first = mine && deg > 0;
    for (int j = 0; j < a.b.k; ++j) first = first && !(j < lane && a.src[j] == s);
    const uint32_t runs = first ? (uint32_t)((deg + kBatchRun - 1) / kBatchRun) : 0u;
    uint32_t upto = runs;
    unsigned long long E = first ? (unsigned long long)deg : 0ull, pairs = mine ? (unsigned long long)deg : 0ull;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = (uint32_t)__shfl_up((int)upto, o, 64);
        if (lane >= o) upto += x;
        E += __shfl_xor(E, o, 64);
        pairs += __shfl_xor(pairs, o, 64);
    }
    const uint32_t all = (uint32_t)__shfl((int)upto, 63, 64);
    const int F = (int)__popcll(__ballot(first));
    const bool fits = all <= (uint32_t)a.b.g.cap;
    if (mine) {
        a.b.D[(size_t)s * kBatchLanes + lane] = 0u;
        atomicOr(a.b.mask + s, 1ull << lane);
        a.b.mu[lane] = 0xFFFFFFFFu;
    }
    if (fits)
        for (uint32_t i0 = 0; i0 < all; i0 += 64) {
            const uint32_t i = i0 + lane;
            int j = 0;  // the source whose run i is
            for (int k = 0; k + 1 < a.b.k; ++k) j += (uint32_t)__shfl((int)upto, k, 64) <= i ? 1 : 0;
            const uint32_t before = (uint32_t)__shfl((int)(upto - runs), j, 64);
            if (i < all) a.b.g.queue[i] = make_uint2((uint32_t)a.src[j], i - before);
        }
    if (lane == 0) {
        ctl[kRgF] = (unsigned long long)F;
        ctl[kRgE] = E;
        ctl[kRgCnt] = fits ? all : 0ull;
        ctl[kRgFlags] = kFlagMarked | (fits ? 0ull : kFlagOver);
        ctl[kRgPairs] = pairs;
    }
}

template <typename T>
using cptr = const T __attribute__((address_space(4))) *;  // read-only: uniform loads are scalar ones
template <typename T>
__device__ __forceinline__ cptr<T> to_constant(const T *p) {
    return (cptr<T>)p;
}
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t arcs_vec __attribute__((ext_vector_type(2 * kBatchArcs), aligned(8)));

// d (+) w in one or two instructions (INF, the largest value, stays).
template <int WT>
__device__ __forceinline__ uint32_t plus_sat(uint32_t d, uint32_t w) {
    if constexpr (WT == 0) return __builtin_elementwise_add_sat(d, w);
    else return __float_as_uint(fminf(__uint_as_float(d) + __uint_as_float(w), __uint_as_float(kInfF32)));
}
// mu (+) w < best, for room = room_of(mu, best): one comparison for uint32.
template <int WT>
__device__ __forceinline__ uint32_t room_of(uint32_t mu, uint32_t best) {
    if constexpr (WT == 0) return __builtin_elementwise_sub_sat(best, mu);
    else return best;
}
template <int WT>
__device__ __forceinline__ bool in_room(uint32_t mu, uint32_t w, uint32_t room) {
    if constexpr (WT == 0) return w < room;
    else return __uint_as_float(mu) + __uint_as_float(w) < __uint_as_float(room);
}

template <int WT>
__global__ __launch_bounds__(256, 8) void k_order_batch(OrderBatchArgs g) {
    const OrderJob &J = g.b.g;
    const int t = threadIdx.x, lane = t & 63;
    gptr<unsigned long long> ctl = to_global(J.ctl);
    const int32_t n = J.n;
    const int s0 = (int)(g.round % 3), s1 = (int)((g.round + 1) % 3), s2 = (int)((g.round + 2) % 3);
    constexpr int slot_words = kOrderRegions * kOrderRegionWords;
    const Totals T = read_slot(ctl + s0 * slot_words);
    const bool pulled = (T.flags & (uint32_t)kFlagPulled) != 0u;
    const bool pull = (T.flags & (uint32_t)kFlagOver) != 0u ||
                      (pulled ? kBatchBack * T.E > (unsigned long long)n + T.read
                              : kOrderBias * (double)T.E * (double)T.E >= (double)n * (double)J.m);
    const bool keep = pull && pulled && (unsigned long long)T.F * kBackShare <= (unsigned long long)n;
    gptr<uint32_t> mus = to_global(g.b.mu);
    if (blockIdx.x == 0) {
        for (int i = t; i < slot_words; i += 256) ctl[s2 * slot_words + i] = 0ull;
        for (int i = t; i < kOrderRegions * 64; i += 256) mus[s2 * kOrderRegions * 64 + i] = 0u;
    }
    const int rg = (int)(blockIdx.x % kOrderRegions);
    gptr<unsigned long long> region = ctl + s1 * slot_words + rg * kOrderRegionWords;
    if (blockIdx.x == 0 && t == 0) {
        gptr<unsigned long long> state = ctl + kOrderState;
        for (int i = 0; i < kOrderRegions; ++i) {
            state[kStPulledArcs] += ctl[s0 * slot_words + i * kOrderRegionWords + kRgRead];
            state[kStPairs] += ctl[s0 * slot_words + i * kOrderRegionWords + kRgPairs];
        }
        if (T.F == 0u) {
            if (state[kStDone] == 0ull) {
                state[kStDone] = 1ull;
                const unsigned long long v[kOrderBatchStatWords] = {1ull, (unsigned long long)g.round, state[kStPulls],
                                                                    state[kStF], state[kStPushed] + state[kStPulledArcs],
                                                                    state[kStPairs]};
#pragma unroll
                for (int i = 1; i < kOrderBatchStatWords; ++i)
                    __hip_atomic_store(g.stat + i, v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                __hip_atomic_store(g.stat, v[0], __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);  // (the host polls it)
            }
        } else {
            if (g.tag != 0ull) __hip_atomic_store(g.stat, g.tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            state[kStF] += T.F;
            if (pull) {
                state[kStPulls] += 1ull;
            } else {
                state[kStPushed] += T.E;
            }
            (void)__hip_atomic_fetch_or(region + kRgFlags,
                                        (pull ? kFlagPulled : 0ull) | (pull && !keep ? kFlagOver : kFlagMarked) |
                                            (T.flags & kFlagMarked ? kFlagWasMarked : 0ull),
                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (T.F == 0u) return;
    gptr<unsigned long long> mask = to_global(g.b.mask);
    gptr<const unsigned long long> on = mask + (size_t)s0 * n;
    gptr<unsigned long long> next = mask + (size_t)s1 * n;
    gptr<uint32_t> D = to_global(g.b.D);
    gptr<const int32_t> ro = to_global(J.ro);
    __shared__ uint32_t sLow[kBatchLanes];
    __shared__ uint32_t sNew, sRead, sKept;
    __shared__ uint32_t sKeep[kBatchKeep];  // keep: the vertices that the block improved
    __shared__ unsigned long long sPairs;
    if (t < kBatchLanes) sLow[t] = 0u;
    if (t == 0) {
        sNew = sRead = sKept = 0u;
        sPairs = 0ull;
    }
    __syncthreads();
    uint32_t low = 0u;             // complement of this lane's smallest improvement
    uint32_t nnew = 0, nread = 0;  // by wave, uniform
    unsigned long long pairs = 0;
    const auto row = [&](uint32_t v) { return D + (size_t)v * kBatchLanes + lane; };
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4u + (uint32_t)(t >> 6)));
    const uint32_t waves = gridDim.x * 4u;
    // the next round's next masks: what marked the frontier before
    if (T.flags & kFlagWasMarked)
        for (int64_t i = (int64_t)blockIdx.x * 256 + t; i < n; i += (int64_t)gridDim.x * 256)
            mask[(size_t)s2 * n + i] = 0ull;
    gptr<u32x2> queue = reinterpret_cast<gptr<u32x2>>(to_global(J.queue));
    gptr<u32x2> to = queue + ((size_t)((g.round + 1) & 1) * kOrderRegions + rg) * J.cap;
    if (!pull) {
        gptr<const u32x2> from = queue + (size_t)(g.round & 1) * kOrderRegions * J.cap;
        gptr<const u32x2> adj = reinterpret_cast<gptr<const u32x2>>(to_global(J.adj));
        uint32_t mine = lane < kOrderRegions ? (uint32_t)ctl[s0 * slot_words + lane * kOrderRegionWords + kRgCnt] : 0u;
        uint32_t upto = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t x = (uint32_t)__shfl_up((int)upto, o, 64);
            if (lane >= o) upto += x;
        }
        const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
        for (uint32_t i = wave; i < all; i += waves) {
            const int q = (int)__popcll(__ballot(upto <= i));
            const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)upto, q);
            const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)mine, q);
            u32x2 ent = from[(size_t)q * J.cap + (i - (end - cnt))];
            ent.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)ent.x);
            ent.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)ent.y);
            // (a lane whose frontier has no such vertex: INF improves nothing)
            const uint32_t du = on[ent.x] >> lane & 1ull
                                    ? __hip_atomic_load(row(ent.x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                    : (WT == 1 ? kInfF32 : kInfU32);
            const int32_t e0 = ro[ent.x] + (int32_t)ent.y * kBatchRun, e1 = min(ro[ent.x + 1], e0 + kBatchRun);
            const u32x2 a = adj[min(e0 + lane, e1 - 1)];
            const int deg1 = __builtin_amdgcn_readfirstlane(e1 - e0);
            unsigned long long won = 0ull;  // the lanes that this lane's arc improved
            for (int j = 0; j < deg1; j += kBatchArcs) {
                uint32_t nd[kBatchArcs], cur[kBatchArcs];
#pragma unroll
                for (int k = 0; k < kBatchArcs; ++k) {
                    const int at = min(j + k, deg1 - 1);
                    nd[k] = plus_sat<WT>(du, (uint32_t)__builtin_amdgcn_readlane((int)a.y, at));
                    cur[k] = *row((uint32_t)__builtin_amdgcn_readlane((int)a.x, at));
                }
#pragma unroll
                for (int k = 0; k < kBatchArcs; ++k) {
                    // (another wave may be lower by now: then the vertex is on the frontier with its value)
                    const bool win = nd[k] < cur[k];
                    const unsigned long long b = __ballot(win);
                    if (b == 0ull) continue;
                    const int at = min(j + k, deg1 - 1);
                    if (win) {
                        (void)__hip_atomic_fetch_min(row((uint32_t)__builtin_amdgcn_readlane((int)a.x, at)), nd[k],
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        low = max(low, ~nd[k]);
                    }
                    if (lane == at) won |= b;
                }
            }
            // (the lane holding the arc marks its head)
            uint32_t runs = 0, deg = 0;
            if (won != 0ull) {
                const unsigned long long was =
                    __hip_atomic_fetch_or(next + a.x, won, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                deg = (uint32_t)(ro[a.x + 1] - ro[a.x]);
                pairs += (unsigned long long)__popcll(won & ~was) * deg;
                if (was == 0ull) runs = (deg + kBatchRun - 1) / kBatchRun;
            }
            const unsigned long long fresh = __ballot(runs != 0u);
            if (fresh == 0ull) continue;
            uint32_t before = runs;
            unsigned long long sum = runs ? deg : 0u;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t x = (uint32_t)__shfl_up((int)before, o, 64);
                if (lane >= o) before += x;
                sum += __shfl_xor(sum, o, 64);
            }
            const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)before, 63);
            unsigned long long base = 0;
            if (lane == 0) {
                base = __hip_atomic_fetch_add(region + kRgCnt, (unsigned long long)total, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
                (void)__hip_atomic_fetch_add(region + kRgE, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            nnew += (uint32_t)__popcll(fresh);
            base = (unsigned long long)__shfl((long long)base, 0, 64);
            if (base + total > (unsigned long long)J.cap) {  // the next round pulls
                if (lane == 0)
                    (void)__hip_atomic_fetch_or(region + kRgFlags, kFlagOver, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                continue;
            }
            const uint32_t at = (uint32_t)base + before - runs;
            for (uint32_t r = 0; r < runs; ++r) to[at + r] = u32x2{a.x, r};
        }
    } else {
        cptr<int32_t> ri = to_constant(J.ro_in), rc = to_constant(J.ro);
        cptr<uint2> arc = to_constant(J.arc);
        uint32_t mu = 0u;
#pragma unroll
        for (int i = 0; i < kOrderRegions; ++i) mu = max(mu, mus[(s0 * kOrderRegions + i) * 64 + lane]);
        // (INF for a lane whose frontier is empty: its arcs are all ruled out)
        mu = min(~mu, WT == 1 ? kInfF32 : kInfU32);
        // a vertex that the lanes w improved (one: by this wave alone) and that goes to the queue
        const auto kept = [&](uint32_t v, unsigned long long w, bool one) {
            if (lane != 0) return;
            if (one) next[v] = w;
            else if (__hip_atomic_fetch_or(next + v, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0ull) return;
            const uint32_t at = atomicAdd(&sKept, 1u);
            if (at < (uint32_t)kBatchKeep) sKeep[at] = v;
        };
        // the arcs [e, e1) of a row, in order of weight, against the lanes' best
        const auto walk = [&](int32_t e, int32_t e1, uint32_t &best) {
            for (; e < e1; e += kBatchArcs) {
                const arcs_vec a = *(cptr<arcs_vec>)(arc + e);  // (past the last row: the table after the arcs)
                const uint32_t room = room_of<WT>(mu, best);
                uint32_t d[kBatchArcs];
                bool in[kBatchArcs];
#pragma unroll
                for (int k = 0; k < kBatchArcs; ++k) {
                    in[k] = e + k < e1 && __ballot(in_room<WT>(mu, a[2 * k + 1], room)) != 0ull;
                    if (in[k]) d[k] = *row(a[2 * k]);
                }
#pragma unroll
                for (int k = 0; k < kBatchArcs; ++k)
                    if (in[k]) {
                        best = min(best, plus_sat<WT>(d[k], a[2 * k + 1]));
                        ++nread;
                    }
                if (!in[kBatchArcs - 1]) return;  // out for every lane: so are those after it
            }
        };
        for (uint32_t v0 = wave * kBatchVerts; v0 < (uint32_t)n; v0 += waves * kBatchVerts) {
            const u32x8 a0 = *(cptr<u32x8>)(to_constant(J.a0) + v0), a1 = *(cptr<u32x8>)(to_constant(J.a1) + v0);
            const u32x4 w2 = *(cptr<u32x4>)(to_constant(J.w2) + v0);
            uint32_t b[kBatchVerts], best[kBatchVerts], d0[kBatchVerts], d1[kBatchVerts];
            bool has[kBatchVerts], in0[kBatchVerts], in1[kBatchVerts];
#pragma unroll
            for (int k = 0; k < kBatchVerts; ++k) {
                has[k] = v0 + k < (uint32_t)n && a0[2 * k] != kOrderNone;
                if (has[k]) b[k] = *row(v0 + k);
            }
#pragma unroll
            for (int k = 0; k < kBatchVerts; ++k) {
                in0[k] = in1[k] = false;
                if (has[k]) {
                    const uint32_t room = room_of<WT>(mu, b[k]);
                    in0[k] = __ballot(in_room<WT>(mu, a0[2 * k + 1], room)) != 0ull;
                    in1[k] = in0[k] && a1[2 * k] != kOrderNone && __ballot(in_room<WT>(mu, a1[2 * k + 1], room)) != 0ull;
                }
                if (in0[k]) d0[k] = *row(a0[2 * k]);
                if (in1[k]) d1[k] = *row(a1[2 * k]);
            }
#pragma unroll
            for (int k = 0; k < kBatchVerts; ++k) {
                if (!in0[k]) continue;
                ++nread;
                best[k] = min(b[k], plus_sat<WT>(d0[k], a0[2 * k + 1]));
                if (in1[k]) {
                    ++nread;
                    best[k] = min(best[k], plus_sat<WT>(d1[k], a1[2 * k + 1]));
                    if (__ballot(in_room<WT>(mu, w2[k], room_of<WT>(mu, best[k]))) != 0ull)
                        walk(ri[v0 + k] + 2, ri[v0 + k + 1], best[k]);
                }
                const bool won = best[k] < b[k];
                const unsigned long long w = __ballot(won);
                if (w == 0ull) continue;
                if (won) {
                    *row(v0 + k) = best[k];
                    low = max(low, ~best[k]);
                }
                const unsigned long long x = (unsigned long long)__popcll(w) * (uint32_t)(rc[v0 + k + 1] - rc[v0 + k]);
                pairs += lane == 0 ? x : 0ull;
                ++nnew;
                if (keep) kept(v0 + k, w, true);
            }
        }
        // long rows: a wave per chunk
        for (uint32_t c = wave; c < (uint32_t)J.nchunks; c += waves) {
            const u32x4 ch = *(cptr<u32x4>)(to_constant(J.chunk) + c);
            const uint32_t b = __hip_atomic_load(row(ch.x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            uint32_t best = b;
            walk((int32_t)ch.y, (int32_t)ch.z, best);
            bool won = best < b;
            if (won)
                won = best < __hip_atomic_fetch_min(row(ch.x), best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long w = __ballot(won);
            if (w == 0ull) continue;
            if (won) low = max(low, ~best);
            const unsigned long long x = (unsigned long long)__popcll(w) * (uint32_t)(rc[ch.x + 1] - rc[ch.x]);
            pairs += lane == 0 ? x : 0ull;
            ++nnew;
            if (keep) kept(ch.x, w, false);
        }
        if (keep) {
            __syncthreads();
            const uint32_t cnt = min(sKept, (uint32_t)kBatchKeep);
            if (t == 0 && cnt < sKept)
                (void)__hip_atomic_fetch_or(region + kRgFlags, kFlagOver, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (uint32_t i = (uint32_t)t; __ballot(i < cnt) != 0ull; i += 256u) {
                const bool on[1] = {i < cnt};
                const uint32_t v[1] = {on[0] ? sKeep[i] : 0u};
                enqueue<1, kBatchRun>(ro, J.cap, region, to, v, on, false);
            }
        }
    }
    if (low != 0u) atomicMax(&sLow[lane], low);
    if (lane == 0 && nnew) atomicAdd(&sNew, nnew);
    if (lane == 0 && nread) atomicAdd(&sRead, nread);
    if (pairs) atomicAdd(&sPairs, pairs);
    __syncthreads();
    if (t < kBatchLanes && sLow[t] != 0u)
        (void)__hip_atomic_fetch_max(mus + (s1 * kOrderRegions + rg) * 64 + t, sLow[t], __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
    if (t == 0) {
        if (sNew) (void)__hip_atomic_fetch_add(region + kRgF, (unsigned long long)sNew, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (sRead) (void)__hip_atomic_fetch_add(region + kRgRead, (unsigned long long)sRead, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (sPairs) (void)__hip_atomic_fetch_add(region + kRgPairs, sPairs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ---- layout ------------------------------------------------------------------

// Rows of up to 64 arcs: a wave each, sorted across its lanes.
__device__ __forceinline__ unsigned long long wave_sort(unsigned long long key) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 2; k <= 64; k <<= 1)
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
            const unsigned long long other = __shfl_xor(key, j, 64);
            const bool keep_low = ((lane & j) == 0) == ((lane & k) == 0);
            key = (key < other) == keep_low ? key : other;
        }
    return key;
}

__device__ __forceinline__ uint2 key_arc(unsigned long long k) { return make_uint2((uint32_t)k, (uint32_t)(k >> 32)); }

__device__ __forceinline__ void order_lightest(int32_t v, int32_t deg, unsigned long long k0, unsigned long long k1,
                                               unsigned long long k2, uint32_t inf, uint2 *a0, uint2 *a1, uint32_t *w2) {
    const bool own = deg <= kOrderChunk;  // long rows go by chunks
    a0[v] = own && deg > 0 ? key_arc(k0) : make_uint2(kOrderNone, inf);
    a1[v] = own && deg > 1 ? key_arc(k1) : make_uint2(kOrderNone, inf);
    w2[v] = own && deg > 2 ? (uint32_t)(k2 >> 32) : inf;
}

__global__ __launch_bounds__(256) void k_order_short(int32_t n, const int32_t *ro, const uint2 *adj, uint2 *arc,
                                                     uint32_t inf, uint2 *a0, uint2 *a1, uint32_t *w2) {
    const int lane = threadIdx.x & 63;
    for (int64_t v = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); v < n; v += (int64_t)gridDim.x * 4) {
        const int32_t e0 = ro[v], deg = ro[v + 1] - e0;
        if (deg > 64) continue;
        unsigned long long key = ~0ull;
        if (lane < deg) {
            const uint2 a = adj[e0 + lane];
            key = (unsigned long long)a.y << 32 | a.x;
        }
        if (deg > 1) key = wave_sort(key);
        if (lane < deg) arc[e0 + lane] = key_arc(key);
        const unsigned long long k0 = __shfl(key, 0, 64), k1 = __shfl(key, 1, 64), k2 = __shfl(key, 2, 64);
        if (lane == 0) order_lightest((int32_t)v, deg, k0, k1, k2, inf, a0, a1, w2);
    }
}

// Longer rows: a block per run of up to kOrderChunk arcs, sorted in LDS.  runs:
// (vertex, first arc, its entry in chunk or kOrderNone).
__global__ __launch_bounds__(256) void k_order_long(const uint4 *runs, const int32_t *ro, const uint2 *adj, uint2 *arc,
                                                    uint32_t inf, uint2 *a0, uint2 *a1, uint32_t *w2, uint4 *chunk) {
    __shared__ unsigned long long key[kOrderChunk];
    const int t = threadIdx.x;
    const uint4 r = runs[blockIdx.x];
    const int32_t v = (int32_t)r.x, e0 = (int32_t)r.y, deg = ro[v + 1] - ro[v], n = min(ro[v + 1] - e0, kOrderChunk);
    int size = 128;
    while (size < n) size <<= 1;
    for (int i = t; i < size; i += 256) {
        unsigned long long k = ~0ull;
        if (i < n) {
            const uint2 a = adj[e0 + i];
            k = (unsigned long long)a.y << 32 | a.x;
        }
        key[i] = k;
    }
    for (int k = 2; k <= size; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            __syncthreads();
            for (int i = t; i < size / 2; i += 256) {
                const int a = 2 * i - (i & (j - 1)), b = a + j;
                const unsigned long long x = key[a], y = key[b];
                if ((x > y) == ((a & k) == 0)) {
                    key[a] = y;
                    key[b] = x;
                }
            }
        }
    __syncthreads();
    for (int i = t; i < n; i += 256) arc[e0 + i] = key_arc(key[i]);
    if (t == 0 && e0 == ro[v]) order_lightest(v, deg, key[0], key[1], key[2], inf, a0, a1, w2);
    if (t == 0 && r.z != kOrderNone) chunk[r.z] = make_uint4(r.x, r.y, (uint32_t)(e0 + n), (uint32_t)(key[0] >> 32));
}

inline size_t al256(size_t x) { return (x + 255) & ~size_t(255); }
inline int32_t bit_words(int32_t n) { return (int32_t)(((int64_t)n + kOrderVerts - 1) / kOrderVerts * (kOrderVerts / 64)); }
inline int32_t queue_cap(int32_t n) { return std::clamp(n / 64, 1024, 65536); }

}  // namespace

hipError_t order_build(OrderSet *out, int32_t n, int32_t m, const int32_t *ro_in, const uint2 *adj_in,
                       const int32_t *h_ro_in, int wt, size_t limit, hipStream_t st) {
    *out = OrderSet{};
    std::vector<uint4> runs;
    uint32_t nchunks = 0;
    for (int32_t v = 0; v < n; ++v) {
        const int32_t d = h_ro_in[v + 1] - h_ro_in[v];
        if (d <= 64) continue;
        for (int32_t e = h_ro_in[v]; e < h_ro_in[v + 1]; e += kOrderChunk) {
            runs.push_back(make_uint4((uint32_t)v, (uint32_t)e, d > kOrderChunk ? nchunks++ : kOrderNone, 0u));
            if (h_ro_in[v + 1] - e <= kOrderChunk) break;  // (e + kOrderChunk may pass 2^31)
        }
    }
    const size_t bn = al256(sizeof(uint32_t) * (size_t)n), bm = al256(sizeof(uint2) * (size_t)std::max(m, 1)),
                 bc = al256(sizeof(uint4) * std::max<size_t>(nchunks, 1)), b2 = al256(sizeof(uint2) * (size_t)n);
    OrderSet s;
    s.bytes = bm + bn + 2 * b2 + bc;
    if (s.bytes > limit) return hipErrorOutOfMemory;
    hipError_t e = hipMalloc(&s.base, s.bytes);
    if (e != hipSuccess) return e;
    char *p = static_cast<char *>(s.base);
    s.arc = reinterpret_cast<uint2 *>(p);
    p += bm;
    s.a0 = reinterpret_cast<uint2 *>(p);
    p += b2;
    s.a1 = reinterpret_cast<uint2 *>(p);
    p += b2;
    s.w2 = reinterpret_cast<uint32_t *>(p);
    p += bn;
    s.chunk = reinterpret_cast<uint4 *>(p);
    s.nchunks = (int32_t)nchunks;
    void *d_runs = nullptr;
    const uint32_t inf = wt == 1 ? kInfF32 : kInfU32;
    if (!runs.empty()) e = hipMallocAsync(&d_runs, sizeof(uint4) * runs.size(), st);
    if (e == hipSuccess && !runs.empty())
        e = hipMemcpyAsync(d_runs, runs.data(), sizeof(uint4) * runs.size(), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) {
        const unsigned blocks = (unsigned)std::min<int64_t>(((int64_t)n + 3) / 4, 8192);
        hipLaunchKernelGGL(k_order_short, dim3(blocks), dim3(256), 0, st, n, ro_in, adj_in, s.arc, inf, s.a0, s.a1, s.w2);
        if (!runs.empty())
            hipLaunchKernelGGL(k_order_long, dim3((unsigned)runs.size()), dim3(256), 0, st,
                               static_cast<const uint4 *>(d_runs), ro_in, adj_in, s.arc, inf, s.a0, s.a1, s.w2, s.chunk);
        e = hipGetLastError();
    }
    if (d_runs) (void)hipFreeAsync(d_runs, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        (void)hipFree(s.base);
        return e;
    }
    *out = s;
    return hipSuccess;
}

size_t order_ws_bytes(int32_t n) {
    return al256(kOrderCtlWords * 8) + al256(2 * (size_t)bit_words(n) * 8) +
           al256(2 * (size_t)kOrderRegions * (size_t)queue_cap(n) * sizeof(uint2));
}

void order_carve(OrderJob *j, void *ws) {
    char *p = static_cast<char *>(ws);
    j->ctl = reinterpret_cast<unsigned long long *>(p);
    p += al256(kOrderCtlWords * 8);
    j->nword = bit_words(j->n);
    j->bits = reinterpret_cast<uint64_t *>(p);
    p += al256(2 * (size_t)j->nword * 8);
    j->cap = queue_cap(j->n);
    j->queue = reinterpret_cast<uint2 *>(p);
}

hipError_t order_begin(const OrderJob *jobs, int32_t k, int wt, OrderJob *table, hipStream_t st) {
    if (k < 1 || k > kOrderMaxJobs || wt < 0 || wt > 2) return hipErrorInvalidValue;
    for (int32_t b = 0; b < k; b += kBeginJobs) {
        BeginArgs a{};
        const int32_t c = std::min(kBeginJobs, k - b);
        int32_t big = 1;
        for (int32_t i = 0; i < c; ++i) {
            const OrderJob &j = jobs[b + i];
            if (j.n < 1 || j.src < 0 || j.src >= j.n || !j.dist || !j.arc || !j.ctl) return hipErrorInvalidValue;
            a.job[i] = j;
            big = std::max(big, j.n);
        }
        a.table = table + b;
        a.inf = wt == 1 ? kInfF32 : kInfU32;
        const int32_t blocks = (int32_t)std::min<int64_t>(((int64_t)big + 1023) / 1024, 1024);
        hipLaunchKernelGGL(k_order_begin, dim3((unsigned)blocks, (unsigned)c), dim3(256), 0, st, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool AHEAD>
static void launch_order(int wt, dim3 grid, hipStream_t st, const OrderArgs &a) {
    if (wt == 0) hipLaunchKernelGGL((k_order<0, AHEAD>), grid, dim3(256), 0, st, a);
    else if (wt == 1) hipLaunchKernelGGL((k_order<1, AHEAD>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_order<2, AHEAD>), grid, dim3(256), 0, st, a);
}

hipError_t order_rounds(const OrderJob *jobs, int32_t k, int wt, const OrderJob *table, int64_t first, int32_t rounds,
                        unsigned long long *stat, hipStream_t st) {
    // blocks for the vertices, and for the long rows (16 chunks each)
    int64_t blocks = 64, big = 0;
    for (int32_t i = 0; i < k; ++i) {
        big = std::max<int64_t>(big, jobs[i].n);
        blocks = std::max<int64_t>(blocks, std::min<int64_t>(((int64_t)jobs[i].n + kOrderVerts - 1) / kOrderVerts, 8192) +
                                               std::min<int64_t>(((int64_t)jobs[i].nchunks + 15) / 16, 1024));
    }
    const dim3 grid((unsigned)blocks, (unsigned)k);
    const bool ahead = big >= kOrderAhead;
    OrderArgs a{table, 0, stat, 0};
    for (int32_t r = 0; r < rounds; ++r) {
        a.round = first + r;
        a.tag = r + 1 == rounds ? 2ull * (unsigned long long)(first + rounds) : 0ull;
        if (ahead) launch_order<true>(wt, grid, st, a);
        else launch_order<false>(wt, grid, st, a);
    }
    return hipGetLastError();
}

size_t order_batch_bytes(int32_t n) {
    return al256(kOrderCtlWords * 8) + al256(3 * kOrderRegions * 64 * 4) + al256((size_t)n * kBatchLanes * 4) +
           al256(3 * (size_t)n * 8) + al256(2 * (size_t)kOrderRegions * (size_t)queue_cap(n) * sizeof(uint2));
}

void order_batch_carve(OrderBatch *b, void *ws) {
    char *p = static_cast<char *>(ws);
    const size_t n = (size_t)b->g.n;
    b->g.ctl = reinterpret_cast<unsigned long long *>(p);
    p += al256(kOrderCtlWords * 8);
    b->mu = reinterpret_cast<uint32_t *>(p);
    p += al256(3 * kOrderRegions * 64 * 4);
    b->D = reinterpret_cast<uint32_t *>(p);
    p += al256(n * kBatchLanes * 4);
    b->mask = reinterpret_cast<unsigned long long *>(p);
    p += al256(3 * n * 8);
    b->g.cap = queue_cap(b->g.n);
    b->g.queue = reinterpret_cast<uint2 *>(p);
}

hipError_t order_batch_begin(const OrderBatch &b, const int32_t *srcs, int wt, hipStream_t st) {
    const int32_t k = b.k;
    if (k < 1 || k > kBatchLanes || wt < 0 || wt > 1 || b.g.n < 1 || !b.g.arc || !b.D) return hipErrorInvalidValue;
    BatchBeginArgs a{};
    a.b = b;
    for (int32_t i = 0; i < k; ++i) {
        if (srcs[i] < 0 || srcs[i] >= b.g.n) return hipErrorInvalidValue;
        a.src[i] = srcs[i];
    }
    const unsigned blocks = (unsigned)std::min<int64_t>(((int64_t)b.g.n + 15) / 16, 4096);
    hipLaunchKernelGGL(k_order_batch_clear, dim3(blocks), dim3(256), 0, st, b, wt == 1 ? kInfF32 : kInfU32);
    hipLaunchKernelGGL(k_order_batch_begin, dim3(1), dim3(64), 0, st, a);
    return hipGetLastError();
}

hipError_t order_batch_rounds(const OrderBatch &b, int wt, int64_t first, int32_t rounds, int num_cu,
                              unsigned long long *stat, hipStream_t st) {
    // one block per 16 vertices, or four times the blocks that the chip holds
    // (rows differ in length: 2061 us for 64 sources of a scale-20 R-MAT graph,
    // 2182 with just what it holds, 2330 with eight times as many)
    const int64_t blocks = std::min<int64_t>(((int64_t)b.g.n + 4 * kBatchVerts - 1) / (4 * kBatchVerts), (int64_t)num_cu * 32);
    OrderBatchArgs a{b, 0, stat, 0};
    for (int32_t r = 0; r < rounds; ++r) {
        a.round = first + r;
        a.tag = r + 1 == rounds ? 2ull * (unsigned long long)(first + rounds) : 0ull;
        if (wt == 0) hipLaunchKernelGGL((k_order_batch<0>), dim3((unsigned)blocks), dim3(256), 0, st, a);
        else hipLaunchKernelGGL((k_order_batch<1>), dim3((unsigned)blocks), dim3(256), 0, st, a);
    }
    return hipGetLastError();
}

}  // namespace gr
