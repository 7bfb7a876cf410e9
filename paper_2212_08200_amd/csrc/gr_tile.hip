// Tiled asynchronous loop (Section III-A's asynchronous policy over Section
// III-D's partitioned graph: a tile is a partition, and its inbox the message
// queue of Section III-B).
//
// Mesh-like graphs take thousands of hops, each a handful of relaxations: a
// round of the other loops costs a launch, or a chain of memory-side atomics
// per hop, so they run at the latency of that chain.  Here the chain of a hop
// stays inside a compute unit.  A workgroup of 1024 threads holds one tile of
// up to 4096 vertices: the distances in LDS, and each thread's four vertices
// with their arcs in registers.  A sweep reads the thread's four LDS words,
// and a vertex whose word fell since its last expansion offers its arcs to
// its neighbours' words with LDS atomic mins: no list, no reply, no counter.
// Sweeps run freely; every kTileSweeps of them one workgroup barrier decides
// whether anything moved.  What crosses a tile's border goes to the target
// tile's inbox word with a memory-side atomic min, between sweeps.
//
// Protocol across workgroups (every shared access is an atomic at device
// scope; a dependent access is issued after the earlier one returned):
//   inbox[i]   lowest offer to a border vertex so far; only falls
//   flag[q]    bit 0: an offer may wait in q's inbox; bit 1: a workgroup
//              holds q.  A sender lowers an inbox word, then sets bit 0; if
//              neither bit was set it also queues q.  The holder clears bit 0
//              before it reads the inbox, and lets q go only by taking the
//              flag from 2 to 0: a later offer finds 0 and queues q again.
//   ring       queue of tiles: positions are handed out by an atomic add on
//              either end; a consumer waits for its own position.  A tile is
//              queued at most once, so at most as many entries as tiles are
//              outstanding, and a producer waits for the position's last
//              entry to be taken (by a workgroup that already waits for it).
//   active     tokens: one for every flag whose bit 0 is set, and those held
//              by running workgroups.  A workgroup that sets a bit 0 passes
//              one of its own tokens on, and returns what it holds when it
//              has nothing to do, after its writes were performed.  active =
//              0 thus means that no offer is left anywhere: the query ends.
// Any single resident workgroup makes progress alone, so the launch needs no
// co-residency.  dist is both the output and what survives of a tile between
// runs: the holder writes the words it lowered before it lets the tile go.
#include "gr_tile.h"

#include "gr_device.h"

namespace gr {

namespace {

// Sweeps between two workgroup barriers.
constexpr int kTileSweeps = 6;
// Tokens a workgroup takes at once; it tops up below what one send pass can pass on.
constexpr int kTileTokens = 8 * kTileMaxExt;
constexpr uint64_t kTileIdleTicks = 300;  // wall clock ticks (10 ns) a workgroup keeps its tokens while it waits

// Control words (8 bytes each, hot ones on 256-byte lines of their own).
constexpr int kTcStatus = 0;
constexpr int kTcHead = 32;
constexpr int kTcTail = 64;
constexpr int kTcActive = 96;
constexpr int kTcArcs = 128;
constexpr int kTcItems = 129;
constexpr int kTcExits = 130;
constexpr int kTcWords = 160;

template <typename T>
using gptr = T __attribute__((address_space(1))) *;

template <typename T>
__device__ __forceinline__ gptr<T> to_global(T *p) {
    return (gptr<T>)p;
}

template <typename T>
__device__ __forceinline__ T ld_dev(gptr<T> p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct TileArgs {
    const TileJob *job;
    uint32_t *ring;
    uint32_t mask;  // ring entries - 1
    unsigned long long *ctl;
    uint64_t spin_ticks;
    unsigned long long *stat;
    int32_t linger;  // keep a quiet tile while no other tile waits for a workgroup
};

constexpr int kInitJobs = 16;
struct TileInitArgs {
    TileJob job[kInitJobs];
    TileJob *table;  // of this launch's first job
    uint32_t *ring;
    uint32_t ring_len;
    unsigned long long *ctl;
    int32_t k, base, wt;
};

// Job blockIdx.y: distances and inbox to INF, flags to 0 (the source's tile
// queued), the job table, and with job 0 the queue and the counters.
__global__ __launch_bounds__(256) void k_tile_init(TileInitArgs a) {
    const TileJob j = a.job[blockIdx.y];
    const int32_t t = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
    const int32_t job = a.base + (int32_t)blockIdx.y;
    const uint32_t inf = a.wt == 1 ? kInfF32 : kInfU32;
    const int32_t st = j.pos[j.src] >> kTileShift;
    for (int64_t i = t; i < j.n; i += step) j.dist[i] = inf;
    for (int64_t i = t; i < j.ninbox; i += step) j.inbox[i] = inf;
    for (int64_t i = t; i < (int64_t)j.ntiles * kTileFlagStride; i += step)
        j.flags[i] = i == (int64_t)st * kTileFlagStride ? 1u : 0u;
    if (t == 0) {
        a.table[blockIdx.y] = j;
        a.ring[job] = ((uint32_t)job << 24 | (uint32_t)st) + 1u;
    }
    if (job == 0) {
        for (int64_t i = a.k + t; i < a.ring_len; i += step) a.ring[i] = 0u;
        for (int32_t i = t; i < kTcWords; i += step)
            a.ctl[i] = i == kTcTail || i == kTcActive ? (unsigned long long)a.k : 0ull;
    }
}

// plus() with the saturation in the add itself where the type has one.
template <int WT>
__device__ __forceinline__ uint32_t tile_plus(uint32_t d, uint32_t w) {
    if constexpr (WT == 1) return min(__float_as_uint(__uint_as_float(d) + __uint_as_float(w)), kInfF32);
    else return __builtin_elementwise_add_sat(d, WT == 2 ? 1u : w);
}

// Lanes with want set raise flag[q] and queue q when no workgroup holds it;
// one lane per distinct tile of the wave acts.  Returns the number of
// tokens passed on by this lane.
__device__ __forceinline__ int tile_wake(const TileArgs &a, gptr<uint32_t> flags, uint32_t job, uint32_t q,
                                         bool want) {
    bool lead = false;
    for (unsigned long long m = __ballot(want); m;) {
        const int l = __ffsll(m) - 1;
        const uint32_t q0 = (uint32_t)__builtin_amdgcn_readlane((int)q, l);
        lead = lead || (int)(threadIdx.x & 63) == l;
        m &= ~__ballot(want && q == q0);
    }
    if (!lead) return 0;
    const uint32_t old =
        __hip_atomic_fetch_or(flags + (size_t)q * kTileFlagStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old & 1u) return 0;
    if (!(old & 2u)) {
        gptr<unsigned long long> ctl = to_global(a.ctl);
        const unsigned long long p =
            __hip_atomic_fetch_add(ctl + kTcTail, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        gptr<uint32_t> slot = to_global(a.ring) + ((uint32_t)p & a.mask);
        while (ld_dev(slot) != 0u && ld_dev(ctl + kTcStatus) == 0ull) __builtin_amdgcn_s_sleep(1);
        __hip_atomic_store(slot, (job << 24 | q) + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return 1;
}

__device__ __forceinline__ uint32_t *at_byte(uint32_t *p, uint32_t off) {
    return reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(p) + off);
}

// Every store this thread issued has been performed.
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

enum : int { kTileGot = 0, kTileExit = -1 };

// WT: 0 uint32, 1 binary32, 2 unit steps; D: arc slots per vertex.
template <int WT, int D>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_tile(
    TileArgs a) {
    __shared__ uint32_t sD[kTileVerts];
    __shared__ int sFlag[3];
    __shared__ int sCmd;
    __shared__ int sTok;  // tokens this workgroup holds
    __shared__ unsigned long long sArcs, sItems;
    constexpr uint32_t kInf = WT == 1 ? kInfF32 : kInfU32;
    const int t = threadIdx.x;
    gptr<unsigned long long> ctl = to_global(a.ctl);
    gptr<uint32_t> ring = to_global(a.ring);
    uint32_t items = 0, arcs = 0;
    if (t == 0) {
        sTok = 0;
        sArcs = 0ull;
        sItems = 0ull;
    }
    // thread 0: returns the workgroup's tokens; the one that leaves none ends
    // the query
    const auto give_tokens = [&]() {
        if (sTok == 0) return;
        const unsigned long long x = (unsigned long long)sTok;
        sTok = 0;
        const unsigned long long old =
            __hip_atomic_fetch_add(ctl + kTcActive, 0ull - x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (old == x) __hip_atomic_store(ctl + kTcStatus, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // thread 0: takes tokens (the caller holds at least one).  Called before
    // every send pass, each of which passes on at most kTileMaxExt: while the
    // other threads run one pass, more than that many are left.
    const auto take_tokens = [&]() {
        if (__hip_atomic_load(&sTok, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > 3 * kTileMaxExt) return;
        (void)__hip_atomic_fetch_add(ctl + kTcActive, (unsigned long long)kTileTokens, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
        wait_stores();
        (void)atomicAdd(&sTok, kTileTokens);
    };
    for (;;) {
        // 1. the next tile
        if (t == 0) {
            const unsigned long long p =
                __hip_atomic_fetch_add(ctl + kTcHead, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            gptr<uint32_t> slot = ring + ((uint32_t)p & a.mask);
            const uint64_t t0 = wall_clock64();
            int cmd = kTileExit;
            for (;;) {
                const uint32_t x = ld_dev(slot);
                const unsigned long long s = ld_dev(ctl + kTcStatus);
                if (x != 0u) {
                    __hip_atomic_store(slot, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    cmd = (int)(x - 1u);
                    break;
                }
                if (s != 0ull) break;
                const uint64_t dt = wall_clock64() - t0;
                if (dt > kTileIdleTicks) give_tokens();
                if (dt > a.spin_ticks)
                    __hip_atomic_store(ctl + kTcStatus, 3ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __builtin_amdgcn_s_sleep(2);
            }
            sCmd = cmd;
        }
        __syncthreads();
        const int cmd = __builtin_amdgcn_readfirstlane(sCmd);
        if (cmd == kTileExit) break;
        const uint32_t job = (uint32_t)cmd >> 24, tile = (uint32_t)cmd & 0xFFFFFFu;
        const TileJob &J = a.job[job];
        gptr<uint32_t> flags = to_global(J.flags);
        gptr<uint32_t> flag = flags + (size_t)tile * kTileFlagStride;
        if (t == 0) {
            // held, and bit 0 cleared before the inbox is read
            (void)__hip_atomic_exchange(flag, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sTok += 1;  // the entry's token
            take_tokens();
            wait_stores();
            sFlag[0] = sFlag[1] = sFlag[2] = 0;
        }
        // 2. the tile: distances, arcs, the arcs that leave it
        const size_t base = (size_t)tile << kTileShift;
        gptr<const int32_t> vid = to_global(J.vid) + base;
        gptr<uint32_t> dist = to_global(J.dist);
        uint32_t last[kTileVpt], w[kTileVpt][D], hd[kTileVpt][D / 2];
        uint32_t dirty = 0;
        {
            int32_t v[kTileVpt];
#pragma unroll
            for (int i = 0; i < kTileVpt; ++i) v[i] = vid[tile_place(t, i)];
            gptr<const uint32_t> pw = to_global(J.w) + base * D;
            gptr<const uint32_t> ph = to_global(J.head) + base * (D / 2);
#pragma unroll
            for (int s = 0; s < D; ++s)
#pragma unroll
                for (int i = 0; i < kTileVpt; ++i) w[i][s] = WT == 2 ? 1u : pw[s * kTileVerts + tile_place(t, i)];
#pragma unroll
            for (int s = 0; s < D / 2; ++s)
#pragma unroll
                for (int i = 0; i < kTileVpt; ++i) hd[i][s] = ph[s * kTileVerts + tile_place(t, i)];
            // (places past the end read vertex 0)
#pragma unroll
            for (int i = 0; i < kTileVpt; ++i) last[i] = ld_dev(dist + max(v[i], 0));
#pragma unroll
            for (int i = 0; i < kTileVpt; ++i) {
                last[i] = v[i] < 0 ? kInf : last[i];
                sD[tile_place(t, i)] = last[i];
            }
        }
        gptr<const int32_t> ino = to_global(J.in_off), exo = to_global(J.ext_off);
        const int32_t ib = ino[tile], nb = ino[tile + 1] - ib;
        const int32_t eb = exo[tile], ne = exo[tile + 1] - eb;
        gptr<uint32_t> box = to_global(J.inbox) + ib;
        gptr<uint32_t> boxes = to_global(J.inbox);
        gptr<const int32_t> ina = to_global(J.in_at) + ib;
        int32_t bl[2];  // local places of this thread's inbox words
#pragma unroll
        for (int k = 0; k < 2; ++k) bl[k] = ina[min(k * kTileThreads + t, max(nb - 1, 0))];
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        u32x4 ex[2];
        uint32_t sent[2];
#pragma unroll
        for (int k = 0; k < 2; ++k)
            ex[k] = reinterpret_cast<gptr<const u32x4>>(to_global(J.ext))[eb + min(k * kTileThreads + t, max(ne - 1, 0))];
        const int32_t spos = J.pos[J.src];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 2; ++k) sent[k] = k * kTileThreads + t < ne ? sD[ex[k].x] : 0u;
        __syncthreads();
        if (t == 0 && (uint32_t)spos >> kTileShift == tile) sD[spos & (kTileVerts - 1)] = 0u;
        bool again = true;  // the inbox was not read since bit 0 was cleared
        int p = 0;
        for (;;) {
            if (again) {
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    if (k * kTileThreads + t < nb)
                        (void)__hip_atomic_fetch_min(&sD[bl[k]], ld_dev(box + (k * kTileThreads + t)), __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_WORKGROUP);
                again = false;
                __syncthreads();
            }
            // 3. sweeps, while new offers are on their way from the inbox
            bool any = false;
            uint32_t x[2];
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (k * kTileThreads + t < nb) x[k] = ld_dev(box + (k * kTileThreads + t));
            for (int r = 0; r < kTileSweeps; ++r) {
                uint32_t cur[kTileVpt];
                bool c = false;
#pragma unroll
                for (int i = 0; i < kTileVpt; ++i) {
                    cur[i] = __hip_atomic_load(&sD[tile_place(t, i)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    c = c || cur[i] < last[i];
                }
                if (c) {
                    any = true;
#pragma unroll
                    for (int i = 0; i < kTileVpt; ++i)
                        if (cur[i] < last[i]) {
                            last[i] = cur[i];
                            dirty |= 1u << i;
                            ++items;
#pragma unroll
                            for (int s = 0; s < D; ++s) {
                                uint32_t h2 = hd[i][s / 2];
                                asm volatile("" : "+v"(h2));  // unpacked here: hoisted, it takes a register per arc
                                (void)__hip_atomic_fetch_min(at_byte(sD, s & 1 ? h2 >> 16 : h2 & 0xFFFFu),
                                                             tile_plus<WT>(cur[i], w[i][s]), __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_WORKGROUP);
                            }
                        }
                }
            }
            // 4. offers that arrived meanwhile
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (k * kTileThreads + t < nb &&
                    x[k] < __hip_atomic_load(&sD[bl[k]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) {
                    (void)__hip_atomic_fetch_min(&sD[bl[k]], x[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    any = true;
                }
            // 5. arcs out of the tile whose tail fell since they were last sent
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                if (k * kTileThreads >= ne) continue;  // uniform
                bool want = false;
                uint32_t q = 0;
                const uint32_t du = __hip_atomic_load(&sD[ex[k].x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (du < sent[k]) {
                    sent[k] = du;
                    ++arcs;
                    const uint32_t nd = tile_plus<WT>(du, ex[k].w);
                    q = ex[k].y;
                    if (q & kTileInner) {
                        (void)__hip_atomic_fetch_min(&sD[q & 0xFFFFu], nd, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_WORKGROUP);
                        any = true;
                    } else {
                        want = nd < __hip_atomic_fetch_min(boxes + ex[k].z, nd, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
                const int passed = tile_wake(a, flags, job, q, want);
                if (passed) (void)atomicSub(&sTok, passed);
            }
            if (any) sFlag[p] = 1;
            const int pn = p == 2 ? 0 : p + 1;
            if (t == 0) sFlag[pn] = 0;  // last read two barriers ago
            __syncthreads();
            const bool more = sFlag[p] != 0;
            p = pn;
            if (more) {
                if (t == 0) take_tokens();
                continue;
            }
            // 6. quiet: what fell goes to memory, then the tile waits for
            // offers or is let go
            if (dirty) {
#pragma unroll
                for (int i = 0; i < kTileVpt; ++i)
                    if (dirty >> i & 1u)
                        __hip_atomic_store(dist + vid[tile_place(t, i)], last[i], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                dirty = 0;
            }
            wait_stores();
            __syncthreads();
            if (t == 0) {
                int next = 0;  // 0: let go, 1: again
                const uint64_t t0 = wall_clock64();
                for (;;) {
                    const uint32_t f = ld_dev(flag);
                    if (f & 1u) {
                        (void)__hip_atomic_exchange(flag, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        sTok += 1;
                        take_tokens();
                        wait_stores();
                        next = 1;
                        break;
                    }
                    const uint64_t dt = wall_clock64() - t0;
                    const bool over = ld_dev(ctl + kTcStatus) != 0ull;
                    const bool wanted = !a.linger || over || ld_dev(ctl + kTcTail) > ld_dev(ctl + kTcHead);
                    if (wanted) {
                        uint32_t held = 2u;
                        if (__hip_atomic_compare_exchange_strong(flag, &held, 0u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                                 __HIP_MEMORY_SCOPE_AGENT))
                            break;
                        if (over) break;
                        continue;
                    }
                    if (dt > kTileIdleTicks) give_tokens();
                    if (dt > a.spin_ticks)
                        __hip_atomic_store(ctl + kTcStatus, 3ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __builtin_amdgcn_s_sleep(2);
                }
                sCmd = next;
            }
            __syncthreads();
            again = sCmd != 0;
            if (!again) break;
        }
        __syncthreads();  // sD, sCmd reuse
    }
    atomicAdd(&sItems, (unsigned long long)items);
    atomicAdd(&sArcs, (unsigned long long)arcs + (unsigned long long)items * D);
    __syncthreads();
    if (t == 0) {
        (void)__hip_atomic_fetch_add(ctl + kTcItems, sItems, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        (void)__hip_atomic_fetch_add(ctl + kTcArcs, sArcs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        wait_stores();
        const unsigned long long x =
            __hip_atomic_fetch_add(ctl + kTcExits, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (x + 1ull == gridDim.x) {  // the last one: statistics to the host
            __hip_atomic_store(a.stat + 1, ld_dev(ctl + kTcArcs), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(a.stat + 2, ld_dev(ctl + kTcItems), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(a.stat + 0, ld_dev(ctl + kTcStatus), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

inline size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

uint32_t ring_entries(int64_t tiles) {
    uint32_t r = 1024;
    while ((int64_t)r < 2 * tiles + 2048) r <<= 1;
    return r;
}

}  // namespace

size_t tile_ws_bytes(const TileSet *const *sets, int32_t k) {
    int64_t tiles = 0;
    size_t b = al256(kTcWords * 8) + al256(sizeof(TileJob) * (size_t)k);
    for (int32_t i = 0; i < k; ++i) {
        tiles += sets[i]->ntiles;
        b += al256((size_t)sets[i]->ntiles * kTileFlagStride * 4) + al256((size_t)sets[i]->inbox * 4);
    }
    return b + al256((size_t)ring_entries(tiles) * 4);
}

hipError_t launch_tiles(const TileSet *const *sets, const int32_t *srcs, uint32_t *const *dist, int32_t k, int wt,
                        void *ws, int num_cu, uint64_t spin_ticks, unsigned long long *stat, hipStream_t st) {
    if (k < 1 || k > kTileMaxJobs || wt < 0 || wt > 2 || !ws || !stat) return hipErrorInvalidValue;
    int64_t tiles = 0;
    for (int32_t i = 0; i < k; ++i) {
        const TileSet &s = *sets[i];
        if (s.ntiles < 1 || s.ntiles > kTileMaxTiles || s.slots != sets[0]->slots || srcs[i] < 0 || srcs[i] >= s.n ||
            !dist[i])
            return hipErrorInvalidValue;
        tiles += s.ntiles;
    }
    char *p = static_cast<char *>(ws);
    TileArgs a{};
    a.ctl = reinterpret_cast<unsigned long long *>(p);
    p += al256(kTcWords * 8);
    TileJob *table = reinterpret_cast<TileJob *>(p);
    a.job = table;
    p += al256(sizeof(TileJob) * (size_t)k);
    a.ring = reinterpret_cast<uint32_t *>(p);
    const uint32_t rl = ring_entries(tiles);
    a.mask = rl - 1;
    p += al256((size_t)rl * 4);
    a.spin_ticks = spin_ticks;
    a.stat = stat;
    for (int32_t b = 0; b < k; b += kInitJobs) {
        TileInitArgs ia{};
        const int32_t c = k - b < kInitJobs ? k - b : kInitJobs;
        int32_t big = 1;
        for (int32_t i = 0; i < c; ++i) {
            const TileSet &s = *sets[b + i];
            TileJob &j = ia.job[i];
            j.pos = s.pos;
            j.vid = s.vid;
            j.w = s.w;
            j.head = s.head;
            j.ext = s.ext;
            j.ext_off = s.ext_off;
            j.in_off = s.in_off;
            j.in_at = s.in_at;
            j.dist = dist[b + i];
            j.flags = reinterpret_cast<uint32_t *>(p);
            p += al256((size_t)s.ntiles * kTileFlagStride * 4);
            j.inbox = reinterpret_cast<uint32_t *>(p);
            p += al256((size_t)s.inbox * 4);
            j.n = s.n;
            j.ntiles = s.ntiles;
            j.ninbox = s.inbox;
            j.src = srcs[b + i];
            big = s.n > big ? s.n : big;
        }
        ia.table = table + b;
        ia.ring = a.ring;
        ia.ring_len = rl;
        ia.ctl = a.ctl;
        ia.k = k;
        ia.base = b;
        ia.wt = wt;
        const int blocks = (int)((big + 1023) / 1024 < 4 * num_cu ? (big + 1023) / 1024 : 4 * num_cu);
        hipLaunchKernelGGL(k_tile_init, dim3((unsigned)blocks, (unsigned)c), dim3(256), 0, st, ia);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // one workgroup per tile, up to what the chip holds (2048 threads per compute unit;
    // eight slots take the registers of one workgroup per compute unit)
    const int64_t room = (int64_t)num_cu;
    const unsigned grid = (unsigned)(tiles < room ? tiles : room);
    a.linger = 1;
    const dim3 g(grid), blk(kTileThreads);
#define TILE_LAUNCH(WT, D) hipLaunchKernelGGL((k_tile<WT, D>), g, blk, 0, st, a)
    if (sets[0]->slots == 4) {
        if (wt == 0) TILE_LAUNCH(0, 4);
        else if (wt == 1) TILE_LAUNCH(1, 4);
        else TILE_LAUNCH(2, 4);
    } else {
        if (wt == 0) TILE_LAUNCH(0, 8);
        else if (wt == 1) TILE_LAUNCH(1, 8);
        else TILE_LAUNCH(2, 8);
    }
#undef TILE_LAUNCH
    return hipGetLastError();
}

}  // namespace gr
