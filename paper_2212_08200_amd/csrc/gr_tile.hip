// Tiled asynchronous loop (Section III-A's asynchronous policy over Section
// III-D's partitioned graph: a tile is a partition, and its mail the message
// queue of Section III-B).
//
// Mesh-like graphs take thousands of hops, each a handful of relaxations: a
// round of the other loops costs a launch, or a chain of memory-side atomics
// per hop, so they run at the latency of that chain.  Here the chain of a hop
// stays inside a compute unit.  A workgroup of 16 waves holds one tile of up to
// kTileFill vertices: the distances in LDS, and each thread's four vertices
// with their arcs in registers.
//   14 waves sweep: a thread reads its four LDS words, and a vertex whose word
//     fell since its last expansion offers its arcs to its neighbours' words
//     with LDS atomic mins -- no list, no reply, no counter, no barrier.  0.2 us
//     per hop on a path (a round of the single-workgroup loop's lists: 0.45).
//   One wave sends: it watches the tails of the arcs that leave the tile and
//     stores what fell to the arc's mail word (one writer per word, so a plain
//     write-through store; contiguous per target tile).
//   One wave receives: it polls the mail words of the arcs that enter, and
//     finds out when the tile is quiet.
// About 2 us pass from a tile to the next.  The waves never wait for one another
// while the tile runs; with sends and receipts between the sweeps, behind a
// barrier every six sweeps, a mesh of 1024^2 took 1.18 ms against 0.90 (2048^2:
// 2.2 against 1.7; 173 x 229: 0.26 against 0.21), and a road-like 2048^2, where
// tiles change hands 25 times per workgroup, 0.94 against 1.17.  Measured and
// not taken: 8 vertices per thread (half the tiles, but each wave's pass twice
// as long: 1.5x the time), two workgroups per compute unit in 64 registers
// (spills), holding back vertices above a window over the tile's minimum (20
// to 100 times fewer expansions, the same time: expansions ride in idle lanes).
//
// Protocol across workgroups (every shared access is an atomic at device
// scope; a dependent access is issued after the earlier one was performed):
//   mail[e]    lowest offer along arc e so far; only falls
//   flag[q]    bit 0: q may have mail; bit 1: a workgroup holds q.  A sender
//              stores mail, then sets bit 0; if neither bit was set it also
//              queues q.  The holder clears bit 0 before it reads the mail, and
//              lets q go only by taking the flag from 2 to 0: a later sender
//              finds 0 and queues q again.
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
//   beat       progress, counted every few hundred microseconds while any tile
//              runs.  A workgroup may wait for as long as others do (on a path
//              all but one or two wait), so a wait has outlasted its bound only
//              if this did not change meanwhile.
// Any single resident workgroup makes progress alone, so the launch needs no
// co-residency.  dist is both the output and what survives of a tile between
// runs: the holder writes the words it lowered before it lets the tile go.
#include "gr_tile.h"

#include <algorithm>

#include "gr_device.h"

namespace gr {

namespace {

// Sweeps of a wave between two looks at the tile's state.
constexpr int kTileSweeps = 4;
constexpr int kTileNap = 8;  // s_sleep (64 cycles) of a wave whose block of sweeps found nothing (1: meshes 1% longer)
constexpr int kRegs = 5;  // arcs out, and mail words, that the two courier waves keep in registers, per lane
// Tokens a workgroup takes at once; it does so below what one pass over the arcs
// out can pass on.
constexpr int kTileTokens = 4 * kTileMaxExt;
// The receiving wave counts progress every so many passes (0.2 to 0.5 ms; by the
// clock, looked at every 16 passes, the meshes below took 1-2% longer), and a
// wait is bounded by no less than kTileMinSpin.
constexpr uint32_t kTileLooks = 256, kTileMinSpin = 1000000;
constexpr uint32_t kTileIdleTicks = 100;  // wall clock ticks (10 ns) a workgroup keeps its tokens while it waits

// Control words (8 bytes each, hot ones on 256-byte lines of their own).
constexpr int kTcStatus = 0;
constexpr int kTcHead = 32;
constexpr int kTcTail = 64;
constexpr int kTcActive = 96;
constexpr int kTcArcs = 128;
constexpr int kTcItems = 129;
constexpr int kTcExits = 130;
constexpr int kTcBeat = 160;
constexpr int kTcWords = 192;

template <typename T>
using gptr = T __attribute__((address_space(1))) *;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

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
    uint32_t spin;  // bound on a wait without progress, wall clock ticks
    unsigned long long *stat;
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

// Job blockIdx.y: distances and mail to INF, flags to 0 (the source's tile
// queued), the job table, and with job 0 the queue and the counters.
__global__ __launch_bounds__(256) void k_tile_init(TileInitArgs a) {
    const TileJob j = a.job[blockIdx.y];
    const int32_t t = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
    const int32_t job = a.base + (int32_t)blockIdx.y;
    const uint32_t inf = a.wt == 1 ? kInfF32 : kInfU32;
    const int32_t st = j.pos[j.src] >> kTileShift;
    for (int64_t i = t; i < j.n; i += step) j.dist[i] = inf;
    for (int64_t i = t; i < j.nmail; i += step) j.mail[i] = inf;
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

// A lane raises flag[q] and queues q if no workgroup holds it.  True when it
// passed a token on.
__device__ __forceinline__ bool tile_wake(const TileArgs &a, gptr<uint32_t> flags, uint32_t job, uint32_t q) {
    const uint32_t old =
        __hip_atomic_fetch_or(flags + (size_t)q * kTileFlagStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old == 0u) {
        gptr<unsigned long long> ctl = to_global(a.ctl);
        const unsigned long long p =
            __hip_atomic_fetch_add(ctl + kTcTail, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        gptr<uint32_t> slot = to_global(a.ring) + ((uint32_t)p & a.mask);
        while (ld_dev(slot) != 0u && ld_dev(ctl + kTcStatus) == 0ull) __builtin_amdgcn_s_sleep(1);
        __hip_atomic_store(slot, (job << 24 | q) + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return !(old & 1u);
}

constexpr int kTileExit = -1;

__device__ __forceinline__ uint32_t *at_byte(uint32_t *p, uint32_t off) {
    return reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(p) + off);
}

__device__ __forceinline__ uint32_t ld_lds(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void st_lds(uint32_t *p, uint32_t x) {
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void min_lds(uint32_t *p, uint32_t x) {
    (void)__hip_atomic_fetch_min(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Minimum over the first N lanes of every run of N, in every lane (N = 16: rows).
template <int N>
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
#define DPPMIN(ctrl) x = min(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, ctrl, 0xF, 0xF, false))
    DPPMIN(0xB1);   // quad_perm 1,0,3,2
    DPPMIN(0x4E);   // quad_perm 2,3,0,1
    DPPMIN(0x141);  // row_half_mirror
    DPPMIN(0x140);  // row_mirror
#undef DPPMIN
    if constexpr (N == 16) return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
    const uint32_t a = min((uint32_t)__builtin_amdgcn_readlane((int)x, 0), (uint32_t)__builtin_amdgcn_readlane((int)x, 16));
    const uint32_t b = min((uint32_t)__builtin_amdgcn_readlane((int)x, 32), (uint32_t)__builtin_amdgcn_readlane((int)x, 48));
    return min(a, b);
}

// Everything this wave sent to memory has been performed.
__device__ __forceinline__ void wait_mem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// WT: 0 uint32, 1 binary32, 2 unit steps; D: arc slots per vertex; COUNT:
// whether arcs are counted for the statistics (1% of the time of a mesh).  One workgroup
// fills a compute unit; with four slots its registers leave room for a wave
// per SIMD of other launches (a server's sessions: 48 mixed queries 5.6 ms
// against 6.3).
template <int WT, int D, bool COUNT>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(D == 4 ? 5 : 4))) void k_tile(
    TileArgs a) {
    __shared__ __attribute__((aligned(16))) uint32_t sD[kTileVerts];
    __shared__ uint32_t sSent[kTileMaxExt];  // tail distance each outgoing arc was last sent with
    __shared__ uint32_t sExtQ[kTileMaxExt], sExtW[kTileMaxExt];
    __shared__ uint32_t sInWord[kTileMaxExt];
    __shared__ uint16_t sExtU[kTileMaxExt], sInAt[kTileMaxExt];
    // by wave: sweeps done (low half), and the last of them that expanded
    // anything (high half, written first)
    __shared__ unsigned long long sSeq[kTileThreads / 64];
    __shared__ uint32_t sWake[64];
    __shared__ uint32_t sPark;
    __shared__ int sCmd;
    __shared__ int sTok;  // tokens the workgroup holds
    __shared__ unsigned long long sArcs, sItems;
    constexpr uint32_t kInf = WT == 1 ? kInfF32 : kInfU32;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const bool courier = wave == kInWave;
    gptr<unsigned long long> ctl = to_global(a.ctl);
    gptr<uint32_t> ring = to_global(a.ring);
    uint32_t items = 0, arcs = 0, seq = 0;
    if (t == 0) {
        sArcs = 0ull;
        sItems = 0ull;
        sTok = 0;
    }
    __syncthreads();
    const auto give_tokens = [&]() {  // one lane; the workgroup that leaves none ends the query
        if (sTok == 0) return;
        const unsigned long long x = (unsigned long long)sTok;
        sTok = 0;
        const unsigned long long old =
            __hip_atomic_fetch_add(ctl + kTcActive, 0ull - x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (old == x) __hip_atomic_store(ctl + kTcStatus, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    uint32_t looks = 0;  // the receiving wave's passes
    // one lane, waiting since t0; seen: beat when t0 was last set
    const auto waiting = [&](uint32_t &t0, uint32_t &seen) {
        const uint32_t now = (uint32_t)wall_clock64();
        if (now - t0 > kTileIdleTicks) give_tokens();
        if (now - t0 <= a.spin) return;
        const uint32_t b = (uint32_t)ld_dev(ctl + kTcBeat);
        if (b == seen) __hip_atomic_store(ctl + kTcStatus, 3ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        seen = b;
        t0 = now;
    };
    for (;;) {
        // 1. the next tile
        if (courier && lane == 0) {
            int cmd = kTileExit;
            {
                const unsigned long long p =
                    __hip_atomic_fetch_add(ctl + kTcHead, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                gptr<uint32_t> slot = ring + ((uint32_t)p & a.mask);
                uint32_t since = (uint32_t)wall_clock64(), seen = ~0u;
                for (;;) {
                    const uint32_t x = ld_dev(slot);
                    const unsigned long long s = ld_dev(ctl + kTcStatus);
                    if (x != 0u) {
                        __hip_atomic_store(slot, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        cmd = (int)(x - 1u);
                        break;
                    }
                    if (s != 0ull) break;
                    waiting(since, seen);
                    __builtin_amdgcn_s_sleep(2);
                }
                sCmd = cmd;
                sPark = 0u;
            }
        }
        __syncthreads();
        const int cmd = __builtin_amdgcn_readfirstlane(sCmd);
        if (cmd == kTileExit) break;
        const uint32_t job = (uint32_t)cmd >> 24, tile = (uint32_t)cmd & 0xFFFFFFu;
        const TileJob &J = a.job[job];
        gptr<uint32_t> flags = to_global(J.flags);
        gptr<uint32_t> flag = flags + (size_t)tile * kTileFlagStride;
        gptr<const int32_t> ino = to_global(J.in_off), exo = to_global(J.ext_off);
        const int32_t ib = ino[tile], nb = ino[tile + 1] - ib;
        const int32_t eb = exo[tile], ne = exo[tile + 1] - eb;
        if (courier && lane == 0) {
            // held, and bit 0 cleared before the mail is read
            (void)__hip_atomic_exchange(flag, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            wait_mem();
            sTok += 1;  // the entry's token
        }
        // 2. the tile: distances, arcs, the arcs that leave and enter it
        const size_t base = (size_t)tile << kTileShift;
        gptr<const int32_t> vid = to_global(J.vid) + base;
        gptr<uint32_t> dist = to_global(J.dist);
        uint32_t last[kTileVpt], w[kTileVpt][D], hd[kTileVpt][D / 2];
        uint32_t dirty = 0, deg = 0;  // deg: arcs in the columns (empty slots lead back), a byte per vertex
        {
            const u32x4 v = reinterpret_cast<gptr<const u32x4>>(vid)[t];
            gptr<const u32x4> pw = reinterpret_cast<gptr<const u32x4>>(to_global(J.w) + base * D) + t;
            gptr<const u32x4> ph = reinterpret_cast<gptr<const u32x4>>(to_global(J.head) + base * (D / 2)) + t;
#pragma unroll
            for (int s = 0; s < D; ++s) {
                const u32x4 x = WT == 2 ? u32x4{1u, 1u, 1u, 1u} : pw[s * kTileThreads];
#pragma unroll
                for (int i = 0; i < kTileVpt; ++i) w[i][s] = x[i];
            }
#pragma unroll
            for (int s = 0; s < D / 2; ++s) {
                const u32x4 x = ph[s * kTileThreads];
#pragma unroll
                for (int i = 0; i < kTileVpt; ++i) {
                    const uint32_t own = 4u * (uint32_t)tile_place(t, i);
                    hd[i][s] = x[i];
                    deg += ((x[i] & 0xFFFFu) != own ? 1u : 0u) << (8 * i);
                    deg += (x[i] >> 16 != own ? 1u : 0u) << (8 * i);
                }
            }
            // (places past the end read vertex 0)
#pragma unroll
            for (int i = 0; i < kTileVpt; ++i) last[i] = ld_dev(dist + max((int32_t)v[i], 0));
#pragma unroll
            for (int i = 0; i < kTileVpt; ++i) last[i] = (int32_t)v[i] < 0 ? kInf : last[i];
            *reinterpret_cast<u32x4 *>(&sD[t * kTileVpt]) = u32x4{last[0], last[1], last[2], last[3]};
        }
        {
            gptr<const u32x4> ext = reinterpret_cast<gptr<const u32x4>>(to_global(J.ext)) + eb;
            for (int32_t j = t; j < ne; j += kTileThreads) {
                const u32x4 e = ext[j];
                sExtU[j] = (uint16_t)e.x;
                sExtQ[j] = e.y;
                sExtW[j] = e.w;
            }
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            gptr<const u32x2> in = reinterpret_cast<gptr<const u32x2>>(to_global(J.in)) + ib;
            for (int32_t j = t; j < nb; j += kTileThreads) {
                const u32x2 e = in[j];
                sInWord[j] = e.x;
                sInAt[j] = (uint16_t)e.y;
            }
        }
        __syncthreads();
        for (int32_t j = t; j < ne; j += kTileThreads) sSent[j] = sD[sExtU[j]];
        if (lane == 0) sSeq[wave] = (unsigned long long)seq << 32 | seq;
        uint32_t *const my_seq = reinterpret_cast<uint32_t *>(sSeq + wave);
        __syncthreads();
        if (wave < kTileWaves) {
            // 3. sweeps, until the tile is found quiet
            for (;;) {
                do {
                    unsigned long long moved = 0ull;
#pragma unroll
                    for (int r = 0; r < kTileSweeps; ++r) {
                        asm volatile("" ::: "memory");  // the words are read again
                        const u32x4 cur = *reinterpret_cast<const u32x4 *>(&sD[t * kTileVpt]);
                        unsigned long long m[kTileVpt], any = 0ull;
#pragma unroll
                        for (int i = 0; i < kTileVpt; ++i) {
                            m[i] = __ballot(cur[i] < last[i]);
                            any |= m[i];
                        }
                        if (any == 0ull) continue;
                        moved |= any;
#pragma unroll
                        for (int i = 0; i < kTileVpt; ++i) {
                            if (m[i] == 0ull) continue;
                            items += (uint32_t)__popcll(m[i]);
                            if (cur[i] < last[i]) {
                                last[i] = cur[i];
                                dirty |= 1u << i;
                                if constexpr (COUNT) arcs = __builtin_amdgcn_udot4(deg, 1u << (8 * i), arcs, false);
#pragma unroll
                                for (int s = 0; s < D; ++s) {
                                    uint32_t h2 = hd[i][s / 2];
                                    // unpacked here: hoisted, it takes a register per arc
                                    asm volatile("" : "+v"(h2));
                                    min_lds(at_byte(sD, s & 1 ? h2 >> 16 : h2 & 0xFFFFu),
                                            tile_plus<WT>(cur[i], w[i][s]));
                                }
                            }
                        }
                    }
                    seq += kTileSweeps;
                    if (moved != 0ull) st_lds(my_seq + 1, seq);
                    else __builtin_amdgcn_s_sleep(kTileNap);
                    st_lds(my_seq, seq);
                } while (ld_lds(&sPark) == 0u);
                // quiet: what fell goes to memory
#pragma unroll
                for (int i = 0; i < kTileVpt; ++i)
                    if (dirty >> i & 1u)
                        __hip_atomic_store(dist + vid[tile_place(t, i)], last[i], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                dirty = 0;
                wait_mem();
                __syncthreads();
                __syncthreads();
                if (sCmd == 0) break;
            }
        } else if (wave == kOutWave) {
            // 4. offers out: arcs whose tail fell since they were last sent.
            // A pass counts as a block of sweeps of the other waves.
            gptr<uint32_t> mail = to_global(J.mail) + eb;
            // the first arcs' tails (byte offsets) and what they were last sent with, in registers
            uint32_t eu[kRegs], sent[kRegs];
#pragma unroll
            for (int k = 0; k < kRegs; ++k) {
                const int j = min(k * 64 + lane, max(ne - 1, 0));
                eu[k] = 4u * sExtU[j] & (4u * kTileVerts - 1);
                sent[k] = sSent[j];
            }
            for (;;) {
                do {
                    int tok = __builtin_amdgcn_readfirstlane(sTok);
                    if (tok <= kTileMaxExt) {
                        if (lane == 0)
                            (void)__hip_atomic_fetch_add(ctl + kTcActive, (unsigned long long)kTileTokens,
                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        wait_mem();
                        tok += kTileTokens;
                        sTok = tok;
                    }
                    int nw = 0;  // tiles to wake; the arcs are sorted by target tile
                    uint32_t lastq = kTileInner;
                    bool moved = false;
                    const auto wake = [&]() {
                        // (their offers have been performed)
                        wait_mem();
                        bool passed = false;
                        if (lane < nw) passed = tile_wake(a, flags, job, sWake[lane]);
                        tok -= (int)__popcll(__ballot(passed));
                        nw = 0;
                    };
                    const auto send = [&](int32_t j, bool fell, uint32_t du) {
                        moved = true;
                        uint32_t q = kTileInner;
                        if (fell) {
                            if constexpr (COUNT) ++arcs;
                            const uint32_t nd = tile_plus<WT>(du, sExtW[j]);
                            q = sExtQ[j];
                            if (q & kTileInner) min_lds(&sD[q & 0xFFFFu], nd);
                            else __hip_atomic_store(mail + j, nd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
                        for (unsigned long long m = __ballot(!(q & kTileInner)); m;) {
                            const uint32_t q0 = (uint32_t)__builtin_amdgcn_readlane((int)q, __ffsll(m) - 1);
                            m &= ~__ballot(q == q0);
                            if (q0 == lastq) continue;
                            lastq = q0;
                            if (nw == 64) wake();
                            if (lane == 0) sWake[nw] = q0;
                            ++nw;
                        }
                    };
                    uint32_t du[kRegs];
#pragma unroll
                    for (int k = 0; k < kRegs; ++k) du[k] = ld_lds(at_byte(sD, eu[k]));
#pragma unroll
                    for (int k = 0; k < kRegs; ++k) {
                        const bool fell = k * 64 + lane < ne && du[k] < sent[k];
                        if (__ballot(fell) == 0ull) continue;
                        if (fell) sent[k] = du[k];
                        send(k * 64 + lane, fell, du[k]);
                    }
                    for (int32_t j0 = kRegs * 64; j0 < ne; j0 += 64) {
                        const int32_t j = min(j0 + lane, ne - 1);
                        const uint32_t d = ld_lds(&sD[sExtU[j]]);
                        const bool fell = j0 + lane < ne && d < sSent[j];
                        if (__ballot(fell) == 0ull) continue;
                        if (fell) sSent[j] = d;
                        send(j, fell, d);
                    }
                    if (nw) {
                        wake();
                        sTok = tok;
                    }
                    seq += kTileSweeps;
                    if (moved) st_lds(my_seq + 1, seq);
                    st_lds(my_seq, seq);
                } while (ld_lds(&sPark) == 0u);
                __syncthreads();
                __syncthreads();
                if (sCmd == 0) break;
            }
        } else {
            // 5. offers in, and when the tile is quiet
            gptr<uint32_t> mail = to_global(J.mail);
            const uint32_t spos = (uint32_t)J.pos[J.src];
            if (lane == 0 && spos >> kTileShift == tile) min_lds(&sD[spos & (kTileVerts - 1)], 0u);
            // the first words, their vertices and what was taken from them, in registers
            uint32_t in_at[kRegs], in_word[kRegs], got[kRegs];
#pragma unroll
            for (int k = 0; k < kRegs; ++k) {
                const int i = min(k * 64 + lane, max(nb - 1, 0));
                in_at[k] = 4u * sInAt[i] & (4u * kTileVerts - 1);
                in_word[k] = nb > 0 ? sInWord[i] : 0u;
                got[k] = kInf;
            }
            const auto ran = [&]() {
                return __hip_atomic_load(&sSeq[min(lane, kTileWaves)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            };
            bool moved = true;  // something came in since the snapshot
            uint32_t snap = 0;
            for (;;) {
                uint32_t x[kRegs];
#pragma unroll
                for (int k = 0; k < kRegs; ++k)
                    if (k * 64 < nb) x[k] = ld_dev(mail + in_word[k]);
#pragma unroll
                for (int k = 0; k < kRegs; ++k)
                    if (k * 64 < nb) {
                        const bool less = x[k] < got[k];  // words past the end repeat the last one
                        if (__ballot(less) == 0ull) continue;
                        if (less) {
                            got[k] = x[k];
                            min_lds(at_byte(sD, in_at[k]), x[k]);
                        }
                        moved = true;
                    }
                for (int32_t j0 = kRegs * 64; j0 < nb; j0 += 256) {
                    uint32_t y[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) y[k] = ld_dev(mail + sInWord[min(j0 + k * 64 + lane, nb - 1)]);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const uint32_t l = sInAt[min(j0 + k * 64 + lane, nb - 1)];
                        const bool less = y[k] < ld_lds(&sD[l]);
                        if (less) min_lds(&sD[l], y[k]);
                        moved = moved || __ballot(less) != 0ull;
                    }
                }
                // quiet: since a snapshot no wave expanded or sent anything,
                // each began and ended a pass, and nothing came in.  (What a
                // wave, or this one, offered before the snapshot had landed by
                // then.)
                bool quiet = false;
                while (!moved) {
                    const unsigned long long z = ran();
                    if (__ballot((int32_t)((uint32_t)(z >> 32) - snap) > 0) != 0ull) break;
                    quiet = __ballot((int32_t)((uint32_t)z - snap) < 2 * kTileSweeps) == 0ull;
                    if (quiet) break;
                }
                if (!quiet) {
                    snap = (uint32_t)ran();
                    moved = false;
                    if ((++looks % kTileLooks) == 0u && lane == 0)
                        (void)__hip_atomic_fetch_add(ctl + kTcBeat, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    continue;
                }
                // its distances go to memory; it waits for mail, or is let go
                if (lane == 0) st_lds(&sPark, 1u);
                __syncthreads();
                int next = 0;  // 0: let go, 1: again
                if (lane == 0) {
                    uint32_t since = (uint32_t)wall_clock64(), seen = ~0u;
                    for (;;) {
                        if (ld_dev(flag) & 1u) {
                            (void)__hip_atomic_exchange(flag, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            wait_mem();
                            sTok += 1;
                            next = 1;
                            break;
                        }
                        const bool over = ld_dev(ctl + kTcStatus) != 0ull;
                        if (over || ld_dev(ctl + kTcTail) > ld_dev(ctl + kTcHead)) {
                            uint32_t held = 2u;
                            if (__hip_atomic_compare_exchange_strong(flag, &held, 0u, __ATOMIC_RELAXED,
                                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ||
                                over)
                                break;
                            continue;
                        }
                        waiting(since, seen);
                        __builtin_amdgcn_s_sleep(1);
                    }
                    sCmd = next;
                    st_lds(&sPark, 0u);
                }
                next = __builtin_amdgcn_readfirstlane(next);
                __syncthreads();
                if (next == 0) break;
                moved = true;
            }
        }
        __syncthreads();  // LDS reuse
    }
    // (items is the wave's, arcs the lane's)
    if (lane == 0) atomicAdd(&sItems, (unsigned long long)items);
    if constexpr (COUNT) atomicAdd(&sArcs, (unsigned long long)arcs);
    __syncthreads();
    if (t == 0) {
        (void)__hip_atomic_fetch_add(ctl + kTcItems, sItems, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if constexpr (COUNT) {
            (void)__hip_atomic_fetch_add(ctl + kTcArcs, sArcs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        wait_mem();
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
        b += al256((size_t)sets[i]->ntiles * kTileFlagStride * 4) + al256((size_t)sets[i]->mail * 4);
    }
    return b + al256((size_t)ring_entries(tiles) * 4);
}

size_t tile_query_bytes(const TileSet &set) {
    // its flags and mail, its entry in the table, and its share of the queue:
    // ring_entries(t1 + t2 + ...) < 4 (t1 + t2 + ...) + 4096
    return al256((size_t)set.ntiles * kTileFlagStride * 4) + al256((size_t)set.mail * 4) +
           4 * (4 * (size_t)set.ntiles + 4096) + al256(kTcWords * 8) + al256(sizeof(TileJob)) + 256;
}

hipError_t launch_tiles(const TileSet *const *sets, const int32_t *srcs, uint32_t *const *dist, int32_t k, int wt,
                        void *ws, int num_cu, uint64_t spin_ticks, bool count, unsigned long long *stat, hipStream_t st) {
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
    a.spin = (uint32_t)std::clamp<uint64_t>(spin_ticks, kTileMinSpin, INT32_MAX);
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
            j.in = s.in;
            j.in_off = s.in_off;
            j.dist = dist[b + i];
            j.flags = reinterpret_cast<uint32_t *>(p);
            p += al256((size_t)s.ntiles * kTileFlagStride * 4);
            j.mail = reinterpret_cast<uint32_t *>(p);
            p += al256((size_t)s.mail * 4);
            j.n = s.n;
            j.ntiles = s.ntiles;
            j.nmail = s.mail;
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
    // one workgroup per tile, up to one per compute unit (its registers leave no
    // room for another)
    const int64_t room = (int64_t)num_cu;
    const unsigned grid = (unsigned)(tiles < room ? tiles : room);
    const dim3 g(grid), blk(kTileThreads);
#define TILE_LAUNCH(WT, D)                                                            \
    do {                                                                              \
        if (count) hipLaunchKernelGGL((k_tile<WT, D, true>), g, blk, 0, st, a);       \
        else hipLaunchKernelGGL((k_tile<WT, D, false>), g, blk, 0, st, a);            \
    } while (0)
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
