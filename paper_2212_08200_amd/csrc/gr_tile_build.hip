// Builds the tiled layout (gr_tile.h): the vertices of a mesh-like graph cut
// into tiles of at most kTileFill with most arcs inside.
//
// 1. Cells: one seed vertex per run of kCellVerts ids; sweeps over the arcs
//    give every other vertex the cell of a neighbour (a graph Voronoi diagram
//    in hops, level by level, so cells stay compact).
// 2. Merge (host): cells are joined along their most frequent borders, taken
//    from a sample of the border arcs, until a tile is full.  A few thousand
//    cells, whatever the graph's ids look like.
// 3. Layout: a tile's vertices sorted by cell and id; the arcs inside the tile in `slots` columns, the others in a list.
//
// A graph is left without tiles when its vertices have too many arcs for the
// columns, when too many arcs leave the cells or the tiles (graphs without
// locality: the messages would be the work), or when a border outgrows what a
// workgroup keeps in registers.
#include "gr_tile.h"

#include <algorithm>
#include <deque>
#include <vector>

#include "gr_device.h"

namespace gr {

namespace {

// Vertices per cell: fine cells fill the tiles better, coarse ones keep the
// host's merge short.
int32_t cell_verts(int32_t n) { return n > (1 << 15) ? 256 : 128; }
constexpr int kSweepBatch = 8;
constexpr int kMaxSweeps = 96;
constexpr int32_t kMaxPairs = 1 << 20;

// (the finalizer "lowbias32" of C. Wellons' hash-prospector)
__device__ __forceinline__ uint32_t hash32(uint32_t x) {
    x ^= x >> 16;
    x *= 0x7FEB352Du;
    x ^= x >> 15;
    x *= 0x846CA68Bu;
    return x ^ (x >> 16);
}

// A label: of a cell, -1 for none yet, and -2 - cell for a vertex of more than
// kCellHub arcs, which is in the cell but hands it on to nobody: its arcs lead
// anywhere, and a cell that grows from all of their ends fits no tile.
constexpr int32_t kCellHub = 16;
__device__ __forceinline__ int32_t hub_label(int32_t l, int32_t deg) { return l >= 0 && deg > kCellHub ? -2 - l : l; }

__global__ __launch_bounds__(256) void k_cell_seed(int32_t n, int32_t s, const int32_t *ro, int32_t *label) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= n) return;
    const int32_t b = (int32_t)(v / s), off = (int32_t)(v - (int64_t)b * s);
    const int32_t len = (int32_t)min((int64_t)s, n - (int64_t)b * s);
    const bool seed = off == (int32_t)(hash32((uint32_t)b) % (uint32_t)len);
    label[v] = seed ? hub_label(b, ro[v + 1] - ro[v]) : -1;
}

// One level: an unlabelled vertex takes a neighbour's label of the level before.
// left (optional): counts the vertices still unlabelled.
__global__ __launch_bounds__(256) void k_cell_sweep(int32_t n, const int32_t *ro, const uint2 *adj,
                                                    const int32_t *was, int32_t *now, uint32_t salt,
                                                    unsigned int *left) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int32_t l = 0;
    if (v < n) {
        l = was[v];
        if (l == -1) {
            const int32_t e0 = ro[v], d = ro[v + 1] - e0;
            int32_t at = d > 0 ? (int32_t)(hash32((uint32_t)v ^ salt) % (uint32_t)d) : 0;
            for (int32_t k = 0; k < d && l < 0; ++k) {
                l = was[adj[e0 + at].x];
                if (++at == d) at = 0;
            }
            l = l < 0 ? -1 : hub_label(l, d);
        }
        now[v] = l;
    }
    if (left) {
        const unsigned long long m = __ballot(v < n && l == -1);
        if ((threadIdx.x & 63) == 0 && m) atomicAdd(left, (unsigned int)__popcll(m));
    }
}

// Unreached vertices (other components) form cells by id; cell sizes.
__global__ __launch_bounds__(256) void k_cell_size(int32_t n, int32_t s, int32_t cells, int32_t *label,
                                                   unsigned int *size) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= n) return;
    int32_t l = label[v];
    if (l < 0) label[v] = l = l == -1 ? cells + (int32_t)(v / s) : -2 - l;
    atomicAdd(size + l, 1u);
}

// Border arcs between cells: their count (cnt[0]) and a sample of the cell
// pairs (cnt[1] of them; those past the capacity are dropped).
__global__ __launch_bounds__(256) void k_cell_border(int32_t n, const int32_t *ro, const uint2 *adj,
                                                     const int32_t *label, uint32_t sample_mask, uint2 *pairs,
                                                     unsigned int *cnt) {
    // (a block asks for its pairs' places at once: one by one, 0.74 ms of
    // atomics to one word on a mesh of 1024^2)
    __shared__ unsigned int sCut, sTake, sFirst;
    if (threadIdx.x == 0) sCut = sTake = 0u;
    __syncthreads();
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    unsigned int cut = 0, take = 0;
    const int32_t l = v < n ? label[v] : 0, e0 = v < n ? ro[v] : 0, e1 = v < n ? ro[v + 1] : 0;
    for (int32_t e = e0; e < e1; ++e) {
        if (label[adj[e].x] == l) continue;
        ++cut;
        take += (hash32((uint32_t)e) & sample_mask) == 0u ? 1u : 0u;
    }
    if (cut) atomicAdd(&sCut, cut);
    unsigned int at = take ? atomicAdd(&sTake, take) : 0u;
    __syncthreads();
    if (threadIdx.x == 0) {
        if (sCut) atomicAdd(cnt, sCut);
        sFirst = sTake ? atomicAdd(cnt + 32, sTake) : 0u;
    }
    __syncthreads();
    at += sFirst;
    for (int32_t e = e0; e < e1 && take; ++e) {
        const int32_t x = label[adj[e].x];
        if (x == l || (hash32((uint32_t)e) & sample_mask) != 0u) continue;
        if (at < (unsigned int)kMaxPairs) pairs[at] = make_uint2((uint32_t)l, (uint32_t)x);
        ++at;
        --take;
    }
}

__global__ __launch_bounds__(256) void k_tile_place(int32_t n, const int32_t *label, int32_t *cursor, int32_t *vid,
                                                    int32_t *pos) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= n) return;
    const int32_t p = atomicAdd(cursor + label[v], 1);
    vid[p] = (int32_t)v;
    pos[v] = p;
}

// One workgroup per tile: its vertices sorted by cell and id (a wave then owns
// a compact patch, and most waves are idle while a front crosses the tile).
__global__ __launch_bounds__(kTileThreads) void k_tile_sort(const int32_t *label, int32_t *vid, int32_t *pos) {
    __shared__ unsigned long long key[kTileVerts];
    const int t = threadIdx.x;
    const size_t base = (size_t)blockIdx.x << kTileShift;
    for (int i = t; i < kTileVerts; i += kTileThreads) {
        const int32_t v = vid[base + i];
        key[i] = v < 0 ? ~0ull : (unsigned long long)(uint32_t)label[v] << 32 | (uint32_t)v;
    }
    for (int k = 2; k <= kTileVerts; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            __syncthreads();
            for (int i = t; i < kTileVerts / 2; i += kTileThreads) {
                const int a = 2 * i - (i & (j - 1)), b = a + j;
                const unsigned long long x = key[a], y = key[b];
                if ((x > y) == ((a & k) == 0)) {
                    key[a] = y;
                    key[b] = x;
                }
            }
        }
    __syncthreads();
    for (int i = t; i < kTileVerts; i += kTileThreads) {
        const int32_t v = key[i] == ~0ull ? -1 : (int32_t)(uint32_t)key[i];
        vid[base + i] = v;
        if (v >= 0) pos[v] = (int32_t)(base + i);
    }
}

// One workgroup per tile.  FILL 0: the arcs inside (the first `slots` of each
// vertex) into the columns, and the number of the others; 1: the others.
template <int FILL>
__global__ __launch_bounds__(kTileThreads) void k_tile_arcs(int slots, uint32_t inf, const int32_t *ro,
                                                            const uint2 *adj, const int32_t *pos, const int32_t *vid,
                                                            uint32_t *w, uint16_t *head, int32_t *next, int32_t *nin,
                                                            const int32_t *ext_off, uint4 *ext) {
    __shared__ int sN;
    const int t = threadIdx.x;
    const int32_t tile = blockIdx.x;
    const size_t base = (size_t)tile << kTileShift;
    if (t == 0) sN = 0;
    __syncthreads();
    for (int i = t; i < kTileVerts; i += kTileThreads) {
        const int32_t v = vid[base + i];
        int used = 0, out = 0;
        if (v >= 0) {
            for (int32_t e = ro[v]; e < ro[v + 1]; ++e) {
                const uint2 a = adj[e];
                if (a.x == (uint32_t)v) continue;  // a self-loop never improves
                const int32_t p = pos[a.x], q = p >> kTileShift;
                const uint32_t l = (uint32_t)p & (kTileVerts - 1);
                if (q == tile && used < slots) {
                    if (FILL == 0) {
                        w[base * slots + (size_t)used * kTileVerts + i] = a.y;
                        head[(base * (slots / 2) + (size_t)(used / 2) * kTileVerts + i) * 2 + (used & 1)] = (uint16_t)(4 * l);
                    }
                    ++used;
                } else if (FILL == 0) {
                    ++out;
                    if (q != tile) atomicAdd(nin + q, 1);
                } else {
                    const int c = atomicAdd(&sN, 1);
                    ext[ext_off[tile] + c] = make_uint4((uint32_t)i, q == tile ? kTileInner | l : (uint32_t)q, l, a.y);
                }
            }
        }
        if (FILL == 0) {
            // empty slots offer INF to the vertex itself
            for (; used < slots; ++used) {
                w[base * slots + (size_t)used * kTileVerts + i] = inf;
                head[(base * (slots / 2) + (size_t)(used / 2) * kTileVerts + i) * 2 + (used & 1)] = (uint16_t)(4 * i);
            }
            if (out) atomicAdd(&sN, out);
        }
    }
    if (FILL == 0) {
        __syncthreads();
        if (t == 0) next[tile] = sN;
    }
}

// Sorts n <= kTileMaxExt keys in LDS (size: a power of two >= n, the keys past
// n all ones).
__device__ __forceinline__ void sort_keys(unsigned long long *key, int size) {
    for (int k = 2; k <= size; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            __syncthreads();
            for (int i = threadIdx.x; i < size / 2; i += kTileThreads) {
                const int a = 2 * i - (i & (j - 1)), b = a + j;
                const unsigned long long x = key[a], y = key[b];
                if ((x > y) == ((a & k) == 0)) {
                    key[a] = y;
                    key[b] = x;
                }
            }
        }
    __syncthreads();
}

// One workgroup per tile: its arcs of ext sorted by head's tile (those inside
// last), so that offers to one tile go out together; then listed with the
// tiles they enter.
__global__ __launch_bounds__(kTileThreads) void k_tile_ext_sort(const int32_t *ext_off, uint4 *ext, int32_t *in_cur,
                                                                uint2 *in) {
    __shared__ uint4 sE[kTileMaxExt];
    __shared__ unsigned long long key[4096];
    static_assert(kTileMaxExt <= 4096, "the list fits the sort");
    const int t = threadIdx.x;
    const int32_t e0 = ext_off[blockIdx.x], n = ext_off[blockIdx.x + 1] - e0;
    int size = 64;
    while (size < n) size <<= 1;
    for (int i = t; i < size; i += kTileThreads) {
        if (i < n) sE[i] = ext[e0 + i];
        // (head's tile, head, tail): one order, but for parallel arcs
        key[i] = i < n ? (unsigned long long)sE[i].y << 32 | (unsigned long long)sE[i].z << 19 |
                             (unsigned long long)(sE[i].x & 127u) << 12 | (unsigned long long)i
                       : ~0ull;
    }
    sort_keys(key, size);
    for (int i = t; i < n; i += kTileThreads) {
        const uint4 x = sE[(uint32_t)key[i] & 4095u];
        ext[e0 + i] = x;
        if (!(x.y & kTileInner)) in[atomicAdd(in_cur + x.y, 1)] = make_uint2((uint32_t)(e0 + i), x.z);
    }
}

// One workgroup per tile: the arcs that enter it, sorted by mail word.
__global__ __launch_bounds__(kTileThreads) void k_tile_in_sort(const int32_t *in_off, uint2 *in) {
    __shared__ unsigned long long key[4096];
    const int t = threadIdx.x;
    const int32_t e0 = in_off[blockIdx.x], n = in_off[blockIdx.x + 1] - e0;
    int size = 64;
    while (size < n) size <<= 1;
    for (int i = t; i < size; i += kTileThreads)
        key[i] = i < n ? (unsigned long long)in[e0 + i].x << 32 | in[e0 + i].y : ~0ull;
    sort_keys(key, size);
    for (int i = t; i < n; i += kTileThreads) in[e0 + i] = make_uint2((uint32_t)(key[i] >> 32), (uint32_t)key[i]);
}

// Joins the cells into tiles of at most kTileFill vertices: a tile grows by
// the neighbouring cell it shares most sampled border arcs with, among those
// that fit; the next tile starts beside the tiles made so far.  Returns the
// number of tiles, or -1 when a cell is too large or the graph has no locality.
int32_t merge_cells(const std::vector<unsigned int> &size, const std::vector<uint2> &pairs,
                    std::vector<int32_t> *tile_of) {
    const int32_t c = (int32_t)size.size();
    std::vector<int32_t> off((size_t)c + 1, 0), nb(2 * pairs.size());
    for (const uint2 &p : pairs) {
        ++off[p.x + 1];
        ++off[p.y + 1];
    }
    for (int32_t i = 0; i < c; ++i) off[i + 1] += off[i];
    {
        std::vector<int32_t> at(off.begin(), off.end() - 1);
        for (const uint2 &p : pairs) {
            nb[at[p.x]++] = (int32_t)p.y;
            nb[at[p.y]++] = (int32_t)p.x;
        }
    }
    // Cells of a mesh meet a few others along many arcs (6 to 20 along 64 and
    // more, each counted four times here), those of a random graph another one
    // with nearly every arc: where the sample has enough arcs per cell to tell,
    // the latter end here (uniform of 500,000 vertices and degree 3, whose cells
    // are trees with a third of their arcs on the border: created in 11.9 ms,
    // 8.2 so, 3.1 without trying).
    if ((int64_t)nb.size() >= 64 * (int64_t)c) {
        std::vector<int32_t> seen((size_t)c, -1);
        int64_t distinct = 0;
        for (int32_t i = 0; i < c; ++i)
            for (int32_t k = off[i]; k < off[i + 1]; ++k)
                if (seen[nb[k]] != i) {
                    seen[nb[k]] = i;
                    ++distinct;
                }
        if (5 * distinct > (int64_t)nb.size()) return -1;
    }
    tile_of->assign((size_t)c, -1);
    std::vector<int32_t> gain((size_t)c, 0), front, todo;
    std::vector<int64_t> fill;
    std::deque<int32_t> starts;
    auto grow = [&](int32_t s) {
        const int32_t t = (int32_t)fill.size();
        int64_t have = 0;
        front.clear();
        int32_t add = s;
        while (add >= 0) {
            (*tile_of)[add] = t;
            have += size[add];
            for (int32_t k = off[add]; k < off[add + 1]; ++k) {
                const int32_t x = nb[k];
                if ((*tile_of)[x] >= 0) continue;
                if (gain[x]++ == 0) front.push_back(x);
            }
            add = -1;
            int32_t best = 0;
            size_t keep = 0;
            for (const int32_t x : front) {
                if ((*tile_of)[x] >= 0) {
                    gain[x] = 0;
                    continue;
                }
                front[keep++] = x;
                if (gain[x] > best && have + size[x] <= kTileFill) {
                    best = gain[x];
                    add = x;
                }
            }
            front.resize(keep);
        }
        for (const int32_t x : front) {
            gain[x] = 0;
            starts.push_back(x);
        }
        fill.push_back(have);
    };
    for (int32_t i = 0; i < c; ++i) {
        if (size[i] > (unsigned)kTileFill) return -1;
        if (size[i] == 0 || (*tile_of)[i] >= 0) continue;
        starts.push_back(i);
        while (!starts.empty()) {
            const int32_t s = starts.front();
            starts.pop_front();
            if ((*tile_of)[s] < 0) grow(s);
        }
    }
    // small tiles join a neighbour they fit into, else any small one
    const int32_t nt = (int32_t)fill.size();
    std::vector<int32_t> into((size_t)nt);
    for (int32_t t = 0; t < nt; ++t) into[t] = t;
    std::vector<std::vector<int32_t>> cells((size_t)nt);
    for (int32_t i = 0; i < c; ++i)
        if ((*tile_of)[i] >= 0) cells[(*tile_of)[i]].push_back(i);
    std::vector<int32_t> links((size_t)nt, 0);
    int32_t spare = -1;
    for (int32_t t = 0; t < nt; ++t) {
        if (fill[t] * 2 > kTileFill) continue;
        todo.clear();
        for (const int32_t i : cells[t])
            for (int32_t k = off[i]; k < off[i + 1]; ++k) {
                const int32_t x = (*tile_of)[nb[k]];
                if (x == t || fill[x] == 0) continue;
                if (links[x]++ == 0) todo.push_back(x);
            }
        int32_t best = -1;
        for (const int32_t x : todo)
            if (fill[x] + fill[t] <= kTileFill && (best < 0 || links[x] > links[best])) best = x;
        for (const int32_t x : todo) links[x] = 0;
        if (best < 0 && spare >= 0 && spare != t && fill[spare] > 0 && fill[spare] + fill[t] <= kTileFill) best = spare;
        if (best < 0) {
            spare = t;
            continue;
        }
        for (const int32_t i : cells[t]) (*tile_of)[i] = best;
        cells[best].insert(cells[best].end(), cells[t].begin(), cells[t].end());
        cells[t].clear();
        fill[best] += fill[t];
        fill[t] = 0;
    }
    int32_t out = 0;
    for (int32_t t = 0; t < nt; ++t) into[t] = fill[t] > 0 ? out++ : -1;
    for (int32_t i = 0; i < c; ++i)
        if ((*tile_of)[i] >= 0) (*tile_of)[i] = into[(*tile_of)[i]];
    return out;
}

inline size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

// Stream-ordered scratch, freed on every path.
struct Temp {
    hipStream_t st;
    std::vector<void *> ptrs;
    ~Temp() {
        for (void *p : ptrs) (void)hipFreeAsync(p, st);
    }
    template <class T>
    hipError_t get(T **p, size_t count) {
        void *q = nullptr;
        const hipError_t e = hipMallocAsync(&q, std::max<size_t>(count, 1) * sizeof(T), st);
        if (e == hipSuccess) ptrs.push_back(q);
        *p = static_cast<T *>(q);
        return e;
    }
};

#define TRY(call)                          \
    do {                                   \
        const hipError_t _e = (call);      \
        if (_e != hipSuccess) return _e;   \
    } while (0)

}  // namespace

hipError_t tile_build(TileSet *out, int32_t n, int32_t m, const int32_t *ro, const uint2 *adj, int wt, int64_t over4,
                      int64_t over8, size_t limit, hipStream_t st) {
    *out = TileSet{};
    // four columns where nearly every vertex has at most four arcs, else eight
    // (an arc without a column is walked by the send pass)
    const int slots = over4 * 50 <= m ? 4 : 8;
    if (m < 1 || (slots == 8 && over8 * 50 > m)) return hipSuccess;
    const dim3 grid((unsigned)(((int64_t)n + 255) / 256)), blk(256);
    Temp tmp{st, {}};
    const int32_t s = cell_verts(n), cells = n <= kTileFill ? 1 : (int32_t)(((int64_t)n + s - 1) / s);
    int32_t *la = nullptr, *lb = nullptr, *cursor = nullptr;
    unsigned int *cnt = nullptr, *size = nullptr;
    uint2 *pairs = nullptr;
    TRY(tmp.get(&la, n));
    TRY(tmp.get(&lb, n));
    TRY(tmp.get(&size, 2 * (size_t)cells));
    TRY(tmp.get(&cnt, 64));
    std::vector<unsigned int> hsize((size_t)cells * 2, 0u);
    std::vector<int32_t> tile_of, hcur((size_t)cells * 2, 0);
    int32_t nt = 1;
    if (n <= kTileFill) {
        TRY(hipMemsetAsync(la, 0, sizeof(int32_t) * (size_t)n, st));
        hsize[0] = (unsigned)n;
    } else {
        TRY(tmp.get(&pairs, kMaxPairs));
        hipLaunchKernelGGL(k_cell_seed, grid, blk, 0, st, n, s, ro, la);
        unsigned int left = (unsigned)n, before = 0;
        for (int k = 0; k < kMaxSweeps && left > 0 && left != before; k += kSweepBatch) {
            before = left;
            TRY(hipMemsetAsync(cnt, 0, 256, st));
            for (int j = 0; j < kSweepBatch; ++j) {
                hipLaunchKernelGGL(k_cell_sweep, grid, blk, 0, st, n, ro, adj, la, lb, (uint32_t)(k + j) * 0x9E3779B9u,
                                   j == kSweepBatch - 1 ? cnt : nullptr);
                std::swap(la, lb);
            }
            TRY(hipMemcpyAsync(&left, cnt, sizeof left, hipMemcpyDeviceToHost, st));
            TRY(hipStreamSynchronize(st));
        }
        TRY(hipMemsetAsync(size, 0, sizeof(unsigned int) * 2 * (size_t)cells, st));
        TRY(hipMemsetAsync(cnt, 0, 256, st));
        hipLaunchKernelGGL(k_cell_size, grid, blk, 0, st, n, s, cells, la, size);
        uint32_t mask = 0;
        while ((int64_t)m / (8 * ((int64_t)mask + 1)) > kMaxPairs / 2) mask = mask * 2 + 1;
        hipLaunchKernelGGL(k_cell_border, grid, blk, 0, st, n, ro, adj, la, mask, pairs, cnt);
        unsigned int hc[64];
        TRY(hipMemcpyAsync(hc, cnt, sizeof hc, hipMemcpyDeviceToHost, st));
        TRY(hipMemcpyAsync(hsize.data(), size, sizeof(unsigned int) * hsize.size(), hipMemcpyDeviceToHost, st));
        TRY(hipStreamSynchronize(st));
        // cells of a mesh lose a tenth to a third of their arcs; those of a
        // random graph are trees, which hold half of four arcs per vertex and
        // less of more
        if ((int64_t)hc[0] * 20 > (int64_t)m * 9) return hipSuccess;
        std::vector<uint2> hp(std::min<unsigned int>(hc[32], (unsigned)kMaxPairs));
        if (!hp.empty()) {
            TRY(hipMemcpyAsync(hp.data(), pairs, sizeof(uint2) * hp.size(), hipMemcpyDeviceToHost, st));
            TRY(hipStreamSynchronize(st));
        }
        nt = merge_cells(hsize, hp, &tile_of);
        if (nt < 1 || nt > kTileMaxTiles || (int64_t)nt << kTileShift > INT32_MAX) return hipSuccess;
        std::vector<int32_t> fill((size_t)nt, 0);
        for (size_t i = 0; i < hsize.size(); ++i)
            if (hsize[i] > 0) {
                const int32_t t = tile_of[i];
                hcur[i] = (t << kTileShift) + fill[t];
                fill[t] += (int32_t)hsize[i];
            }
    }
    // one allocation for the layout up to the border arcs' list, whose length is not known yet
    const size_t places = (size_t)nt << kTileShift;
    const size_t b_pos = al256(sizeof(int32_t) * (size_t)n), b_vid = sizeof(int32_t) * places,
                 b_w = sizeof(uint32_t) * places * slots, b_h = b_w / 2,
                 b_off = al256(sizeof(int32_t) * ((size_t)nt + 1));
    const size_t b_ext = sizeof(uint4) * ((size_t)m / 5 + 1), b_in = sizeof(uint2) * ((size_t)m / 5 + 1);
    void *base = nullptr;
    const size_t bytes = b_pos + b_vid + b_w + b_h + 2 * b_off + b_ext + b_in;
    if (bytes > limit) return hipErrorOutOfMemory;
    TRY(hipMalloc(&base, bytes));
    struct Guard {
        void *p;
        ~Guard() {
            if (p) (void)hipFree(p);
        }
    } guard{base};
    TileSet ts;
    char *p = static_cast<char *>(base);
    ts.base = base;
    ts.bytes = bytes;
    ts.n = n;
    ts.ntiles = nt;
    ts.slots = slots;
    ts.pos = reinterpret_cast<int32_t *>(p);
    p += b_pos;
    ts.vid = reinterpret_cast<int32_t *>(p);
    p += b_vid;
    ts.w = reinterpret_cast<uint32_t *>(p);
    p += b_w;
    ts.head = reinterpret_cast<uint32_t *>(p);
    p += b_h;
    ts.ext_off = reinterpret_cast<int32_t *>(p);
    p += b_off;
    ts.in_off = reinterpret_cast<int32_t *>(p);
    p += b_off;
    ts.ext = reinterpret_cast<uint4 *>(p);
    p += b_ext;
    ts.in = reinterpret_cast<uint2 *>(p);
    int32_t *nb = nullptr;
    TRY(tmp.get(&nb, 2 * (size_t)nt));  // arcs that leave each tile, and that enter it
    TRY(tmp.get(&cursor, 2 * (size_t)cells));
    TRY(hipMemcpyAsync(cursor, hcur.data(), sizeof(int32_t) * hcur.size(), hipMemcpyHostToDevice, st));
    TRY(hipMemsetAsync(ts.vid, 0xFF, b_vid, st));
    TRY(hipMemsetAsync(nb, 0, sizeof(int32_t) * 2 * (size_t)nt, st));
    hipLaunchKernelGGL(k_tile_place, grid, blk, 0, st, n, la, cursor, ts.vid, ts.pos);
    const dim3 tg((unsigned)nt), tb(kTileThreads);
    const uint32_t inf = wt == 1 ? kInfF32 : kInfU32;
    hipLaunchKernelGGL(k_tile_sort, tg, tb, 0, st, la, ts.vid, ts.pos);
    hipLaunchKernelGGL((k_tile_arcs<0>), tg, tb, 0, st, slots, inf, ro, adj, ts.pos, ts.vid, ts.w,
                       reinterpret_cast<uint16_t *>(ts.head), nb, nb + nt, nullptr, nullptr);
    TRY(hipGetLastError());
    std::vector<int32_t> hn(2 * (size_t)nt), ioff((size_t)nt + 1, 0), eoff((size_t)nt + 1, 0);
    TRY(hipMemcpyAsync(hn.data(), nb, sizeof(int32_t) * hn.size(), hipMemcpyDeviceToHost, st));
    TRY(hipStreamSynchronize(st));
    int64_t ext = 0;
    for (int32_t i = 0; i < nt; ++i) {
        if (hn[i] > kTileMaxExt || hn[(size_t)nt + i] > kTileMaxExt) return hipSuccess;
        ext += hn[i];
        if (ext > (int64_t)m / 5) return hipSuccess;
        eoff[i + 1] = (int32_t)ext;
        ioff[i + 1] = ioff[i] + hn[(size_t)nt + i];
    }
    ts.mail = (int32_t)ext;
    TRY(hipMemcpyAsync(ts.ext_off, eoff.data(), sizeof(int32_t) * eoff.size(), hipMemcpyHostToDevice, st));
    TRY(hipMemcpyAsync(ts.in_off, ioff.data(), sizeof(int32_t) * ioff.size(), hipMemcpyHostToDevice, st));
    TRY(hipMemcpyAsync(nb, ts.in_off, sizeof(int32_t) * (size_t)nt, hipMemcpyDeviceToDevice, st));  // fill cursors
    hipLaunchKernelGGL((k_tile_arcs<1>), tg, tb, 0, st, slots, inf, ro, adj, ts.pos, ts.vid, nullptr, nullptr, nullptr,
                       nullptr, ts.ext_off, ts.ext);
    hipLaunchKernelGGL(k_tile_ext_sort, tg, tb, 0, st, ts.ext_off, ts.ext, nb, ts.in);
    hipLaunchKernelGGL(k_tile_in_sort, tg, tb, 0, st, ts.in_off, ts.in);
    TRY(hipGetLastError());
    TRY(hipStreamSynchronize(st));
    guard.p = nullptr;
    *out = ts;
    return hipSuccess;
}

}  // namespace gr
