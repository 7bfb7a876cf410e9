// Tiled asynchronous loop for mesh-like graphs (declarations; see
// gr_tile.hip for the kernels and gr_tile_build.hip for the layout).
//
// The vertices are cut into tiles of at most kTileFill that hold most arcs
// inside; a workgroup runs one tile to its local fixed point with the
// distances in LDS and the arcs in registers, and tiles trade improvements
// through one mail word per arc between them.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace gr {

constexpr int kTileThreads = 1024;
constexpr int kTileVpt = 4;  // vertices per thread
constexpr int kTileShift = 12;
constexpr int kTileVerts = 1 << kTileShift;
static_assert(kTileThreads * kTileVpt == kTileVerts, "a workgroup covers a tile's places");
// The last two waves carry offers in and out and hold no vertices: the places
// that the others cover are filled.
constexpr int kTileWaves = kTileThreads / 64 - 2;
constexpr int kOutWave = kTileWaves, kInWave = kTileWaves + 1;
constexpr int kTileFill = kTileWaves * 64 * kTileVpt;
// Arcs that leave a tile (or find no slot inside), and arcs that enter it from
// other tiles, at most (held in LDS).
constexpr int kTileMaxExt = 3072;

// The tiled layout of a graph (one device allocation, `base`).  A vertex's
// place is tile << kTileShift | local.  Thread t of a workgroup owns the
// places tile_place(t, i): each wave a run of 256 consecutive ones.
__host__ __device__ inline int tile_place(int t, int i) { return t * kTileVpt + i; }
struct TileSet {
    void *base = nullptr;
    size_t bytes = 0;
    int32_t ntiles = 0;
    int32_t slots = 0;  // arc slots per vertex: 4 or 8
    int32_t n = 0;
    int32_t mail = 0;  // mail words: one per arc of ext
    int32_t *pos = nullptr;      // [n] place of each vertex
    int32_t *vid = nullptr;      // [ntiles][kTileVerts] vertex at each place, -1 past the end
    uint32_t *w = nullptr;       // [ntiles][slots][kTileVerts] weight bits
    uint32_t *head = nullptr;    // [ntiles][slots / 2][kTileVerts] two local heads, as 16-bit byte offsets
    uint4 *ext = nullptr;        // the other arcs by tail's tile, sorted by head's: (local tail, head's tile or
                                 // kTileInner | local head, 0, weight)
    int32_t *ext_off = nullptr;  // [ntiles + 1]
    uint2 *in = nullptr;         // the arcs of ext that enter each tile: (arc = mail word, local head)
    int32_t *in_off = nullptr;   // [ntiles + 1]
};
constexpr uint32_t kTileInner = 0x80000000u;

// Builds the layout of a CSR (device arrays, arcs (head, weight bits)) whose
// maximum degree is at most kTileMaxDegree: what a tile's list of other arcs
// holds.  (A few vertices of many arcs do no harm: mesh 1024^2 with a hub of 80
// arcs 0.3 ms against 10 over in-arcs by weight, with one of 2,000 0.2 against 3
// in rounds.)  *out stays empty (ntiles = 0) when the graph does not cut into tiles (see gr_tile_build.hip); over4 / over8:
// arcs beyond the fourth / eighth of their vertex; limit: bytes that the layout
// may take (past them hipErrorOutOfMemory).
constexpr int32_t kTileMaxDegree = kTileMaxExt;
hipError_t tile_build(TileSet *out, int32_t n, int32_t m, const int32_t *ro, const uint2 *adj, int wt, int64_t over4,
                      int64_t over8, size_t limit, hipStream_t st);

// One query of a launch.
struct TileJob {
    const int32_t *pos;
    const int32_t *vid;
    const uint32_t *w;
    const uint32_t *head;
    const uint4 *ext;
    const int32_t *ext_off;
    const uint2 *in;
    const int32_t *in_off;
    uint32_t *dist;   // the query's output, n values
    uint32_t *mail;   // workspace: the lowest offer along each arc of ext
    uint32_t *flags;  // workspace: one word per tile, kTileFlagStride apart
    int32_t n, ntiles, nmail, src;
};
constexpr int kTileFlagStride = 16;
constexpr int kTileMaxJobs = 64;
constexpr int kTileMaxTiles = 1 << 24;  // a queue entry packs (query, tile) in 30 bits
// Statistics words the kernel writes to stat (pinned host memory): status (1
// done, 3 a wait timed out), arcs relaxed (with count), vertex expansions.
constexpr int kTileStatWords = 3;

// Workspace bytes of a launch over these queries' layouts, and the launch: a
// workgroup per compute unit, or per tile if there are fewer.  wt: 0 uint32, 1
// binary32, 2 unit steps; all layouts have the same number of slots; count:
// whether the arcs are counted.
size_t tile_ws_bytes(const TileSet *const *sets, int32_t k);
// A query's share: the sum over a launch's is at least its tile_ws_bytes.
size_t tile_query_bytes(const TileSet &set);
hipError_t launch_tiles(const TileSet *const *sets, const int32_t *srcs, uint32_t *const *dist, int32_t k, int wt,
                        void *ws, int num_cu, uint64_t spin_ticks, bool count, unsigned long long *stat, hipStream_t st);

}  // namespace gr
