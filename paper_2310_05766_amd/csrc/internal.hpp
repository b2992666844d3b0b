// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "../../include/tsdf.h"
#include "patch.hpp"
#include "ray.hpp"

namespace tsdf {

// ---------------------------------------------------------------------------
// Batched integration engine (batch.hip). Every integration, a single scan
// included, is a batch: scans (any maps, several per map allowed) whose rays
// are binned by (map tile, position of the scan among its map's scans in the
// batch); one workgroup per tile then applies the map's scans to that tile in
// submission order.
// ---------------------------------------------------------------------------

constexpr int kBinBlock = 256;   // default binning threads per block (one ray each); 128 and 512 also run
constexpr int kTileBlockDefault = 256;  // default tile workgroup size; 512 also runs
constexpr int kMaxEmit = 6;      // tiles per ray listed in LDS before taking positions (more go
                                  // straight to their runs)
constexpr int32_t kMaxTileGrid = 65536;
constexpr int32_t kMaxSeq = 64;  // scans of one map in one batch

struct MapDev {
    int16_t *sdf, *w;
    int32_t dims[3], origin[3], ring0[3];
    int32_t nt[3];
    uint32_t ntot;       // tiles of this map
    uint32_t tile_base;  // first global tile id of this map
    int32_t tau, w_max;
    int32_t vec_ok;      // 16-byte runs possible (see k_tile)
    int32_t pad;
};

struct ScanDev {
    RayParams rp;        // pose, scale, sensor position, tau
    const float *xyz;
    int64_t n;
    int32_t map;         // map slot in the batch
    int32_t seq;         // position among this map's scans in the batch
    uint32_t block0;     // first binning block of this scan
    Row row;             // final where there are no lengths to try; k_rows
    uint64_t rings;      // the lengths to try (row_rings), 0: none
};
constexpr PatchKind kBinPatch = {32, 32768, 3.5f};
// Where a band may cross more tiles than this, two binning passes take runs: what a
// ray has beyond kMaxEmit goes to its run by an atomic of its own, and the points of
// a patch meet in the same runs. 20 scans of 64 x 1024 and 128 x 1024 points into one
// map, us, patches / runs: at most 9 tiles, room 378 and 714 / 350 and 654, street 341
// and 493 / 354 and 519; 12 tiles, room 674 and 1378 / 575 and 1180, street 648 and
// 851 / 497 and 816; 17 tiles, street 1555 and 1752 / 1137 and 1709. (One pass, 128 x
// 1024 points, 17 tiles, room: 210 / 219.)
constexpr uint32_t kPatchTiles = 10;

struct BatchHdr {
    int32_t lt[3];
    int32_t S;           // sequence slots per tile (most scans of one map)
    int32_t G;           // sequence slots whose candidates a tile workgroup holds at once
    int32_t nmaps, nscans;
    uint32_t gtiles;     // sum of the maps' tile counts
    uint32_t nblocks;    // binning blocks of this batch
    uint32_t cap;        // entry capacity
    uint32_t want_stats;
    uint32_t bin_block;  // binning threads per block (one ray each)
    uint32_t key_shift;  // of the tile pass's 32-bit keys; 0: 64-bit keys
    uint32_t once, emit; // one binning pass (TileList); entries that a point can give
};

// The descriptors of a batch of one scan, handed to the first binning
// kernel as arguments: it reads them from there and stores them for the
// kernels after it, so that no copy precedes the launch (on = 0: the
// descriptors are in device memory already).
struct InlineDesc {
    BatchHdr hdr;
    MapDev map;
    ScanDev scan;
    uint32_t on;
    uint32_t pad[3];
};

constexpr int kQueues = 8;  // tile job queues, one per XCD (workgroup b runs on XCD b % 8)
// Words between two queue counters: each counter on a 128-byte line of its
// own, so that atomics on different queues do not meet in one line.
constexpr int kQueueStride = 32;

struct BatchCtl {
    uint32_t n_nonempty;  // busy tiles with heavy work, listed from the list's start
    uint32_t entries, overflow;
    uint32_t n_light;     // the other busy tiles, listed from the list's end
    uint32_t turn, next_turn;  // of ctl[0] (once_ctl)
    uint32_t pad[26];
    uint32_t work[kQueues * kQueueStride];  // next job of queue q: work[q * kQueueStride]
};

// The entries of a tile where each map has one scan (one binning pass): every
// binning block writes its entries, tile by tile, into a region of its own and
// adds a segment of them to each tile it met. The first kSegs segments lie in
// the list itself, the others in kChains chains of nodes in turn, which one wave
// follows together. All zero between batches (segments may hold anything).
// (Their counters are ctl[1] and ctl[2] in turn, ctl[0] being those of two
// binning passes: a tile pass clears the next batch's. The turn is kept on the
// device, so that a launch that a caller captured finds cleared counters at every
// replay: binning goes by ctl[0].next_turn and leaves it in ctl[0].turn, which the
// tile pass goes by; it then sets next_turn.)
constexpr uint32_t kSegs = 7, kChains = 16;
struct TileList {
    uint32_t nseg, total;   // segments, entries (one 64-bit counter)
    uint2 seg[kSegs];       // first entry, entries
    uint32_t chain[kChains];  // first node + 1, 0: none
};
static_assert(sizeof(TileList) == 128, "a line per tile");
// Nodes (next + 1, first entry, entries, -) of a block: one per slot of its
// table, one per entry that found the table full.
__host__ __device__ inline uint32_t nodes_per_block(uint32_t bin_block, uint32_t emit) { return bin_block * (2u + emit); }
// Per-scan counts of one binning pass: kStatParts lines of 64 bytes per scan, each
// (updated, visits) as one 64-bit counter that the tile pass adds to, and in the
// first line the valid points as its third word. (A kernel that sums over the
// tiles afterwards took 11.8 us for one scan, and the copy of its result to
// pageable memory 9 us more than to pinned memory.)
constexpr uint32_t kStatParts = 8, kStatWords = kStatParts * 16;
constexpr uint64_t kOnceBlocks = 65536;  // binning blocks of a batch that is binned in one pass, at most

// Device addresses of one engine (all inside buffers the engine owns).
struct BatchArrays {
    BatchHdr *hdr;
    MapDev *maps;
    ScanDev *scans;
    uint32_t *block_scan;  // [nblocks] scan of each binning block
    int4 *seq_sensor;      // [nmaps * S] sensor position (fixed point) and tau of the scan at (map, seq)
    uint32_t *counts;      // [S * gtiles] entries per (seq, tile), seq-major; zero between batches
    uint32_t *offsets;     // [S * gtiles] start of each run
    uint32_t *cursor;      // [S * gtiles] fill position
    uint32_t *tile_vis;    // [S * gtiles] visits per (seq, tile), when stats are wanted
    uint32_t *tile_upd;    // [S * gtiles] voxels updated per (seq, tile)
    uint4 *jobs;           // [gtiles] busy tiles: (global tile, map slot, busy sequence slots as a 64-bit mask)
    uint4 *entries;        // [cap] (point index, q.x, q.y, q.z), by tile then seq
    uint4 *entries2;       // [cap] (r, packed band offsets, crossing counts at tile entry, sequence slot)
    uint32_t *valid_part;  // [nblocks] points with a ray per binning block
    uint32_t *scan_stats;  // [nscans * 4] updated, valid, visits, overflow; one binning pass: [nscans * kStatWords]
    BatchCtl *ctl;
    TileList *lists;       // [gtiles], one binning pass
    uint4 *nodes;          // [nblocks * nodes_per_block], one binning pass
};

// A scan's row among the lengths to try (patch.hpp). A whole wave calls.
__device__ __forceinline__ Row find_row(const float *xyz, int64_t n, uint64_t rings, const PatchKind &kind)
{
    const uint32_t lane = __lane_id(), j = lane / kRowSamples, mine = ring_at(rings, j);
    bool counts = false, fits = false;
    if (mine) {
        const float *a = xyz + 3 * row_sample(n, lane % kRowSamples), *b = a + 3 * (int64_t)((uint32_t)n / mine), *c = a + 3 * kRowSpan;
        const float pa[3] = {a[0], a[1], a[2]}, pb[3] = {b[0], b[1], b[2]}, pc[3] = {c[0], c[1], c[2]};
        row_vote(pa, pb, pc, kind.step, counts, fits);
    }
    const uint64_t lanes = ((1ull << kRowSamples) - 1) << (j * kRowSamples);
    const int nc = __popcll(__ballot(counts) & lanes), nf = __popcll(__ballot(fits) & lanes);
    const uint64_t ok = __ballot(row_fits(nc, nf));
    if (!ok) return Row{0, 0, 0};
    const uint32_t r = ring_at(rings, (uint32_t)__builtin_ctzll(ok) / kRowSamples);
    return row_of((uint32_t)n / r, r, kind);
}
// A row held alike by all lanes, in scalar registers.
__device__ __forceinline__ Row uniform_row(const Row &row)
{
    return Row{(uint32_t)__builtin_amdgcn_readfirstlane((int)row.length), (uint32_t)__builtin_amdgcn_readfirstlane((int)row.end),
               (uint32_t)__builtin_amdgcn_readfirstlane((int)row.inverse)};
}

// Upper bound of the tiles one ray's band can fall in.
int32_t max_tiles_per_ray(int32_t tau, const int32_t lt[3]);

// Grid sizes of one launch. Every grid is sized from these capacities and
// the kernels read the batch's real sizes from the header, so a captured
// graph serves every batch that fits them.
struct LaunchCaps {
    uint32_t blocks;      // binning blocks
    uint32_t gtiles;      // global tiles
    uint32_t scans;       // scans
    int32_t tile_grid;    // tile workgroups
    uint32_t tile_lds;    // dynamic LDS bytes of a tile workgroup
    uint32_t bin_block;   // binning threads per block: 128, 256 or 512
    uint32_t tile_block;  // tile workgroup size: 256 or 512
    uint32_t stats;       // per-scan counts wanted: k_stats runs only then
    uint32_t key32;       // 32-bit keys in the tile pass
    uint32_t once;        // one binning pass
    uint32_t rows;        // scans that may have rows: k_rows runs only then
};

// The tile pass's LDS and grid for a tiling, S sequence slots, a truncation and
// the points of the largest scan.
constexpr int kMaxGroup32 = 16, kMaxGroup64 = 8;  // sequence slots a tile workgroup holds at once, by key size
constexpr int kTileStaticLds = 1792;              // k_tile's fixed tables
// Waves per SIMD of the tile pass: its registers would allow seven, but fewer
// LDS bytes per workgroup mean fewer slots per group (5, 6, 7 waves on 50 scans
// of 128 x 1024 points: 267, 264, 268 us; on 64 uneven scans into 16 maps: 331,
// 326, 339; on 32 small scans into 32 maps: 107, 97, 95).
constexpr int kTileWaves = 6;
struct TilePlan {
    uint32_t key_shift;  // 0: 64-bit keys
    int32_t G;
    uint32_t lds;        // dynamic LDS bytes of a workgroup
    int32_t grid;        // workgroups that fill the device
};
TilePlan tile_plan(const int32_t lt[3], int32_t S, int32_t tau, int64_t max_points, int32_t tile_block, int32_t cus);

// The block sizes the kernels are built for.
bool launch_blocks_ok(int32_t bin_block, int32_t tile_block);

// Events recorded (when non-null) after binning and after the tile pass,
// for per-stage timing. inl (when non-null, with on = 1): the descriptors of
// a one-scan batch, stored by the first kernel instead of copied before.
hipError_t launch_batch(const BatchArrays &B, const LaunchCaps &caps, hipStream_t stream, hipEvent_t ev_start,
                        hipEvent_t ev_binned, hipEvent_t ev_tiles, const InlineDesc *inl = nullptr);
hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t stream);

// One scan through the global key volume (interp.hip): with vertical
// interpolation between scan lines (dq > 0), or with free-space carving.
struct InterpScan {
    RayParams rp;
    const float *xyz;  // device points
    int64_t n;
    int64_t dq;        // delta_z of Eq. (3) in 1/2^20 units (0 with carving)
    int64_t up[3];     // the sensor's up vector in 1/1024 units
    int32_t carve;     // walk each ray longer than tau from the sensor as well
    int32_t origin[3], dims[3];
    int32_t ring0[3];  // floor_mod(origin, dims): the slot of the window's first voxel
    int16_t *sdf, *w;
    int32_t w_max;
    unsigned long long *keys;      // [nx*ny*nz] per-scan keys, all EMPTY between scans
    uint8_t *touched;              // [ceil(nx*ny*nz / 64)] runs of 64 slots with a key, all 0 between scans
    // 32-bit keys (key_shift of key32_shift, 0: 64-bit ones): keys32 in the key
    // volume's first half, all ~0 between scans, and carving's marks, a byte per
    // voxel of the window (not of the ring), padded to 4096, all ~0 between scans
    uint32_t key_shift;
    uint32_t *keys32;
    uint8_t *marks;
    Row row;                       // as in ScanDev
    uint64_t rings;
    Row *found;                    // from the band's kernel to the free space's
    int32_t want_stats;            // count valid points, visits and voxels updated
    unsigned long long *counters;  // [kinds][kCtrLines * kCtrStride], added to
};
enum { kCtrValid = 0, kCtrVisits = 1, kCtrUpdated = 2, kCtrAtomics = 3, kCtrKinds = 4 };
constexpr uint32_t kCtrLines = 64, kCtrStride = 16;  // counters of a kind, and words from one to the next
constexpr size_t kCtrWords = (size_t)kCtrLines * kCtrStride;
constexpr PatchKind kKeyPatch = {8, 8192, 6.0f};
// Bytes of a key volume: 64-bit keys, or 32-bit keys and marks.
inline size_t key_marks_offset(int64_t nvox) { return ((size_t)nvox * 4 + 255) / 256 * 256; }
inline size_t key_marks_bytes(int64_t nvox) { return ((size_t)nvox + 4095) / 4096 * 4096; }
inline size_t key_volume_bytes(int64_t nvox)
{
    const size_t narrow = key_marks_offset(nvox) + key_marks_bytes(nvox);
    return (size_t)nvox * 8 > narrow ? (size_t)nvox * 8 : narrow;
}
hipError_t launch_interp(const InterpScan &P, int64_t nvox, hipStream_t stream);

// Point-to-TSDF registration (register.hip).
constexpr int kRegSums = 29;       // H upper triangle (21), J^T r (6), sum r^2, points used
constexpr int kRegRow = 32;        // the same, padded
constexpr int kRegMaxBlocks = 256;  // more points than 256 blocks hold: several per thread
constexpr int kRegFan = 16;        // blocks per arrival counter
// Device memory of a map's registrations (zeroed once; every run leaves the
// counters at zero).
struct RegWork {
    double M[12];  // the next launch's pose
    double step;   // norm of the last step
    int32_t it, stop;
    uint32_t root, pad;
    uint32_t ticket[32 * (kRegMaxBlocks / kRegFan)];  // each counter on a 128-byte line of its own
    double rows[kRegMaxBlocks * kRegRow];
};
// Pinned host memory the last evaluation of a run writes.
struct RegResult {
    double M[12], sums[kRegSums], step;
    int32_t it, done;
};
struct RegArgs {
    double M[12];      // the first launch's pose, rows 0..2
    const float *xyz;  // device points
    int64_t n;
    const int16_t *sdf, *w;
    int32_t dims[3], origin[3];
    int32_t ring0[3];  // floor_mod(origin, dims)
    int32_t tau;
    int32_t first, last;
    double vs, damping;
    RegWork *work;
    RegResult *result;
};
hipError_t launch_reg_step(const RegArgs &A, hipStream_t stream);

// Surface extraction of a box of the window (mesh.hip).
constexpr uint32_t kMeshUnit = 16;  // groups of rows of cubes per workgroup
struct MeshArgs {
    const int16_t *sdf, *w;
    int32_t dims[3];  // the window (slot = floor_mod(g, dims))
    int32_t lo[3];    // first cube's voxel
    int32_t s0[3];    // its slot per axis
    int32_t n[3];     // cubes per axis
    uint32_t nrows;   // n[0] * n[1]
    // a wave takes a group of 64 >> lseg rows of up to 2^lseg voxels side by side,
    // where they are that short, else (lseg 6) one row
    int32_t lseg;
    uint32_t groups;
    double vs;        // voxel size, metres
};
void mesh_groups(MeshArgs &A);  // lseg and groups, from the rest
inline uint32_t mesh_units(const MeshArgs &A) { return (A.groups + kMeshUnit - 1) / kMeshUnit; }
// Triangles per group of rows and per unit of kMeshUnit groups.
hipError_t launch_mesh_count(const MeshArgs &A, uint32_t *group_tris, uint32_t *unit_tris, hipStream_t stream);
// Triangles of `units` units from unit0 on; unit_base: exclusive prefix of
// unit_tris, with the total behind it; base: the first unit's.
hipError_t launch_mesh_emit(const MeshArgs &A, const uint32_t *group_tris, const uint64_t *unit_base, uint32_t unit0,
                            uint32_t units, uint64_t base, float *out, hipStream_t stream);

// ---------------------------------------------------------------------------
// Host-side store of 64^3-voxel chunks that left the window.
// ---------------------------------------------------------------------------
constexpr int kChunk = 64;
constexpr int64_t kChunkVox = (int64_t)kChunk * kChunk * kChunk;

struct ChunkKey {
    int32_t x, y, z;
    bool operator==(const ChunkKey &o) const { return x == o.x && y == o.y && z == o.z; }
};
struct ChunkKeyHash {
    size_t operator()(const ChunkKey &k) const
    {
        uint64_t h = (uint64_t)(uint32_t)k.x * 0x9E3779B97F4A7C15ull;
        h ^= (uint64_t)(uint32_t)k.y * 0xC2B2AE3D27D4EB4Full + (h << 6) + (h >> 2);
        h ^= (uint64_t)(uint32_t)k.z * 0x165667B19E3779F9ull + (h << 6) + (h >> 2);
        return (size_t)h;
    }
};
// A chunk of the host store: kChunkVox sdf values then kChunkVox weights,
// [x][y][z] z fastest, in pinned host memory (a buffer of the map's chunk
// pool), so that a whole chunk crosses the host link in one copy.
struct Chunk {
    int16_t *buf = nullptr;
    int16_t *sdf() const { return buf; }
    int16_t *w() const { return buf + kChunkVox; }
};

// A box of voxels copied between the window and a dense staging buffer:
// global box [lo, lo + ext), staged at `off` (elements) as [x][y][z].
struct BoxXfer {
    int32_t lo[3];
    int32_t ext[3];
    int64_t off;
};
// Slot of a global voxel: floor_mod(g, dims) per axis.
// pack: stage <- window, whose voxels are reset to 0;
// unpack: window <- stage, or <- 0 when stage_sdf is null.
hipError_t launch_pack_boxes(const BoxXfer *boxes_dev, int32_t nboxes, int64_t max_box_vox, int16_t *sdf,
                             int16_t *w, const int32_t dims[3], int16_t *stage_sdf, int16_t *stage_w, hipStream_t stream);
// Lines [line0, line0 + lines) of a box of the window, line = x * ny + y, nz
// voxels each: out gets their sdf values, then their weights, both dense.
struct LinesXfer {
    const int16_t *sdf, *w;
    int32_t dims[3];  // the window
    int32_t s0[3];    // slot of the box's first voxel per axis
    uint32_t ny, nz;  // the box
};
hipError_t launch_pack_lines(const LinesXfer &A, uint32_t line0, uint32_t lines, int16_t *out, hipStream_t stream);
// Whole chunks of a window whose dims are multiples of 64 (lo[j]: the chunk's
// global origin), staged chunk by chunk in the store's layout
// (stage + j * 2 * kChunkVox: sdf, then w). pack clears the window voxels and
// sets flags[j] (pinned host memory, zero beforehand) when chunk j holds a
// non-zero voxel. move copies staged chunks at[j] to (out) or from their pinned
// host buffers host[j].
constexpr int kShiftChunks = 16;  // one chunk layer of a 512 x 512 x 128 window
struct ChunkList {
    int32_t lo[kShiftChunks][3];
};
struct ChunkPtrs {
    int16_t *host[kShiftChunks];
    int32_t at[kShiftChunks];
};
hipError_t launch_pack_chunks(const ChunkList &C, int32_t nchunks, int16_t *sdf, int16_t *w, const int32_t dims[3],
                              int16_t *stage, uint32_t *flags, hipStream_t stream);
hipError_t launch_move_chunks(const ChunkPtrs &P, int32_t nchunks, int16_t *stage, bool out, hipStream_t stream);
hipError_t launch_unpack_chunks(const ChunkList &C, int32_t nchunks, int16_t *sdf, int16_t *w, const int32_t dims[3],
                                const int16_t *stage, hipStream_t stream);
hipError_t launch_unpack_boxes(const BoxXfer *boxes_dev, int32_t nboxes, int64_t max_box_vox, int16_t *sdf,
                               int16_t *w, const int32_t dims[3], const int16_t *stage_sdf,
                               const int16_t *stage_w, hipStream_t stream);

}  // namespace tsdf
