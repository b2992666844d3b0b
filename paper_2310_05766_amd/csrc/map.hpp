// The map object behind the C ABI's opaque tsdf_map, shared by the
// library's translation units (runtime.hip holds its calls).
#pragma once

#include <atomic>
#include <memory>

#include "engine.hpp"

struct tsdf_map {
    tsdf_map_desc d;
    int64_t nvox = 0;
    double scale = 0.0;
    int16_t *sdf = nullptr, *w = nullptr;
    bool own_arrays = false;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    int device = 0;
    int32_t lt[3] = {0, 0, 0};  // integration tiling; {0, 0, 0}: chosen per call
    int32_t tile_grid = 0;      // 0: as many workgroups as fit the device
    int32_t bin_block = 0;      // binning threads per block; 0: the default
    int32_t tile_block = 0;     // tile workgroup size; 0: the default
    std::unique_ptr<tsdf::Engine> engine;  // single-scan integration on the map's stream
    // vertical interpolation between scan lines, or free-space carving (their
    // own path through a key volume over the window, interp.hip)
    int64_t interp_dq = 0;                     // delta_z of Eq. (3), 1/2^20 units; 0: off
    bool carve = false;                        // rays longer than tau walked from the sensor
    unsigned long long *interp_keys = nullptr;  // key volume, all ~0 between scans
    uint8_t *interp_touched = nullptr;          // [ceil(nvox / 64)], 0 between scans
    unsigned long long *interp_ctr = nullptr;   // device counters (kCtrKinds * kCtrWords)
    unsigned long long *interp_ctr_host = nullptr;
    int64_t atomics_seen = 0;                   // atomics counted up to the last tsdf_map_key_atomics
    float *interp_pts = nullptr;                // device copy of host points
    int64_t interp_pts_cap = 0;                 // points
    // registration: device state and rows of sums, pinned result
    tsdf::RegWork *reg_work = nullptr;
    tsdf::RegResult *reg_result = nullptr;
    // surface extraction: triangle counts and places, device and pinned host;
    // device triangles on their way out (two pieces at most)
    void *mesh_dev = nullptr, *mesh_host = nullptr, *mesh_tris = nullptr;
    size_t mesh_dev_cap = 0, mesh_host_cap = 0, mesh_tris_cap = 0;
    bool meshed = false;  // a mesh has left without staging
    // shift / readback / mesh staging
    int16_t *stage_dev = nullptr;  // [2][stage_cap]
    int16_t *stage_host = nullptr;
    int64_t stage_cap = 0;  // voxels per array
    tsdf::BoxXfer *boxes_dev = nullptr;
    tsdf::BoxXfer *boxes_host = nullptr;
    int32_t boxes_cap = 0;
    // whole-chunk shifts: device staging of kShiftChunks chunks leaving and
    // kShiftChunks entering, per-chunk non-zero flags (pinned host), and a
    // second stream for the copies into the window, so that both directions of
    // the host link run together
    int16_t *cstage_dev = nullptr;
    uint32_t *cflags_host = nullptr;
    hipStream_t copy_stream = nullptr;
    hipEvent_t copy_done = nullptr;
    // the store's chunk buffers: pinned host slabs cut into 1 MiB chunks
    std::vector<void *> pool_slabs;
    std::vector<int16_t *> pool_free;
    // per-kernel event timing (pack, unpack)
    bool prof_on = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> prof_ev[TSDF_KERNEL_COUNT];
    std::vector<hipEvent_t> ev_pool;
    // state
    bool poisoned = false;
    std::atomic<int> busy{0};
    std::unordered_map<tsdf::ChunkKey, tsdf::Chunk, tsdf::ChunkKeyHash> store;
};

namespace tsdf {

// One host thread per map: a call holds the map's busy flag while it runs.
struct Guard {
    tsdf_map *m;
    bool ok;
    explicit Guard(tsdf_map *mm) : m(mm), ok(false)
    {
        int expected = 0;
        ok = m->busy.compare_exchange_strong(expected, 1);
    }
    ~Guard()
    {
        if (ok) m->busy.store(0);
    }
};


// Tiles of 2^lt voxels: every lt in [2, 6], the z edge at least 8 (merge
// runs), 2^9..2^12 voxels per tile (12 bytes of LDS per voxel).
// Tilings used while a map has none set. A larger tile has fewer fixed costs per
// scan, a smaller one holds more scans' keys at once and spreads a scan over more
// workgroups. What decides is how many tiles are busy, which the host cannot
// know; it goes by the most scans that one map has in the call, by its points and
// by the windows' voxels. Whole calls, us (16x16x16, 16x16x8, 16x8x8, 8x8x8 voxels;
// * the rule's; S: 64 mm street in 512 x 512 x 256, R: 80 mm room in 256^3, D: 200 mm
// room in 128 x 128 x 64; the first line's rule is that of plain calls, which also
// keeps the allocation-free call's tables small):
//   1 scan    1 map, 128 x 1024       S   26   27*  30   33   R   57   43*  43   40
//             4 maps, 64 x 1024       S   75*  76   87  107   R   71*  67   68   72
//             24 maps, 16 x 1024      S  103* 128  131  149   D   92*  91   91   90
//             6 maps, 128 x 1024      S  118* 117  115  117   D  230  231  163  159*
//             2 maps, 64 x 1024       R   63   62*  63   62   D  106  106   80*  74
//             1 map, 128 x 1024       (in a batch)            D   -   113  100   70*
//   2 scans   1 map, 128 x 1024       S   78   71   71*  75   R  125   92   89*  88
//   4 scans   4 maps, 64 x 1024       S  328  306  291* 319   R  181  161  157* 161
//             16 maps, uneven         R  501  463  489* 536
//             1 map, 128 x 1024       S  129  115  109* 116   R  188  131  124  110*
//   8 scans   1 map, 128 x 1024       S  210  172  158* 163   R  329  222  212  180*
//             16 maps, 32 x 1024      R  508  453  467* 505
//   3 scans   1 map, 128 x 1024       D  277  264  212  163*
// One scan per map of more than kManyPoints points together takes the largest
// tiles, the busy ones being many then, unless the windows are dense, a point for
// every 32 voxels or more (8: very dense; 64 where scans are large): few tiles, with
// many entries each. A point for 64, 100 mm room: 6 maps, 128 x 1024 144, 138, 114,
// 115 us; 32 maps, 16 x 1024 106, -, 117, -.
// (Where the best is not taken, up to 6 % on many maps of 4 and 8 scans, no figure
// that the host has tells that line from the next.)
inline constexpr int32_t kScanTiling[3] = {4, 4, 3};
inline constexpr int32_t kManyScansTiling[3] = {4, 4, 4};
inline constexpr int32_t kFewSeqTiling[3] = {4, 3, 3};
inline constexpr int32_t kBatchTiling[3] = {3, 3, 3};
inline constexpr int64_t kManyPoints = 131072, kLargeScan = 65536;
inline constexpr int32_t kFewSeq = 8;

// seq: the most scans of one map in the call; points: of all its scans; maps, and
// voxels of their windows (0, 0, 0: a plain call).
inline const int32_t *tiling_for(const tsdf_map *m, int32_t seq, int64_t points, int64_t maps, int64_t voxels)
{
    if (m->lt[0] != 0) return m->lt;
    const auto dense = [&](int64_t voxels_per_point) { return voxels > 0 && points >= voxels / voxels_per_point; };
    if (seq > 1) return seq <= kFewSeq && !dense(32) ? kFewSeqTiling : kBatchTiling;
    if (dense(8)) return kBatchTiling;
    if (dense(32) || (dense(64) && points > kLargeScan * maps)) return kFewSeqTiling;
    return points > kManyPoints ? kManyScansTiling : kScanTiling;
}

// The launch shape of an integration on this map (a batch takes its first
// scan's map's).
inline LaunchShape launch_shape(const tsdf_map *m, int32_t seq, int64_t points, int64_t maps, int64_t voxels)
{
    LaunchShape sh;
    const int32_t *lt = tiling_for(m, seq, points, maps, voxels);
    for (int a = 0; a < 3; ++a) sh.lt[a] = lt[a];
    sh.tile_grid = m->tile_grid;
    sh.bin_block = m->bin_block > 0 ? m->bin_block : kBinBlock;
    sh.tile_block = m->tile_block > 0 ? m->tile_block : kTileBlockDefault;
    return sh;
}

}  // namespace tsdf
