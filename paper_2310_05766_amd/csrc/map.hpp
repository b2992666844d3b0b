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
// Tilings used while a map has none set, by the most scans that one map has in
// the call. A larger tile has fewer fixed costs per scan, a smaller one holds
// more scans' keys at once; the tile pass's time, us (tiles of 8x8x8, 16x8x8,
// 16x16x8, 16x16x16 voxels):
//   1 scan    32 maps, 16 x 1024 points each     153 122 110  96
//             4 maps, 64 x 1024                   61  62  60  61
//             1 map, 128 x 1024                   41  36  33  37
//             1 map, 16 x 1024                    17  17  16  19
//   2 scans   1 map, 128 x 1024                   76  69  68  75
//   4 scans   16 maps, uneven                    665 605 567 608
//             4 maps, 64 x 1024                  128 120 129 145
//   8 scans   1 map, 128 x 1024                  147 145 158 191
//             16 maps, 32 x 1024                 466 430 416 473
//   16 scans  4 maps, 64 x 1024                  259 262 293 378
//   50 scans  1 map, 128 x 1024                  502 517 583 817
// (whole calls). One scan per map of more than kManyPoints points together
// takes the largest tiles: the busy tiles are then many more than workgroups.
inline constexpr int32_t kScanTiling[3] = {4, 4, 3};
inline constexpr int32_t kManyScansTiling[3] = {4, 4, 4};
inline constexpr int32_t kFewSeqTiling[3] = {4, 3, 3};
inline constexpr int32_t kBatchTiling[3] = {3, 3, 3};
inline constexpr int64_t kManyPoints = 131072;
inline constexpr int32_t kFewSeq = 8;

// seq: the most scans of one map in the call; points: of all its scans.
inline const int32_t *tiling_for(const tsdf_map *m, int32_t seq, int64_t points)
{
    if (m->lt[0] != 0) return m->lt;
    if (seq <= 1) return points > kManyPoints ? kManyScansTiling : kScanTiling;
    return seq <= kFewSeq ? kFewSeqTiling : kBatchTiling;
}

// The launch shape of an integration on this map (a batch takes its first
// scan's map's).
inline LaunchShape launch_shape(const tsdf_map *m, int32_t seq, int64_t points)
{
    LaunchShape sh;
    const int32_t *lt = tiling_for(m, seq, points);
    for (int a = 0; a < 3; ++a) sh.lt[a] = lt[a];
    sh.tile_grid = m->tile_grid;
    sh.bin_block = m->bin_block > 0 ? m->bin_block : kBinBlock;
    sh.tile_block = m->tile_block > 0 ? m->tile_block : kTileBlockDefault;
    return sh;
}

}  // namespace tsdf
