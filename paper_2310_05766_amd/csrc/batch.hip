// Batched integration (FeatSense, arXiv 2310.05766, Sec. VI): any number of
// registered scans, into any number of maps, in one pass of two to six kernels.
//
// Each map window is cut into tiles of 2^lt voxels per axis (window-relative
// coordinates). The per-scan volume V of the min-tsdf step never reaches HBM:
// a workgroup owns one tile, keeps its candidate keys (|s|, point index, s)
// in LDS and resolves them with ds_min (order independent, one winner per
// voxel), then applies the averaging step, Eq. (1) and Eq. (2), to the tile.
// When several scans of one map share a batch, the tile's SDF and weights
// stay in LDS while its workgroup applies those scans one after another, in
// submission order, and go back to HBM once.
//
//   k_rows        where scans may have rows of points, their lengths (patch.hpp)
//   k_bin<count>  every ray walks its band on the grid of tiles (the exact
//                 walk with tile-sized cells) and counts one entry per tile;
//                 keys are (sequence slot, tile), merged per block in an LDS
//                 table so that each block sends one atomic per distinct key
//   k_alloc       a run of the entry buffer per (sequence slot, tile), runs of
//                 one tile consecutive in sequence order; list of busy tiles
//   k_bin<fill>   the same walk, writing point indices into the runs
//   k_tile        per busy tile, per sequence slot in order: every ray jumps
//                 to its first voxel in the tile (exact crossing counts) and
//                 walks the tile; candidates meet in LDS; then the merge
//   k_stats       per-scan counts, when asked for (one binning pass: the tile
//                 pass adds them up)
//
// Where each map has one scan, binning is one pass (the engine says when), after
// k_rows where there are several:
//   k_bin<once>   the walk once; each block writes its entries, tile by tile,
//                 into a region of its own and adds a segment of them to the
//                 list of each tile it met; who adds a tile's first one lists
//                 the tile as busy
//   k_tile_once   k_tile for these lists
// (128 x 1024 points: 11.7 us, where count, runs and fill took 6.4 + 5.7 + 11.2.)
#include <string.h>

#include <algorithm>

#include "internal.hpp"

namespace tsdf {

namespace {

constexpr int kAllocBlock = 512;

__device__ __forceinline__ uint32_t lane() { return __lane_id(); }

// A map array seen as global memory: through a generic pointer the compiler
// must assume it may alias the LDS buffers, and it then waits for every map
// load before the LDS store that follows it.
typedef __attribute__((address_space(1))) int16_t glob_i16;
__device__ __forceinline__ glob_i16 *glob(int16_t *p) { return (glob_i16 *)p; }

template <int kLog2>
__device__ __forceinline__ uint32_t hash_slot(uint32_t key)
{
    return (key * 2654435761u) >> (32 - kLog2);
}

// Second half of an entry record: what the tile pass needs of the ray
// beyond its point, r = isqrt(|D|^2) and the band offsets off = E - q (both
// exact: r < 2^32, |off_a| <= tau < 2^15), the voxel crossings per axis
// (each < 2^7) up to the event that entered the tile, and the scan's sequence
// slot (< 2^6).
__device__ __forceinline__ uint4 entry_ray(const Ray &R, uint32_t cpack, uint32_t seq)
{
    const uint32_t o0 = (uint32_t)(R.E[0] - R.q[0]) & 0xffffu, o1 = (uint32_t)(R.E[1] - R.q[1]) & 0xffffu,
                   o2 = (uint32_t)(R.E[2] - R.q[2]) & 0xffffu;
    return make_uint4((uint32_t)R.r, o0 | o1 << 16, o2 | (cpack & 0xffffu) << 16, cpack >> 16 | seq << 8);
}

enum { kCount = 0, kFillRuns = 1, kOnce = 2 };

// A tile with this many entries or more is listed first: the persistent tile
// pass then starts the longest tiles early instead of ending on one of them.
constexpr uint32_t kHeavyTile = 2048;

// Adds a block's segment of n entries to a tile's list, in two steps, so that
// other work can go between the atomic and its result: the segments and entries
// listed before, and the segment's place. A tile is listed as busy by its first
// segment (finish_segment is then true, and the caller does it), and once more,
// among the heavy ones, by the segment that makes it heavy: the tile pass takes
// it from there and skips it among the others.
__device__ __forceinline__ unsigned long long begin_segment(const BatchArrays &B, uint32_t tile, uint32_t n)
{
    return atomicAdd(reinterpret_cast<unsigned long long *>(&B.lists[tile]), (unsigned long long)n << 32 | 1ull);
}
__device__ __forceinline__ bool finish_segment(const BatchArrays &B, BatchCtl *ctl, unsigned long long old, uint32_t tile,
                                               uint32_t map, uint32_t pos, uint32_t n, uint32_t node)
{
    TileList *L = &B.lists[tile];
    const uint32_t k = (uint32_t)old, total = (uint32_t)(old >> 32);
    if (k < kSegs) L->seg[k] = make_uint2(pos, n);
    else B.nodes[node] = make_uint4(atomicExch(&L->chain[(k - kSegs) % kChains], node + 1u), pos, n, 0u);
    if (total < kHeavyTile && total + n >= kHeavyTile) {
        const uint32_t h = atomicAdd(&ctl->n_nonempty, 1u);
        B.offsets[h] = tile;
        B.cursor[h] = map;
    }
    return k == 0u;
}

// The rows of a batch's scans, a wave each: 6 us. (By every block of the counting
// pass for itself, 10 us on 50 scans of 128 x 1024 points. The one scan of a plain
// call does that: 0.8 us of 34 where a kernel of its own would take 5.)
__global__ __launch_bounds__(256) void k_rows(BatchArrays B)
{
    const uint32_t s = blockIdx.x * 4u + threadIdx.x / 64u;
    if (s >= (uint32_t)B.hdr->nscans) return;
    ScanDev &SD = B.scans[s];
    if (SD.rings == 0) return;
    const Row row = find_row(SD.xyz, SD.n, SD.rings, kBinPatch);
    if (threadIdx.x % 64u == 0) SD.row = row;
}

// kInline (the first pass only): the batch is one scan whose descriptors are
// I, not yet in memory.
template <int kMode, int kBinBlock, bool kInline>
__global__ __launch_bounds__(kBinBlock) void k_bin(BatchArrays B, InlineDesc I)
{
    constexpr bool kFill = kMode != kCount;       // writes records
    constexpr bool kFirst = kMode != kFillRuns;   // counts valid points
    // the block's (sequence slot, tile) keys: a hash table of two slots per
    // point of the block (a block of 256 OS1-128 points meets about 100
    // tiles), so that clearing and flushing it stays cheap; keys that find it
    // full go straight to their runs
    constexpr int kHashLog2 = kBinBlock == 128 ? 8 : (kBinBlock == 256 ? 9 : 10);
    constexpr uint32_t kHashSlots = 1u << kHashLog2;
    static_assert(kHashSlots == 2 * kBinBlock && kHashSlots <= 1024, "slots fit the 10-bit field below");
    __shared__ uint32_t h_key[kHashSlots];  // key + 1; 0 = free
    __shared__ uint32_t h_cnt[kHashSlots];
    __shared__ uint32_t h_base[kFill ? kHashSlots : 1];
    // per emitted entry: hash slot | crossing counts (7 bits per axis) << 10, and rank
    __shared__ uint32_t s_slot[kFill ? kMaxEmit * kBinBlock : 1];
    __shared__ uint16_t s_rank[kFill ? kMaxEmit * kBinBlock : 1];
    __shared__ uint32_t s_valid, s_extra, s_new, s_job, s_sum[kBinBlock / 64];
    __shared__ Row s_row;
    // a one-scan batch's descriptors come with the counting launch, which
    // stores them for the kernels after it
    constexpr bool inl = kFirst && kInline;
    const BatchHdr H = inl ? I.hdr : *B.hdr;
    if (inl && blockIdx.x == 0 && threadIdx.x == 0) {
        *B.hdr = I.hdr;
        B.maps[0] = I.map;
        B.scans[0] = I.scan;
        B.seq_sensor[0] = make_int4(I.scan.rp.o[0], I.scan.rp.o[1], I.scan.rp.o[2], I.scan.rp.tau);
    }
    if (kMode == kCount && blockIdx.x == 0 && threadIdx.x == 0) {
        // the allocation counters of the previous batch are done with (the
        // grid always has a block 0, also for a batch without points)
        B.ctl->n_nonempty = 0;
        B.ctl->n_light = 0;
        B.ctl->entries = 0;
        B.ctl->overflow = 0;
        for (int q = 0; q < kQueues; ++q) B.ctl->work[q * kQueueStride] = 0;
    }
    const uint32_t turn = kMode == kOnce ? B.ctl->next_turn : 0u;
    if (kMode == kOnce && blockIdx.x == 0 && threadIdx.x == 0) B.ctl->turn = turn;
    if (blockIdx.x >= H.nblocks) return;
    if (kMode == kOnce && H.want_stats)
        for (uint32_t j = blockIdx.x * kBinBlock + threadIdx.x; j < (uint32_t)H.nscans * kStatWords; j += H.nblocks * kBinBlock)
            B.scan_stats[j] = 0;
    for (uint32_t j = threadIdx.x; j < kHashSlots; j += kBinBlock) {
        h_key[j] = 0;
        h_cnt[j] = 0;
    }
    if (threadIdx.x == 0) s_valid = s_extra = s_new = 0;
    // (a one-scan batch's block table is written here, for the fill)
    if (inl && kMode == kCount && threadIdx.x == 0) B.block_scan[blockIdx.x] = 0u;
    const uint32_t s = inl ? 0u : B.block_scan[blockIdx.x];
    const ScanDev &SD = inl ? I.scan : B.scans[s];
    // one scan: every block finds the same row length; several: k_rows has it
    const bool tries = inl && SD.rings != 0;
    if (tries && threadIdx.x < 64u) s_row = find_row(SD.xyz, SD.n, SD.rings, kBinPatch);
    __syncthreads();
    const Row row = uniform_row(tries ? s_row : SD.row);
    if (tries && kMode == kCount && blockIdx.x == 0 && threadIdx.x == 0) B.scans[0].row = row;
    const int64_t i = patch_point<kBinBlock, kBinPatch.rows>(blockIdx.x - SD.block0, threadIdx.x, row);
    const MapDev &MD = inl ? I.map : B.maps[SD.map];
    const RayParams rp = SD.rp;
    Ray R;
    Walk W, Wv;  // the walk on the tile grid; the voxel walk's start (fill)
    bool active = false;
    int32_t q[3] = {0, 0, 0};
    if (i < SD.n) {
        const float *p = SD.xyz + 3 * i;
        if (quantise(p[0], p[1], p[2], rp, q) && make_ray(q, rp, R)) {
            active = true;
            // the tiles of the band's voxels are the cells of the same exact
            // walk on the grid of tiles (floor of a floor division)
            const int32_t lc[3] = {10 + H.lt[0], 10 + H.lt[1], 10 + H.lt[2]};
            const int32_t base[3] = {1024 * MD.origin[0], 1024 * MD.origin[1], 1024 * MD.origin[2]};
            walk_init_cells(R, W, lc, base);
            if (kFill) walk_init(R, Wv);
        }
    }
    const uint32_t valid = active ? 1u : 0u;
    const uint32_t seq = (uint32_t)SD.seq;
    const uint32_t key0 = seq * H.gtiles + MD.tile_base;
    // the map's tile counts in registers: loads through MD inside the walk
    // would be repeated after every atomic (they may alias)
    const uint32_t nt0 = (uint32_t)__builtin_amdgcn_readfirstlane(MD.nt[0]);
    const uint32_t nt1 = (uint32_t)__builtin_amdgcn_readfirstlane(MD.nt[1]);
    const uint32_t nt2 = (uint32_t)__builtin_amdgcn_readfirstlane(MD.nt[2]);
    // one pass: this block's region of the entries, its nodes, the counters
    const uint32_t region = kMode == kOnce ? blockIdx.x * kBinBlock * H.emit : 0u;
    const uint32_t node0 = kMode == kOnce ? blockIdx.x * nodes_per_block(kBinBlock, H.emit) : 0u;
    BatchCtl *ctl = kMode == kOnce ? B.ctl + 1u + turn : B.ctl;
    int ne = 0;
    uint32_t listed = 0;  // fill: bit k set when entry k was listed in LDS (not sent straight to its run)
    double t_in = -1.0;  // event that entered the current tile (none for the first)
    int typ_in = 0;
    while (active) {
        if ((uint32_t)W.g[0] < nt0 && (uint32_t)W.g[1] < nt1 && (uint32_t)W.g[2] < nt2) {
            const uint32_t key =
                key0 + ((uint32_t)W.g[0] * nt1 + (uint32_t)W.g[1]) * nt2 + (uint32_t)W.g[2];
            uint32_t h = hash_slot<kHashLog2>(key), slot = 0xffffu;
            for (uint32_t probe = 0; probe < kHashSlots; ++probe) {
                const uint32_t old = atomicCAS(&h_key[h], 0u, key + 1u);
                if (old == 0u || old == key + 1u) {
                    slot = h;
                    break;
                }
                h = (h + 1u) & (kHashSlots - 1u);
            }
            // voxel crossings of each axis up to the event that entered
            // this tile: the tile pass resumes the voxel walk there
            uint32_t cpack = 0;
            if (kFill && t_in >= 0.0) {
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    cpack |= (uint32_t)crossings_upto(Wv.T[a], Wv.dT[a], Wv.step[a] > 0 ? 0 : 1, t_in, typ_in)
                             << (8 * a);
            }
            if (slot != 0xffffu && (!kFill || ne < kMaxEmit)) {
                const uint32_t rank = atomicAdd(&h_cnt[slot], 1u);
                if (kFill) {
                    s_slot[ne * kBinBlock + threadIdx.x] = slot | counts_8to7(cpack) << 10;
                    s_rank[ne * kBinBlock + threadIdx.x] = (uint16_t)rank;
                    listed |= 1u << ne;
                }
            } else if (kMode == kOnce) {  // a segment of its own, from the region's end
                const uint32_t x = atomicAdd(&s_extra, 1u), pos = region + kBinBlock * H.emit - 1u - x;
                B.entries[pos] = make_uint4((uint32_t)i, (uint32_t)q[0], (uint32_t)q[1], (uint32_t)q[2]);
                B.entries2[pos] = entry_ray(R, cpack, seq);
                if (finish_segment(B, ctl, begin_segment(B, key, 1u), key, (uint32_t)SD.map, pos, 1u,
                                   node0 + 2u * kBinBlock + x))
                    B.jobs[atomicAdd(&ctl->n_light, 1u)] = make_uint4(key, (uint32_t)SD.map, 0u, 0u);
            } else if (kFill) {  // table full or very long band: straight to the tile's run
                const uint32_t pos = atomicAdd(&B.cursor[key], 1u);
                if (pos < H.cap) {
                    B.entries[pos] = make_uint4((uint32_t)i, (uint32_t)q[0], (uint32_t)q[1], (uint32_t)q[2]);
                    B.entries2[pos] = entry_ray(R, cpack, seq);
                } else {
                    atomicOr(&B.ctl->overflow, 1u);
                }
            } else {
                atomicAdd(&B.counts[key], 1u);
            }
            ++ne;
        }
        active = walk_next_event(W, t_in, typ_in);
    }
    const auto write_records = [&]() {
        // each record carries the point's fixed-point position, so the tile pass
        // needs neither the point nor the pose again
        const uint4 rec = make_uint4((uint32_t)i, (uint32_t)q[0], (uint32_t)q[1], (uint32_t)q[2]);
        // the entries listed in LDS: an entry that found the table full went
        // straight to its run and left its LDS place unwritten
        const int nl = ne < kMaxEmit ? ne : kMaxEmit;
        for (int k = 0; k < nl; ++k) {
            if (!((listed >> k) & 1u)) continue;
            const uint32_t sc = s_slot[k * kBinBlock + threadIdx.x];
            const uint32_t pos = h_base[sc & 1023u] + s_rank[k * kBinBlock + threadIdx.x];
            if (kMode == kOnce || pos < H.cap) {
                B.entries[pos] = rec;
                B.entries2[pos] = entry_ray(R, counts_7to8(sc >> 10), seq);
            } else {
                atomicOr(&B.ctl->overflow, 1u);
            }
        }
    };
    if (kFirst && valid) atomicAdd(&s_valid, 1u);
    __syncthreads();
    if (kMode == kOnce) {
        // the block's entries in the order of its table: two slots per thread
        const uint32_t j0 = 2u * threadIdx.x, c0 = h_cnt[j0], c1 = h_cnt[j0 + 1u];
        uint32_t p = c0 + c1;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t v = (uint32_t)__shfl_up((int)p, off);
            if (lane() >= (uint32_t)off) p += v;
        }
        if (lane() == 63u) s_sum[threadIdx.x / 64] = p;
        __syncthreads();
        for (uint32_t w = 0; w < threadIdx.x / 64; ++w) p += s_sum[w];
        const uint32_t at = region + p - c0 - c1;
        h_base[j0] = at;
        h_base[j0 + 1u] = at + c0;
        const uint32_t k0 = h_key[j0] - 1u, k1 = h_key[j0 + 1u] - 1u;
        unsigned long long old0 = 0, old1 = 0;
        if (c0) old0 = begin_segment(B, k0, c0);
        if (c1) old1 = begin_segment(B, k1, c1);
        __syncthreads();
        // the records go out while the atomics are under way
        write_records();
        const bool f0 = c0 && finish_segment(B, ctl, old0, k0, (uint32_t)SD.map, at, c0, node0 + j0);
        const bool f1 = c1 && finish_segment(B, ctl, old1, k1, (uint32_t)SD.map, at + c0, c1, node0 + j0 + 1u);
        // one atomic for all tiles that this block lists
        uint32_t r = 0;
        if (f0 || f1) r = atomicAdd(&s_new, (f0 ? 1u : 0u) + (f1 ? 1u : 0u));
        __syncthreads();
        if (threadIdx.x == 0) {
            if (s_new) s_job = atomicAdd(&ctl->n_light, s_new);
            B.valid_part[blockIdx.x] = s_valid;
        }
        __syncthreads();
        if (f0) B.jobs[s_job + r++] = make_uint4(k0, (uint32_t)SD.map, 0u, 0u);
        if (f1) B.jobs[s_job + r] = make_uint4(k1, (uint32_t)SD.map, 0u, 0u);
        return;
    }
    // one global atomic per distinct key of this block
    for (uint32_t j = threadIdx.x; j < kHashSlots; j += kBinBlock) {
        const uint32_t k1 = h_key[j];
        const uint32_t c = h_cnt[j];
        if (k1 == 0u || c == 0u) continue;
        if (kFill) h_base[j] = atomicAdd(&B.cursor[k1 - 1u], c);
        else atomicAdd(&B.counts[k1 - 1u], c);
    }
    if (!kFill) {
        if (threadIdx.x == 0) B.valid_part[blockIdx.x] = s_valid;
        return;
    }
    __syncthreads();
    write_records();
}

// Map slot of a global tile: the last map whose first tile is <= g.
__device__ __forceinline__ int32_t map_of_tile(const BatchArrays &B, int32_t nmaps, uint32_t g)
{
    int32_t lo = 0, hi = nmaps - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (B.maps[mid].tile_base <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Runs of the entry buffer: one per (sequence slot, tile), a tile's runs
// consecutive in sequence order; the tile is listed as busy. Runs may lie in
// any order, so they are handed out by atomic allocation, one atomic per
// block and counter (same-address device atomics serialise; a block prefix
// keeps them few). Four lanes share a tile, each summing a quarter of its
// sequence slots, so that the chains of count loads stay short.
constexpr int kAllocTiles = kAllocBlock / 4;
constexpr int kAllocPer = kMaxSeq / 4;  // sequence slots per lane, at most
__global__ __launch_bounds__(kAllocBlock) void k_alloc(BatchArrays B)
{
    __shared__ uint32_t s_w[3][kAllocBlock / 64];  // per wave: entries, heavy tiles, light tiles
    __shared__ uint32_t s_base[3];
    const BatchHdr H = *B.hdr;
    if (blockIdx.x * kAllocTiles >= H.gtiles) return;
    const uint32_t t = blockIdx.x * kAllocTiles + threadIdx.x / 4;
    const uint32_t part = threadIdx.x & 3u, wave = threadIdx.x / 64;
    const int per = (H.S + 3) / 4;  // at most kAllocPer
    const int s_lo = (int)part * per, s_hi = min(H.S, s_lo + per);
    // this part's counts, kept for the runs: every load is issued (at a
    // clamped, valid index) before any is used, so all are in flight together
    uint32_t cs[kAllocPer];
    const uint32_t tc = min(t, H.gtiles - 1u);
#pragma unroll
    for (int j = 0; j < kAllocPer; ++j) cs[j] = B.counts[(uint32_t)min(s_lo + j, H.S - 1) * H.gtiles + tc];
#pragma unroll
    for (int j = 0; j < kAllocPer; ++j) cs[j] = (t < H.gtiles && s_lo + j < s_hi) ? cs[j] : 0u;
    uint32_t c = 0;
    uint64_t busy = 0;  // this part's busy sequence slots
#pragma unroll
    for (int j = 0; j < kAllocPer; ++j) {
        c += cs[j];
        busy |= cs[j] ? 1ull << (s_lo + j) : 0ull;
    }
    // the tile's busy slots: the four parts' masks together
#pragma unroll
    for (int x = 1; x < 4; x <<= 1) {
        const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)busy, x);
        const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(busy >> 32), x);
        busy |= (uint64_t)lo | (uint64_t)hi << 32;
    }
    // inclusive prefix of the four parts of a tile, and the tile's total
    uint32_t pq = c;
    {
        uint32_t a = (uint32_t)__shfl_up((int)pq, 1);
        if (part >= 1) pq += a;
        a = (uint32_t)__shfl_up((int)pq, 2);
        if (part >= 2) pq += a;
    }
    const uint32_t tile_c = (uint32_t)__shfl((int)pq, (int)(lane() | 3u));
    // inclusive prefix over the wave's tiles (counted on each tile's last lane)
    const bool heavy = tile_c >= kHeavyTile;
    uint32_t pc = part == 3u ? tile_c : 0u, pn = (part == 3u && heavy) ? 1u : 0u;
    uint32_t pl = (part == 3u && tile_c && !heavy) ? 1u : 0u;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t a = (uint32_t)__shfl_up((int)pc, off);
        const uint32_t b = (uint32_t)__shfl_up((int)pn, off);
        const uint32_t d = (uint32_t)__shfl_up((int)pl, off);
        if (lane() >= (uint32_t)off) {
            pc += a;
            pn += b;
            pl += d;
        }
    }
    pc = (uint32_t)__shfl((int)pc, (int)(lane() | 3u));
    pn = (uint32_t)__shfl((int)pn, (int)(lane() | 3u));
    pl = (uint32_t)__shfl((int)pl, (int)(lane() | 3u));
    if (lane() == 63) {
        s_w[0][wave] = pc;
        s_w[1][wave] = pn;
        s_w[2][wave] = pl;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        // lane a: exclusive prefix of counter a over the waves, then one
        // atomic for the block; the three atomics leave as one instruction
        const int a = (int)threadIdx.x;
        uint32_t sum = 0;
        for (int k = 0; k < kAllocBlock / 64; ++k) {
            const uint32_t v = s_w[a][k];
            s_w[a][k] = sum;
            sum += v;
        }
        uint32_t *ctr = a == 0 ? &B.ctl->entries : (a == 1 ? &B.ctl->n_nonempty : &B.ctl->n_light);
        s_base[a] = sum ? atomicAdd(ctr, sum) : 0u;
    }
    __syncthreads();
    if (tile_c) {
        // this part's first run: after the wave's earlier tiles and the
        // tile's earlier parts
        uint32_t off = s_base[0] + s_w[0][wave] + (pc - tile_c) + (pq - c);
#pragma unroll
        for (int j = 0; j < kAllocPer; ++j) {
            if (!cs[j]) continue;  // runs of empty slots are never read (nor slots past S)
            const uint32_t k = (uint32_t)(s_lo + j) * H.gtiles + t;
            B.offsets[k] = off;
            B.cursor[k] = off;
            off += cs[j];
        }
        if (part == 0u) {
            const uint32_t slot =
                heavy ? s_base[1] + s_w[1][wave] + pn - 1u : H.gtiles - 1u - (s_base[2] + s_w[2][wave] + pl - 1u);
            B.jobs[slot] = make_uint4(t, (uint32_t)map_of_tile(B, H.nmaps, t), (uint32_t)busy, (uint32_t)(busy >> 32));
        }
    }
}

// Eq. (1) with one unit of weight, Eq. (2), on a voxel state held in 32-bit
// registers (the stored int16 values, sign-extended once).
__device__ __forceinline__ void merge_one(int32_t &sdf, int32_t &w, int32_t v, int32_t w_max)
{
    sdf = rdiv_small(__mul24(sdf, w) + v, w + 1);  // |sdf|, w < 2^15: a 24-bit product
    w = w + 1 < w_max ? w + 1 : w_max;
}

__device__ __forceinline__ void merge_one(int16_t &sdf, int16_t &w, int32_t v, int32_t w_max)
{
    int32_t s = sdf, ww = w;
    merge_one(s, ww, v, w_max);
    sdf = (int16_t)s;
    w = (int16_t)ww;
}

// A candidate's key in LDS: 64 bits, or 32 where tau and the point counts
// leave room (key32_shift), which doubles the slots that a group holds.
__device__ __forceinline__ int32_t key_value(uint64_t key, uint32_t) { return tile_key_sdf(key); }
__device__ __forceinline__ int32_t key_value(uint32_t key, uint32_t shift) { return tile_key_sdf(key, shift); }

// Merge the touched voxels of one run of 8 z-consecutive voxels straight
// into HBM (one busy sequence slot on the tile).
template <typename Key>
__device__ __forceinline__ uint32_t merge_run_direct(Key *kr, uint32_t shift, const MapDev &MD, int64_t row,
                                                     int32_t rz0)
{
    constexpr Key kNone = (Key)~(Key)0;
    Key kk[8];
    bool any = false;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        kk[j] = kr[j];
        any |= kk[j] != kNone;
    }
    if (!any) return 0;
    uint32_t updated = 0;
    if (MD.vec_ok) {
        // 8 int16 of sdf and of w in one 16-byte access each
        int32_t sz = rz0 + MD.ring0[2];
        sz -= sz >= MD.dims[2] ? MD.dims[2] : 0;
        int4 sv = *reinterpret_cast<const int4 *>(MD.sdf + row + sz);
        int4 wv = *reinterpret_cast<const int4 *>(MD.w + row + sz);
        int16_t *sp = reinterpret_cast<int16_t *>(&sv);
        int16_t *wp = reinterpret_cast<int16_t *>(&wv);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (kk[j] != kNone) {
                merge_one(sp[j], wp[j], key_value(kk[j], shift), MD.w_max);
                kr[j] = kNone;
                ++updated;
            }
        *reinterpret_cast<int4 *>(MD.sdf + row + sz) = sv;
        *reinterpret_cast<int4 *>(MD.w + row + sz) = wv;
    } else {
        for (int j = 0; j < 8; ++j) {
            if (kk[j] == kNone) continue;
            kr[j] = kNone;
            if (rz0 + j >= MD.dims[2]) continue;  // the tile's part outside the window
            int32_t sz = rz0 + j + MD.ring0[2];
            sz -= sz >= MD.dims[2] ? MD.dims[2] : 0;
            merge_one(MD.sdf[row + sz], MD.w[row + sz], key_value(kk[j], shift), MD.w_max);
            ++updated;
        }
    }
    return updated;
}

// Slot of window-relative voxel r of a map.
__device__ __forceinline__ int64_t slot_of_rel(const MapDev &MD, int32_t rx, int32_t ry, int32_t rz)
{
    int32_t sx = rx + MD.ring0[0], sy = ry + MD.ring0[1], sz = rz + MD.ring0[2];
    sx -= sx >= MD.dims[0] ? MD.dims[0] : 0;
    sy -= sy >= MD.dims[1] ? MD.dims[1] : 0;
    sz -= sz >= MD.dims[2] ? MD.dims[2] : 0;
    return ((int64_t)sx * MD.dims[1] + sy) * MD.dims[2] + sz;
}

// Values every lane of a workgroup holds alike, moved to scalar registers
// (the compiler cannot tell that values read from LDS or memory are uniform,
// and keeps them, and all derived from them, in vector registers otherwise).
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// LDS byte address of a shared-memory pointer, and back: an address kept
// in one integer register needs no base added per access.
typedef __attribute__((address_space(3))) unsigned long long lds_u64;
typedef __attribute__((address_space(3))) unsigned int lds_u32;

__device__ __forceinline__ uint32_t lds_address(void *p) { return (uint32_t)(uintptr_t)(lds_u32 *)(uint32_t *)p; }
__device__ __forceinline__ void lds_min(int32_t a, uint64_t key)
{
    atomicMin((unsigned long long *)(lds_u64 *)(uintptr_t)(uint32_t)a, (unsigned long long)key);
}
__device__ __forceinline__ void lds_min(int32_t a, uint32_t key)
{
    atomicMin((unsigned int *)(lds_u32 *)(uintptr_t)(uint32_t)a, key);
}
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T>
__device__ __forceinline__ T *uniform(T *p)
{
    const uint64_t a = (uint64_t)p;
    return (T *)((uint64_t)uniform((uint32_t)a) | (uint64_t)uniform((uint32_t)(a >> 32)) << 32);
}

__device__ __forceinline__ MapDev uniform_map(const MapDev &m)
{
    MapDev u;
    u.sdf = uniform(m.sdf);
    u.w = uniform(m.w);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        u.dims[a] = uniform(m.dims[a]);
        u.origin[a] = uniform(m.origin[a]);
        u.ring0[a] = uniform(m.ring0[a]);
        u.nt[a] = uniform(m.nt[a]);
    }
    u.ntot = uniform(m.ntot);
    u.tile_base = uniform(m.tile_base);
    u.tau = uniform(m.tau);
    u.w_max = uniform(m.w_max);
    u.vec_ok = uniform(m.vec_ok);
    u.pad = 0;
    return u;
}

// One entry's candidates, from its record to the keys of its slot at `base`:
// the walk is resumed right after the event that entered the tile; its voxels
// inside the tile are one run (the walk carries the key's LDS address itself).
// Returns the visits when kStats. (t0: the tile's first voxel in the window,
// blo: in global coordinates.)
template <bool kStats, typename Key>
__device__ __forceinline__ uint32_t walk_entry(const uint4 &ra, const uint4 &rb, const int32_t o[3], int32_t tau,
                                               uint32_t base, const BatchHdr &H, const MapDev &MD,
                                               const int32_t t0[3], const int32_t blo[3], const int32_t ext[3],
                                               const int32_t shb[3], bool cut)
{
    constexpr int kKeyLog2 = sizeof(Key) == 4 ? 2 : 3;
    const uint32_t i = ra.x;
    const int32_t q[3] = {(int32_t)ra.y, (int32_t)ra.z, (int32_t)ra.w};
    const int32_t off[3] = {(int16_t)(rb.y & 0xffffu), (int16_t)(rb.y >> 16), (int16_t)(rb.z & 0xffffu)};
    const int32_t c[3] = {(int32_t)((rb.z >> 16) & 0xffu), (int32_t)(rb.z >> 24), (int32_t)(rb.w & 0xffu)};
    Ray R;
    BoxWalk V;
    tile_walk_resume(q, off, rb.x, c, o, tau, blo, ext, shb, base, R, V);
    const double taud = (double)tau, rh = R.r + 0.5;
    uint32_t visits = 0;
    // (a candidate outside the window is no visit)
    const auto resident = [&]() {
        const uint32_t v = ((uint32_t)V.lv - base) >> kKeyLog2;
        return (int32_t)(v & ((1u << H.lt[2]) - 1u)) + t0[2] < MD.dims[2] &&
               (int32_t)((v >> H.lt[2]) & ((1u << H.lt[1]) - 1u)) + t0[1] < MD.dims[1] &&
               (int32_t)(v >> (H.lt[1] + H.lt[2])) + t0[0] < MD.dims[0];
    };
    if (sizeof(Key) == 4) {
        do {
            lds_min(V.lv, tile_key32(V.n, rh, R.inv_r2, taud, H.key_shift, i));
            if (kStats) visits += !cut || resident() ? 1u : 0u;
        } while (box_walk_next(V));
    } else {
        const uint32_t ihi = i >> 16, ilo = i << 16;
        do {
            lds_min(V.lv, tile_key(V.n, rh, R.inv_r2, taud, ihi, ilo));
            if (kStats) visits += !cut || resident() ? 1u : 0u;
        } while (box_walk_next(V));
    }
    return visits;
}

// A tile with one busy sequence slot: its keys straight into HBM, runs of 8;
// the voxels updated.
template <int kTileBlock, typename Key>
__device__ __forceinline__ uint32_t merge_tile_direct(Key *keys, uint32_t tvox, const BatchHdr &H, const MapDev &MD,
                                                      const int32_t t0[3], bool cut)
{
    constexpr Key kNone = (Key)~(Key)0;
    uint32_t updated = 0;
    for (uint32_t v0 = threadIdx.x * 8u; v0 < tvox; v0 += kTileBlock * 8u) {
        const int32_t rz0 = (int32_t)(v0 & ((1u << H.lt[2]) - 1u)) + t0[2];
        const int32_t ry = (int32_t)((v0 >> H.lt[2]) & ((1u << H.lt[1]) - 1u)) + t0[1];
        const int32_t rx = (int32_t)(v0 >> (H.lt[1] + H.lt[2])) + t0[0];
        if (cut && (rx >= MD.dims[0] || ry >= MD.dims[1] || rz0 >= MD.dims[2])) {
#pragma unroll
            for (int j = 0; j < 8; ++j) keys[v0 + j] = kNone;
            continue;
        }
        int32_t sx = rx + MD.ring0[0], sy = ry + MD.ring0[1];
        sx -= sx >= MD.dims[0] ? MD.dims[0] : 0;
        sy -= sy >= MD.dims[1] ? MD.dims[1] : 0;
        const int64_t row = ((int64_t)sx * MD.dims[1] + sy) * MD.dims[2];
        updated += merge_run_direct(&keys[v0], H.key_shift, MD, row, rz0);
    }
    return updated;
}

// Persistent tile pass. Workgroup b first takes busy tile b, then pulls
// further tiles from queue b % nq, nq = min(8, workgroups) (one queue per
// XCD keeps same-address atomics spread; with fewer than 8 workgroups each
// queue still has one, so every job is reached). A tile's job record holds
// its map and its busy sequence slots, so that the runs and the map record
// of a tile are requested together, with the sensors of its slots, which come
// from a table indexed by (map, sequence slot). Per tile, the busy sequence
// slots are taken in groups of G: the candidates of a group's runs are computed
// together, one LDS key buffer per slot, then each voxel applies the group's
// scans in submission order. A group's runs lie one after another, and a
// record names its slot, so an entry needs no search for its run. A tile busy
// in several slots keeps its SDF and weights in LDS.
// Bound by instruction issue. Against 64-bit keys alone, a search over the
// group's runs per entry and a set-up through the general walk (96 VGPRs,
// spills), on 50 scans of 128 x 1024 points 333 -> 264 us, on one 29.0 -> 22.8.
template <int kTileBlock, bool kStats, typename Key>
__global__ __launch_bounds__(kTileBlock) __attribute__((amdgpu_waves_per_eu(kTileWaves))) void k_tile(BatchArrays B)
{
    constexpr Key kNone = (Key)~(Key)0;
    constexpr int kGroup = sizeof(Key) == 4 ? kMaxGroup32 : kMaxGroup64;
    constexpr int kKeyLog2 = sizeof(Key) == 4 ? 2 : 3;
    extern __shared__ uint64_t s_dyn[];  // G * tvox keys, then the cached tile: tvox sdf, tvox w
    Key *s_keys = reinterpret_cast<Key *>(s_dyn);
    // (kTileStaticLds bounds these) per busy slot of the tile, in sequence
    // order: first entry, entries, sequence slot; per sequence slot: sensor,
    // and tau | place among the busy slots << 16
    __shared__ uint32_t s_beg[kMaxSeq], s_cnt[kMaxSeq];
    __shared__ uint8_t s_list[kMaxSeq];
    __shared__ int4 s_sens[kMaxSeq];
    __shared__ uint32_t s_vis[kGroup], s_upd[kGroup];
    __shared__ uint32_t s_job;
    const BatchHdr H = *B.hdr;
    const int32_t lsum = H.lt[0] + H.lt[1] + H.lt[2];
    const uint32_t tvox = 1u << lsum;
    const int32_t G = H.G;
    const uint32_t kshift = H.key_shift;
    int16_t *c_sdf = reinterpret_cast<int16_t *>(s_keys + (size_t)G * tvox);
    int16_t *c_w = c_sdf + tvox;
    // heavy tiles first (from the list's start), then the others (from its end)
    const uint32_t nheavy = B.ctl->n_nonempty, nne = nheavy + B.ctl->n_light;
    const uint32_t ez = 1u << H.lt[2], ey = 1u << H.lt[1];
    // LDS address shift per axis, in bytes of keys
    const int32_t shb[3] = {H.lt[1] + H.lt[2] + kKeyLog2, H.lt[2] + kKeyLog2, kKeyLog2};
    const int32_t ext[3] = {1 << H.lt[0], 1 << H.lt[1], 1 << H.lt[2]};
    uint32_t job = blockIdx.x;
    if (job >= nne) return;
    const uint32_t nq = gridDim.x < (uint32_t)kQueues ? gridDim.x : (uint32_t)kQueues;
    const uint32_t queue = blockIdx.x % nq;
    for (uint32_t v = threadIdx.x; v < (uint32_t)G * tvox; v += kTileBlock) s_keys[v] = kNone;
    while (job < nne) {
        const uint32_t at = job < nheavy ? job : H.gtiles - 1u - (job - nheavy);
        const uint4 jb = B.jobs[at];
        const uint32_t g = uniform(jb.x);
        const int32_t mb = uniform((int32_t)jb.y);
        const uint64_t busy = (uint64_t)uniform(jb.z) | (uint64_t)uniform(jb.w) << 32;
        const int nbusy = __popcll(busy);
        // the busy slots' runs and sensors, all in flight together, listed in
        // order, so that groups of G hold busy slots only
        if (threadIdx.x < 64u && ((busy >> threadIdx.x) & 1ull)) {
            const uint32_t k = threadIdx.x * H.gtiles + g;
            const int p = __popcll(busy & ((1ull << threadIdx.x) - 1ull));
            int4 sens = B.seq_sensor[mb * H.S + (int32_t)threadIdx.x];
            s_cnt[p] = B.counts[k];
            s_beg[p] = B.offsets[k];
            s_list[p] = (uint8_t)threadIdx.x;
            sens.w |= p << 16;
            s_sens[threadIdx.x] = sens;
        }
        const MapDev MD = uniform_map(B.maps[mb]);
        const uint32_t t = g - MD.tile_base;
        const uint32_t tz = t % (uint32_t)MD.nt[2];
        const uint32_t txy = t / (uint32_t)MD.nt[2];
        const int32_t t0[3] = {(int32_t)(txy / (uint32_t)MD.nt[1]) << H.lt[0],
                               (int32_t)(txy % (uint32_t)MD.nt[1]) << H.lt[1], (int32_t)tz << H.lt[2]};
        // the tile's first voxel in global coordinates; a tile that the
        // window's edge cuts is walked whole, and its voxels outside get no
        // merge
        int32_t blo[3];
        bool cut = false;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            blo[a] = MD.origin[a] + t0[a];
            cut = cut || t0[a] + (1 << H.lt[a]) > MD.dims[a];
        }
        __syncthreads();
        const bool cached = nbusy > 1;
        if (cached) {
            for (uint32_t v = threadIdx.x; v < tvox; v += kTileBlock) {
                const int32_t rz = (int32_t)(v & (ez - 1)) + t0[2];
                const int32_t ry = (int32_t)((v >> H.lt[2]) & (ey - 1)) + t0[1];
                const int32_t rx = (int32_t)(v >> (H.lt[1] + H.lt[2])) + t0[0];
                if (rx >= MD.dims[0] || ry >= MD.dims[1] || rz >= MD.dims[2]) continue;
                const int64_t slot = slot_of_rel(MD, rx, ry, rz);
                const int16_t sv = glob(MD.sdf)[slot], wv = glob(MD.w)[slot];
                c_sdf[v] = sv;
                c_w[v] = wv;
            }
        }
        for (int j0 = 0; j0 < nbusy; j0 += G) {
            // a group: busy slots j0 .. j0 + ng - 1 of the list, in order;
            // their runs are one stretch of records
            const int ng = min(G, nbusy - j0);
            const uint32_t beg = uniform(s_beg[j0]);
            const uint32_t end = min(uniform(s_beg[j0 + ng - 1] + s_cnt[j0 + ng - 1]), H.cap);
            if (kStats) {
                if (threadIdx.x < (uint32_t)ng) {
                    s_vis[threadIdx.x] = 0;
                    s_upd[threadIdx.x] = 0;
                }
                __syncthreads();
            }
            for (uint32_t e = beg + threadIdx.x; e < end; e += kTileBlock) {
                const uint4 ra = B.entries[e];
                const uint4 rb = B.entries2[e];
                const int4 sens = s_sens[(rb.w >> 8) & (kMaxSeq - 1)];
                const int32_t o[3] = {sens.x, sens.y, sens.z};
                const int32_t r = (sens.w >> 16) - j0;
                const uint32_t base = lds_address(s_keys) + (((uint32_t)r << lsum) << kKeyLog2);
                const uint32_t visits =
                    walk_entry<kStats, Key>(ra, rb, o, sens.w & 0xffff, base, H, MD, t0, blo, ext, shb, cut);
                if (kStats && visits) atomicAdd(&s_vis[r], visits);
            }
            __syncthreads();
            if (cached) {
                // each voxel applies the group's scans in submission order,
                // its cached state held in registers across them
                uint32_t upd[kGroup];
#pragma unroll
                for (int r = 0; r < kGroup; ++r) upd[r] = 0;
                for (uint32_t v = threadIdx.x; v < tvox; v += kTileBlock) {
                    int32_t vs = 0, vw = 0;
                    bool touched = false;
                    if (cut && ((int32_t)(v & (ez - 1)) + t0[2] >= MD.dims[2] ||
                                (int32_t)((v >> H.lt[2]) & (ey - 1)) + t0[1] >= MD.dims[1] ||
                                (int32_t)(v >> (H.lt[1] + H.lt[2])) + t0[0] >= MD.dims[0])) {
                        for (int r = 0; r < ng; ++r) s_keys[(uint32_t)r * tvox + v] = kNone;
                        continue;
                    }
#pragma unroll
                    for (int r = 0; r < kGroup; ++r) {
                        if (r >= ng) break;
                        Key *kp = &s_keys[(uint32_t)r * tvox + v];
                        const Key key = *kp;
                        if (key == kNone) continue;
                        if (!touched) {
                            vs = c_sdf[v];
                            vw = c_w[v];
                            touched = true;
                        }
                        merge_one(vs, vw, key_value(key, kshift), MD.w_max);
                        *kp = kNone;
                        ++upd[r];
                    }
                    if (touched) {
                        c_sdf[v] = (int16_t)vs;
                        c_w[v] = (int16_t)vw;
                    }
                }
                if (kStats)
                    for (int r = 0; r < ng; ++r)
                        if (upd[r]) atomicAdd(&s_upd[r], upd[r]);
            } else {
                const uint32_t updated = merge_tile_direct<kTileBlock, Key>(s_keys, tvox, H, MD, t0, cut);
                if (kStats && updated) atomicAdd(&s_upd[0], updated);
            }
            __syncthreads();
            if (threadIdx.x < (uint32_t)ng) {
                const uint32_t k = (uint32_t)s_list[j0 + threadIdx.x] * H.gtiles + g;  // sequence slot, tile
                B.counts[k] = 0;  // ready for the next batch
                if (kStats) {
                    B.tile_vis[k] = s_vis[threadIdx.x];
                    B.tile_upd[k] = s_upd[threadIdx.x];
                }
            }
        }
        if (cached) {
            for (uint32_t v = threadIdx.x; v < tvox; v += kTileBlock) {
                const int32_t rz = (int32_t)(v & (ez - 1)) + t0[2];
                const int32_t ry = (int32_t)((v >> H.lt[2]) & (ey - 1)) + t0[1];
                const int32_t rx = (int32_t)(v >> (H.lt[1] + H.lt[2])) + t0[0];
                if (rx >= MD.dims[0] || ry >= MD.dims[1] || rz >= MD.dims[2]) continue;
                const int64_t slot = slot_of_rel(MD, rx, ry, rz);
                glob(MD.sdf)[slot] = c_sdf[v];
                glob(MD.w)[slot] = c_w[v];
            }
        }
        // next tile from this workgroup's queue
        if (threadIdx.x == 0)
            s_job = gridDim.x + queue + nq * atomicAdd(&B.ctl->work[queue * kQueueStride], 1u);
        __syncthreads();
        job = uniform(s_job);
    }
}

// The tile pass for the lists of one binning pass (one scan per map): jobs and
// queues as in k_tile. A tile's segments are gathered by the first wave, up to
// 64 at a time: those of the list, then three nodes of each chain (a chain is a
// load after a load, so 16 are followed together); an entry finds its segment
// in their prefix sums. Bound by latency: each tile is a chain of dependent
// loads, as in k_tile, for a hundred entries (128 x 1024 points: 22.6 us against
// k_tile's 24.0, which had its runs laid out for it by two launches more).
template <int kTileBlock, bool kStats, typename Key>
__global__ __launch_bounds__(kTileBlock) __attribute__((amdgpu_waves_per_eu(kTileWaves))) void k_tile_once(BatchArrays B)
{
    constexpr Key kNone = (Key)~(Key)0;
    constexpr int kKeyLog2 = sizeof(Key) == 4 ? 2 : 3, kHops = 3;
    static_assert(kSegs + kHops * kChains <= 64, "a lane per segment");
    extern __shared__ uint64_t s_dyn[];
    Key *s_keys = reinterpret_cast<Key *>(s_dyn);
    // per segment gathered: its place less the entries of those before it, and
    // the entries up to its end
    __shared__ uint32_t s_off[64], s_end[64];
    __shared__ uint32_t s_vis, s_upd, s_more, s_job;
    const BatchHdr H = *B.hdr;
    const uint32_t tvox = 1u << (H.lt[0] + H.lt[1] + H.lt[2]);
    const uint32_t turn = B.ctl->turn;
    BatchCtl *ctl = B.ctl + 1u + turn;
    const uint32_t nheavy = ctl->n_nonempty, nne = nheavy + ctl->n_light;
    if (blockIdx.x == 0) {
        // the next batch's counters
        uint32_t *other = reinterpret_cast<uint32_t *>(B.ctl + (2u - turn));
        if (threadIdx.x == 0) B.ctl->next_turn = 1u - turn;
        for (uint32_t j = threadIdx.x; j < sizeof(BatchCtl) / 4; j += kTileBlock) other[j] = 0;
    }
    if (kStats) {
        // a scan's valid points, over its binning blocks
        for (uint32_t s = blockIdx.x; s < (uint32_t)H.nscans; s += gridDim.x) {
            const ScanDev &SD = B.scans[s];
            const uint32_t nb = (uint32_t)((SD.n + H.bin_block - 1) / H.bin_block);
            if (threadIdx.x == 0) s_vis = 0;
            __syncthreads();
            uint32_t val = 0;
            for (uint32_t b = threadIdx.x; b < nb; b += kTileBlock) val += B.valid_part[SD.block0 + b];
            if (val) atomicAdd(&s_vis, val);
            __syncthreads();
            if (threadIdx.x == 0) B.scan_stats[s * kStatWords + 2u] = s_vis;
        }
    }
    const int32_t shb[3] = {H.lt[1] + H.lt[2] + kKeyLog2, H.lt[2] + kKeyLog2, kKeyLog2};
    const int32_t ext[3] = {1 << H.lt[0], 1 << H.lt[1], 1 << H.lt[2]};
    const uint32_t wl = threadIdx.x < 64u ? threadIdx.x : 64u;  // lane of the first wave
    uint32_t job = blockIdx.x;
    if (job >= nne) return;
    const uint32_t nq = gridDim.x < (uint32_t)kQueues ? gridDim.x : (uint32_t)kQueues;
    const uint32_t queue = blockIdx.x % nq;
    for (uint32_t v = threadIdx.x; v < tvox; v += kTileBlock) s_keys[v] = kNone;
    while (job < nne) {
        const bool from_heavy = job < nheavy;
        uint32_t g, mb;
        if (from_heavy) {
            g = uniform(B.offsets[job]);
            mb = uniform(B.cursor[job]);
        } else {
            const uint4 jb = B.jobs[job - nheavy];
            g = uniform(jb.x);
            mb = uniform(jb.y);
        }
        TileList *L = &B.lists[g];
        const unsigned long long head = *reinterpret_cast<const unsigned long long *>(L);  // in one access
        const uint32_t nseg = uniform((uint32_t)head), total = uniform((uint32_t)(head >> 32));
        // (a heavy tile is listed twice: whoever took it from the heavy ones does
        // it, before or after the other looked)
        if (nseg && (total >= kHeavyTile) == from_heavy) {
            const MapDev MD = uniform_map(B.maps[mb]);
            const int4 sens = B.seq_sensor[mb];
            const int32_t o[3] = {uniform(sens.x), uniform(sens.y), uniform(sens.z)};
            const int32_t tau = uniform(sens.w);
            uint32_t cur = 0;
            uint2 mine = make_uint2(0u, 0u);
            if (wl < kSegs && wl < nseg) mine = L->seg[wl];
            if (wl >= 16u && wl < 16u + kChains && nseg > kSegs) cur = L->chain[wl - 16u];
            if (kStats && threadIdx.x == 0) s_vis = s_upd = 0;
            const uint32_t t = g - MD.tile_base;
            const uint32_t tz = t % (uint32_t)MD.nt[2];
            const uint32_t txy = t / (uint32_t)MD.nt[2];
            const int32_t t0[3] = {(int32_t)(txy / (uint32_t)MD.nt[1]) << H.lt[0],
                                   (int32_t)(txy % (uint32_t)MD.nt[1]) << H.lt[1], (int32_t)tz << H.lt[2]};
            int32_t blo[3];
            bool cut = false;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                blo[a] = MD.origin[a] + t0[a];
                cut = cut || t0[a] + (1 << H.lt[a]) > MD.dims[a];
            }
            uint32_t visits = 0;
            bool more = true;
            while (more) {
                if (wl < 64u) {
                    // segment of lane s: s < kSegs of the list, then hop h of chain c
                    // in lane kSegs + 16 h + c
                    uint2 sg = mine;
                    mine = make_uint2(0u, 0u);
#pragma unroll
                    for (int h = 0; h < kHops; ++h) {
                        uint4 nd = make_uint4(0u, 0u, 0u, 0u);
                        if (cur) nd = B.nodes[cur - 1u];
                        cur = nd.x;
                        const int from = (int)wl - (int)kSegs - (int)kChains * h + 16;  // the chain's lane
                        const uint32_t x = (uint32_t)__shfl((int)nd.y, from & 63), y = (uint32_t)__shfl((int)nd.z, from & 63);
                        if (from >= 16 && from < 16 + (int)kChains) sg = make_uint2(x, y);
                    }
                    uint32_t p = sg.y;
#pragma unroll
                    for (int off = 1; off < 64; off <<= 1) {
                        const uint32_t v = (uint32_t)__shfl_up((int)p, off);
                        if (wl >= (uint32_t)off) p += v;
                    }
                    s_off[wl] = sg.x - (p - sg.y);
                    s_end[wl] = p;
                    const bool left = __any(cur != 0u);
                    if (wl == 0u) s_more = left ? 1u : 0u;
                }
                __syncthreads();
                const uint32_t n = uniform(s_end[63]);
                more = uniform(s_more) != 0u;
                for (uint32_t e = threadIdx.x; e < n; e += kTileBlock) {
                    uint32_t j = 0;
#pragma unroll
                    for (uint32_t step = 32; step > 0; step >>= 1) j += s_end[j + step - 1u] <= e ? step : 0u;
                    const uint32_t at = s_off[j] + e;
                    visits += walk_entry<kStats, Key>(B.entries[at], B.entries2[at], o, tau, lds_address(s_keys), H, MD,
                                                      t0, blo, ext, shb, cut);
                }
                __syncthreads();
            }
            // the list is empty again for the next batch
            if (wl == 0u) *reinterpret_cast<unsigned long long *>(L) = 0ull;
            if (nseg > kSegs && wl >= 16u && wl < 16u + kChains) L->chain[wl - 16u] = 0u;
            const uint32_t updated = merge_tile_direct<kTileBlock, Key>(s_keys, tvox, H, MD, t0, cut);
            if (kStats) {
                if (visits) atomicAdd(&s_vis, visits);
                if (updated) atomicAdd(&s_upd, updated);
                __syncthreads();
                if (threadIdx.x == 0)
                    atomicAdd(reinterpret_cast<unsigned long long *>(
                                  &B.scan_stats[mb * kStatWords + g % kStatParts * 16u]),  // (scan k is map k's)
                              (unsigned long long)s_vis << 32 | s_upd);
            }
        } else {
            __syncthreads();  // every wave has read s_job
        }
        if (threadIdx.x == 0)
            s_job = gridDim.x + queue + nq * atomicAdd(&ctl->work[queue * kQueueStride], 1u);
        __syncthreads();
        job = uniform(s_job);
    }
}

// Per-scan counts (one workgroup per scan): voxels updated and visits over
// the scan's (sequence slot, tile) records, which it clears again, and
// points with a ray over the scan's binning blocks.
__global__ __launch_bounds__(256) void k_stats(BatchArrays B)
{
    __shared__ uint32_t s_sum[3][256];
    const BatchHdr H = *B.hdr;
    const uint32_t s = blockIdx.x;
    if (!H.want_stats || s >= (uint32_t)H.nscans) return;
    const ScanDev &SD = B.scans[s];
    const MapDev &MD = B.maps[SD.map];
    uint32_t vis = 0, upd = 0, val = 0;
    const uint32_t k0 = (uint32_t)SD.seq * H.gtiles + MD.tile_base;
    for (uint32_t t = threadIdx.x; t < MD.ntot; t += 256) {
        vis += B.tile_vis[k0 + t];
        upd += B.tile_upd[k0 + t];
        B.tile_vis[k0 + t] = 0;
        B.tile_upd[k0 + t] = 0;
    }
    const uint32_t nb = (uint32_t)((SD.n + H.bin_block - 1) / H.bin_block);
    for (uint32_t b = threadIdx.x; b < nb; b += 256) val += B.valid_part[SD.block0 + b];
    s_sum[0][threadIdx.x] = upd;
    s_sum[1][threadIdx.x] = val;
    s_sum[2][threadIdx.x] = vis;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (threadIdx.x < (uint32_t)off)
            for (int j = 0; j < 3; ++j) s_sum[j][threadIdx.x] += s_sum[j][threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        B.scan_stats[4 * s + 0] = s_sum[0][0];
        B.scan_stats[4 * s + 1] = s_sum[1][0];
        B.scan_stats[4 * s + 2] = s_sum[2][0];
        B.scan_stats[4 * s + 3] = B.ctl->overflow;
    }
}

__global__ void k_fill_u32(uint32_t *p, int64_t n, uint32_t v)
{
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x)
        p[j] = v;
}

}  // namespace

// Entries one point can emit: the tiles its band segment's walk visits.
int32_t max_tiles_per_ray(int32_t tau, const int32_t lt[3]) { return band_tiles_bound(tau, lt); }

namespace {

template <int kBB>
void launch_bin(int mode, uint32_t bins, const BatchArrays &B, const InlineDesc &I, hipStream_t stream)
{
    const dim3 grid(bins), block(kBB);
    if (mode == kFillRuns) hipLaunchKernelGGL((k_bin<kFillRuns, kBB, false>), grid, block, 0, stream, B, I);
    else if (mode == kCount && I.on) hipLaunchKernelGGL((k_bin<kCount, kBB, true>), grid, block, 0, stream, B, I);
    else if (mode == kCount) hipLaunchKernelGGL((k_bin<kCount, kBB, false>), grid, block, 0, stream, B, I);
    else if (I.on) hipLaunchKernelGGL((k_bin<kOnce, kBB, true>), grid, block, 0, stream, B, I);
    else hipLaunchKernelGGL((k_bin<kOnce, kBB, false>), grid, block, 0, stream, B, I);
}

void launch_bin_any(int mode, uint32_t bins, uint32_t block, const BatchArrays &B, const InlineDesc &I,
                    hipStream_t stream)
{
    if (block == 128) launch_bin<128>(mode, bins, B, I, stream);
    else if (block == 512) launch_bin<512>(mode, bins, B, I, stream);
    else launch_bin<256>(mode, bins, B, I, stream);
}

template <int kTB, bool kStats, typename Key>
void launch_tile_as(const LaunchCaps &caps, const BatchArrays &B, hipStream_t stream)
{
    const dim3 grid((uint32_t)caps.tile_grid), block(kTB);
    if (caps.once) hipLaunchKernelGGL((k_tile_once<kTB, kStats, Key>), grid, block, caps.tile_lds, stream, B);
    else hipLaunchKernelGGL((k_tile<kTB, kStats, Key>), grid, block, caps.tile_lds, stream, B);
}

template <int kTB>
void launch_tile(const LaunchCaps &caps, const BatchArrays &B, hipStream_t stream)
{
    if (caps.key32 && caps.stats) launch_tile_as<kTB, true, uint32_t>(caps, B, stream);
    else if (caps.key32) launch_tile_as<kTB, false, uint32_t>(caps, B, stream);
    else if (caps.stats) launch_tile_as<kTB, true, uint64_t>(caps, B, stream);
    else launch_tile_as<kTB, false, uint64_t>(caps, B, stream);
}

}  // namespace

TilePlan tile_plan(const int32_t lt[3], int32_t S, int32_t tau, int64_t max_points, int32_t tile_block, int32_t cus)
{
    TilePlan P;
    P.key_shift = key32_shift(tau, max_points);
    const int64_t key = P.key_shift ? 4 : 8, most = P.key_shift ? kMaxGroup32 : kMaxGroup64;
    // LDS of a tile workgroup: G key buffers and the cached tile (4 bytes per
    // voxel). G as large as lets the workgroups a CU holds (kTileWaves per
    // 256 threads) share its 160 KB, 128 granules of 1280 bytes; the
    // persistent grid fills the CUs.
    const int64_t tvox = (int64_t)1 << (lt[0] + lt[1] + lt[2]);
    const int64_t granules = 128 / kTileWaves;  // of 1280 bytes, per 256 threads
    const int64_t budget = granules * 1280 * (tile_block / 256) - kTileStaticLds;
    const int64_t gfit = (budget / tvox - 4) / key;
    P.G = (int32_t)std::max<int64_t>(1, std::min<int64_t>({gfit, most, (int64_t)S}));
    P.lds = (uint32_t)((key * P.G + 4) * tvox);
    const int by_waves = 4 * kTileWaves / (tile_block / 64);  // four SIMDs
    const int per_cu = (int)std::max<size_t>(
        1, std::min<size_t>((size_t)by_waves, (size_t)(160 * 1024) / (P.lds + (uint32_t)kTileStaticLds)));
    P.grid = cus * per_cu;
    return P;
}

bool launch_blocks_ok(int32_t bin_block, int32_t tile_block)
{
    return (bin_block == 128 || bin_block == 256 || bin_block == 512) && (tile_block == 256 || tile_block == 512);
}

hipError_t launch_batch(const BatchArrays &B, const LaunchCaps &caps, hipStream_t stream, hipEvent_t ev_start,
                        hipEvent_t ev_binned, hipEvent_t ev_tiles, const InlineDesc *inl)
{
    hipError_t e;
    if (ev_start && (e = hipEventRecord(ev_start, stream)) != hipSuccess) return e;
    const uint32_t bins = caps.blocks > 0 ? caps.blocks : 1u;
    InlineDesc none;
    memset(&none, 0, sizeof(none));
    if (caps.rows) hipLaunchKernelGGL(k_rows, dim3((caps.scans + 3) / 4), dim3(256), 0, stream, B);
    if (caps.once) {
        launch_bin_any(kOnce, bins, caps.bin_block, B, inl ? *inl : none, stream);
    } else {
        launch_bin_any(kCount, bins, caps.bin_block, B, inl ? *inl : none, stream);
        hipLaunchKernelGGL(k_alloc, dim3((caps.gtiles + kAllocTiles - 1) / kAllocTiles), dim3(kAllocBlock), 0, stream,
                           B);
        launch_bin_any(kFillRuns, bins, caps.bin_block, B, none, stream);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (ev_binned && (e = hipEventRecord(ev_binned, stream)) != hipSuccess) return e;
    // the per-scan counts are a template switch: without them the walk and
    // the merges carry no counters
    if (caps.tile_block == 512) launch_tile<512>(caps, B, stream);
    else launch_tile<256>(caps, B, stream);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (ev_tiles && (e = hipEventRecord(ev_tiles, stream)) != hipSuccess) return e;
    if (caps.stats && !caps.once) hipLaunchKernelGGL(k_stats, dim3(caps.scans > 0 ? caps.scans : 1u), dim3(256), 0, stream, B);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill_u32, dim3((uint32_t)blocks), dim3(256), 0, stream, p, n, v);
    return hipGetLastError();
}

}  // namespace tsdf
