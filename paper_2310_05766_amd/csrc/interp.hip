// Vertical interpolation between scan lines (FeatSense, arXiv 2310.05766,
// Sec. VI, Eq. (3) and Eq. (4)): every band voxel of a ray also gives its
// value to the voxels along the interpolation vector int = d x (d x up),
// up to the height h = delta_z * len above and below the ray, where len is
// the voxel's distance along the ray. The filled voxels of one band voxel
// are the exact floor-set of the segment [c - e, c + e] around its centre c,
// with e = h int / |int| in fixed point; each receives the band voxel's key,
// and the per-scan minimum over all keys (band and fill, all rays) decides.
//
// A fill reaches across tiles, so this form does not use the tiled engine:
// candidates meet in a key volume over the window (all ~0 between scans) by
// atomicMin, with one byte per run of 64 slots that tells whether it holds a
// key (a plain store: an atomic that returns the old key, to mark only on the
// first candidate, is slower). Scattered atomics run at about 20 per ns on this
// card, whatever they hit, and a band voxel is met by neighbouring rays: a block
// takes a patch of rays and merges its candidates in LDS (KeyTable) before any
// goes out. A second kernel, one wave per 64 runs, merges the keys of touched
// runs (Eq. (1), Eq. (2)) and empties them again. Keys are 32 bits wide where
// tau and the point count let them (key32_shift), else 64: half the bytes in the
// table and in the merge. 128 x 1024 points in a 512 x 512 x 256 window, fills
// of 3.8 M visits: 206 us + 53 us of merge with a ray per lane and 3.83 M 64-bit
// atomics, now 109 us + 38 us with 1.23 M.
//
// Free-space carving uses the same key volume: a ray longer than tau also
// walks [o, S] from the sensor to the start of its band (the long walk, clipped
// to the window), whose voxels take the ray's key like band voxels. With 32-bit
// keys a scan takes three kernels:
//   k_carve_band   the band, and the last voxels before S whose distance is
//                  not truncated: 32-bit atomicMin, and a mark per voxel that
//                  got a key, 2 where its |s| is tau, 4 where it is less
//   k_carve_free   the free space proper, where every candidate is +tau. Such
//                  a candidate changes a voxel only where nothing lies below
//                  it, so it needs no atomic: it leaves the mark 1 on an
//                  unmarked voxel (a plain byte store, the same from every
//                  ray) and nothing elsewhere; only where the band left |s| =
//                  tau (mark 2) does the point index decide between +tau and
//                  -tau, and the candidate's key is offered like the band's
//   k_carve_merge  marks 1 take +tau, other marks their key
// The marks lie in the second half of the key volume (an unmarked voxel is ~0
// like an empty key, so that either width finds the volume as it needs it),
// an eighth of the bytes of 64-bit keys. On the same points (24.6 M visits, 7.3 M
// voxels updated) the free space took 6.6 M atomics before, and the scan 581 us +
// 94 us of merge; the three kernels take 54, 79 and 76 us.
// Wider scans go through k_carve_scan and 64-bit keys: a visit reads the key
// first and issues the atomic only when it would lower it (keys only fall
// during a scan, so a stale read at worst costs an atomic), and marks the run
// only when it read EMPTY; that path is bound by how many scattered 64-bit
// atomics and stores the L2 takes per second.
//
// Integer ranges (all exact): d = rdiv(1024 D, r) has |d| <= 1026, the up
// vector U is in 1/1024 units, so |int| < 2^31 and int . int < 2^62; a fill
// applies to rays of r < 2^30 (|D|^2 < 2^62); h is capped at 65535 (64
// voxels), so a fill segment spans |2 e_a| < 2^17 per axis, the range the
// exact walk is built for.
#include <algorithm>

#include "internal.hpp"

namespace tsdf {

namespace {

constexpr int kInterpBlock = 256;
// Blocks of the band scans: a patch of 64 rays (8 rows), whose candidates meet
// in the block's table. Neighbouring lanes share a ray, each taking every
// kFillLanes-th (kBandLanes-th) voxel of its band: bands differ a lot in length
// and in the length of their fills, and a ray on one lane kept the launch
// waiting for its longest. Interpolating 128 x 1024 points: 202 us with a ray
// per lane and 256 rays per block, 116 with 4 lanes and 64 rays, 109 with a
// table twice as large; 2 and 8 lanes 147 and 139. (Carving's bands, without
// fills: 58, 62, 62; 54 with 2 lanes. Its atomics alone take 43 us.)
constexpr int kKeyRays = 64, kFillLanes = 4, kBandLanes = 2;
constexpr int kCarveChunkLog2 = 3;
constexpr int kCarvePieces = 16;  // of a ray's free segment, one wave each per 64 rays
constexpr int kCarveAhead = 2;    // voxels whose marks are requested together

// rdiv(n, d) = sign(n) floor((2|n| + d) / 2d), to nearest with ties away
// from zero, for a divisor 0 < d < 2^32 fixed per ray (given as 2d and
// 1 / 2d correctly rounded) and |n| < 2^61 with a quotient below 2^31: the
// float64 estimate is within one of the quotient, and one exact 64-bit
// correction each way fixes it (no integer division). Here, once per ray:
// d = r < 2^30 with n = 1024 D_a (the fills of each band voxel take the
// float64 forms band_len and fill_offset).
__device__ __forceinline__ int64_t rdiv_by(int64_t n, uint64_t d2, double inv_d2)
{
    const uint64_t a = (uint64_t)(n < 0 ? -n : n);
    const uint64_t num = 2 * a + (d2 >> 1);
    uint64_t k = (uint64_t)((double)num * inv_d2);
    k -= k * d2 > num ? 1u : 0u;
    k += (k + 1) * d2 <= num ? 1u : 0u;
    return n < 0 ? -(int64_t)k : (int64_t)k;
}

// Slot of a voxel inside the window: floor_mod(g_a, dims_a) per axis, z
// fastest.
__device__ __forceinline__ int64_t window_slot(const InterpScan &P, const int32_t g[3])
{
    int64_t sl = 0;
    for (int a = 0; a < 3; ++a) {
        int32_t v = g[a] - P.origin[a] + P.ring0[a];
        v -= v >= P.dims[a] ? P.dims[a] : 0;
        sl = sl * P.dims[a] + v;
    }
    return sl;
}

// Eq. (1) with one unit of weight, Eq. (2) (|g w + v| <= tau (w + 1)).
__device__ __forceinline__ void merge_value(int16_t &sdf, int16_t &w, int32_t v, int32_t w_max)
{
    const int32_t gw = w;
    sdf = (int16_t)rdiv_small(sdf * gw + v, gw + 1);
    w = (int16_t)(gw + 1 < w_max ? gw + 1 : w_max);
}

// s of a key of the volume.
__device__ __forceinline__ int32_t volume_value(const InterpScan &, uint64_t key)
{
    return (int16_t)(uint16_t)(key & 0xffffu);
}
__device__ __forceinline__ int32_t volume_value(const InterpScan &P, uint32_t key)
{
    return tile_key_sdf(key, P.key_shift);
}

// Adds a block's sum to its counter of one kind (kCtrLines of them per kind, a
// 128-byte line each: additions on one address queue).
__device__ __forceinline__ void block_add(uint64_t v, const InterpScan &P, int kind)
{
    if (kind != kCtrAtomics && !P.want_stats) return;
    __shared__ unsigned long long s_sum;
    if (threadIdx.x == 0) s_sum = 0;
    __syncthreads();
    if (v) atomicAdd(&s_sum, (unsigned long long)v);
    __syncthreads();
    if (threadIdx.x == 0 && s_sum)
        atomicAdd(&P.counters[(kind * kCtrLines + blockIdx.x % kCtrLines) * kCtrStride], s_sum);
    __syncthreads();
}

// Window-relative index of a voxel (marks; no ring).
__device__ __forceinline__ uint32_t rel_index(const InterpScan &P, const int32_t g[3])
{
    return ((uint32_t)(g[0] - P.origin[0]) * (uint32_t)P.dims[1] + (uint32_t)(g[1] - P.origin[1])) * (uint32_t)P.dims[2] +
           (uint32_t)(g[2] - P.origin[2]);
}

// Ring slot of a window-relative index.
__device__ __forceinline__ uint32_t slot_of_index(const InterpScan &P, uint32_t idx)
{
    const uint32_t row = idx / (uint32_t)P.dims[2];
    int32_t z = (int32_t)(idx - row * (uint32_t)P.dims[2]) + P.ring0[2];
    const uint32_t rx = row / (uint32_t)P.dims[1];
    int32_t y = (int32_t)(row - rx * (uint32_t)P.dims[1]) + P.ring0[1], x = (int32_t)rx + P.ring0[0];
    x -= x >= P.dims[0] ? P.dims[0] : 0;
    y -= y >= P.dims[1] ? P.dims[1] : 0;
    z -= z >= P.dims[2] ? P.dims[2] : 0;
    return ((uint32_t)x * (uint32_t)P.dims[1] + (uint32_t)y) * (uint32_t)P.dims[2] + (uint32_t)z;
}

__device__ __forceinline__ void lds_key_min(uint32_t *p, uint32_t k) { atomicMin(p, k); }
__device__ __forceinline__ void lds_key_min(uint64_t *p, uint64_t k)
{
    atomicMin((unsigned long long *)p, (unsigned long long)k);
}

// A block's candidates, merged in LDS before any goes to the key volume: a
// table of voxel (window-relative index) and smallest key. Neighbouring rays
// meet the same voxels (3.8 candidates a voxel on 128 x 1024 interpolated
// points), a block holds a patch of rays, and scattered atomics run at about 20
// per ns whatever they hit, so that each one saved is time saved. A candidate
// that finds its places taken goes to the volume by itself.
template <typename Key, int kBlock, int kLog2>
struct KeyTable {
    static constexpr Key kNone = (Key)~(Key)0;
    static constexpr uint32_t kSlots = 1u << kLog2, kProbes = 8;
    uint32_t idx[kSlots];
    Key key[kSlots];

    __device__ __forceinline__ void clear()
    {
        for (uint32_t j = threadIdx.x; j < kSlots; j += kBlock) {
            idx[j] = 0xffffffffu;  // (a window has fewer than 2^31 voxels)
            key[j] = kNone;
        }
        __syncthreads();
    }
    __device__ __forceinline__ bool offer(uint32_t at, Key k)
    {
        uint32_t h = (at * 2654435761u) >> (32 - kLog2);
        for (uint32_t p = 0; p < kProbes; ++p) {
            uint32_t there = idx[h];
            if (there == 0xffffffffu) there = atomicCAS(&idx[h], 0xffffffffu, at);
            if (there == 0xffffffffu || there == at) {
                lds_key_min(&key[h], k);
                return true;
            }
            h = (h + 1u) & (kSlots - 1u);
        }
        return false;
    }
    // send(voxel, smallest key) for every voxel met; the sum of what it returns
    template <class Send>
    __device__ __forceinline__ uint64_t flush(Send send)
    {
        __syncthreads();
        uint64_t n = 0;
        for (uint32_t j = threadIdx.x; j < kSlots; j += kBlock)
            if (idx[j] != 0xffffffffu) n += send(idx[j], key[j]);
        return n;
    }
};

// One candidate to the key volume, its run of 64 slots marked; 1 (an atomic).
__device__ __forceinline__ uint32_t send_key(const InterpScan &P, uint32_t idx, uint32_t key)
{
    const uint32_t slot = slot_of_index(P, idx);
    atomicMin(&P.keys32[slot], key);
    P.touched[slot >> 6] = 1;
    return 1;
}
__device__ __forceinline__ uint32_t send_key(const InterpScan &P, uint32_t idx, uint64_t key)
{
    const uint32_t slot = slot_of_index(P, idx);
    atomicMin(&P.keys[slot], (unsigned long long)key);
    P.touched[slot >> 6] = 1;
    return 1;
}

// Whether no voxel within `reach` voxels of a ray's band lies in the window.
__device__ __forceinline__ bool band_outside(const InterpScan &P, const Ray &R, int32_t reach)
{
    bool out = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int32_t g0 = min(R.S[a], R.E[a]) >> 10, g1 = max(R.S[a], R.E[a]) >> 10;
        out = out || g1 + reach < P.origin[a] || g0 - reach >= P.origin[a] + P.dims[a];
    }
    return out;
}

template <typename Key>
__global__ __launch_bounds__(kKeyRays * kFillLanes) void k_interp_scan(InterpScan P, uint32_t block0)
{
    __shared__ KeyTable<Key, kKeyRays * kFillLanes, sizeof(Key) == 4 ? 12 : 11> T;
    __shared__ Row s_row;
    const bool tries = P.rings != 0;
    if (tries && threadIdx.x < 64u) s_row = find_row(P.xyz, P.n, P.rings, kKeyPatch);
    T.clear();
    const Row row = tries ? uniform_row(s_row) : P.row;
    const int64_t i = patch_point<kKeyRays, kKeyPatch.rows>(block0 + blockIdx.x, threadIdx.x / kFillLanes, row);
    const int sub = (int)(threadIdx.x % kFillLanes);
    uint64_t valid = 0, visits = 0, atomics = 0;
    int32_t q[3];
    Ray R;
    if (i < P.n && quantise(P.xyz[3 * i], P.xyz[3 * i + 1], P.xyz[3 * i + 2], P.rp, q) && make_ray(q, P.rp, R)) {
        valid = sub == 0 ? 1 : 0;
        const int64_t rr = (int64_t)R.r;
        int64_t Di[3], v[3] = {0, 0, 0}, nv = 0, dd = 0;
        double vd[3] = {0.0, 0.0, 0.0}, nvh = 0.0, tt = 0.0;
        for (int a = 0; a < 3; ++a) Di[a] = (int64_t)R.D[a];
        const bool fills = P.dq > 0 && rr < ((int64_t)1 << 30);
        const uint64_t r2 = 2 * (uint64_t)rr;
        const double inv_r2 = 1.0 / (double)r2;
        uint64_t nv2 = 0;
        double inv_nv2 = 0.0;
        if (fills) {
            int64_t d[3], w[3];
            for (int a = 0; a < 3; ++a) {
                d[a] = rdiv_by(1024 * Di[a], r2, inv_r2);
                dd += Di[a] * Di[a];
            }
            w[0] = d[1] * P.up[2] - d[2] * P.up[1];
            w[1] = d[2] * P.up[0] - d[0] * P.up[2];
            w[2] = d[0] * P.up[1] - d[1] * P.up[0];
            v[0] = d[1] * w[2] - d[2] * w[1];
            v[1] = d[2] * w[0] - d[0] * w[2];
            v[2] = d[0] * w[1] - d[1] * w[0];
            nv = (int64_t)isqrt_u64((uint64_t)(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]));
            nv2 = 2 * (uint64_t)nv;
            inv_nv2 = nv > 0 ? 1.0 / (double)nv2 : 0.0;
            for (int a = 0; a < 3; ++a) vd[a] = (double)v[a];
            nvh = (double)nv + 0.5;
            tt = (double)(dd - rr * rr);  // |D|^2 - r^2, in [0, 2r]
        }
        // (a fill reaches 64 voxels at most, and less the nearer the ray: its
        // height grows with the voxel's distance along the ray, len = rdiv((c - o)
        // . D, r). The band ends (1 + tau / r) |D| from the sensor, a centre lies
        // within 888 units of it, and |D|^2 <= r^2 + 2r, so len is at most
        // (r + tau)(1 + 2 / r) + 888 sqrt(3): a few units from the sensor much
        // more than r + tau)
        const double reach = (R.r + (double)P.rp.tau) * (1.0 + 4.0 * R.inv_r2) + 2048.0;
        const double top = fills ? fmin((double)P.dq * reach * 0x1p-30 + 3.0, 66.0) : 0.0;
        Walk W;
        walk_init(R, W);
        bool more = !band_outside(P, R, (int32_t)top);
        for (int k = 0; k < sub; ++k) more = more && walk_next(W);
        const double taud = (double)P.rp.tau, rh = R.r + 0.5;
        const uint32_t ihi = (uint32_t)i >> 16, ilo = (uint32_t)i << 16;
        while (more) {
            // a voxel of the band walk: band_key is pack_key(voxel_sdf(...))
            const Key key = sizeof(Key) == 4 ? (Key)tile_key32(W.n, rh, R.inv_r2, taud, P.key_shift, (uint32_t)i)
                                             : (Key)band_key(W.n, rh, R.inv_r2, taud, ihi, ilo);
            // the fill segment of this band voxel: [c - e, c + e]
            int64_t e[3] = {0, 0, 0};
            if (fills && nv > 0) {
                // len = rdiv((c - o) . D, r), (c - o) . D = |D|^2 - n
                const double len = band_len(W.n, tt, R);
                if (len > 0.0) {
                    // h = rdiv(dq len, 2^20): dq len < 2^51 is exact, the
                    // scaling by 2^-20 too
                    const double h = fmin(floor(__fma_rn((double)P.dq, len, 524288.0) * 0x1p-20), 65535.0);
                    for (int a = 0; a < 3; ++a) e[a] = fill_offset(h * vd[a], nvh, inv_nv2);
                }
            }
            Ray F;  // a segment only: the fill walk needs no distances
            for (int a = 0; a < 3; ++a) {
                const int32_t c = 1024 * W.g[a] + 512;
                F.S[a] = c - (int32_t)e[a];
                F.E[a] = c + (int32_t)e[a];
                F.q[a] = 0;
                F.D[a] = 0.0;
            }
            Walk FW;
            walk_init(F, FW);
            do {
                bool inside = true;
                for (int a = 0; a < 3; ++a)
                    inside = inside && FW.g[a] >= P.origin[a] && FW.g[a] < P.origin[a] + P.dims[a];
                if (inside) {
                    const uint32_t idx = rel_index(P, FW.g);
                    if (!T.offer(idx, key)) atomics += send_key(P, idx, key);
                    ++visits;
                }
            } while (walk_next(FW));
#pragma unroll
            for (int k = 0; k < kFillLanes; ++k) more = more && walk_next(W);
        }
    }
    atomics += T.flush([&](uint32_t idx, Key key) { return send_key(P, idx, key); });
    block_add(valid, P, kCtrValid);
    block_add(visits, P, kCtrVisits);
    block_add(atomics, P, kCtrAtomics);
}

// One candidate: the atomic only when it would lower the key read, the
// run's mark only by a thread that read EMPTY (the first atomic on a slot in
// a scan comes from such a thread: no key can be read before one is written).
// Returns 1 when it issued the atomic.
__device__ __forceinline__ uint32_t offer_key(const InterpScan &P, int64_t sl, uint64_t key)
{
    unsigned long long *k = &P.keys[sl];
    const unsigned long long seen = *k;
    if (seen > key) {
        atomicMin(k, (unsigned long long)key);
        if (seen == kEmptyKey) P.touched[sl >> 6] = 1;
        return 1;
    }
    return 0;
}

// Free-space walks of neighbouring points (consecutive indices: neighbouring
// columns of one scan line) that start in the same voxel visit the voxels
// they share at the same step, so the wave walks in lockstep and a lane
// whose left neighbour holds the same slot with a smaller key leaves the
// candidate to it (that neighbour offers it, or is covered the same way by
// a smaller key further left). A lane whose walk has ended still shows the
// last candidate it held, which was offered.
// Free-space walks differ a lot in length (a wave runs as long as its longest
// lane), so each ray's free segment is cut into chunks: chunk c walks only
// the slab of voxels [(k0 + c) C, (k0 + c + 1) C) along the segment's longest
// axis, slabs of C = 2^kCarveChunkLog2 voxels in global coordinates counted
// from the slab k0 that holds the segment's lowest voxel inside the window.
// A wave holds one chunk of 64 consecutive rays, and consecutive waves take
// the chunks of one group of rays in turn (wave w: rays 64 (w / nch) + lane,
// chunk w mod nch), which spreads the atomics near the sensor, where all rays
// meet, over the whole launch instead of its first waves. Chunk 0 also walks
// the band. Four waves per SIMD: held to five, the walk state spills.
__global__ __launch_bounds__(kInterpBlock) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_carve_scan(InterpScan P,
                                                                                                      int64_t nch,
                                                                                                      int64_t block0)
{
    // block0: this launch's first block of the whole grid (the grid may be
    // split over several launches)
    const int64_t t = (block0 + (int64_t)blockIdx.x) * kInterpBlock + threadIdx.x;
    const int64_t w = t >> 6;
    const int64_t i = (w / nch) * 64 + (t & 63);
    const int32_t chunk = (int32_t)(w % nch);
    const int lane = (int)(threadIdx.x & 63u);
    uint64_t valid = 0, visits = 0, atomics = 0;
    int32_t q[3];
    Ray R;
    int32_t lo[3], hi[3];
    for (int a = 0; a < 3; ++a) {
        lo[a] = P.origin[a];
        hi[a] = P.origin[a] + P.dims[a];
    }
    const bool ray = i < P.n && quantise(P.xyz[3 * i], P.xyz[3 * i + 1], P.xyz[3 * i + 2], P.rp, q) &&
                     make_ray(q, P.rp, R);
    FreeWalk F;
    bool act = false;
    if (ray && R.r > (double)P.rp.tau) {
        // the free segment [o, S]: its longest axis and its voxel range there
        int da = 0;
        int64_t best = -1;
        for (int a = 0; a < 3; ++a) {
            const int64_t L = (int64_t)R.S[a] - P.rp.o[a];
            const int64_t m = L < 0 ? -L : L;
            if (m > best) {
                best = m;
                da = a;
            }
        }
        const int32_t g0 = P.rp.o[da] >> 10, g1 = R.S[da] >> 10;
        int32_t gmin = g0 < g1 ? g0 : g1, gmax = g0 < g1 ? g1 : g0;
        gmin = gmin > lo[da] ? gmin : lo[da];
        gmax = gmax < hi[da] - 1 ? gmax : hi[da] - 1;
        const int32_t k = (gmin >> kCarveChunkLog2) + chunk;  // arithmetic shift: floor division
        const int32_t slo = k * (1 << kCarveChunkLog2), shi = slo + (1 << kCarveChunkLog2);
        if (gmin <= gmax && slo <= gmax) {
            lo[da] = lo[da] > slo ? lo[da] : slo;
            hi[da] = hi[da] < shi ? hi[da] : shi;
            act = lo[da] < hi[da] && free_walk_init(R, P.rp, lo, hi, F);
        }
        for (int a = 0; a < 3; ++a) {
            lo[a] = P.origin[a];
            hi[a] = P.origin[a] + P.dims[a];
        }
    }
    int64_t sl = -1;
    uint64_t key = 0;
    while (__any(act)) {
        if (act) {
            sl = window_slot(P, F.W.g);
            key = free_walk_key(F, R, P.rp.tau, (uint32_t)i);
        }
        const int64_t left_sl = __shfl_up(sl, 1);
        const uint64_t left_key = __shfl_up(key, 1);
        if (act) {
            if (!(lane > 0 && left_sl == sl && left_key <= key)) atomics += offer_key(P, sl, key);
            ++visits;
            act = free_walk_next(F);
        }
    }
    if (ray && chunk == 0) {
        valid = 1;
        Walk W;
        walk_init(R, W);
        do {
            bool inside = true;
            for (int a = 0; a < 3; ++a) inside = inside && W.g[a] >= lo[a] && W.g[a] < hi[a];
            if (inside) {
                atomics += offer_key(P, window_slot(P, W.g), pack_key(voxel_sdf(W.n, R, P.rp.tau), (uint32_t)i));
                ++visits;
            }
        } while (walk_next(W));
    }
    block_add(valid, P, kCtrValid);
    block_add(visits, P, kCtrVisits);
    block_add(atomics, P, kCtrAtomics);
}

// One wave per group of 64 runs of 64 slots: the wave reads the group's 64
// touched bytes at once and clears them, then merges the touched runs
// kMergeBatch at a time: the batch's keys are all requested together, then
// the voxels of its touched slots, so that a wave waits on two dependent
// reads per batch instead of per run.
constexpr int kMergeBatch = 8;

template <typename Key>
__global__ __launch_bounds__(256) void k_interp_merge(InterpScan P, int64_t nvox)
{
    constexpr Key kNone = (Key)~(Key)0;
    Key *keys = sizeof(Key) == 4 ? (Key *)P.keys32 : (Key *)P.keys;
    uint64_t updated = 0;
    const int64_t nruns = (nvox + 63) / 64;
    const int64_t ngroups = (nruns + 63) / 64;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64;
    const int64_t waves = (int64_t)gridDim.x * blockDim.x / 64;
    const int lane = (int)(threadIdx.x & 63u);
    for (int64_t gi = wave; gi < ngroups; gi += waves) {
        const int64_t b0 = gi * 64;
        const bool t = b0 + lane < nruns && P.touched[b0 + lane] != 0;
        if (t) P.touched[b0 + lane] = 0;
        uint64_t mask = __ballot(t);  // the same for the whole wave
        while (mask) {
            int64_t j[kMergeBatch];
            Key key[kMergeBatch];
#pragma unroll
            for (int b = 0; b < kMergeBatch; ++b) {
                j[b] = 0;
                key[b] = kNone;
                if (mask) {
                    j[b] = (b0 + __builtin_ctzll(mask)) * 64 + lane;
                    mask &= mask - 1;
                    if (j[b] < nvox) key[b] = keys[j[b]];
                }
            }
            int16_t sv[kMergeBatch], wv[kMergeBatch];
#pragma unroll
            for (int b = 0; b < kMergeBatch; ++b) {
                sv[b] = 0;
                wv[b] = 0;
                if (key[b] != kNone) {
                    sv[b] = P.sdf[j[b]];
                    wv[b] = P.w[j[b]];
                }
            }
#pragma unroll
            for (int b = 0; b < kMergeBatch; ++b) {
                if (key[b] == kNone) continue;
                merge_value(sv[b], wv[b], volume_value(P, key[b]), P.w_max);
                P.sdf[j[b]] = sv[b];
                P.w[j[b]] = wv[b];
                keys[j[b]] = kNone;
                ++updated;
            }
        }
    }
    block_add(updated, P, kCtrUpdated);
}

// --- carving with 32-bit keys ----------------------------------------------

constexpr uint8_t kNoMark = 0xff, kMarkFree = 1, kMarkTau = 2, kMarkKey = 4;
constexpr int kMarkQuads = 2, kMarkGroup = kMarkQuads * 1024;  // marks of a wave of the merge

// Where the window is large and the scan small for it, a byte per group of marks
// (in P.touched, which these scans have no other use for) tells the merge whether
// it holds any, or it would read the whole window for every scan; read first, as
// its few lines are hot. A look per newly marked voxel costs the band and the free
// space of 128 x 1024 points 18 us of 145, so the line lies where the merge of all
// marks costs more: at 2^27 voxels, and at a third of them for each step that the
// scan can take (points times the longest side). us a call, all marks / groups: 16
// x 1024 points in 512 x 512 x 256 113 / 126, in 1024 x 1024 x 512 259 / 191, in
// 1024^3 356 / 205; 2 x 256 points in 1024^3 248 / 80; 128 x 1024 points in 512 x 512
// x 256 219 / 237, in 1024 x 1024 x 512 380 / 335, in 2048 x 2048 x 128 1099 / 1170.
constexpr int64_t kGroupedWindow = (int64_t)1 << 27;
__device__ __forceinline__ void touch_group(const InterpScan &P, uint32_t idx)
{
    uint8_t *t = &P.touched[idx / (uint32_t)kMarkGroup];
    if (*t == 0) *t = 1;
}

// A candidate of the band to the volume, its voxel marked: 2 where |s| is tau,
// else 4; 1 (an atomic). Marks 2 and 4 may overwrite each other: both are
// stored only where some |s| below tau was offered, and there 2 costs the free
// space an atomic and decides nothing.
template <bool kGrouped>
__device__ __forceinline__ uint32_t send_marked(const InterpScan &P, uint32_t idx, uint32_t key)
{
    atomicMin(&P.keys32[slot_of_index(P, idx)], key);
    P.marks[idx] = (int32_t)(key >> P.key_shift) == P.rp.tau ? kMarkTau : kMarkKey;
    if (kGrouped) touch_group(P, idx);
    return 1;
}

// The axis along which a ray's free segment [o, S] is longest.
__device__ __forceinline__ int free_axis(const Ray &R, const RayParams &P)
{
    int da = 0;
    int64_t best = -1;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int64_t L = (int64_t)R.S[a] - P.o[a];
        const int64_t m = L < 0 ? -L : L;
        if (m > best) {
            best = m;
            da = a;
        }
    }
    return da;
}

// The band of each ray, and the end of its free segment: a voxel centre lies
// within 887 units (half a voxel's diagonal) of the segment's stretch in it, so
// a free voxel whose distance rounds below tau is met less than a voxel's
// length before S: in the last two voxels along the longest axis (three are
// walked).
template <bool kGrouped>
__global__ __launch_bounds__(kKeyRays * kBandLanes) void k_carve_band(InterpScan P)
{
    __shared__ KeyTable<uint32_t, kKeyRays * kBandLanes, 11> T;
    __shared__ Row s_row;
    const bool tries = P.rings != 0;
    if (tries && threadIdx.x < 64u) s_row = find_row(P.xyz, P.n, P.rings, kKeyPatch);
    T.clear();
    const Row row = tries ? uniform_row(s_row) : P.row;
    if (blockIdx.x == 0 && threadIdx.x == 0) *P.found = row;
    const int64_t i = patch_point<kKeyRays, kKeyPatch.rows>(blockIdx.x, threadIdx.x / kBandLanes, row);
    const int sub = (int)(threadIdx.x % kBandLanes);
    const auto offer = [&](const int32_t g[3], uint32_t key) -> uint32_t {
        const uint32_t idx = rel_index(P, g);
        return T.offer(idx, key) ? 0u : send_marked<kGrouped>(P, idx, key);
    };
    uint64_t valid = 0, visits = 0, atomics = 0;
    int32_t q[3];
    Ray R;
    if (i < P.n && quantise(P.xyz[3 * i], P.xyz[3 * i + 1], P.xyz[3 * i + 2], P.rp, q) && make_ray(q, P.rp, R)) {
        valid = sub == 0 ? 1 : 0;
        int32_t lo[3], hi[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = P.origin[a];
            hi[a] = P.origin[a] + P.dims[a];
        }
        if (sub == kBandLanes - 1 && R.r > (double)P.rp.tau) {
            const int da = free_axis(R, P.rp);
            int32_t tlo[3], thi[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const int32_t g1 = R.S[a] >> 10;
                tlo[a] = a == da && g1 - 2 > lo[a] ? g1 - 2 : lo[a];
                thi[a] = a == da && g1 + 3 < hi[a] ? g1 + 3 : hi[a];
            }
            FreeWalk F;
            if (thi[0] > tlo[0] && thi[1] > tlo[1] && thi[2] > tlo[2] && free_walk_init(R, P.rp, tlo, thi, F)) do {
                    if (F.u >= kFreeBias) continue;  // free space proper: k_carve_free's
                    const uint64_t key = free_walk_key(F, R, P.rp.tau, 0u);
                    const uint32_t as = (uint32_t)(key >> 48);
                    atomics += offer(F.W.g, as << P.key_shift | (uint32_t)i << 1 | (uint32_t)((key >> 15) & 1u));
                    ++visits;
                } while (free_walk_next(F));
        }
        Walk W;
        walk_init(R, W);
        const double taud = (double)P.rp.tau, rh = R.r + 0.5;
        bool more = !band_outside(P, R, 0);
        for (int k = 0; k < sub; ++k) more = more && walk_next(W);
        while (more) {
            bool inside = true;
#pragma unroll
            for (int a = 0; a < 3; ++a) inside = inside && W.g[a] >= lo[a] && W.g[a] < hi[a];
            if (inside) {
                atomics += offer(W.g, tile_key32(W.n, rh, R.inv_r2, taud, P.key_shift, (uint32_t)i));
                ++visits;
            }
#pragma unroll
            for (int k = 0; k < kBandLanes; ++k) more = more && walk_next(W);
        }
    }
    atomics += T.flush([&](uint32_t idx, uint32_t key) { return send_marked<kGrouped>(P, idx, key); });
    block_add(valid, P, kCtrValid);
    block_add(visits, P, kCtrVisits);
    block_add(atomics, P, kCtrAtomics);
}

// A visit of the free space whose voxel held mark m: 1 when it took an atomic.
template <bool kGrouped>
__device__ __forceinline__ uint32_t mark_free(const InterpScan &P, uint32_t idx, uint8_t m, uint32_t key)
{
    if (m == kNoMark) {
        P.marks[idx] = kMarkFree;
        if (kGrouped) touch_group(P, idx);
    }
    if (m != kMarkTau) return 0;
    uint32_t *k = &P.keys32[slot_of_index(P, idx)];
    if (*k <= key) return 0;
    atomicMin(k, key);
    return 1;
}

// The free space of each ray: a wave holds one of kCarvePieces equal pieces
// (along the longest axis, of the part inside the window) of a patch of 64 rays;
// consecutive waves hold the pieces of one patch. Near rays walk as FreeRun
// (about 40 instructions a step), others as FreeWalk. Bound by how many lines a
// wave's loads and stores of marks touch: the rays of neighbouring rings differ
// in z, the axis that is contiguous. Waves of 64 points of one ring, of 8 x 8,
// 32 x 2 and 64 x 1 points: 139, 79, 79, 88 us. 8, 16, 32 pieces: 88 (64 x 1),
// 79, 109 us (fewer leave the launch waiting for its longest, more set down more
// walks); 2, 4, 8 marks at a time 139, 142, 149 us (one ring).
template <bool kGrouped>
__global__ __launch_bounds__(kInterpBlock) void k_carve_free(InterpScan P, int64_t block0)
{
    const int64_t w = ((block0 + (int64_t)blockIdx.x) * kInterpBlock + threadIdx.x) >> 6;
    const int64_t i = patch_point<64, kKeyPatch.rows>((uint32_t)(w / kCarvePieces), threadIdx.x & 63u, *P.found);
    const int32_t piece = (int32_t)(w % kCarvePieces);
    uint64_t visits = 0, atomics = 0;
    int32_t q[3];
    Ray R;
    if (i < P.n && quantise(P.xyz[3 * i], P.xyz[3 * i + 1], P.xyz[3 * i + 2], P.rp, q) && make_ray(q, P.rp, R) &&
        R.r > (double)P.rp.tau) {
        const int da = free_axis(R, P.rp);
        int32_t lo[3], hi[3];
        bool some = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = P.origin[a];
            hi[a] = P.origin[a] + P.dims[a];
            if (a != da) continue;
            const int32_t g0 = P.rp.o[a] >> 10, g1 = R.S[a] >> 10;
            const int32_t gmin = max(min(g0, g1), lo[a]), gmax = min(max(g0, g1), hi[a] - 1);
            some = gmin <= gmax;
            const int32_t len = some ? gmax - gmin + 1 : 0;  // below 2^22
            lo[a] = gmin + len * piece / kCarvePieces;
            hi[a] = gmin + len * (piece + 1) / kCarvePieces;
            some = some && lo[a] < hi[a];
        }
        const uint32_t key = (uint32_t)P.rp.tau << P.key_shift | (uint32_t)i << 1;
        if (some && free_run_near(R, P.rp)) {
            FreeRun F;
            const int32_t stride[3] = {P.dims[1] * P.dims[2], P.dims[2], 1};
            bool go = free_run_init(R, P.rp, lo, hi, P.origin, stride, F);
            while (go) {
                // kCarveAhead voxels at a time: their marks are requested
                // together, a step needs none of them
                uint32_t at[kCarveAhead];
                bool on[kCarveAhead];
                uint8_t m[kCarveAhead];
#pragma unroll
                for (int k = 0; k < kCarveAhead; ++k) {
                    at[k] = F.idx;
                    on[k] = go;
                    const bool next = free_run_next(F);
                    go = go && next;
                }
#pragma unroll
                for (int k = 0; k < kCarveAhead; ++k) m[k] = on[k] ? P.marks[at[k]] : kMarkKey;
#pragma unroll
                for (int k = 0; k < kCarveAhead; ++k) {
                    atomics += mark_free<kGrouped>(P, at[k], m[k], key);
                    visits += on[k] ? 1u : 0u;
                }
            }
        } else if (some) {
            FreeWalk F;
            if (free_walk_init(R, P.rp, lo, hi, F)) do {
                    if (F.u < kFreeBias) break;  // from here on k_carve_band's
                    const uint32_t idx = rel_index(P, F.W.g);
                    atomics += mark_free<kGrouped>(P, idx, P.marks[idx], key);
                    ++visits;
                } while (free_walk_next(F));
        }
    }
    block_add(visits, P, kCtrVisits);
    block_add(atomics, P, kCtrAtomics);
}

// A wave per kMarkGroup marks: it takes the runs of 64 that hold one, kMergeBatch
// at a time (the marks from LDS; their keys and voxels requested together), and
// clears marks and keys. Bound by memory: 67 MB of marks and, at 128 x 1024
// carved points, 330 thousand runs of 64 voxels read and written, about 280 MB
// in 76 us. 1, 2, 4 K marks a wave: 78, 76, 82 us. (Whole runs stored, changed or
// not: 82 us.)
template <bool kGrouped>
__global__ __launch_bounds__(256) void k_carve_merge(InterpScan P, int64_t nvox)
{
    __shared__ uint4 s_mark[4][kMarkQuads * 64];
    uint64_t updated = 0;
    const int64_t ngroups = (nvox + kMarkGroup - 1) / kMarkGroup;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64;
    const int64_t waves = (int64_t)gridDim.x * blockDim.x / 64;
    const int lane = (int)(threadIdx.x & 63u);
    uint4 *mine = s_mark[threadIdx.x / 64];
    const uint8_t *bytes = reinterpret_cast<const uint8_t *>(mine);
    const bool rows = P.dims[2] % 64 == 0;
    // the wave's groups, wave + k waves, 64 at a time: a lane looks at one
    for (int64_t g0 = wave; g0 < ngroups; g0 += 64 * waves) {
        const int64_t own = g0 + lane * waves;
        const bool hold = own < ngroups && (!kGrouped || P.touched[own] != 0);
        if (hold && kGrouped) P.touched[own] = 0;
        uint64_t held = __ballot(hold);
        while (held) {
            const int64_t gi = g0 + __builtin_ctzll(held) * waves;
            held &= held - 1;
            // (the marks are padded to whole groups)
            uint4 *m = reinterpret_cast<uint4 *>(P.marks + gi * kMarkGroup);
            uint64_t mask = 0;
#pragma unroll
            for (int k = 0; k < kMarkQuads; ++k) {
                // 16 runs of four lanes each: run r of them in bit 4 r, then in bit r
                const uint4 v = m[64 * k + lane];
                mine[64 * k + lane] = v;
                const bool any = (v.x & v.y & v.z & v.w) != 0xffffffffu;
                if (any) m[64 * k + lane] = make_uint4(0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu);
                uint64_t some = __ballot(any);
                some |= some >> 1;
                some |= some >> 2;
                some &= 0x1111111111111111ull;
                some = (some | some >> 3) & 0x0303030303030303ull;
                some = (some | some >> 6) & 0x000f000f000f000full;
                some = (some | some >> 12) & 0x000000ff000000ffull;
                some = (some | some >> 24) & 0xffffull;
                mask |= some << (16 * k);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            while (mask) {
                uint32_t j[kMergeBatch];
                uint8_t f[kMergeBatch];
#pragma unroll
                for (int b = 0; b < kMergeBatch; ++b) {
                    f[b] = kNoMark;
                    j[b] = 0;
                    if (mask) {
                        const uint32_t run = (uint32_t)__builtin_ctzll(mask);
                        j[b] = (uint32_t)(gi * kMarkGroup) + run * 64u + (uint32_t)lane;
                        mask &= mask - 1;
                        f[b] = bytes[run * 64u + (uint32_t)lane];
                    }
                }
                uint32_t sl[kMergeBatch], key[kMergeBatch];
                int16_t sv[kMergeBatch], wv[kMergeBatch];
                // (where a row is whole runs, a run's row is the wave's: its
                // divisions are scalar)
#pragma unroll
                for (int b = 0; b < kMergeBatch; ++b) {
                    sl[b] = 0;
                    key[b] = (uint32_t)P.rp.tau << P.key_shift;
                    sv[b] = wv[b] = 0;
                    if (f[b] != kNoMark) {
                        if (rows) {
                            const uint32_t j0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(j[b] & ~63u));
                            const uint32_t s0 = slot_of_index(P, j0), z0 = j0 % (uint32_t)P.dims[2];
                            // (the slot of the run's row and its z, wrapped per lane)
                            int32_t z = (int32_t)(z0 + (j[b] & 63u)) + P.ring0[2];
                            z -= z >= P.dims[2] ? P.dims[2] : 0;
                            sl[b] = s0 / (uint32_t)P.dims[2] * (uint32_t)P.dims[2] + (uint32_t)z;
                        } else {
                            sl[b] = slot_of_index(P, j[b]);
                        }
                        if (f[b] != kMarkFree) key[b] = P.keys32[sl[b]];
                        sv[b] = P.sdf[sl[b]];
                        wv[b] = P.w[sl[b]];
                    }
                }
#pragma unroll
                for (int b = 0; b < kMergeBatch; ++b) {
                    if (f[b] == kNoMark) continue;
                    const int32_t gw = wv[b];
                    P.sdf[sl[b]] = (int16_t)rdiv_small(sv[b] * gw + tile_key_sdf(key[b], P.key_shift), gw + 1);
                    P.w[sl[b]] = (int16_t)(gw + 1 < P.w_max ? gw + 1 : P.w_max);
                    if (f[b] != kMarkFree) P.keys32[sl[b]] = 0xffffffffu;
                    ++updated;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    }
    block_add(updated, P, kCtrUpdated);
}

// (in launches of at most 2^31 work-items, like the free walks: a ray takes kFillLanes)
void launch_interp_scan(const InterpScan &P, uint32_t blocks, hipStream_t stream)
{
    const uint32_t per = (uint32_t)1 << 23;
    static_assert(((uint64_t)kKeyRays * kFillLanes << 23) <= (uint64_t)1 << 31, "work-items of a launch");
    for (uint32_t b0 = 0; b0 < blocks; b0 += per) {
        const dim3 grid(blocks - b0 < per ? blocks - b0 : per), block(kKeyRays * kFillLanes);
        if (P.key_shift) hipLaunchKernelGGL((k_interp_scan<uint32_t>), grid, block, 0, stream, P, b0);
        else hipLaunchKernelGGL((k_interp_scan<uint64_t>), grid, block, 0, stream, P, b0);
    }
}

// The band and the free space of a carving scan with 32-bit keys.
template <bool kGrouped>
void launch_carve(const InterpScan &P, hipStream_t stream)
{
    hipLaunchKernelGGL(k_carve_band<kGrouped>, dim3((uint32_t)((P.n + kKeyRays - 1) / kKeyRays)), dim3(kKeyRays * kBandLanes), 0,
                       stream, P);
    const int64_t total = (P.n + 63) / 64 * kCarvePieces * 64 / kInterpBlock + 1, per = (int64_t)1 << 23;
    for (int64_t b0 = 0; b0 < total; b0 += per) {
        const int64_t nb = total - b0 < per ? total - b0 : per;
        hipLaunchKernelGGL(k_carve_free<kGrouped>, dim3((uint32_t)nb), dim3(kInterpBlock), 0, stream, P, b0);
    }
}

}  // namespace

hipError_t launch_interp(const InterpScan &P, int64_t nvox, hipStream_t stream)
{
    const int32_t side = std::max(P.dims[0], std::max(P.dims[1], P.dims[2]));
    const bool grouped = nvox > kGroupedWindow && nvox / 3 > P.n * side;
    if (P.n > 0) {
        const int64_t blocks = (P.n + kInterpBlock - 1) / kInterpBlock;
        if (P.carve && P.key_shift) {
            if (grouped) launch_carve<true>(P, stream);
            else launch_carve<false>(P, stream);
        } else if (P.carve) {
            // chunks of a ray: as many slabs as the window's longest side
            // spans, plus one for a slab boundary inside it
            int32_t dmax = P.dims[0] > P.dims[1] ? P.dims[0] : P.dims[1];
            dmax = dmax > P.dims[2] ? dmax : P.dims[2];
            const int64_t nchunk = ((int64_t)dmax + (1 << kCarveChunkLog2) - 1) / (1 << kCarveChunkLog2) + 1;
            // blocks * nchunk blocks in launches of at most 2^23 blocks
            // (2^31 work-items), so that no grid exceeds a launch's limits
            const int64_t total = blocks * nchunk, per = (int64_t)1 << 23;
            for (int64_t b0 = 0; b0 < total; b0 += per) {
                const int64_t nb = total - b0 < per ? total - b0 : per;
                hipLaunchKernelGGL(k_carve_scan, dim3((uint32_t)nb), dim3(kInterpBlock), 0, stream, P, nchunk, b0);
            }
        } else
            launch_interp_scan(P, (uint32_t)((P.n + kKeyRays - 1) / kKeyRays), stream);
    }
    // four waves per block, one group of 64 runs per wave
    int64_t mblocks = ((nvox + 63) / 64 + 255) / 256;
    if (mblocks > 8192) mblocks = 8192;
    if (P.carve && P.key_shift) {
        mblocks = (nvox + 4 * kMarkGroup - 1) / (4 * kMarkGroup);
        const dim3 grid((uint32_t)(mblocks < 8192 ? mblocks : 8192));
        if (grouped) hipLaunchKernelGGL(k_carve_merge<true>, grid, dim3(256), 0, stream, P, nvox);
        else hipLaunchKernelGGL(k_carve_merge<false>, grid, dim3(256), 0, stream, P, nvox);
        return hipGetLastError();
    }
    const dim3 mg((uint32_t)(mblocks > 0 ? mblocks : 1));
    if (P.key_shift) hipLaunchKernelGGL((k_interp_merge<uint32_t>), mg, dim3(256), 0, stream, P, nvox);
    else hipLaunchKernelGGL((k_interp_merge<uint64_t>), mg, dim3(256), 0, stream, P, nvox);
    return hipGetLastError();
}

}  // namespace tsdf
