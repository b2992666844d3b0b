// The order in which blocks take the points of a scan. A block takes a patch,
// kRows rows of an organised scan (point = row * columns + column) with
// neighbouring columns of each, instead of one run of points: rows that follow
// each other are neighbouring rings of the sensor, whose points share tiles and
// voxels, so that a binning block meets fewer tiles, sends fewer atomics and
// writes longer stretches of a run, and a block of the key-volume scans merges
// more candidates. Count and fill of 50 street scans of 128 x 1024 points, runs /
// patches: 136 + 157 / 104 + 131 us.
//
// The calls do not say how long a row is, and patches cut at a wrong length
// scatter a block's points. So the host lists the row lengths that a scan of n
// points may have (row_rings), and the device tries them on a few samples
// (row_vote); where none fits, blocks take runs. Count and fill of 32 street scans
// of 128 x 900 points: 54 + 61 us in runs, 76 + 78 cut at 1024, 51 + 54 at 900.
//
// A power of two needs no samples: its rows are powers of two long, and patches
// cut at 1024 then hold the rings of one direction (two rows of 512, one of
// 1024) or of two opposite ones (half rows of 2048). 32 scans of 128 x 512 points
// in a room, cut at 512 / 1024: 48 + 55 / 48 + 55 us; of 128 x 2048, cut at 2048 /
// 1024: 184 + 196 / 131 + 188 us in the room (fewer lanes of a wave count in the
// same place of the block's table), 115 + 112 / 115 + 124 in the street.
#pragma once

#include <stdint.h>

namespace tsdf {

constexpr int kRowLengths = 8, kRowSamples = 8;  // of a scan: a wave tries all at once
static_assert(kRowLengths * kRowSamples == 64, "a lane per length and sample");
constexpr uint32_t kRowSpan = 32;  // points of a row that a step from row to row is compared with (row_vote)

// What patches a kernel takes: their rows (a power of two), the fewest points of a
// scan in patches (that many rows of 1024), and the longest step from row to row that pays, in steps along a row.
struct PatchKind {
    uint32_t rows;
    int64_t points;
    float step;
};

// A row's length, and what patch_point needs of it.
struct Row {
    uint32_t length;  // points, 0: the scan is taken in runs
    uint32_t end;     // columns of all whole bands, one after another
    uint32_t inverse; // 2^32 / length, rounded up
};

__host__ __device__ __forceinline__ Row row_of(uint32_t length, uint32_t rings, const PatchKind &kind)
{
    return Row{length, rings / kind.rows * length, 0xffffffffu / length + 1u};
}

// The row to take the points of a scan of n points by, where there are no lengths
// to try; else these, as numbers of rings (length n / rings, of at least 256
// points), a byte each from the low end, the most first (0: no more): the usual
// numbers, then any from 128 down to 16. (Eight Rows in the kernels' arguments,
// 96 bytes, cost every call 0.4 us: 17.5 -> 18.0 for a scan of 16 x 1024 points.)
inline Row row_rings(int64_t n, const PatchKind &kind, uint64_t &rings)
{
    rings = 0;
    if (n < kind.points || n >= (int64_t)1 << 32) return Row{0, 0, 0};
    if ((n & (n - 1)) == 0) return row_of(1024, (uint32_t)(n / 1024), kind);
    const uint32_t points = (uint32_t)n, most = points / 256 < 128 ? points / 256 : 128;
    uint32_t found[kRowLengths];
    int k = 0;
    const auto add = [&](uint32_t r) {
        if (k == kRowLengths || r < kind.rows || r > most || points % r != 0) return;
        int at = 0;
        while (at < k && found[at] > r) ++at;
        if (at < k && found[at] == r) return;
        for (int j = k++; j > at; --j) found[j] = found[j - 1];
        found[at] = r;
    };
    for (uint32_t r : {128u, 64u, 32u, 16u, 40u, 80u}) add(r);
    for (uint32_t r = most; r >= 16 && k < kRowLengths; --r) add(r);
    for (int j = 0; j < k; ++j) rings |= (uint64_t)found[j] << 8 * j;
    return Row{0, 0, 0};
}
__host__ __device__ __forceinline__ uint32_t ring_at(uint64_t rings, uint32_t k) { return (uint32_t)(rings >> 8 * k) & 255u; }

// Sample j's first point: points at + length and at + kRowSpan exist for every
// length (at most n / 16).
__host__ __device__ __forceinline__ int64_t row_sample(int64_t n, uint32_t j)
{
    return (n - n / 16 - kRowSpan - 1) * (2 * j + 1) / (2 * kRowSamples);
}

// What a sample says of a length: a, b and c are the points at, at + length and
// at + kRowSpan. It counts if all three are returns, and speaks for the length
// if the angle from a to b is at most `step` steps along the row, kRowSpan of
// which are the angle from a to c.
__host__ __device__ __forceinline__ void row_vote(const float a[3], const float b[3], const float c[3], float step, bool &counts,
                                                  bool &fits)
{
    float ab = 0.f, ac = 0.f, len[3] = {0.f, 0.f, 0.f};
    for (int k = 0; k < 3; ++k) {
        ab += a[k] * b[k];
        ac += a[k] * c[k];
        len[0] += a[k] * a[k];
        len[1] += b[k] * b[k];
        len[2] += c[k] * c[k];
    }
    counts = true;
    for (int k = 0; k < 3; ++k) counts = counts && len[k] > 0.f && len[k] < 1e12f;  // (a NaN is neither)
    float xb = 0.f, xc = 0.f;
    for (int k = 0; k < 3; ++k) {
        const int i = (k + 1) % 3, j = (k + 2) % 3;
        const float vb = a[i] * b[j] - a[j] * b[i], vc = a[i] * c[j] - a[j] * c[i];
        xb += vb * vb;
        xc += vc * vc;
    }
    // (tangents for angles: a row of 256 points and more has its 32nd within 45 degrees)
    const float most = step / kRowSpan;
    fits = counts && ab > 0.f && ac > 0.f && xb * (ac * ac) <= most * most * (xc * (ab * ab));
}

// Whether a length is the scan's, by the samples that count and fit.
__host__ __device__ __forceinline__ bool row_fits(int counts, int fits) { return counts >= 3 && 4 * fits >= 3 * counts; }

// The point of thread t of a scan's block b (runs where row.length is 0). Block
// by block, kRun columns of a band of kRows rows, the bands' columns in one
// sequence (a block that ends a band begins the next); the points after the last
// whole band in order. Every point is some thread's, once. (The band by its
// inverse: two divisions a thread were 5 % of the fill, 129 -> 135 us on 50
// scans of 128 x 1024 points.)
template <int kBlock, uint32_t kRows>
__host__ __device__ __forceinline__ int64_t patch_point(uint32_t b, uint32_t t, const Row &row)
{
    constexpr uint32_t kRun = kBlock / kRows;
    static_assert(kRun * kRows == kBlock && kRun <= 256, "whole columns; at most a row's");
    const uint32_t col0 = b * kRun;
    if (col0 >= row.end) return (int64_t)b * kBlock + t;
    uint32_t band = (uint32_t)((uint64_t)col0 * row.inverse >> 32);  // the quotient, or one more
    band -= band * row.length > col0 ? 1u : 0u;
    const uint32_t slot = col0 + t % kRun;
    if (slot >= row.end) return (int64_t)slot * kRows + t / kRun;
    uint32_t col = slot - band * row.length;
    if (col >= row.length) {
        col -= row.length;
        ++band;
    }
    return (int64_t)(band * kRows + t / kRun) * row.length + col;
}

}  // namespace tsdf
