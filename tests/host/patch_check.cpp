// Host build of the order in which blocks take a scan's points (csrc/patch.hpp):
// whatever the row length, every point belongs to one thread; the samples of a
// scan find its row length, also with missing returns, and none where points
// have no rows; and a block of 256 points meets no more 8-voxel tiles than a run
// of points does, over scans of a room whose rows have many different lengths
// (counted block by block, at 64 mm).
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <vector>
#define __host__
#define __device__
#define __forceinline__ inline
#include PATCH_HPP
using namespace tsdf;

// as the kernels have them (internal.hpp)
static const PatchKind bin = {32, 32768, 3.5f}, keys = {8, 8192, 6.0f};

static long bad = 0;
#define CHECK(c, ...)                       \
    do {                                    \
        if (!(c) && ++bad < 10) {           \
            printf(__VA_ARGS__);            \
            printf("\n");                   \
        }                                   \
    } while (0)

template <int kBlock, uint32_t kRows>
static void once_each(int64_t n, const Row &row)
{
    std::vector<uint8_t> seen((size_t)n, 0);
    const uint32_t blocks = (uint32_t)((n + kBlock - 1) / kBlock);
    long twice = 0, all = 0;
    for (uint32_t b = 0; b < blocks; ++b)
        for (uint32_t t = 0; t < kBlock; ++t) {
            const int64_t i = patch_point<kBlock, kRows>(b, t, row);
            if (i < 0 || i >= n) continue;
            twice += seen[(size_t)i]++ ? 1 : 0;
            ++all;
        }
    CHECK(twice == 0 && all == n, "block %d rows %u: n %lld row %u: %ld points, %ld twice", kBlock, kRows, (long long)n, row.length, all, twice);
}

struct Scan {
    std::vector<float> p;
    int64_t n() const { return (int64_t)p.size() / 3; }
};

// rings x cols points on the walls of a room of 16 x 12 x 3.6 m, a share of them missing
static Scan room(int rings, int cols, double fov, double missing, std::mt19937_64 &rng)
{
    Scan s;
    std::uniform_real_distribution<double> u(0.0, 1.0);
    const double half[3] = {8.0, 6.0, 1.8}, pos[3] = {1.3, -0.7, 0.2};
    for (int r = 0; r < rings; ++r)
        for (int c = 0; c < cols; ++c) {
            const double el = (rings > 1 ? -fov / 2 + fov * r / (rings - 1) : 0.0) * M_PI / 180, az = 2 * M_PI * c / cols;
            const double d[3] = {cos(el) * cos(az), cos(el) * sin(az), sin(el)};
            double t = 1e9;
            for (int a = 0; a < 3; ++a)
                if (d[a] != 0) t = std::min(t, ((d[a] > 0 ? half[a] : -half[a]) - pos[a]) / d[a]);
            const bool lost = u(rng) < missing;
            for (int a = 0; a < 3; ++a) s.p.push_back(lost ? NAN : (float)(d[a] * t));
        }
    return s;
}

// as a wave finds it on the device
static Row find_row(const Scan &s, const PatchKind &kind)
{
    uint64_t rings;
    const Row row = row_rings(s.n(), kind, rings);
    uint32_t last = 0;
    for (int k = 0; k < kRowLengths && ring_at(rings, k); ++k) {
        const Row len = row_of((uint32_t)s.n() / ring_at(rings, k), ring_at(rings, k), kind);
        CHECK(len.length > last, "lengths out of order");
        last = len.length;
        int nc = 0, nf = 0;
        for (uint32_t j = 0; j < kRowSamples; ++j) {
            const int64_t i = row_sample(s.n(), j);
            bool c, f;
            CHECK(i >= 0 && i + len.length < s.n() && i + kRowSpan < s.n(), "sample past the scan");
            row_vote(&s.p[3 * i], &s.p[3 * (i + len.length)], &s.p[3 * (i + kRowSpan)], kind.step, c, f);
            nc += c;
            nf += f;
        }
        if (row_fits(nc, nf)) return len;
    }
    return row;
}
static uint32_t find(const Scan &s, const PatchKind &kind) { return find_row(s, kind).length; }

static double tiles_per_block(const Scan &s, const Row &row)
{
    long tiles = 0;
    const uint32_t blocks = (uint32_t)((s.n() + 255) / 256);
    for (uint32_t b = 0; b < blocks; ++b) {
        std::set<int64_t> met;
        for (uint32_t t = 0; t < 256; ++t) {
            const int64_t i = patch_point<256, 32>(b, t, row);
            if (i >= s.n() || std::isnan(s.p[3 * i])) continue;
            int64_t key = 0;
            for (int a = 0; a < 3; ++a) key = key * 4096 + (int64_t)floor((s.p[3 * i + a] + 50.0) / (8 * 0.064));
            met.insert(key);
        }
        tiles += (long)met.size();
    }
    return (double)tiles / blocks;
}

int main()
{
    std::mt19937_64 rng(3);
    for (int64_t n : {(int64_t)1, (int64_t)255, (int64_t)8192, (int64_t)32768, (int64_t)57616, (int64_t)131072, (int64_t)65344,
                      (int64_t)115200, (int64_t)100003, (int64_t)128 * 2083, (int64_t)40 * 1800, (int64_t)1 << 22})
        for (const bool key : {false, true}) {
            uint64_t rings;
            Row row = row_rings(n, key ? keys : bin, rings);
            for (int k = 0; k <= kRowLengths; ++k) {
                if (k > 0) {
                    const uint32_t r = ring_at(rings, k - 1);
                    if (r == 0) break;
                    row = row_of((uint32_t)n / r, r, key ? keys : bin);
                }
                if (key) {
                    once_each<64, 8>(n, row);
                } else {
                    once_each<128, 32>(n, row);
                    once_each<256, 32>(n, row);
                    once_each<512, 32>(n, row);
                }
            }
        }
    // the band of a column by the row's inverse, over the longest sequences
    for (int k = 0; k < 2000000; ++k) {
        const uint32_t length = std::uniform_int_distribution<uint32_t>(256, 1u << 28)(rng), kRun = 8;
        const uint32_t end = std::uniform_int_distribution<uint32_t>(1, 0x7ffffffu / (length < 0x7ffffffu ? length : 0x7ffffffu))(rng) * length;
        const Row row{length, end, row_of(length, 32, bin).inverse};
        if (end <= kRun) continue;
        const uint32_t col = std::uniform_int_distribution<uint32_t>(0, end - 1)(rng) / kRun * kRun;
        CHECK((patch_point<256, 32>(col / kRun, 0, row) == (int64_t)(col / length * 32) * length + col % length), "column %u of rows of %u", col,
              length);
    }
    struct {
        int rings, cols;
        double fov;
    } scans[] = {{128, 1024, 45}, {128, 512, 45}, {128, 2048, 45}, {64, 1024, 33}, {64, 2048, 33}, {32, 1024, 40}, {32, 2083, 40},
                 {64, 1021, 45},  {104, 554, 45}, {128, 720, 45},  {128, 900, 90}, {64, 1800, 45}, {64, 2083, 45}, {80, 1440, 40},
                 {40, 1800, 25},  {57, 743, 45}, {93, 512, 45}, {128, 700, 45}, {128, 870, 45},  {128, 800, 45}, {96, 1000, 45}, {128, 333, 45}, {64, 512, 45}};
    for (auto &c : scans)
        for (double missing : {0.0, 0.3}) {
            const Scan s = room(c.rings, c.cols, c.fov, missing, rng);
            const Row found = find_row(s, bin);
            const uint32_t row = found.length;
            const double run = tiles_per_block(s, Row{0, 0, 0}), patch = tiles_per_block(s, found);
            if (missing == 0.0) printf("%d x %d: row %u, tiles per block %.1f -> %.1f\n", c.rings, c.cols, row, run, patch);
            // (a power of two is not tried: 32 rings at 40 degrees are 4 steps apart)
            const bool tried = (s.n() & (s.n() - 1)) != 0;
            CHECK(tried ? row == 0 || row % c.cols == 0 : row == 1024, "%d x %d: row %u", c.rings, c.cols, row);
            CHECK(patch <= (tried ? 1.0 : 1.05) * run, "%d x %d: tiles %.1f -> %.1f", c.rings, c.cols, run, patch);
        }
    for (auto &c : {scans[0], scans[7], scans[8], scans[10], scans[16]}) CHECK(find(room(c.rings, c.cols, c.fov, 0.1, rng), bin) == (uint32_t)c.cols, "%d x %d", c.rings, c.cols);
    // no rows: shuffled points, one ring of many points, too few points, no returns
    Scan s = room(128, 1000, 45, 0.0, rng);
    for (int64_t i = s.n() - 1; i > 0; --i) {
        const int64_t j = std::uniform_int_distribution<int64_t>(0, i)(rng);
        for (int a = 0; a < 3; ++a) std::swap(s.p[3 * i + a], s.p[3 * j + a]);
    }
    CHECK(find(s, bin) == 0, "rows among shuffled points");
    CHECK(find(room(1, 128000, 0, 0.0, rng), bin) == 0, "rows of one ring");
    CHECK(find(room(2, 64000, 2, 0.0, rng), bin) == 0, "rows of two rings");
    CHECK(find(room(16, 1000, 30, 0.0, rng), bin) == 0, "rows of a small scan");
    CHECK(find(room(128, 1000, 45, 1.0, rng), bin) == 0, "rows without returns");
    CHECK(find(room(16, 1000, 30, 0.0, rng), keys) == 1000, "16 rings in patches of 8 rows");
    CHECK(find(room(17, 584, 30, 0.0, rng), keys) == 584, "17 rings in patches of 8 rows");
    CHECK(find(room(93, 512, 45, 0.0, rng), bin) == 512, "93 rings");
    CHECK(find(room(64, 1800, 45, 0.0, rng), keys) == 1800, "64 rings in patches of 8 rows");
    printf("mismatches %ld\n", bad);
    return bad != 0;
}
