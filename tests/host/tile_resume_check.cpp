// Host build of the tile pass's resume as the tile pass calls it (csrc/ray.hpp):
// for random rays and every tiling that a map may have, the binning side walks
// the band on the grid of tiles and takes, at each tile, the voxel walk's
// crossing counts up to the event that entered it; the tile side gets the entry
// record (q, r, 16-bit band offsets, 7-bit counts) and the whole tile, not cut
// to a window, and has no other way to place the walk. So the voxel at these
// counts must lie in the tile, the box walk must visit exactly the plain voxel
// walk's voxels of the tile, in order, with their distance numerators, and no
// key address of a visited voxel may lie outside the tile's slot of the key
// buffer. Rays with ties (on faces, edges and corners of voxels and tiles), flat
// axes, points a few units from the sensor, r around tau, the farthest
// positions and the largest tau. The hardware's reciprocal is 1 / d with a
// relative error up to 2^-21. The test driver defines RAY_HPP.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
static double g_err = 0.0;
#define __device__
#define __forceinline__ inline
#define __fma_rn(a, b, c) std::fma((a), (b), (c))
#define __dmul_rn(a, b) ((a) * (b))
#define __builtin_amdgcn_rcp(x) ((1.0 + g_err) / (x))
#define __builtin_amdgcn_rsq(x) (1.0 / std::sqrt(x))
using std::fabs;
using std::floor;
using std::fmin;
using std::isfinite;
using std::rint;
using std::sqrt;
#include RAY_HPP
using namespace tsdf;

struct Vox {
    int32_t g[3];
    double n;
};

int main(int argc, char **argv)
{
    std::mt19937_64 rng(argc > 1 ? strtoull(argv[1], nullptr, 10) : 1);
    const int iters = argc > 2 ? atoi(argv[2]) : 20000;
    auto pick = [&](int64_t lo, int64_t hi) { return std::uniform_int_distribution<int64_t>(lo, hi)(rng); };
    long bad = 0, rays = 0, tiles = 0, visits = 0;
    int32_t max_count = 0;
    for (int it = 0; it < iters; ++it) {
        g_err = it % 3 == 0 ? 0.0 : std::ldexp((double)pick(-1000, 1000) / 1000.0, -21);
        RayParams P{};
        P.tau = (int32_t)(it % 5 == 0 ? 32767 : it % 5 == 1 ? 5120 : it % 5 == 2 ? pick(1, 64) : pick(1, 32767));
        const int mode = it % 8;
        // lattice of ties: voxel half-units in mode 0, tile corners in mode 1
        const int64_t snap = mode == 0 ? 512 : mode == 1 ? 8192 : 1;
        const int64_t far = mode == 6 ? (1ll << 30) - 1 : 1ll << 22;
        const int64_t lim = mode == 2 ? 4 : mode == 3 ? 2ll * P.tau + 1 : mode == 6 ? (1ll << 30) - 1 : 1ll << pick(0, 24);
        int32_t q[3];
        for (int a = 0; a < 3; ++a) {
            const int64_t o = pick(-far, far) / snap * snap;
            int64_t d = pick(-lim, lim) / snap * snap;
            if (mode == 4 && a == (it / 8) % 3) d = 0;
            if (mode == 5 && a != (it / 8) % 3) d = 0;
            P.o[a] = (int32_t)o;
            q[a] = (int32_t)std::max<int64_t>(-(1ll << 30) + 1, std::min<int64_t>((1ll << 30) - 1, o + d));
        }
        Ray R;
        if (!make_ray(q, P, R)) continue;
        ++rays;
        std::vector<Vox> all;
        Walk W;
        walk_init(R, W);
        do all.push_back({{W.g[0], W.g[1], W.g[2]}, W.n});
        while (walk_next(W) && all.size() < 100000);
        int32_t lt[3];
        do {
            for (int a = 0; a < 3; ++a) lt[a] = (int32_t)pick(a == 2 ? 3 : 2, 6);
        } while (lt[0] + lt[1] + lt[2] < 9 || lt[0] + lt[1] + lt[2] > 12);
        int32_t org[3];
        for (int a = 0; a < 3; ++a) org[a] = (int32_t)(mode == 1 ? 8 * pick(-100, 100) : pick(-1000, 1000));
        if (far > (1ll << 22))
            for (int a = 0; a < 3; ++a) org[a] = (int32_t)std::max<int64_t>(-(1 << 20), std::min<int64_t>((1 << 20) - 1, q[a] >> 10));
        const int32_t lc[3] = {10 + lt[0], 10 + lt[1], 10 + lt[2]};
        const int32_t base[3] = {1024 * org[0], 1024 * org[1], 1024 * org[2]};
        const int32_t key_log2 = it % 2 ? 2 : 3, ext[3] = {1 << lt[0], 1 << lt[1], 1 << lt[2]};
        const int32_t sh[3] = {lt[1] + lt[2] + key_log2, lt[2] + key_log2, key_log2};
        const uint32_t slot = 1u << (lt[0] + lt[1] + lt[2] + key_log2), lds = slot * (uint32_t)pick(0, 3) + 1792u;
        Walk T, Wv;
        walk_init_cells(R, T, lc, base);
        walk_init(R, Wv);
        double t_in = -1.0;
        int typ_in = 0;
        size_t at = 0;  // the plain walk's voxels lie in the tiles one after another
        do {
            ++tiles;
            uint32_t c8 = 0;
            if (t_in >= 0.0)
                for (int a = 0; a < 3; ++a)
                    c8 |= (uint32_t)crossings_upto(Wv.T[a], Wv.dT[a], Wv.step[a] > 0 ? 0 : 1, t_in, typ_in) << (8 * a);
            const uint32_t back = counts_7to8(counts_8to7(c8));
            const int32_t c[3] = {(int32_t)(back & 0xffu), (int32_t)((back >> 8) & 0xffu), (int32_t)((back >> 16) & 0xffu)};
            const int32_t off[3] = {(int16_t)(uint16_t)(R.E[0] - R.q[0]), (int16_t)(uint16_t)(R.E[1] - R.q[1]),
                                    (int16_t)(uint16_t)(R.E[2] - R.q[2])};
            int32_t blo[3];
            bool in = true;
            for (int a = 0; a < 3; ++a) {
                max_count = std::max(max_count, c[a]);
                blo[a] = org[a] + (T.g[a] << lt[a]);
                const int32_t g = (R.S[a] >> 10) + Wv.step[a] * c[a];
                in = in && g >= blo[a] && g < blo[a] + ext[a];
            }
            if (!in) {
                if (bad < 5) printf("ray %d: the resumed voxel lies outside its tile\n", it);
                ++bad;
                continue;
            }
            Ray Rd;
            BoxWalk V;
            tile_walk_resume(R.q, off, (uint32_t)R.r, c, P.o, P.tau, blo, ext, sh, lds, Rd, V);
            bool ok = Rd.r == R.r;
            size_t n = 0;
            do {
                const uint32_t v = (uint32_t)V.lv - lds;
                ok = ok && (uint32_t)V.lv >= lds && v < slot && at + n < all.size();
                if (!ok) break;
                uint32_t want = 0;
                for (int a = 0; a < 3; ++a) {
                    const int32_t rel = all[at + n].g[a] - blo[a];
                    ok = ok && rel >= 0 && rel < ext[a];
                    want += (uint32_t)rel << sh[a];
                }
                ok = ok && v == want && V.n == all[at + n].n;
                ++n;
            } while (box_walk_next(V) && n < 100000);
            at += n;
            visits += (long)n;
            if (!ok) {
                if (bad < 5) printf("ray %d: voxel %zu of tile (%d %d %d) differs\n", it, n, T.g[0], T.g[1], T.g[2]);
                ++bad;
                break;
            }
        } while (walk_next_event(T, t_in, typ_in));
        if (at != all.size()) {
            if (bad < 5) printf("ray %d: %zu of %zu voxels in its tiles\n", it, at, all.size());
            ++bad;
        }
    }
    printf("rays %ld tiles %ld visits %ld largest crossing count %d mismatches %ld\n", rays, tiles, visits, max_count, bad);
    return bad != 0 || visits == 0;
}
