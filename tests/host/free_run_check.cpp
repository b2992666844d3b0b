// Host build of carving's near free walk (FreeRun in csrc/ray.hpp) against the
// general one (FreeWalk): for random near rays and boxes, the indices it visits
// are, in order, those of FreeWalk's voxels from its first up to the first whose
// candidate is not +tau. Rays with ties (on faces, edges, corners), flat axes,
// sensors inside and outside the box, slabs along the longest axis as the
// carving scan cuts them, and extents up to the near walk's limit. The hardware
// reciprocal is replaced by 1 / d with a relative error up to 2^-18. The test
// driver defines RAY_HPP (ray.hpp with its inline-asm minimum replaced).
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
using std::fmax;
using std::fmin;
using std::isfinite;
using std::rint;
using std::sqrt;
#include RAY_HPP
using namespace tsdf;

int main(int argc, char **argv)
{
    std::mt19937_64 rng(argc > 1 ? strtoull(argv[1], nullptr, 10) : 1);
    const int iters = argc > 2 ? atoi(argv[2]) : 20000;
    auto pick = [&](int64_t lo, int64_t hi) { return std::uniform_int_distribution<int64_t>(lo, hi)(rng); };
    long bad = 0, cases = 0, visits = 0, rays = 0;
    for (int it = 0; it < iters; ++it) {
        g_err = it % 4 == 0 ? 0.0 : std::ldexp((double)pick(-1000, 1000) / 1000.0, -18);
        const int mode = it % 7;
        const int64_t span = mode == 0 ? 20000 : mode == 1 ? 400000 : mode == 2 ? 4000000 : mode == 3 ? 3000 : mode == 4 ? 60
                             : mode == 5 ? 60000 : 16000000;
        RayParams P{};
        int32_t q[3];
        for (int a = 0; a < 3; ++a) {
            P.o[a] = (int32_t)pick(-span, span);
            q[a] = (int32_t)pick(-span, span);
            if (mode == 4) {
                P.o[a] *= 512;
                q[a] *= 512;
            }
            if (mode == 5 && a == (it / 7) % 3) q[a] = P.o[a];
            if (mode == 3 && a != (it / 7) % 3 && it % 2) q[a] = P.o[a];  // axis rays
        }
        P.tau = it % 3 == 0 ? 5120 : (int32_t)pick(1, 32767);
        Ray R;
        if (!make_ray(q, P, R) || !(R.r > (double)P.tau) || !free_run_near(R, P)) continue;
        ++rays;
        // a window around a point of the segment, and boxes inside it
        const double t = (double)pick(0, 1000) / 1000.0;
        int32_t w0[3], dims[3];
        for (int a = 0; a < 3; ++a) {
            dims[a] = (int32_t)pick(1, 200);
            const int32_t at = (int32_t)std::floor((P.o[a] + t * (R.S[a] - P.o[a])) / 1024.0);
            w0[a] = at - (int32_t)pick(0, dims[a]);
        }
        const int32_t stride[3] = {dims[1] * dims[2], dims[2], 1};
        for (int b = 0; b < 4; ++b) {
            int32_t lo[3], hi[3];
            for (int a = 0; a < 3; ++a) {
                lo[a] = w0[a];
                hi[a] = w0[a] + dims[a];
                const bool slab = b == 3 ? a == it % 3 : b > 0;
                if (slab) {
                    lo[a] = (int32_t)pick(w0[a], w0[a] + dims[a] - 1);
                    hi[a] = (int32_t)pick(lo[a] + 1, w0[a] + dims[a]);
                }
            }
            std::vector<uint32_t> want, got;
            FreeWalk W;
            if (free_walk_init(R, P, lo, hi, W)) do {
                    if (W.u < kFreeBias) break;
                    uint32_t idx = 0;
                    for (int a = 0; a < 3; ++a) idx += (uint32_t)(W.W.g[a] - w0[a]) * (uint32_t)stride[a];
                    want.push_back(idx);
                } while (free_walk_next(W) && want.size() < 100000);
            FreeRun F;
            if (free_run_init(R, P, lo, hi, w0, stride, F)) do got.push_back(F.idx);
                while (free_run_next(F) && got.size() < 100000);
            ++cases;
            visits += (long)want.size();
            if (want != got) {
                if (bad < 5) printf("mismatch: ray %d mode %d box %d: %zu voxels, want %zu\n", it, mode, b, got.size(), want.size());
                ++bad;
            }
        }
    }
    printf("rays %ld cases %ld visits %ld mismatches %ld\n", rays, cases, visits, bad);
    return bad != 0 || visits == 0;
}
