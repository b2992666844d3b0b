// Point-to-TSDF registration (the paper's stated next step; HATSDF, which
// FeatSense's mapping comes from, localises directly in the TSDF): damped
// Gauss-Newton on sum phi(R p + t)^2, phi the map's signed distance in
// metres, trilinear between the 8 voxel centres around the point (all
// resident, observed, not truncated, else the point is left out), with the
// left update R' = exp([theta]x) R, t' = exp([theta]x) t + rho and the
// Jacobian row J = (grad phi, w x grad phi).
//
// One launch per evaluation of the normal equations, and no wait for the host
// between them: the launch's last block adds the blocks' rows of 29 sums (H
// upper triangle, J^T r, sum r^2, points used), solves the 6 x 6 system and
// leaves the next pose in device memory for the next launch. An evaluation is
// bound by latency: 131,072 points are two waves per SIMD, and of 14.8 us per
// launch the points and their corners take 5 (uncoalesced 4-byte loads), the
// wave sums 3, the rows of the blocks through memory 4. A 10-step run takes
// 185 us; with the block rows copied to the host, a solve there and a wait per
// step it took 570 us, 22 us of each step in the kernel.
//
// The sums do not depend on scheduling: a wave's points, the waves of a block,
// and the blocks (in 16 interleaved chains, then the chains in order) are all
// added in an order fixed by n.
#include "internal.hpp"

namespace tsdf {

namespace {

constexpr int kRegBlock = 512;

// phi (metres), its gradient (per metre) and the world point of point p;
// false when the point is left out. The 16 corner loads leave together.
__device__ __forceinline__ bool reg_point(const RegArgs &A, const double M[12], float px, float py, float pz,
                                          double &phi, double grad[3], double w[3])
{
    if (!isfinite(px) || !isfinite(py) || !isfinite(pz)) return false;
    const double x = px, y = py, z = pz;
    int32_t s0[3], s1[3];  // slots of the lower and the upper corner
    double f[3];
    bool inside = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        w[a] = __fma_rn(M[4 * a + 0], x, __fma_rn(M[4 * a + 1], y, __fma_rn(M[4 * a + 2], z, M[4 * a + 3])));
        const double u = w[a] / A.vs - 0.5;  // voxel g's centre is at u = g
        const bool near = fabs(u) < 1073741824.0;
        const double fl = floor(u);
        f[a] = u - fl;
        // |g| < 2^30 + 1 and |origin| <= 2^20: no overflow
        const int32_t rel = (near ? (int32_t)fl : 0) - A.origin[a];
        inside = inside && near && rel >= 0 && rel + 1 < A.dims[a];
        const int32_t v0 = rel + A.ring0[a], v1 = v0 + 1;
        s0[a] = v0 - (v0 >= A.dims[a] ? A.dims[a] : 0);
        s1[a] = v1 - (v1 >= A.dims[a] ? A.dims[a] : 0);
    }
    if (!inside) return false;
    // the two corners of a z pair lie side by side (one 4-byte load of each
    // array) unless the window's ring buffer wraps between them
    int32_t sq[8], wq[8];
    const char *ps = (const char *)A.sdf, *pw = (const char *)A.w;
    const bool side = s1[2] == s0[2] + 1;
    uint32_t ds[4], dw[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int32_t vx = k & 1 ? s1[0] : s0[0], vy = k & 2 ? s1[1] : s0[1];
        const uint32_t at = 2u * (uint32_t)((vx * A.dims[1] + vy) * A.dims[2]);  // slots stay below 2^31
        if (side) {
            __builtin_memcpy(&ds[k], ps + (at + 2u * (uint32_t)s0[2]), 4);
            __builtin_memcpy(&dw[k], pw + (at + 2u * (uint32_t)s0[2]), 4);
        } else {
            uint16_t l, h;
            __builtin_memcpy(&l, ps + (at + 2u * (uint32_t)s0[2]), 2);
            __builtin_memcpy(&h, ps + (at + 2u * (uint32_t)s1[2]), 2);
            ds[k] = l | (uint32_t)h << 16;
            __builtin_memcpy(&l, pw + (at + 2u * (uint32_t)s0[2]), 2);
            __builtin_memcpy(&h, pw + (at + 2u * (uint32_t)s1[2]), 2);
            dw[k] = l | (uint32_t)h << 16;
        }
    }
    double c[8];
    bool used = true;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        sq[k] = k & 4 ? (int32_t)ds[k & 3] >> 16 : (int16_t)(ds[k & 3] & 0xffffu);
        wq[k] = k & 4 ? (int32_t)dw[k & 3] >> 16 : (int16_t)(dw[k & 3] & 0xffffu);
        used = used && wq[k] > 0 && sq[k] > -A.tau && sq[k] < A.tau;
        c[k] = (double)sq[k] * A.vs / 1024.0;
    }
    if (!used) return false;
    // trilinear value and its derivatives along x, y, z (per voxel)
    const double c00 = c[0] + f[0] * (c[1] - c[0]), c10 = c[2] + f[0] * (c[3] - c[2]);
    const double c01 = c[4] + f[0] * (c[5] - c[4]), c11 = c[6] + f[0] * (c[7] - c[6]);
    const double c0 = c00 + f[1] * (c10 - c00), c1 = c01 + f[1] * (c11 - c01);
    phi = c0 + f[2] * (c1 - c0);
    const double dx0 = (c[1] - c[0]) + f[1] * ((c[3] - c[2]) - (c[1] - c[0]));
    const double dx1 = (c[5] - c[4]) + f[1] * ((c[7] - c[6]) - (c[5] - c[4]));
    grad[0] = (dx0 + f[2] * (dx1 - dx0)) / A.vs;
    grad[1] = ((c10 - c00) + f[2] * ((c11 - c01) - (c10 - c00))) / A.vs;
    grad[2] = (c1 - c0) / A.vs;
    return true;
}

typedef double double4 __attribute__((ext_vector_type(4)));

// The sums of a wave's 64 points are X^T X for the 64 x 8 matrix X of
// (J, phi, 1) rows: eight v_mfma_f64_16x16x4f64, each fed by one LDS read
// (A and B of X^T X are the same register), rows 0..7 of the 16 holding
// points p..p+3 and rows 8..15 points p+4..p+7, so that the two 8 x 8
// diagonal blocks of the result hold the sums (products on the vector unit and
// a halving exchange of doubles: 23.1 us per launch, this 17.7).
constexpr int kFeat = 8;

// (H + lambda I) d = -g by Cholesky; then the pose exp([theta]x) applied on
// the left with translation rho (d = (rho, theta)). false when H + lambda I
// is not positive definite.
__device__ bool reg_update(const double *sums, double lambda, const double M[12], double out[12], double d[6])
{
    double H[6][6], L[6][6], inv[6], y[6];
    int k = 0;
#pragma unroll
    for (int a = 0; a < 6; ++a)
#pragma unroll
        for (int b = a; b < 6; ++b) H[b][a] = sums[k++];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
#pragma unroll
        for (int j = 0; j < i; ++j) {
            double s = H[i][j];
#pragma unroll
            for (int q = 0; q < j; ++q) s -= L[i][q] * L[j][q];
            L[i][j] = s * inv[j];
        }
        double s = H[i][i] + lambda;
#pragma unroll
        for (int q = 0; q < i; ++q) s -= L[i][q] * L[i][q];
        if (!(s > 0.0)) return false;
        L[i][i] = sqrt(s);
        inv[i] = 1.0 / L[i][i];  // the chain is serial: one division per row, products elsewhere
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        double s = -sums[21 + i];
#pragma unroll
        for (int q = 0; q < i; ++q) s -= L[i][q] * y[q];
        y[i] = s * inv[i];
    }
#pragma unroll
    for (int i = 5; i >= 0; --i) {
        double s = y[i];
#pragma unroll
        for (int q = i + 1; q < 6; ++q) s -= L[q][i] * d[q];
        d[i] = s * inv[i];
    }
    const double ax = d[3], ay = d[4], az = d[5];
    const double ang = sqrt(ax * ax + ay * ay + az * az);
    const double a = ang > 1e-12 ? sin(ang) / ang : 1.0;
    const double b = ang > 1e-12 ? (1.0 - cos(ang)) / (ang * ang) : 0.5;
    // exp(K) = I + a K + b K^2, K = [theta]x
    const double K[3][3] = {{0.0, -az, ay}, {az, 0.0, -ax}, {-ay, ax, 0.0}};
    double R[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            double k2 = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) k2 += K[i][q] * K[q][j];
            R[i][j] = (i == j ? 1.0 : 0.0) + a * K[i][j] + b * k2;
        }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double s = j == 3 ? d[i] : 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) s += R[i][q] * M[4 * q + j];
            out[4 * i + j] = s;
        }
    }
    return true;
}

// Orders a wave's LDS accesses with each other (no other wave uses them).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Waits until this wave's stores are done. A relaxed agent-scope store goes
// through the L2 to where every XCD sees it, so once it is done the row it
// belongs to may be counted in; a release fence would write the whole L2's
// dirty lines back as well, three times per block.
__device__ __forceinline__ void arrived()
{
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// One evaluation. A.first: the pose is A.M, else what the previous launch
// left in A.work. A.last: no step follows (the sums at this pose are the
// answer). A launch after the run has stopped does nothing.
__global__ __launch_bounds__(kRegBlock) void k_reg_step(RegArgs A)
{
    __shared__ double s_x[kRegBlock / 64][64 * kFeat];
    __shared__ double s_w[2 * kRegBlock / 64][kFeat * kFeat];
    __shared__ double s_chain[kRegBlock / kRegRow][kRegRow];
    __shared__ uint32_t s_last;
    RegWork &S = *A.work;
    if (!A.first && S.stop) return;
    double M[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) M[k] = A.first ? A.M[k] : S.M[k];
    const int lane = (int)(threadIdx.x & 63u), wave = (int)(threadIdx.x / 64u);
    // sum k = threadIdx.x is entry (a, b) of X^T X (worked out here, beside
    // the loads)
    int entry = 0;
    if (threadIdx.x < kRegSums) {
        const int k = (int)threadIdx.x;
        int a = 0, b = k;
        while (a < 5 && b >= 6 - a) b -= 6 - a++;
        b += a;
        if (k >= 21) a = k < 27 ? k - 21 : (k == 27 ? 6 : 7), b = k < 28 ? 6 : 7;
        entry = a * kFeat + b;
    }
    double4 acc = {0.0, 0.0, 0.0, 0.0};
    double *x = s_x[wave];
    // every wave takes the same number of rounds: the matrix instruction
    // wants all lanes
    const int64_t stride = (int64_t)gridDim.x * kRegBlock;
    // Workgroup b runs on XCD b % 8: it takes four runs of 128 points, 1024
    // apart, so that an XCD keeps to one sector of an organised scan's columns
    // in every ring, and the map lines that a column's points share are
    // fetched by one L2 instead of eight (17.7 -> 15.2 us per launch on 131,072
    // points).
    const int64_t group = (int64_t)(blockIdx.x / 8u) * (8 * kRegBlock) + (blockIdx.x % 8u) * (kRegBlock / 4) +
                          (threadIdx.x / (kRegBlock / 4)) * (2 * kRegBlock) + threadIdx.x % (kRegBlock / 4);
    for (int64_t i0 = 0; i0 < A.n; i0 += stride) {
        const int64_t i = i0 + group;
        double phi = 0.0, one = 0.0, g[3] = {0.0, 0.0, 0.0}, w[3] = {0.0, 0.0, 0.0};
        if (i < A.n && reg_point(A, M, A.xyz[3 * i], A.xyz[3 * i + 1], A.xyz[3 * i + 2], phi, g, w)) {
            one = 1.0;
        } else {
            phi = 0.0;
#pragma unroll
            for (int a = 0; a < 3; ++a) g[a] = w[a] = 0.0;
        }
        const double f[kFeat] = {g[0], g[1], g[2], w[1] * g[2] - w[2] * g[1], w[2] * g[0] - w[0] * g[2],
                                 w[0] * g[1] - w[1] * g[0], phi, one};
#pragma unroll
        for (int k = 0; k < kFeat; ++k) x[lane * kFeat + k] = f[k];
        wave_sync();
        // lane l of step m: row l % 16 (feature % 8 of point half * 4 + l / 16)
#pragma unroll
        for (int m = 0; m < 64 / 8; ++m) {
            const double a = x[(8 * m + ((lane >> 3) & 1) * 4 + (lane >> 4)) * kFeat + (lane & 7)];
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, a, acc, 0, 0, 0);
        }
        wave_sync();
    }
    // result register v of lane l: row l / 16 + 4 v, column l % 16
    {
        const bool low = (lane & 8) == 0;
        double *d = s_w[2 * wave + (low ? 0 : 1)];
        d[(lane >> 4) * kFeat + (lane & 7)] = low ? acc[0] : acc[2];
        d[((lane >> 4) + 4) * kFeat + (lane & 7)] = low ? acc[1] : acc[3];
    }
    __syncthreads();
    double *row = S.rows + (size_t)blockIdx.x * kRegRow;
    if (threadIdx.x < kRegRow) {
        double s = 0.0;
        if (threadIdx.x < kRegSums) {
#pragma unroll
            for (int q = 0; q < 2 * kRegBlock / 64; ++q) s += s_w[q][entry];
        }
        __hip_atomic_store(&row[threadIdx.x], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        arrived();
    }
    __syncthreads();
    // the last block to arrive: counters of kRegFan blocks each, then one
    // over those (additions on one address queue at the memory side)
    if (threadIdx.x == 0) {
        const uint32_t q = blockIdx.x / kRegFan, groups = (gridDim.x + kRegFan - 1) / kRegFan;
        const uint32_t members = q + 1 < groups ? kRegFan : gridDim.x - q * kRegFan;
        uint32_t last = 0;
        if (__hip_atomic_fetch_add(&S.ticket[32 * q], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == members - 1)
            last = __hip_atomic_fetch_add(&S.root, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == groups - 1;
        s_last = last;
    }
    __syncthreads();
    if (!s_last) return;
    {
        // chain c adds rows c, c + 16, ...; then the chains in order
        constexpr uint32_t kChains = kRegBlock / kRegRow;
        const uint32_t k = threadIdx.x % kRegRow, c = threadIdx.x / kRegRow;
        double r[kRegMaxBlocks / kChains], s = 0.0;
        // (rows past the last are read as the last, and not added)
#pragma unroll
        for (uint32_t j = 0; j < kRegMaxBlocks / kChains; ++j)
            r[j] = __hip_atomic_load(&S.rows[(size_t)min(c + j * kChains, gridDim.x - 1u) * kRegRow + k],
                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (uint32_t j = 0; j < kRegMaxBlocks / kChains; ++j) s += c + j * kChains < gridDim.x ? r[j] : 0.0;
        s_chain[c][k] = s;
        __syncthreads();
        if (threadIdx.x < kRegRow) {
            double t = 0.0;
            for (uint32_t q = 0; q < kChains; ++q) t += s_chain[q][threadIdx.x];
            s_chain[0][threadIdx.x] = t;
        }
        // ready for the next launch
        if (threadIdx.x < kRegMaxBlocks / kRegFan) S.ticket[32 * threadIdx.x] = 0;
        if (threadIdx.x == 0) S.root = 0;
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    const double *sums = s_chain[0];
    int32_t it = A.first ? 0 : S.it;
    double step = A.first ? 0.0 : S.step, next[12], d[6];
    const bool go = !A.last && sums[28] >= 6.0 && reg_update(sums, A.damping, M, next, d);
    if (go) {
#pragma unroll
        for (int k = 0; k < 12; ++k) S.M[k] = next[k];
        S.step = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + d[3] * d[3] + d[4] * d[4] + d[5] * d[5]);
        S.it = it + 1;
        S.stop = 0;
        return;
    }
    S.stop = 1;
    RegResult &O = *A.result;
#pragma unroll
    for (int k = 0; k < 12; ++k) O.M[k] = M[k];
    for (int k = 0; k < kRegSums; ++k) O.sums[k] = sums[k];
    O.step = step;
    O.it = it;
    O.done = 1;
}

}  // namespace

hipError_t launch_reg_step(const RegArgs &A, hipStream_t stream)
{
    int64_t blocks = (A.n + 8 * kRegBlock - 1) / (8 * kRegBlock) * 8;  // whole groups of eight (one per XCD)
    blocks = blocks < 8 ? 8 : (blocks > kRegMaxBlocks ? kRegMaxBlocks : blocks);
    hipLaunchKernelGGL(k_reg_step, dim3((uint32_t)blocks), dim3(kRegBlock), 0, stream, A);
    return hipGetLastError();
}

}  // namespace tsdf
