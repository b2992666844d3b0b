// Surface extraction for inspection: the zero level set of the resident
// window in a box, by marching tetrahedra (each cube of 8 observed voxel
// centres cut into the 6 tetrahedra around its 0-7 diagonal; one or two
// triangles per tetrahedron with a sign change; edge points at
// t = s_a / (s_a - s_b) in float64). Two passes give a deterministic order,
// cube by cube (x, then y, then z): a count per row of cubes, and, after an
// exclusive scan over units of 16 rows on the host, an emit pass.
//
// Almost all cubes hold no surface (1 in 45 of a window around a room), so
// both passes look at 63 cubes of a row at once: a wave reads 64 voxels of the
// four voxel rows around them, ballots "observed" and "negative", and works
// out on eight 64-bit masks which cubes are complete and change sign; where no
// cube is complete, the distances are not read at all. Only then do lanes look
// up what their cube holds in a table over its eight signs. The emit pass
// spreads a wave's triangles over its lanes, one triangle per lane, however
// many each cube gives. A 512 x 512 x 256 window with 5.8 M triangles: count
// 770 -> 160 us (bound by instruction issue, 1.3 M spans), emit 2.7 -> 1.5 ms,
// beside the copies to the host, which take 3.5 ms (60 GB/s) and bound the
// call (24.1 -> 6.0 ms with those copies and their page faults shared by
// several host threads).
#include <algorithm>

#include "internal.hpp"

namespace tsdf {

namespace {

constexpr int kMeshBlock = 256;
constexpr int kMeshWaves = kMeshBlock / 64;
// The emit pass has a wave per row: where a wall lies along y, its few rows
// hold thousands of triangles each.
constexpr int kEmitWaves = (int)kMeshUnit, kEmitBlock = 64 * kEmitWaves;
constexpr int kMostTris = 12;  // six tetrahedra, two triangles each
// Units per launch: 2^31 work-items, half of what a grid may hold (a thin, wide
// window has up to 2^30 rows of cubes).
constexpr uint32_t kCountUnits = 0x80000000u / kMeshBlock, kEmitUnits = 0x80000000u / kEmitBlock;

// What a cube holds, by its signs (bit k: corner k = (k & 1, k >> 1 & 1,
// k >> 2 & 1) is negative): the number of triangles, and for each, 6 bits per
// vertex, the edge (from | to << 3) it lies on.
struct MeshTable {
    uint8_t count[256];
    uint32_t tri[256][kMostTris];
};

constexpr MeshTable make_table()
{
    constexpr int tet[6][4] = {{0, 1, 3, 7}, {0, 3, 2, 7}, {0, 2, 6, 7}, {0, 6, 4, 7}, {0, 4, 5, 7}, {0, 5, 1, 7}};
    MeshTable T{};
    for (int signs = 0; signs < 256; ++signs) {
        int n = 0;
        for (int t = 0; t < 6; ++t) {
            int v[4] = {}, in[4] = {}, nin = 0;
            for (int k = 0; k < 4; ++k) {
                v[k] = tet[t][k];
                in[k] = (signs >> v[k]) & 1;
                nin += in[k];
            }
            if (nin == 0 || nin == 4) continue;
            if (nin == 1 || nin == 3) {
                // the lone vertex: inside when one is inside, outside when three are
                int lone = 0;
                for (int k = 0; k < 4; ++k)
                    if (in[k] == (nin == 1 ? 1 : 0)) lone = k;
                uint32_t e = 0;
                int at = 0;
                for (int k = 0; k < 4; ++k)
                    if (k != lone) e |= (uint32_t)(v[lone] | v[k] << 3) << (6 * at++);
                T.tri[signs][n++] = e;
            } else {
                int i[2] = {}, o[2] = {}, ni = 0, no = 0;
                for (int k = 0; k < 4; ++k) {
                    if (in[k]) i[ni++] = v[k];
                    else o[no++] = v[k];
                }
                // the quad i0o0, i0o1, i1o1, i1o0 as triangles (0 1 2), (0 2 3)
                const uint32_t q[4] = {(uint32_t)(i[0] | o[0] << 3), (uint32_t)(i[0] | o[1] << 3),
                                       (uint32_t)(i[1] | o[1] << 3), (uint32_t)(i[1] | o[0] << 3)};
                T.tri[signs][n++] = q[0] | q[1] << 6 | q[2] << 12;
                T.tri[signs][n++] = q[0] | q[2] << 6 | q[3] << 12;
            }
        }
        T.count[signs] = (uint8_t)n;
    }
    return T;
}

__constant__ MeshTable kTable = make_table();

// 63 cubes (64 voxels) of a row from voxel z0 on. q = (x | y << 1) numbers
// the four voxel rows.
struct MeshSpan {
    uint64_t act;    // complete cubes whose signs differ
    int32_t s[4];    // this lane's voxel of each row (where act != 0)
    uint32_t signs;  // this lane's cube (where its bit of act is set)
};

// Slots of the four voxel rows around cube row r of the box (32 bits: a
// window has fewer than 2^31 voxels).
__device__ __forceinline__ void mesh_rows(const MeshArgs &A, uint32_t r, int32_t row[4])
{
    const int32_t x = (int32_t)(r / (uint32_t)A.n[1]), y = (int32_t)(r % (uint32_t)A.n[1]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        int32_t sx = A.s0[0] + x + (q & 1), sy = A.s0[1] + y + (q >> 1);
        sx -= sx >= A.dims[0] ? A.dims[0] : 0;
        sy -= sy >= A.dims[1] ? A.dims[1] : 0;
        row[q] = (sx * A.dims[1] + sy) * A.dims[2];
    }
}

__device__ __forceinline__ MeshSpan mesh_span(const MeshArgs &A, const int32_t row[4], int32_t z0, int lane)
{
    MeshSpan P;
    P.act = 0;
    P.signs = 0;
    const int32_t z = z0 + lane;
    const bool valid = z <= A.n[2];  // n cubes are n + 1 voxels
    int32_t sz = A.s0[2] + z;
    sz -= sz >= A.dims[2] ? A.dims[2] : 0;
    sz = valid ? sz : 0;
    int32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = A.w[row[q] + sz];
    uint64_t seen = __ballot(valid);
#pragma unroll
    for (int q = 0; q < 4; ++q) seen &= __ballot(w[q] > 0);
    const uint64_t cubes = seen & (seen >> 1);  // (the last voxel of a span starts no cube)
    if (!cubes) return P;
#pragma unroll
    for (int q = 0; q < 4; ++q) P.s[q] = A.sdf[row[q] + sz];
    uint64_t any = 0, all = ~0ull;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint64_t neg = __ballot(P.s[q] < 0);
        any |= neg;
        all &= neg;
    }
    any |= any >> 1;
    all &= all >> 1;
    P.act = cubes & any & ~all;
    if (!P.act) return P;
    uint32_t own = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) own |= (P.s[q] < 0 ? 1u : 0u) << q;
    P.signs = own | (uint32_t)__shfl_down((int)own, 1) << 4;
    return P;
}

__global__ __launch_bounds__(kMeshBlock) void k_mesh_count(MeshArgs A, uint32_t *row_tris, uint32_t *unit_tris,
                                                           uint32_t unit0)
{
    const uint32_t u = unit0 + blockIdx.x;
    __shared__ uint32_t s_sum;
    if (threadIdx.x == 0) s_sum = 0;
    __syncthreads();
    const int lane = (int)(threadIdx.x & 63u);
    for (uint32_t j = threadIdx.x / 64; j < kMeshUnit; j += kMeshWaves) {
        const uint32_t r = u * kMeshUnit + j;
        if (r >= A.nrows) break;
        int32_t row[4];
        mesh_rows(A, r, row);
        uint32_t n = 0;
        for (int32_t z0 = 0; z0 < A.n[2]; z0 += 63) {
            const MeshSpan P = mesh_span(A, row, z0, lane);
            if ((P.act >> lane) & 1ull) n += kTable.count[P.signs];
        }
        if (__any(n != 0)) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) n += (uint32_t)__shfl_xor((int)n, off);
        }
        if (lane == 0) {
            row_tris[r] = n;
            if (n) atomicAdd(&s_sum, n);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) unit_tris[u] = s_sum;
}

__device__ __forceinline__ void mesh_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Units unit0 + blockIdx.x; unit u's triangles go to out at unit_base[u] -
// base.
__global__ __launch_bounds__(kEmitBlock) void k_mesh_emit(MeshArgs A, const uint32_t *row_tris,
                                                          const uint64_t *unit_base, uint32_t unit0, uint64_t base,
                                                          float *out)
{
    __shared__ uint32_t s_row[kMeshUnit];
    __shared__ int16_t s_val[kEmitWaves][4][64];
    __shared__ uint8_t s_signs[kEmitWaves][64], s_owner[kEmitWaves][64 * kMostTris];
    __shared__ uint16_t s_off[kEmitWaves][64];
    const uint32_t u = unit0 + blockIdx.x;
    if (unit_base[u + 1] == unit_base[u]) return;
    if (threadIdx.x < kMeshUnit) {
        const uint32_t r = u * kMeshUnit + threadIdx.x;
        s_row[threadIdx.x] = r < A.nrows ? row_tris[r] : 0u;
    }
    __syncthreads();
    const int lane = (int)(threadIdx.x & 63u), wave = (int)(threadIdx.x / 64u);
    const uint32_t j = (uint32_t)wave;  // this wave's row
    if (s_row[j] != 0) {
        uint64_t at = unit_base[u] - base;
        for (uint32_t k = 0; k < j; ++k) at += s_row[k];
        const uint32_t r = u * kMeshUnit + j;
        int32_t row[4];
        mesh_rows(A, r, row);
        const int32_t gx = A.lo[0] + (int32_t)(r / (uint32_t)A.n[1]), gy = A.lo[1] + (int32_t)(r % (uint32_t)A.n[1]);
        for (int32_t z0 = 0; z0 < A.n[2]; z0 += 63) {
            const MeshSpan P = mesh_span(A, row, z0, lane);
            if (!P.act) continue;
            const uint32_t n = (P.act >> lane) & 1ull ? kTable.count[P.signs] : 0u;
            uint32_t pre = n;  // inclusive prefix over the wave
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t a = (uint32_t)__shfl_up((int)pre, off);
                pre += lane >= off ? a : 0u;
            }
            const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)pre, 63);
#pragma unroll
            for (int q = 0; q < 4; ++q) s_val[wave][q][lane] = (int16_t)P.s[q];
            s_signs[wave][lane] = (uint8_t)P.signs;
            s_off[wave][lane] = (uint16_t)(pre - n);
            for (uint32_t k = 0; k < n; ++k) s_owner[wave][pre - n + k] = (uint8_t)lane;
            mesh_wave_sync();
            for (uint32_t t = (uint32_t)lane; t < total; t += 64) {
                const int o = s_owner[wave][t];
                const uint32_t tri = kTable.tri[s_signs[wave][o]][t - s_off[wave][o]];
                const int32_t g[3] = {gx, gy, A.lo[2] + z0 + o};
                float *p = out + 9 * (at + t);
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const int a = (int)(tri >> (6 * e)) & 7, b = (int)(tri >> (6 * e + 3)) & 7;
                    const int32_t sa = s_val[wave][a & 3][o + (a >> 2)], sb = s_val[wave][b & 3][o + (b >> 2)];
                    const double f = (double)sa / ((double)sa - (double)sb);
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const double ga = (double)(g[k] + ((a >> k) & 1)) + 0.5;
                        const double gb = (double)(g[k] + ((b >> k) & 1)) + 0.5;
                        p[3 * e + k] = (float)((ga + f * (gb - ga)) * A.vs);
                    }
                }
            }
            mesh_wave_sync();
            at += total;
        }
    }
}

}  // namespace

hipError_t launch_mesh_count(const MeshArgs &A, uint32_t *row_tris, uint32_t *unit_tris, hipStream_t stream)
{
    const uint32_t units = mesh_units(A.nrows);
    for (uint32_t u = 0; u < units; u += kCountUnits) {
        hipLaunchKernelGGL(k_mesh_count, dim3(std::min(kCountUnits, units - u)), dim3(kMeshBlock), 0, stream, A, row_tris,
                           unit_tris, u);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_mesh_emit(const MeshArgs &A, const uint32_t *row_tris, const uint64_t *unit_base, uint32_t unit0,
                            uint32_t units, uint64_t base, float *out, hipStream_t stream)
{
    for (uint32_t u = 0; u < units; u += kEmitUnits) {
        hipLaunchKernelGGL(k_mesh_emit, dim3(std::min(kEmitUnits, units - u)), dim3(kEmitBlock), 0, stream, A, row_tris,
                           unit_base, unit0 + u, base, out);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace tsdf
