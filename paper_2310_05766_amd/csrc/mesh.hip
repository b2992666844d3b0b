// Surface extraction for inspection: the zero level set of the resident
// window in a box, by marching tetrahedra (each cube of 8 observed voxel
// centres cut into the 6 tetrahedra around its 0-7 diagonal; one or two
// triangles per tetrahedron with a sign change; edge points at
// t = s_a / (s_a - s_b) in float64). Two passes give a deterministic order,
// cube by cube (x, then y, then z): a count per row of cubes (per group of short
// rows, which share a wave), and, after an exclusive scan over units of 16 rows
// (groups) on the host, an emit pass.
//
// Almost all cubes hold no surface (1 in 45 of a window around a room), so
// both passes look at 63 cubes of a row at once: a wave reads 64 voxels of the
// four voxel rows around them, ballots "observed" and "negative", and works
// out on eight 64-bit masks which cubes are complete and change sign; where no
// cube is complete, the distances are not read at all. Only then do lanes look
// up what their cube holds in a table over its eight signs. The emit pass
// spreads a wave's triangles over its lanes, one triangle per lane, however
// many each cube gives. Rows of at most 31 cubes (a slice of the ground) share
// a wave, or most of its lanes would idle: 512 x 512 voxels, 2 layers, count 41 ->
// 25 us and emit 29 -> 20 (a thread per cube: 16 and 43), 9 layers 41 -> 20 and 31 ->
// 20 (27 and 61). A 512 x 512 x 256 window with 5.8 M triangles: count
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
// The emit pass has a wave per row (group): where a wall lies along y, its few rows
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

// The cubes of a wave: 63 (64 voxels) of one row from voxel z0 on, or, in thin
// boxes, a group of rows side by side, 2^lseg lanes each. q = (x | y << 1) numbers
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

// Slot of a row's voxel z of the box, 0 past the box.
__device__ __forceinline__ int32_t mesh_z(const MeshArgs &A, int32_t z, bool valid)
{
    int32_t sz = A.s0[2] + z;
    sz -= sz >= A.dims[2] ? A.dims[2] : 0;
    return valid ? sz : 0;
}

// valid: this lane has a voxel of the box; ends: lanes that end a row of a group.
__device__ __forceinline__ MeshSpan mesh_span(const MeshArgs &A, const int32_t row[4], int32_t sz, bool valid, uint64_t ends)
{
    MeshSpan P;
    P.act = 0;
    P.signs = 0;
    int32_t w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) w[q] = A.w[row[q] + sz];
    uint64_t seen = __ballot(valid);
#pragma unroll
    for (int q = 0; q < 4; ++q) seen &= __ballot(w[q] > 0);
    const uint64_t cubes = seen & (seen >> 1) & ~ends;  // (the last voxel of a span or row starts no cube)
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

__device__ __forceinline__ uint32_t wave_sum(uint32_t n)
{
    if (__any(n != 0)) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) n += (uint32_t)__shfl_xor((int)n, off);
    }
    return n;
}

// A workgroup per unit, its waves take the unit's groups in turn.
template <bool kThin>
__global__ __launch_bounds__(kMeshBlock) void k_mesh_count(MeshArgs A, uint32_t *group_tris, uint32_t *unit_tris,
                                                           uint32_t unit0)
{
    constexpr uint32_t kPasses = kMeshUnit / kMeshWaves;
    const uint32_t u = unit0 + blockIdx.x;
    __shared__ uint32_t s_sum;
    if (threadIdx.x == 0) s_sum = 0;
    __syncthreads();
    const int lane = (int)(threadIdx.x & 63u);
    const uint32_t group0 = u * kMeshUnit + threadIdx.x / 64;
    const auto store = [&](uint32_t group, uint32_t n) {
        n = wave_sum(n);
        if (lane == 0) {
            group_tris[group] = n;
            if (n) atomicAdd(&s_sum, n);
        }
    };
    if (kThin) {
        // the first of each row's four voxel rows, of all passes together: in most
        // groups it holds nothing observed
        const int32_t z = lane & ((1 << A.lseg) - 1);
        const uint64_t ends = __ballot(z == (1 << A.lseg) - 1);
        const int32_t sz = mesh_z(A, z, z <= A.n[2]);
        int32_t row[kPasses][4], first[kPasses];
#pragma unroll
        for (uint32_t k = 0; k < kPasses; ++k) {
            const uint32_t r = (group0 + k * kMeshWaves) * (64u >> A.lseg) + (uint32_t)(lane >> A.lseg);
            const bool in = r < A.nrows && z <= A.n[2];
            mesh_rows(A, in ? r : 0u, row[k]);
            first[k] = in ? A.w[row[k][0] + sz] : 0;
        }
#pragma unroll
        for (uint32_t k = 0; k < kPasses; ++k) {
            if (group0 + k * kMeshWaves >= A.groups) break;
            uint32_t n = 0;
            if (__any(first[k] > 0)) {
                const MeshSpan P = mesh_span(A, row[k], sz, first[k] > 0, ends);
                if ((P.act >> lane) & 1ull) n = kTable.count[P.signs];
            }
            store(group0 + k * kMeshWaves, n);
        }
    } else {
        for (uint32_t k = 0; k < kPasses; ++k) {
            const uint32_t r = group0 + k * kMeshWaves;
            if (r >= A.groups) break;
            int32_t row[4];
            mesh_rows(A, r, row);
            uint32_t n = 0;
            for (int32_t z0 = 0; z0 < A.n[2]; z0 += 63) {
                const bool valid = z0 + lane <= A.n[2];  // n cubes are n + 1 voxels
                const MeshSpan P = mesh_span(A, row, mesh_z(A, z0 + lane, valid), valid, 0);
                if ((P.act >> lane) & 1ull) n += kTable.count[P.signs];
            }
            store(r, n);
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
template <bool kThin>
__global__ __launch_bounds__(kEmitBlock) void k_mesh_emit(MeshArgs A, const uint32_t *group_tris,
                                                          const uint64_t *unit_base, uint32_t unit0, uint64_t base,
                                                          float *out)
{
    __shared__ uint32_t s_group[kMeshUnit];
    __shared__ int16_t s_val[kEmitWaves][4][64];
    __shared__ uint8_t s_signs[kEmitWaves][64], s_owner[kEmitWaves][64 * kMostTris];
    __shared__ uint16_t s_off[kEmitWaves][64];
    const uint32_t u = unit0 + blockIdx.x;
    if (unit_base[u + 1] == unit_base[u]) return;
    if (threadIdx.x < kMeshUnit) {
        const uint32_t g = u * kMeshUnit + threadIdx.x;
        s_group[threadIdx.x] = g < A.groups ? group_tris[g] : 0u;
    }
    __syncthreads();
    const int lane = (int)(threadIdx.x & 63u), wave = (int)(threadIdx.x / 64u);
    const uint32_t j = (uint32_t)wave;  // this wave's group
    if (s_group[j] != 0) {
        uint64_t at = unit_base[u] - base;
        for (uint32_t k = 0; k < j; ++k) at += s_group[k];
        const int lseg = kThin ? A.lseg : 6;
        const uint32_t r0 = (u * kMeshUnit + j) << (6 - lseg), r = r0 + (uint32_t)(lane >> lseg);
        const int32_t zl = lane & ((1 << lseg) - 1);
        const uint64_t ends = kThin ? __ballot(zl == (1 << lseg) - 1) : 0ull;
        const bool in = r < A.nrows;
        int32_t row[4];
        mesh_rows(A, in ? r : 0u, row);
        const int32_t gx = A.lo[0] + (int32_t)(r0 / (uint32_t)A.n[1]), gy = A.lo[1] + (int32_t)(r0 % (uint32_t)A.n[1]);
        for (int32_t z0 = 0; z0 < A.n[2]; z0 += 63) {  // (once in thin boxes)
            const bool valid = in && z0 + zl <= A.n[2];
            const MeshSpan P = mesh_span(A, row, mesh_z(A, z0 + zl, valid), valid, ends);
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
                int32_t g[3] = {gx, gy, A.lo[2] + z0 + (o & ((1 << lseg) - 1))};
                if (kThin) {
                    const uint32_t ro = r0 + (uint32_t)(o >> lseg);
                    g[0] = A.lo[0] + (int32_t)(ro / (uint32_t)A.n[1]);
                    g[1] = A.lo[1] + (int32_t)(ro % (uint32_t)A.n[1]);
                }
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

void mesh_groups(MeshArgs &A)
{
    A.lseg = 1;
    while (A.lseg < 6 && A.n[2] >= 1 << A.lseg) ++A.lseg;
    const uint32_t per = 64u >> A.lseg;
    A.groups = (A.nrows + per - 1) / per;
}

hipError_t launch_mesh_count(const MeshArgs &A, uint32_t *group_tris, uint32_t *unit_tris, hipStream_t stream)
{
    const uint32_t units = mesh_units(A);
    for (uint32_t u = 0; u < units; u += kCountUnits) {
        const dim3 grid(std::min(kCountUnits, units - u)), block(kMeshBlock);
        if (A.lseg < 6) hipLaunchKernelGGL(k_mesh_count<true>, grid, block, 0, stream, A, group_tris, unit_tris, u);
        else hipLaunchKernelGGL(k_mesh_count<false>, grid, block, 0, stream, A, group_tris, unit_tris, u);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_mesh_emit(const MeshArgs &A, const uint32_t *group_tris, const uint64_t *unit_base, uint32_t unit0,
                            uint32_t units, uint64_t base, float *out, hipStream_t stream)
{
    for (uint32_t u = 0; u < units; u += kEmitUnits) {
        const dim3 grid(std::min(kEmitUnits, units - u)), block(kEmitBlock);
        if (A.lseg < 6) hipLaunchKernelGGL(k_mesh_emit<true>, grid, block, 0, stream, A, group_tris, unit_base, unit0 + u, base, out);
        else hipLaunchKernelGGL(k_mesh_emit<false>, grid, block, 0, stream, A, group_tris, unit_base, unit0 + u, base, out);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace tsdf
