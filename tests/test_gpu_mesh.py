"""GPU parity of surface extraction (marching tetrahedra over the resident
window): triangles in the same order and bit-identical to the oracle's."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def test_mesh_config1_and_sub_boxes():
    from paper_2310_05766_amd.tsdf import TsdfMap
    w = synth.config1()
    spec, sc = w.maps[0], w.scans[0]
    gm = TsdfMap.from_spec(spec)
    om = oracle.OracleMap.from_spec(spec)
    for k, p in enumerate([sc.pose, synth.fuzz_pose((71, 0), 0.3)]):
        gm.integrate(sc.xyz, p)
        om.integrate(sc.xyz, p)
    lo, hi = spec.origin, tuple(spec.origin[a] + spec.dims[a] for a in range(3))
    boxes = [(lo, hi), ((lo[0] + 3, lo[1] + 10, lo[2] + 1), (hi[0] - 7, hi[1] - 2, lo[2] + 60)),
             ((0, 0, 0), (1, 1, 1)), ((5, 5, 5), (5, 9, 9))]
    for blo, bhi in boxes:
        g = gm.mesh(blo, bhi)
        o = om.mesh(blo, bhi)
        say("box", blo, bhi, "triangles", g.shape[0])
        assert g.shape == o.shape
        assert np.array_equal(g, o)
    assert gm.mesh(lo, hi).shape[0] > 10000
    gm.close()
    om.close()


def test_mesh_after_shift_and_errors():
    """The ring buffer's slot addressing after a shift; boxes outside the
    window are rejected; a too small output is reported."""
    from paper_2310_05766_amd import TsdfError
    from paper_2310_05766_amd import _abi
    import ctypes as C
    from paper_2310_05766_amd.tsdf import TsdfMap
    dims, origin = (64, 64, 64), (-32, -32, -32)
    gm = TsdfMap(dims, origin, 0.05, 3072, 64)
    om = oracle.OracleMap(dims, origin, 0.05, 3072, 64)
    for k in range(3):
        xyz = synth.fuzz_scan((72, k), 4000, extent_m=1.2, nan_frac=0.02)
        pose = synth.fuzz_pose((73, k), 0.3)
        gm.integrate(xyz, pose)
        om.integrate(xyz, pose)
    new = (-32 + 19, -32 - 7, -32)
    gm.shift(new)
    om.shift(new)
    hi = tuple(new[a] + dims[a] for a in range(3))
    assert np.array_equal(gm.mesh(new, hi), om.mesh(new, hi))
    with pytest.raises(TsdfError):
        gm.mesh(origin, (origin[0] + 64, origin[1] + 64, origin[2] + 64))
    lo_a, hi_a = (C.c_int32 * 3)(*new), (C.c_int32 * 3)(*hi)
    n = C.c_int64()
    assert _abi.lib().tsdf_mesh(gm.handle, lo_a, hi_a, None, 0, C.byref(n)) == 0 and n.value > 0
    small = np.zeros((1, 9), np.float32)
    rc = _abi.lib().tsdf_mesh(gm.handle, lo_a, hi_a, small.ctypes.data_as(C.POINTER(C.c_float)), 1, C.byref(n))
    assert rc == _abi.TSDF_ERANGE
    gm.close()
    om.close()


def _random_pair(dims, origin, seen, seed):
    """A GPU map on caller-owned arrays and an oracle map with the same random
    voxels: a share `seen` of them observed, every sign pattern among them."""
    import torch
    from paper_2310_05766_amd.tsdf import TsdfMap
    g = np.random.Generator(np.random.PCG64(seed))
    w = (g.random(dims) < seen).astype(np.int16) * g.integers(1, 65, dims, dtype=np.int16)
    sdf = np.where(w > 0, g.integers(-3072, 3073, dims), 0).astype(np.int16)
    hi = tuple(origin[a] + dims[a] for a in range(3))
    om = oracle.OracleMap(dims, origin, 0.05, 3072, 64)
    om.set_voxels(origin, hi, sdf, w)
    # slot s of an axis holds the voxel origin + (s - origin) mod n
    ix = np.ix_(*[(np.arange(n) - o) % n for n, o in zip(dims, origin)])
    arrays = [torch.from_numpy(np.ascontiguousarray(v[ix])).to("cuda") for v in (sdf, w)]
    scratch = torch.zeros(TsdfMap.scratch_bytes(dims, origin, 0.05, 3072, 64), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    return TsdfMap(dims, origin, 0.05, 3072, 64, arrays=(*arrays, scratch)), om


@pytest.mark.parametrize("cubes", [(1, 1, 1), (3, 5, 62), (3, 5, 63), (2, 8, 64), (1, 17, 126), (5, 3, 127), (4, 4, 140)])
def test_mesh_row_and_unit_edges(cubes):
    """Rows of cubes around one and two spans of a wave, units of rows that
    are cut, and the ring buffer's wrap inside the box: bit-identical."""
    dims, origin = (9, 19, 143), (-4, -13, -61)
    gm, om = _random_pair(dims, origin, 0.97, 5)
    lo = tuple(origin[a] + (dims[a] - cubes[a]) // 2 for a in range(3))
    hi = tuple(lo[a] + cubes[a] + 1 for a in range(3))
    g, o = gm.mesh(lo, hi), om.mesh(lo, hi)
    say(cubes, g.shape)
    assert g.shape == o.shape and np.array_equal(g, o)
    gm.close()
    om.close()


@pytest.mark.parametrize("dims", [(40, 44, 63), (60, 66, 150), (70, 90, 150)])
def test_mesh_through_staging_slots(dims):
    """Results of some, of more than one, and of more than two pieces of
    staging: every slot and buffer is used again."""
    origin = (-11, 5, -40)
    gm, om = _random_pair(dims, origin, 0.92, 6)
    hi = tuple(origin[a] + dims[a] for a in range(3))
    g, o = gm.mesh(origin, hi), om.mesh(origin, hi)
    say(dims, g.shape, g.nbytes)
    assert g.shape == o.shape and np.array_equal(g, o)
    gm.close()
    om.close()


@pytest.mark.parametrize("dims", [(12, 14, 63), (40, 44, 63)])
def test_mesh_with_and_without_staging(dims):
    """A map's first mesh leaves without staging, a later one of more than 4 MB
    through it, and a small one after that through what is there."""
    origin = (-11, 5, -40)
    gm, om = _random_pair(dims, origin, 0.92, 7)
    hi = tuple(origin[a] + dims[a] for a in range(3))
    o, part = om.mesh(origin, hi), om.mesh(origin, (origin[0] + 5, origin[1] + 6, hi[2]))
    for k in range(3):
        g = gm.mesh(origin, hi)
        say(dims, k, g.shape, g.nbytes)
        assert g.shape == o.shape and np.array_equal(g, o)
    g = gm.mesh(origin, (origin[0] + 5, origin[1] + 6, hi[2]))
    assert g.shape == part.shape and np.array_equal(g, part)
    gm.close()
    om.close()


def test_mesh_of_a_thin_wide_window():
    """More rows of cubes than one launch holds work-items for (2^28 rows in
    units of 16 under 256 threads to count, 2^26 under 1024 to emit): the scans
    of a corner and of the far corner, in the order of a small window's meshes."""
    from paper_2310_05766_amd.tsdf import TsdfMap
    dims, origin = (16384, 16400, 4), (-8192, -8200, -2)
    assert (dims[0] - 1) * (dims[1] - 1) > 1 << 28
    gm = TsdfMap(dims, origin, 0.1, 3072, 64)
    parts = []
    for corner in (0, 1):
        at = [origin[a] + corner * (dims[a] - 48) for a in range(2)]
        small = TsdfMap((48, 48, 4), (at[0], at[1], -2), 0.1, 3072, 64)
        pose = np.eye(4)
        pose[:3, 3] = ((at[0] + 24) * 0.1, (at[1] + 24) * 0.1, 0.6)
        g = np.random.default_rng((74, corner))
        xyz = np.concatenate([g.uniform(-1.5, 1.5, (20000, 2)), g.uniform(-0.65, -0.55, (20000, 1))], 1).astype(np.float32)
        for m in (gm, small):
            m.integrate(xyz, pose)
        parts.append(small.mesh((at[0], at[1], -2), (at[0] + 48, at[1] + 48, 2)))
        small.close()
    say("mesh of", dims, "triangles", [p.shape[0] for p in parts])
    assert min(p.shape[0] for p in parts) > 1000
    import torch
    gm.synchronize()
    free = torch.cuda.mem_get_info()[0]
    g = gm.mesh(origin, tuple(origin[a] + dims[a] for a in range(3)))
    want = np.concatenate(parts)
    assert g.shape == want.shape and np.array_equal(g, want)
    assert free - torch.cuda.mem_get_info()[0] < 40 << 20  # (counts of all rows are given back)
    gm.close()


@pytest.mark.parametrize("layers", [1, 2, 3, 4, 7, 8, 15, 16, 30, 31, 32])
@pytest.mark.parametrize("rows", [(1, 1), (7, 9), (40, 37)])
def test_mesh_of_thin_boxes(rows, layers):
    """Short rows of cubes that share a wave, around every number of lanes that
    a row may take: groups and units that are cut, the ring buffer's wrap inside
    the box; bit-identical."""
    dims, origin = (43, 41, 37), (-20, -13, -15)
    gm, om = _random_pair(dims, origin, 0.95, 8)
    lo = tuple(origin[a] + (dims[a] - c) // 2 for a, c in enumerate((*rows, layers)))
    hi = tuple(lo[a] + c + 1 for a, c in enumerate((*rows, layers)))
    g, o = gm.mesh(lo, hi), om.mesh(lo, hi)
    say(rows, layers, g.shape)
    assert g.shape == o.shape and np.array_equal(g, o)
    gm.close()
    om.close()


def test_mesh_of_a_tall_window():
    """Units of more triangles than a staging slot should hold (16 rows of 9,000
    cubes) leave without staging, and their memory is given back; twice."""
    import torch
    dims, origin = (5, 5, 9000), (-2, -3, -4500)
    gm, om = _random_pair(dims, origin, 0.97, 9)
    hi = tuple(origin[a] + dims[a] for a in range(3))
    o = om.mesh(origin, hi)
    free = torch.cuda.mem_get_info()[0]
    for k in range(2):
        g = gm.mesh(origin, hi)
        say(dims, g.shape, g.nbytes)
        assert g.shape == o.shape and np.array_equal(g, o)
    assert g.nbytes * 8 > 64 << 20 and free - torch.cuda.mem_get_info()[0] < 80 << 20
    gm.close()
    om.close()
