"""GPU parity of the batched forms: ordered multi-scan batches on one map,
interleaved batches over several maps, batches longer than one chunk, and
every candidate tiling -- each bit-exact with the oracle applied scan by
scan in submission order."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def gpu_map(dims, origin, vs, tau, wmax):
    from paper_2310_05766_amd.tsdf import TsdfMap
    return TsdfMap(dims, origin, vs, tau, wmax)


def same(gm, om, dims):
    o = gm.origin
    hi = tuple(o[a] + dims[a] for a in range(3))
    g = gm.readback(o, hi)
    r = om.readback(o, hi)
    return np.array_equal(g[0], r[0]) and np.array_equal(g[1], r[1])


def test_config2_ordered_batch():
    from paper_2310_05766_amd.tsdf import integrate_batch
    w = synth.config2(20)
    spec = w.maps[0]
    say("config2: 20 scans, one batch")
    om = oracle.OracleMap.from_spec(spec)
    ost = [om.integrate(s.xyz, s.pose) for s in w.scans]
    gm = gpu_map(spec.dims, spec.origin, spec.voxel_size, spec.tau_u, spec.w_max)
    gst = integrate_batch([(gm, s.xyz, s.pose) for s in w.scans], stats=True)
    assert gst == ost
    assert same(gm, om, spec.dims)
    gm.close()
    om.close()


def test_config2_full_batch_as_benchmarked():
    """The benchmark's launch shape: all 50 OS1-128 scans of the sequence as
    one ordered batch, points already in device memory, on a stream of its
    own, graph launch on; the second batch replays the captured graph."""
    import torch
    from paper_2310_05766_amd.tsdf import TsdfMap, integrate_batch, set_graph_launch
    w = synth.config2()
    spec = w.maps[0]
    set_graph_launch(True)
    st = torch.cuda.Stream()
    dev = [torch.from_numpy(s.xyz).to("cuda") for s in w.scans]
    torch.cuda.synchronize()
    gm = TsdfMap.from_spec(spec, stream=st)
    om = oracle.OracleMap.from_spec(spec)
    for rep in range(2):
        say("config2: batch of 50, pass", rep)
        integrate_batch([(gm, x, s.pose) for x, s in zip(dev, w.scans)], stream=st)
        for s in w.scans:
            om.integrate(s.xyz, s.pose)
        gm.synchronize()
        assert same(gm, om, spec.dims), rep
    gm.close()
    om.close()


def test_interleaved_maps_and_long_batches():
    """Three maps, scans interleaved in random order; one map gets 70 scans
    (more than one chunk of 64)."""
    from paper_2310_05766_amd.tsdf import integrate_batch
    specs = [((48, 40, 24), (-24, -20, -12), 0.05, 3072, 5),
             ((33, 65, 17), (-16, -30, -8), 0.08, 5120, 64),
             ((64, 64, 64), (-32, -32, -32), 0.064, 5120, 64)]
    g = np.random.default_rng(5)
    order = [0] * 70 + [1] * 12 + [2] * 9
    g.shuffle(order)
    items, refs = [], []
    gms = [gpu_map(*s) for s in specs]
    oms = [oracle.OracleMap(*s) for s in specs]
    for k, m in enumerate(order):
        xyz = synth.fuzz_scan((77, k), 1500 + 97 * (k % 5), extent_m=1.5, nan_frac=0.05,
                              grid_snap=0.05 if k % 7 == 0 else None)
        pose = synth.fuzz_pose((78, k), max_t=0.3)
        items.append((gms[m], xyz, pose))
        refs.append(oms[m].integrate(xyz, pose))
    say("interleaved batch of", len(items), "scans")
    st = integrate_batch(items, stats=True)
    assert st == refs
    for k, s in enumerate(specs):
        assert same(gms[k], oms[k], s[0]), k
        gms[k].close()
        oms[k].close()


TILINGS = [(3, 3, 3), (2, 3, 4), (3, 4, 5), (4, 4, 4), (2, 2, 5), (4, 3, 3), (3, 3, 6), (4, 4, 3)]


@pytest.mark.parametrize("lt", TILINGS)
def test_every_tiling_gives_the_same_map(lt):
    from paper_2310_05766_amd.tsdf import integrate_batch
    w = synth.config1()
    spec, sc = w.maps[0], w.scans[0]
    om = oracle.OracleMap.from_spec(spec)
    gm = gpu_map(spec.dims, spec.origin, spec.voxel_size, spec.tau_u, spec.w_max)
    gm.set_tiling(lt)
    assert gm.get_tiling()[0] == tuple(lt)
    poses = [sc.pose] + [synth.fuzz_pose((lt, k), 0.4) for k in range(5)]
    for p in poses[:2]:
        assert gm.integrate(sc.xyz, p, stats=True) == om.integrate(sc.xyz, p)
    st = integrate_batch([(gm, sc.xyz, p) for p in poses[2:]], stats=True)
    assert st == [om.integrate(sc.xyz, p) for p in poses[2:]]
    assert same(gm, om, spec.dims)
    gm.close()
    om.close()


@pytest.mark.parametrize("workgroups", [1, 3, 7, 8, 9])
def test_few_tile_workgroups_drain_every_queue(workgroups):
    """Grids smaller than the number of work queues (one per XCD): every busy
    tile is still processed, over two batches in a row (the second starts
    from the per-tile counts the first left), bit-exact with the oracle."""
    from paper_2310_05766_amd.tsdf import integrate_batch
    w = synth.config1()
    spec, sc = w.maps[0], w.scans[0]
    om = oracle.OracleMap.from_spec(spec)
    gm = gpu_map(spec.dims, spec.origin, spec.voxel_size, spec.tau_u, spec.w_max)
    gm.set_tiling((3, 3, 3), workgroups)
    assert gm.get_tiling() == ((3, 3, 3), workgroups)
    for b in range(2):
        poses = [synth.fuzz_pose((workgroups, b, k), 0.4) for k in range(3)]
        st = integrate_batch([(gm, sc.xyz, p) for p in poses], stats=True)
        assert st == [om.integrate(sc.xyz, p) for p in poses], (workgroups, b)
        assert gm.integrate(sc.xyz, sc.pose, stats=True) == om.integrate(sc.xyz, sc.pose)
    assert same(gm, om, spec.dims)
    gm.close()
    om.close()


@pytest.mark.parametrize("blocks", [(128, 256), (512, 256), (256, 512), (512, 512), (128, 512)])
def test_every_block_size_gives_the_same_map(blocks):
    """Binning blocks of 128, 256 and 512 points and tile workgroups of 256
    and 512 threads: the same map and counts as the oracle, for single
    scans and for a batch of several scans of one map."""
    from paper_2310_05766_amd import TsdfError
    from paper_2310_05766_amd.tsdf import integrate_batch
    w = synth.config1()
    spec, sc = w.maps[0], w.scans[0]
    om = oracle.OracleMap.from_spec(spec)
    gm = gpu_map(spec.dims, spec.origin, spec.voxel_size, spec.tau_u, spec.w_max)
    gm.set_blocks(*blocks)
    assert gm.get_blocks() == tuple(blocks)
    poses = [sc.pose] + [synth.fuzz_pose((blocks, k), 0.4) for k in range(9)]
    for p in poses[:2]:
        assert gm.integrate(sc.xyz, p, stats=True) == om.integrate(sc.xyz, p)
    st = integrate_batch([(gm, sc.xyz, p) for p in poses[2:]], stats=True)
    assert st == [om.integrate(sc.xyz, p) for p in poses[2:]]
    assert same(gm, om, spec.dims)
    for bad in [(64, 256), (256, 128), (300, 256), (-1, 0)]:
        with pytest.raises(TsdfError):
            gm.set_blocks(*bad)
    gm.set_blocks(0, 0)
    assert gm.get_blocks() == (256, 256)
    gm.close()
    om.close()


def test_invalid_tilings_rejected():
    from paper_2310_05766_amd import TsdfError
    gm = gpu_map((32, 32, 32), (-16, -16, -16), 0.05, 3072, 64)
    assert gm.get_tiling()[0] == (0, 0, 0)  # chosen per call until set
    for lt in [(1, 4, 4), (3, 3, 2), (7, 3, 3), (2, 2, 3), (5, 5, 5), (0, 3, 3)]:
        with pytest.raises(TsdfError):
            gm.set_tiling(lt)
    gm.set_tiling((4, 4, 4))
    gm.set_tiling((0, 0, 0))
    assert gm.get_tiling()[0] == (0, 0, 0)
    gm.close()


def test_batch_of_nothing_and_empty_scans():
    from paper_2310_05766_amd.tsdf import integrate_batch
    gm = gpu_map((16, 16, 16), (-8, -8, -8), 0.1, 3072, 64)
    om = oracle.OracleMap((16, 16, 16), (-8, -8, -8), 0.1, 3072, 64)
    assert integrate_batch([]) is None
    xyz = synth.fuzz_scan(91, 300, extent_m=0.7)
    items = [(gm, np.zeros((0, 3), np.float32), np.eye(4)), (gm, xyz, np.eye(4)),
             (gm, np.full((5, 3), np.nan, np.float32), np.eye(4))]
    st = integrate_batch(items, stats=True)
    ref = [om.integrate(x, p) for _, x, p in items]
    assert st == ref
    assert same(gm, om, (16, 16, 16))
    gm.close()
    om.close()


def test_graph_replays_match_direct_launches():
    """Captured graphs replayed many times, with eager work and syncs in
    between, give the same maps as direct launches and as the oracle."""
    from paper_2310_05766_amd.tsdf import integrate_batch, set_graph_launch
    w = synth.config1()
    spec, sc = w.maps[0], w.scans[0]
    om = oracle.OracleMap.from_spec(spec)
    maps = {}
    try:
        for mode in (True, False):
            set_graph_launch(mode)
            gm = gpu_map(spec.dims, spec.origin, spec.voxel_size, spec.tau_u, spec.w_max)
            snaps = []
            for k in range(6):
                poses = [synth.fuzz_pose((k, j, 5), 0.4) for j in range(1 + k % 3)]
                if k % 2:
                    integrate_batch([(gm, sc.xyz[: 4000 + 1000 * j], p) for j, p in enumerate(poses)])
                else:
                    for j, p in enumerate(poses):
                        gm.integrate(sc.xyz[: 4000 + 1000 * j], p)
                gm.synchronize()
                snaps.append(gm.readback_window())
                if mode:
                    for j, p in enumerate(poses):
                        om.integrate(sc.xyz[: 4000 + 1000 * j], p)
                    ref = om.readback(spec.origin, tuple(spec.origin[a] + spec.dims[a] for a in range(3)))
                    assert np.array_equal(snaps[-1][0], ref[0]) and np.array_equal(snaps[-1][1], ref[1]), k
            maps[mode] = snaps
            gm.close()
    finally:
        set_graph_launch(True)
    for a, b in zip(maps[True], maps[False]):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    om.close()


def test_autotuner_candidates_agree(tmp_path, monkeypatch):
    import torch
    from paper_2310_05766_amd.autotune import autotune
    monkeypatch.setenv("XDG_CACHE_HOME", str(tmp_path))
    w = synth.config1()
    spec, sc = w.maps[0], w.scans[0]
    sample = [(torch.from_numpy(sc.xyz).to("cuda"), synth.fuzz_pose((3, k), 0.3)) for k in range(4)]
    torch.cuda.synchronize()
    best = autotune(spec, sample, mode="batch", reps=1)
    assert tuple(best["lt"]) in [tuple(c["lt"]) for c in best["candidates"]]
    # all three knobs were searched and are recorded: tiling, workgroups, block sizes
    seen = {(c["bin_block"], c["tile_block"]) for c in best["candidates"]}
    assert {(256, 256), (128, 256), (512, 256), (256, 512), (512, 512)} <= seen
    again = autotune(spec, sample, mode="batch", reps=1)
    assert again["cached"] and tuple(again["lt"]) == tuple(best["lt"])
    assert (again["bin_block"], again["tile_block"]) == (best["bin_block"], best["tile_block"])


@pytest.mark.parametrize("lt", [(2, 2, 5), (3, 3, 6), (4, 4, 4), (0, 0, 0)])
def test_longest_bands_resume_at_tile_entries(lt):
    """tau = 32767 (a band of 64 voxels) on rays along z that enter a tile
    after 64 or more voxel crossings on z: the resume counts of the tile
    pass reach their largest values (up to 66 per axis)."""
    from paper_2310_05766_amd.tsdf import integrate_batch
    vs, tau = 1.0, 32767
    dims, origin = (8, 8, 256), (-4, -4, 0)
    om = oracle.OracleMap(dims, origin, vs, tau, 64)
    gm = gpu_map(dims, origin, vs, tau, 64)
    gm.set_tiling(lt)
    pose = np.eye(4)
    pose[:3, 3] = [0.5, 0.5, 0.5]  # sensor on a voxel centre
    pts = []
    for k, zk in enumerate((1, 2, 3, 4, 5)):
        for dz in (2, 10, 500, 1000, 1023):
            # band start S_z = 1024 * 32 * zk + dz (fixed point): 64 crossings
            qz = 1024 * 32 * zk + dz + tau
            pts.append([0.0, 0.0, (qz - 512) / 1024.0])
            pts.append([0.25 * (k - 2) / 1024.0, 0.0, (qz - 512 + 1) / 1024.0])  # nearly vertical
    xyz = np.array(pts, dtype=np.float32)
    assert gm.integrate(xyz, pose, stats=True) == om.integrate(xyz, pose)
    poses = [pose.copy() for _ in range(3)]
    for j, p in enumerate(poses):
        p[:3, 3] = [0.5 - j, 0.5 + j, 0.5 + 7 * j]
    st = integrate_batch([(gm, xyz, p) for p in poses], stats=True)
    assert st == [om.integrate(xyz, p) for p in poses]
    assert same(gm, om, dims)
    gm.close()
    om.close()


@pytest.mark.parametrize("bin_block", [128, 256, 512])
def test_full_binning_table_sends_entries_straight_to_runs(bin_block):
    """Points scattered over a wide window with the longest band (tau =
    32767): each ray crosses about ten tiles, so a binning block meets far
    more (sequence slot, tile) keys than its hash table holds (two slots per
    point) and more tiles per point than it lists in LDS; those entries go
    straight to their runs. Bit-exact with the oracle, one scan and a batch."""
    from paper_2310_05766_amd.tsdf import integrate_batch
    vs, tau = 0.1, 32767
    dims, origin = (256, 256, 64), (-128, -128, -32)
    rng = np.random.default_rng(bin_block)
    xyz = rng.uniform([-12.0, -12.0, -3.0], [12.0, 12.0, 3.0], size=(3000, 3)).astype(np.float32)
    poses = []
    for j in range(3):
        p = np.eye(4)
        p[:3, 3] = [0.03 + 0.4 * j, -0.02 - 0.3 * j, 0.01 + 0.1 * j]
        poses.append(p)
    om = oracle.OracleMap(dims, origin, vs, tau, 64)
    gm = gpu_map(dims, origin, vs, tau, 64)
    gm.set_blocks(bin_block, 0)
    say(f"bin block {bin_block}: one scan")
    assert gm.integrate(xyz, poses[0], stats=True) == om.integrate(xyz, poses[0])
    say(f"bin block {bin_block}: batch of two")
    st = integrate_batch([(gm, xyz, p) for p in poses[1:]], stats=True)
    assert st == [om.integrate(xyz, p) for p in poses[1:]]
    assert same(gm, om, dims)
    gm.close()
    om.close()


@pytest.mark.parametrize("graphs", [True, False])
def test_one_scan_and_multi_scan_batches_interleaved_on_one_stream(graphs):
    """One-scan batches (their descriptors handed to the first kernel, in a
    table of their own) and batches of several scans (descriptor tables
    copied on the engine's copy stream, two device copies used in turn)
    interleaved on one stream, device points, with graph replays and with
    direct launches: the map equals the oracle's scan by scan."""
    torch = pytest.importorskip("torch")
    from paper_2310_05766_amd.tsdf import integrate_batch, set_graph_launch
    w = synth.config2(12)
    spec = w.maps[0]
    say("one-scan and multi-scan batches interleaved, graphs", graphs)
    om = oracle.OracleMap.from_spec(spec)
    for s in w.scans:
        om.integrate(s.xyz, s.pose)
    dev = [torch.from_numpy(s.xyz).to("cuda") for s in w.scans]
    st = torch.cuda.Stream()
    set_graph_launch(graphs)
    try:
        from paper_2310_05766_amd.tsdf import TsdfMap
        gm = TsdfMap.from_spec(spec, stream=st)
        # sizes 1, 3, 1, 2, 1, 4: every batch kind follows every other
        k = 0
        for n in (1, 3, 1, 2, 1, 4):
            integrate_batch([(gm, dev[j], w.scans[j].pose) for j in range(k, k + n)], stream=st)
            k += n
        assert k == len(w.scans)
        assert same(gm, om, spec.dims)
        gm.close()
    finally:
        set_graph_launch(True)


@pytest.mark.parametrize("n", [32767, 32768, 32769, 65535, 70001])
@pytest.mark.parametrize("bin_block", [128, 256, 512])
def test_every_point_is_binned_once(n, bin_block):
    """Binning blocks take patches of 32 rows of a scan's points while whole
    groups of 32 x 1024 points are left, then points in order: around the group
    size, counts and maps are the oracle's (a point left out or taken twice
    changes points_valid and visits)."""
    dims, origin = (64, 72, 56), (-32, -36, -28)
    om = oracle.OracleMap(dims, origin, 0.1, 3072, 64)
    gm = gpu_map(dims, origin, 0.1, 3072, 64)
    gm.set_blocks(bin_block, 0)
    for k in range(2):
        xyz, pose = synth.fuzz_scan((91, n, k), n, extent_m=3.0, nan_frac=0.02), synth.fuzz_pose((92, k), 0.5)
        assert gm.integrate(xyz, pose, stats=True) == om.integrate(xyz, pose)
    assert same(gm, om, dims)
    gm.close()
    om.close()


@pytest.mark.parametrize("tau,n", [(5120, 1 << 18), (5120, (1 << 18) + 1), (8190, 1 << 18), (8191, 1 << 18),
                                   (32767, 1 << 15), (32767, (1 << 15) + 1), (1, 1), (4095, 4097)])
def test_key_widths_of_the_tile_pass(tau, n):
    """On both sides of where the tile pass's keys fit 32 bits (bits of tau,
    bits of the largest point index, one for the sign; no key may equal the
    empty one), on a window whose edges cut tiles: one slot per tile and
    several, ties of |s| among many points of one voxel decided by the index."""
    from paper_2310_05766_amd.tsdf import integrate_batch
    dims, origin = (41, 39, 35), (-20, -19, -17)
    om = oracle.OracleMap(dims, origin, 0.1, tau, 64)
    gm = gpu_map(dims, origin, 0.1, tau, 64)
    scans = [(synth.fuzz_scan((93, tau, k), n if k == 0 else 3000, extent_m=2.5, nan_frac=0.02, grid_snap=0.05),
              synth.fuzz_pose((94, k), 0.3)) for k in range(3)]
    ost = [om.integrate(x, p) for x, p in scans]
    assert gm.integrate(*scans[0], stats=True) == ost[0]
    assert integrate_batch([(gm, x, p) for x, p in scans[1:]], stats=True) == ost[1:]
    assert same(gm, om, dims)
    ost = [om.integrate(x, p) for x, p in scans]
    assert integrate_batch([(gm, x, p) for x, p in scans], stats=True) == ost
    assert same(gm, om, dims)
    gm.close()
    om.close()


@pytest.mark.parametrize("maps,per_map,n", [(3, 1, 43690), (3, 1, 43691), (2, 2, 5000), (2, 8, 3000), (2, 9, 3000)])
def test_automatic_tilings(maps, per_map, n):
    """A batch's tiling follows from the most scans of one map and, for one
    scan each, from the points of all (more than 131,072): on both sides of
    each line, counts and maps are the oracle's."""
    from paper_2310_05766_amd.tsdf import integrate_batch
    dims, origin = (50, 46, 37), (-25, -23, -18)
    gms = [gpu_map(dims, origin, 0.1, 4000, 64) for _ in range(maps)]
    oms = [oracle.OracleMap(dims, origin, 0.1, 4000, 64) for _ in range(maps)]
    items, ost = [], []
    for k in range(maps * per_map):
        x, p = synth.fuzz_scan((95, n, k), n, extent_m=2.5, nan_frac=0.02), synth.fuzz_pose((96, k), 0.3)
        items.append((gms[k % maps], x, p))
        ost.append(oms[k % maps].integrate(x, p))
    assert integrate_batch(items, stats=True) == ost
    for g, o in zip(gms, oms):
        assert same(g, o, dims)
        g.close()
        o.close()


@pytest.mark.parametrize("case", ["one_tile", "small_tiles", "long_bands", "several_maps", "many_blocks", "wide_keys"])
def test_one_binning_pass(case):
    """Batches of one scan per map, binned in one pass: tiles with more
    segments than their list and the first chains hold (every block meets the
    same few tiles) and heavy ones, blocks that meet more tiles than their
    table has slots, rays with more tiles than a block lists, several maps,
    many blocks, 64-bit keys; counts and maps are the oracle's, twice in a row
    (the lists are empty again)."""
    from paper_2310_05766_amd.tsdf import integrate_batch
    dims, origin, tau, extent, maps, n, tiling = (41, 39, 35), (-20, -19, -17), 5120, 2.0, 1, 20000, None
    if case == "one_tile":
        extent, n = 0.35, 70000
    elif case == "small_tiles":
        dims, origin, tau, extent, tiling, n = (120, 117, 64), (-60, -58, -32), 10240, 5.0, (3, 3, 3), 6000
    elif case == "long_bands":
        tau, tiling, n = 32767, (3, 3, 3), 3000
    elif case == "several_maps":
        maps, n = 5, 7001
    elif case == "many_blocks":
        n = (1 << 20) + 1
    else:
        tau, n = 32767, 40000
    gms = [gpu_map(dims, origin, 0.1, tau, 64) for _ in range(maps)]
    oms = [oracle.OracleMap(dims, origin, 0.1, tau, 64) for _ in range(maps)]
    for k in range(2):
        items, ost = [], []
        for m in range(maps):
            if tiling:
                gms[m].set_tiling(tiling)
            x = synth.fuzz_scan((101, k, m), n - 1000 * m, extent_m=extent, nan_frac=0.02)
            p = synth.fuzz_pose((102, k, m), 0.3)
            items.append((gms[m], x, p))
            ost.append(oms[m].integrate(x, p))
        if maps == 1:
            assert gms[0].integrate(items[0][1], items[0][2], stats=True) == ost[0]
        else:
            assert integrate_batch(items, stats=True) == ost
    for g, o in zip(gms, oms):
        assert same(g, o, dims)
        g.close()
        o.close()


def test_one_binning_pass_where_memory_is_short():
    """A scan whose one-pass buffers (about 14 GB) do not fit the memory that
    is left, while those of two passes (about 9) do: the same map and counts as
    with all memory, and the size that failed is not tried again."""
    import torch
    from paper_2310_05766_amd.tsdf import TsdfMap
    spec, n = ((64, 60, 56), (-32, -30, -28), 0.1, 10240, 64), 65536 * 512
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    xyz = torch.randn(n, 3, generator=g, device="cuda")
    xyz *= (3.0 / xyz.norm(dim=1, keepdim=True)) * (0.8 + 0.4 * torch.rand(n, 1, generator=g, device="cuda"))
    torch.cuda.synchronize()

    def made():
        m = TsdfMap(*spec)
        m.set_tiling((3, 3, 3))
        m.set_blocks(512, 256)
        return m

    ref = made()
    want = [ref.integrate(xyz, synth.fuzz_pose((103, k), 0.3), stats=True) for k in range(3)]
    arrays = ref.readback_window()
    ref.close()
    gm = made()
    gm.integrate(xyz[:1000], np.eye(4))
    gm.close()  # (what the first use of a path loads is loaded)
    gm = made()
    torch.cuda.empty_cache()
    GB = 1 << 30
    held = []
    while torch.cuda.mem_get_info()[0] > 12.5 * GB:
        held.append(torch.empty(int(min(16 * GB, torch.cuda.mem_get_info()[0] - 12 * GB)), dtype=torch.uint8, device="cuda"))
    say("free", torch.cuda.mem_get_info()[0] / GB)
    got = [gm.integrate(xyz, synth.fuzz_pose((103, k), 0.3), stats=True) for k in range(2)]
    say("free", torch.cuda.mem_get_info()[0] / GB)
    del held
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    got.append(gm.integrate(xyz, synth.fuzz_pose((103, 2), 0.3), stats=True))
    assert free - torch.cuda.mem_get_info()[0] < GB
    assert got == want
    assert all(np.array_equal(a, b) for a, b in zip(gm.readback_window(), arrays))
    gm.close()


@pytest.mark.parametrize("dims", [(41, 39, 35), (64, 48, 40), (130, 9, 70)])
def test_one_binning_pass_on_caller_owned_memory(dims):
    """A map in the caller's arrays and in scratch of exactly the stated size:
    the tile lists lie in the scratch behind the tables for coarse tiles and in
    memory of their own for the finest, and the scratch is cut anew when tiles
    get finer. Automatic, fine and automatic tiling again, with and without
    counts, a batch of two scans between; nothing behind the scratch is
    written."""
    import torch
    from paper_2310_05766_amd.tsdf import TsdfMap, integrate_batch
    args = (dims, tuple(-(n // 2) for n in dims), 0.1, 3072, 64)
    nv, sb, guard = dims[0] * dims[1] * dims[2], TsdfMap.scratch_bytes(*args), 4096
    sdf, w = (torch.zeros(nv + guard, dtype=torch.int16, device="cuda") for _ in range(2))
    scratch = torch.full((sb + guard,), 0xA5, dtype=torch.uint8, device="cuda")
    sdf[nv:] = w[nv:] = 0x5A5A
    torch.cuda.synchronize()
    gm, om = TsdfMap(*args, arrays=(sdf[:nv], w[:nv], scratch[:sb])), oracle.OracleMap(*args)
    say("scratch of", sb, "bytes for", dims)
    k = 0
    for tiling in (None, (3, 3, 3), (2, 2, 5), None, (4, 4, 4)):
        gm.set_tiling(tiling or (0, 0, 0))
        for stats in (True, False, True):
            x, p = synth.fuzz_scan((104, k), 9000, extent_m=2.5, nan_frac=0.03), synth.fuzz_pose((105, k), 0.3)
            got, want = gm.integrate(x, p, stats=stats), om.integrate(x, p)
            assert got == (want if stats else None), (tiling, k)
            k += 1
        assert same(gm, om, dims), tiling
        x, p = synth.fuzz_scan((106, k), 5000, extent_m=2.5), synth.fuzz_pose((107, k), 0.3)
        assert integrate_batch([(gm, x, p), (gm, x[:3000], p)], stats=True) == [om.integrate(x, p), om.integrate(x[:3000], p)]
    assert same(gm, om, dims)
    torch.cuda.synchronize()
    assert bool((scratch[sb:] == 0xA5).all()) and bool((sdf[nv:] == 0x5A5A).all()) and bool((w[nv:] == 0x5A5A).all())
    gm.close()
    om.close()


def _rings(rings, cols, seed, missing=0.02):
    """An organised scan of a small room, in the sensor frame."""
    g = np.random.default_rng(seed)
    el = np.deg2rad(np.linspace(-22.5, 22.5, rings))[:, None]
    az = 2 * np.pi * np.arange(cols)[None] / cols
    d = np.stack([np.cos(el) * np.cos(az), np.cos(el) * np.sin(az), np.sin(el) * np.ones_like(az)], -1).reshape(-1, 3)
    half, pos = np.array([3.0, 2.4, 1.3]), np.array([0.4, -0.3, 0.1])
    with np.errstate(divide="ignore"):
        t = (np.where(d > 0, half - pos, half + pos) / np.abs(d)).min(1) + 0.01 * g.standard_normal(len(d))
    xyz = (d * t[:, None]).astype(np.float32)
    xyz[g.random(len(d)) < missing] = np.nan
    return xyz


@pytest.mark.parametrize("rings,cols", [(104, 554), (64, 1021), (128, 900), (128, 333), (40, 1800), (32, 1025), (64, 512), (33, 1024)])
def test_patches_of_rows_of_any_length(rings, cols):
    """Scans whose rows the binning finds (or not) take their points in patches:
    every point once. One scan, a batch of several scans of a map, one per map,
    interpolating and carving maps, and the allocation-free call, against the
    oracle; the same points shuffled, which have no rows."""
    import ctypes as C

    import torch
    from paper_2310_05766_amd import _abi
    from paper_2310_05766_amd.tsdf import integrate_batch
    spec = ((72, 64, 40), (-36, -32, -20), 0.1, 3072, 64)
    scans = [(_rings(rings, cols, (108, k)), synth.fuzz_pose((109, k), 0.2)) for k in range(3)]
    scans.append((np.random.default_rng(110).permutation(scans[0][0]), scans[0][1]))
    dev = [(torch.from_numpy(x).to("cuda"), p) for x, p in scans]
    gms, oms = [gpu_map(*spec) for _ in range(5)], [oracle.OracleMap(*spec) for _ in range(5)]
    for m in (gms[2], oms[2]):
        m.set_interpolation(45.0, 64)
    for m in (gms[3], oms[3]):
        m.set_carving(True)
    say(rings, "x", cols)
    for k in range(4):
        for m in (0, 2, 3):
            assert gms[m].integrate(*dev[k], stats=True) == oms[m].integrate(*scans[k]), (k, m)
        M, st = np.ascontiguousarray(scans[k][1], dtype=np.float64), _abi.ScanStats()
        torch.cuda.synchronize()
        assert _abi.lib().tsdf_integrate_scan_noalloc(gms[4].handle, dev[k][0].data_ptr(), dev[k][0].shape[0],
                                                      M.ctypes.data_as(C.POINTER(C.c_double)), C.byref(st)) == 0
        assert dict((f, getattr(st, f)) for f, _ in st._fields_) == oms[4].integrate(*scans[k]), k
    items = [(0, 0), (1, 1), (0, 2), (0, 3), (1, 0)]
    assert integrate_batch([(gms[m], *dev[k]) for m, k in items], stats=True) == [oms[m].integrate(*scans[k]) for m, k in items]
    items = [(0, 1), (1, 2)]
    assert integrate_batch([(gms[m], *dev[k]) for m, k in items], stats=True) == [oms[m].integrate(*scans[k]) for m, k in items]
    for g, o in zip(gms, oms):
        assert same(g, o, spec[0])
        g.close()
        o.close()
