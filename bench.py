#!/usr/bin/env python3
"""Benchmark of the TSDF integration path on one MI355X.

Workload: 50 OS1-128-shaped scans (128 rings x 1024 columns, seeded
synthetic outdoor scene, FP64 poses along a straight path) integrated into a
fixed 512 x 512 x 256 map at 6.4 cm with tau = 5 voxels and w_max = 64. One
step = the whole 50-scan sequence (transform, band traversal, min-tsdf,
merge) with the points already resident in HBM.

Prints ONE JSON line. Extra legs (all outside the timed region):
  * per-kernel durations from HIP events recorded on the map's stream, for
    the roofline of the dominant kernel;
  * synchronous per-scan latency (p50 / p99);
  * the ring-buffer shift of a 512 x 512 x 128 window (host-link bound);
  * 256 uneven scans into 16 maps: one launch, launches of 16, one call per
    scan;
  * vertical interpolation between scan lines on 10 of the same scans;
  * the serving loop on 48 sessions (real-time and compressed replays);
  * the CPU oracle on a bounded sample of the same workload.
"""
from __future__ import annotations

import argparse
import gc
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
METRIC = "voxel updates/s + scans/s (OS1-128 scan→512²×256 map); p99 scan latency"


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def sources_digest() -> str:
    h = hashlib.sha256()
    csrc = os.path.join(ROOT, "paper_2310_05766_amd", "csrc")
    for f in sorted(os.listdir(csrc)):
        with open(os.path.join(csrc, f), "rb") as fh:
            h.update(f.encode())
            h.update(fh.read())
    return h.hexdigest()[:16]


def read_traffic(kernel: str, workload_tag: str):
    """HBM bytes per launch from the committed rocprofv3 counter summary, or
    None when it is missing or was taken on other kernel sources."""
    path = os.path.join(ROOT, "profiles", f"traffic_{kernel}_{workload_tag}.txt")
    if not os.path.exists(path):
        return None
    kv = {}
    for line in open(path):
        if ":" in line and not line.startswith("#"):
            k, v = line.split(":", 1)
            kv[k.strip()] = v.strip()
    if kv.get("sources_sha256") != sources_digest():
        return None
    try:
        return float(kv["hbm_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


# VALU issue capacity: 256 CUs x 4 SIMDs, one wave64 instruction per SIMD
# every 4 cycles (16 lanes per cycle), at 2.4 GHz
VALU_WAVE_INSTS_PER_S = 256 * 4 * 2.4e9 / 4


def read_valu_insts(kernel: str, workload_tag: str):
    """SQ_INSTS_VALU per dispatch (wave instructions) from the committed
    rocprofv3 counter summary, or None when it is missing or was taken on
    other kernel sources."""
    path = os.path.join(ROOT, "profiles", f"sq_counters_{workload_tag}.txt")
    if not os.path.exists(path):
        return None
    lines = open(path).read().splitlines()
    if not any(line.strip() == f"kernel sources sha256[:16]: {sources_digest()}" for line in lines):
        return None
    head = next((line for line in lines if line.startswith("| kernel |")), None)
    row = next((line for line in lines if line.startswith(f"| `{kernel}` |")), None)
    if head is None or row is None:
        return None
    cols = [c.strip() for c in head.strip("|").split("|")]
    vals = [c.strip() for c in row.strip("|").split("|")]
    try:
        return float(vals[cols.index("SQ_INSTS_VALU")])
    except (ValueError, IndexError):
        return None


def cpu_baseline(workload, max_seconds: float):
    """The oracle, single-threaded and pinned to one host core, on the first
    scans of the same sequence: the first run takes scans until a third of
    max_seconds of integrate time is spent; that sample is run three times
    in all, each time on a fresh oracle map, and the median is reported."""
    import oracle

    spec = workload.maps[0]
    core = min(os.sched_getaffinity(0))
    saved = os.sched_getaffinity(0)
    os.sched_setaffinity(0, {core})
    try:
        runs, n_scans, upd, pts = [], None, 0, 0
        for rep in range(3):
            om = oracle.OracleMap.from_spec(spec)
            t_total, u, k, p = 0.0, 0, 0, 0
            for sc in workload.scans[:n_scans] if n_scans else workload.scans:
                t0 = time.perf_counter()
                st = om.integrate(sc.xyz, sc.pose)
                t_total += time.perf_counter() - t0
                u += st["voxels_updated"]
                p += st["points_in"]
                k += 1
                if n_scans is None and t_total >= max_seconds / 3:
                    break
            om.close()
            n_scans, upd, pts = k, u, p
            runs.append(t_total)
    finally:
        os.sched_setaffinity(0, saved)
    t_med = sorted(runs)[1]
    return {
        "value": upd / t_med,
        "unit": "voxel updates/s",
        "cores": 1,
        "kind": "oracle",
        "sample": f"first {n_scans} of the {len(workload.scans)} scans ({pts} points), integrate calls only, "
                  f"single-threaded C oracle pinned to host core {core}, median of 3 runs "
                  f"({', '.join(f'{t:.2f}' for t in runs)} s)",
        "scans_per_s": n_scans / t_med,
        "cpu": cpu_model(),
        "host_cores": len(saved),
    }


def _copy_device(torch, dst, src_ptr: int, nbytes: int):
    """Device-to-device copy from a raw address (the map's weight array)."""
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so.7")
    hip.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
    torch.cuda.synchronize()
    rc = hip.hipMemcpy(ctypes.c_void_p(dst.data_ptr()), ctypes.c_void_p(src_ptr), nbytes, 3)
    if rc != 0:
        raise RuntimeError(f"hipMemcpy failed ({rc})")


def bandwidth_leg(torch) -> dict:
    """Measured ceilings next to the nominal 8 TB/s: a device-to-device copy
    of 1 GiB (2 GiB of HBM traffic per copy), and pinned host <-> device
    copies of 256 MiB each way, best of 5, HIP events on torch's stream."""
    def best(fn, reps=5):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        fn()
        out = []
        for _ in range(reps):
            e0.record()
            fn()
            e1.record()
            e1.synchronize()
            out.append(e0.elapsed_time(e1) * 1e-3)
        return min(out)

    n = 1 << 30
    a = torch.empty(n, dtype=torch.uint8, device="cuda")
    b = torch.empty_like(a)
    a.fill_(1)
    t_copy = best(lambda: b.copy_(a))
    del a, b
    m = 256 << 20
    h = torch.empty(m, dtype=torch.uint8, pin_memory=True)
    d = torch.empty(m, dtype=torch.uint8, device="cuda")
    h.fill_(1)
    t_h2d = best(lambda: d.copy_(h, non_blocking=True))
    t_d2h = best(lambda: h.copy_(d, non_blocking=True))
    del h, d
    return {"device_copy_GBps": 2 * n / t_copy / 1e9, "device_copy_bytes": 2 * n,
            "pinned_h2d_GBps": m / t_h2d / 1e9, "pinned_d2h_GBps": m / t_d2h / 1e9, "pinned_bytes": m}


def cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def shift_leg(torch, TsdfMap, synth, bw=None):
    """One-chunk shifts of a 512 x 512 x 128 ring window at 5 cm, back and
    forth between two origins 64 voxels apart, with observed data in both
    end slabs: config-1 room scans spread along y at the window's left end,
    then (after one shift) at its right end. Every timed shift then sends the
    16 chunks of the slab that leaves out to the host store (1 MiB each,
    sdf + w) and loads the 16 of the slab that enters back from it."""
    import numpy as np

    dims = (512, 512, 128)
    vs = 0.05
    a_org = (-256, -256, -64)
    b_org = (-192, -256, -64)
    m = TsdfMap(dims, a_org, vs, 3072, 64)
    sc = synth.config1().scans[0]
    ys = [-11.0 + 22.0 * k / 7 for k in range(8)]

    def fill(x):
        for y in ys:
            pose = np.eye(4)
            pose[:3, 3] = [x, y, 0.0]
            m.integrate(sc.xyz, pose)

    fill(-11.2)  # the slab [-12.8, -9.6) m at the left end of the window at a_org
    m.shift(b_org)
    fill(14.4)   # the slab [12.8, 16.0) m at the right end of the window at b_org
    m.synchronize()
    times, moved_out, moved_in = [], 0, 0
    chunk_bytes = 64 ** 3 * 4
    loaded = None
    for k in range(6):
        new = a_org if k % 2 == 0 else b_org
        c0, _ = m.store_info()
        t0 = time.perf_counter()
        m.shift(new)
        times.append(time.perf_counter() - t0)
        c1, _ = m.store_info()
        # every shift brings back what the shift before it evicted (its
        # inverse); the store count moves by the evicted minus the loaded
        if loaded is None:
            loaded = 16  # the left slab, evicted by the set-up shift
        evicted = c1 - c0 + loaded
        moved_out += evicted * chunk_bytes
        moved_in += loaded * chunk_bytes
        loaded = evicted
    m.close()
    t = sum(times)
    out = {"window": list(dims), "shift_vox": 64, "shifts": len(times), "ms_per_shift": 1e3 * t / len(times),
           "bytes_out": moved_out, "bytes_in": moved_in, "host_link_GBps": (moved_out + moved_in) / t / 1e9}
    if bw:
        # the same bytes at the measured pinned rates, one direction after
        # the other (the shift overlaps the two directions, so this can pass 1)
        ideal = moved_out / (bw["pinned_d2h_GBps"] * 1e9) + moved_in / (bw["pinned_h2d_GBps"] * 1e9)
        out["frac_of_pinned"] = ideal / t
    return out


ATOMIC_BOUND = "scattered 64-bit atomicMin, probe_atomic_min_rate: 2048 waves x 64 lanes x 128 atomics"


def atomic_rates(torch, n_keys: int, stream) -> dict:
    """Scattered 64-bit atomicMin per second on a key volume of n_keys (the
    bound of the key-volume paths), and on an L2-resident 4 MiB."""
    from paper_2310_05766_amd.probe import atomic_probe
    keys = torch.empty(n_keys, dtype=torch.int64, device="cuda")
    out = {}
    for pattern, name in ((0, "window_key_volume"), (1, "l2_resident_4MiB")):
        atomic_probe(keys, 2048, 16, pattern, stream=stream)  # warm
        ms = min(atomic_probe(keys, 2048, 128, pattern, stream=stream) for _ in range(3))
        out[name] = 2048 * 64 * 128 / (ms * 1e-3)
    del keys
    return out


def interp_leg(torch, synth, TsdfMap, n_scans: int = 10, reps: int = 5):
    """Vertical interpolation between scan lines (45 deg over 128 lines, the
    OS1-128's) on the first scans of the config-2 sequence, one call per
    scan on the map's stream, timed with HIP events on that stream."""
    w = synth.config2(n_scans)
    spec = w.maps[0]
    dev = [torch.from_numpy(sc.xyz).to("cuda") for sc in w.scans]
    st = torch.cuda.Stream()
    m = TsdfMap.from_spec(spec, stream=st)
    dq = m.set_interpolation(45.0, 128)
    stats = [m.integrate(x, sc.pose, stats=True) for x, sc in zip(dev, w.scans)]
    upd = sum(x["voxels_updated"] for x in stats)
    visits = sum(x["visits"] for x in stats)
    pts = sum(x["points_in"] for x in stats)
    for x, sc in zip(dev, w.scans):  # warm
        m.integrate(x, sc.pose)
    m.key_atomics()  # restart the count of issued atomics
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    st.synchronize()
    e0.record(st)
    t0 = time.perf_counter()
    for _ in range(reps):
        for x, sc in zip(dev, w.scans):
            m.integrate(x, sc.pose)
    e1.record(st)
    st.synchronize()
    wall = time.perf_counter() - t0
    gpu_s = e0.elapsed_time(e1) * 1e-3
    atomics = m.key_atomics()
    m.close()
    n = reps * n_scans
    B = 12.0 * pts + 128.0 * n_scans + 8.0 * upd  # per pass over the scans
    probe = atomic_rates(torch, spec.n_voxels, st)
    vps = visits * reps / gpu_s
    aps = atomics / gpu_s
    return {"scans": n_scans, "delta_z_q20": dq, "visits_per_scan": visits / n_scans,
            "voxel_updates_per_scan": upd / n_scans, "scans_per_s": n / wall,
            "voxel_updates_per_s": upd * reps / wall, "visits_per_s": vps, "gpu_ms_per_scan": 1e3 * gpu_s / n,
            "algorithmic_GBps": B * reps / gpu_s / 1e9, "hbm_frac": B * reps / gpu_s / 1e9 / HBM_PEAK_GBS,
            "atomic_roofline": {"bound": ATOMIC_BOUND, "probe_atomics_per_s": probe,
                                "issued_atomics_per_s": aps, "visits_per_s": vps,
                                "frac": aps / probe["window_key_volume"],
                                "note": "issued atomics counted on the device (a block merges its candidates before it issues any; 32-bit where keys fit)"}}


def carve_leg(torch, synth, TsdfMap, n_scans: int = 50, reps: int = 3):
    """Free-space carving on the config-2 sequence (every ray also walked
    from the sensor to its band; sensors outside the window for the first
    and last scans), one call per scan on the map's stream, timed with HIP
    events on that stream."""
    w = synth.config2(n_scans)
    spec = w.maps[0]
    dev = [torch.from_numpy(sc.xyz).to("cuda") for sc in w.scans]
    st = torch.cuda.Stream()
    m = TsdfMap.from_spec(spec, stream=st)
    m.set_carving(True)
    stats = [m.integrate(x, sc.pose, stats=True) for x, sc in zip(dev, w.scans)]
    upd = sum(x["voxels_updated"] for x in stats)
    visits = sum(x["visits"] for x in stats)
    pts = sum(x["points_in"] for x in stats)
    m.key_atomics()  # restart the count of issued atomics
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    st.synchronize()
    e0.record(st)
    t0 = time.perf_counter()
    for _ in range(reps):
        for x, sc in zip(dev, w.scans):
            m.integrate(x, sc.pose)
    e1.record(st)
    st.synchronize()
    wall = time.perf_counter() - t0
    gpu_s = e0.elapsed_time(e1) * 1e-3
    atomics = m.key_atomics()
    m.close()
    n = reps * n_scans
    B = 12.0 * pts + 128.0 * n_scans + 8.0 * upd  # per pass over the scans
    probe = atomic_rates(torch, spec.n_voxels, st)
    vps = visits * reps / gpu_s
    aps = atomics / gpu_s
    return {"scans": n_scans, "visits_per_scan": visits / n_scans, "voxel_updates_per_scan": upd / n_scans,
            "scans_per_s": n / wall, "voxel_updates_per_s": upd * reps / wall, "visits_per_s": vps,
            "gpu_ms_per_scan": 1e3 * gpu_s / n, "algorithmic_GBps": B * reps / gpu_s / 1e9,
            "hbm_frac": B * reps / gpu_s / 1e9 / HBM_PEAK_GBS,
            "atomics_per_scan": atomics / n,
            "atomic_roofline": {"bound": ATOMIC_BOUND, "probe_atomics_per_s": probe,
                                "issued_atomics_per_s": aps, "visits_per_s": vps,
                                "frac": aps / probe["window_key_volume"],
                                "note": "issued atomics counted on the device; free-space visits mark voxels "
                                        "without one, and a block merges its band's candidates"}}


def uneven_batch_leg(torch, synth, reps: int = 3):
    """Config 4: 256 scans of uneven shapes (16x512 .. 128x2048) into 16 maps
    of 256^3 at 8 cm, scan i into map i mod 16. Three forms on the same
    resident points, each rep starting from fresh maps: one launch for all
    256 scans (16 per map, in order), 16 launches of one scan per map, and
    one tsdf_integrate_scan per scan. The autotuner picks the batch tiling
    on the first 16 scans."""
    from paper_2310_05766_amd.autotune import autotune
    from paper_2310_05766_amd.tsdf import TsdfMap, integrate_batch

    shapes = synth.config4_shapes()
    scans = [synth.config4_scan(i, shapes[i]) for i in range(256)]
    spec = synth.MapSpec((256, 256, 256), (-128, -128, -128), 0.08, 5120, 64)
    dev = [torch.from_numpy(sc.xyz).to("cuda") for sc in scans]
    poses = [sc.pose for sc in scans]
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    best = autotune(spec, list(zip(dev[:16], poses[:16])), mode="batch", reps=2, use_cache=False)
    lt = tuple(best["lt"])

    def fresh(tiling):
        ms = [TsdfMap.from_spec(spec, stream=st) for _ in range(16)]
        if tiling:
            for m in ms:
                m.set_tiling(tiling, best["workgroups"])
                m.set_blocks(best["bin_block"], best["tile_block"])
        return ms

    def timed(form, tiling):
        out = []
        for _ in range(reps):
            ms = fresh(tiling)
            items = [(ms[i % 16], dev[i], poses[i]) for i in range(256)]
            st.synchronize()
            t0 = time.perf_counter()
            if form == "all":
                integrate_batch(items, stream=st)
            elif form == "per16":
                for b in range(0, 256, 16):
                    integrate_batch(items[b:b + 16], stream=st)
            else:
                for m, x, p in items:
                    m.integrate(x, p)
            st.synchronize()
            out.append(time.perf_counter() - t0)
            for m in ms:
                m.close()
        return min(out)

    ms = fresh(lt)
    stats = integrate_batch([(ms[i % 16], dev[i], poses[i]) for i in range(256)], stream=st, stats=True)
    st.synchronize()
    for m in ms:
        m.close()
    upd = sum(x["voxels_updated"] for x in stats)
    timed("all", lt)  # warm every engine and graph shape once
    timed("per16", lt)
    timed("plain", None)
    t_all, t_16, t_plain = timed("all", lt), timed("per16", lt), timed("plain", None)
    return {"scans": 256, "points": int(sum(d.shape[0] for d in dev)), "voxel_updates": upd,
            "autotuned": {"lt": list(lt), "workgroups": best["workgroups"], "bin_block": best["bin_block"],
                          "tile_block": best["tile_block"]},
            "one_launch": {"scans_per_s": 256 / t_all, "voxel_updates_per_s": upd / t_all, "ms": 1e3 * t_all},
            "launch_per_16": {"scans_per_s": 256 / t_16, "voxel_updates_per_s": upd / t_16, "ms": 1e3 * t_16},
            "plain": {"scans_per_s": 256 / t_plain, "voxel_updates_per_s": upd / t_plain, "ms": 1e3 * t_plain}}


def _session_scans(args):
    """All scans of one config-5 session as stacked arrays (a worker job)."""
    import numpy as np

    import synth
    sid, n_sessions, duration = args
    sess = synth.config5(n_sessions=n_sessions, duration_s=duration)[sid]
    n = len(sess.arrivals)
    xyz = np.empty((n, 16 * 1024, 3), np.float32)
    poses = np.empty((n, 4, 4), np.float64)
    for k in range(n):
        sc = sess.scan(k)
        xyz[k] = sc.xyz
        poses[k] = sc.pose
    return sid, xyz, poses


def _digest_window(m, spec) -> str:
    import numpy as np
    o = spec.origin
    sdf, w = m.readback(o, tuple(o[a] + spec.dims[a] for a in range(3)))
    h = hashlib.sha256()
    h.update(np.ascontiguousarray(sdf).tobytes())
    h.update(np.ascontiguousarray(w).tobytes())
    return h.hexdigest()


def serving_leg(torch, synth, seconds: float, speedup: float, workers: int = 15):
    """Config-5 serving: 48 sessions (maps 256^3 / 384^3 / 512x512x256 at
    6.4 cm), 16x1024 scans arriving Poisson at 10 Hz per session for 60 s,
    every scan distinct (about 28,800, generated ahead by worker processes).
    A real-time replay of the first `seconds` of arrivals gives p50/p99
    latency. The whole trace compressed `speedup` times gives the peak served
    rate; its 48 final maps are then read back and compared with the
    oracle's digests (tests/golden/oracle_digests.json). The same scans
    integrated one call per scan, in arrival order, give the plain rate."""
    import multiprocessing as mp

    from paper_2310_05766_amd.serve import GpuExecutor, Server, latency_summary, replay
    from paper_2310_05766_amd.tsdf import TsdfMap

    duration = 60.0
    sessions = synth.config5(n_sessions=48, duration_s=duration)
    t0 = time.perf_counter()
    nw = max(1, min(workers, len(os.sched_getaffinity(0)) - 1))
    with mp.get_context("spawn").Pool(nw) as pool:
        data = {sid: (x, p) for sid, x, p in pool.imap_unordered(_session_scans,
                                                               [(s.sid, 48, duration) for s in sessions])}
    t_gen = time.perf_counter() - t0

    def scans_of(sid, k):
        x, p = data[sid]
        return x[k], p[k]

    n_scans = sum(len(s.arrivals) for s in sessions)
    out = {"sessions": len(sessions), "scans": n_scans, "trace_s": duration,
           "offered_scans_per_s": n_scans / duration, "scan_generation_s": t_gen}
    # real time: the first `seconds` of arrivals
    trace = [(s.sid, s.spec, s.arrivals[s.arrivals < seconds]) for s in sessions]
    trace = [t for t in trace if len(t[2])]
    ex = GpuExecutor(lanes=2)
    srv = Server(ex, budget_bytes=200 * 10 ** 9, lanes=2, max_batch=64)
    t0 = time.perf_counter()
    recs = replay(srv, trace, scans_of, speedup=1.0)
    wall = time.perf_counter() - t0
    ex.close()
    out["realtime"] = dict(latency_summary(recs), speedup=1.0, replayed_s=seconds, wall_s=wall,
                           scans_per_s=len(recs) / wall, batches=srv.batches)
    # the whole trace, compressed; maps kept for the check
    golden = None
    gpath = os.path.join(ROOT, "tests", "golden", "oracle_digests.json")
    if os.path.exists(gpath):
        golden = json.load(open(gpath)).get("config5")
    ex = GpuExecutor(lanes=2)
    srv = Server(ex, budget_bytes=200 * 10 ** 9, lanes=2, max_batch=64)
    trace = [(s.sid, s.spec, s.arrivals) for s in sessions]
    t0 = time.perf_counter()
    recs = replay(srv, trace, scans_of, speedup=speedup, close_at_end=False)
    wall = time.perf_counter() - t0
    for st in ex.streams:
        st.synchronize()
    exact = 0
    for s in sessions:
        m = srv.sessions[s.sid].map
        dig = _digest_window(m, s.spec)
        exact += int(golden is not None and golden.get(str(s.sid), {}).get("window_sha256") == dig)
        srv.close_session(s.sid)
    ex.close()
    out["compressed"] = dict(latency_summary(recs), speedup=speedup, wall_s=wall, scans_per_s=len(recs) / wall,
                             batches=srv.batches, maps_bit_exact_with_oracle=exact,
                             checked_against="tests/golden/oracle_digests.json" if golden else None)
    # plain: one call per scan, arrival order, one stream, maps resident
    st = torch.cuda.Stream()
    maps = {s.sid: TsdfMap.from_spec(s.spec, stream=st) for s in sessions}
    events = sorted((t, s.sid, k) for s in sessions for k, t in enumerate(s.arrivals))
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _, sid, k in events:
        x, p = scans_of(sid, k)
        maps[sid].integrate(x, p)
    st.synchronize()
    wall = time.perf_counter() - t0
    for m in maps.values():
        m.close()
    out["plain_scans_per_s"] = len(events) / wall
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--scans", type=int, default=50)
    ap.add_argument("--cpu-seconds", type=float, default=15.0, help="budget of the oracle baseline leg")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-shift", action="store_true")
    ap.add_argument("--no-serving", action="store_true")
    ap.add_argument("--no-uneven", action="store_true", help="skip the 256 uneven scans leg")
    ap.add_argument("--no-interp", action="store_true", help="skip the vertical interpolation leg")
    ap.add_argument("--interp-only", action="store_true",
                    help="with --profile-only: the interpolating path on 10 config-2 scans only")
    ap.add_argument("--no-carve", action="store_true", help="skip the free-space carving leg")
    ap.add_argument("--carve-only", action="store_true",
                    help="with --profile-only: the carving path on the config-2 sequence only")
    ap.add_argument("--serving-seconds", type=float, default=10.0, help="real-time replay length (seconds)")
    ap.add_argument("--blocks", type=str, default="",
                    help="binning block and tile workgroup sizes for the main map, e.g. 512,256 (default: the "
                         "library's)")
    ap.add_argument("--tiling", type=str, default="",
                    help="log2 tile edges for the main map, e.g. 3,3,3 (default: the library's)")
    ap.add_argument("--prewarm-seconds", type=float, default=2.0,
                    help="untimed batched steps before any timed leg (the device clocks up)")
    ap.add_argument("--profile-only", action="store_true", help="warmup + timed steps only (for rocprofv3)")
    ap.add_argument("--plain-only", action="store_true", help="with --profile-only: per-scan calls only")
    ap.add_argument("--batched-only", action="store_true", help="with --profile-only: batched steps only")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only a plain 256 MiB device copy, three times (calibrates HBM byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py: measures one GPU only; --gpus {args.gpus} is not supported "
              "(every workload fits one MI355X; maps and sessions would shard whole across GPUs)", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    # Python's cyclic garbage collector stays paused for the whole run, as
    # timeit pauses it: with torch and the synthetic scans loaded, a full
    # collection takes tens of milliseconds, longer than a whole timed window
    # of batched steps, and would land in one now and then. Reference
    # counting still frees everything the run drops.
    gc.collect()
    gc.disable()

    if args.copy_calibration:
        n = 256 * 1024 * 1024
        a = torch.ones(n // 4, dtype=torch.float32, device="cuda")
        b = torch.empty_like(a)
        torch.cuda.synchronize()
        for _ in range(3):
            b.copy_(a)
        torch.cuda.synchronize()
        log(f"copied {n} bytes three times")
        return

    import synth
    from paper_2310_05766_amd.tsdf import TsdfMap, integrate_batch

    torch.cuda.set_device(0)
    if args.profile_only and args.interp_only:
        log(f"profile-only: interpolation {interp_leg(torch, synth, TsdfMap, reps=max(1, args.steps // 4))}")
        return
    if args.profile_only and args.carve_only:
        log(f"profile-only: carving {carve_leg(torch, synth, TsdfMap, reps=max(1, args.steps // 10))}")
        return
    log("generating config-2 scans")
    w = synth.config2(args.scans)
    spec = w.maps[0]
    dev = [torch.from_numpy(s.xyz).to("cuda") for s in w.scans]
    poses = [s.pose for s in w.scans]
    torch.cuda.synchronize()
    # a stream of our own (default priority): the map, its batches and the
    # timing events all live on it
    stream = torch.cuda.Stream()
    gm = TsdfMap.from_spec(spec, stream=stream)
    if args.blocks:
        gm.set_blocks(*[int(v) for v in args.blocks.split(",")])
    if args.tiling:
        gm.set_tiling(tuple(int(v) for v in args.tiling.split(",")))

    batch_items = [(gm, x, p) for x, p in zip(dev, poses)]

    def step_plain():
        for x, p in zip(dev, poses):
            gm.integrate(x, p)

    def step_batched():
        integrate_batch(batch_items, stream=stream)

    def timed(step):
        for _ in range(args.warmup):
            step()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            step()
        torch.cuda.synchronize()
        return time.perf_counter() - t0

    if args.profile_only:
        # the launches a profiler should see, and nothing else: warmup and
        # timed steps of the chosen form on the fresh map
        parts = []
        if not args.batched_only:
            parts.append(("plain", timed(step_plain)))
        if not args.plain_only:
            parts.append(("batched", timed(step_batched)))
        log("profile-only: " + ", ".join(f"{k} {v * 1e3 / args.steps:.3f} ms/step" for k, v in parts))
        gm.close()
        return

    # per-scan counts (state independent): U, visits, valid points; on the
    # fresh map, the voxels any scan touches (the union) are those with w > 0
    stats = [gm.integrate(x, p, stats=True) for x, p in zip(dev, poses)]
    U_step = sum(s["voxels_updated"] for s in stats)
    N_step = sum(s["points_in"] for s in stats)
    visits_step = sum(s["visits"] for s in stats)
    _sdf_ptr, w_ptr, _st = gm.device_arrays()
    w_view = torch.empty(spec.n_voxels, dtype=torch.int16, device="cuda")
    _copy_device(torch, w_view, w_ptr, spec.n_voxels * 2)
    U_union = int((w_view > 0).sum().item())
    del w_view
    n_scans = len(dev)

    # the device needs a moment of work to clock up from idle: untimed
    # batched steps before anything is timed
    log("device pre-warm")
    t_end = time.perf_counter() + args.prewarm_seconds
    while time.perf_counter() < t_end:
        step_batched()
        torch.cuda.synchronize()
    log("batched steps")
    dt = timed(step_batched)
    # (the result is the window above; four more show what a stall of the host would do to it)
    dt_again = [timed(step_batched) for _ in range(4)]
    log("plain per-scan steps")
    dt_plain = timed(step_plain)

    def stage_times(step, reps):
        gm.profile(True)
        for _ in range(reps):
            step()
        out = {}
        for k in ("k_bin", "k_tile"):
            ms, n = gm.profile_read(k)
            if n:
                out[k] = {"total_ms": ms, "launches": n, "avg_us": 1e3 * ms / n}
        gm.profile(False)
        return out

    log("kernel timing")
    kt_plain = stage_times(step_plain, max(3, args.steps // 4))
    # batched launches: stage events of the stream's batch engine
    from paper_2310_05766_amd.tsdf import batch_profile, batch_profile_read
    # (the same K steps again, launched directly: stage events sit between
    # kernels, so these launches are not graph replays)
    batch_profile(stream, True)
    for _ in range(args.steps):
        step_batched()
    kt = {}
    for name, stage in (("bin", "bin"), ("k_tile", "tile"), ("stats", "stats"), ("launch", "launch")):
        ms, n = batch_profile_read(stream, stage)
        kt[name] = {"total_ms": ms, "launches": n, "avg_us": 1e3 * ms / max(n, 1)}
    batch_profile(stream, False)

    # algorithmic bytes per scan: 12 per point (no-return slots included),
    # 128 per pose, 8 per voxel update (int16 sdf + int16 w, read once and
    # written once); per launch, summed over the batch's scans
    B_scans = 12.0 * N_step + 128.0 * n_scans + 8.0 * U_step
    # the same with each voxel counted once per batch (what one pass over
    # the batch must move at least): a secondary figure
    B_distinct = 12.0 * N_step + 128.0 * n_scans + 8.0 * U_union
    achieved = B_scans / (kt["k_tile"]["avg_us"] * 1e-6) / 1e9
    traffic = read_traffic("k_tile", "config2_batch")
    step_traffic = read_traffic("step", "config2_batch")
    log("bandwidth ceilings")
    bw = bandwidth_leg(torch)

    # synchronous per-scan latency (plain path)
    log("latency")
    lat = []
    for _ in range(3):
        for x, p in zip(dev, poses):
            t1 = time.perf_counter()
            gm.integrate(x, p)
            gm.synchronize()
            lat.append(time.perf_counter() - t1)
    lat_ms = np.array(lat) * 1e3
    # surface extraction of the whole window after the sequence (inspection)
    lo = spec.origin
    hi = tuple(spec.origin[a] + spec.dims[a] for a in range(3))
    gm.synchronize()
    t0 = time.perf_counter()
    tris = gm.mesh(lo, hi)
    t_mesh = time.perf_counter() - t0
    mesh = {"box": [list(lo), list(hi)], "triangles": int(tris.shape[0]), "ms": 1e3 * t_mesh,
            "cubes_per_s": float(np.prod([spec.dims[a] - 1 for a in range(3)])) / t_mesh,
            "includes": "count pass, host scan, emit pass, device-to-host copy of the triangles"}
    del tris
    # point-to-TSDF registration of one scan of the sequence against the map
    # (from 5 cm and 1.1 deg off)
    import math
    k_reg = n_scans // 2
    P0 = poses[k_reg].copy()
    P0[0, 3] += 0.04
    P0[1, 3] -= 0.03
    c, s_ = math.cos(0.02), math.sin(0.02)
    P0[:3, :3] = np.array([[c, -s_, 0], [s_, c, 0], [0, 0, 1]]) @ P0[:3, :3]
    gm.register(dev[k_reg], P0, 2)  # warm
    iters = 10
    t0 = time.perf_counter()
    P, info = gm.register(dev[k_reg], P0, iters, 1e-6)
    t_reg = time.perf_counter() - t0
    registration = {"scan": k_reg, "points": int(dev[k_reg].shape[0]), "points_used": info["points"],
                    "steps": info["steps"], "ms_per_step": 1e3 * t_reg / max(info["steps"] + 1, 1),
                    "points_per_s": dev[k_reg].shape[0] * (info["steps"] + 1) / t_reg,
                    "translation_error_m": float(np.linalg.norm(P[:3, 3] - poses[k_reg][:3, 3])),
                    "includes": "normal-equation kernel with the 6x6 solve in its last block, per step, plus the "
                                "final evaluation"}
    gm.close()

    shift = None if args.no_shift else shift_leg(torch, TsdfMap, synth, bw)
    interp = None
    if not args.no_interp:
        log("vertical interpolation")
        interp = interp_leg(torch, synth, TsdfMap)
    carve = None
    if not args.no_carve:
        log("free-space carving")
        carve = carve_leg(torch, synth, TsdfMap)
    uneven = None
    if not args.no_uneven:
        log("uneven batches (config 4)")
        uneven = uneven_batch_leg(torch, synth)
    serving = None
    if not args.no_serving:
        log("serving (config 5)")
        serving = serving_leg(torch, synth, args.serving_seconds, speedup=1000.0)
    cpu = None
    if not args.no_cpu_baseline:
        log("cpu baseline (oracle)")
        cpu = cpu_baseline(w, args.cpu_seconds)

    value = U_step * args.steps / dt
    valu_insts = read_valu_insts("k_tile", "config2_batch")
    valu_issue = None
    if valu_insts is not None:
        t_tile = kt["k_tile"]["avg_us"] * 1e-6
        valu_issue = {"wave_insts_per_launch": valu_insts, "peak_wave_insts_per_s": VALU_WAVE_INSTS_PER_S,
                      "busy_frac": valu_insts / t_tile / VALU_WAVE_INSTS_PER_S}
    line = {
        "metric": METRIC,
        "value": value,
        "unit": "voxel updates/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": dt * 1e3 / args.steps,
        "ms_per_step_again": [t * 1e3 / args.steps for t in dt_again],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {
            "workload": f"{n_scans} OS1-128-shaped scans (128x1024, seeded outdoor scene, FP64 poses) -> "
                        "fixed 512x512x256 map at 6.4 cm, tau 5 voxels, w_max 64; one step = the whole sequence, "
                        "integrated as one ordered batch",
            "scans_per_step": n_scans,
            "points_per_step": N_step,
            "voxel_updates_per_step": U_step,
            "distinct_voxels_per_step": U_union,
            "visits_per_step": visits_step,
            "storage": "int16 sdf + int16 weight per voxel",
        },
        "scans_per_s": n_scans * args.steps / dt,
        "latency_ms": {"p50": float(np.percentile(lat_ms, 50)), "p99": float(np.percentile(lat_ms, 99)),
                       "max": float(lat_ms.max()), "mode": "synchronous per-scan call"},
        "plain": {
            "value": U_step * args.steps / dt_plain,
            "scans_per_s": n_scans * args.steps / dt_plain,
            "ms_per_step": dt_plain * 1e3 / args.steps,
            "kernels": kt_plain,
        },
        "kernels": kt,
        "roofline": {
            "bound": "hbm",
            "kernel": "k_tile",
            "achieved": achieved,
            "peak": HBM_PEAK_GBS,
            "unit": "GB/s",
            "frac": achieved / HBM_PEAK_GBS,
            "traffic": traffic,
            "algorithmic_bytes_per_launch": B_scans,
            "bytes_per_unit": "12 per point + 128 per pose + 8 per voxel update, summed over the launch's scans",
            "kernel_avg_us": kt["k_tile"]["avg_us"],
            "frac_of_device_copy": achieved / bw["device_copy_GBps"],
            "distinct_voxel_bytes_per_launch": B_distinct,
            # what does bound it: VALU issue (committed SQ counters of the
            # same kernel sources, over the live launch time)
            "valu_issue": valu_issue,
        },
        "step_roofline": {
            "algorithmic_bytes": B_scans,
            "kernel_time_us": kt["launch"]["avg_us"],
            "frac_kernel_time": B_scans / (kt["launch"]["avg_us"] * 1e-6) / 1e9 / HBM_PEAK_GBS,
            "wall_ms": dt * 1e3 / args.steps,
            "frac_wall": B_scans / (dt / args.steps) / 1e9 / HBM_PEAK_GBS,
            "traffic": step_traffic,
        },
        "bandwidth": bw,
        "shift": shift,
        "mesh": mesh,
        "registration": registration,
        "carving": carve,
        "uneven_batches": uneven,
        "interpolation": interp,
        "serving": serving,
        "cpu_baseline": cpu,
        "sources_sha256": sources_digest(),
    }
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
