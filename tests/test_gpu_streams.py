"""Device points written on torch's stream just before a call: the library's
stream must wait for them (a torch event, skipped only when torch's stream
has nothing left to do). The points are produced after a long device-side
delay on torch's current stream, so a call that did not wait would read
memory that is not written yet; the result must equal the same scan given
as host points."""
import sys

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _late_points(torch, xyz):
    """A device copy of xyz that torch's current stream writes only after
    about 20 ms of spinning (torch.cuda._sleep)."""
    src = torch.from_numpy(np.ascontiguousarray(xyz, dtype=np.float32)).to("cuda")
    torch.cuda.synchronize()
    torch.cuda._sleep(50_000_000)
    out = torch.empty_like(src)
    out.copy_(src)  # queued behind the spin on the same stream
    return out


def _host_reference(spec, scans):
    from paper_2310_05766_amd.tsdf import TsdfMap

    m = TsdfMap.from_spec(spec)
    for sc in scans:
        m.integrate(sc.xyz, sc.pose)
    sdf, w = m.readback_window()
    m.close()
    return sdf, w


def test_plain_call_waits_for_points_written_on_torch_stream():
    torch = pytest.importorskip("torch")
    from paper_2310_05766_amd.tsdf import TsdfMap

    w = synth.config1()
    spec, sc = w.maps[0], w.scans[0]
    say("plain call, late points", spec.dims)
    want_sdf, want_w = _host_reference(spec, [sc])
    m = TsdfMap.from_spec(spec)  # the library's own stream, not torch's
    x = _late_points(torch, sc.xyz)
    assert not torch.cuda.current_stream().query()  # still spinning: the call must order itself
    m.integrate(x, sc.pose)
    del x  # the map keeps the points alive until its stream has read them
    sdf, ww = m.readback_window()
    m.close()
    assert (ww > 0).sum() > 10000
    assert np.array_equal(sdf, want_sdf) and np.array_equal(ww, want_w)


def test_batch_waits_for_points_written_on_torch_stream():
    torch = pytest.importorskip("torch")
    from paper_2310_05766_amd.tsdf import TsdfMap, integrate_batch

    w = synth.config1()
    spec = w.maps[0]
    base = w.scans[0]
    # the same points from three poses: the batch merges them in order
    scans = [base] + [synth.Scan(xyz=base.xyz, pose=synth.fuzz_pose(s, max_t=0.2), rings=base.rings, cols=base.cols)
                      for s in (3, 4)]
    say("batch, late points", len(scans))
    want_sdf, want_w = _host_reference(spec, scans)
    st = torch.cuda.Stream()
    m = TsdfMap.from_spec(spec, stream=st)
    xs = [_late_points(torch, s.xyz) for s in scans]
    assert not torch.cuda.current_stream().query()
    integrate_batch([(m, x, s.pose) for x, s in zip(xs, scans)], stream=st)
    del xs  # recorded on the batch's stream: kept until it has read them
    sdf, ww = m.readback_window()
    m.close()
    assert (ww > 0).sum() > 10000
    assert np.array_equal(sdf, want_sdf) and np.array_equal(ww, want_w)


@pytest.mark.parametrize("option", ["none", "interpolation", "carving"])
@pytest.mark.parametrize("calls", [1, 2, 3])
def test_calls_in_a_captured_graph_replay(calls, option):
    """One-scan calls of device points, captured by the caller once the map has
    its memory, give at every replay what eager calls give: replays follow one
    another and other calls (a scan, a batch of two) come between."""
    torch = pytest.importorskip("torch")
    import oracle
    from paper_2310_05766_amd.tsdf import TsdfMap, integrate_batch

    spec = ((48, 40, 32), (-24, -20, -16), 0.1, 3072, 64)
    st = torch.cuda.Stream()
    gm, om = TsdfMap(*spec, stream=st), oracle.OracleMap(*spec)
    for m in (gm, om):
        if option == "interpolation":
            m.set_interpolation(30.0, 16)
        elif option == "carving":
            m.set_carving(True)
    scans = [(synth.fuzz_scan((71, k), 3000, extent_m=1.6, nan_frac=0.05), synth.fuzz_pose((72, k), 0.4)) for k in range(5)]
    dev = [torch.from_numpy(x).to("cuda") for x, _ in scans]
    torch.cuda.synchronize()

    def eager(k):
        with torch.cuda.stream(st):
            gm.integrate(dev[k], scans[k][1])
        om.integrate(*scans[k])

    def same():
        lo, hi = spec[1], tuple(spec[1][a] + spec[0][a] for a in range(3))
        return all(np.array_equal(a, b) for a, b in zip(gm.readback(lo, hi), om.readback(lo, hi)))

    for k in range(len(scans)):
        eager(k)
    torch.cuda.synchronize()
    say("capture of", calls, "calls,", option)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        for k in range(calls):
            gm.integrate(dev[k], scans[k][1])
    for step in range(6):
        for _ in range(1 + step % 3):
            with torch.cuda.stream(st):
                graph.replay()
            for k in range(calls):
                om.integrate(*scans[k])
        if step % 2:
            eager(step % len(scans))
        if step == 3:
            integrate_batch([(gm, dev[k], scans[k][1]) for k in (3, 4)], stream=st)
            for k in (3, 4):
                om.integrate(*scans[k])
        torch.cuda.synchronize()
        assert same(), step
    gm.close()
    om.close()
