"""GPU parity at the sizes where a kernel or a dispatch rule changes its path:
block and room edges, remainders, smallest launches. Bars as in the other GPU
tests: 1e-5 of the largest value for renders, 1e-4 for gradients, against the
FP64 oracle."""
import ctypes
import threading

import numpy as np
import pytest
import torch

from gpu_util import announce, oracle_render, rel_err, stop_ambiguous, tdev, tiny_camera, upload
from oracle import core as OC
from paper_2202_06088_amd import _lib, ops
from workloads import make_scene, make_scene_per_point, scene_for_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tiny():
    """The tiny workload's view, an upstream gradient (zero where the stop test is within rounding) and its oracle."""
    sc = scene_for_workload("tiny")
    cam = tiny_camera(sc)
    o, d = OC.pinhole_rays(64, 64, cam.intr(), cam.c2w)
    g = np.random.default_rng(61).normal(size=(o.shape[0], 3)).astype(np.float32)
    g[stop_ambiguous(oracle_render(sc, o, d, None, 4.0, 1e-4, g_rgb=g), label="tiny")] = 0.0
    return sc, o, d, g, oracle_render(sc, o, d, None, 4.0, 1e-4, g_rgb=g)


@pytest.mark.parametrize("records", [None, "1", "130", "4100"])
@pytest.mark.parametrize("cap", [1, 127, 128, 129, 2000, 20_000])
def test_room_edges(tiny, cap, records, monkeypatch):
    """Traces and records that end inside, at and just after a block of the room: samples without room are walked
    or scattered, and the gradients are the same."""
    sc, o, d, g, ref = tiny
    if records is None:
        monkeypatch.delenv("NEUVV_BWD_RECORDS", raising=False)
    else:
        monkeypatch.setenv("NEUVV_BWD_RECORDS", records)
    tree, oo, dd = upload(sc), tdev(o), tdev(d)
    trace = ops.Trace(o.shape[0], cap, oo.device)
    rgb, alpha, _, nsamp = ops.render(tree, oo, dd, 4.0, None, 1e-4, 64, trace=trace)
    gl, gb = ops.render_backward(tree, oo, dd, rgb, alpha, nsamp, tdev(g), None, 4.0, None, 1e-4, 64, trace=trace)
    torch.cuda.synchronize()
    hh, ws = tree.unpack_grad(gl)
    e = [rel_err(hh.cpu().numpy(), ref["grad_hh"]), rel_err(ws.cpu().numpy(), ref["grad_wsig"]),
         rel_err(gb.cpu().numpy(), ref["grad_basis"])]
    announce(f"cap={cap} records={records}: grad rel errors {e}")
    assert max(e) <= 1e-4, e


@pytest.mark.parametrize("width,height", [(1, 1), (1, 70), (257, 1), (1237, 31), (64, 64)])
def test_pinhole_edges(width, height):
    """Camera rays equal the oracle's bit for bit (both round one float64 value), whole images and pixel lists."""
    c = np.random.default_rng(width).normal(size=(3, 4)).astype(np.float32)
    intr = np.array([1.3 * width, 0.9 * width, 0.4 * width, 0.55 * height], np.float32)
    cam = _lib.make_camera(width, height, *intr, c)
    for pix in (None, np.arange(width * height, dtype=np.int32)[::-3].copy()):
        ro, rd = OC.pinhole_rays(width, height, intr, c, pix)
        o, d = ops.pinhole_rays(cam, None if pix is None else torch.from_numpy(pix).cuda())
        assert np.array_equal(o.cpu().numpy(), ro) and np.array_equal(d.cpu().numpy(), rd)


@pytest.mark.parametrize("layout", [_lib.LAYOUT_LEAF_ROWS, _lib.LAYOUT_VEC_SOA])
@pytest.mark.parametrize("K,C,Cg", [(16, 8, 0), (14, 31, 31), (30, 31, 0), (14, 8, 0), (1, 1, 0), (30, 64, 64)])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 257, 70_001])
def test_unpack_grad_rows_edges(n, K, C, Cg, layout):
    """Rows to payload vectors is a rearrangement: every value, and zeros in the padding, for leaf counts around a
    wavefront's share and rows of fewer and of more than 64 values."""
    R = _lib.neuvv_grad_row_elems(K, C, Cg)
    rows = torch.arange(n * R, dtype=torch.float32, device="cuda").remainder_(65_521.0).view(n, R) + 1.0
    parts = [(0, 3 * K), (3 * K, C)] + ([(3 * K + C, Cg)] if Cg else [])
    out = [torch.full((-(-r // 4) * 4 * n,), -1.0, device="cuda") for _, r in parts]
    _lib.neuvv_unpack_grad_rows(K, C, Cg, layout, n, rows, *out)
    for (start, r), got in zip(parts, out):
        want = torch.zeros(n, -(-r // 4) * 4, device="cuda")
        want[:, :r] = rows[:, start:start + r]
        if layout == _lib.LAYOUT_VEC_SOA:
            want = want.view(n, -1, 4).permute(1, 0, 2)
        assert torch.equal(got, want.reshape(-1))


@pytest.mark.parametrize("records", [None, "1", "300"])
@pytest.mark.parametrize("cap", [0, 300, None])
def test_per_point_timed_reduction(cap, records, monkeypatch):
    """Per-point leaves with a time per ray: traced, partly traced and walked rays, with room for every record, for
    some and for one, on a tree whose leaf count is no multiple of a batch; against the oracle."""
    if records is None:
        monkeypatch.delenv("NEUVV_BWD_RECORDS", raising=False)
    else:
        monkeypatch.setenv("NEUVV_BWD_RECORDS", records)
    sc = make_scene_per_point(5, 3000, "random", T=12, seed=7)
    cam = tiny_camera(sc)
    o, d = OC.pinhole_rays(64, 64, cam.intr(), cam.c2w)
    n, rng = o.shape[0], np.random.default_rng(71)
    t = rng.uniform(0, sc.T - 1, n).astype(np.float32)
    g = rng.normal(size=(n, 3)).astype(np.float32)
    g[stop_ambiguous(oracle_render(sc, o, d, t, 0.0, 1e-4, g_rgb=g), label="per-point timed")] = 0.0
    ref = oracle_render(sc, o, d, t, 0.0, 1e-4, g_rgb=g)
    tree, oo, dd, tt = upload(sc), tdev(o), tdev(d), tdev(t)
    trace = ops.Trace(n, 32 * n if cap is None else cap, oo.device)
    rgb, alpha, _, nsamp = ops.render(tree, oo, dd, tt, None, 1e-4, 64, trace=trace)
    out = ops.render_backward(tree, oo, dd, rgb, alpha, nsamp, tdev(g), None, tt, None, 1e-4, 64, trace=trace)
    torch.cuda.synchronize()
    hh, ws, wg = tree.unpack_grad(out[0])
    got = dict(grad_hh=hh, grad_wsig=ws, grad_wgam=wg, grad_basis=out[1], grad_basis_g=out[2])
    e = {k: rel_err(v.cpu().numpy(), ref[k]) for k, v in got.items()}
    announce(f"per-point timed cap={cap} records={records}: grad rel errors {e}")
    assert int(nsamp.sum()) > 1000 and max(e.values()) <= 1e-4, e


def test_kept_scratch(tiny):
    """Scratch kept between calls: growing and shrinking calls on two streams whose work overlaps, streams made and
    dropped beyond the kept blocks, calls of four threads, and calls after a release all give the one-call results."""
    sc, o, d, g, _ = tiny
    tree, oo, dd, gg = upload(sc), tdev(o), tdev(d), tdev(g)

    def once(m, stream):
        with torch.cuda.stream(stream):
            rgb, alpha, _, ns = ops.render(tree, oo[:m], dd[:m], 4.0, None, 1e-4, 64, want_depth=False)
            grads = ops.render_backward(tree, oo[:m], dd[:m], rgb, alpha, ns, gg[:m], None, 4.0, None, 1e-4, 64)
        return rgb, ns, grads[0]

    def same(got, want):
        return torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and \
            rel_err(got[2].cpu().numpy(), want[2].cpu().numpy()) <= 1e-5   # summation order of float32 atomics

    sizes = [64, 4096, 640, 2048, 64, 4096]
    main = torch.cuda.current_stream()
    want = {m: once(m, main) for m in set(sizes)}
    torch.cuda.synchronize()
    two = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = [(m, once(m, s)) for _ in range(5) for m in sizes for s in two]
    torch.cuda.synchronize()
    assert all(same(r, want[m]) for m, r in got)
    got = [(m, once(m, torch.cuda.Stream())) for k in range(40) for m in (64, 4096)]
    torch.cuda.synchronize()
    assert all(same(r, want[m]) for m, r in got)
    results = []

    def worker(stream):
        results.extend((m, once(m, stream)) for m in sizes)

    threads = [threading.Thread(target=worker, args=(s,)) for s in (main, main, two[0], two[1])]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    torch.cuda.synchronize()
    assert len(results) == 4 * len(sizes) and all(same(r, want[m]) for m, r in results)
    _lib.neuvv_release_scratch()
    r = once(4096, main)
    torch.cuda.synchronize()
    assert same(r, want[4096])


@pytest.mark.parametrize("traced", [False, True])
@pytest.mark.parametrize("width,n", [(1, 333), (7, 400), (8, 512), (9, 513), (63, 4000), (64, 4096), (65, 3999),
                                     (513, 4096), (4096, 4096), (5000, 4096)])
def test_cull_segments(tiny, width, n, traced):
    """Images whose rows and columns end inside a tile, a segment of tiles and an XCD's part: the outputs are those of
    the same rays as a list, bit for bit, and so are the gradients up to summation order."""
    sc, o, d, g, _ = tiny
    tree, oo, dd, gg = upload(sc), tdev(o[:n]), tdev(d[:n]), tdev(g[:n])
    got = []
    for w in (0, width):
        trace = ops.Trace(n, 4 * n, oo.device) if traced else None
        out = ops.render(tree, oo, dd, 4.0, None, 1e-4, w, trace=trace)
        got.append(out + ops.render_backward(tree, oo, dd, out[0], out[1], out[3], gg, None, 4.0, None, 1e-4, w,
                                             trace=trace))
    torch.cuda.synchronize()
    for a, b in zip(got[0][:4], got[1][:4]):
        assert torch.equal(a, b)
    for a, b in zip(got[0][4:], got[1][4:]):
        assert rel_err(a.cpu().numpy(), b.cpu().numpy()) <= 1e-5


@pytest.mark.parametrize("form", ["global", "wide", "per_point"])
@pytest.mark.parametrize("timed", [False, True])
@pytest.mark.parametrize("records", [None, "0", "1", "9000"])
def test_fresh_gradients(form, timed, records, monkeypatch):
    """Gradient rows written by the call itself (the buffer starts as NaN) are those that a call adds to a cleared
    buffer, with room for every record, for some and for none, traced, partly traced and walked, and for no rays."""
    if records is None:
        monkeypatch.delenv("NEUVV_BWD_RECORDS", raising=False)
    else:
        monkeypatch.setenv("NEUVV_BWD_RECORDS", records)
    sc = make_scene_per_point(5, 3000, "random", T=12, seed=7) if form == "per_point" else \
        make_scene(5, 3001, "random", K=30 if form == "wide" else 16, C=31 if form == "wide" else 8, T=12, seed=8)
    tree, cam = upload(sc), tiny_camera(sc)
    o, d = (tdev(v) for v in OC.pinhole_rays(64, 64, cam.intr(), cam.c2w))
    n, rng = o.shape[0], np.random.default_rng(81)
    t = tdev(rng.uniform(0, sc.T - 1, n)) if timed else 3.25
    g = tdev(rng.normal(size=(n, 3)))
    for m, cap in ((n, None), (n, 0), (n, 900), (n, 64 * n), (0, None)):
        tt = t[:m].contiguous() if timed else t
        trace = None if cap is None else ops.Trace(m, cap, o.device)
        rgb, alpha, _, ns = ops.render(tree, o[:m], d[:m], tt, None, 1e-4, 64, trace=trace)
        want = ops.render_backward(tree, o[:m], d[:m], rgb, alpha, ns, g[:m], None, tt, None, 1e-4, 64,
                                   grads=tree.zero_grads(), trace=trace)
        got = tree.zero_grads()
        got[0].fill_(float("nan"))
        _lib.neuvv_render_backward_fresh(tree.struct(), None, m, o, d, tt if timed else None, 0.0 if timed else tt, 64,
                                         1e-4, rgb, alpha, ns, g, None, got[0], got[1], got[2] if tree.Cg else None,
                                         None if trace is None else trace.buf, 0 if trace is None else trace.cap)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert rel_err(a.cpu().numpy(), b.cpu().numpy()) <= 1e-5   # summation order of float32 atomics
        assert m == 0 or float(want[0].abs().max()) > 0


@pytest.mark.parametrize("depth,leaves", [(2, 1), (3, 63), (3, 65), (5, 1000), (6, 16_383), (6, 16_384), (6, 16_385)])
@pytest.mark.parametrize("traced", [False, True])
def test_timed_reduction_lists(depth, leaves, traced):
    """Per-point leaves with a time per ray: trees small enough for several record lists per leaf (below 16,384 leaves
    for these 4,096 rays) and at the edge of that rule, for stored and for added rows; against the oracle."""
    sc = make_scene_per_point(depth, leaves, "random", T=12, seed=9)
    cam = tiny_camera(sc)
    o, d = OC.pinhole_rays(64, 64, cam.intr(), cam.c2w)
    n, rng = o.shape[0], np.random.default_rng(91)
    t = rng.uniform(0, sc.T - 1, n).astype(np.float32)
    g = rng.normal(size=(n, 3)).astype(np.float32)
    g[stop_ambiguous(oracle_render(sc, o, d, t, 0.0, 1e-4, g_rgb=g), label="timed lists")] = 0.0
    ref = oracle_render(sc, o, d, t, 0.0, 1e-4, g_rgb=g)
    tree, oo, dd, tt = upload(sc), tdev(o), tdev(d), tdev(t)
    trace = ops.Trace(n, 64 * n, oo.device) if traced else None
    rgb, alpha, _, nsamp = ops.render(tree, oo, dd, tt, None, 1e-4, 64, trace=trace)
    for grads in (None, tree.zero_grads()):
        out = ops.render_backward(tree, oo, dd, rgb, alpha, nsamp, tdev(g), None, tt, None, 1e-4, 64, grads=grads,
                                  trace=trace)
        torch.cuda.synchronize()
        hh, ws, wg = tree.unpack_grad(out[0])
        got = dict(grad_hh=hh, grad_wsig=ws, grad_wgam=wg, grad_basis=out[1], grad_basis_g=out[2])
        e = {k: rel_err(v.cpu().numpy(), ref[k]) for k, v in got.items()}
        announce(f"timed lists {depth} {leaves} {traced}: grad rel errors {e}")
        assert max(e.values()) <= 1e-4, e


def _fastest(call):
    """Milliseconds of the fastest of six calls."""
    ms = []
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        ms.append(a.elapsed_time(b))
    return min(ms)


def test_timed_reduction_small_tree_time(monkeypatch):
    """262,144 rays with times of their own on 1,000 per-point leaves: the adjoint with records takes no longer than
    half as much again as with none (the lists of a small tree once ran on 16 wavefronts and took ten times as long)."""
    sc = make_scene_per_point(5, 1000, "random", T=12, seed=9)
    cam = tiny_camera(sc)
    o, d = (tdev(np.repeat(v, 64, 0)) for v in OC.pinhole_rays(64, 64, cam.intr(), cam.c2w))
    n, rng, tree = o.shape[0], np.random.default_rng(92), upload(sc)
    t, g = tdev(rng.uniform(0, sc.T - 1, n)), tdev(rng.normal(size=(n, 3)))
    rgb, alpha, _, nsamp = ops.render(tree, o, d, t)
    ms = {}
    for records in ("4000000", "0"):
        monkeypatch.setenv("NEUVV_BWD_RECORDS", records)
        ms[records] = _fastest(lambda: ops.render_backward(tree, o, d, rgb, alpha, nsamp, g, None, t))
    announce(f"timed reduction of a small tree: {ms} ms, {int(nsamp.sum())} samples")
    assert ms["4000000"] <= 1.5 * ms["0"], ms


@pytest.mark.parametrize("records", ["0", "1000"])
def test_traced_adjoint_without_room_for_records(tiny, records, monkeypatch):
    """A traced adjoint that has records for few samples or none takes no longer than half as much again as the
    untraced one (it once made a basis for every sample, one lane at a time, and took three times as long), and its
    gradients are the oracle's."""
    sc, o, d, g, ref = tiny
    monkeypatch.setenv("NEUVV_BWD_RECORDS", records)
    tree, rep = upload(sc), 64
    oo, dd, gg = (tdev(np.repeat(v, rep, 0)) for v in (o, d, g))
    n, ms = oo.shape[0], {}
    trace = ops.Trace(n, 16 * n, oo.device)
    rgb, alpha, _, nsamp = ops.render(tree, oo, dd, 4.0, trace=trace)
    for name, tr in (("untraced", None), ("traced", trace)):
        ms[name] = _fastest(lambda: ops.render_backward(tree, oo, dd, rgb, alpha, nsamp, gg, None, 4.0, trace=tr))
    gl, gb = ops.render_backward(tree, oo, dd, rgb, alpha, nsamp, gg, None, 4.0, trace=trace)
    hh, ws = tree.unpack_grad(gl)
    e = [rel_err(hh.cpu().numpy() / rep, ref["grad_hh"]), rel_err(ws.cpu().numpy() / rep, ref["grad_wsig"]),
         rel_err(gb.cpu().numpy() / rep, ref["grad_basis"])]
    announce(f"traced without room: {ms} ms, grad rel errors {e}")
    assert max(e) <= 1e-4, e
    assert ms["traced"] <= 1.5 * ms["untraced"], ms


def _hip():
    """The HIP runtime that this process has loaded."""
    path = next(ln.split()[-1] for ln in open("/proc/self/maps") if "libamdhip64" in ln)
    lib = ctypes.CDLL(path)
    lib.hipStreamCreateWithFlags.argtypes = [ctypes.c_void_p, ctypes.c_uint]
    lib.hipStreamDestroy.argtypes = [ctypes.c_void_p]
    return lib


def test_scratch_of_destroyed_streams(tiny):
    """Streams of the runtime that are destroyed while their work is queued, so that later streams may get their
    handles: more of them than blocks are kept, two calls in flight at a time, and calls on the per-thread stream."""
    sc, o, d, g, _ = tiny
    hip, tree = _hip(), upload(sc)
    oo, dd, gg = (tdev(np.repeat(v, 64, 0)) for v in (o, d, g))
    sizes = [oo.shape[0], 64, 4096]

    def once(m, stream, out):
        ops.render(tree, oo[:m], dd[:m], 4.0, out=out[:4], stream=stream)
        ops.render_backward(tree, oo[:m], dd[:m], out[0], out[1], out[3], gg[:m], None, 4.0, grads=out[4:],
                            stream=stream)

    def outputs(m):
        return (torch.empty(m, 3, device="cuda"), torch.empty(m, device="cuda"), torch.empty(m, device="cuda"),
                torch.empty(m, dtype=torch.int32, device="cuda")) + tree.zero_grads()

    want = {m: outputs(m) for m in sizes}
    for m in sizes:
        once(m, None, want[m])
    work = [(sizes[k % 3], outputs(sizes[k % 3])) for k in range(45)]
    torch.cuda.synchronize()
    streams, handles = [], set()
    for k, (m, out) in enumerate(work):
        if k % 9 == 8:
            once(m, 2, out)   # hipStreamPerThread
            continue
        s = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0   # non-blocking, default priority
        handles.add(s.value)
        streams.append(s)
        once(m, s.value, out)
        if len(streams) == 2:
            assert hip.hipStreamDestroy(streams.pop(0)) == 0
    for s in streams:
        assert hip.hipStreamDestroy(s) == 0
    torch.cuda.synchronize()
    announce(f"{len(handles)} handles of 40 streams")
    for m, out in work:
        for a, b in zip(out[:4], want[m][:4]):
            assert torch.equal(a, b)
        for a, b in zip(out[4:], want[m][4:]):
            assert rel_err(a.cpu().numpy(), b.cpu().numpy()) <= 1e-5   # summation order of float32 atomics
    _lib.neuvv_release_scratch()


def test_captured_calls(tiny):
    """Calls captured in a graph, whose scratch is the graph's, beside eager calls on kept scratch: every replay gives
    the eager results."""
    sc, o, d, g, _ = tiny
    tree, oo, dd, gg = upload(sc), tdev(o), tdev(d), tdev(g)
    want = ops.render(tree, oo, dd, 4.0, None, 1e-4, 64)
    wg = ops.render_backward(tree, oo, dd, want[0], want[1], want[3], gg, None, 4.0, None, 1e-4, 64)
    out, grads = tuple(torch.empty_like(v) for v in want), tree.zero_grads()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ops.render(tree, oo, dd, 4.0, None, 1e-4, 64, out=out)
        ops.render_backward(tree, oo, dd, out[0], out[1], out[3], gg, None, 4.0, None, 1e-4, 64, grads=grads)
    for _ in range(4):
        for v in out + tuple(grads):
            v.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want))
        assert all(rel_err(a.cpu().numpy(), b.cpu().numpy()) <= 1e-5 for a, b in zip(grads, wg))
        again = ops.render(tree, oo, dd, 4.0, None, 1e-4, 64)
        assert all(torch.equal(a, b) for a, b in zip(again, want))


@pytest.mark.parametrize("traced", [False, True])
@pytest.mark.parametrize("n", [16_383 * 64, 16_384 * 64 - 37, 16_384 * 64, 16_384 * 64 + 1])
def test_cull_groups(tiny, n, traced):
    """Lists of rays on both sides of the size (16,384 chunks of 64) from which a wavefront culls more of them at a time,
    ragged at the end: the outputs are those of the same rays as an image, bit for bit, gradients up to summation
    order, rows written by the call itself as well as added."""
    sc, o, d, g, _ = tiny
    shift = 1237   # (rays of every part of the view in each group)
    pick = (np.arange(n) * shift) % o.shape[0]
    tree, oo, dd, gg = upload(sc), tdev(o[pick]), tdev(d[pick]), tdev(g[pick])
    got = []
    for w in (0, 1024):
        trace = ops.Trace(n, n, oo.device) if traced else None
        out = ops.render(tree, oo, dd, 4.0, None, 1e-4, w, trace=trace)
        for grads in (None, tree.zero_grads()):
            got.append(out + ops.render_backward(tree, oo, dd, out[0], out[1], out[3], gg, None, 4.0, None, 1e-4, w,
                                                 grads=grads, trace=trace))
    torch.cuda.synchronize()
    assert int(got[0][3].sum()) > n // 4
    for other in got[1:]:
        for a, b in zip(got[0][:4], other[:4]):
            assert torch.equal(a, b)
        for a, b in zip(got[0][4:], other[4:]):
            assert rel_err(a.cpu().numpy(), b.cpu().numpy()) <= 1e-4   # the gradients' bar: lists of thousands of records
