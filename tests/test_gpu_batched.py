"""Batching: segmented Reduce over many uneven vectors in one persistent
launch, and chains of skeleton calls captured in a graph and replayed.

Segment lengths follow the batched workload: floor(exp(U[ln 32, ln 2^20])),
values N(0, 1); parity against the oracle's per-segment binary64 Reduce with
|r - r*| <= 1e-5 * sum |x| of the segment (MIN / MAX exact).
"""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

RED_OPS = {"sum": 0, "min": 1, "max": 2}


def check_segments(skel, oracle_mod, x, off, op, variant):
    out = skel.Container.empty(skel.F32, off.size - 1)
    skel.skel_reduce_segments(RED_OPS[op], skel.Container.from_numpy(x),
                              skel.Container.from_numpy(off), out, variant=variant)
    got = out.to_numpy().astype(np.float64)
    ref = oracle_mod.reduce_segments(op, x, off)
    if op == "sum":
        mag = oracle_mod.reduce_segments("sum", np.abs(x), off)
        bad = np.abs(got - ref) > 1e-5 * mag + 1e-30
    else:
        bad = got != ref
    assert not bad.any(), (op, variant, np.flatnonzero(bad)[:5])


@pytest.mark.parametrize("op", list(RED_OPS))
def test_segments_small_and_edge_cases(skel, oracle_mod, op):
    x = si.normal_f32(200003, 2, 0)
    cases = [
        np.array([0, x.size], np.int64),                      # one segment
        np.array([0, 0, 0], np.int64),                        # only empty segments
        np.array([0, 1, 2, 3, 16387, 16387, 50000, 200003], np.int64),  # mixed, ragged
        np.array([0, 16384, 32768, 32769, 200003], np.int64),  # chunk boundaries
        np.array([5, 9, 17], np.int64),                       # not starting at 0, unaligned
    ]
    for off in cases:
        for v in range(skel.skel_variant_count(skel.SK_REDUCE_SEGMENTS)):
            check_segments(skel, oracle_mod, x, off, op, v)
    skel.skel_sync()


@pytest.mark.parametrize("op", list(RED_OPS))
@pytest.mark.parametrize("lens", [
    [4095, 1, 4096, 4097, 0, 0, 1023, 1, 1024, 2048, 3],      # chunk and slice edges
    [0, 0, 1, 0, 4095, 0, 0],                                 # empty ones at the edges
    [1] * 20000 + [0] * 700 + [2] * 5000,                     # many starts in a chunk
    [5, 15 * 4096, 1, 16 * 4096, 3, 17 * 4096 - 1, 4],        # few pieces and many
    [100, 4200 * 4096 + 17, 7, 0],                            # one long vector
], ids=["edges", "empty", "short", "pieces", "long"])
def test_segments_across_chunks(skel, oracle_mod, op, lens):
    """B1 divides the elements into chunks of 4096 (slices of 1024): segments
    that start, end or span at those edges, at the end of the data, and with
    elements before the first and after the last offset; two calls give the
    same bits."""
    for lead, trail in ((0, 0), (3, 9000)):
        off = (lead + np.concatenate([[0], np.cumsum(lens)])).astype(np.int64)
        x = si.normal_f32(int(off[-1]) + trail, 2, 31)
        check_segments(skel, oracle_mod, x, off, op, 1)
    cx, co = skel.Container.from_numpy(x), skel.Container.from_numpy(off)
    got = []
    for _ in range(2):
        out = skel.Container.empty(skel.F32, len(lens))
        skel.skel_reduce_segments(RED_OPS[op], cx, co, out, variant=1)
        got.append(out.to_numpy())
    assert np.array_equal(got[0], got[1])
    skel.skel_sync()


@pytest.mark.parametrize("op", list(RED_OPS))
@pytest.mark.parametrize("lens,lead,trail", [
    ([4 * 4096, 4 * 4096 + 1, 5 * 4096, 5 * 4096 - 1, 6 * 4096, 1], 4096, 3 * 4096),
    ([7, 0, 90 * 4096, 0, 3, 70 * 4096 + 5] * 3, 2 * 4096 + 7, 1),
    ([0, 0, 0], 3 * 4096, 0),                                  # all at the end of the data
    ([0, 5, 0, 0], 0, 4 * 4096),                               # chunks past the last offset
    ([3, 1023 * 4096, 1024 * 4096, 1025 * 4096, 2], 0, 0),     # pieces of one wavefront
], ids=["own", "shared", "end", "past", "pieces"])
def test_segments_first_of_each_chunk(skel, oracle_mod, op, lens, lead, trail):
    """The table of each chunk's first segment: entries written by one lane (up
    to four chunks per segment) and by a wavefront, chunks before the first and
    after the last offset, and segments of about 1024 chunks."""
    off = (lead + np.concatenate([[0], np.cumsum(lens)])).astype(np.int64)
    x = si.normal_f32(int(off[-1]) + trail, 2, 33)
    check_segments(skel, oracle_mod, x, off, op, 1)
    skel.skel_sync()


def test_segments_log_uniform_batch(skel, oracle_mod):
    lens = si.log_uniform_lengths(512, 32, 1 << 20, config=2, index=10)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    x = si.normal_f32(int(off[-1]), 2, 11)
    for v in (0, 1):
        check_segments(skel, oracle_mod, x, off, "sum", v)
    # repeated calls reuse the counters and slots (fresh epoch per call)
    for k in range(3):
        check_segments(skel, oracle_mod, x, off, "max", 1)
    skel.skel_sync()


def test_segments_reject_bad_offsets(skel):
    x = skel.Container.from_numpy(np.ones(1000, np.float32))
    bad = skel.Container.from_numpy(np.array([0, 600, 500, 1000], np.int64))
    out = skel.Container.empty(skel.F32, 3)
    with pytest.raises(skel.SkelError) as e:
        skel.skel_reduce_segments(skel.SUM, x, bad, out, variant=0)
    assert e.value.status == skel.E_INVAL
    # the persistent variant checks on the device: no work, flag at sync
    skel.skel_reduce_segments(skel.SUM, x, bad, out, variant=1)
    with pytest.raises(skel.SkelError) as e:
        skel.skel_sync()
    assert e.value.status == skel.E_TIMEOUT and "flag 0x4" in str(e.value)
    skel.skel_sync()  # the flag was cleared
    # and the next good call is unaffected
    good = skel.Container.from_numpy(np.array([0, 500, 600, 1000], np.int64))
    skel.skel_reduce_segments(skel.SUM, x, good, out, variant=1)
    assert out.to_numpy().tolist() == [500.0, 100.0, 400.0]
    with pytest.raises(skel.SkelError) as e:
        skel.skel_reduce_segments(skel.SUM, x, good, skel.Container.empty(skel.F32, 2))
    assert e.value.status == skel.E_SHAPE


def test_graph_capture_replays(skel, oracle_mod):
    """A chain Map -> MapReduce -> Scan captured once and replayed with new
    inputs between replays; every replay is checked against the oracle.  The
    look-back scan and the ticket reduction hand values between workgroups
    through epoch-tagged words, so a replay that reused the previous replay's
    epoch would read stale descriptors: the changing inputs catch that."""
    import torch
    n = (1 << 20) + 5
    x0 = si.normal_f32(n, 5, 0)
    y = si.normal_f32(n, 5, 1)
    ci = si.int_uniform_i32(n, 1000, 5, 2)
    cx, cy = skel.Container.from_numpy(x0), skel.Container.from_numpy(y)
    cz = skel.Container.empty(skel.F32, n)
    r = skel.Container.empty(skel.F32, 1)
    csi = skel.Container.from_numpy(ci)
    cso = skel.Container.empty(skel.I64, n)
    stream = torch.cuda.Stream()

    def chain():
        skel.skel_map(skel.MAP_AFFINE, [2.0, 1.0], [cx], cz, stream=stream)
        skel.skel_mapreduce(skel.MAP_MUL, None, [cz, cy], skel.SUM, r, variant=2,
                            stream=stream)
        skel.skel_scan(csi, cso, skel.EXCLUSIVE, skel.SUM, variant=2, stream=stream)

    with torch.cuda.stream(stream):
        chain()  # outside capture: sizes workspaces, makes device copies valid
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            chain()
    torch.cuda.synchronize()
    for rep in range(4):
        xk = si.normal_f32(n, 6, rep)
        ik = si.int_uniform_i32(n, 1000, 6, 10 + rep)
        cx.write_numpy(xk)
        csi.write_numpy(ik)
        for c in (cx, csi):  # eager device reads make the new data resident
            skel.skel_container_acquire(c, skel.DEVICE, skel.READ, stream)
            skel.skel_container_release(c, skel.DEVICE, stream)
        # eager work of the same kinds between replays
        tmp = skel.Container.empty(skel.I64, n)
        skel.skel_scan(csi, tmp, skel.INCLUSIVE, skel.SUM, variant=2, stream=stream)
        with torch.cuda.stream(stream):
            g.replay()
        for c in (cz, r, cso):
            c.mark_device_written(stream)
        zref = oracle_mod.map_f32("affine", [2.0, 1.0], xk).astype(np.float32)
        ref, mag = oracle_mod.mapreduce("mul", None, zref, y)
        assert abs(float(r.to_numpy()[0]) - ref) <= 1e-5 * mag, rep
        assert np.array_equal(cso.to_numpy(), oracle_mod.scan(ik, "exclusive", "sum",
                                                              np.int64)), rep
        assert np.array_equal(tmp.to_numpy(), oracle_mod.scan(ik, "inclusive", "sum",
                                                              np.int64)), rep
    skel.skel_sync(stream)


@pytest.mark.parametrize("op", ["sum", "max"])
def test_reduce_segments_many_empty(skel, op):
    """Runs of a million empty segments: at the start, inside and at the end of the data, at
    a chunk's border, and with no data at all."""
    import torch
    m = 1_000_000
    for before, after in ((0, 0), (0, 5), (5, 0), (4096, 4096), (5000, 300), (1, 9000)):
        lens = np.r_[np.full(int(before > 0), before, np.int64), np.zeros(m, np.int64),
                     np.full(int(after > 0), after, np.int64)]
        off = np.r_[0, np.cumsum(lens)]
        x = si.normal_f32(before + after, 31, before)
        cx = (skel.Container.from_numpy(x) if x.size else skel.Container.empty(skel.F32, 1, 0))
        out = skel.Container.empty(skel.F32, lens.size)
        skel.skel_reduce_segments(skel.SUM if op == "sum" else skel.MAX, cx,
                                  skel.Container.from_numpy(off), out, variant=1)
        got = out.to_numpy()
        ident = np.float32(0 if op == "sum" else -np.inf)
        full = np.flatnonzero(lens)
        assert np.all(np.delete(got, full) == ident), (op, before, after)
        for s in full:
            part = x[off[s]:off[s + 1]].astype(np.float64)
            if op == "max":
                assert got[s] == part.max()
            else:
                assert abs(got[s] - part.sum()) <= 1e-5 * np.abs(part).sum()
    skel.skel_sync()


def test_graph_replays_batched_layer_and_persistent_scan(skel, oracle_mod):
    """The batched forms and the persistent scan captured once (a batched-field
    stencil, a row-wise scan, its reverse, the batched transpose, and an S3
    scan whose workgroups share a tile counter reset on the device) and
    replayed with new inputs and eager calls of the same kinds in between;
    every replay is checked against the oracle."""
    import torch
    dev = torch.device("cuda", 0)
    F, H, W = 6, 96, 136
    n = (1 << 18) + 77
    w5 = si.five_point_weights(0.5, 0.1, 0.2, 0.05, 0.15)
    x = torch.empty(F * H, W, device=dev)
    y, z, gz, gy, gx = (torch.empty_like(x) for _ in range(5))
    si_t = torch.empty(n, dtype=torch.int32, device=dev)
    so_t = torch.empty(n, dtype=torch.int64, device=dev)
    stream = torch.cuda.Stream()
    cs = [skel.wrap_tensor(t, stream) for t in (x, y, z, gz, gy, gx, si_t, so_t)]
    cx, cy, cz, cgz, cgy, cgx, csi, cso = cs

    def chain():
        skel.skel_mapoverlap2d_fields(cx, cy, F, w2d=w5, stream=stream)
        skel.skel_scan_rows(cy, cz, skel.INCLUSIVE, skel.SUM, stream=stream)
        skel.skel_scan_rows(cgz, cgy, skel.REVERSE_INCLUSIVE, skel.SUM, stream=stream)
        skel.skel_mapoverlap2d_fields_backward(cgy, cgx, F, w2d=w5, stream=stream)
        skel.skel_scan(csi, cso, skel.EXCLUSIVE, skel.SUM, variant=3, stream=stream)

    with torch.cuda.stream(stream):
        chain()  # outside capture: sizes workspaces
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            chain()
    torch.cuda.synchronize()
    tmp = torch.empty(n, dtype=torch.int64, device=dev)
    ctmp = skel.wrap_tensor(tmp, stream)
    for rep in range(4):
        xh = si.normal_f32(F * H * W, 7, rep).reshape(F * H, W)
        gh = si.normal_f32(F * H * W, 7, 10 + rep).reshape(F * H, W)
        ih = si.int_uniform_i32(n, 1000, 7, 20 + rep)
        with torch.cuda.stream(stream):
            x.copy_(torch.from_numpy(xh))
            gz.copy_(torch.from_numpy(gh))
            si_t.copy_(torch.from_numpy(ih))
            # eager calls of the same kinds between replays
            skel.skel_scan(csi, ctmp, skel.INCLUSIVE, skel.SUM, variant=3, stream=stream)
            skel.skel_scan_rows(cgz, cgx, skel.INCLUSIVE, skel.SUM, stream=stream)
            g.replay()
        stream.synchronize()
        zr = z.cpu().numpy()
        gxr = gx.cpu().numpy()
        for f in range(F):
            blk = slice(f * H, (f + 1) * H)
            yref, ymag = oracle_mod.mapoverlap2d(xh[blk], 1, 1, w2d=w5, edge="clamp")
            zref, _ = oracle_mod.scan_rows(yref.astype(np.float32), "inclusive")
            zmag = oracle_mod.scan_rows(ymag.astype(np.float32), "inclusive")[0]
            assert np.all(np.abs(zr[blk] - zref) <= 1e-5 * zmag + 1e-30), (rep, f)
            gyref, gymag = oracle_mod.scan_rows(gh[blk], "reverse_inclusive")
            dref, _ = oracle_mod.mapoverlap2d_adjoint(gyref.astype(np.float32), 1, 1, w2d=w5,
                                                      edge="clamp")
            _, dmag = oracle_mod.mapoverlap2d_adjoint(gymag.astype(np.float32), 1, 1,
                                                      w2d=np.abs(w5), edge="clamp")
            assert np.all(np.abs(gxr[blk] - dref) <= 1e-5 * dmag + 1e-30), (rep, f)
        assert np.array_equal(so_t.cpu().numpy(), oracle_mod.scan(ih, "exclusive", "sum",
                                                                 np.int64)), rep
        assert np.array_equal(tmp.cpu().numpy(), oracle_mod.scan(ih, "inclusive", "sum",
                                                                np.int64)), rep
    skel.skel_sync(stream)
    for c in cs + [ctmp]:
        c.destroy()


def test_containers_collected_during_capture_are_destroyed_after(skel):
    """A container that Python collects while a graph is being captured is not
    destroyed then (that would wait for the device and free pinned memory,
    invalidating the capture): it is destroyed after the capture."""
    import gc
    import torch
    n = 1 << 16
    x = torch.ones(n, device="cuda")
    y = torch.empty_like(x)
    stream = torch.cuda.Stream()
    cx, cy = skel.wrap_tensor(x, stream), skel.wrap_tensor(y, stream)
    garbage = [skel.Container.from_numpy(np.ones(1000, np.float32)) for _ in range(4)]
    for c in garbage:  # device copies with pending work, pinned host copies
        skel.skel_map(skel.MAP_AFFINE, [2.0, 0.0], [c], c, stream=stream)
    with torch.cuda.stream(stream):
        skel.skel_map(skel.MAP_AFFINE, [2.0, 1.0], [cx], cy, stream=stream)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            del garbage
            gc.collect()  # collected inside the capture
            skel.skel_map(skel.MAP_AFFINE, [2.0, 1.0], [cx], cy, stream=stream)
        g.replay()
    stream.synchronize()
    assert torch.all(y == 3.0)
    skel.skel_sync(stream)  # the deferred containers are destroyed here
    cx.destroy()
    cy.destroy()
