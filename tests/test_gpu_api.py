"""The C ABI on the GPU: argument validation (no side effects on failure),
selectability of forced variants, transfer accounting of the smart containers
over a chain of dependent skeleton calls (Section IV), and cross-stream
ordering through container events (Section V)."""
import ctypes as C

import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


def status_of(fn, *a, **k):
    import paper_1405_2915_amd as skel
    try:
        fn(*a, **k)
    except skel.SkelError as e:
        return e.status
    return skel.OK


def test_validation_statuses(skel):
    x = skel.Container.from_numpy(np.ones(100, np.float32))
    xi = skel.Container.from_numpy(np.ones(100, np.int32))
    y = skel.Container.from_numpy(np.ones(50, np.float32))
    r = skel.Container.empty(skel.F32, 1)
    r2 = skel.Container.empty(skel.F32, 2)
    assert status_of(skel.skel_map, 99, [], [x], x) == skel.E_INVAL
    assert status_of(skel.skel_map, skel.MAP_AXPY, [2.5], [x], x) == skel.E_INVAL  # 1 input
    assert status_of(skel.skel_map, skel.MAP_AXPY, [], [x, x], x) == skel.E_INVAL  # no p0
    assert status_of(skel.skel_map, skel.MAP_MUL, [], [x, y], x) == skel.E_SHAPE
    assert status_of(skel.skel_map, skel.MAP_SQUARE, [], [xi], x) == skel.E_DTYPE
    assert status_of(skel.skel_reduce, skel.SUM, x, r2) == skel.E_SHAPE
    assert status_of(skel.skel_reduce, skel.SUM, x, x) == skel.E_INVAL
    assert status_of(skel.skel_reduce, skel.SUM, xi, r) == skel.E_DTYPE  # i32 -> f32
    assert status_of(skel.skel_reduce, 7, x, r) == skel.E_INVAL
    assert status_of(skel.skel_reduce, skel.SUM, x, r, variant=17) == skel.E_UNSUPPORTED
    assert status_of(skel.skel_reduce, skel.MAX, x, r, variant=3) == skel.E_UNSUPPORTED
    assert status_of(skel.skel_scan, x, x, 5, skel.SUM) == skel.E_INVAL
    assert status_of(skel.skel_scan, xi, y, skel.INCLUSIVE, skel.SUM) == skel.E_DTYPE
    assert status_of(skel.skel_mapoverlap1d, x, x, [1, 1, 1], 1) == skel.E_INVAL
    big = np.ones(2 * 65 + 1, np.float32)
    o = skel.Container.empty(skel.F32, 100)
    assert status_of(skel.skel_mapoverlap1d, x, o, big, 65) == skel.E_INVAL
    img = skel.Container.from_numpy(np.ones((8, 8), np.float32))
    img2 = skel.Container.empty(skel.F32, 8, 9)
    assert status_of(skel.skel_mapoverlap2d, img, img2, wy=[1, 1, 1], wx=[1, 1, 1]) \
        == skel.E_SHAPE
    img3 = skel.Container.empty(skel.F32, 8, 8)
    assert status_of(skel.skel_mapoverlap2d, img, img3, w2d=np.ones((3, 3)), variant=2) \
        == skel.E_UNSUPPORTED
    # failed calls moved nothing and counted nothing
    for c in (x, xi, y, r, r2):
        s = c.stats()
        assert s["h2d"] == 0 and s["eager_equiv"] == 0, s
    # an uninitialised container cannot be read
    u = skel.Container.empty(skel.F32, 100)
    assert status_of(skel.skel_reduce, skel.SUM, u, r) == skel.E_STATE
    assert "uninitialised" in skel.skel_last_error()


def test_chain_of_twenty_calls_counts_copies(skel, oracle_mod):
    # Section IV: in a loop of calls, lazy copying moves each operand once.
    n = (1 << 20) + 3
    x = si.uniform_f32(n, -1.0, 1.0, 0, 0)
    y = si.uniform_f32(n, -1.0, 1.0, 0, 1)
    cx, cy = skel.Container.from_numpy(x), skel.Container.from_numpy(y)
    want = y.copy()
    for _ in range(20):
        skel.skel_map(skel.MAP_AXPY, [2.5], [cx, cy], cy)
        # the oracle's binary64 value rounded once = the fused multiply-add result
        want = oracle_mod.map_f32("axpy", [2.5], x, want).astype(np.float32)
    assert np.array_equal(cy.to_numpy(), want)
    sx, sy = cx.stats(), cy.stats()
    assert (sx["h2d"], sx["d2h"], sx["eager_equiv"]) == (1, 0, 20)
    assert (sy["h2d"], sy["d2h"], sy["eager_equiv"]) == (1, 1, 40)
    # the lazy scheme moved 3 copies where an eager one moves 60
    assert sx["h2d"] + sx["d2h"] + sy["h2d"] + sy["d2h"] == 3
    assert sy["d2h_bytes"] == 4 * n


def test_device_pointer_and_host_write(skel):
    import torch
    n = 4096
    c = skel.Container.from_numpy(np.arange(n, dtype=np.float32))
    ptr = skel.skel_container_acquire(c, skel.DEVICE, skel.READ)
    assert ptr % 256 == 0
    skel.skel_container_release(c, skel.DEVICE)
    c.write_numpy(np.full(n, 3.0, np.float32))  # host write invalidates device copy
    r = skel.Container.empty(skel.F32, 1)
    skel.skel_reduce(skel.SUM, c, r)
    assert r.to_numpy()[0] == 3.0 * n
    assert c.stats()["h2d"] == 2
    torch.cuda.synchronize()


def test_cross_stream_dependence(skel):
    import torch
    n = 1 << 22
    x = si.uniform_f32(n, -1.0, 1.0, 0, 5)
    cx = skel.Container.from_numpy(x)
    cy = skel.Container.empty(skel.F32, n)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(3):
        skel.skel_map(skel.MAP_AFFINE, [2.0, 1.0], [cx], cy, stream=s1)
        r = skel.Container.empty(skel.F32, 1)
        # reads cy on another stream: must wait for the write on s1
        skel.skel_reduce(skel.SUM, cy, r, stream=s2)
        got = float(r.to_numpy()[0])
        ref = float(np.sum(2.0 * x.astype(np.float64) + 1.0))
        assert abs(got - ref) <= 1e-5 * float(np.sum(np.abs(2.0 * x.astype(np.float64) + 1.0)))
    skel.skel_sync(s1)
    skel.skel_sync(s2)


def test_variant_names_and_plan(skel):
    names = {sk: [skel.skel_variant_name(sk, v) for v in range(skel.skel_variant_count(sk))]
             for sk in range(6)}
    assert names[skel.SK_REDUCE] == ["R0_single_wg", "R1_two_pass", "R2_ticket", "R3_atomic",
                                     "R4_compensated", "R5_pairwise", "R6_gather"]
    assert names[skel.SK_MAPREDUCE][4:] == ["MR4_compensated", "MR5_pairwise",
                                            "MR6_fused_gather"]
    assert names[skel.SK_SCAN][2:] == ["S2_decoupled_lookback", "S3_persistent_lookback",
                                       "S4_small_tile_lookback", "S5_flat_lookback"]
    # the tuned plan picks one of the single-pass variants for a large scan
    assert skel.skel_select_variant(skel.SK_SCAN, skel.I32, 1 << 27) in (2, 3)


def test_sync_reports_no_error(skel):
    skel.skel_sync()
    skel.skel_sync(0)


def test_range_granular_coherence(skel, oracle_mod):
    """After the host rewrites a few elements of a device-resident operand,
    the next skeleton call moves only those elements; a host read of part of
    a device-written result moves only that part."""
    import synth_inputs as si
    n = (1 << 22) + 3
    xh = si.normal_f32(n, 11, 0)
    x = skel.Container.from_numpy(xh)
    y = skel.Container.empty(skel.F32, n)
    skel.skel_map(skel.MAP_AFFINE, [2.0, 1.0], [x], y)
    assert x.stats()["h2d_bytes"] == 4 * n
    patch = si.normal_f32(1000, 11, 1)
    x.write_range(123457, patch)
    xh[123457:124457] = patch
    assert x.valid_ranges(skel.DEVICE) == [(0, 123457), (124457, n)]
    skel.skel_map(skel.MAP_AFFINE, [2.0, 1.0], [x], y)
    s = x.stats()
    assert s["h2d"] == 2 and s["h2d_bytes"] == 4 * n + 4000
    part = y.read_range(123000, 2000)
    assert y.stats()["d2h_bytes"] == 8000
    ref = oracle_mod.map_f32("affine", [2.0, 1.0], xh[123000:125000])
    assert np.all(np.abs(part - ref) <= 1e-6 * (2 * np.abs(xh[123000:125000]) + 1))
    full = y.to_numpy()  # the rest of the result, in two runs around the part read
    assert y.stats()["d2h"] == 3 and y.stats()["d2h_bytes"] == 4 * n
    assert np.all(np.abs(full - oracle_mod.map_f32("affine", [2.0, 1.0], xh))
                  <= 1e-6 * (2 * np.abs(xh) + 1))


def test_failed_call_keeps_coherence_state(skel):
    """A call that fails after its operands were acquired -- here a first,
    larger unfused MapReduce inside a graph capture, whose scratch memory (the
    stored products) cannot grow there -- returns SKEL_E_STATE and leaves its
    output's validity as it was: both copies still current, nothing counted."""
    import torch
    mr0 = skel.variant_index(skel.SK_MAPREDUCE, "MR0_unfused")
    s = torch.cuda.Stream()
    small = skel.Container.from_numpy(si.uniform_f32(1000, -1.0, 1.0, 3, 90))
    r = skel.Container.empty(skel.F32, 1)
    with torch.cuda.stream(s):  # the stream's workspace, sized for the small call
        skel.skel_mapreduce(skel.MAP_MUL, None, [small, small], skel.SUM, r, variant=mr0)
    n = 1 << 20  # 4 MiB of products: more scratch than the small call made
    x = skel.Container.from_numpy(si.uniform_f32(n, -1.0, 1.0, 3, 91))
    out = skel.Container.from_numpy(np.array([42.0], np.float32))
    with torch.cuda.stream(s):  # device copies current before the capture
        for c in (x, out):
            skel.skel_container_acquire(c, skel.DEVICE, skel.READ)
            skel.skel_container_release(c, skel.DEVICE)
    skel.skel_sync(s)
    before = (out.valid_ranges(skel.HOST), out.valid_ranges(skel.DEVICE), out.stats())
    assert before[0] == before[1] == [(0, 1)]
    g = torch.cuda.CUDAGraph()
    status = None
    try:
        with torch.cuda.graph(g, stream=s):
            try:
                skel.skel_mapreduce(skel.MAP_MUL, None, [x, x], skel.SUM, out, variant=mr0)
            except skel.SkelError as e:
                status = e.status
    except RuntimeError:
        pass  # torch may refuse an empty capture; the call's own status is what counts
    assert status == skel.E_STATE
    assert out.valid_ranges(skel.HOST) == before[0]
    assert out.valid_ranges(skel.DEVICE) == before[1]
    assert out.stats()["eager_equiv"] == before[2]["eager_equiv"]
    assert out.to_numpy()[0] == 42.0


def test_plain_and_converted_arguments_agree(skel):
    """Calls whose arguments are plain (containers, numbers, float32 arrays) go
    straight to the library; the same values in other forms (lists, float64 and
    strided arrays, numpy scalars, a Container subclass) are converted first.
    Both give the same bits and raise the same errors."""
    import torch

    class Sub(skel.Container):
        """a second name of another container's handle, which that one frees"""

        def __del__(self):
            pass

    def sub(c):
        d = object.__new__(Sub)
        d.__dict__.update(c.__dict__)
        return d

    n = 3000
    x = skel.Container.from_numpy(si.uniform_f32(n, -1.0, 1.0, 61, 0).reshape(50, 60))
    k = skel.Container.from_numpy(si.int_uniform_i32(n, 100, 61, 1).reshape(50, 60))
    off = skel.Container.from_numpy(np.array([0, 7, 7, 2999, 3000], np.int64))
    w1 = si.uniform_f32(5, -1.0, 1.0, 61, 2)
    w2 = si.uniform_f32(15, -1.0, 1.0, 61, 3).reshape(3, 5)
    wy, wx = si.uniform_f32(3, 0.0, 1.0, 61, 4), si.uniform_f32(7, 0.0, 1.0, 61, 5)
    f64 = lambda a: a.astype(np.float64)
    strided = lambda a: np.repeat(a, 2, axis=-1)[..., ::2]
    f32 = lambda *s: skel.Container.empty(skel.F32, *s)
    i64 = lambda *s: skel.Container.empty(skel.I64, *s)
    st = torch.cuda.current_stream()
    calls = [
        (f32, (50, 60), lambda o, c, a, p: skel.skel_map(skel.MAP_AFFINE, p([2.0, 0.5]), [c(x)], o)),
        (f32, (1,), lambda o, c, a, p: skel.skel_reduce(skel.SUM, c(x), o)),
        (f32, (1,), lambda o, c, a, p: skel.skel_mapreduce(skel.MAP_AXPY, p([3]), (c(x), c(x)),
                                                           skel.MAX, o)),
        (f32, (50, 60), lambda o, c, a, p: skel.skel_mapoverlap1d(c(x), o, a(w1), 2,
                                                                  skel.EDGE_CONST, 0.25)),
        (f32, (50, 60), lambda o, c, a, p: skel.skel_mapoverlap1d_backward(c(x), o, a(w1), 2)),
        (f32, (50, 60), lambda o, c, a, p: skel.skel_mapoverlap2d(c(x), o, w2d=a(w2))),
        (f32, (50, 60), lambda o, c, a, p: skel.skel_mapoverlap2d_fields(c(x), o, 2, wy=a(wy),
                                                                         wx=a(wx))),
        (f32, (50, 60), lambda o, c, a, p: skel.skel_mapoverlap2d_backward(c(x), o, wy=a(wy),
                                                                           wx=a(wx), stream=st)),
        (f32, (50, 60), lambda o, c, a, p: skel.skel_mapoverlap2d_fields_backward(
            c(x), o, 5, w2d=a(w2), ry=1, rx=2)),
        (i64, (50, 60), lambda o, c, a, p: skel.skel_scan(c(k), o, skel.EXCLUSIVE, skel.SUM)),
        (i64, (50, 60), lambda o, c, a, p: skel.skel_scan_rows(c(k), o, skel.REVERSE_INCLUSIVE)),
        (f32, (4,), lambda o, c, a, p: skel.skel_reduce_segments(skel.MIN, c(x), off, o)),
    ]
    same = lambda v: v
    forms = [(same, same, same), (sub, f64, lambda p: [np.float64(v) for v in p]),
             (same, strided, tuple), (same, lambda a: a.tolist(), same)]
    for i, (make, shape, call) in enumerate(calls):
        got = []
        for c, a, p in forms:
            o = make(*shape)
            call(o, c, a, p)
            got.append(o.to_numpy())
        for g in got[1:]:
            assert np.array_equal(got[0], g), i
    # errors: the status of a call that the library refuses, the exceptions of
    # arguments that the binding refuses
    o = f32(50, 60)
    for bad in (lambda: skel.skel_map(skel.MAP_AXPY, [2.5], [x], o),
                lambda: skel.skel_map(skel.MAP_AXPY, np.array([2.5]), [x], o),
                lambda: skel.skel_mapoverlap2d(x, x, w2d=w2)):
        with pytest.raises(skel.SkelError) as e:
            bad()
        assert e.value.status == skel.E_INVAL
    with pytest.raises(ValueError):
        skel.skel_mapoverlap1d(x, o, w1, 3)
    with pytest.raises(ValueError):
        skel.skel_mapoverlap2d(x, o, wy=wy, wx=wx, ry=2)
    dead = f32(4)
    dead.destroy()
    with pytest.raises(TypeError):
        skel.skel_reduce(skel.SUM, dead, f32(1))


def test_containers_outlive_another_init(skel):
    """A container made before the library was initialised again still frees its memory
    through the callbacks it was made with."""
    import gc
    made = [skel.Container.from_numpy(np.ones(1000 + k, np.float32)) for k in range(8)]
    for c in made:  # device copies
        skel.skel_map(skel.MAP_AFFINE, [2.0, 0.0], [c], c)
    for _ in range(3):
        skel.skel_init(0, "torch")
        gc.collect()
    for c in made:
        assert np.all(c.to_numpy() == 2.0)
        c.destroy()
