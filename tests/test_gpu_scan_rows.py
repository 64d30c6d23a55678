"""GPU parity of the row-wise Scan (every row of a matrix scanned on its own)
against the oracle, through the C ABI, for both variants.

Bars as the flat Scan: integers bit-exact; float32 sums within
|y - y*| <= 1e-5 * (sum of |x| over the terms), float32 min/max exact.
"""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

RED_OPS = {"sum": 0, "min": 1, "max": 2}
KINDS = {"inclusive": 0, "exclusive": 1, "reverse_inclusive": 2, "reverse_exclusive": 3}
# widths around the one-wavefront chunk (2048), odd widths (element accesses),
# a long row (several chunks) and many short rows
SHAPES = [(1, 1), (3, 5), (7, 64), (5, 2048), (4, 2049), (2, 5000), (300, 7), (65, 4096),
          (2, (1 << 17) + 3), (1, 1 << 17)]
SR0, SR1 = 0, 1


def aligned(cols, in_size, out_size):
    return (cols * in_size) % 16 == 0 and (cols * out_size) % 16 == 0


def ints(g, shape, din):
    if din == np.int32:
        return g.integers(-2 ** 31, 2 ** 31, shape, dtype=np.int64).astype(np.int32)
    return g.integers(-2 ** 62, 2 ** 62, shape, dtype=np.int64)


@pytest.mark.parametrize("pair", ["i32_i32", "i32_i64", "i64_i64"])
@pytest.mark.parametrize("op", list(RED_OPS))
def test_scan_rows_int_bit_exact(skel, oracle_mod, pair, op):
    din, dout, sk_in, sk_out = {"i32_i32": (np.int32, np.int32, skel.I32, skel.I32),
                                "i32_i64": (np.int32, np.int64, skel.I32, skel.I64),
                                "i64_i64": (np.int64, np.int64, skel.I64, skel.I64)}[pair]
    for shape in SHAPES:
        x = ints(si.rng(21, shape[0] * 7919 + shape[1]), shape, din)
        cx = skel.Container.from_numpy(x)
        vs = [SR1] + ([SR0] if aligned(shape[1], x.itemsize, np.dtype(dout).itemsize) else [])
        for kind, code in KINDS.items():
            ref = oracle_mod.scan_rows(x, kind, op, dout)
            for v in vs:
                out = skel.Container.empty(sk_out, *shape)
                skel.skel_scan_rows(cx, out, code, RED_OPS[op], variant=v)
                got = out.to_numpy().reshape(shape)
                assert np.array_equal(got, ref), (pair, op, shape, kind, v,
                                                  np.argwhere(got != ref)[:5])
    skel.skel_sync()


@pytest.mark.parametrize("op", list(RED_OPS))
def test_scan_rows_f32(skel, oracle_mod, op):
    for shape in SHAPES:
        x = si.normal_f32(shape[0] * shape[1], 21, shape[1]).reshape(shape)
        cx = skel.Container.from_numpy(x)
        vs = [SR1] + ([SR0] if shape[1] % 4 == 0 else [])
        for kind, code in KINDS.items():
            ref, mag = oracle_mod.scan_rows(x, kind, op)
            for v in vs:
                out = skel.Container.empty(skel.F32, *shape)
                skel.skel_scan_rows(cx, out, code, RED_OPS[op], variant=v)
                got = out.to_numpy().reshape(shape).astype(np.float64)
                bad = np.abs(got - ref) > 1e-5 * mag + 1e-30 if op == "sum" else got != ref
                assert not bad.any(), (op, shape, kind, v, np.argwhere(bad)[:5])
    skel.skel_sync()


def test_scan_rows_in_place_and_errors(skel, oracle_mod):
    for shape in [(9, 2048), (9, 2047)]:
        x = si.int_uniform_i32(shape[0] * shape[1], 100, 21, 3).reshape(shape)
        c = skel.Container.from_numpy(x)
        skel.skel_scan_rows(c, c, skel.INCLUSIVE, skel.SUM)  # in place
        assert np.array_equal(c.to_numpy().reshape(shape), oracle_mod.scan_rows(x))
    # the per-row single-pass form needs 16-byte aligned rows
    x = np.ones((3, 6), np.int32)
    out = skel.Container.empty(skel.I64, 3, 6)
    with pytest.raises(skel.SkelError) as e:
        skel.skel_scan_rows(skel.Container.from_numpy(x), out, skel.INCLUSIVE, skel.SUM,
                            variant=SR0)
    assert e.value.status == skel.E_UNSUPPORTED
    with pytest.raises(skel.SkelError) as e:
        skel.skel_scan_rows(skel.Container.from_numpy(x), skel.Container.empty(skel.I64, 2, 9),
                            skel.INCLUSIVE, skel.SUM)
    assert e.value.status == skel.E_SHAPE
    skel.skel_sync()


def test_scan_rows_many_rows(skel, oracle_mod):
    # the field layout of the batched layer: many rows of 2048, widening
    shape = (8192, 2048)
    x = si.int_uniform_i32(shape[0] * shape[1], 1000, 21, 4).reshape(shape)
    cx = skel.Container.from_numpy(x)
    for kind in ("exclusive", "reverse_inclusive"):
        ref = oracle_mod.scan_rows(x, kind, "sum", np.int64)
        for v in (SR0, SR1):
            out = skel.Container.empty(skel.I64, *shape)
            skel.skel_scan_rows(cx, out, KINDS[kind], skel.SUM, variant=v)
            assert np.array_equal(out.to_numpy().reshape(shape), ref), (kind, v)
    skel.skel_sync()


def test_scan_rows_more_rows_than_one_grid(skel, oracle_mod):
    # the kernels step over rows in a grid of at most 2^20 workgroups; sampled
    # rows around that stride are checked against the oracle one by one
    for cols in (3, 4):  # element accesses, then 16-byte vectors
        rows = (1 << 20) + 5
        x = si.int_uniform_i32(rows * cols, 1000, 21, 5 + cols).reshape(rows, cols)
        out = skel.Container.empty(skel.I64, rows, cols)
        skel.skel_scan_rows(skel.Container.from_numpy(x), out, skel.EXCLUSIVE, skel.SUM,
                            variant=SR1)
        got = out.to_numpy().reshape(rows, cols)
        for r in (0, 1, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, rows - 1):
            assert np.array_equal(got[r], oracle_mod.scan(x[r], "exclusive", "sum", np.int64)), \
                (cols, r)
    skel.skel_sync()



def test_scan_rows_more_rows_than_one_launch_of_short_rows(skel):
    """2^29 rows of one element at 8 lanes each are more work items than one
    launch can number: they take two."""
    import torch
    rows = (1 << 29) + 3
    x = torch.empty(rows, 1, dtype=torch.int32, device="cuda").random_(-1000, 1000)
    y = torch.full_like(x, 7)
    cx, cy = skel.wrap_tensor(x), skel.wrap_tensor(y)
    skel.skel_scan_rows(cx, cy, skel.INCLUSIVE, skel.SUM, variant=SR1)
    assert torch.equal(x, y)
    skel.skel_scan_rows(cx, cy, skel.REVERSE_EXCLUSIVE, skel.SUM, variant=SR1)
    assert not y.any()
    skel.skel_sync()
    for c in (cx, cy):
        c.destroy()


from hypothesis import HealthCheck, given, settings, strategies as st  # noqa: E402


@settings(max_examples=60, deadline=None, suppress_health_check=list(HealthCheck))
@given(rows=st.integers(1, 40), cols=st.integers(1, 5000),
       pair=st.sampled_from(["i32_i32", "i32_i64", "i64_i64"]),
       kind=st.sampled_from(list(KINDS)), op=st.sampled_from(list(RED_OPS)),
       variant=st.sampled_from([SR0, SR1]), seed=st.integers(0, 1000))
def test_scan_rows_drawn_shapes(skel, oracle_mod, rows, cols, pair, kind, op, variant, seed):
    din, dout, sk_out = {"i32_i32": (np.int32, np.int32, skel.I32),
                         "i32_i64": (np.int32, np.int64, skel.I64),
                         "i64_i64": (np.int64, np.int64, skel.I64)}[pair]
    if variant == SR0 and not aligned(cols, np.dtype(din).itemsize, np.dtype(dout).itemsize):
        variant = SR1
    x = ints(si.rng(23, seed), (rows, cols), din)
    out = skel.Container.empty(sk_out, rows, cols)
    skel.skel_scan_rows(skel.Container.from_numpy(x), out, KINDS[kind], RED_OPS[op],
                        variant=variant)
    assert np.array_equal(out.to_numpy().reshape(rows, cols),
                          oracle_mod.scan_rows(x, kind, op, dout))


# the forms of the single launch: 8, 16 and 32 lanes per row, a wavefront per row
# with 1, 2, 4 and 8 vectors per lane, one workgroup of 4 and of 16 wavefronts per
# row, the flat look-back within rows, the decoupled look-back within rows -- each
# at its edges, rows at any alignment
FORM_SHAPES = [(9, 15), (33, 31), (70, 33), (130, 65), (31, 127), (9, 129), (70, 257), (41, 1023),
               (1030, 2047), (3, 4097), (700, 4099), (230, 8193), (40, 32769), (2, 500001),
               (90, 65537), (300, 32767)]


@pytest.mark.parametrize("pair", ["f32", "i32_i32", "i32_i64", "i64_i64"])
def test_scan_rows_forms(skel, oracle_mod, pair):
    din, dout, npd, npo = {"f32": (skel.F32, skel.F32, np.float32, np.float32),
                           "i32_i32": (skel.I32, skel.I32, np.int32, np.int32),
                           "i32_i64": (skel.I32, skel.I64, np.int32, np.int64),
                           "i64_i64": (skel.I64, skel.I64, np.int64, np.int64)}[pair]
    for rows, cols in FORM_SHAPES:
        if pair == "f32":
            x = si.normal_f32(rows * cols, 23, cols).reshape(rows, cols)
        else:
            x = si.int_uniform_i32(rows * cols, 1000, 23, cols).astype(npd).reshape(rows, cols)
        cx = skel.Container.from_numpy(x)
        for k, kind in enumerate(("inclusive", "exclusive", "reverse_inclusive",
                                  "reverse_exclusive")):
            out = skel.Container.empty(dout, rows, cols)
            skel.skel_scan_rows(cx, out, k, skel.SUM, variant=SR1)
            got = out.to_numpy().reshape(rows, cols)
            v = x[:, ::-1] if k >= 2 else x
            wide = np.cumsum(v, axis=1, dtype=np.float64 if pair == "f32" else np.int64)
            if k % 2:
                wide = wide - v
            ref = wide[:, ::-1] if k >= 2 else wide
            if pair == "f32":
                mag = np.cumsum(np.abs(v), axis=1, dtype=np.float64)
                mag = mag[:, ::-1] if k >= 2 else mag
                bad = np.abs(got - ref) > 1e-5 * mag + 1e-30
            else:
                bad = got != ref.astype(npo)
            assert not bad.any(), (pair, rows, cols, kind, np.argwhere(bad)[:3])
    skel.skel_sync()


@pytest.mark.parametrize("pair", ["f32", "i32_i32", "i32_i64", "i64_i64"])
@pytest.mark.parametrize("op", list(RED_OPS))
def test_scan_rows_around_a_wavefront(skel, oracle_mod, pair, op):
    """Rows of about 64 vectors, of 64 elements at a time, and their neighbours, aligned and not;
    more rows than wavefronts of the last workgroup."""
    din, dout, npd, npo = {"f32": (skel.F32, skel.F32, np.float32, np.float32),
                           "i32_i32": (skel.I32, skel.I32, np.int32, np.int32),
                           "i32_i64": (skel.I32, skel.I64, np.int32, np.int64),
                           "i64_i64": (skel.I64, skel.I64, np.int64, np.int64)}[pair]
    for rows, cols in ((5, 127), (6, 128), (7, 129), (9, 130), (9, 192), (11, 193), (5, 254),
                       (6, 255), (7, 256), (5, 257), (1025, 66), (1030, 127), (1025, 129),
                       (1027, 256)):
        x = (si.normal_f32(rows * cols, 25, cols).reshape(rows, cols) if pair == "f32"
             else ints(si.rng(25, cols), (rows, cols), npd))
        cx = skel.Container.from_numpy(x)
        for kind, code in KINDS.items():
            out = skel.Container.empty(dout, rows, cols)
            skel.skel_scan_rows(cx, out, code, RED_OPS[op], variant=SR1)
            got = out.to_numpy().reshape(rows, cols)
            if pair == "f32":
                ref, mag = oracle_mod.scan_rows(x, kind, op)
                bad = (np.abs(got.astype(np.float64) - ref) > 1e-5 * mag + 1e-30 if op == "sum"
                       else got != ref)
            else:
                bad = got != oracle_mod.scan_rows(x, kind, op, npo)
            assert not bad.any(), (pair, op, rows, cols, kind, np.argwhere(bad)[:3])
    skel.skel_sync()


@pytest.mark.parametrize("op", ["min", "max"])
def test_scan_rows_forms_min_max_in_place(skel, op):
    """In place; a NaN leaves the running minimum or maximum as it is."""
    fn = np.fmin if op == "min" else np.fmax
    for rows, cols in FORM_SHAPES:
        x = si.normal_f32(rows * cols, 24, cols).reshape(rows, cols)
        x[:, cols // 2] = np.nan
        x[:, 0] = np.inf if op == "max" else -np.inf
        c = skel.Container.from_numpy(x)
        skel.skel_scan_rows(c, c, skel.REVERSE_INCLUSIVE, skel.MIN if op == "min" else skel.MAX,
                            variant=SR1)
        ref = fn.accumulate(x[:, ::-1], axis=1)[:, ::-1]
        ident = np.float32(np.inf if op == "min" else -np.inf)
        ref = np.where(np.isnan(ref), ident, ref)
        assert np.array_equal(c.to_numpy().reshape(rows, cols), ref), (op, rows, cols)


def test_scan_rows_tiled_form_under_capture(skel):
    """A tiled shape whose descriptors were never allocated on the stream is
    served inside a capture by the form that needs none; repeated replays give
    the eager result."""
    import torch
    rows, cols = 90, 65537
    xt = torch.randint(0, 1000, (rows, cols), device="cuda", dtype=torch.int32)
    yt = torch.empty_like(xt)
    cx, cy = skel.wrap_tensor(xt), skel.wrap_tensor(yt)
    s = torch.cuda.Stream()
    small = skel.wrap_tensor(xt[:1, :100].contiguous())
    with torch.cuda.stream(s):  # the stream's workspace exists, its descriptors do not
        skel.skel_map(skel.MAP_IDENTITY, None, [skel.Container.from_numpy(np.ones(4, np.float32))],
                      skel.Container.empty(skel.F32, 4))
    torch.cuda.synchronize()
    want = torch.cumsum(xt.to(torch.int64), 1).to(torch.int32)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        skel.skel_scan_rows(cx, cy, skel.INCLUSIVE, skel.SUM, variant=SR1)
    for _ in range(3):
        yt.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(yt, want)
    with torch.cuda.stream(s):
        yt.zero_()
        skel.skel_scan_rows(cx, cy, skel.INCLUSIVE, skel.SUM, variant=SR1)
    torch.cuda.synchronize()
    assert torch.equal(yt, want)
    for c in (cx, cy, small):
        c.destroy()


def test_scan_rows_f32_sums_keep_their_bits(skel):
    """binary32 row sums are the same bits on every run and inside a captured graph,
    whichever form serves the shape (a workgroup per row, rows cut into chunks, a
    wavefront per row), beside a busy second stream too."""
    import torch
    s, other = torch.cuda.Stream(), torch.cuda.Stream()
    load = torch.randn(2048, 2048, device="cuda")
    torch.cuda.synchronize()
    for rows, cols in ((300, 5001), (40, 30000), (1, 32769), (40, 50001), (300, 100001),
                       (3, 1000003), (1, 5000009)):
        x = torch.randn(rows, cols, device="cuda")
        y = torch.empty_like(x)
        cx, cy = skel.wrap_tensor(x), skel.wrap_tensor(y)
        torch.cuda.synchronize()
        for kind in range(4):
            with torch.cuda.stream(s):
                skel.skel_scan_rows(cx, cy, kind, skel.SUM, variant=SR1)
                first = y.clone()
                for rep in range(6):
                    with torch.cuda.stream(other):
                        load.mul_(1.0)
                    y.fill_(float("nan"))
                    skel.skel_scan_rows(cx, cy, kind, skel.SUM, variant=SR1)
                    assert torch.equal(y, first), (rows, cols, kind, rep)
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                skel.skel_scan_rows(cx, cy, kind, skel.SUM, variant=SR1)
            for rep in range(3):
                y.fill_(float("nan"))
                torch.cuda.synchronize()
                g.replay()
                torch.cuda.synchronize()
                assert torch.equal(y, first), (rows, cols, kind, "replay", rep)
        for c in (cx, cy):
            c.destroy()
    skel.skel_sync()


def test_row_scans_leave_captured_scans_intact(skel):
    """A flat scan captured on a stream replays correctly after row scans on the
    same stream have enlarged the descriptor array: words left on the array that
    the graph uses never pass for a new call's."""
    import torch
    n = 5 * 32768 + 3
    xt = torch.randint(0, 1000, (n,), device="cuda", dtype=torch.int32)
    yt = torch.empty_like(xt)
    cx, cy = skel.wrap_tensor(xt), skel.wrap_tensor(yt)
    rows, cols = 700, 16 * 32768  # 700 x 16 tiles: more than the first array's words
    rx = torch.ones((rows, cols), device="cuda", dtype=torch.int32)
    crx = skel.wrap_tensor(rx)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        skel.skel_scan(cx, cy, skel.INCLUSIVE, skel.SUM, variant=2)
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        skel.skel_scan(cx, cy, skel.INCLUSIVE, skel.SUM, variant=2)
    with torch.cuda.stream(s):
        for _ in range(4):
            g.replay()
        skel.skel_scan_rows(crx, crx, skel.INCLUSIVE, skel.SUM, variant=SR1)
    torch.cuda.synchronize()
    assert int(rx[:, -1].min()) == cols == int(rx[:, -1].max())
    # the old array holds the tags of the 5th call; were the epoch counted anew
    # from the enlarging call, the next replay would be the 5th again
    with torch.cuda.stream(s):
        for _ in range(3):
            skel.skel_scan_rows(crx, crx, skel.INCLUSIVE, skel.MAX, variant=SR1)
    torch.cuda.synchronize()
    for k in range(3):
        xt.copy_(torch.randint(0, 1000, (n,), device="cuda", dtype=torch.int32))
        yt.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            g.replay()
        torch.cuda.synchronize()
        assert torch.equal(yt, torch.cumsum(xt.to(torch.int64), 0).to(torch.int32)), k
    for c in (cx, cy, crx):
        c.destroy()


def test_row_scans_beside_replays_of_the_streams_graphs(skel):
    """A graph captured on a stream and replayed on another one runs beside eager row
    scans on the first: they share no counters, descriptors or scratch."""
    import torch
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    n = (1 << 22) + 40961
    x = torch.randint(0, 1000, (n,), device="cuda", dtype=torch.int32)
    f = torch.randn(n, device="cuda")
    y, r = torch.empty_like(x), torch.empty(1, device="cuda")
    cx, cy, cf, cr = (skel.wrap_tensor(t) for t in (x, y, f, r))
    rows = [(torch.randint(0, 1000, s, device="cuda", dtype=d), torch.empty(s, device="cuda", dtype=d))
            for s, d in (((90, 65537), torch.int32), ((3, 1000003), torch.int32))]
    rows.append((torch.randn(200, 50001, device="cuda"), torch.empty(200, 50001, device="cuda")))
    crows = [(skel.wrap_tensor(p), skel.wrap_tensor(q)) for p, q in rows]
    torch.cuda.synchronize()

    def graphed():
        skel.skel_scan(cx, cy, skel.INCLUSIVE, skel.SUM, variant=2)
        skel.skel_scan(cx, cy, skel.INCLUSIVE, skel.SUM, variant=3)
        skel.skel_reduce(skel.SUM, cf, cr, variant=1)

    with torch.cuda.stream(a):
        graphed()
        for p, q in crows:
            skel.skel_scan_rows(p, q, skel.INCLUSIVE, skel.SUM, variant=SR1)
    torch.cuda.synchronize()
    want, total = y.clone(), r.clone()
    wrows = [q.clone() for _, q in rows]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=a):
        graphed()
    for rep in range(20):
        y.zero_(), r.zero_()
        for _, q in rows:
            q.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(b):
            g.replay()
        with torch.cuda.stream(a):
            for p, q in crows:
                skel.skel_scan_rows(p, q, skel.INCLUSIVE, skel.SUM, variant=SR1)
        torch.cuda.synchronize()
        assert torch.equal(y, want) and torch.equal(r, total), rep
        for (_, q), w in zip(rows, wrows):
            assert torch.equal(q, w), rep
    for c in (cx, cy, cf, cr, *(c for pq in crows for c in pq)):
        c.destroy()
    skel.skel_sync(a)
