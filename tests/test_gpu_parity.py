"""GPU parity: every skeleton variant of libskel against the CPU oracle on the
same seeded inputs, called through the C ABI (via the ctypes binding).

Bars (stated per skeleton in the oracle's definitions):
  * integer Reduce / Scan: bit-exact (wrapping in the output width);
  * Map: |y - y*| <= 1e-6 * (magnitude of the terms of f);
  * Reduce / MapReduce (floating point): |r - r*| <= 1e-5 * sum |terms|;
  * MapOverlap: |y - y*| <= 1e-6 * sum_k |w_k x_k| per output;
  * floating-point Scan: |y_i - y*_i| <= 1e-5 * sum_{j<=i} |x_j|;
  * MIN / MAX: exact.
Sizes span several tiles, ragged tails, empty and one-element inputs.
"""
import math

import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

SIZES = [0, 1, 3, 4, 5, 63, 64, 65, 255, 1000, 4095, 4096, 4097, 65537, (1 << 20) + 3]
MAP_OPS = {"identity": 0, "axpy": 1, "affine": 2, "tanh": 3, "affine_tanh": 4, "mul": 5,
           "square": 6}
RED_OPS = {"sum": 0, "min": 1, "max": 2}
EDGES = {"clamp": 0, "const": 1, "cyclic": 2}


def variants(skel, sk):
    return list(range(skel.skel_variant_count(sk)))


def cont(skel, arr, dtype=None):
    return skel.Container.from_numpy(arr, dtype)


def scalar_out(skel, dtype):
    return skel.Container.empty(dtype, 1)


# ----------------------------------------------------------------------- Map
def map_mag(op, p, x, y):
    """Magnitude scale of f's terms, the reference for the 1e-6 bound."""
    x = np.abs(x.astype(np.float64))
    y = np.abs(y.astype(np.float64)) if y is not None else 0
    if op == "identity":
        return x
    if op == "axpy":
        return abs(p[0]) * x + y
    if op == "affine":
        return abs(p[0]) * x + abs(p[1])
    if op == "tanh":
        return np.maximum(1, x)
    if op == "affine_tanh":
        return np.maximum(1, abs(p[0]) * x + abs(p[1]))
    if op == "mul":
        return x * y
    return x * x


@pytest.mark.parametrize("op", list(MAP_OPS))
def test_map(skel, oracle_mod, op):
    params = {"axpy": [2.5], "affine": [-1.5, 0.25], "affine_tanh": [0.75, -0.5]}.get(op, [])
    two = op in oracle_mod.TWO_INPUT_MAP_OPS
    for n in SIZES:
        x = si.uniform_f32(n, -1.0, 1.0, 0, 0) * np.float32(3)
        y = si.uniform_f32(n, -1.0, 1.0, 0, 1) if two else None
        ref = oracle_mod.map_f32(op, [np.float32(p) for p in params], x, y)
        tol = 1e-6 * map_mag(op, params, x, y) + 1e-30
        for v in variants(skel, skel.SK_MAP):
            cx = cont(skel, x)
            out = skel.Container.empty(skel.F32, n)
            ins = [cx, cont(skel, y)] if two else [cx]
            skel.skel_map(MAP_OPS[op], params, ins, out, variant=v)
            got = out.to_numpy().astype(np.float64)
            bad = np.abs(got - ref) > tol
            assert not bad.any(), (op, n, v, np.flatnonzero(bad)[:5])


def test_map_saxpy_bit_exact_and_in_place(skel, oracle_mod):
    # x, y on the 2^-23 grid: 2.5x + y is exact in binary64, so the fused
    # multiply-add's single rounding gives exactly fp32(oracle)
    n = (1 << 20) + 7
    x = si.uniform_f32(n, -1.0, 1.0, 0, 0)
    y = si.uniform_f32(n, -1.0, 1.0, 0, 1)
    want = oracle_mod.map_f32("axpy", [2.5], x, y).astype(np.float32)
    for v in variants(skel, skel.SK_MAP):
        cx, cy = cont(skel, x), cont(skel, y)
        skel.skel_map(skel.MAP_AXPY, [2.5], [cx, cy], cy, variant=v)  # in place
        assert np.array_equal(cy.to_numpy(), want), v


# -------------------------------------------------------------------- Reduce
def check_fp(got, ref, mag, rel=1e-5):
    assert abs(float(got) - ref) <= rel * mag + 1e-30, (got, ref, mag)


@pytest.mark.parametrize("op", list(RED_OPS))
def test_reduce_f32(skel, oracle_mod, op):
    for n in SIZES:
        x = si.normal_f32(n, 1, 2)
        ref = oracle_mod.reduce(op, x)
        mag = oracle_mod.abs_sum(x)
        for v in variants(skel, skel.SK_REDUCE):
            if v in (3, 4, 5) and op != "sum":  # atomic, compensated, pairwise: sums only
                with pytest.raises(skel.SkelError) as e:
                    skel.skel_reduce(RED_OPS[op], cont(skel, x), scalar_out(skel, skel.F32),
                                     variant=v)
                assert e.value.status == skel.E_UNSUPPORTED
                continue
            out = scalar_out(skel, skel.F32)
            skel.skel_reduce(RED_OPS[op], cont(skel, x), out, variant=v)
            got = out.to_numpy()[0]
            if op == "sum":
                check_fp(got, ref, mag)
            else:
                assert float(got) == ref, (op, n, v)


@pytest.mark.parametrize("n", [1, 64, 65536, 1 << 20, 1 << 24])
def test_reduce_sum_of_indices(skel, n):
    # sum_{i<n} i = n(n-1)/2; binary32 holds every i exactly for n <= 2^24
    exact = n * (n - 1) // 2
    xi = np.arange(n, dtype=np.int32)
    for v in variants(skel, skel.SK_REDUCE):
        if v not in (4, 5):  # compensated and pairwise: floating point only
            o32, o64 = scalar_out(skel, skel.I32), scalar_out(skel, skel.I64)
            skel.skel_reduce(skel.SUM, cont(skel, xi), o32, variant=v)
            skel.skel_reduce(skel.SUM, cont(skel, xi), o64, variant=v)
            assert int(o64.to_numpy()[0]) == exact
            assert int(o32.to_numpy()[0]) == ((exact + 2 ** 31) % 2 ** 32) - 2 ** 31
        of = scalar_out(skel, skel.F32)
        skel.skel_reduce(skel.SUM, cont(skel, xi.astype(np.float32)), of, variant=v)
        assert abs(float(of.to_numpy()[0]) - exact) <= 1e-5 * exact


@pytest.mark.parametrize("pair", ["i32_i32", "i32_i64", "i64_i64"])
@pytest.mark.parametrize("op", list(RED_OPS))
def test_reduce_int_bit_exact(skel, oracle_mod, pair, op):
    din, dout = {"i32_i32": (skel.I32, skel.I32), "i32_i64": (skel.I32, skel.I64),
                 "i64_i64": (skel.I64, skel.I64)}[pair]
    for n in SIZES:
        g = si.rng(7, n)
        if din == skel.I32:
            x = g.integers(-2 ** 31, 2 ** 31, n, dtype=np.int64).astype(np.int32)
        else:
            x = g.integers(-2 ** 62, 2 ** 62, n, dtype=np.int64)
        ref = oracle_mod.reduce(op, x, np.int64 if dout == skel.I64 else np.int32)
        for v in variants(skel, skel.SK_REDUCE):
            out = scalar_out(skel, dout)
            if v in (4, 5):
                with pytest.raises(skel.SkelError) as e:
                    skel.skel_reduce(RED_OPS[op], cont(skel, x), out, variant=v)
                assert e.value.status == skel.E_UNSUPPORTED
                continue
            skel.skel_reduce(RED_OPS[op], cont(skel, x), out, variant=v)
            assert int(out.to_numpy()[0]) == ref, (pair, op, n, v)


def test_reduce_deterministic_variants(skel):
    x = si.normal_f32((1 << 22) + 11, 1, 9)
    for v in (0, 1, 2, 4, 5):
        vals = set()
        for _ in range(3):
            out = scalar_out(skel, skel.F32)
            skel.skel_reduce(skel.SUM, cont(skel, x), out, variant=v)
            vals.add(out.to_numpy()[0].tobytes())
        assert len(vals) == 1, v


# ----------------------------------------------------------------- MapReduce
@pytest.mark.parametrize("mop", ["mul", "square", "identity", "axpy", "affine_tanh"])
@pytest.mark.parametrize("op", list(RED_OPS))
def test_mapreduce_f32(skel, oracle_mod, mop, op):
    params = {"axpy": [2.5], "affine_tanh": [0.5, 0.125]}.get(mop, [])
    two = mop in oracle_mod.TWO_INPUT_MAP_OPS
    for n in SIZES:
        x = si.normal_f32(n, 1, 0)
        y = si.normal_f32(n, 1, 1) if two else None
        ref, mag = oracle_mod.mapreduce(mop, params, x, y, op)
        if op != "sum":
            # min/max of f32 element results: compare with the f32-rounded values
            vals = oracle_mod.map_f32(mop, params, x, y)
            tol = 1e-6 * (np.max(map_mag(mop, params, x, y)) if n else 0)
        for v in variants(skel, skel.SK_MAPREDUCE):
            out = scalar_out(skel, skel.F32)
            ins = [cont(skel, x), cont(skel, y)] if two else [cont(skel, x)]
            if v in (4, 5) and op != "sum":  # compensated, pairwise: sums only
                with pytest.raises(skel.SkelError) as e:
                    skel.skel_mapreduce(MAP_OPS[mop], params, ins, RED_OPS[op], out,
                                        variant=v)
                assert e.value.status == skel.E_UNSUPPORTED
                continue
            skel.skel_mapreduce(MAP_OPS[mop], params, ins, RED_OPS[op], out, variant=v)
            got = float(out.to_numpy()[0])
            if op == "sum":
                check_fp(got, ref, mag)
            elif n == 0:
                assert got == ref
            else:
                assert abs(got - ref) <= tol + 1e-30, (mop, op, n, v, got, ref)


def test_mapreduce_bf16_inputs(skel, oracle_mod):
    for n in (0, 1, 7, 8, 9, 4097, (1 << 20) + 5):
        xb = si.log_uniform_signed_bf16(n, config=4, index=1)
        yb = si.log_uniform_signed_bf16(n, config=4, index=2)
        xf, yf = si.bf16_bits_to_f32(xb), si.bf16_bits_to_f32(yb)
        ref, mag = oracle_mod.mapreduce("mul", None, xf, yf)
        rsum = oracle_mod.reduce("sum", xf)
        asum = oracle_mod.abs_sum(xf)
        for v in (1, 2, 3, 4, 5):
            out = scalar_out(skel, skel.F32)
            skel.skel_mapreduce(skel.MAP_MUL, None, [cont(skel, xb, skel.BF16),
                                                     cont(skel, yb, skel.BF16)],
                                skel.SUM, out, variant=v)
            check_fp(out.to_numpy()[0], ref, mag)
        for v in variants(skel, skel.SK_REDUCE):
            out = scalar_out(skel, skel.F32)
            skel.skel_reduce(skel.SUM, cont(skel, xb, skel.BF16), out, variant=v)
            check_fp(out.to_numpy()[0], rsum, asum)
        with pytest.raises(skel.SkelError):  # the unfused form maps in f32 only
            skel.skel_mapreduce(skel.MAP_MUL, None, [cont(skel, xb, skel.BF16),
                                                     cont(skel, yb, skel.BF16)],
                                skel.SUM, scalar_out(skel, skel.F32), variant=0)


def test_mapreduce_identities(skel, oracle_mod):
    n = (1 << 20) + 1
    x = si.normal_f32(n, 1, 3)
    e = np.zeros(n, np.float32)
    e[12345] = 1
    out = scalar_out(skel, skel.F32)
    skel.skel_mapreduce(skel.MAP_MUL, None, [cont(skel, e), cont(skel, x)], skel.SUM, out)
    assert out.to_numpy()[0] == x[12345]
    out2 = scalar_out(skel, skel.F32)
    skel.skel_mapreduce(skel.MAP_MUL, None, [cont(skel, x), cont(skel, np.ones_like(x))],
                        skel.SUM, out2)
    check_fp(out2.to_numpy()[0], oracle_mod.reduce("sum", x), oracle_mod.abs_sum(x))


# ---------------------------------------------------------------- MapOverlap
@pytest.mark.parametrize("edge", list(EDGES))
@pytest.mark.parametrize("r", [0, 1, 2, 4, 7])
def test_mapoverlap1d(skel, oracle_mod, edge, r):
    w = si.uniform_f32(2 * r + 1, -1.0, 1.0, 3, r)
    for n in (1, 2, 5, 17, 1000, 1023, 1024, 1025, 4099, (1 << 20) + 2):
        x = si.uniform_f32(n, -1.0, 1.0, 0, 3)
        ref, mag = oracle_mod.mapoverlap1d(x, w, r, edge, 0.625)
        for v in variants(skel, skel.SK_MAPOVERLAP1D):
            out = skel.Container.empty(skel.F32, n)
            if v == 2 and r > 4:  # cross-lane variant reaches 4 neighbours per side
                with pytest.raises(skel.SkelError) as e:
                    skel.skel_mapoverlap1d(cont(skel, x), out, w, r, EDGES[edge], 0.625,
                                           variant=v)
                assert e.value.status == skel.E_UNSUPPORTED
                continue
            skel.skel_mapoverlap1d(cont(skel, x), out, w, r, EDGES[edge], 0.625, variant=v)
            got = out.to_numpy().astype(np.float64)
            bad = np.abs(got - ref) > 1e-6 * mag + 1e-30
            assert not bad.any(), (edge, r, n, v, np.flatnonzero(bad)[:5])


SHAPES_2D = [(1, 1), (1, 17), (13, 1), (3, 5), (64, 64), (65, 63), (100, 130), (257, 300)]
RADII_2D = [(4, 4), (1, 1), (2, 2), (3, 1), (0, 2), (8, 8)]


@pytest.mark.parametrize("edge", list(EDGES))
@pytest.mark.parametrize("r", [3, 5, 8, 31, 63, 64])
def test_mapoverlap1d_window(skel, oracle_mod, edge, r):
    """The LDS window (O1b) and the transpose that runs it: both tile sizes
    (256 and 1024 outputs) at their edges, arrays shorter than the radius, both
    remainders of 2r + 1 by four taps.  At most 2r + 1 fused multiply-adds in
    turn, and an end element's coefficients and lane sums rounded once more:
    2r + 4 roundings of 2^-24 of the terms' magnitude."""
    v = skel.variant_index(skel.SK_MAPOVERLAP1D, "O1b_lds_tile")
    w = si.uniform_f32(2 * r + 1, -1.0, 1.0, 31, r)
    tol = (2 * r + 4) * 2.0 ** -24
    for n in (1, 2, r, r + 1, 255, 256, 257, 1000, 256 * 5 + 2, (1 << 17) + 1, (1 << 17) + 1024 + r):
        x = si.uniform_f32(n, -1.0, 1.0, 31, 100)
        y, dx = skel.Container.empty(skel.F32, n), skel.Container.empty(skel.F32, n)
        skel.skel_mapoverlap1d(cont(skel, x), y, w, r, EDGES[edge], pad=0.25, variant=v)
        skel.skel_mapoverlap1d_backward(cont(skel, x), dx, w, r, EDGES[edge])
        for got, (ref, mag) in ((y, oracle_mod.mapoverlap1d(x, w, r, edge, 0.25)),
                                (dx, oracle_mod.mapoverlap1d_adjoint(x, w, r, edge))):
            bad = np.abs(got.to_numpy().astype(np.float64) - ref) > tol * mag + 1e-30
            assert not bad.any(), (edge, r, n, got is dx, np.flatnonzero(bad)[:5])


@pytest.mark.parametrize("edge", list(EDGES))
@pytest.mark.parametrize("ry,rx", RADII_2D)
def test_mapoverlap2d(skel, oracle_mod, edge, ry, rx):
    wy = si.uniform_f32(2 * ry + 1, 0.0, 1.0, 3, 10 + ry)
    wx = si.uniform_f32(2 * rx + 1, -1.0, 1.0, 3, 20 + rx)
    w2d = si.uniform_f32((2 * ry + 1) * (2 * rx + 1), -1.0, 1.0, 3, 30).reshape(
        2 * ry + 1, 2 * rx + 1)
    for shape in SHAPES_2D:
        x = si.uniform_f32(shape[0] * shape[1], 0.0, 1.0, 1, shape[0]).reshape(shape)
        for sep in (True, False):
            kw = dict(wy=wy, wx=wx) if sep else dict(w2d=w2d)
            ref, mag = oracle_mod.mapoverlap2d(x, ry, rx, edge=edge, pad=-0.25, **kw)
            for v in variants(skel, skel.SK_MAPOVERLAP2D):
                if v in (2, 3) and not sep:  # separable variants
                    continue
                if v == 4 and max(ry, rx) > 4:  # marching window: radii up to 4
                    continue
                out = skel.Container.empty(skel.F32, shape[0], shape[1])
                skel.skel_mapoverlap2d(cont(skel, x), out, ry=ry, rx=rx, edge=EDGES[edge],
                                       pad=-0.25, variant=v, **kw)
                got = out.to_numpy().reshape(shape).astype(np.float64)
                bad = np.abs(got - ref) > 1e-6 * mag + 1e-30
                assert not bad.any(), (edge, ry, rx, shape, sep, v, np.argwhere(bad)[:5])


# The marching-window variant's straight-line path runs for whole 256-column
# strips of images with at least 4 rows: rows beyond the image ends and the
# chunks beyond a row's two ends are mapped by the edge rule without branches.
# These shapes put strips at both row ends (widths that are multiples of 256),
# a ragged last strip (260, 772), images of 4 and 5 rows (rows wrapped or
# clamped up to 4 away) and strips that end mid-strip in height.
# images at the edges of the 64-column tiles of 16 rows, unaligned rows
TILE_SHAPES = [(1, 70), (70, 1), (2, 2), (15, 63), (16, 64), (17, 65), (33, 130), (100, 333)]
TILE_RADII = [(0, 0), (0, 3), (3, 0), (1, 2), (5, 5), (2, 6), (7, 7), (8, 1), (8, 8)]


@pytest.mark.parametrize("edge", list(EDGES))
@pytest.mark.parametrize("ry,rx", TILE_RADII)
def test_mapoverlap2d_tiles_and_transpose(skel, oracle_mod, edge, ry, rx):
    """The LDS tiles for every column radius, and the transpose whose border
    pixels run beside the tiles: each output is at most (2ry+1)(2rx+1) fused
    multiply-adds in turn (a row and a column pass for factors), and a border
    pixel's coefficients are sums of weights rounded in turn: that many
    roundings of 2^-24 of the terms' magnitude, and eight more."""
    wy = si.uniform_f32(2 * ry + 1, -1.0, 1.0, 51, ry)
    wx = si.uniform_f32(2 * rx + 1, -1.0, 1.0, 51, 20 + rx)
    w2d = si.uniform_f32((2 * ry + 1) * (2 * rx + 1), -1.0, 1.0, 51, 40).reshape(2 * ry + 1, -1)
    tol = ((2 * ry + 1) * (2 * rx + 1) + 8) * 2.0 ** -24
    for shape in TILE_SHAPES:
        x = si.uniform_f32(shape[0] * shape[1], -1.0, 1.0, 51, 60).reshape(shape)
        for names, kw in ((["O2b_lds_tile"], {"w2d": w2d}),
                          (["O2c_lds_separable", "O2d_separable_l1"], {"wy": wy, "wx": wx})):
            ref, mag = oracle_mod.mapoverlap2d(x, ry, rx, edge=edge, pad=0.5, **kw)
            for name in names:
                out = skel.Container.empty(skel.F32, *shape)
                skel.skel_mapoverlap2d(cont(skel, x), out, ry=ry, rx=rx, edge=EDGES[edge], pad=0.5,
                                       variant=skel.variant_index(skel.SK_MAPOVERLAP2D, name), **kw)
                got = out.to_numpy().reshape(shape).astype(np.float64)
                bad = np.abs(got - ref) > tol * mag + 1e-30
                assert not bad.any(), (edge, ry, rx, shape, name, np.argwhere(bad)[:3])
            ref, mag = oracle_mod.mapoverlap2d_adjoint(x, ry, rx, edge=edge, **kw)
            out = skel.Container.empty(skel.F32, *shape)
            skel.skel_mapoverlap2d_backward(cont(skel, x), out, ry=ry, rx=rx, edge=EDGES[edge], **kw)
            got = out.to_numpy().reshape(shape).astype(np.float64)
            bad = np.abs(got - ref) > tol * mag + 1e-30
            assert not bad.any(), (edge, ry, rx, shape, "transpose", np.argwhere(bad)[:3])


@pytest.mark.parametrize("mirror", ["both", "rows", "cols"])
@pytest.mark.parametrize("ry,rx", [(1, 1), (0, 1), (1, 0), (0, 0), (1, 2), (2, 1)])
def test_mapoverlap2d_transpose_of_mirrored_weights(skel, oracle_mod, ry, rx, mirror):
    """Weights that mirror along both axes make a clamped map of radii up to 1
    its own transpose; along one axis only, or beyond radius 1, they do not.
    Tolerance as for the tiles, on images of one tile and of marching strips."""
    ny, nx = 2 * ry + 1, 2 * rx + 1
    w2d = si.uniform_f32(ny * nx, -1.0, 1.0, 53, 1).reshape(ny, nx)
    wy, wx = si.uniform_f32(ny, -1.0, 1.0, 53, 2), si.uniform_f32(nx, -1.0, 1.0, 53, 3)
    if mirror != "cols":
        w2d, wy = np.maximum(w2d, w2d[::-1]), np.maximum(wy, wy[::-1])
    if mirror != "rows":
        w2d, wx = np.maximum(w2d, w2d[:, ::-1]), np.maximum(wx, wx[::-1])
    tol = (ny * nx + 8) * 2.0 ** -24
    for shape, fields in (((1, 70), 1), ((70, 1), 1), ((2, 2), 1), ((17, 65), 3), ((12, 1024), 90)):
        x = si.uniform_f32(fields * shape[0] * shape[1], -1.0, 1.0, 53, 4)
        x = x.reshape(fields * shape[0], shape[1])
        for kw in ({"w2d": w2d}, {"wy": wy, "wx": wx}):
            out = skel.Container.empty(skel.F32, *x.shape)
            skel.skel_mapoverlap2d_fields_backward(cont(skel, x), out, fields, ry=ry, rx=rx,
                                                   edge=EDGES["clamp"], **kw)
            got = out.to_numpy().reshape(x.shape).astype(np.float64)
            for f in (0, fields - 1):
                part = slice(f * shape[0], (f + 1) * shape[0])
                ref, mag = oracle_mod.mapoverlap2d_adjoint(x[part], ry, rx, edge="clamp", **kw)
                bad = np.abs(got[part] - ref) > tol * mag + 1e-30
                assert not bad.any(), (shape, f, list(kw), np.argwhere(bad)[:3])


@pytest.mark.parametrize("sep", [False, True])
def test_mapoverlap2d_two_row_tiles(skel, oracle_mod, sep):
    """2^23 pixels and more: two rows per lane; unaligned rows, a ragged last
    tile.  Compared with the oracle on sampled rows."""
    rows, cols, r = 2900, 2903, 3
    wy, wx = si.uniform_f32(7, 0.0, 1.0, 52, 1), si.uniform_f32(7, -1.0, 1.0, 52, 2)
    kw = {"wy": wy, "wx": wx} if sep else {"w2d": si.uniform_f32(49, -1.0, 1.0, 52, 3).reshape(7, 7)}
    x = si.uniform_f32(rows * cols, -1.0, 1.0, 52, 4).reshape(rows, cols)
    out, dx = skel.Container.empty(skel.F32, rows, cols), skel.Container.empty(skel.F32, rows, cols)
    skel.skel_mapoverlap2d(cont(skel, x), out, ry=r, rx=r, edge=EDGES["clamp"], **kw)
    skel.skel_mapoverlap2d_backward(cont(skel, x), dx, ry=r, rx=r, edge=EDGES["clamp"], **kw)
    tol = (49 + 8) * 2.0 ** -24
    for fn, got in ((oracle_mod.mapoverlap2d, out), (oracle_mod.mapoverlap2d_adjoint, dx)):
        got = got.to_numpy().reshape(rows, cols).astype(np.float64)
        for a, b in ((0, 40), (1440, 1480), (rows - 40, rows)):
            # a band of the image with its own halo is exact away from the cut
            lo, hi = max(0, a - 2 * r), min(rows, b + 2 * r)
            ref, mag = fn(x[lo:hi], r, r, edge="clamp", **kw)
            s = slice(r if lo else 0, (hi - lo) - (r if hi < rows else 0))
            bad = np.abs(got[lo:hi][s] - ref[s]) > tol * mag[s] + 1e-30
            assert not bad.any(), (sep, a, np.argwhere(bad)[:3])


MARCH_SHAPES = [(4, 256), (5, 512), (37, 768), (70, 1024), (20, 260), (9, 772)]
MARCH_RADII = [(1, 1), (2, 2), (4, 4), (3, 1), (0, 2), (4, 0)]


@pytest.mark.parametrize("edge", list(EDGES))
@pytest.mark.parametrize("ry,rx", MARCH_RADII)
def test_mapoverlap2d_march_paths(skel, oracle_mod, edge, ry, rx):
    v = skel.variant_index(skel.SK_MAPOVERLAP2D, "O2e_march")
    wy = si.uniform_f32(2 * ry + 1, -1.0, 1.0, 41, 10 + ry)
    wx = si.uniform_f32(2 * rx + 1, -1.0, 1.0, 41, 20 + rx)
    w2d = si.uniform_f32((2 * ry + 1) * (2 * rx + 1), -1.0, 1.0, 41, 30).reshape(
        2 * ry + 1, 2 * rx + 1)
    for shape in MARCH_SHAPES:
        x = si.uniform_f32(shape[0] * shape[1], -1.0, 1.0, 42, shape[1]).reshape(shape)
        for kw in (dict(w2d=w2d), dict(wy=wy, wx=wx)):
            ref, mag = oracle_mod.mapoverlap2d(x, ry, rx, edge=edge, pad=0.625, **kw)
            out = skel.Container.empty(skel.F32, shape[0], shape[1])
            skel.skel_mapoverlap2d(cont(skel, x), out, ry=ry, rx=rx, edge=EDGES[edge],
                                   pad=0.625, variant=v, **kw)
            got = out.to_numpy().reshape(shape).astype(np.float64)
            bad = np.abs(got - ref) > 1e-6 * mag + 1e-30
            assert not bad.any(), (edge, ry, rx, shape, list(kw), np.argwhere(bad)[:5])


@pytest.mark.parametrize("edge", list(EDGES))
@pytest.mark.parametrize("ry,rx", [(1, 1), (2, 2), (1, 2), (0, 2), (3, 1)])
def test_mapoverlap2d_march_ragged(skel, oracle_mod, edge, ry, rx):
    """Rows that are not whole vectors, strips past a ragged row end, heights below, at
    and past the 16 rows of a strip."""
    v = skel.variant_index(skel.SK_MAPOVERLAP2D, "O2e_march")
    wy, wx = (si.uniform_f32(2 * r + 1, -1.0, 1.0, 44, 10 + r) for r in (ry, rx))
    w2d = si.uniform_f32((2 * ry + 1) * (2 * rx + 1), -1.0, 1.0, 44, 30).reshape(2 * ry + 1, -1)
    for rows in (12, 16, 37):
        for cols in (261, 515, 1001):
            x = si.uniform_f32(rows * cols, -1.0, 1.0, 45, cols).reshape(rows, cols)
            for kw in (dict(w2d=w2d), dict(wy=wy, wx=wx)):
                ref, mag = oracle_mod.mapoverlap2d(x, ry, rx, edge=edge, pad=0.625, **kw)
                out = skel.Container.empty(skel.F32, rows, cols)
                skel.skel_mapoverlap2d(cont(skel, x), out, ry=ry, rx=rx, edge=EDGES[edge],
                                       pad=0.625, variant=v, **kw)
                got = out.to_numpy().reshape(rows, cols).astype(np.float64)
                bad = np.abs(got - ref) > 1e-6 * mag + 1e-30
                assert not bad.any(), (edge, ry, rx, rows, cols, list(kw), np.argwhere(bad)[:5])


@pytest.mark.parametrize("variant,r", [("O2c_lds_separable", 2), ("O2c_lds_separable", 8),
                                       ("O2d_separable_l1", 5), ("O2b_lds_tile", 8)])
def test_mapoverlap2d_two_row_tile_forms(skel, oracle_mod, variant, r):
    """The forms with two rows per lane (2^23 pixels and more) and their widest halos,
    compared with the oracle on bands of rows."""
    rows, cols = 2900, 2903
    wy, wx = si.uniform_f32(2 * r + 1, 0.0, 1.0, 53, 1), si.uniform_f32(2 * r + 1, -1.0, 1.0, 53, 2)
    kw = {"wy": wy, "wx": wx} if "separable" in variant else {"w2d": np.outer(wy, wx)}
    x = si.uniform_f32(rows * cols, -1.0, 1.0, 53, 4).reshape(rows, cols)
    out = skel.Container.empty(skel.F32, rows, cols)
    skel.skel_mapoverlap2d(cont(skel, x), out, ry=r, rx=r, edge=EDGES["cyclic"],
                           variant=skel.variant_index(skel.SK_MAPOVERLAP2D, variant), **kw)
    got = out.to_numpy().reshape(rows, cols).astype(np.float64)
    tol = ((2 * r + 1) ** 2 + 8) * 2.0 ** -24
    for a, b in ((0, 20), (1440, 1470), (rows - 20, rows)):
        band = np.take(x, np.arange(a - r, b + r), axis=0, mode="wrap")  # with its halo
        ref, mag = oracle_mod.mapoverlap2d(band, r, r, edge="cyclic", **kw)
        bad = np.abs(got[a:b] - ref[r:-r]) > tol * mag[r:-r] + 1e-30
        assert not bad.any(), (variant, r, a, np.argwhere(bad)[:3])


def test_mapoverlap_constant_field_and_impulse(skel):
    g = si.gaussian_weights(4, 2.0)
    sw = math.fsum(float(v) for v in g)
    c = np.float32(0.75)
    x = np.full((129, 257), c, np.float32)
    for v in variants(skel, skel.SK_MAPOVERLAP2D):
        out = skel.Container.empty(skel.F32, 129, 257)
        skel.skel_mapoverlap2d(cont(skel, x), out, wy=g, wx=g, variant=v)
        got = out.to_numpy().astype(np.float64)
        assert np.all(np.abs(got - float(c) * sw * sw) <= 1e-6), v
    # impulse: the response is W flipped in both axes (correlation orientation)
    w = np.arange(1, 16, dtype=np.float32).reshape(3, 5)
    x = np.zeros((9, 11), np.float32)
    x[4, 5] = 1
    for v in (0, 1):
        out = skel.Container.empty(skel.F32, 9, 11)
        skel.skel_mapoverlap2d(cont(skel, x), out, w2d=w, variant=v)
        got = out.to_numpy()
        assert np.array_equal(got[3:6, 3:8], w[::-1, ::-1]), v
        assert np.count_nonzero(got) == 15


# ---------------------------------------------------------------------- Scan
# tiles are 32768 elements for 4-byte inputs and 16384 for 8-byte inputs
SCAN_SIZES = [0, 1, 2, 63, 64, 65, 2047, 2049, 8193, 16383, 16384, 16385, 32767, 32768,
              32769, 3 * 32768 + 5, 70000, (1 << 20) + 3]


@pytest.mark.parametrize("pair", ["i32_i32", "i32_i64", "i64_i64"])
@pytest.mark.parametrize("kind", ["inclusive", "exclusive"])
@pytest.mark.parametrize("op", list(RED_OPS))
def test_scan_int_bit_exact(skel, oracle_mod, pair, kind, op):
    din, dout = {"i32_i32": (skel.I32, skel.I32), "i32_i64": (skel.I32, skel.I64),
                 "i64_i64": (skel.I64, skel.I64)}[pair]
    K = {"inclusive": skel.INCLUSIVE, "exclusive": skel.EXCLUSIVE}[kind]
    for n in SCAN_SIZES:
        g = si.rng(8, n)
        if din == skel.I32:
            x = g.integers(-2 ** 31, 2 ** 31, n, dtype=np.int64).astype(np.int32)
        else:
            x = g.integers(-2 ** 62, 2 ** 62, n, dtype=np.int64)
        ref = oracle_mod.scan(x, kind, op, np.int64 if dout == skel.I64 else np.int32)
        for v in variants(skel, skel.SK_SCAN):
            out = skel.Container.empty(dout, n)
            skel.skel_scan(cont(skel, x), out, K, RED_OPS[op], variant=v)
            got = out.to_numpy()
            assert np.array_equal(got, ref), (pair, kind, op, n, v,
                                              np.flatnonzero(got != ref)[:5])
    skel.skel_sync()


@pytest.mark.parametrize("kind", ["inclusive", "exclusive"])
@pytest.mark.parametrize("op", list(RED_OPS))
def test_scan_f32(skel, oracle_mod, kind, op):
    K = {"inclusive": skel.INCLUSIVE, "exclusive": skel.EXCLUSIVE}[kind]
    for n in SCAN_SIZES:
        x = si.normal_f32(n, 3, 1)
        ref, mag = oracle_mod.scan(x, kind, op)
        for v in variants(skel, skel.SK_SCAN):
            out = skel.Container.empty(skel.F32, n)
            skel.skel_scan(cont(skel, x), out, K, RED_OPS[op], variant=v)
            got = out.to_numpy().astype(np.float64)
            if op == "sum":
                bad = np.abs(got - ref) > 1e-5 * mag + 1e-30
            else:
                bad = got != ref
            assert not bad.any(), (kind, op, n, v, np.flatnonzero(bad)[:5])
    skel.skel_sync()


def test_scan_in_place_and_closed_forms(skel, oracle_mod):
    n = (1 << 20) + 9
    ones = np.ones(n, np.int32)
    for v in variants(skel, skel.SK_SCAN):
        c = cont(skel, ones)
        skel.skel_scan(c, c, skel.INCLUSIVE, skel.SUM, variant=v)  # in place
        assert np.array_equal(c.to_numpy(), np.arange(1, n + 1, dtype=np.int32)), v
        x = si.int_uniform_i32(n, 100, 0, 7)
        inc, red = skel.Container.empty(skel.I64, n), scalar_out(skel, skel.I64)
        skel.skel_scan(cont(skel, x), inc, skel.INCLUSIVE, skel.SUM, variant=v)
        skel.skel_reduce(skel.SUM, cont(skel, x), red)
        assert inc.to_numpy()[-1] == red.to_numpy()[0]
    skel.skel_sync()


# ragged sizes past S3's middle ones, whose tiles are flat: its persistent workgroups
# loop over tile ids there
@pytest.mark.parametrize("pair", ["f32", "i32_i32", "i32_i64", "i64_i64"])
@pytest.mark.parametrize("op", list(RED_OPS))
def test_scan_persistent_lookback(skel, pair, op):
    import torch
    din, dout = {"f32": (torch.float32,) * 2, "i32_i32": (torch.int32,) * 2,
                 "i32_i64": (torch.int32, torch.int64), "i64_i64": (torch.int64,) * 2}[pair]
    for n in ((1 << 22) + (1 << 20) + 5, (1 << 23) + 32771, 20 * (1 << 20) + 1):
        if n < 1 << 23 and din != torch.int64:
            continue
        x = (torch.randn(n, device="cuda") if din == torch.float32 else
             torch.randint(-1000, 1000, (n,), device="cuda", dtype=din))
        y = torch.empty(n, device="cuda", dtype=dout)
        cx, cy = skel.wrap_tensor(x), skel.wrap_tensor(y)
        for kind in range(4):
            y.fill_(-7)
            skel.skel_scan(cx, cy, kind, RED_OPS[op], variant=3)
            v = x.flip(0) if kind >= 2 else x
            wide = torch.float64 if din == torch.float32 else torch.int64
            if op == "sum":
                ref = v.to(wide).cumsum(0)
                if kind % 2:
                    ref = ref - v
            else:
                ref = (v.to(wide).cummin(0) if op == "min" else v.to(wide).cummax(0)).values
                if kind % 2:  # the first element is the identity
                    ref = torch.cat([ref[:1], ref[:-1]])
            got = y.flip(0) if kind >= 2 else y
            first = 1 if kind % 2 and op != "sum" else 0
            if din == torch.float32 and op == "sum":
                bad = (got - ref).abs() > 1e-5 * v.abs().double().cumsum(0)
            else:
                bad = got.to(wide) != ref
                if dout == torch.int32:
                    bad = got != ref.to(torch.int32)
            assert not bool(bad[first:].any()), (pair, op, n, kind)
        for c in (cx, cy):
            c.destroy()
    skel.skel_sync()


def test_scan_persistent_lookback_in_a_graph(skel):
    """The persistent workgroups' counters are reset on the device: replays, with
    eager calls of the same kind between them, give the eager result."""
    import torch
    n = (1 << 23) + 32771
    x = torch.randint(0, 1000, (n,), device="cuda", dtype=torch.int32)
    y, z = torch.empty_like(x), torch.empty_like(x)
    s = torch.cuda.Stream()
    cx, cy, cz = (skel.wrap_tensor(t, s) for t in (x, y, z))
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        skel.skel_scan(cx, cy, skel.EXCLUSIVE, skel.SUM, variant=3)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            skel.skel_scan(cx, cy, skel.EXCLUSIVE, skel.SUM, variant=3)
    torch.cuda.synchronize()
    for rep in range(4):
        with torch.cuda.stream(s):
            x.copy_(torch.randint(0, 1000, (n,), device="cuda", dtype=torch.int32))
            y.fill_(-1)
            skel.skel_scan(cx, cz, skel.REVERSE_INCLUSIVE, skel.SUM, variant=3)
            g.replay()
        s.synchronize()
        want = torch.cumsum(x.to(torch.int64), 0)
        assert torch.equal(y, (want - x).to(torch.int32)), rep
        assert torch.equal(z, (want[-1] - want + x).to(torch.int32)), rep
    skel.skel_sync(s)
    for c in (cx, cy, cz):
        c.destroy()


def test_scan_repeated_calls_reuse_descriptors(skel, oracle_mod):
    # the look-back descriptors and counters are reused across calls (a fresh
    # epoch each call): alternate sizes and the four single-pass variants
    # without clearing anything
    for k in range(24):
        n = [(1 << 20) + 1, 9000, (1 << 18) + 77][k % 3]
        x = si.int_uniform_i32(n, 1000, 5, k)
        out = skel.Container.empty(skel.I64, n)
        skel.skel_scan(cont(skel, x), out, skel.EXCLUSIVE, skel.SUM, variant=2 + (k // 3) % 4)
        assert np.array_equal(out.to_numpy(), oracle_mod.scan(x, "exclusive", "sum",
                                                              np.int64)), k
    skel.skel_sync()


# ------------------------------------------- drawn tiny shapes (hypothesis)
from hypothesis import HealthCheck, given, settings, strategies as st  # noqa: E402


@settings(max_examples=40, deadline=None, suppress_health_check=list(HealthCheck))
@given(rows=st.integers(1, 90), cols=st.sampled_from([252, 255, 256, 257, 260, 512, 516, 768]),
       ry=st.integers(0, 4), rx=st.integers(0, 4), edge=st.sampled_from(list(EDGES)),
       sep=st.booleans(), seed=st.integers(0, 1000))
def test_mapoverlap2d_march_drawn_shapes(skel, oracle_mod, rows, cols, ry, rx, edge, sep, seed):
    # widths around whole 256-column strips, where the marching window
    # switches between its straight-line and general paths
    img = si.uniform_f32(rows * cols, -1.0, 1.0, 43, seed).reshape(rows, cols)
    wy = si.uniform_f32(2 * ry + 1, -1.0, 1.0, 43, 2000 + seed)
    wx = si.uniform_f32(2 * rx + 1, -1.0, 1.0, 43, 3000 + seed)
    kw = {"wy": wy, "wx": wx} if sep else {
        "w2d": (wy.astype(np.float64)[:, None] * wx.astype(np.float64)[None, :]).astype(
            np.float32)}
    ref, mag = oracle_mod.mapoverlap2d(img, ry, rx, edge=edge, pad=-0.5, **kw)
    out = skel.Container.empty(skel.F32, rows, cols)
    skel.skel_mapoverlap2d(cont(skel, img), out, ry=ry, rx=rx, edge=EDGES[edge], pad=-0.5,
                           variant=skel.variant_index(skel.SK_MAPOVERLAP2D, "O2e_march"), **kw)
    got = out.to_numpy().reshape(rows, cols).astype(np.float64)
    assert np.all(np.abs(got - ref) <= 1e-6 * mag + 1e-30), (rows, cols, ry, rx, edge, sep)


@settings(max_examples=60, deadline=None, suppress_health_check=list(HealthCheck))
@given(rows=st.integers(1, 40), cols=st.integers(1, 40), ry=st.integers(0, 8),
       rx=st.integers(0, 8), edge=st.sampled_from(list(EDGES)), sep=st.booleans(),
       seed=st.integers(0, 1000))
def test_mapoverlap2d_drawn_shapes(skel, oracle_mod, rows, cols, ry, rx, edge, sep, seed):
    img = si.uniform_f32(rows * cols, -1.0, 1.0, 13, seed).reshape(rows, cols)
    wy = si.uniform_f32(2 * ry + 1, -1.0, 1.0, 13, 2000 + seed)
    wx = si.uniform_f32(2 * rx + 1, -1.0, 1.0, 13, 3000 + seed)
    kw = {"wy": wy, "wx": wx} if sep else {
        "w2d": (wy.astype(np.float64)[:, None] * wx.astype(np.float64)[None, :]).astype(
            np.float32)}
    ref, mag = oracle_mod.mapoverlap2d(img, ry, rx, edge=edge, pad=0.375, **kw)
    for v in variants(skel, skel.SK_MAPOVERLAP2D):
        if (v in (2, 3) and not sep) or (v == 4 and max(ry, rx) > 4):
            continue
        out = skel.Container.empty(skel.F32, rows, cols)
        skel.skel_mapoverlap2d(cont(skel, img), out, ry=ry, rx=rx, edge=EDGES[edge],
                               pad=0.375, variant=v, **kw)
        got = out.to_numpy().reshape(rows, cols).astype(np.float64)
        assert np.all(np.abs(got - ref) <= 1e-6 * mag + 1e-30), (v, rows, cols, ry, rx, edge)


@settings(max_examples=60, deadline=None, suppress_health_check=list(HealthCheck))
@given(n=st.integers(1, 3000), r=st.integers(0, 9), edge=st.sampled_from(list(EDGES)),
       seed=st.integers(0, 1000))
def test_mapoverlap1d_drawn_sizes(skel, oracle_mod, n, r, edge, seed):
    x = si.uniform_f32(n, -1.0, 1.0, 14, seed)
    w = si.uniform_f32(2 * r + 1, -1.0, 1.0, 14, 2000 + seed)
    ref, mag = oracle_mod.mapoverlap1d(x, w, r, edge, -0.5)
    for v in variants(skel, skel.SK_MAPOVERLAP1D):
        if v == 2 and r > 4:
            continue
        out = skel.Container.empty(skel.F32, n)
        skel.skel_mapoverlap1d(cont(skel, x), out, w, r, EDGES[edge], -0.5, variant=v)
        assert np.all(np.abs(out.to_numpy() - ref) <= 1e-6 * mag + 1e-30), (v, n, r, edge)
    # and the adjoint on the same draw
    ga, gm = oracle_mod.mapoverlap1d_adjoint(x, w, r, edge)
    for v in range(skel.skel_variant_count(skel.SK_MAPOVERLAP1D_BACKWARD)):
        out = skel.Container.empty(skel.F32, n)
        skel.skel_mapoverlap1d_backward(cont(skel, x), out, w, r, EDGES[edge], variant=v)
        assert np.all(np.abs(out.to_numpy() - ga) <= 1e-6 * gm + 1e-30), (n, r, edge, v)
