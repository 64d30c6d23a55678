"""GPU parity of the batched-field 2D MapOverlap and its transpose: every
field of a (fields * H) x W container is mapped on its own, so each field must
match the oracle's single-image result, for every variant and edge rule.

Bars as the single-image calls: |y - y*| <= 1e-6 * sum of |terms| per pixel."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

EDGES = {"clamp": 0, "const": 1, "cyclic": 2}
SHAPES = [(3, 37, 45), (5, 64, 64), (2, 1, 9), (4, 130, 7)]


def weights(sep, r, seed):
    wy = si.uniform_f32(2 * r + 1, -1.0, 1.0, 22, seed)
    wx = si.uniform_f32(2 * r + 1, -1.0, 1.0, 22, seed + 1)
    if sep:
        return {"wy": wy, "wx": wx}
    return {"w2d": si.uniform_f32((2 * r + 1) ** 2, -1.0, 1.0, 22, seed + 2)
            .reshape(2 * r + 1, 2 * r + 1)}


@pytest.mark.parametrize("edge", list(EDGES))
@pytest.mark.parametrize("sep", [False, True])
@pytest.mark.parametrize("r", [1, 4])
def test_fields_forward_and_backward(skel, oracle_mod, edge, sep, r):
    w = weights(sep, r, 10 * r + sep)
    for f, h, wd in SHAPES:
        x = si.uniform_f32(f * h * wd, -1.0, 1.0, 22, f * 1000 + h).reshape(f * h, wd)
        cx = skel.Container.from_numpy(x)
        for v in range(skel.skel_variant_count(skel.SK_MAPOVERLAP2D)):
            name = skel.skel_variant_name(skel.SK_MAPOVERLAP2D, v)
            if not sep and "separable" in name:
                continue
            out = skel.Container.empty(skel.F32, f * h, wd)
            skel.skel_mapoverlap2d_fields(cx, out, f, edge=EDGES[edge], pad=0.25, variant=v,
                                          **w)
            got = out.to_numpy().reshape(f, h, wd)
            for k in range(f):
                ref, mag = oracle_mod.mapoverlap2d(x[k * h:(k + 1) * h], r, r, edge=edge,
                                                   pad=0.25, **w)
                bad = np.abs(got[k] - ref) > 1e-6 * mag + 1e-30
                assert not bad.any(), (edge, sep, r, (f, h, wd), name, k, np.argwhere(bad)[:3])
        for v in range(skel.skel_variant_count(skel.SK_MAPOVERLAP2D_BACKWARD)):
            out = skel.Container.empty(skel.F32, f * h, wd)
            skel.skel_mapoverlap2d_fields_backward(cx, out, f, edge=EDGES[edge], variant=v, **w)
            got = out.to_numpy().reshape(f, h, wd)
            for k in range(f):
                ref, mag = oracle_mod.mapoverlap2d_adjoint(x[k * h:(k + 1) * h], r, r,
                                                           edge=edge, **w)
                bad = np.abs(got[k] - ref) > 1e-6 * mag + 1e-30
                assert not bad.any(), (edge, sep, r, (f, h, wd), "adjoint", v, k,
                                       np.argwhere(bad)[:3])
    skel.skel_sync()


# images of 1, 2, 3, 6, 8, 9, 12 and 17 tiles of 64 x 16: every remainder of the tile
# count over the eight XCDs that matters, and axes shorter than the halo
@pytest.mark.parametrize("edge", list(EDGES))
@pytest.mark.parametrize("r", [1, 2, 6])
def test_fields_of_few_tiles(skel, oracle_mod, edge, r):
    for f, h, wd in ((7, 16, 16), (3, 5, 70), (3, 3, 130), (2, 33, 65), (2, 49, 100),
                     (2, 33, 131), (2, 49, 130), (2, 260, 3)):
        x = si.uniform_f32(f * h * wd, -1.0, 1.0, 26, f * 1000 + h).reshape(f * h, wd)
        cx = skel.Container.from_numpy(x)
        for sep in (False, True):
            w = weights(sep, r, 50 * r + sep)
            calls = [("map", v) for v in (1, 2, 3, 4) if (sep or v in (1, 4)) and (v < 4 or r <= 4)]
            for what, v in calls + [("transpose", 1)]:
                out = skel.Container.empty(skel.F32, f * h, wd)
                if what == "map":
                    skel.skel_mapoverlap2d_fields(cx, out, f, edge=EDGES[edge], pad=0.25,
                                                  variant=v, **w)
                else:
                    skel.skel_mapoverlap2d_fields_backward(cx, out, f, edge=EDGES[edge],
                                                           variant=v, **w)
                got = out.to_numpy().reshape(f, h, wd)
                for k in range(f):
                    img = x[k * h:(k + 1) * h]
                    ref, mag = (oracle_mod.mapoverlap2d(img, r, r, edge=edge, pad=0.25, **w)
                                if what == "map" else
                                oracle_mod.mapoverlap2d_adjoint(img, r, r, edge=edge, **w))
                    bad = np.abs(got[k] - ref) > 1e-6 * mag + 1e-30
                    assert not bad.any(), (edge, sep, r, (f, h, wd), what, v, k,
                                           np.argwhere(bad)[:3])
    skel.skel_sync()


@pytest.mark.parametrize("edge", list(EDGES))
def test_image_of_more_tiles_than_one_launch(skel, edge):
    """A column of 2^29 + 37 pixels: its tiles and, clamped, the transpose's border
    are more work items than one launch can number.  Weights are eighths and pixels
    small integers, so that every sum is exact."""
    import torch
    n = (1 << 29) + 37
    w = np.array([[1, 2, 0], [3, 1, 2], [2, 0, 5]], np.float32) / 8
    x = torch.empty(n, 1, device="cuda").random_(-8, 9)
    y = torch.empty_like(x)
    cx, cy = skel.wrap_tensor(x), skel.wrap_tensor(y)
    # one column: with a border rule that reads it back, a row's weights add up
    a = (w[:, 1] if edge == "const" else w.sum(1)).astype(float)
    up, down = torch.roll(x, 1, 0), torch.roll(x, -1, 0)  # x[i - 1], x[i + 1]
    if edge != "cyclic":
        up[0] = x[0] if edge == "clamp" else 0
        down[-1] = x[-1] if edge == "clamp" else 0
    skel.skel_mapoverlap2d_fields(cx, cy, 1, w2d=w, edge=EDGES[edge], pad=0.0)
    assert torch.equal(y, a[0] * up + a[1] * x + a[2] * down)
    skel.skel_mapoverlap2d_fields_backward(cx, cy, 1, w2d=w, edge=EDGES[edge])
    if edge != "cyclic":
        up[0] = down[-1] = 0
    want = a[2] * up + a[1] * x + a[0] * down
    if edge == "clamp":
        want[0] += a[0] * x[0]
        want[-1] += a[2] * x[-1]
    assert torch.equal(y, want)
    skel.skel_sync()
    for c in (cx, cy):
        c.destroy()


def test_fields_beyond_one_launch(skel, oracle_mod):
    # more fields than one launch's grid holds (65535): the launcher splits them
    f, h, wd = 70001, 2, 4
    x = si.uniform_f32(f * h * wd, -1.0, 1.0, 22, 99).reshape(f * h, wd)
    w = si.five_point_weights(0.5, 0.1, 0.2, 0.05, 0.15)
    cx = skel.Container.from_numpy(x)
    out = skel.Container.empty(skel.F32, f * h, wd)
    skel.skel_mapoverlap2d_fields(cx, out, f, w2d=w, edge=skel.EDGE_CLAMP)
    got = out.to_numpy().reshape(f, h, wd)
    back = skel.Container.empty(skel.F32, f * h, wd)
    skel.skel_mapoverlap2d_fields_backward(cx, back, f, w2d=w, edge=skel.EDGE_CLAMP)
    gb = back.to_numpy().reshape(f, h, wd)
    for k in (0, 1, 65534, 65535, 65536, f - 1):
        xf = x[k * h:(k + 1) * h]
        ref, mag = oracle_mod.mapoverlap2d(xf, 1, 1, w2d=w, edge="clamp")
        assert np.all(np.abs(got[k] - ref) <= 1e-6 * mag + 1e-30), k
        ref, mag = oracle_mod.mapoverlap2d_adjoint(xf, 1, 1, w2d=w, edge="clamp")
        assert np.all(np.abs(gb[k] - ref) <= 1e-6 * mag + 1e-30), k
    skel.skel_sync()


def test_fields_shape_errors(skel):
    x = skel.Container.from_numpy(np.zeros((10, 8), np.float32))
    out = skel.Container.empty(skel.F32, 10, 8)
    w = np.ones((3, 3), np.float32)
    for bad in (3, 0, -1):  # 3 does not divide 10 rows
        with pytest.raises(skel.SkelError) as e:
            skel.skel_mapoverlap2d_fields(x, out, bad, w2d=w)
        assert e.value.status == skel.E_SHAPE
        with pytest.raises(skel.SkelError) as e:
            skel.skel_mapoverlap2d_fields_backward(x, out, bad, w2d=w)
        assert e.value.status == skel.E_SHAPE
    skel.skel_mapoverlap2d_fields(x, out, 10, w2d=w)  # ten 1 x 8 fields
    skel.skel_sync()


from hypothesis import HealthCheck, given, settings, strategies as st  # noqa: E402


@settings(max_examples=60, deadline=None, suppress_health_check=list(HealthCheck))
@given(f=st.integers(1, 5), h=st.integers(1, 40), wd=st.integers(1, 40), ry=st.integers(0, 3),
       rx=st.integers(0, 3), edge=st.sampled_from(list(EDGES)), sep=st.booleans(),
       seed=st.integers(0, 1000))
def test_fields_drawn_shapes(skel, oracle_mod, f, h, wd, ry, rx, edge, sep, seed):
    x = si.uniform_f32(f * h * wd, -1.0, 1.0, 24, seed).reshape(f * h, wd)
    wy = si.uniform_f32(2 * ry + 1, -1.0, 1.0, 24, 2000 + seed)
    wx = si.uniform_f32(2 * rx + 1, -1.0, 1.0, 24, 3000 + seed)
    w = {"wy": wy, "wx": wx} if sep else {"w2d": np.outer(wy, wx).astype(np.float32)}
    cx = skel.Container.from_numpy(x)
    out = skel.Container.empty(skel.F32, f * h, wd)
    skel.skel_mapoverlap2d_fields(cx, out, f, edge=EDGES[edge], pad=0.5, **w)
    back = skel.Container.empty(skel.F32, f * h, wd)
    skel.skel_mapoverlap2d_fields_backward(cx, back, f, edge=EDGES[edge], **w)
    got, gb = out.to_numpy().reshape(f, h, wd), back.to_numpy().reshape(f, h, wd)
    for k in range(f):
        xf = x[k * h:(k + 1) * h]
        ref, mag = oracle_mod.mapoverlap2d(xf, ry, rx, edge=edge, pad=0.5, **w)
        assert np.all(np.abs(got[k] - ref) <= 1e-6 * mag + 1e-30), k
        ref, mag = oracle_mod.mapoverlap2d_adjoint(xf, ry, rx, edge=edge, **w)
        assert np.all(np.abs(gb[k] - ref) <= 1e-6 * mag + 1e-30), k
