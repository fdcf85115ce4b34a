"""GPU parity of RoIAlign at sampling ratios other than 2 on the 7x7 and 14x14 grids (the
adaptive grid and fixed ratios) against the CPU oracle: the footprint forward and the tile
gather that RE_BWD_AUTO takes with a plan, at the sizes where their panels and tiles end,
with non-finite values, and with levels that are not the plan's.

Tolerances are those of the other parity tests (gpu_helpers): a pixel's weight is a sum of
at most 2 x 64 products of binary32 fractions, each correct to a few units of 2^-24, far
inside 1e-5 of the result.
"""
import numpy as np
import pytest

import oracle
import paper_1906_07155_amd as rex
from paper_1906_07155_amd import workloads as W
from gpu_helpers import as_f64, check_bwd, check_fwd, from_device, log, to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rex.lib()


SHAPES = [(2, 70, 25, 90), (2, 70, 13, 45), (2, 70, 7, 23)]
SCALES = [0.25, 0.125, 0.0625]


def _setup(rois, shapes, scales, dt, layout, levels=None, seed=0):
    rng = np.random.default_rng(seed)
    feats = [rng.standard_normal(s, dtype=np.float32) for s in shapes]
    if dt == "bf16":
        feats = [W.f32_to_bf16_bits(f) for f in feats]
    r = torch.from_numpy(rois).cuda()
    dev = [to_device(f, dt, layout) for f in feats]
    lv, ws = rex.plan(dev, scales, r, 56.0)
    lv_np = oracle.level_map(rois, len(shapes), 56.0)
    if levels is not None:
        lv_np = np.asarray(levels(lv_np), np.int32)
        lv = torch.from_numpy(lv_np).cuda()
    return rng, feats, dev, r, lv, ws, lv_np


def _run(name, rois, P, S, aligned=True, dt="f32", layout="cl", levels=None, zero_init=True,
         shapes=SHAPES, scales=SCALES):
    log("adaptive case %s: K=%d P=%d S=%d aligned=%d %s %s" % (
        name, rois.shape[0], P, S, aligned, dt, layout))
    rng, feats, dev, r, lv, ws, lv_np = _setup(rois, shapes, scales, dt, layout, levels)
    K, C = rois.shape[0], shapes[0][1]
    out = rex.roi_align_fwd(dev, scales, r, lv, (P, P), S, aligned, workspace=ws)
    f64 = [as_f64(f, dt) for f in feats]
    ref = oracle.roi_align_fwd(f64, scales, rois, lv_np, P, P, S, aligned, "parity")
    check_fwd(from_device(out), ref, dt == "bf16", name + " forward")
    g = rng.standard_normal((K, C, P, P), dtype=np.float32)
    if dt == "bf16":
        g = W.f32_to_bf16_bits(g)
    g64 = as_f64(g, dt)
    gref = oracle.roi_align_bwd(g64, shapes, scales, rois, lv_np, P, P, S, aligned, "parity")
    aref = oracle.roi_align_bwd(np.abs(g64), shapes, scales, rois, lv_np, P, P, S, aligned,
                                "parity")
    grads = [torch.full(s, 7.0, dtype=torch.float32, device="cuda") for s in shapes]
    if layout == "cl":
        grads = [x.contiguous(memory_format=torch.channels_last) for x in grads]
    rex.roi_align_bwd(to_device(g, dt, "nchw"), r, lv, (P, P), S, aligned, grads, scales,
                      zero_init=zero_init, workspace=ws)
    torch.cuda.synchronize()
    base = 0.0 if zero_init else 7.0
    for l in range(len(shapes)):
        check_bwd(from_device(grads[l]) - base, gref[l], aref[l] + base * 2.0 ** -20 / 1e-4, False,
                  "%s backward level %d" % (name, l))


def _mixed_rois():
    """Boxes of every size, among them one as wide as the map (two column panels), one as
    tall, and boxes without width, outside the map and of an image that is not there."""
    rng = np.random.default_rng(3)
    rois = W.draw_rois(rng, 2, 17, (100, 360), (1.0, 300.0))
    extra = np.array([[0, 0, 40, 360, 52], [1, 3, 0, 20, 100], [0, 30, 30, 30, 60],
                      [1, 500, 20, 600, 50], [2, 10, 10, 60, 60], [0, -80, -60, 30, 25]], np.float32)
    return np.concatenate([rois, extra])


@pytest.mark.parametrize("S", [0, 1, 3, 4])
@pytest.mark.parametrize("P", [7, 14])
def test_sampling_ratios(P, S):
    _run("ratios", _mixed_rois(), P, S, aligned=S != 3)


@pytest.mark.parametrize("P", [7, 14])
@pytest.mark.parametrize("dt,layout", [("bf16", "cl"), ("f32", "nchw"), ("bf16", "nchw")])
def test_types_and_layouts(P, dt, layout):
    _run("types", _mixed_rois(), P, 0, dt=dt, layout=layout, zero_init=layout == "cl")


@pytest.mark.parametrize("C", [1, 3, 64, 129])
def test_channels(C):
    shapes = [(n, C, h, w) for n, _, h, w in SHAPES]
    _run("channels", _mixed_rois(), 7, 0, shapes=shapes)


def test_many_samples():
    # one level: bins of up to 300 / 7 = 43 and 70 pixels (the grid is capped at 64 samples),
    # so a wave's bin rows and the columns both take several panels
    rois = np.array([[0, 0, 0, 300, 200], [0, 2, 1, 500, 190], [0, 5, 7, 40, 199]], np.float32)
    _run("many", rois, 7, 0, shapes=[(1, 5, 200, 500)], scales=[1.0])


WIDE = np.array([[0, 0, 0, 300, 200], [1, 2, 1, 500, 190], [0, 5, 7, 40, 199], [1, 100, 20, 480, 44],
                 [0, -90, -50, 460, 300], [1, 10, 10, 30, 30], [0, 0, 60, 499, 66]], np.float32)


@pytest.mark.parametrize("copies", [1, 80])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("P,S", [(7, 1), (7, 3), (7, 4), (7, 33), (14, 1), (14, 3), (14, 17)])
def test_few_samples_in_wide_bins(P, S, dt, copies):
    # bins many pixels wide: the forward takes the samples' taps where they are fewer than the
    # pixels between them, on either axis, in one panel (S = 1, 3, 4) and in several, in grids
    # that leave the chip idle and in larger ones
    shapes = [(2, 70, 200, 500)]
    if copies == 1:
        _run("wide", WIDE, P, S, dt=dt, shapes=shapes, scales=[1.0], aligned=S != 3)
    elif S <= 4:
        _forward("wide, many", np.tile(WIDE, (copies, 1)), P, S, dt, shapes, [1.0])


def _forward(name, rois, P, S, dt, shapes, scales, aligned=True):
    log("adaptive forward %s: K=%d P=%d S=%d %s" % (name, rois.shape[0], P, S, dt))
    rng, feats, dev, r, lv, ws, lv_np = _setup(rois, shapes, scales, dt, "cl")
    out = rex.roi_align_fwd(dev, scales, r, lv, (P, P), S, aligned, workspace=ws)
    ref = oracle.roi_align_fwd([as_f64(f, dt) for f in feats], scales, rois, lv_np, P, P, S, aligned,
                               "parity")
    check_fwd(from_device(out), ref, dt == "bf16", name)


@pytest.mark.parametrize("C", [64, 129])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("P", [7, 14])
def test_grid_sizes(P, dt, C):
    # workgroups around the counts up to which a workgroup has one wave per bin row
    few = 512 if P == 7 else 256
    slices = -(-C // (128 if dt == "bf16" and P == 7 and C % 2 == 0 else 64))
    rois = np.tile(_mixed_rois(), (13, 1))
    shapes = [(n, C, h, w) for n, _, h, w in SHAPES]
    for k in (few // slices, few // slices + 1):
        _forward("grid", rois[:k], P, 0, dt, shapes, SCALES)


@pytest.mark.parametrize("S", [1, 4])
def test_non_finite_feature_in_wide_bins(S):
    shapes = [(2, 6, 200, 500)]
    rng = np.random.default_rng(S)
    feats = rng.standard_normal(shapes[0], dtype=np.float32)
    for value in (np.inf, -np.inf, np.nan):
        for _ in range(40):
            feats[rng.integers(2), rng.integers(6), rng.integers(200), rng.integers(500)] = value
    feats[:, 5, ::2] = np.inf    # (rows that some samples tap with weight zero)
    rois = np.concatenate([WIDE, np.array([[0, 10.5, 0.5, 290.5, 112.5]], np.float32)])
    lv = np.zeros(len(rois), np.int32)
    out = from_device(rex.roi_align_fwd([to_device(feats, "f32", "cl")], [1.0], torch.from_numpy(rois).cuda(),
                                        torch.from_numpy(lv).cuda(), (7, 7), S, True))
    ref = oracle.roi_align_fwd([feats.astype(np.float64)], [1.0], rois, lv, 7, 7, S, True, "parity")
    assert np.array_equal(np.isfinite(out), np.isfinite(ref)) and not np.isfinite(ref).all()
    ok = np.isfinite(ref)
    check_fwd(np.where(ok, out, 0), np.where(ok, ref, 0), False, "non-finite feature, wide bins")


@pytest.mark.parametrize("S", [3, 4, 64])
def test_samples_closer_than_a_unit(S):
    # boxes a few units in the last place wide: all samples of a bin round to one position, which
    # at the map's edges is cut or clamped as a whole (the window over the samples is compared
    # with the sum over all of them on the CPU, test_any_window_cpu.py)
    rois = []
    for x, y in ((362, 40), (361, 102), (-2, 3), (-1.9, -2), (30, 30)):
        x2, y2 = np.float32(x), np.float32(y)
        for _ in range(3):
            x2, y2 = np.nextafter(x2, np.float32(np.inf)), np.nextafter(y2, np.float32(np.inf))
            rois += [[0, x, y, x2, y2], [1, x, 20, x2, 50], [0, 100, y, 160, y2]]
    _run("tiny", np.array(rois, np.float32), 7, S)


def test_levels_not_the_plans():
    # a caller's own levels: the tile lists hold the RoIs on the plan's levels only
    _run("stray", _mixed_rois(), 7, 0, levels=lambda lv: (lv + (np.arange(lv.size) % 3 == 0)) % 3)


def test_non_finite_feature():
    # an infinity and a NaN reach exactly the bins whose samples read them
    rois = _mixed_rois()
    rng, feats, dev, r, lv, ws, lv_np = _setup(rois, SHAPES, SCALES, "f32", "cl")
    feats[0][0, 3, 10, 40] = np.inf
    feats[1][1, 69, 5, 20] = np.nan
    dev = [to_device(f, "f32", "cl") for f in feats]
    for P in (7, 14):
        out = from_device(rex.roi_align_fwd(dev, SCALES, r, lv, (P, P), 0, True, workspace=ws))
        ref = oracle.roi_align_fwd([f.astype(np.float64) for f in feats], SCALES, rois, lv_np, P, P,
                                   0, True, "parity")
        assert np.array_equal(np.isfinite(out), np.isfinite(ref))
        ok = np.isfinite(ref)
        check_fwd(np.where(ok, out, 0), np.where(ok, ref, 0), False, "non-finite feature")


def _as_the_scatter(rois, g, P, S, aligned, layout, zero_init):
    """RE_BWD_AUTO's pyramid has the scatter's infinities and NaNs, element by element."""
    rng, feats, dev, r, lv, ws, lv_np = _setup(rois, SHAPES, SCALES, "f32", layout)
    gd = g.cuda()
    res = []
    for algo in ("auto", "scatter"):
        grads = [torch.full(s, 7.0, dtype=torch.float32, device="cuda") for s in SHAPES]
        if layout == "cl":
            grads = [x.contiguous(memory_format=torch.channels_last) for x in grads]
        rex.roi_align_bwd(gd, r, lv, (P, P), S, aligned, grads, SCALES, zero_init=zero_init,
                          workspace=ws, algorithm=algo)
        res.append([from_device(x) for x in grads])
    for a, s in zip(*res):
        assert np.array_equal(np.isnan(a), np.isnan(s))
        assert np.array_equal(np.isposinf(a), np.isposinf(s))
        assert np.array_equal(np.isneginf(a), np.isneginf(s))
        ok = np.isfinite(s)
        # the same products in two orders: 1e-4 of the sums' scale, as the gather against
        # the oracle
        assert np.all(np.abs(a[ok] - s[ok]) <= 1e-4 * np.maximum(np.abs(s[ok]), 1.0))
    return res[1]


@pytest.mark.parametrize("zero_init", [True, False])
@pytest.mark.parametrize("layout", ["cl", "nchw"])
def test_non_finite_gradient(layout, zero_init):
    # as the scatter: exactly the tapped pixels take the value
    rois = _mixed_rois()
    g = torch.from_numpy(np.random.default_rng(1).standard_normal((rois.shape[0], 70, 7, 7),
                                                                  dtype=np.float32))
    g[4, 2, 3, 3] = np.inf
    g[20, 69, 0, 6] = np.nan
    _as_the_scatter(rois, g, 7, 0, True, layout, zero_init)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("P,S,zero_init", [(7, 0, True), (7, 1, True), (7, 3, False), (7, 4, True),
                                           (14, 0, False), (14, 4, True)])
def test_non_finite_gradient_on_integer_samples(P, S, zero_init, dt):
    # A sample on a pixel taps the next one with weight zero, and zero times an infinity is NaN,
    # whatever other samples of the bin give that pixel; so does a sample on the last pixel (or
    # clamped to it) with that pixel, and one clamped to pixel 0 with pixel 1.  Boxes on level 0
    # (scale 1/4, 25 x 90 pixels) whose bins are 1, 2 or 4 pixels wide from a quarter of a pixel on.
    rois = []
    for bin_ in (1.0, 2.0, 0.25):
        for at in (3.0, 3.5, 3.25, -1.0, -0.5, 88.0 - 7 * bin_, 89.5 - 7 * bin_, 91.0 - 7 * bin_):
            for top in (2.0, 2.5, -0.5, 20.5 - 7 * bin_):
                x1, y1 = (at + 0.5) * 4, (top + 0.5) * 4
                rois.append([len(rois) % 2, x1, y1, x1 + P * bin_ * 4, y1 + P * bin_ * 4])
    rois = np.array(rois, np.float32)
    rng = np.random.default_rng(P + S)
    g = rng.standard_normal((len(rois), 70, P, P), dtype=np.float32)
    for value in (np.inf, -np.inf, np.nan, 2e38):
        for _ in range(60):
            g[rng.integers(len(rois)), rng.integers(70), rng.integers(P), rng.integers(P)] = value
    g = torch.from_numpy(g)
    if dt == "bf16":
        g = g.to(torch.bfloat16)
    s = _as_the_scatter(rois, g, P, S, True, "cl", zero_init)
    assert np.isnan(s[0]).any() and np.isposinf(s[0]).any() and np.isneginf(s[0]).any()


def _adds(rois, S, streams):
    """Every stream adds one upstream gradient into one pyramid; the sum against the oracle."""
    rng, feats, dev, r, lv, ws, lv_np = _setup(rois, SHAPES, SCALES, "f32", "cl")
    g = rng.standard_normal((len(streams), rois.shape[0], 70, 7, 7), dtype=np.float32)
    gd = torch.from_numpy(g).cuda()
    grads = [torch.full(s, 7.0, device="cuda").contiguous(memory_format=torch.channels_last) for s in SHAPES]
    torch.cuda.synchronize()
    for i, st in enumerate(streams):
        rex.roi_align_bwd(gd[i], r, lv, (7, 7), S, True, grads, SCALES, zero_init=False,
                          workspace=ws, stream=st)
    torch.cuda.synchronize()
    for l in range(len(SHAPES)):
        ref = sum(oracle.roi_align_bwd(x.astype(np.float64), SHAPES, SCALES, rois, lv_np, 7, 7, S, True,
                                       "parity")[l] for x in g)
        aref = sum(oracle.roi_align_bwd(np.abs(x).astype(np.float64), SHAPES, SCALES, rois, lv_np, 7, 7, S,
                                        True, "parity")[l] for x in g)
        # (7 and the partial sums round to binary32: 2^-20 of them covers the few additions)
        check_bwd(from_device(grads[l]) - 7.0, ref, aref + 7.0 * 2.0 ** -20 / 1e-4, False, "added")


@pytest.mark.parametrize("S", [0, 3])
def test_accumulating_calls_may_overlap(S):
    # calls that add into one pyramid on several streams lose nothing (atomics, as the scatter)
    _adds(_mixed_rois(), S, [torch.cuda.Stream() for _ in range(4)] * 2)


def test_levels_that_share_memory():
    # one tensor as two levels: both levels' gradients end up in it, which a gather that stores
    # every element cannot do
    rois = np.concatenate([_mixed_rois(), np.array([[0, 10, 0, 200, 98], [1, 100, 5, 300, 95]], np.float32)])
    shapes, scales = [SHAPES[0], SHAPES[0]], [0.25, 0.25]
    rng, feats, dev, r, lv, ws, lv_np = _setup(rois, shapes, scales, "f32", "cl")
    assert 0 < int((lv_np == 1).sum()) < rois.shape[0]
    g = rng.standard_normal((rois.shape[0], 70, 7, 7), dtype=np.float32)
    grad = torch.full(shapes[0], 7.0, device="cuda").contiguous(memory_format=torch.channels_last)
    rex.roi_align_bwd(torch.from_numpy(g).cuda(), r, lv, (7, 7), 3, True, [grad, grad], scales,
                      zero_init=True, workspace=ws)
    refs = [sum(oracle.roi_align_bwd(x.astype(np.float64), shapes, scales, rois, lv_np, 7, 7, 3, True,
                                     "parity")) for x in (g, np.abs(g))]
    check_bwd(from_device(grad), refs[0], refs[1], False, "shared levels")
