"""GPU edge cases and invariants, each against the CPU oracle.

Small shapes that still span several channel slices with a ragged tail, every
kernel family (channels-last fast path, general strided path), both dtypes, and
the degenerate inputs the operator has.
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


def _feats(rng, shapes, fdt):
    out = []
    for s in shapes:
        x = rng.standard_normal(s, dtype=np.float32)
        out.append(W.f32_to_bf16_bits(x) if fdt == "bf16" else x)
    return out


def _device_levels(feats_np, fdt, layout):
    if layout in ("cl", "nchw"):
        return [to_device(f, fdt, layout) for f in feats_np]
    # strided views into larger tensors: 'cl_view' keeps stride_c == 1, 'nchw_view' does not
    views = []
    for f in feats_np:
        n, c, h, w = f.shape
        big = np.zeros((n, c + 5, h + 2, w + 3), dtype=f.dtype)
        big[:, 2:2 + c, 1:1 + h, :w] = f
        t = to_device(big, fdt, "cl" if layout == "cl_view" else "nchw")
        views.append(t[:, 2:2 + c, 1:1 + h, :w])
    return views


def _rois(rng, K, n_images, img_w, img_h, outside=0.2):
    a = rng.uniform(-outside * img_w, (1 + outside) * img_w, (K, 2))
    b = rng.uniform(-outside * img_h, (1 + outside) * img_h, (K, 2))
    r = np.zeros((K, 5), np.float32)
    r[:, 0] = rng.integers(0, n_images, K)
    r[:, 1], r[:, 3] = a.min(1), a.max(1)
    r[:, 2], r[:, 4] = b.min(1), b.max(1)
    return r


def run(name, shapes, scales, rois, out_hw=(7, 7), S=2, aligned=True, fdt="f32", odt="f32",
        gdt="f32", layout="cl", roi_levels=None, use_plan=True, seed=0, backward=True,
        zero_init=True):
    log("edge case %s: shapes=%s K=%d out=%s S=%d aligned=%d %s->%s layout=%s" % (
        name, shapes, rois.shape[0], out_hw, S, aligned, fdt, odt, layout))
    rng = np.random.default_rng(seed)
    feats_np = _feats(rng, shapes, fdt)
    feats = _device_levels(feats_np, fdt, layout)
    K = rois.shape[0]
    C = shapes[0][1]
    L = len(shapes)
    r_dev = torch.from_numpy(rois).cuda()
    ws = None
    if roi_levels is None:
        lv_dev, ws = rex.plan(feats, scales, r_dev, 56.0)
        lv = oracle.level_map(rois, L, 56.0)
        if not use_plan:
            ws = None
    else:
        lv = np.asarray(roi_levels, np.int32)
        lv_dev = torch.from_numpy(lv).cuda()
    odt_t = torch.bfloat16 if odt == "bf16" else torch.float32
    out = rex.roi_align_fwd(feats, scales, r_dev, lv_dev, out_hw, S, aligned, out_dtype=odt_t,
                            workspace=ws)
    torch.cuda.synchronize()
    f64 = [as_f64(f, fdt) for f in feats_np]
    ref = oracle.roi_align_fwd(f64, scales, rois, lv, out_hw[0], out_hw[1], S, aligned, "parity")
    check_fwd(from_device(out), ref, fdt == "bf16" or odt == "bf16", name + " forward")
    if not backward:
        return out
    g = rng.standard_normal((K, C) + tuple(out_hw), dtype=np.float32)
    if gdt == "bf16":
        g = W.f32_to_bf16_bits(g)
    g64 = as_f64(g, gdt)
    gref = oracle.roi_align_bwd(g64, shapes, scales, rois, lv, out_hw[0], out_hw[1], S, aligned,
                                "parity")
    aref = oracle.roi_align_bwd(np.abs(g64), shapes, scales, rois, lv, out_hw[0], out_hw[1], S,
                                aligned, "parity")
    # scatter always; the gather where it applies (plan, 7x7 / 14x14, S = 2; any level
    # layout whose images span less than 2^30 bytes, channels-last or NCHW)
    algos = ["scatter"]
    if ws is not None and S == 2 and tuple(out_hw) in ((7, 7), (14, 14)):
        algos.append("gather")
    for algo in algos:
        grads = [torch.full(s, 7.0, dtype=torch.float32, device="cuda") for s in shapes]
        if layout in ("cl", "cl_view"):
            grads = [x.contiguous(memory_format=torch.channels_last) for x in grads]
        rex.roi_align_bwd(to_device(g, gdt, "nchw"), r_dev, lv_dev, out_hw, S, aligned, grads,
                          scales, zero_init=zero_init, workspace=ws, algorithm=algo)
        torch.cuda.synchronize()
        base = 0.0 if zero_init else 7.0
        for l in range(L):
            # accumulating onto `base` adds one binary32 rounding of base + sum
            scale = aref[l] + base * 2.0 ** -20 / 1e-4
            check_bwd(from_device(grads[l]) - base, gref[l], scale, False,
                      "%s backward (%s) level %d" % (name, algo, l))
    return out


PYR = [(2, 100, 24, 40), (2, 100, 12, 20), (2, 100, 6, 10), (2, 100, 3, 5)]
SC = [0.25, 0.125, 0.0625, 0.03125]


def _pyr(c):
    return [(n, c, h, w) for (n, _, h, w) in PYR]


@pytest.mark.parametrize("gdt", ["f32", "bf16"])
@pytest.mark.parametrize("out_hw", [(7, 7), (14, 14)])
@pytest.mark.parametrize("C", [1, 3, 100, 256, 320])
def test_channels_ragged(out_hw, C, gdt):
    # channel counts that leave the last 64-channel group partial (or make it the only
    # one): the lanes past the last channel must neither read nor write
    rng = np.random.default_rng(C)
    rois = W.draw_rois(rng, 2, 19, (96, 160), (4.0, 200.0))
    run("C=%d %s g=%s" % (C, out_hw, gdt), _pyr(C), SC, rois, out_hw=out_hw, gdt=gdt)


@pytest.mark.parametrize("S", [0, 1, 2, 3])
@pytest.mark.parametrize("aligned", [True, False])
def test_sampling_and_alignment(S, aligned):
    rng = np.random.default_rng(10 + S)
    rois = _rois(rng, 29, 2, 160, 96)
    run("S=%d aligned=%d" % (S, aligned), _pyr(40), SC, rois, S=S, aligned=aligned)


@pytest.mark.parametrize("layout", ["nchw", "cl_view", "nchw_view"])
def test_layouts(layout):
    rng = np.random.default_rng(20)
    rois = _rois(rng, 23, 2, 160, 96)
    run("layout %s" % layout, _pyr(70), SC, rois, layout=layout)
    run("layout %s mask" % layout, _pyr(70), SC, rois, out_hw=(14, 14), layout=layout)


@pytest.mark.parametrize("fdt,odt,gdt", [("bf16", "bf16", "bf16"), ("bf16", "f32", "f32"),
                                         ("f32", "bf16", "bf16")])
def test_dtypes(fdt, odt, gdt):
    rng = np.random.default_rng(30)
    rois = W.draw_rois(rng, 2, 21, (96, 160), (4.0, 200.0))
    run("dtypes %s/%s/%s" % (fdt, odt, gdt), _pyr(130), SC, rois, fdt=fdt, odt=odt, gdt=gdt)
    run("dtypes %s/%s/%s mask" % (fdt, odt, gdt), _pyr(130), SC, rois, out_hw=(14, 14),
        fdt=fdt, odt=odt, gdt=gdt)


@pytest.mark.parametrize("layout", ["nchw", "nchw_view"])
@pytest.mark.parametrize("fdt,odt,gdt", [("bf16", "bf16", "bf16"), ("f32", "bf16", "f32")])
def test_layouts_dtypes(layout, fdt, odt, gdt):
    """Levels in separate channel planes with bf16 features, outputs or upstream
    gradients, on both specialised grids; 70 channels leave a partial last channel
    group."""
    rng = np.random.default_rng(35)
    rois = W.draw_rois(rng, 2, 19, (96, 160), (4.0, 200.0))
    for out_hw in ((7, 7), (14, 14)):
        run("layout %s dtypes %s/%s/%s %s" % (layout, fdt, odt, gdt, out_hw), _pyr(70), SC,
            rois, out_hw=out_hw, fdt=fdt, odt=odt, gdt=gdt, layout=layout)


def test_other_output_sizes():
    rng = np.random.default_rng(40)
    rois = _rois(rng, 17, 2, 160, 96)
    run("out 5x3", _pyr(33), SC, rois, out_hw=(5, 3))
    run("out 1x1", _pyr(33), SC, rois, out_hw=(1, 1), S=0)


def test_degenerate_boxes_and_maps():
    rng = np.random.default_rng(50)
    shapes = [(2, 70, 1, 1), (2, 70, 2, 3)]
    scales = [0.5, 0.25]
    rois = np.array([[0, 0.0, 0.0, 0.0, 0.0],          # zero size
                     [1, 0.5, 0.5, 0.5, 3.0],          # zero width
                     [0, -50, -50, -10, -10],          # entirely outside, low side
                     [1, 30, 30, 60, 60],              # entirely outside, high side
                     [0, -3, -3, 5, 5],                # straddles the origin
                     [1, 0, 0, 2, 2]], np.float32)
    lv = np.array([0, 1, 0, 1, 0, 1], np.int32)
    for S in (0, 2):
        for out_hw in ((7, 7), (14, 14), (2, 2)):
            run("degenerate S=%d %s" % (S, out_hw), shapes, scales, rois, out_hw=out_hw, S=S,
                roi_levels=lv)


def test_invalid_batch_and_level_indices():
    rng = np.random.default_rng(60)
    rois = W.draw_rois(rng, 2, 6, (96, 160), (8.0, 90.0))
    rois[0, 0] = -1.0
    rois[1, 0] = 2.0          # N = 2: names no image
    rois[2, 0] = 1.9          # truncates to image 1
    lv = np.array([0, 1, 2, 3, 7, -1, 0, 1, 2, 3, 0, 1], np.int32)
    out = run("invalid indices", _pyr(64), SC, rois, roi_levels=lv)
    o = out.cpu()
    for k in (0, 1, 4, 5):
        assert not o[k].any()


def test_one_and_zero_rois():
    rng = np.random.default_rng(70)
    rois = W.draw_rois(rng, 1, 1, (96, 160), (30.0, 60.0))
    run("K=1", [(1, 100, 24, 40), (1, 100, 12, 20)], SC[:2], rois)
    shapes = [(1, 100, 24, 40), (1, 100, 12, 20)]
    feats = [to_device(np.zeros(s, np.float32), "f32") for s in shapes]
    empty = torch.zeros((0, 5), dtype=torch.float32, device="cuda")
    lv, ws = rex.plan(feats, SC[:2], empty)
    out = rex.roi_align_fwd(feats, SC[:2], empty, lv, (7, 7), 2, True, workspace=ws)
    grads = [torch.ones(s, device="cuda") for s in shapes]
    rex.roi_align_bwd(torch.zeros((0, 100, 7, 7), device="cuda"), empty, lv, (7, 7), 2, True,
                      grads, SC[:2], zero_init=True, workspace=ws)
    torch.cuda.synchronize()
    assert out.shape == (0, 100, 7, 7)
    assert all(not g.any() for g in grads)


@pytest.mark.parametrize("out_hw", [(7, 7), (14, 14)])
def test_backward_accumulates_without_zero_init(out_hw):
    rng = np.random.default_rng(85)
    rois = W.draw_rois(rng, 2, 33, (96, 160), (4.0, 200.0))
    run("accumulate %s" % (out_hw,), _pyr(96), SC, rois, out_hw=out_hw, zero_init=False)
    run("accumulate %s bf16 grad" % (out_hw,), _pyr(96), SC, rois, out_hw=out_hw,
        zero_init=False, gdt="bf16")


def test_dense_rois_on_one_tile():
    """Many RoIs on top of each other (long tile lists, heavy duplication)."""
    rng = np.random.default_rng(86)
    base = np.array([0, 20.0, 12.0, 60.0, 44.0], np.float32)
    rois = np.tile(base, (150, 1))
    rois[:, 1:] += rng.uniform(-3, 3, (150, 4)).astype(np.float32)
    rois[:, 0] = rng.integers(0, 2, 150)
    run("150 stacked RoIs", _pyr(64), SC, rois)
    run("150 stacked RoIs bf16 grad", _pyr(64), SC, rois, gdt="bf16")
    run("150 stacked RoIs mask", _pyr(64), SC, rois, out_hw=(14, 14))
    # the cut lists' partial sums added onto existing gradients
    run("150 stacked RoIs accumulate", _pyr(64), SC, rois, zero_init=False)
    run("150 stacked RoIs mask accumulate bf16 grad", _pyr(64), SC, rois, out_hw=(14, 14),
        zero_init=False, gdt="bf16")


def test_many_long_tile_lists():
    """40 hot spots of 40 RoIs each on one image: many long tile lists, whose workgroups
    run first (longest-first tile order)."""
    rng = np.random.default_rng(87)
    shapes = [(1, 64, 128, 128), (1, 64, 64, 64), (1, 64, 32, 32), (1, 64, 16, 16)]
    centres = rng.uniform(40, 472, (40, 2))
    rows = []
    for cx, cy in centres:
        half = rng.uniform(8, 24, (40, 2))
        jit = rng.uniform(-6, 6, (40, 2))
        x1 = np.clip(cx + jit[:, 0] - half[:, 0], 0, 512)
        x2 = np.clip(cx + jit[:, 0] + half[:, 0], 0, 512)
        y1 = np.clip(cy + jit[:, 1] - half[:, 1], 0, 512)
        y2 = np.clip(cy + jit[:, 1] + half[:, 1], 0, 512)
        rows.append(np.stack([np.zeros(40), x1, y1, x2, y2], 1))
    rois = np.concatenate(rows).astype(np.float32)
    run("40 hot spots", shapes, SC, rois)
    run("40 hot spots accumulate", shapes, SC, rois, zero_init=False)
    run("40 hot spots mask bf16 grad", shapes, SC, rois, out_hw=(14, 14), gdt="bf16")


def test_plan_five_kernel_path():
    """More RoIs than the one-launch plan takes (8192): the plan runs as five kernels
    (device-wide counting, scan, fill, tile order), and the forward and the gather
    backward use its order and tile lists."""
    rng = np.random.default_rng(89)
    rois = W.draw_rois(rng, 2, 4700, (96, 160), (4.0, 200.0))
    run("9400 RoIs (five-kernel plan)", _pyr(16), SC, rois)
    run("9400 RoIs (five-kernel plan) mask", _pyr(16), SC, rois, out_hw=(14, 14))


def test_wide_tiles_on_a_large_map():
    """Maps with more 16-pixel tiles than the plan bins (one 2048 x 2048 or 4096 x 4096
    image): the tile layout widens the tiles to 32 or 64 pixels, so a gather workgroup
    owns a band of four 8 x 8 quadrants (8 x 32 pixels) of a tile instead of a whole
    16 x 16 tile (4 or 16 workgroups per tile)."""
    rng = np.random.default_rng(90)
    rois = _rois(rng, 48, 1, 8192, 8192, outside=0.05)
    run("2048 x 2048 map, 32-pixel tiles", [(1, 8, 2048, 2048)], [0.25], rois)
    # 4096 x 4096: 64-pixel tiles, 16 workgroups per tile
    rois = _rois(rng, 24, 1, 4096, 4096, outside=0.05)
    run("4096 x 4096 map, 64-pixel tiles", [(1, 4, 4096, 4096)], [1.0], rois)


def test_forward_many_rois_ragged_slices():
    """Enough RoIs that a forward workgroup takes several 64-channel slices of its RoI:
    300 channels = 4 slices + one of 44, so RoIs split 4 + 1 across two workgroups."""
    rng = np.random.default_rng(88)
    rois = W.draw_rois(rng, 2, 2048, (96, 160), (4.0, 200.0))
    run("4096 RoIs, 300 channels", _pyr(300), SC, rois, backward=False)


def test_plan_order_is_irrelevant_to_results():
    rng = np.random.default_rng(80)
    rois = W.draw_rois(rng, 2, 40, (96, 160), (4.0, 200.0))
    a = run("with plan", _pyr(96), SC, rois, backward=False)
    b = run("without plan", _pyr(96), SC, rois, use_plan=False, backward=False)
    assert torch.equal(a, b)


def test_threshold_boxes_bit_exact():
    """Boxes whose areas sit at the level thresholds, one binary32 step either side."""
    log("level map at thresholds")
    rows = []
    for side in (112.0, 224.0, 448.0):
        s = np.float32(side)
        for w in (np.nextafter(s, np.float32(0)), s, np.nextafter(s, np.float32(1e9))):
            for h in (np.nextafter(s, np.float32(0)), s, np.nextafter(s, np.float32(1e9))):
                for x in (0.0, 13.25, 300.5):
                    rows.append([0, x, x, np.float32(x) + w, np.float32(x) + h])
    rois = np.array(rows, np.float32)
    ref = oracle.level_map(rois, 4, 56.0)
    got = rex.fpn_level_map(torch.from_numpy(rois).cuda(), 4, 56.0).cpu().numpy()
    assert np.array_equal(got, ref)
    assert len(set(ref.tolist())) == 4


def test_level_map_pixel_boxes():
    """Boxes as inclusive pixel ranges (RE_BOX_PIXELS): the level map, the plan's
    levels and a forward on them, against the oracle with box_plus1; thresholds hit
    exactly (sides one below, at and one binary32 step around 112, 224, 448 minus 1)
    and random boxes with fractional corners."""
    log("level map, inclusive pixel boxes: threshold neighbourhoods and random boxes")
    rows = []
    for side in (111.0, 223.0, 447.0):
        s = np.float32(side)
        for w in (np.nextafter(s, np.float32(0)), s, np.nextafter(s, np.float32(1e9))):
            for h in (np.float32(side - 1), s, np.nextafter(s, np.float32(1e9))):
                for x in (0.0, 13.25, 300.5):
                    rows.append([0, x, x, np.float32(x) + w, np.float32(x) + h])
    rng = np.random.default_rng(91)
    rows += W.draw_rois(rng, 2, 300, (800, 1344), (4.0, 800.0)).tolist()
    rois = np.array(rows, np.float32)
    rois[:, 0] = np.minimum(rois[:, 0], 1)
    ref = oracle.level_map(rois, 4, 56.0, box_plus1=True)
    r_dev = torch.from_numpy(rois).cuda()
    got = rex.fpn_level_map(r_dev, 4, 56.0, box_pixels=True).cpu().numpy()
    assert np.array_equal(got, ref)
    assert len(set(ref.tolist())) == 4
    assert not np.array_equal(ref, oracle.level_map(rois, 4, 56.0))   # the convention matters
    # the plan computes the same levels, and the forward reads the level they name
    shapes = [(2, 16, 200, 336), (2, 16, 100, 168), (2, 16, 50, 84), (2, 16, 25, 42)]
    scales = [0.25, 0.125, 0.0625, 0.03125]
    feats_np = [rng.standard_normal(sh, dtype=np.float32) for sh in shapes]
    feats = [torch.from_numpy(f).cuda().contiguous(memory_format=torch.channels_last)
             for f in feats_np]
    lv, ws = rex.plan(feats, scales, r_dev, 56.0, box_pixels=True)
    assert np.array_equal(lv.cpu().numpy(), ref)
    out = rex.roi_align_fwd(feats, scales, r_dev, lv, (7, 7), 2, True, workspace=ws)
    torch.cuda.synchronize()
    exp = oracle.roi_align_fwd([f.astype(np.float64) for f in feats_np], scales, rois, ref,
                               7, 7, 2, True)
    check_fwd(from_device(out), exp, False, "forward on pixel-box levels")


def test_gpu_invariants():
    """Constant maps give constants; the backward conserves mass and is the adjoint."""
    log("invariants: constant, mass, adjoint (fp32 on the GPU)")
    rng = np.random.default_rng(90)
    shapes = _pyr(128)
    scales = SC
    rois = W.draw_rois(rng, 2, 50, (96, 160), (4.0, 150.0))
    r_dev = torch.from_numpy(rois).cuda()
    const = [torch.full(s, 1.5 + l, device="cuda").contiguous(memory_format=torch.channels_last)
             for l, s in enumerate(shapes)]
    lv, ws = rex.plan(const, scales, r_dev)
    out = rex.roi_align_fwd(const, scales, r_dev, lv, (7, 7), 2, True, workspace=ws)
    exp = (1.5 + lv.float())[:, None, None, None].expand_as(out)
    assert torch.allclose(out, exp, rtol=1e-6, atol=1e-6)
    g = torch.randn((rois.shape[0], 128, 7, 7), device="cuda")
    grads = [torch.empty(s, device="cuda").contiguous(memory_format=torch.channels_last)
             for s in shapes]
    rex.roi_align_bwd(g, r_dev, lv, (7, 7), 2, True, grads, scales, zero_init=True, workspace=ws)
    tot = sum(x.double().sum() for x in grads)
    assert abs(tot.item() - g.double().sum().item()) <= 1e-4 * g.abs().sum().item()
    x = [torch.randn(s, device="cuda").contiguous(memory_format=torch.channels_last)
         for s in shapes]
    y = rex.roi_align_fwd(x, scales, r_dev, lv, (7, 7), 2, True, workspace=ws)
    lhs = (y.double() * g.double()).sum().item()
    rhs = sum((a.double() * b.double()).sum().item() for a, b in zip(x, grads))
    assert abs(lhs - rhs) <= 1e-5 * (y.double().abs() * g.double().abs()).sum().item()


@pytest.mark.parametrize("out_hw", [(7, 7), (14, 14)])
def test_non_finite_features(out_hw):
    """NaN and infinities in the footprint reach exactly the bins whose samples read
    them (a zero bilinear weight times an infinity included), as in the definition."""
    rng = np.random.default_rng(80)
    shapes = _pyr(100)
    rois = W.draw_rois(rng, 2, 12, (96, 160), (6.0, 120.0))
    feats_np = _feats(rng, shapes, "f32")
    lv = oracle.level_map(rois, len(shapes), 56.0)
    planted = [np.nan, np.inf, -np.inf]
    for i, k in enumerate(range(0, rois.shape[0], 3)):
        l, b = lv[k], int(rois[k, 0])
        _, _, H, Wd = shapes[l]
        y = min(H - 1, max(0, int((rois[k, 2] + rois[k, 4]) * 0.5 * SC[l])))
        x = min(Wd - 1, max(0, int((rois[k, 1] + rois[k, 3]) * 0.5 * SC[l])))
        feats_np[l][b, (7 * i) % 100, y, x] = planted[i % 3]
        feats_np[l][b, (7 * i + 50) % 100, y, min(Wd - 1, x + 1)] = planted[(i + 1) % 3]
    log("non-finite features: %s, K=%d" % (out_hw, rois.shape[0]))
    feats = [to_device(f, "f32", "cl") for f in feats_np]
    r_dev = torch.from_numpy(rois).cuda()
    lv_dev, ws = rex.plan(feats, SC, r_dev, 56.0)
    out = rex.roi_align_fwd(feats, SC, r_dev, lv_dev, out_hw, 2, True, workspace=ws)
    torch.cuda.synchronize()
    got = from_device(out)
    ref = oracle.roi_align_fwd([as_f64(f, "f32") for f in feats_np], SC, rois, lv, *out_hw, 2,
                               True, "parity")
    assert np.isnan(ref).any() and np.isinf(ref).any(), "the planted values reach the outputs"
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.isposinf(got), np.isposinf(ref))
    assert np.array_equal(np.isneginf(got), np.isneginf(ref))
    fin = np.isfinite(ref)
    check_fwd(np.where(fin, got, 0.0), np.where(fin, ref, 0.0), False, "non-finite features")


def _odd_views(arrs):
    """bf16 channels-last views whose pixels do not lie at multiples of 4 bytes: one starting at an
    odd element (even strides), one with an odd pixel stride, in turn over the levels."""
    out = []
    for i, a in enumerate(arrs):
        n, c, h, w = a.shape
        pad = 2 if i % 2 == 0 else 1
        big = torch.empty((n, h, w, c + pad), dtype=torch.bfloat16, device="cuda")
        big.fill_(float("nan"))
        v = (big[..., 1:c + 1] if pad == 2 else big[..., :c]).permute(0, 3, 1, 2)
        v.copy_(to_device(a, "bf16", "nchw"))
        assert v.stride(1) == 1 and (v.data_ptr() % 4 != 0 or v.stride(3) % 2 == 1)
        out.append(v)
    return out


@pytest.mark.parametrize("S", [2, 0, 1])
@pytest.mark.parametrize("P", [7, 14])
def test_bf16_views_off_a_word(P, S):
    # an even channel count, but no aligned pairs of channels: same result, one head and several
    rng = np.random.default_rng(P)
    shapes, scales = [(2, 70, 25, 90), (2, 70, 13, 45)], [0.25, 0.125]
    feats = [W.f32_to_bf16_bits(rng.standard_normal(s, dtype=np.float32)) for s in shapes]
    rois = W.draw_rois(rng, 2, 24, (100, 360), (1.0, 300.0))
    r = torch.from_numpy(rois).cuda()
    views = _odd_views(feats)
    lv, ws = rex.plan(views, scales, r, 56.0)
    lv_np = oracle.level_map(rois, 2, 56.0)
    ref = oracle.roi_align_fwd([as_f64(f, "bf16") for f in feats], scales, rois, lv_np, P, P, S, True,
                               "parity")
    out = rex.roi_align_fwd(views, scales, r, lv, (P, P), S, True, workspace=ws)
    check_fwd(from_device(out), ref, True, "views off a word")
    heads = [dict(rois=r, roi_levels=lv, out_size=(p, p), sampling_ratio=S, workspace=ws) for p in (7, 14)]
    multi = rex.roi_align_fwd_multi(views, scales, heads)
    assert torch.equal(multi[P == 14], out)
