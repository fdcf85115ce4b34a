"""GPU parity of the tile-gather backward of 14x14 grids, against the CPU oracle.  In full grids
binary32 blocks are staged in two parts of bin rows; in few workgroups whole, and bf16 blocks in
two slots.  Gradients that start off 16 bytes (the one-element copies), partial channel groups,
RoIs whose parts meet different tiles or none, and grids on both sides of the rule."""
import numpy as np
import pytest

import oracle
import paper_1906_07155_amd as rex
from paper_1906_07155_amd import workloads as W
from gpu_helpers import check_bwd, from_device, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rex.lib()


@pytest.mark.parametrize("C", [1, 5, 64, 70])
@pytest.mark.parametrize("offset", [0, 1, 2])
@pytest.mark.parametrize("images", [2, 9])
def test_parts(C, offset, images):
    # two images: few workgroups; nine, and more than 1536 RoIs x channel groups: two parts
    log("gather parts C=%d, gradient starting %d values into its storage, %d images" % (C, offset, images))
    rng = np.random.default_rng(C)
    shapes, scales = [(images, C, 50, 41), (images, C, 25, 21)], [0.25, 0.125]
    rois = np.concatenate([
        # more than one batch per tile
        W.draw_rois(rng, images, 40 if images == 2 else 180 // -(-C // 64), (200, 164), (2.0, 200.0)),
        np.array([[0, 5, -60, 90, 40], [1, 5, 150, 90, 290], [0, 20, 0, 60, 200]], np.float32)])
    grads = [torch.full(s, 3.0, device="cuda").contiguous(memory_format=torch.channels_last)
             for s in shapes]
    r = torch.from_numpy(rois).cuda()
    lv, ws = rex.plan(grads, scales, r, 56.0)
    g = rng.standard_normal((rois.shape[0], C, 14, 14), dtype=np.float32)
    store = torch.empty(g.size + offset, device="cuda")
    view = store[offset:].view(g.shape)
    view.copy_(torch.from_numpy(g))
    lv_np = lv.cpu().numpy()
    g64 = g.astype(np.float64)
    ref = oracle.roi_align_bwd(g64, shapes, scales, rois, lv_np, 14, 14, 2, True, "parity")
    mag = oracle.roi_align_bwd(np.abs(g64), shapes, scales, rois, lv_np, 14, 14, 2, True, "parity")
    rex.roi_align_bwd(view, r, lv, (14, 14), 2, True, grads, scales, workspace=ws,
                      algorithm="gather")
    for l in range(2):
        check_bwd(from_device(grads[l]), ref[l], mag[l], False, "parts level %d" % l)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("C", [65, 66, 72])
@pytest.mark.parametrize("images", [1, 18])
def test_grid_forms(images, C, dt):
    # 58 and 1044 workgroups, on both sides of the rule's 1024; bf16 channel counts whose blocks
    # start at odd values, at odd words and at multiples of 16 bytes; one head and two
    log("gather forms: %d images, C=%d, %s" % (images, C, dt))
    rng = np.random.default_rng(C)
    shapes, scales = [(images, C, 100, 41), (images, C, 50, 21)], [0.25, 0.125]
    grads = [torch.full(s, 3.0, device="cuda").contiguous(memory_format=torch.channels_last) for s in shapes]
    heads, ref, mag = [], [0.0, 0.0], [0.0, 0.0]
    for P, n in ((7, 4), (14, 5)):
        rois = W.draw_rois(rng, images, n, (400, 164), (4.0, 300.0))
        r = torch.from_numpy(rois).cuda()
        lv, ws = rex.plan(grads, scales, r, 56.0)
        g = torch.from_numpy(rng.standard_normal((rois.shape[0], C, P, P), dtype=np.float32))
        if dt == "bf16":
            g = g.to(torch.bfloat16)
        g64 = g.double().numpy()
        one = oracle.roi_align_bwd(g64, shapes, scales, rois, lv.cpu().numpy(), P, P, 2, True, "parity")
        am = oracle.roi_align_bwd(np.abs(g64), shapes, scales, rois, lv.cpu().numpy(), P, P, 2, True, "parity")
        gd = g.cuda()
        rex.roi_align_bwd(gd, r, lv, (P, P), 2, True, grads, scales, workspace=ws, algorithm="gather")
        for l in range(2):
            check_bwd(from_device(grads[l]), one[l], am[l], False, "one head %d level %d" % (P, l))
            ref[l], mag[l] = ref[l] + one[l], mag[l] + am[l]
        heads.append(dict(grad_out=gd, rois=r, roi_levels=lv, out_size=(P, P), workspace=ws))
    for pair in (heads, heads[::-1]):
        rex.roi_align_bwd_multi(pair, grads, scales)
        for l in range(2):
            check_bwd(from_device(grads[l]), ref[l], mag[l], False, "two heads level %d" % l)
