"""GPU parity of the tile-gather backward of binary32 14x14 grids, whose blocks are staged in
two parts of bin rows: gradients that start off 16 bytes (the one-element copies), partial
channel groups, and RoIs whose parts meet different tiles or none, against the CPU oracle."""
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
def test_parts(C, offset):
    log("gather parts C=%d, gradient starting %d values into its storage" % (C, offset))
    rng = np.random.default_rng(C)
    shapes, scales = [(2, C, 50, 41), (2, C, 25, 21)], [0.25, 0.125]
    rois = np.concatenate([
        W.draw_rois(rng, 2, 40, (200, 164), (2.0, 200.0)),      # more than one batch per tile
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
