"""GPU parity of the tile-gather backward with bf16 upstream gradients (packed in LDS) where
the staged block's layout can go wrong: channel counts that leave partial groups or blocks
that are not a multiple of 16 bytes apart, gradients that do not start on 16 bytes, one and two
heads, against the CPU oracle with the tolerance of the other bf16 parity tests."""
import numpy as np
import pytest

import oracle
import paper_1906_07155_amd as rex
from paper_1906_07155_amd import workloads as W
from gpu_helpers import as_f64, check_bwd, from_device, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rex.lib()


@pytest.mark.parametrize("C", [1, 2, 3, 63, 64, 66, 100, 136])
@pytest.mark.parametrize("offset", [0, 1, 2, 4])
def test_blocks(C, offset):
    log("gather bf16 C=%d, gradient starting %d values into its storage" % (C, offset))
    rng = np.random.default_rng(C)
    shapes = [(2, C, 25, 41), (2, C, 13, 21)]
    scales = [0.25, 0.125]
    heads, ref = [], [0.0, 0.0]
    scale = [0.0, 0.0]
    grads = [torch.full(s, 3.0, device="cuda").contiguous(memory_format=torch.channels_last)
             for s in shapes]
    for P, n in ((7, 9), (14, 5)):
        rois = W.draw_rois(rng, 2, n, (100, 164), (4.0, 150.0))
        r = torch.from_numpy(rois).cuda()
        lv, ws = rex.plan(grads, scales, r, 28.0)
        g = W.f32_to_bf16_bits(rng.standard_normal((2 * n, C, P, P), dtype=np.float32))
        store = torch.empty(g.size + offset, dtype=torch.int16, device="cuda")
        view = store[offset:].view(g.shape)
        view.copy_(torch.from_numpy(g.view(np.int16)))
        heads.append({"grad_out": view.view(torch.bfloat16), "rois": r, "roi_levels": lv,
                      "out_size": (P, P), "workspace": ws})
        lv_np = lv.cpu().numpy()
        g64 = as_f64(g, "bf16")
        one = oracle.roi_align_bwd(g64, shapes, scales, rois, lv_np, P, P, 2, True, "parity")
        mag = oracle.roi_align_bwd(np.abs(g64), shapes, scales, rois, lv_np, P, P, 2, True, "parity")
        h = heads[-1]
        rex.roi_align_bwd(h["grad_out"], r, lv, (P, P), 2, True, grads, scales, workspace=ws,
                          algorithm="gather")
        for l in range(2):
            check_bwd(from_device(grads[l]), one[l], mag[l], False, "one head %d level %d" % (P, l))
            ref[l] = ref[l] + one[l]
            scale[l] = scale[l] + mag[l]
    rex.roi_align_bwd_multi(heads, grads, scales)
    for l in range(2):
        check_bwd(from_device(grads[l]), ref[l], scale[l], False, "two heads level %d" % l)
