"""GPU parity of the contiguous-NCHW forward where a workgroup takes several chunks of
channels: runs that end in a partial chunk or past the channels, RoIs with no valid sample,
with every sample tap distinct and with non-finite features beside the map's edge, against
the CPU oracle (tolerances of the other forward tests)."""
import numpy as np
import pytest

from paper_1906_07155_amd import workloads as W
from test_gpu_edges import run

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("fdt,odt", [("f32", "f32"), ("bf16", "bf16"), ("f32", "bf16")])
@pytest.mark.parametrize("P,K,C", [(7, 310, 67), (7, 1100, 33), (14, 260, 35), (7, 5, 9), (14, 3, 1)])
def test_runs(P, K, C, fdt, odt):
    rng = np.random.default_rng(K)
    rois = W.draw_rois(rng, 2, (K + 1) // 2, (96, 160), (2.0, 160.0))[:K]
    rois[0, 1:] = [300, 10, 340, 40]           # off the map
    rois[1, 1:] = [-40, -30, 20, 20]           # half off it
    rois[2, 0] = 7                             # of an image that is not there
    run("runs", [(2, C, 24, 40), (2, C, 12, 20)], [0.25, 0.125], rois, out_hw=(P, P), fdt=fdt,
        odt=odt, layout="nchw", backward=False)
