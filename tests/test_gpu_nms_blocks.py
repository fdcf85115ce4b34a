"""GPU parity of box_nms against the CPU oracle (exact: the definition fixes every decision)
where the block-parallel form can go wrong: box counts around the 64-box blocks and the
per-wave block counts, overlap lists longer than the LDS holds, long chains of dependent
decisions, every kind of threshold, and boxes that are no boxes."""
import numpy as np
import pytest

import oracle
from paper_1906_07155_amd import workloads as W
from test_gpu_nms import run

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _boxes(n, seed=0, size=(100, 160), sides=(8.0, 60.0)):
    rng = np.random.default_rng(seed)
    b, s, _ = W.draw_proposals(rng, 1, n, size, sides, 0.5)
    return b, s


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 129, 192, 193, 320, 1024, 1025, 3072, 3073])
def test_sizes(n):
    b, s = _boxes(n, n)
    run("n=%d" % n, b, s, 0.5)
    run("n=%d limited" % n, b, s, 0.6, max_keep=max(1, n // 7))


@pytest.mark.parametrize("thr", [-1.0, 0.0, 1e-30, 0.3, 1.0, 2.0, float("inf")])
def test_thresholds(thr):
    b, s = _boxes(500, 3)
    run("thr", b, s, thr, cats=(np.arange(500) % 3 - 1).astype(np.int32))


def test_dense_lists():
    # every box overlaps nearly every other: lists far longer than the LDS entries
    rng = np.random.default_rng(5)
    n = 2500
    b = np.tile(np.array([10, 10, 60, 50], np.float32), (n, 1)) + \
        rng.uniform(-4, 4, (n, 4)).astype(np.float32)
    run("dense", b, rng.uniform(0, 1, n).astype(np.float32), 0.5)
    run("identical", np.tile(b[:1], (700, 1)), np.full(700, 0.5, np.float32), 0.9)


@pytest.mark.parametrize("objects,jitter", [(10, 0.1), (20, 0.15), (3, 0.05)])
@pytest.mark.parametrize("thr", [0.5, 0.7])
def test_crowds(objects, jitter, thr):
    # the largest call, its boxes around a few objects of each image as a detector's proposals
    # are: hundreds of thousands of overlap words, nearly all boxes removed, and rows that wait
    # for more words than a wave keeps
    rng = np.random.default_rng(objects)
    b = []
    for _ in range(2):
        c = rng.uniform(0, (1333, 800), (objects, 2))
        wh = np.exp(rng.uniform(np.log(40), np.log(400), (objects, 2)))
        o = rng.integers(0, objects, 4096)
        b.append(np.concatenate([c - wh / 2, c + wh / 2], 1)[o] +
                 rng.uniform(-jitter, jitter, (4096, 4)) * np.tile(wh[o], 2))
    run("crowds", np.concatenate(b).astype(np.float32), rng.uniform(0, 1, 8192).astype(np.float32), thr,
        cats=np.repeat(np.arange(2, dtype=np.int32), 4096))


@pytest.mark.parametrize("shift", [1, 64, 65])
def test_chains(shift):
    # box r overlaps only boxes r - shift and r + shift in rank order: every decision waits
    # for the one before it, as many rounds as the blocks allow
    n = 1500
    pos = np.arange(n)
    x = (pos // shift).astype(np.float32) * 4.0
    y = (pos % shift).astype(np.float32) * 20.0
    b = np.stack([x, y, x + 10, y + 10], 1).astype(np.float32)
    s = (1.0 - pos / (2.0 * n)).astype(np.float32)
    run("chain", b, s, 0.4)


def test_odd_boxes():
    rng = np.random.default_rng(9)
    b, s = _boxes(400, 11)
    b[3] = [np.nan, 1, 5, 9]
    b[50] = [0, 0, np.inf, np.inf]
    b[51] = [-np.inf, 0, 10, 10]
    b[70:80] = b[70:80, [2, 3, 0, 1]]                  # inverted
    b[90:100, 2] = b[90:100, 0]                        # no width
    b[100:140] = b[100:140] * np.float32(1e-22)        # areas among the denormals
    b[140:150] = b[140:141] * np.float32(1e-22)
    b[150:160] = b[150:151] * np.float32(1e18)         # areas overflow
    s[200:210] = np.nan
    s[210:220] = -0.0
    s[220:230] = 0.0
    s[230:240] = np.inf
    for thr in (-0.5, 0.0, 0.5, 0.9):
        run("odd", b, s, thr)
