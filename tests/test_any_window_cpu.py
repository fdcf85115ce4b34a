"""The sample window of the RoIAlign kernels for any sampling ratio, on the CPU: `any_weight`
looks only at the samples that can tap a pixel.  Its own source (adaptive.hip) is compiled for
the host and compared, for every pixel near a box and near the map's edges, with the sum over
all samples of the bin: the weight bit for bit, and whether any sample taps the pixel.  The
hardware reciprocal is within a unit in the last place of the quotient; the comparison runs
with the quotient and with its neighbours on both sides.
"""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1906_07155_amd", "csrc")

DRIVER = r"""
#include "hip/hip_runtime.h"
static int g_ulp;
static float emu_rcp(float x) {
    float r = 1.0f / x;
    for (int i = 0; i < g_ulp; ++i) r = std::nextafter(r, INFINITY);
    for (int i = 0; i > g_ulp; --i) r = std::nextafter(r, 0.0f);
    return std::fabs(x) < 1.17549435e-38f ? std::copysign(INFINITY, x) : r;
}
#define __builtin_amdgcn_rcpf emu_rcp
#include "common.hpp"
namespace rex {
constexpr int kAnyGrid = kGridCap;
#include "any_functions.inc"
}
using namespace rex;
int main(int argc, char **argv) {
    struct Box { float c1, c2, scale; int aligned, P, S, size; };
    FILE *f = std::fopen(argv[1], "rb");
    Box b;
    long pixels = 0, tapped = 0, bad = 0;
    while (std::fread(&b, sizeof b, 1, f) == 1) {
        const Axis a = axis_setup(b.c1, b.c2, b.scale, b.aligned, b.P, b.S);
        std::vector<int> near = {0, 1, 2, b.size - 3, b.size - 2, b.size - 1};
        for (int p = 0; p < b.P; ++p) {
            float pos[kAnyGrid];
            for (int i = 0; i < a.grid; ++i) {
                pos[i] = any_position(a, p, i, b.size);
                if (pos[i] >= 0.0f)
                    for (int d = -2; d <= 3; ++d) near.push_back((int)pos[i] + d);
            }
            std::sort(near.begin(), near.end());
            near.erase(std::unique(near.begin(), near.end()), near.end());
            for (int X : near) {
                if (X < 0 || X >= b.size) continue;
                float w = 0.0f;
                bool hit = false;
                for (int i = 0; i < a.grid; ++i) {
                    const Tap t = axis_tap(a, p, i, b.size);
                    if (t.lo < 0) continue;
                    w += t.lo == X ? t.wlo : 0.0f;
                    w += t.hi == X && t.hi != t.lo ? t.whi : 0.0f;
                    hit = hit || t.lo == X || t.hi == X;
                }
                for (g_ulp = -1; g_ulp <= 1; ++g_ulp) {
                    bool h = false;
                    const float got = any_weight(pos, a, p, X, b.size, h);
                    if (got != w || h != hit) {
                        if (bad++ < 10)
                            std::printf("box %.9g %.9g scale %g aligned %d P %d S %d size %d: bin %d "
                                        "pixel %d: %.9g hit %d, all samples %.9g hit %d\n", b.c1, b.c2,
                                        b.scale, b.aligned, b.P, b.S, b.size, p, X, got, h, w, hit);
                    }
                }
                ++pixels;
                tapped += hit;
            }
        }
    }
    std::printf("pixels %ld tapped %ld bad %ld\n", pixels, tapped, bad);
    return bad != 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = str(tmp_path_factory.mktemp("any"))
    src = open(os.path.join(CSRC, "adaptive.hip")).read()
    a = src.index("__device__ __forceinline__ float any_position(")
    b = src.index("// Positions of every sample of both axes into pos")
    with open(os.path.join(d, "any_functions.inc"), "w") as f:
        f.write(src[a:b])
    with open(os.path.join(d, "driver.cpp"), "w") as f:
        f.write(DRIVER)
    out = os.path.join(d, "driver")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-Wno-attributes",
                           "-I" + os.path.join(HERE, "emulate"), "-I" + d, "-I" + CSRC,
                           os.path.join(d, "driver.cpp"), "-o", out])
    return out


BOX = np.dtype([("c1", "f4"), ("c2", "f4"), ("scale", "f4"), ("aligned", "i4"), ("P", "i4"),
                ("S", "i4"), ("size", "i4")])


def _check(driver, tmp_path, boxes):
    path = str(tmp_path / "boxes.bin")
    np.array(boxes, BOX).tofile(path)
    r = subprocess.run([driver, path], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[3]) > 0, r.stdout   # some pixel is tapped


def _random(rng, n, size, scale, lengths, starts):
    out = []
    for _ in range(n):
        c1 = np.float32(starts(rng) / scale)
        ln = np.exp(rng.uniform(*np.log(lengths))) / scale
        out.append((c1, np.float32(c1 + ln), scale, int(rng.integers(2)), int(rng.choice([7, 14])),
                    int(rng.choice([0, 1, 3, 4, 5, 8, 16, 33, 64])), size))
    return out


@pytest.mark.parametrize("size,scale", [(25, 1 / 32), (336, 0.25), (1, 0.125), (2, 1.0),
                                        (4096, 1.0), (60000, 1.0)])
def test_boxes(driver, tmp_path, size, scale):
    rng = np.random.default_rng(size)
    boxes = _random(rng, 400, size, scale, (0.3, 2.0 * size + 2), lambda r: r.uniform(-size, size))
    # at the map's edges, where samples are cut and clamped
    for at in (-1.0, -0.5, 0.0, 0.5, 1.0, size - 1.0, size - 0.5, float(size), size + 0.5):
        boxes += _random(rng, 40, size, scale, (1e-6, 3.0), lambda r: at + r.uniform(-1e-4, 1e-4))
        boxes += _random(rng, 40, size, scale, (1e-3, 8.0), lambda r: at + r.normal() * 0.5)
    _check(driver, tmp_path, boxes)


def test_samples_closer_than_a_unit(driver, tmp_path):
    # boxes a few units in the last place wide: a bin's samples round to one position, at the
    # map's edges to the cut or to the clamped one
    boxes = []
    for size, scale in ((336, 0.25), (25, 1.0), (4096, 0.5)):
        for aligned in (0, 1):
            for x in (-1.0, -0.9, -0.5, 0.0, 0.5, 3.0, 17.25, size - 1.0, size - 0.5, size, size + 0.5):
                x1 = np.float32((x + 0.5 * aligned) / scale)
                for steps in (1, 2, 5, 40):
                    x2 = x1
                    for _ in range(steps):
                        x2 = np.nextafter(x2, np.float32(np.inf))
                    for S in (1, 3, 4, 64):
                        boxes.append((x1, x2, scale, aligned, 7, S, size))
    _check(driver, tmp_path, boxes)


def test_clamped_samples(driver, tmp_path):
    # samples left of pixel 0 are moved onto it and tap pixel 1 with weight zero
    boxes = [(np.float32(-0.9 + 0.5 + 0.01 * i), np.float32(-0.9 + 0.5 + 0.01 * i + 0.35), 1.0, 1, 7, 4, 20)
             for i in range(60)]
    _check(driver, tmp_path, boxes)


def test_values_that_are_no_boxes(driver, tmp_path):
    v = [np.float32(x) for x in (0, 5, 1e-38, 1e-42, 1e30, -1e30, 3e38, -3e38, np.inf, -np.inf, np.nan)]
    _check(driver, tmp_path, [(a, b, 1.0, al, 7, S, 30) for a in v for b in v for al in (0, 1)
                              for S in (0, 1, 4, 64)])
