"""The deciding half of greedy suppression run on the CPU (``emulate/emu_nms.cpp``: its own
source, one fiber per work-item, AddressSanitizer and UndefinedBehaviorSanitizer) against a walk
in rank order, on overlaps that no boxes need to have: random ones from hardly any to nearly
all, crowds, chains in which every decision waits for the one before it, and rows that wait for
more words than a wave keeps.  The waves wait for each other's decisions, so a run that does not
end in time is a failure.
"""
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    sys.path.insert(0, os.path.join(HERE, "emulate"))
    import emu_build
    return emu_build.build_nms(str(tmp_path_factory.mktemp("nms")))


def _check(emu, tmp_path, overlaps, lg):
    """overlaps: bool [n, n]; row i's entries j < i count."""
    n = overlaps.shape[0]
    inp, out = str(tmp_path / "in.bin"), str(tmp_path / "out.bin")
    kept = np.zeros(n, bool)
    with open(inp, "wb") as f:
        np.array([n, lg], np.int32).tofile(f)
        for i in range(n):
            js = np.flatnonzero(overlaps[i, :i]).astype(np.int32)
            np.array([js.size], np.int32).tofile(f)
            js.tofile(f)
            kept[i] = not kept[js].any()
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=1",
               UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([emu, inp, out], capture_output=True, text=True, timeout=120, env=env)
    assert r.returncode == 0 and "done" in r.stdout, (r.stdout + r.stderr)[-3000:]
    assert np.array_equal(np.fromfile(out, np.uint8).astype(bool), kept)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 130, 1000, 1024, 1100])
@pytest.mark.parametrize("density", [0.001, 0.05, 0.9])
def test_random(emu, tmp_path, n, density):
    rng = np.random.default_rng(n)
    _check(emu, tmp_path, rng.random((n, n)) < density, 3 if n % 2 else 1)


@pytest.mark.parametrize("step", [1, 63, 64, 65, 200])
def test_chains(emu, tmp_path, step):
    n = 1030
    i = np.arange(n)
    _check(emu, tmp_path, (i[:, None] - i[None, :]) == step, 3)


@pytest.mark.parametrize("width", [70, 400])
def test_slides(emu, tmp_path, width):
    # every box overlaps the `width` before it: each block waits for the one before it, with as
    # many waiting words as its rows have neighbours
    n = 1100
    i = np.arange(n)
    d = i[:, None] - i[None, :]
    _check(emu, tmp_path, (d > 0) & (d < width), 1)


def test_crowds(emu, tmp_path):
    rng = np.random.default_rng(3)
    n = 1500
    crowd = rng.integers(0, 6, n)
    _check(emu, tmp_path, (crowd[:, None] == crowd[None, :]) & (rng.random((n, n)) < 0.8), 3)


def test_more_waiting_words_than_a_wave_keeps(emu, tmp_path):
    # the blocks before the last hang on one chain, and every row of the last overlaps one box of
    # each of them: hundreds of words that can only wait
    n = 64 * 16
    o = np.zeros((n, n), bool)
    i = np.arange(n)
    o[i[64:-64], i[64:-64] - 64] = True
    o[-64:, :-64] = np.random.default_rng(4).random((64, n - 64)) < 0.03
    _check(emu, tmp_path, o, 3)
    _check(emu, tmp_path, o, 1)
