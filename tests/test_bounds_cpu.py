"""The plain arithmetic of ``csrc/bounds.h``, which keeps row and tile indices
inside their buffers, compiled with g++ and run on the host."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from paper_2606_22541_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
BIG = 2**31 - 1

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("bounds") / "bounds")
    cmd = ["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
           "-I", build.CSRC, os.path.join(HERE, "bounds_main.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0 and "sanitize" in r.stderr:
        pytest.skip("sanitizer runtime not available: " + r.stderr[-300:])
    assert r.returncode == 0, r.stderr
    return exe


def _run(driver, what, *numbers):
    r = subprocess.run([driver, what], input=" ".join(str(int(n)) for n in numbers), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return [int(v) for v in r.stdout.split()]


@pytest.mark.parametrize("counts,n", [
    ([BIG, BIG, BIG], 300),                          # the third total wraps in 32 bits
    ([10, BIG, 5, BIG, BIG], 300),
    ([BIG] * 256, BIG),
    ([-1, -2**31, 7, 0, 300], 300),
    ([1 << 25] * 256, BIG),                          # 64 lanes of valid counts pass 2^31
    ([100, 100, 100], 300),
    ([100, 100, 101], 300),
    ([0] * 65 + [3], 0),
])
def test_grouped_counts_never_pass_the_buffer(driver, counts, n):
    got = _run(driver, "counts", n, len(counts), *counts)
    want = oracle.grouped_counts(counts, n).tolist()
    assert got[:-1] == want
    assert sum(got[:-1]) <= n
    assert got[-1] == int(want != list(counts))


def test_grouped_counts_of_any_value(driver):
    rng = np.random.default_rng(7)
    for _ in range(200):
        n = int(rng.integers(0, 2**int(rng.integers(1, 32)) - 1))
        top = 2**int(rng.integers(1, 32)) - 1
        counts = rng.integers(-top, top + 1, int(rng.integers(1, 257))).tolist()
        counts = [c if rng.random() < 0.5 else 0 for c in counts]
        got = _run(driver, "counts", n, len(counts), *counts)
        assert got[:-1] == oracle.grouped_counts(counts, n).tolist()
