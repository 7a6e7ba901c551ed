"""The plain arithmetic of ``csrc/bounds.h``, which keeps row and tile indices
inside their buffers, of ``csrc/deal.h``, which deals work items to lists, and of
``csrc/errors.h``, compiled with g++ and run on the host."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from paper_2606_22541_amd import build
from paper_2606_22541_amd import moe_stage as C

HERE = os.path.dirname(os.path.abspath(__file__))
BIG = 2**31 - 1

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("bounds") / "bounds")
    cmd = ["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
           "-I", build.CSRC, "-I", build.INCLUDE, os.path.join(HERE, "bounds_main.cpp"), "-o", exe]
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


def test_tile_offsets_fit_32_bits(driver):
    """Every row length that the stage takes (256 rows of it fit) gets tiles
    whose rows' byte offsets fit, and the largest such up to the tiles' own
    limit of 10 blocks."""
    edge = [(2**31 - 1) // (64 * b) for b in (8, 9, 10)]
    cols = sorted({128, 7168, 2**21} | {e // 128 * 128 + 128 * j for e in edge for j in (-1, 0, 1)})
    got = _run(driver, "blocks", len(cols), *[v for c in cols for v in (10, c)])
    for c, blocks, taken in zip(cols, got[::2], got[1::2]):
        assert taken == int(256 * c * 2 < 2**31), c
        if taken:
            assert 32 * blocks * c * 2 < 2**31, (c, blocks)
            assert blocks == 10 or 32 * (blocks + 1) * c * 2 >= 2**31, (c, blocks)


def test_descriptors_are_taken_up_to_the_least_tile():
    """Row lengths on both sides of what the least tile can address are
    accepted and refused by the library (host only)."""
    for cols, ok in ((4194176, True), (4194304, False), (3355392, True), (3355520, True)):
        for d, f in ((cols, 128), (128, cols)):
            desc = C.make_desc(d, f, 8, 0, 1, 2, 160, n_slots=1)
            if ok:
                assert C.moe_stage_workspace_bytes(desc) > 0
            else:
                with pytest.raises(C.MoEStageError) as e:
                    C.moe_stage_workspace_bytes(desc)
                assert e.value.status == C.MOE_EINVAL


def test_a_stalled_pass_is_reported_before_any_other_error(driver):
    """All bits of the error word are cleared together, so the one that says
    that rows are wrong through no fault of the caller must not be hidden."""
    words = list(range(32))
    order = ((16, C.MOE_EHIP), (1, C.MOE_EBADID), (2, C.MOE_EBADLAYER), (8, C.MOE_EBADCOUNT), (4, C.MOE_ETIMEOUT))
    want = [next((s for bit, s in order if w & bit), C.MOE_OK) for w in words]
    assert _run(driver, "status", len(words), *words) == want


@pytest.mark.parametrize("row_bytes", [896, 1024])
@pytest.mark.parametrize("phases", [1, 2, 3])
@pytest.mark.parametrize("P", [1, 3, 7, 8, 16, 24, 248, 256, 304])
def test_every_item_is_dealt_once_and_few_are_spread(driver, P, phases, row_bytes):
    """All items of both products are in the lists exactly once, the fixed ones
    are the first of each list, and with up to three quarters as many gate/up items
    as workgroups no list has more than its even share (rows of 1 KB and more;
    shorter rows, and more items, fill the lists one after the other)."""
    rng = np.random.default_rng(P)
    sizes = [(0, 0), (1, 1), (8, 8), (9, 1), (32, 56), (128, 448), (192, 9), (193, 9), (255, 1), (256, 224), (257, 3000)]
    sizes += [tuple(int(v) for v in 2**rng.uniform(0, 12, 2)) for _ in range(12)]
    for g, d in sizes:
        out = _run(driver, "deal", P, g, d, phases, row_bytes)
        lists, run, fixed, rest = out[0], out[1], out[2:2 + P], out[2 + P:]
        assert lists == (1 if P % 8 else 8)
        got = {}
        for p in range(2):
            for y in range(lists):
                n = rest.pop(0)
                got[p, y], rest = rest[:n], rest[n:]
        assert not rest
        for p, n in ((0, g if phases & 1 else 0), (1, d if phases & 2 else 0)):
            assert sorted(i for y in range(lists) for i in got[p, y]) == list(range(n)), (P, g, d, p)
        for y in range(lists):
            assert [f for f in fixed[y::lists] if f >= 0] == got[0, y][:run], (P, g, d, y)
            share = -(-g // lists)
            few = row_bytes >= 1024 and 4 * share <= 3 * (P // lists)
            if phases & 1 and few:
                assert len(got[0, y]) <= max(share, 1), (P, g, d, y)
            if phases & 1 and g <= P and not few:
                assert len(got[0, y]) == min(P // lists, max(0, g - y * (P // lists))), (P, g, d, y)


def test_products_are_split_where_other_streams_can_use_the_gpu(driver):
    """One launch on one stream, for several rounds and for short streams of
    weights; a launch per product for one round on several streams."""
    MB = 2**20
    cases = []                                 # streams, fp8, items, bytes, workgroups, expected
    for streams in (1, 2, 3):
        for fp8 in (0, 1):
            for items in (1, 256, 257, 1056):
                for size in (159, 160, 704):
                    want = streams >= (2 if fp8 else 3) and items <= 256 and size >= 160
                    cases.append((streams, fp8, items, size * MB, 256, want))
    got = _run(driver, "split", len(cases), *[v for c in cases for v in c[:5]])
    assert got == [int(c[5]) for c in cases]
