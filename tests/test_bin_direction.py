"""Which way the costs run over the cell index, as the binned schedule's queue
order uses it (within a bin the order runs against the index where they grow): the
host build of the device code against the covariance of block and bin in exact
integers, with last blocks from one cell to a full one, fields that rise, fall,
are mostly cheap or dear, or have no direction, and the largest counts."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2112_05834_amd", "csrc")
BLOCK = 4096


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("dir") / "bin_direction")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           "-I", CSRC, os.path.join(HERE, "bin_direction_driver.cpp"), "-o", exe])
    return exe


def _run(driver, fields):
    text = "\n".join("%d %s" % (len(c), " ".join(str(int(v)) for v in np.concatenate(c))) for c in fields)
    r = subprocess.run([driver], input=text, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return [int(v) for v in r.stdout.split()]


def _counts(bins):
    """[blocks][9] of a cell's bins in index order."""
    return [np.append(np.bincount(bins[lo:lo + BLOCK], minlength=8), 1) for lo in range(0, len(bins), BLOCK)]


def _grows(counts):
    c = [[int(v) for v in row[:8]] for row in counts]
    n = sum(map(sum, c))
    sk = sum(k * sum(row) for k, row in enumerate(c))
    sb = sum(b * v for row in c for b, v in enumerate(row))
    return int(n * sum(k * b * v for k, row in enumerate(c) for b, v in enumerate(row)) - sk * sb > 0)


@pytest.mark.parametrize("n", [1, 100, 4096, 4097, 8192, 8200, 12305, 16384, 16411, 20481, 65537])
def test_direction_is_the_covariance(driver, n):
    rng = np.random.Generator(np.random.PCG64(n))
    fields, known = [], []
    for cheap in (0.0, 0.5, 0.8, 0.99):              # share of the cells in bin 0, or in bin 7
        for low in (0, 7):
            b = np.where(rng.random(n) < cheap, low, rng.integers(0, 8, n))
            for way, f in ((1, np.sort(b)), (0, np.sort(b)[::-1]), (None, b)):
                fields.append(_counts(f))
                several = len(fields[-1]) > 1 and (fields[-1][0][:8] * len(b) != np.bincount(b, minlength=8) * min(n, BLOCK)).any()
                known.append(way if several else None)
    fields.append(_counts(np.full(n, 3)))
    known.append(0)                                  # all alike: no direction
    got = _run(driver, fields)
    assert got == [_grows(f) for f in fields]
    for g, k, f in zip(got, known, fields):
        assert k is None or g == k
        assert len(f) > 1 or g == 0                  # one block has no direction


def test_direction_at_the_largest_counts(driver):
    """2^31 - 1 cells: 524288 blocks, the last one a cell short."""
    nblk = 1 << 19
    up = np.zeros((nblk, 9), np.int64)
    up[: nblk // 2, 0] = BLOCK
    up[nblk // 2:, 7] = BLOCK
    up[-1, 7] -= 1
    down = np.zeros_like(up)
    down[: nblk // 2, 7] = BLOCK
    down[nblk // 2:, 0] = BLOCK
    down[-1, 0] -= 1
    assert _run(driver, [up, down]) == [1, 0]
