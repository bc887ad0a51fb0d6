"""Bounds of the workgroup integration's LU and solves, checked on the CPU.

`tests/wide_lu_m_bounds.c` replays their loops, loads and guards thread by
thread, with every LDS and HBM buffer allocated on its own at exactly the kernel's
size, built with AddressSanitizer, for every state size of the workgroup kernel
(65..256): two, three and four groups of rows, every width of the last panel.
Uninitialised buffers and padding rows hold NaN. The factors, rows' order and
first zero pivot must equal the oracle's in every bit, the solutions to rounding.
"""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import oracle as O

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "wide_lu_m_bounds.c")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("gcc") is None:
        pytest.skip("gcc not available")
    d = tmp_path_factory.mktemp("wlm")
    out = str(d / "wide_lu_m_bounds")
    subprocess.check_call(["gcc", "-std=gnu11", "-O1", "-g", "-fno-omit-frame-pointer", "-ffp-contract=off",
                           "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-o", out, SRC, "-lm"])
    return out, str(d)


def _read(path):
    raw, off = open(path, "rb").read(), 0

    def take(dtype, count):
        nonlocal off
        v = np.frombuffer(raw, dtype=dtype, count=count, offset=off)
        off += v.nbytes
        return v

    while off < len(raw):
        n, ld, info = (int(v) for v in take(np.int32, 3))
        yield (n, info, take(np.float64, n * n).reshape(n, n), take(np.float64, n * n).reshape(n, n),
               take(np.int32, n), take(np.float64, n))


# every size on random matrices; the other patterns on windows that hold every
# width of the last panel, in each number of row groups
CASES = [(0, 65, 256)] + [(p, lo, lo + 15) for p in (1, 2, 3, 4, 5) for lo in (113, 177, 241)]


@pytest.mark.parametrize("pattern,n_lo,n_hi", CASES)
def test_integration_lu_in_bounds(exe, pattern, n_lo, n_hi):
    path, d = exe
    out = os.path.join(d, "r_%d_%d.bin" % (pattern, n_lo))
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:exitcode=23")
    r = subprocess.run([path, out, str(n_lo), str(n_hi), str(pattern)], env=env, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    seen = []
    for n, info, A, F, pos, x in _read(out):
        seen.append(n)
        LU, piv, inf = O.lu(A)
        rows = np.arange(n)
        for k, p in enumerate(piv):
            rows[[k, p]] = rows[[p, k]]
        assert info == inf == {3: n, 4: n // 2 + 1}.get(pattern, 0), n
        assert np.array_equal(pos[rows], np.arange(n)), n
        assert np.array_equal(F, LU), n
        if pattern in (0, 1, 2):
            xo = O.lu_solve(LU, piv, np.arange(n, dtype=float) + 1)
            assert np.max(np.abs(x - xo)) <= 1e-12 * np.max(np.abs(xo)), n
        if pattern == 1:
            assert (piv[:-1] == n - 1).all(), n
    assert seen == list(range(n_lo, n_hi + 1))
