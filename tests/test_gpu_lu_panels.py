"""The one-cell-per-wave LU works in panels of four columns: its pivot search
orders candidates by their high words and falls back to an exact search, and
its trailing updates run as broadcast multiply-adds per tile of 16 columns.
With several cells per wave the LU goes column by column, the pivot row
through LDS. Sizes at the edges of panels and tiles (10, 41, 55, 64; several
cells per wave 10, 13, 16, 26, 32), each against the oracle's LU:

* integer matrices A = L U with L's entries +-1 and U's diagonal +-2^k, so
  that every column ties (the pivot is the first row) and every operation is
  exact: pivots and factors equal in every bit;
* columns whose candidates differ in the low word only, in the first column
  and inside a later panel: pivots equal;
* a pivot from the last row at every step, and a zero column (info).
"""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2112_05834_amd import chem, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SIZES = {10: (9, 20, 4, 0, 9, False, 1), "10 by 4": (9, 20, 4, 0, 9, False, 4), 13: (12, 36, 4, 2, 1012, True, 4),
         16: (15, 45, 5, 2, 1015, True, 4), 26: (25, 90, 10, 3, 1025, True, 2), 32: (31, 110, 12, 4, 1031, True, 2), 41: (40, 160, 20, 6, 1040, True, 0), 55: (54, 269, 40, 12, 54, True, 0),
         64: (63, 250, 30, 8, 1063, True, 0)}


def _solver(n, tmp_path):
    ns, nr, n3, nt, seed, by_class, cpw = SIZES[n]
    mech = synth.generate_mechanism(ns, nr, n3, nt, seed, ea_by_class=by_class)
    path = synth.write_mech(mech, str(tmp_path / "m.mech"))
    return chem.Solver(chem.Mechanism(path), chem.default_opts(cells_per_wave=cpw), device=0), ns + 1


def _lu(S, A, b=None):
    r = S.lu_batch(torch.from_numpy(A.copy()).to(DEV), None if b is None else torch.from_numpy(b.copy()).to(DEV))
    torch.cuda.synchronize()
    return [None if t is None else t.cpu().numpy() for t in r]


@pytest.mark.parametrize("n", list(SIZES))
def test_lu_ties_and_special_columns(n, tmp_path):
    S, n = _solver(n, tmp_path)
    rng = np.random.Generator(np.random.PCG64(n))
    A = np.zeros((12, n, n))
    for c in range(6):                              # every column ties, exact arithmetic
        L = np.tril(rng.choice([-1.0, 1.0], size=(n, n)), -1) + np.eye(n)
        U = np.triu(rng.integers(-3, 4, size=(n, n)).astype(float), 1)
        U += np.diag(rng.choice([-1.0, 1.0], size=n) * 2.0 ** rng.integers(0, 3, size=n))
        A[c] = L @ U
    for c, k in ((6, 0), (7, 5), (8, n - 7)):       # high words equal in column k
        A[c] = rng.normal(size=(n, n))
        A[c, :k] = 0.0
        A[c, :k, :k] = 4.0 * np.eye(k)
        A[c, k:, k] = -(1.5 + rng.permutation(n - k) * 2.0 ** -40)
    A[9] = rng.normal(size=(n, n)) * 0.01 + np.diag(np.full(n - 1, 4.0), 1)
    A[9, n - 1, 0] = 4.0                            # pivot of column 0 from the last row
    A[10] = np.diag(np.arange(1.0, n + 1.0))[::-1]  # an interchange at every step
    A[11] = rng.normal(size=(n, n)) + 3.0 * np.eye(n)
    A[11, :, n // 2] = 0.0                          # singular
    Ag, piv, info, _ = _lu(S, A)
    for c in range(len(A)):
        LU, pr, inf = O.lu(A[c])
        assert np.array_equal(piv[c], pr), c
        assert info[c] == inf, c
        if c < 6 or c == 10:
            assert np.array_equal(Ag[c], LU), c
        else:
            assert np.max(np.abs(Ag[c] - LU)) <= 1e-12 * np.max(np.abs(A[c])), c
    assert info[11] == n // 2 + 1


@pytest.mark.parametrize("n", list(SIZES))
def test_lu_batch_remainders(n, tmp_path):
    """Batches that leave a block's last waves without a matrix."""
    S, n = _solver(n, tmp_path)
    rng = np.random.Generator(np.random.PCG64(100 + n))
    A = rng.normal(size=(13, n, n)) + 3.0 * np.eye(n)[None]
    b = rng.normal(size=(13, n))
    for batch in (1, 5, 13):
        Ag, piv, info, bg = _lu(S, A[:batch], b[:batch])
        assert (info == 0).all()
        for c in range(batch):
            LU, pr, _ = O.lu(A[c])
            assert np.array_equal(piv[c], pr), (batch, c)
            x = O.lu_solve(LU, pr, b[c])
            assert np.max(np.abs(bg[c] - x)) <= 1e-10 * np.max(np.abs(x)), (batch, c)
