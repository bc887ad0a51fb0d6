"""The LU that the integration runs above 64 state components (panels of 16
columns, blocks of 8, groups of 64 rows: two up to a leading dimension of 128,
three up to 192, then four), on given matrices: the factors of g I - A, the rows'
order and the first zero pivot equal the oracle's in every bit, since every
element receives the unblocked algorithm's operations in its order; the solves
(another order, reciprocals) agree to 1e-10.

Sizes: one column past two groups' first panels, a leading dimension equal to n,
the edges of two, three and four groups, ragged last panels of 1, 8 and 9
columns, the largest size.
"""
import ctypes

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2112_05834_amd import chem, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(S, g, A, b):
    f = chem.lib().chem_check_lu_integration
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_double] + [ctypes.c_void_p] * 5
    At, bt = torch.from_numpy(A.copy()).to(DEV), torch.from_numpy(b.copy()).to(DEV)
    rows = torch.empty(A.shape[:2], dtype=torch.int32, device=DEV)
    info = torch.empty(len(A), dtype=torch.int32, device=DEV)
    rc = f(S._h, len(A), g, At.data_ptr(), rows.data_ptr(), info.data_ptr(), bt.data_ptr(),
           torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in (At, rows, info, bt)]


def _order(piv):
    rows = np.arange(len(piv))
    for k, p in enumerate(piv):
        rows[[k, p]] = rows[[p, k]]
    return rows


def _last_row_pivots(rng, n):
    """P L U, |l| <= 1/2: the pivot is the last row at every step."""
    L = np.tril(rng.uniform(-0.5, 0.5, (n, n)), -1) + np.eye(n)
    U = np.triu(rng.uniform(-1, 1, (n, n)), 1) + np.diag(rng.uniform(2, 3, n))
    arr = np.arange(n)
    for k in range(n - 2, -1, -1):
        arr[[k, n - 1]] = arr[[n - 1, k]]
    return (L @ U)[arr]


@pytest.mark.parametrize("n", [65, 80, 105, 112, 128, 129, 145, 161, 177, 192, 193, 200, 217, 256])
def test_integration_lu_equals_oracle(n, tmp_path):
    mech = synth.generate_mechanism(n - 1, 2 * n, n // 8, n // 16, 4000 + n, ea_by_class=True)
    path = synth.write_mech(mech, str(tmp_path / "m.mech"))
    S = chem.Solver(chem.Mechanism(path), device=0)
    rng = np.random.Generator(np.random.PCG64(n))
    g = 2.5
    M = rng.normal(size=(10, n, n))
    M[0] += 3.0 * np.eye(n)
    M[2] = _last_row_pivots(rng, n)
    # every column ties, every operation is exact
    M[3] = ((np.tril(rng.choice([-1.0, 1.0], (n, n)), -1) + np.eye(n))
            @ (np.triu(rng.integers(-1, 2, (n, n)).astype(float), 1) + np.diag(rng.choice([-1.0, 1.0], n))))
    # candidates that differ in the low word only
    for c, k in ((4, 0), (5, 21), (6, n - 9)):
        M[c, :k] = 0.0
        M[c, :k, :k] = 4.0 * np.eye(k)
        M[c, k:, k] = -(1.5 + rng.permutation(n - k) * 2.0 ** -40)
    M[7, :, n // 2] = 0.0                               # a zero pivot inside
    M[8, :, n - 1] = 0.0                                # and at the end
    M[9] += np.diag(np.full(n, 40.0))                   # no interchange
    A = g * np.eye(n)[None] - M
    want = np.where(np.eye(n, dtype=bool)[None], g, 0.0) - A     # as the kernel forms it
    b = rng.normal(size=(len(A), n))
    F, rows, info, x = _check(S, g, A, b)
    again = _check(S, g, A, b)
    for u, v in zip((F, rows, info, x), again):
        assert np.array_equal(u, v, equal_nan=u.dtype == np.float64)
    for c in range(len(A)):
        LU, piv, inf = O.lu(want[c])
        assert info[c] == inf, c
        assert np.array_equal(rows[c], _order(piv)), c
        assert np.array_equal(F[c], LU), (c, np.max(np.abs(F[c] - LU)))
        if c in (0, 2, 9):                              # well conditioned
            xo = O.lu_solve(LU, piv, b[c])
            assert np.max(np.abs(x[c] - xo)) <= 1e-10 * np.max(np.abs(xo)), c
    assert info[7] == n // 2 + 1 and info[8] == n
    assert (rows[9] == np.arange(n)).all()


def test_small_state_sizes_are_refused(tmp_path):
    mech = synth.generate_mechanism(9, 20, 4, 0, 9)
    S = chem.Solver(chem.Mechanism(synth.write_mech(mech, str(tmp_path / "m.mech"))), device=0)
    f = chem.lib().chem_check_lu_integration
    f.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_double] + [ctypes.c_void_p] * 5
    d = torch.zeros(100, dtype=torch.float64, device=DEV)
    i = torch.zeros(100, dtype=torch.int32, device=DEV)
    assert f(S._h, 1, 0.0, d.data_ptr(), i.data_ptr(), i.data_ptr(), None, None) == -6
    assert f(S._h, 1, 0.0, None, i.data_ptr(), i.data_ptr(), None, None) == -1
