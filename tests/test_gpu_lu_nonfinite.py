"""Matrices that are not finite beside finite ones, in the batched LU and in
integrations with several cells per wave: a wave's other matrices and cells
keep every bit, and the pivots stay rows of the matrix.

A column whose remaining candidates are all NaN keeps its diagonal as pivot
(nothing compares; the oracle's search does the same).
"""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2112_05834_amd import chem, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# species, cells per wave (0: the default): exact and padded sizes of every
# compiled variant, and one workgroup per matrix
SIZES = [(9, 4), (9, 1), (12, 4), (15, 4), (25, 2), (31, 2), (40, 0), (54, 0), (59, 0), (63, 0), (70, 0)]


def _path(ns, tmp_path):
    mech = (synth.generate_mechanism(9, 20, 4, 0, 9) if ns == 9 else
            synth.generate_mechanism(ns, 3 * ns, ns // 4, ns // 10, 1000 + ns, ea_by_class=True))
    return mech, synth.write_mech(mech, str(tmp_path / "m.mech"))


def _lu(S, A, b):
    r = S.lu_batch(torch.from_numpy(A.copy()).to(DEV), torch.from_numpy(b.copy()).to(DEV))
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in r]


@pytest.mark.parametrize("ns,cpw", SIZES)
def test_lu_batch_beside_nonfinite(ns, cpw, tmp_path):
    _, path = _path(ns, tmp_path)
    S = chem.Solver(chem.Mechanism(path), chem.default_opts(cells_per_wave=cpw), device=0)
    n = ns + 1
    rng = np.random.Generator(np.random.PCG64(n))
    bad = []
    for k in range(7):
        A = rng.normal(size=(n, n)) + 3.0 * np.eye(n)
        if k == 0:
            A[:] = np.nan
        elif k == 1:
            A[:, 0] = np.nan                # nothing to compare in the first column
        elif k == 2:
            A[n - 1, n - 1] = np.nan        # only the last candidate of the last column
        elif k == 3:
            A[0, 0] = np.nan
        elif k == 4:
            A[n // 2, :] = np.inf
        elif k == 5:
            A[:, n // 2] = -np.nan
            A[n // 3, n // 3] = np.inf
        else:
            A[n // 2:, n // 2:] = np.nan    # several columns without a candidate
        bad.append(A)
    good = rng.normal(size=(len(bad) + 1, n, n)) + 3.0 * np.eye(n)
    gb = rng.normal(size=(len(good), n))
    alone = _lu(S, good, gb)
    # alternating, so that a wave with several matrices holds both
    A = np.empty((2 * len(bad) + 1, n, n))
    b = np.empty((len(A), n))
    A[0::2], A[1::2] = good, np.stack(bad)
    b[0::2], b[1::2] = gb, 1.0
    got = _lu(S, A, b)
    for g, a in zip(got, alone):
        assert np.array_equal(g[0::2], a)
    piv = got[1]
    assert (piv >= np.arange(n)).all() and (piv < n).all()
    assert np.array_equal(piv[1], np.arange(n))             # all NaN: diagonals
    for k, c in enumerate(bad):
        if k in (0, 1, 2):                                  # one possible choice everywhere
            _, p, info = O.lu(c)
            assert np.array_equal(piv[2 * k + 1], p) and got[2][2 * k + 1] == info, k


@pytest.mark.parametrize("schedule", ["plain", "persistent"])
@pytest.mark.parametrize("ns,cpw", [(9, 4), (12, 4), (15, 4), (25, 2), (31, 2), (40, 0), (54, 0), (63, 0)])
def test_integration_beside_cells_without_mass(ns, cpw, schedule, tmp_path):
    """Cells whose mass fractions are all zero have no density: their
    right-hand side is not a number and no step of theirs is accepted."""
    mech, path = _path(ns, tmp_path)
    phi = synth.generate_states(mech, 37, 6.0e6, "bimodal", 3)
    dt = 1e-7
    code = {"plain": chem.PLAIN, "persistent": chem.PERSISTENT}[schedule]
    S = chem.Solver(chem.Mechanism(path), chem.default_opts(schedule=code, cells_per_wave=cpw), device=0)
    ref = S.integrate(torch.from_numpy(phi).to(DEV), dt)
    mixed = phi.copy()
    mixed[1::3, 2:] = 0.0
    r = S.integrate(torch.from_numpy(mixed).to(DEV), dt)
    torch.cuda.synchronize()
    keep = np.ones(len(phi), bool)
    keep[1::3] = False
    keep = torch.from_numpy(keep).to(DEV)
    for name in ("phi", "h", "n_acc", "n_rej", "status"):
        assert torch.equal(getattr(r, name)[keep], getattr(ref, name)[keep]), name
    _, _, na, nr, st = O.Mech(path).integrate(mixed, dt)
    assert np.array_equal(r.status.cpu().numpy(), st)
    assert (r.n_acc.cpu().numpy()[1::3] == 0).all() and (na[1::3] == 0).all()
