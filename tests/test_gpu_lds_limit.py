"""The largest mechanisms whose work areas fit the LDS of a CU with one wave of
several cells: image of the mechanism plus, for each cell, J and rates of every
reaction. They run, and agree with the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2112_05834_amd import chem, synth

pytestmark = pytest.mark.gpu

LDS = 160 * 1024


def _reactions(n, nn, cells):
    """Most reactions A -> B (16 bytes of words and two 2-byte list entries each)
    beside: species offsets, 64 reciprocal weights; per cell J, a pivot row, the
    five rates of each reaction and three vectors of the species."""
    up = lambda x: (x + 15) // 16 * 16
    nr = 0
    while True:
        k = nr + 1
        image = 16 * k + up(2 * n) + up(4 * k) + 8 * 64
        cell = nn * nn + (nn + 2) // 2 * 2 + max(5 * k, 3 * nn) + 3 * (nn - 1)
        if image + 8 * cells * cell > LDS:
            return nr
        nr = k


@pytest.mark.parametrize("n,nn,cpw", [(10, 10, 4), (16, 16, 4), (12, 16, 4), (32, 32, 2)])
def test_largest_mechanism_of_one_wave(n, nn, cpw, tmp_path):
    ns = n - 1
    mech = synth.generate_mechanism(9, 20, 4, 0, 9) if ns == 9 else synth.generate_mechanism(ns, 3 * ns, 0, 0, 2000 + ns)
    rng = np.random.Generator(np.random.PCG64(n))
    mech.reactions = []
    for k in range(_reactions(n, nn, cpw)):
        a, b = (int(s) for s in rng.choice(ns, size=2, replace=False))
        mech.reactions.append(synth.Reaction(0, False, [(a, 1)], [(b, 1)], float(10.0 ** rng.uniform(0, 3)), 0.0, 0.0))
    path = synth.write_mech(mech, str(tmp_path / "m.mech"))
    phi = synth.generate_states(mech, 9, synth.P_ATM, "uniform", 5)
    S = chem.Solver(chem.Mechanism(path), chem.default_opts(schedule=chem.PERSISTENT, cells_per_wave=cpw), device=0)
    r = S.integrate(torch.from_numpy(phi).cuda(), 1e-6)
    torch.cuda.synchronize()
    ref, _, na, nr, st = O.Mech(path).integrate(phi, 1e-6)
    assert np.array_equal(r.status.cpu().numpy(), st) and (st == 0).all()
    got = r.phi.cpu().numpy()
    assert np.all(np.abs(got[:, 0] - ref[:, 0]) <= 1e-8 * ref[:, 0])
    assert np.all(np.abs(got[:, 2:] - ref[:, 2:]) <= 1e-10 + 1e-6 * np.abs(ref[:, 2:]))
