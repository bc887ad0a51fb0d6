"""The workgroup-per-cell integration at the edges of its LU's blocks (panels of
16 columns, blocks of 8, groups of 64 rows: two up to a leading dimension of
128, three up to 192, then four), on the GPU through the C ABI, against the CPU
oracle:

  n =  65  two groups, a last panel of one column
  n = 112  n equals the leading dimension: every panel and load is full
  n = 128  the largest size of two groups
  n = 161  three groups, a last panel of one column
  n = 177  the largest leading dimension of three groups, a ragged last one
  n = 200  four groups, half a panel

The bar is that of the other integration tests: at most one cell on another step
sequence than the oracle's, the others to rel 1e-8 in T and 1e-6 in Y.
"""
import os

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2112_05834_amd import chem, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,scheme", [(64, "rodas3"), (111, "ros4"), (127, "rodas3"), (160, "ros4"), (176, "rodas3"),
                                       (199, "rodas3")])
def test_wide_integration_at_block_edges(tmp_path, ns, scheme):
    mech = synth.generate_mechanism(ns, 3 * ns, ns // 4, ns // 10, 3000 + ns, ea_by_class=True)
    path = synth.write_mech(mech, str(tmp_path / "m.mech"))
    phi = synth.generate_states(mech, 16, 6.0e6, "bimodal", 9000 + ns)
    dt = 1e-6
    code = {"rodas3": chem.RODAS3, "ros4": chem.ROS4}[scheme]
    S = chem.Solver(chem.Mechanism(path), chem.default_opts(schedule=chem.PERSISTENT, scheme=code), device=0)
    r = S.integrate(torch.from_numpy(phi).cuda(), dt)
    torch.cuda.synchronize()
    gphi, gna, gnr, gst = (t.cpu().numpy() for t in (r.phi, r.n_acc, r.n_rej, r.status))
    ref, _, na, nr_, st = O.Mech(path).integrate(phi, dt, scheme=code, n_threads=max(1, min(16, os.cpu_count() or 1)))
    assert np.array_equal(gst, st)
    same = (gna == na) & (gnr == nr_)
    assert (~same).sum() <= 1
    assert not (same & (np.abs(gphi[:, 0] - ref[:, 0]) > 1e-8 * np.abs(ref[:, 0]))).any()
    dY = np.abs(gphi[:, 2:] - ref[:, 2:])
    assert not (same[:, None] & (dY > 1e-10 + 1e-6 * np.abs(ref[:, 2:]))).any()
