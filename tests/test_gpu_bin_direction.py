"""The binned schedule's queue order where costs grow with the cell index (the
order inside a bin then runs against the index) and where they do not: every
cell is integrated exactly once, with the bits of the plain schedule.

Sizes: one block of the binning kernels (4096 cells), its edge, several blocks
with a ragged last one. The costs are given, so that the direction is known.
"""
import numpy as np
import pytest
import torch

from paper_2112_05834_amd import chem, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 100, 4096, 4097, 3 * 4096 + 17])
@pytest.mark.parametrize("way", ["ascending", "descending", "mixed", "one"])
def test_binned_order_either_direction(tmp_path, n, way):
    mech = synth.generate_mechanism(9, 20, 4, 0, 9)
    path = synth.write_mech(mech, str(tmp_path / "m.mech"))
    x = torch.from_numpy(synth.generate_states(mech, n, synth.P_ATM, "uniform", 5)).cuda()
    S = chem.Solver(chem.Mechanism(path), chem.default_opts(schedule=chem.PLAIN), device=0)
    rng = np.random.default_rng(n)
    cost = {"ascending": np.linspace(0.0, 6.0, n), "descending": np.linspace(6.0, 0.0, n),
            "mixed": rng.uniform(0.0, 6.0, n), "one": np.full(n, 2.0)}[way].astype(np.float32)
    S.model_set(np.zeros(4545, np.float32), edges=np.linspace(0.5, 5.5, 7).astype(np.float32))
    ref = S.integrate(x, 1e-6)
    S.set_opts(chem.default_opts(schedule=chem.PERSISTENT_BINNED))
    S.set_cost_override(torch.from_numpy(cost).cuda())
    out = torch.full_like(x, float("nan"))
    got = S.integrate(x, 1e-6, out=out)
    torch.cuda.synchronize()
    S.set_cost_override(None)
    assert S.last_binning_used()
    assert torch.equal(out, ref.phi)
    assert torch.equal(got.n_acc, ref.n_acc) and torch.equal(got.n_rej, ref.n_rej) and torch.equal(got.status, ref.status)
