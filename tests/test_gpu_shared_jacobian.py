"""Pairs of waves that share a Jacobian buffer (state sizes 33 to 55, two
waves a block or more) against one wave per block with a buffer of its own:
equal in every bit, for blocks of 2, 3 (the last wave alone with its buffer)
and 4 waves, counts that leave waves of a pair without a cell, cells with
rejected attempts (whose Jacobian is formed again), every method option, and
the evaluation counters."""
import numpy as np
import pytest
import torch

from paper_2112_05834_amd import chem, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(S, x, dt, **kw):
    S.set_opts(chem.default_opts(**kw))
    n = x.shape[0]
    nj = torch.zeros(n, dtype=torch.int32, device=DEV)
    nf = torch.zeros(n, dtype=torch.int32, device=DEV)
    S.eval_counters(nj, nf)
    r = S.integrate(x, dt)
    torch.cuda.synchronize()
    S.eval_counters(None, None)
    return [r.phi, r.h, r.n_acc, r.n_rej, r.status, nj, nf]


@pytest.mark.parametrize("ns,nr,n3,nt", [(33, 120, 15, 5), (40, 160, 20, 6), (54, 269, 40, 12)])
@pytest.mark.parametrize("opts", [{}, {"scheme": chem.ROS4}, {"state": chem.STATE_NO_BATH},
                                  {"jacobian": chem.JAC_FD}])
def test_shared_buffer_equals_own(tmp_path, ns, nr, n3, nt, opts):
    mech = synth.generate_mechanism(ns, nr, n3, nt, 54 if ns == 54 else 1000 + ns, ea_by_class=True)
    path = synth.write_mech(mech, str(tmp_path / "m.mech"))
    n = 67 if "jacobian" in opts else 261
    x = torch.from_numpy(synth.generate_states(mech, n, 6.0e6, "bimodal", 7)).to(DEV)
    S = chem.Solver(chem.Mechanism(path), device=0)
    ref = _run(S, x, 1e-6, waves_per_block=1, **opts)
    assert int(ref[3].sum()) > 0 and not ref[4].any()
    for schedule in (chem.PLAIN, chem.PERSISTENT):
        for wpb in (2, 3, 4):
            got = _run(S, x, 1e-6, waves_per_block=wpb, schedule=schedule, **opts)
            for u, v in zip(ref, got):
                assert torch.equal(u, v), (schedule, wpb)
    # a failing cell beside its partner
    y = x.clone()
    y[3, 0] = float("nan")
    got = _run(S, y, 1e-6, waves_per_block=4, schedule=chem.PERSISTENT, **opts)
    keep = torch.arange(n, device=DEV) != 3
    assert got[4][3].item() == chem.CELL_NONFINITE
    for u, v in zip(ref, got):
        assert torch.equal(u[keep], v[keep])
