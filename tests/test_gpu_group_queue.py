"""Several cells per wave on the persistent queue: a lane group that finishes
its cell takes the next one while the wave's other groups go on. Against the
static schedule, equal in every bit: groups that refill many times (one
block), chunks, a queue order, counts below one wave's groups, cells that fail
at once or hit the attempt limit beside long ones; the evaluation counters and
the cost log, whose records belong to the right cells."""
import numpy as np
import pytest
import torch

from paper_2112_05834_amd import chem, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MECHS = {4: (9, 20, 4, 0, 9, False, 1e5, "uniform"), 2: (25, 90, 10, 3, 1025, True, 6.0e6, "bimodal")}


def _run(S, x, **kw):
    n = x.shape[0]
    S.set_opts(chem.default_opts(**kw))
    nj = torch.zeros(n, dtype=torch.int32, device=DEV)
    nf = torch.zeros(n, dtype=torch.int32, device=DEV)
    S.eval_counters(nj, nf)
    S.log_enable(2 * n)
    r = S.integrate(x, 1e-6)
    f, t = S.log_fetch(2 * n)
    S.log_enable(0)
    S.eval_counters(None, None)
    rec = np.concatenate([f.cpu().numpy(), t.cpu().numpy()[:, None]], axis=1)
    return [r.phi, r.h, r.n_acc, r.n_rej, r.status, nj, nf], rec[np.lexsort(rec.T[::-1])]


@pytest.mark.parametrize("cpw", [4, 2])
@pytest.mark.parametrize("opts", [{}, {"scheme": chem.ROS4, "state": chem.STATE_NO_BATH}])
def test_refilled_groups_equal_static_map(tmp_path, cpw, opts):
    ns, nr, n3, nt, seed, by_class, p, recipe = MECHS[cpw]
    mech = synth.generate_mechanism(ns, nr, n3, nt, seed, ea_by_class=by_class)
    path = synth.write_mech(mech, str(tmp_path / "m.mech"))
    S = chem.Solver(chem.Mechanism(path), device=0)
    for n, max_steps in ((1, 100000), (3, 100000), (150, 100000), (150, 20)):
        x = torch.from_numpy(synth.generate_states(mech, n, p, recipe, 7)).to(DEV)
        if n > 100:
            x[5, 0] = float("nan")
            x[n - 1, 1] = -1.0
        ref, log = _run(S, x, schedule=chem.PLAIN, cells_per_wave=cpw, max_steps=max_steps, **opts)
        for kw in ({}, {"blocks": 1, "waves_per_block": 1}, {"blocks": 1, "queue_chunk": 7}, {"queue_chunk": 64}):
            got, log2 = _run(S, x, schedule=chem.PERSISTENT, cells_per_wave=cpw, max_steps=max_steps, **opts, **kw)
            for u, v in zip(ref, got):
                assert np.array_equal(u.cpu().numpy().view(np.uint8), v.cpu().numpy().view(np.uint8)), (n, kw)
            assert np.array_equal(log.view(np.uint8), log2.view(np.uint8)), (n, kw)
    # through a queue order
    n = 150
    x = torch.from_numpy(synth.generate_states(mech, n, p, recipe, 9)).to(DEV)
    ref, _ = _run(S, x, schedule=chem.PLAIN, cells_per_wave=cpw, **opts)
    S.model_set(np.zeros(4545, dtype=np.float32), None, np.linspace(0.5, 6.0, 7).astype(np.float32))
    S.set_cost_override(torch.log((ref[2] + ref[3]).clamp(min=1).float()))
    got, _ = _run(S, x, schedule=chem.PERSISTENT_BINNED, cells_per_wave=cpw, blocks=2, **opts)
    assert S.last_binning_used()
    for u, v in zip(ref, got):
        assert torch.equal(u, v)
