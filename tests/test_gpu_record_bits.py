"""Right-hand side and Jacobian by the packed reaction records have the bits of
the general reaction words, for sides of every form that the records hold (A,
2A, A + B, 2A + B, A + B + C), at all state sizes that read them and for every
number of cells per wave. Both are compared with the oracle too.

The general words are reached by one more reaction whose form has no record:
of the last type, so that the others keep their places, and of a rate that
changes no sum.
"""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2112_05834_amd import chem, synth

from .test_reaction_records import FORMS, _mech, _scaled, _side

pytestmark = pytest.mark.gpu


def _forms(ns):
    if ns > 9:
        return _mech(ns, ns)
    mech = synth.generate_mechanism(9, 20, 4, 0, 9)
    rng = np.random.Generator(np.random.PCG64(ns))
    for k, (fo, po) in enumerate((a, b) for a in FORMS.values() for b in FORMS.values()):
        eff = [(int(s), float(rng.uniform(0.3, 12.0))) for s in rng.choice(ns, size=k % 7, replace=False)]
        mech.reactions.append(synth.Reaction(k % 2, k % 3 > 0, _side(rng, ns, fo), _side(rng, ns, po),
                                             10.0 ** rng.uniform(1.0, 3.0) * 1e-3 ** (sum(fo) - 1),
                                             float(rng.uniform(-0.5, 0.5)), float(rng.uniform(0, 2e4)),
                                             eff=eff if k % 2 else []))
    return mech


@pytest.mark.parametrize("ns,cpw", [(9, 4), (9, 1), (12, 4), (15, 4), (25, 2), (31, 2), (33, 0), (54, 0), (63, 0)])
def test_records_have_the_bits_of_the_general_words(ns, cpw, tmp_path):
    mech = _forms(ns)
    path = synth.write_mech(mech, str(tmp_path / "m.mech"))
    more = _forms(ns)
    more.reactions.append(synth.Reaction(2, False, [(0, 1), (1, 2)], [(2, 1)], 1e-280, 0.0, 0.0,
                                         troe=(1e-285, 0.0, 0.0, 0.6, 150.0, 2500.0, 4000.0, 0.0)))
    gen = synth.write_mech(more, str(tmp_path / "g.mech"))
    phi = synth.generate_states(mech, 13, 6.0e6, "bimodal", 5)
    x = torch.from_numpy(phi).to("cuda:0")
    out = []
    for p in (path, gen):
        S = chem.Solver(chem.Mechanism(p), chem.default_opts(cells_per_wave=cpw), device=0)
        f, J = S.eval_rhs_jac(x)
        f2, _ = S.eval_rhs_jac(x, jac=False)
        torch.cuda.synchronize()
        assert torch.equal(f, f2)
        out.append((f.cpu().numpy(), J.cpu().numpy()))
    (f, J), (fg, Jg) = out
    M = O.Mech(path)
    for c in range(len(phi)):
        y = np.concatenate([[phi[c, 0]], phi[c, 2:]])
        fr, Jr = M.rhs(phi[c, 1], y), M.jac(phi[c, 1], y)
        scale = np.abs(Jr).sum(axis=1) * np.maximum(np.abs(y), 1e-8).max() + np.abs(fr)
        B = _scaled(Jr, y)
        assert np.all(np.abs(f[c] - fr) <= 1e-9 * np.abs(fr) + 1e-12 * scale), c
        assert np.all(np.abs(_scaled(J[c], y) - B) <= 1e-9 * np.abs(B) + 1e-12 * np.abs(B).max(axis=1, keepdims=True)), c
    assert np.array_equal(f, fg)
    assert np.array_equal(J, Jg)
