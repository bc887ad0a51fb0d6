"""The per-wave kernel's reaction records (state sizes 33 to 64) and the rule
that chooses them: a mechanism whose reaction sides all have one of the forms
A, 2A, A + B, 2A + B, A + B + C uses the records, any other the general
reaction words.

On the CPU the records of generated mechanisms with every form are decoded
and compared with the parsed reactions. On the GPU the right-hand side and
Jacobian of such mechanisms are compared with the oracle, and with the
general words: the same mechanism with one more reaction of negligible rate
whose form has no record."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2112_05834_amd import synth

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2112_05834_amd", "csrc")

FORMS = {"A": [1], "2A": [2], "A+B": [1, 1], "2A+B": [2, 1], "A+B+C": [1, 1, 1]}
OTHER = {"3A": [3], "A+2B": [1, 2], "2A+2B": [2, 2], "A+B+2C": [1, 1, 2]}


def _side(rng, ns, orders):
    return list(zip((int(s) for s in rng.choice(ns, size=len(orders), replace=False)), orders))


def _mech(ns, seed, extra=None):
    """Generated mechanism plus every pair of forms as reactant and product
    sides, in every type and direction (rates of ordinary size, balance not
    needed here); extra: a side without a record, at a negligible rate."""
    mech = synth.generate_mechanism(ns, 3 * ns, 8, 3, 1000 + ns, ea_by_class=True)
    rng = np.random.Generator(np.random.PCG64(seed))
    k = 0
    for fo in FORMS.values():
        for po in FORMS.values():
            rtype, rev = k % 3, (k // 3) % 2 == 0
            k += 1
            A = 10.0 ** rng.uniform(1.0, 3.0) * 1e-3 ** (sum(fo) - 1)
            eff = [] if rtype == 0 else [(int(s), float(rng.uniform(0.3, 12.0)))
                                         for s in rng.choice(ns, size=k % 11, replace=False)]
            troe = (A * 10.0, -1.0, 500.0, 0.6, 150.0, 2500.0, 4000.0, float(k % 2)) if rtype == 2 else None
            kw = {"troe": troe} if troe else {}
            mech.reactions.append(synth.Reaction(rtype, rev, _side(rng, ns, fo), _side(rng, ns, po), A,
                                                 float(rng.uniform(-0.5, 0.5)), float(rng.uniform(0, 2e4)), eff=eff,
                                                 **kw))
    if extra:
        mech.reactions.append(synth.Reaction(0, False, _side(rng, ns, extra), _side(rng, ns, [1]), 1e-280, 0.0, 0.0))
    return mech


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("rec") / "rec_driver")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           "-I", CSRC, os.path.join(HERE, "rec_driver.cpp"), os.path.join(CSRC, "mech.cpp"),
                           "-o", exe])
    return exe


def test_records_decode_to_the_reactions(driver, tmp_path):
    files, want = [], []
    for ns in (33, 40, 54, 63, 64):
        for extra in [None] + list(OTHER.values()):
            path = synth.write_mech(_mech(ns, ns, extra), str(tmp_path / ("m%d.mech" % len(files))))
            files.append(path)
            want.append("records" if extra is None and ns <= 63 else "general")
    for name in ("tiny9", "spray54"):
        files.append(synth.mech_cached(name, str(tmp_path))[1])
        want.append("records")
    r = subprocess.run([driver] + files, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-500:] + r.stderr[-2000:]
    assert r.stdout.split() == want


def _scaled(J, y):
    s = np.abs(y).copy()
    s[0] = max(s[0], 1.0)
    s[1:] = np.maximum(s[1:], 1e-8)
    return J * s[None, :] / s[:, None]


@pytest.mark.gpu
@pytest.mark.parametrize("ns", [33, 40, 54, 63])
def test_records_match_oracle_and_general_words(ns, tmp_path):
    import torch

    from oracle import oracle as O
    from paper_2112_05834_amd import chem

    mech = _mech(ns, ns)
    path = synth.write_mech(mech, str(tmp_path / "m.mech"))
    gen = synth.write_mech(_mech(ns, ns, OTHER["A+2B"]), str(tmp_path / "g.mech"))
    phi = synth.generate_states(mech, 12, 6.0e6, "bimodal", 5)
    out = []
    for p in (path, gen):
        S = chem.Solver(chem.Mechanism(p), device=0)
        x = torch.from_numpy(phi).to("cuda:0")
        f, J = S.eval_rhs_jac(x)
        f2, _ = S.eval_rhs_jac(x, jac=False)
        torch.cuda.synchronize()
        assert torch.equal(f, f2)
        out.append((f.cpu().numpy(), J.cpu().numpy()))
    M = O.Mech(path)
    for c in range(len(phi)):
        y = np.concatenate([[phi[c, 0]], phi[c, 2:]])
        fr = M.rhs(phi[c, 1], y)
        Jr = M.jac(phi[c, 1], y)
        scale = np.abs(Jr).sum(axis=1) * np.maximum(np.abs(y), 1e-8).max() + np.abs(fr)
        B = _scaled(Jr, y)
        rowmax = np.abs(B).max(axis=1, keepdims=True)
        for f, J in out:
            assert np.all(np.abs(f[c] - fr) <= 1e-9 * np.abs(fr) + 1e-12 * scale), c
            assert np.all(np.abs(_scaled(J[c], y) - B) <= 1e-9 * np.abs(B) + 1e-12 * rowmax), c
        (f, J), (fg, Jg) = out
        assert np.all(np.abs(f[c] - fg[c]) <= 1e-9 * np.abs(fg[c]) + 1e-12 * scale), c
        assert np.all(np.abs(_scaled(J[c], y) - _scaled(Jg[c], y)) <= 1e-9 * np.abs(B) + 1e-12 * rowmax), c
