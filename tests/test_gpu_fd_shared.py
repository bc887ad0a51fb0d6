"""Forward-difference Jacobians do not hold the buffer that two waves share: a
block of two waves takes little longer than blocks of one with buffers of their
own, and gives the same bits, also without the bath gas (whose column and row
are cleared on the way into the registers)."""
import pytest
import torch

from paper_2112_05834_amd import chem, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _mechanism(tmp_path, ns, nr, n3, nt):
    mech = synth.generate_mechanism(ns, nr, n3, nt, 1000 + ns, ea_by_class=True)
    return mech, chem.Mechanism(synth.write_mech(mech, str(tmp_path / "m.mech")))


@pytest.mark.parametrize("ns,nr,n3,nt", [(33, 120, 15, 5), (54, 269, 40, 12)])
@pytest.mark.parametrize("scheme", [chem.RODAS3, chem.ROS4])
def test_differences_without_the_bath_gas(tmp_path, ns, nr, n3, nt, scheme):
    mech, handle = _mechanism(tmp_path, ns, nr, n3, nt)
    x = torch.from_numpy(synth.generate_states(mech, 19, 6.0e6, "bimodal", 7)).to(DEV)
    out = []
    for wpb in (1, 2, 3):
        S = chem.Solver(handle, chem.default_opts(schedule=chem.PERSISTENT, waves_per_block=wpb, scheme=scheme,
                                                  jacobian=chem.JAC_FD, state=chem.STATE_NO_BATH), device=0)
        r = S.integrate(x, 1e-6)
        torch.cuda.synchronize()
        out.append([r.phi, r.h, r.n_acc, r.n_rej, r.status])
    assert not out[0][4].any()
    for got in out[1:]:
        for u, v in zip(out[0], got):
            assert torch.equal(u, v)


def test_two_waves_run_beside_each_other(tmp_path):
    """Eight copies of one long cell, each wave with a SIMD of its own. Nearly all
    of a step is differences: a pair that excludes itself there takes twice a
    single wave's time, one that does not about the same; the line is between."""
    mech, handle = _mechanism(tmp_path, 40, 160, 20, 6)
    x = torch.from_numpy(synth.generate_states(mech, 64, 6.0e6, "bimodal", 7)).to(DEV)
    steps = chem.Solver(handle, device=0).integrate(x, 1e-6).n_acc
    x = x[int(steps.argmax())].repeat(8, 1).contiguous()
    ms = {1: [], 2: []}
    for turn in range(4):
        for wpb in ms:
            S = chem.Solver(handle, chem.default_opts(waves_per_block=wpb, jacobian=chem.JAC_FD), device=0)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            S.integrate(x, 1e-6)
            b.record()
            b.synchronize()
            if turn:                          # the first one loads the kernel
                ms[wpb].append(a.elapsed_time(b))
    assert min(ms[2]) < 1.4 * min(ms[1]), ms
