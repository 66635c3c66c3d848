"""The gradient pass contracts each coupling once and counts it twice; W~ is
formed from the summed amplitudes (needs an MI355X).  Checked against the
oracle's gradient at fragment kinds and widths where the terms differ: dimers
alone, one trimer, unequal OSV counts on either side of a 16-row block, strong
Fock coupling, and pair domains past the LDS-resident solver's 128."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def m():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2603_16575_amd as pkg
    pkg._lib.load()
    return pkg


@pytest.mark.parametrize("n_occ,n_vir,n_aux,r,dimers_only", [
    (2, 24, 40, (3, 9), False), (3, 24, 40, (2, 17), False), (4, 40, 64, (7, 18), True),
    (4, 80, 96, (15, 33), False), (3, 120, 150, (50, 72), False)])
def test_gradient_terms(m, n_occ, n_vir, n_aux, r, dimers_only):
    import torch
    print(f"case: {n_occ} LMOs, r {r}, dimers only {dimers_only}", flush=True)
    prob = synth.micro(n_occ=n_occ, n_vir=n_vir, n_aux=n_aux, r=r, seed=11)
    f = prob.f_occ.copy()
    off = ~np.eye(n_occ, dtype=bool)
    f[off] *= 4.0
    prob = dataclasses.replace(prob, f_occ=f)
    if dimers_only:
        prob = dataclasses.replace(prob, trimers=np.zeros((0, 3), dtype=np.int32))
    ref = oracle.gradient(prob)
    h = m.from_problem(prob, device="cuda:0", warm_start=False)
    out = h.forward(grad=True)
    dF = torch.empty((n_occ, n_occ), dtype=torch.float64, device="cuda:0")
    dB, _ = h.mbe3_backward(out["gamma"], out["W"], dEdF=dF)
    gB = np.stack([ref["dB"][i] for i in range(n_occ)])
    # tol 1e-12 on both sides: the same iterates, apart from rounding
    assert np.abs(dF.cpu().numpy() - ref["df"]).max() <= 1e-10 * np.abs(ref["df"]).max()
    assert np.abs(dB.cpu().numpy() - gB).max() <= 1e-10 * np.abs(gB).max()
    h.close()
