"""The range finder's steps at sizes around its splits (needs an MI355X): virtuals
under, over and between multiples of 64, 256, 512 and 1024, one accepted row, row
counts around groups of four and of sixty-four, against the oracle."""
import numpy as np
import pytest

import synth
from oracle import rosv as R

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def m():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2603_16575_amd as pkg
    pkg._lib.load()
    return pkg


@pytest.mark.parametrize("n_vir,n_aux,n_max", [
    (9, 12, 3), (66, 70, 1), (130, 150, 65), (257, 200, 30), (520, 260, 70), (1100, 400, 5)])
def test_rosv_sizes(m, n_vir, n_aux, n_max):
    print(f"case: {n_vir} virtuals, {n_max} rows", flush=True)
    prob = synth.micro(n_occ=2, n_vir=n_vir, n_aux=n_aux, r=(2, 4), seed=21)
    h = m.from_problem(prob, device="cuda:0")
    out = {k: v.cpu().numpy() for k, v in h.rosv(n_max=n_max).items()}
    for i in range(prob.n_occ):
        ref = R.lmo_rosv(prob, i, n_max=n_max)
        k = len(ref["w"])
        assert out["rows"][i] == ref["rows"] and out["n_osv"][i] == k
        # as for the helix's LMOs: w relative, the projector entry by entry
        assert np.abs(out["w"][i, :k] - ref["w"]).max() <= 1e-10 * ref["w"].max()
        Q = out["Q"][i, :k].T
        assert np.abs(Q @ Q.T - ref["Q"] @ ref["Q"].T).max() <= 1e-9
    h.close()
