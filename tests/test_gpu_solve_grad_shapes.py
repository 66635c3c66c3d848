"""Multipliers and dE/df of fragment_solve at every shape of the solver's work
split, from T = 0 and from the pairs' own fragments (needs an MI355X): the stored
amplitudes, the gradient pass with its shared row blocks, and, with three LMOs
(one trimer) and four (trimers that share pairs), first sweeps without and with the
pairs' coupling sums.  The oracle makes the same iterates; what is left is the
rounding of sums over at most 4 r terms."""
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


@pytest.mark.parametrize("n,warm", [(4, False), (4, True), (3, True)])
@pytest.mark.parametrize("r", [(1, 1), (5, 5), (8, 8), (12, 13), (16, 17), (23, 24), (25, 32),
                               (33, 33), (38, 40), (41, 41), (47, 48), (49, 52), (57, 57),
                               (64, 64), (1, 40), (3, 64), (30, 78), (70, 78)])
def test_gradient_shapes(m, r, n, warm):
    import torch
    print(f"case: {n} LMOs, r {r}, warm start {warm}", flush=True)
    prob = synth.micro(n_occ=n, n_vir=max(24, 4 * r[1]), n_aux=max(32, 5 * r[1]), r=r,
                       seed=100 * r[0] + r[1] + n, tol=1e-9)
    ref = oracle.run(prob, keep_T=True, warm_start=warm)
    W, df = {}, np.zeros((n, n))
    for f, c, T in zip(prob.frags, oracle.mbe3_coefficients(n, prob.frags), ref["T"]):
        Tt, g = oracle.fragment_gradient(ref["oracle"], f, T)
        for t, v in Tt.items():
            W[t] = W.get(t, 0.0) + c * v
        df += c * g
    slots = [(p, p) for p in range(n)] + [tuple(int(x) for x in pq) for pq in prob.pairs]
    Wref = np.concatenate([W[t].ravel() for t in slots])
    h = m.from_problem(prob, device="cuda:0", warm_start=warm)
    out = h.forward(grad=True)
    dF = torch.empty((n, n), dtype=torch.float64, device="cuda:0")
    h.mbe3_backward(out["gamma"], out["W"], dEdF=dF)
    assert np.array_equal(out["iters"].cpu().numpy(), ref["iters"])
    for name, got, want in (("W", out["W"], Wref), ("dE/df", dF, 0.5 * (df + df.T))):
        err = np.abs(got.cpu().numpy() - want).max()
        assert err <= 1e-11 * np.abs(want).max(), name
    h.close()
