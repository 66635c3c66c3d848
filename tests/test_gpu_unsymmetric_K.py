"""Exchange blocks K_pp that are not symmetric (needs an MI355X).  fragment_solve
takes any K buffer and returns <2T - T^T, K + R>, the multipliers 2T - T^T and
the functional's explicit dE/df for it; the amplitudes of a diagonal pair are
then not symmetric either.  Checked against the oracle with the same blocks at
the widths of every solver instance, the 160-wide one among them, from T = 0 and
from the pairs' own fragments.  Both sides make the same iterates; what is left is
the rounding of sums over at most 4 r terms."""
import numpy as np
import pytest

import oracle
import synth
from oracle.mbe3 import orbs, prepare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def m():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2603_16575_amd as pkg
    pkg._lib.load()
    return pkg


def explicit_df(ora, o, T):
    """d e_frag / df at fixed amplitudes: the residual's terms with f, over p <= q."""
    g = np.zeros((ora.prob.n_occ, ora.prob.n_occ))
    for (p, q), v in T.items():
        Tt = (1.0 if p == q else 2.0) * (2.0 * v - v.T)
        for k in o:
            Sa = ora.Sblk(orbs(p, q), orbs(k, q))
            g[p, k] -= np.sum(Tt * (Sa @ ora.get_T(T, k, q) @ Sa.T))
            Sb = ora.Sblk(orbs(p, q), orbs(p, k))
            g[k, q] -= np.sum(Tt * (Sb @ ora.get_T(T, p, k) @ Sb.T))
    return g


@pytest.mark.parametrize("n,warm", [(3, False), (3, True), (4, True)])
@pytest.mark.parametrize("r", [(2, 3), (9, 12), (23, 24), (30, 40), (41, 48), (49, 55),
                               (57, 64), (70, 78)])
def test_unsymmetric_diagonal_blocks(m, r, n, warm):
    import torch
    print(f"case: {n} LMOs, r {r}, warm start {warm}", flush=True)
    prob = synth.micro(n_occ=n, n_vir=max(24, 4 * r[1]), n_aux=max(32, 5 * r[1]), r=r,
                       seed=10 * r[0] + r[1], tol=1e-9)
    h = m.from_problem(prob, device="cuda:0", warm_start=warm)
    K = h.pair_K(h.osv_project(h.empty_gamma()), h.empty_K())
    ora = oracle.Oracle(prob)
    prepare(ora, prob.frags)
    g = np.random.default_rng(r[0])
    host = K.cpu().numpy()
    for p in range(n):
        d = int(prob.r[p])
        a = g.standard_normal((d, d))
        blk = ora.Kbar(p, p).copy()
        blk += 0.3 * np.abs(blk).max() * (a - a.T)
        ora._K[(p, p)] = blk
        host[h.k_off[p]:h.k_off[p + 1]] = blk.ravel()
    K.copy_(torch.from_numpy(host))
    ref = oracle.run(prob, keep_T=True, ora=ora, warm_start=warm)
    c = oracle.mbe3_coefficients(n, prob.frags)
    W, df = {}, np.zeros((n, n))
    for f, cF, T in zip(prob.frags, c, ref["T"]):
        for t, v in T.items():
            W[t] = W.get(t, 0.0) + cF * (2.0 * v - v.T)
        df += cF * explicit_df(ora, [int(x) for x in f if x >= 0], T)
    slots = [(p, p) for p in range(n)] + [tuple(int(x) for x in pq) for pq in prob.pairs]
    Wref = np.concatenate([W[t].ravel() for t in slots])

    e = torch.empty(prob.n_frag, dtype=torch.float64, device="cuda:0")
    it = torch.empty(prob.n_frag, dtype=torch.int32, device="cuda:0")
    Wd = h.empty_K()
    h.fragment_solve(K, e, it, Wd)
    dF = torch.empty((n, n), dtype=torch.float64, device="cuda:0")
    h.mbe3_backward(h.osv_project(h.empty_gamma()), Wd, dEdF=dF)
    assert np.array_equal(it.cpu().numpy(), ref["iters"])
    for got, want in ((e, ref["e_frag"]), (Wd, Wref), (dF, 0.5 * (df + df.T))):
        assert np.abs(got.cpu().numpy() - want).max() <= 1e-11 * np.abs(want).max()
    # energy alone: without the gradient the amplitudes are not stored
    e2 = torch.empty_like(e)
    h.fragment_solve(K, e2, it)
    assert np.abs(e2.cpu().numpy() - ref["e_frag"]).max() <= 1e-11 * np.abs(ref["e_frag"]).max()
    h.close()
