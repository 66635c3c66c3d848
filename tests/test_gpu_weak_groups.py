"""Screening and weak pairs take a column block per second LMO: pair lists in any
order, with repeats and with one partner or many, unequal OSV counts on either
side of a 16- and a 32-row block, diagonal blocks that are not symmetric (needs an
MI355X).  Against the oracle, pair by pair."""
import numpy as np
import pytest

import oracle
import synth
from oracle import weak

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def m():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2603_16575_amd as pkg
    pkg._lib.load()
    return pkg


@pytest.mark.parametrize("n_occ,n_vir,n_aux,r", [
    (2, 4, 6, (1, 2)), (4, 37, 41, (3, 17)), (12, 50, 67, (14, 35)), (3, 120, 130, (60, 72))])
def test_weak_groups(m, n_occ, n_vir, n_aux, r):
    import torch
    print(f"case: {n_occ} LMOs, r {r}", flush=True)
    prob = synth.micro(n_occ=n_occ, n_vir=n_vir, n_aux=n_aux, r=r, seed=5)
    ora = oracle.Oracle(prob)
    h = m.from_problem(prob, device="cuda:0")
    gamma = h.osv_project(h.empty_gamma())
    rng = np.random.default_rng(3)
    Td, W = [], np.zeros(int(h.k_off[-1]))
    for i in range(n_occ):
        ri = int(round((h.k_off[i + 1] - h.k_off[i]) ** 0.5))
        b = 0.05 * rng.standard_normal((ri, ri))
        Td.append(b)
        W[h.k_off[i]:h.k_off[i + 1]] = b.ravel()
    Wd = torch.as_tensor(W, device="cuda:0")
    pr = np.array([(i, j) for i in range(n_occ) for j in range(i + 1, n_occ)], dtype=np.int32)
    pr = rng.permutation(np.concatenate([pr, pr[:1]]))
    ref = np.array([weak.weak_energies(ora, p[None], Td)[0] for p in pr])
    for sel in (slice(None), slice(0, 1)):
        e = h.weak_pairs(pr[sel], gamma, Wd).cpu().numpy()
        # FP64 sums of at most 130 x 72 terms, conditioned bases: as the chain's pairs
        assert np.abs(e - ref[sel]).max() <= 1e-9 * np.abs(ref).max()
    both = rng.permutation(np.concatenate([pr, pr[:, ::-1]]))
    s = h.screen(both).cpu().numpy()
    sref = np.array([weak.s2b(ora, int(i), int(j)) for i, j in both])
    assert np.abs(s - sref).max() <= 1e-13 * np.abs(sref).max()
    h.close()


def test_kept_blocks(m):
    """Calls whose device blocks the handle keeps give the same bits whatever the
    calls before left in them: mixed calls of several sizes against the first of
    their kind on a handle of its own."""
    import torch
    prob = synth.micro(n_occ=6, n_vir=70, n_aux=90, r=(9, 20), seed=8)
    pr = np.array([(i, j) for i in range(6) for j in range(i + 1, 6)], dtype=np.int32)

    def calls(h):
        gamma = h.osv_project(h.empty_gamma())
        W = h.pair_K(gamma, h.empty_K())
        s = h.fit_metric()
        cut = float(s.median())
        return [lambda: h.screen(pr), lambda: h.weak_pairs(pr, gamma, W),
                lambda: h.screen(pr[:2]), lambda: h.project_fit(s, 0.0, h.empty_gamma()),
                lambda: h.pair_K_fit(s, cut, h.empty_K()), lambda: h.rosv(n_max=30)["Q"],
                lambda: h.weak_pairs(pr[3:5], gamma, W), lambda: h.project_fit(s, cut, h.empty_gamma()),
                lambda: h.rosv(n_max=12, s_fit=s, l_fit=cut)["Q"]]

    ref = []
    for k in range(9):
        h = m.from_problem(prob, device="cuda:0")
        ref.append(calls(h)[k]().cpu())
        h.close()
    h = m.from_problem(prob, device="cuda:0")
    c = calls(h)
    for k in np.random.default_rng(2).integers(0, 9, 40):
        assert torch.equal(c[k]().cpu(), ref[k]), k
    h.close()
