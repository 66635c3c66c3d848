"""Slabs with more rows or columns than one launch's grid takes in its second
dimension (needs an MI355X): 65535 groups of 16 rows of a regenerated slab, of 16
columns of its split planes, of 64 rows of compacted columns.  Projections
against Q^T B of the oracle's slab.  A product differs from the exact one by the
rounding of a sum of n terms and of the normals (4 ulp each): well below 1e-12 of
sum |q b|; split precision, 2^-22 of it."""
import types

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def m():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2603_16575_amd as pkg
    pkg._lib.load()
    return pkg


@pytest.mark.parametrize("form,n_vir,n_aux", [
    ("slab", 65535 * 16 + 19, 3), ("split", 9, 65535 * 16 + 19), ("columns", 65535 * 64 + 67, 2)])
def test_past_one_grid(m, form, n_vir, n_aux):
    import torch
    print(f"case: {form}, {n_vir} x {n_aux}", flush=True)
    n = 2
    g = np.random.default_rng(3)
    p = types.SimpleNamespace(seed=17, n_vir=n_vir, n_aux=n_aux,
                              w_ia=g.uniform(0.05, 0.1, (n, n_vir)),
                              w_iP=g.uniform(0.2, 1.0, (n, n_aux)))
    Q = g.standard_normal((n, n_vir))
    Q /= np.linalg.norm(Q, axis=1)[:, None]
    dev = dict(device="cuda:0", dtype=torch.float64)
    f = np.array([[-0.9, 0.02], [0.02, -0.7]])
    h = m.Mbe3(r=[1, 1], Q=torch.as_tensor(Q, **dev),
                 eps_vir=torch.linspace(0.2, 4.0, n_vir, **dev), f_occ=torch.as_tensor(f, **dev),
                 pairs=[[0, 1]], frags=[[0, -1, -1], [1, -1, -1], [0, 1, -1]], seed=p.seed,
                 w_ia=torch.as_tensor(p.w_ia, **dev), w_iP=torch.as_tensor(p.w_iP, **dev),
                 precision=m.MBE3_MIXED_BF16_PROJ if form == "split" else m.MBE3_FP64)
    gamma = h.empty_gamma()
    if form == "columns":
        s_fit = torch.ones((n, n_aux), **dev)
        h.project_fit(s_fit, 0.5, gamma)
    else:
        h.osv_project(gamma)
    got = gamma.cpu().numpy().reshape(n, n, n_aux)  # [i][x][P], one OSV each
    eps = 2.0 ** -22 if form == "split" else 1e-12
    for i in range(n):
        B = oracle.mbe3.slab(p, i)
        assert np.all(np.abs(got[i] - Q @ B) <= eps * (np.abs(Q) @ np.abs(B)))
    h.close()
