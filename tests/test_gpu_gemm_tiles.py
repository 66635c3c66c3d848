"""Grouped FP64 products at the edges of their tiles (needs an MI355X): slab
dimensions below, at and past the 16-deep steps and the 32- to 128-wide tiles,
odd ones (rows at 8-byte alignment, a last chunk that is shifted) and ones that
take the general kernel (a single row or column), through every tile shape:
projection, pair_K, dE/dGamma and dE/dB against plain FP64 products."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def m():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2603_16575_amd as pkg
    pkg._lib.load()
    return pkg


@pytest.mark.parametrize("n_vir,n_aux,r", [
    (1, 1, (1, 1, 1)), (2, 2, (1, 2, 1)), (2, 1, (1, 2, 2)), (3, 5, (3, 1, 2)),
    (15, 16, (5, 7, 3)), (16, 17, (16, 3, 8)), (17, 31, (17, 9, 1)), (33, 32, (20, 33, 2)),
    (64, 127, (31, 32, 33)), (95, 129, (47, 48, 49)), (130, 97, (64, 65, 15)),
    (257, 191, (70, 12, 64))])
def test_products_at_tile_edges(m, n_vir, n_aux, r):
    import torch
    print(f"case: n_vir {n_vir}, n_aux {n_aux}, r {r}", flush=True)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(n_vir * 1000 + n_aux)
    rnd = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64, device="cuda:0")
    n = 3
    slab, Q = rnd(n, n_vir, n_aux), rnd(sum(r), n_vir)
    pairs = np.array([[0, 1], [0, 2], [1, 2]], dtype=np.int32)
    frags = np.array([[0, -1, -1], [1, -1, -1], [2, -1, -1]], dtype=np.int32)
    h = m.Mbe3(r=np.array(r), Q=Q, eps_vir=rnd(n_vir).abs() + 1.0,
               f_occ=-torch.eye(n, dtype=torch.float64, device="cuda:0"), pairs=pairs,
               frags=frags, slab=slab)
    W = rnd(int(h.layout.k_elems))
    off = np.concatenate([[0], np.cumsum(r)])
    q = [Q[off[i]:off[i + 1]] for i in range(n)]
    G = [[qx @ slab[i] for qx in q] for i in range(n)]  # N+(i) is everything
    slots = [(i, i) for i in range(n)] + [tuple(p) for p in pairs.tolist()]
    eps = 2.0 ** -52

    def close(x, ref, bound):
        assert bool((x - ref).abs().le(bound + 1e-300).all()), float((x - ref).abs().max())

    refG = torch.cat([torch.cat(Gi) for Gi in G]).reshape(-1)
    absG = torch.cat([torch.cat([qx.abs() @ slab[i].abs() for qx in q]) for i in range(n)])
    refB = torch.zeros_like(slab)
    absB = torch.zeros_like(slab)
    refK, absK = [], []
    for s, (a, b) in enumerate(slots):
        o = [a] if a == b else [a, b]
        L, R = torch.cat([G[a][x] for x in o]), torch.cat([G[b][x] for x in o])
        refK.append((L @ R.T).reshape(-1))
        absK.append((L.abs() @ R.abs().T).reshape(-1))
        V = torch.cat([q[x] for x in o])
        w = W[h.k_off[s]:h.k_off[s + 1]].reshape(len(V), len(V))
        c = 2.0 if a == b else 4.0
        refB[a] += c * V.T @ (w @ R)
        refB[b] += c * V.T @ (w.T @ L)
        absB[a] += c * V.abs().T @ (w.abs() @ (V.abs() @ slab[b].abs()))
        absB[b] += c * V.abs().T @ (w.abs().T @ (V.abs() @ slab[a].abs()))
    first = None
    for shape in range(6):
        h.set_gemm_shape(shape)
        gamma = h.osv_project(h.empty_gamma())
        K = h.pair_K(gamma, h.empty_K())
        # sums over n terms in any order differ by at most n eps of sum |a b|
        close(gamma, refG, 2 * n_vir * eps * absG.reshape(-1))
        close(K, torch.cat(refK), 4 * (n_aux + n_vir) * eps * torch.cat(absK) * 4)
        if h.n_vir > 1:
            h.pair_K(gamma, K)
            e = torch.empty(n, dtype=torch.float64, device="cuda:0")
            it = torch.empty(n, dtype=torch.int32, device="cuda:0")
            Wd = h.empty_K()
            h.fragment_solve(K, e, it, Wd, check=False)  # plans the gradient
            h.set_gemm_shape(shape)
            dB, _ = h.mbe3_backward(gamma, W)
            terms = n_vir + 2 * max(r) * n + n * max(r)
            close(dB, refB, 8 * terms * eps * absB)
            out = torch.cat([gamma, K, dB.reshape(-1)])
        else:
            out = torch.cat([gamma, K])
        first = out if first is None else first
        assert torch.equal(out, first)  # every shape sums in the same order
    h.close()
