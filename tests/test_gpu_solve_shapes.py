"""Fragment solver at every shape of its work split (needs an MI355X): OSV
counts that give diagonal targets of 1 - 8 and pair targets of 1 - 8 row blocks
(one block shared by all waves, blocks shared by two or four, the fifth block of
80-wide domains, whole blocks), source dimensions on both sides of the 16-row
padding and of its four-row steps, unequal orbitals in one trimer, starts from
T = 0 and from the pairs' own fragments, and the 160-wide instance.  Fragment
energies and update counts against the oracle."""
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


@pytest.mark.parametrize("warm", [False, True])
@pytest.mark.parametrize("r", [(1, 1), (5, 5), (8, 8), (9, 9), (12, 13), (16, 17), (23, 24),
                               (25, 32), (33, 33), (38, 40), (41, 41), (47, 48), (49, 52),
                               (57, 57), (64, 64), (1, 40), (3, 64), (30, 78), (70, 78)])
def test_solve_shapes(m, r, warm):
    print(f"case: r {r}, warm start {warm}", flush=True)
    prob = synth.micro(n_occ=4, n_vir=max(24, 4 * r[1]), n_aux=max(32, 5 * r[1]), r=r,
                       seed=100 * r[0] + r[1], tol=1e-9)
    ref = oracle.run(prob, warm_start=warm)
    h = m.from_problem(prob, device="cuda:0", warm_start=warm)
    out = h.forward(grad=True)
    e = out["e_frag"].cpu().numpy()
    assert np.array_equal(out["iters"].cpu().numpy(), ref["iters"])
    # the same iterates on both sides: rounding of sums over at most 4 r terms
    scale = np.abs(ref["e_frag"]).max()
    assert np.abs(e - ref["e_frag"]).max() <= 1e-12 * scale + 1e-15
    h.close()
