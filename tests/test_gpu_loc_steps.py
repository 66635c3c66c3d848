"""The antidiagonal steps of mbe3_pm_localize against the oracle's pair-by-pair
sweeps (needs an MI355X): one orbital, one pair, odd and even orbital counts,
one atom, atom counts around the lanes of an angle, column groups at and past a
workgroup's share, and charges past the two-buffer limit (64 MiB), which are
rotated in place."""
import numpy as np
import pytest

from oracle import loc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def m():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2603_16575_amd as pkg
    pkg._lib.load()
    return pkg


@pytest.mark.parametrize("n,na,max_sweeps", [
    (1, 3, 4), (2, 1, 4), (2, 17, 4), (3, 5, 4), (4, 16, 4), (7, 15, 4), (8, 40, 4),
    (9, 17, 4), (33, 12, 3), (24, 30000, 2)])
def test_pm_steps_match_pair_order(m, n, na, max_sweeps):
    import torch
    print(f"case: {n} orbitals, {na} atoms, {max_sweeps} sweeps", flush=True)
    g = np.random.default_rng(1000 * n + na)
    per = max(1, -(-2 * n // na))  # AOs per atom
    C, _ = np.linalg.qr(g.standard_normal((na * per, n)))
    if na == 1:  # orthonormal columns on one atom have no angle: any C does
        C = g.standard_normal(C.shape)
    off = np.arange(na + 1, dtype=np.int32) * per
    out = m.pm_localize(torch.as_tensor(C, device="cuda:0"), off, l_loc=-1.0,
                        max_sweeps=max_sweeps, check=False)
    ref = loc.jacobi_pm(loc.charges(C, off), l_loc=-1.0, max_sweeps=max_sweeps)
    assert out["sweeps"] == ref["sweeps"]
    assert np.array_equal(out["rotations"][:1], np.array(ref["rotations"])[:1])
    U, P = out["U"].cpu().numpy(), np.transpose(out["P"].cpu().numpy(), (2, 0, 1))
    # early sweeps are not contracting: rounding differences grow along the path
    assert abs(out["dL"][0] - ref["dL"][0]) <= 1e-9 * max(abs(ref["dL"][0]), 1e-9)
    assert np.abs(U - ref["U"]).max() <= 1e-6
    assert np.abs(P - ref["P"]).max() <= 1e-6
    assert np.abs(U.T @ U - np.eye(n)).max() <= 1e-12
    assert np.abs(P - loc.charges(C @ U, off)).max() <= 1e-12 * max(1.0, np.abs(P).max())
