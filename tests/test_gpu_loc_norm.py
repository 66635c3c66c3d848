"""The rotations of mbe3_pm_localize keep lengths to rounding (needs an MI355X):
no bias in the norms of the columns of U after many of them.  With cosine and sine
rounded at random, a column turned R times is off by about 2^-53 sqrt(R) (the
rounding of c^2 + s^2 and of the column's elements, a random walk), and the mean of
n columns by less; a cosine and sine that are too short by half an ulp each time
would give 2^-53 R."""
import numpy as np
import pytest

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


@pytest.mark.parametrize("k", [0, 1, "random 60", "random 96"])
def test_rotations_keep_lengths(m, k):
    import torch
    print(f"case: {k}", flush=True)
    if k in (0, 1):
        lp = synth.loc_config(k)
        C, off = lp.C, lp.ao_off
    else:
        n = int(k.split()[1])
        na = 3 * n // 4
        C, _ = np.linalg.qr(np.random.default_rng(n).standard_normal((6 * na, n)))
        off = np.arange(na + 1, dtype=np.int32) * 6
    out = m.pm_localize(torch.as_tensor(C, device="cuda:0"), off, l_loc=1e-6, max_sweeps=40,
                        check=False)
    U = out["U"].cpu().numpy().astype(np.longdouble)
    turns = 2.0 * np.sum(out["rotations"]) / U.shape[1]  # a column's share
    d = np.sum(U * U, axis=0) - 1
    print(f"  {turns:.0f} turns per column, mean {float(d.mean()):.2e}, max "
          f"{float(np.abs(d).max()):.2e}", flush=True)
    assert abs(d.mean()) <= 2.0 ** -53 * np.sqrt(turns)
