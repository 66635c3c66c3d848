"""Screening and weak pairs of more pairs than one launch of a workgroup each takes
(2^32 threads: 2^24 workgroups of 256), one pair listed over and over: every
result is that of the pair by itself (needs an MI355X)."""
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


def test_more_pairs_than_workgroups(m):
    import torch
    n = (1 << 24) + 3
    print(f"case: {n} pairs", flush=True)
    prob = synth.micro(n_occ=2, n_vir=16, n_aux=24, r=(1, 1))
    h = m.from_problem(prob, device="cuda:0")
    out = h.forward(grad=True)
    one = np.array([[0, 1]], dtype=np.int32)
    pairs = np.tile(one, (n, 1))
    for name, got, want in (
            ("screen", h.screen(pairs), h.screen(one)),
            ("weak", h.weak_pairs(pairs, out["gamma"], out["W"]),
             h.weak_pairs(one, out["gamma"], out["W"]))):
        print(f"  {name}", flush=True)
        assert float(want[0]) != 0.0
        assert bool((got == want[0]).all()), name
    h.close()
    torch.cuda.empty_cache()
