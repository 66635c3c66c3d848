"""Runs a piece of Python in a child process whose library calls the stand-in HIP
runtime of fake_hip.c (no GPU needed): `fake` is that runtime, `lib` the library,
`problem(prob)` an mbe3_problem over host arrays, `handle(prob)` a created handle."""
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = textwrap.dedent("""
    import ctypes, sys
    sys.path.insert(0, {root!r})
    fake = ctypes.CDLL({so!r}, mode=ctypes.RTLD_GLOBAL)
    for f in ("refuse", "capacity", "in_use", "asked", "launches"):
        getattr(fake, "fake_" + f).restype = ctypes.c_int64
    for f in ("refuse", "capacity", "asked"):
        getattr(fake, "fake_" + f).argtypes = [ctypes.c_size_t]
    import numpy as np
    import paper_2603_16575_amd as m
    import synth
    lib = m._lib.load()
    ptr = m._lib.ptr
    keep = []

    def problem(prob, warm_start=True):
        p = m._lib.Mbe3Problem()
        a = [np.ascontiguousarray(x) for x in (prob.r, prob.QT_packed, prob.eps_vir, prob.f_occ,
                                               prob.w_ia, prob.w_iP, prob.pairs, prob.frags)]
        keep.append(a)
        p.n_occ, p.n_vir, p.n_aux, p.seed = prob.n_occ, prob.n_vir, prob.n_aux, prob.seed
        p.r, p.Q, p.eps_vir, p.f_occ, p.w_ia, p.w_iP, p.pairs, p.frags = map(ptr, a)
        p.n_pair, p.n_frag, p.tol, p.max_iter = len(a[6]), len(a[7]), prob.tol, prob.max_iter
        p.tau_S, p.warm_start = prob.tau_S, int(warm_start)
        return p

    def handle(prob, **kw):
        h = ctypes.c_void_p()
        rc = lib.mbe3_create(ctypes.byref(h), ctypes.byref(problem(prob, **kw)), None)
        assert rc == 0, lib.mbe3_last_error(None)
        lay = m._lib.Mbe3Layout()
        lib.mbe3_get_layout(h, ctypes.byref(lay))
        return h, lay

    def solve(h, lay, W=False):
        K = np.zeros(lay.k_elems)
        e, it = np.zeros(lay.n_frag), np.zeros(lay.n_frag, dtype=np.int32)
        keep.append((K, e, it))
        return lib.fragment_solve(h, ptr(K), ptr(e), ptr(it), ptr(np.zeros_like(K)) if W else None)
""")


def run(tmp_path, body):
    """Child process over PRELUDE + body; fails the test with its output."""
    so = str(tmp_path / "fake_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.c"), "-o", so],
                   check=True)
    src = PRELUDE.format(root=ROOT, so=so) + textwrap.dedent(body)
    res = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, (res.stdout + res.stderr)[-4000:]
    return res.stdout
