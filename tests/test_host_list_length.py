"""mbe3_screen_lists with a count far above the number of distinct pairs: the list is
refused where it first repeats or leaves the range, without memory in proportion to
the count (no GPU needed; in a child process, which an exception would end)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import sys
sys.path.insert(0, {root!r})
import numpy as np
import paper_2603_16575_amd as m
lib, ptr = m._lib.load(), m._lib.ptr
nc, nw, nt = (np.zeros(1, dtype=np.int64) for _ in range(3))
s = np.full(8, 0.5)
for pairs, word in (([[0, 1], [1, 2], [2, 0], [1, 0]], "repeats"), ([[0, 1], [0, 3]], "range")):
    p = np.array(pairs, dtype=np.int32)
    for n in (len(p), 2 ** 40, 2 ** 61, 2 ** 63 - 1):
        rc = lib.mbe3_screen_lists(3, ptr(p), n, ptr(s), m.S2B_DISTANT, m.S2B_CLOSE, m.S3B_KEEP,
                                   None, None, ptr(nc), None, ptr(nw), None, 0, ptr(nt))
        assert rc == m.MBE3_EINVAL, (n, rc)
        assert word in lib.mbe3_last_error(None).decode()
print("refused")
"""


def test_counts_beyond_the_distinct_pairs():
    res = subprocess.run([sys.executable, "-c", CHILD.format(root=ROOT)], capture_output=True,
                         text=True, timeout=120)
    assert res.returncode == 0 and "refused" in res.stdout, (res.returncode, res.stderr[-2000:])
