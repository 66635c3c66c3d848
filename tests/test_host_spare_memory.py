"""Stores that only save time are done without where memory is short (no GPU
needed; the stand-in HIP runtime refuses the allocation)."""
import _fake

BASE = """
    prob = synth.micro(n_occ=5, n_vir=40, n_aux=60, r=(7, 21))
    D = lambda d: (int(d) + 15) // 16 * 16
    want = 8 * sum(D(prob.r[p]) ** 2 + D(prob.r[q]) ** 2 + D(prob.r[p] + prob.r[q]) ** 2
                   for p, q in prob.pairs)
"""


def test_create_without_the_coupling_sums(tmp_path):
    """The sums of a dimer's couplings are a shortcut of its trimers' first sweep:
    without room for them the handle is made and the trimers form their own."""
    _fake.run(tmp_path, BASE + """
    h, lay = handle(prob)
    assert fake.fake_asked(want) == 1, "the store is not where this test looks for it"
    assert solve(h, lay) == 0 and fake.fake_launches(b"ELi3ELi") > 0
    lib.mbe3_destroy(h)
    assert fake.fake_in_use() == 0
    fake.fake_refuse(want)
    before = fake.fake_launches(b"ELi3ELi")
    h, lay = handle(prob)
    assert solve(h, lay) == 0 and solve(h, lay, W=True) == 0
    assert fake.fake_launches(b"ELi3ELi") == before
    lib.mbe3_destroy(h)
    assert fake.fake_in_use() == 0
    """)


def test_coupling_sums_make_room(tmp_path):
    """They are given up for an allocation of the handle that fails beside them (the
    gradient's workspace), but not while a recorded graph names them."""
    _fake.run(tmp_path, BASE + """
    h, lay = handle(prob)
    assert solve(h, lay) == 0
    used = fake.fake_in_use()
    n0 = fake.fake_launches(b"ELi3ELi")
    assert solve(h, lay, W=True) == 0
    need = fake.fake_in_use() - used
    lib.mbe3_destroy(h)
    for recorded in (False, True):
        h, lay = handle(prob)
        assert solve(h, lay) == 0 and fake.fake_in_use() == used
        if recorded:
            assert lib.mbe3_graph_begin(h, 0) == 0 and solve(h, lay) == 0
            assert lib.mbe3_graph_end(h) == 0
        n0 = fake.fake_launches(b"ELi3ELi")
        fake.fake_capacity(used + need - want // 2)
        rc = solve(h, lay, W=True)
        fake.fake_capacity(2 ** 62)
        if recorded:
            assert rc == m.MBE3_ENOMEM
        else:
            assert rc == 0 and fake.fake_launches(b"ELi3ELi") == n0
            assert fake.fake_in_use() == used + need - want
        lib.mbe3_destroy(h)
        assert fake.fake_in_use() == 0
    """)


def test_localization_without_a_second_buffer(tmp_path):
    """Charges of up to 64 MiB move between two buffers; where the second does not fit
    they are turned in place."""
    _fake.run(tmp_path, """
    n, na = 24, 18
    C = np.zeros((n * 4, n)); off = np.arange(na + 1, dtype=np.int32); off[-1] = n * 4
    P, U, ns = np.zeros((n, n, na)), np.zeros((n, n)), np.zeros(1, dtype=np.int32)
    def call():
        return lib.mbe3_pm_localize(ptr(C), ptr(off), n * 4, n, na, 1e-3, 5, ptr(P), ptr(U), None,
                                    None, ptr(ns), None)
    assert call() == 0 and fake.fake_asked(P.nbytes) == 1
    assert fake.fake_launches(b"pm_step") == 2 * n - 3 and fake.fake_launches(b"pm_angle") == 0
    fake.fake_refuse(P.nbytes)
    assert call() == 0, lib.mbe3_last_error(None)
    assert fake.fake_launches(b"pm_step") == 4 * n - 6
    assert fake.fake_launches(b"pm_angle") == 2 * n - 3
    assert ns[0] == 1 and fake.fake_in_use() == 0
    """)
