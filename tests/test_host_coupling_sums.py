"""Which pairs' coupling sums a warm-started handle stores: those of pairs in
trimers that the LDS-resident solver takes, and none where the trimers share too few
pairs for the sums to pay (no GPU needed; stand-in HIP runtime)."""
import _fake

BODY = """
    import dataclasses
    D = lambda d: (int(d) + 15) // 16 * 16

    def used(prob, tri, warm=True):
        # bytes of the store of these trimers' pairs, were it allocated and launched?
        prob = dataclasses.replace(prob, trimers=np.array(tri, dtype=np.int32).reshape(-1, 3))
        prs = sorted({(t[a], t[b]) for t in prob.trimers.tolist() for a, b in ((0, 1), (0, 2), (1, 2))})
        want = 8 * sum(D(prob.r[p]) ** 2 + D(prob.r[q]) ** 2 + D(prob.r[p] + prob.r[q]) ** 2
                       for p, q in prs)
        n0, a0 = fake.fake_launches(b"ELi3ELi"), fake.fake_asked(want)
        u0 = fake.fake_in_use()
        h, lay = handle(prob, warm_start=warm)
        got = fake.fake_asked(want) - a0 if prs else 0
        assert solve(h, lay) == 0
        launched = fake.fake_launches(b"ELi3ELi") - n0
        lib.mbe3_destroy(h)
        assert fake.fake_in_use() == u0
        assert (got > 0) == (launched > 0), (got, launched)
        return launched > 0

    def all_of(n):
        return [[i, j, k] for i in range(n) for j in range(i + 1, n) for k in range(j + 1, n)]
"""


def test_shared_pairs_only(tmp_path):
    _fake.run(tmp_path, BODY + """
    prob = synth.micro(n_occ=9, n_vir=60, n_aux=80, r=(17, 23))
    assert not used(prob, [])
    assert not used(prob, [[0, 1, 2]]) and not used(prob, [[0, 1, 2], [3, 4, 5]])
    assert not used(prob, [[0, 1, 2], [0, 1, 3], [0, 1, 4]])  # 9 sides over 7 pairs
    assert used(prob, all_of(4))  # 12 sides over 6 pairs, of the 36 pairs kept
    assert used(prob, all_of(9)) and not used(prob, all_of(9), warm=False)
    """)


def test_wide_trimers_have_none(tmp_path):
    _fake.run(tmp_path, BODY + """
    prob = synth.micro(n_occ=6, n_vir=200, n_aux=220, r=(10, 10))
    r = np.array([70, 10, 10, 10, 10, 70], dtype=np.int32)
    g = np.random.default_rng(0)
    Q = [np.linalg.qr(g.standard_normal((200, k)))[0] for k in r]
    prob = dataclasses.replace(prob, r=r, Q=Q)
    # pair (0, 5) is 140 wide: its trimers run in the wide solver and read no sums
    assert not used(prob, [[0, 1, 5], [0, 2, 5], [0, 3, 5], [0, 4, 5]])
    assert used(prob, [[i, j, k] for i, j, k in all_of(6) if not (i == 0 and k == 5)])
    """)
