"""Device blocks that a handle keeps from its allocating calls: reused by the next
one, given back by mbe3_release_blocks, to an allocation that fails beside them and
with the handle, and never more than 512 MiB (no GPU needed; stand-in HIP runtime)."""
import _fake

BODY = """
    prob = synth.micro(n_occ=5, n_vir=40, n_aux=60, r=(7, 21))
    h, lay = handle(prob)
    idle = fake.fake_in_use()
    pairs = np.array([[i, j] for i in range(5) for j in range(i)], dtype=np.int32)

    def screen(times=1):
        pr, out = np.tile(pairs, (times, 1)), np.zeros(len(pairs) * times)
        return lib.mbe3_screen(h, ptr(pr), len(pr), ptr(out))
"""


def test_blocks_are_released(tmp_path):
    _fake.run(tmp_path, BODY + """
    assert screen() == 0
    kept = fake.fake_in_use() - idle
    assert 0 < kept <= 512 << 20
    assert screen() == 0 and fake.fake_in_use() == idle + kept  # reused
    assert lib.mbe3_release_blocks(h) == 0 and fake.fake_in_use() == idle
    assert lib.mbe3_release_blocks(h) == 0
    assert screen() == 0 and fake.fake_in_use() == idle + kept
    assert lib.mbe3_graph_begin(h, 0) == 0
    assert lib.mbe3_release_blocks(h) == m.MBE3_EINVAL  # and the recording is lost
    assert lib.mbe3_graph_end(h) == m.MBE3_EINVAL
    assert lib.mbe3_release_blocks(None) == m.MBE3_EINVAL
    lib.mbe3_destroy(h)
    assert fake.fake_in_use() == 0
    """)


def test_blocks_are_bounded(tmp_path):
    _fake.run(tmp_path, BODY + """
    for times in (1, 300, 40000, 20, 30000, 60000, 1):
        assert screen(times) == 0
        assert fake.fake_in_use() - idle <= 512 << 20, times
    assert fake.fake_in_use() - idle > 256 << 20
    # an allocation of the handle that finds no room takes them back
    fake.fake_capacity(fake.fake_in_use())
    assert screen(4000) == 0 and fake.fake_in_use() > idle
    lib.mbe3_destroy(h)
    assert fake.fake_in_use() == 0
    """)
