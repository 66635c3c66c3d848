"""bench.py prints one JSON line, which has to stay short enough to be read from the
end of a log: the tuner's part is a summary whatever the number of task lists."""
import json

import bench

SHAPES = ["64x64", "128x128", "32x32", "32x128", "64x128", "96x96"]


def test_tuner_summary_is_short():
    n = 140
    report = "".join(
        f"{k} cross {k} (1234 tasks): " + " ".join(f"{s} {1.0 + i} ms" for i, s in enumerate(SHAPES))
        + f" -> {SHAPES[k % 4]} (was {SHAPES[0]})\n" for k in range(n))
    out = bench.tune_choices(report)
    assert out["lists"] == n
    assert out["chosen"] == {s: n // 4 for s in SHAPES[:4]}
    assert len(json.dumps(out)) < 200
