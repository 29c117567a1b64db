"""The autotuner records no workgroup size that has no effect: FP64 generation does not go by the setting,
so whatever the timings, the size set before stays.  The timings are made up; no GPU."""
import itertools


def test_fp64_workgroup_size_is_kept(monkeypatch):
    from paper_1002_3446_amd import autotune, bg
    falling = itertools.count(1000.0, -1.0)   # each candidate seems faster than the one before
    monkeypatch.setattr(bg, "generate", lambda *a, **k: {})
    monkeypatch.setattr(autotune, "_time", lambda fn, reps=3: next(falling))
    try:
        for size in (64, 128, 256):
            for n in autotune.NS:
                bg.set_launch(n, 64, size, 1)
            shapes = autotune.tune_single(64, log=lambda *a: None)
            assert {s[0] for s in shapes.values()} == {size}
            assert {bg.get_launch(n, 64)[0] for n in autotune.NS} == {size}
        assert {s[0] for s in autotune.tune_single(32, log=lambda *a: None).values()} <= {64, 256}
    finally:
        for n in autotune.NS:
            for prec in (32, 64):
                bg.set_launch(n, prec, 0, 0)
                bg.set_lanes(n, prec, 0)
                bg.set_form(n, prec, 0)
        bg.load_tuning()
