"""The tuner times no schedule twice: settings that run the same kernel over the same
tiles (unroll, and min_waves with one lane per ray) appear once."""

from paper_1611_09048_amd import autotune


def test_no_schedule_twice():
    seen = set()
    for w, x, u, g, m, p in autotune.candidates():
        key = (w, x, g, m if g > 1 else None, p)
        assert key not in seen, key
        seen.add(key)


def test_given_axes_are_kept():
    assert {c[4] for c in autotune.candidates(min_waves=(4,), lanes=(1, 4))} == {4}
    assert {c[2] for c in autotune.candidates(unrolls=(2,), min_waves=(0,), lanes=(1,))} == {2}
