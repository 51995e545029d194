"""FP16 and BF16 fields read in place: the aligned window that holds both x corners
of a scalar or 3-vector must give the values of the derive pass, which reads them
one by one, whatever the parity of rows, planes and of the field's first byte, on
the last voxels of the range too; fields that are not x-adjacent keep their loop."""

import dataclasses

import numpy as np
import pytest

from scenes import configs, relayout

pytestmark = pytest.mark.gpu

LAYOUTS = [dict(pitch_align=2), dict(pitch_align=4), dict(pitch_align=256), dict(pitch_align=2, extra_layers=1),
           dict(pitch_align=2, extra_layers=2), dict(pitch_align=2, flip=(False, True, False)),
           dict(pitch_align=2, flip=(False, False, True)), dict(pitch_align=2, order=(0, 2, 1)),
           dict(pitch_align=2, order=(1, 0, 2)), dict(pitch_align=2, flip=(True, False, False))]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("layout", range(len(LAYOUTS)))
def test_half_pairs_equal_derived(dtype, layout):
    from paper_1611_09048_amd import DERIVE, DIRECT, Context, device
    for dims in ((1, 1, 1), (2, 3, 1), (7, 5, 6), (24, 17, 13)):
        sc = configs.pic3(seed=3 + layout, dims=dims, width=67, height=58, dtype=dtype, n_clip=0)
        sc = sc.with_(sources=[relayout(s, **LAYOUTS[layout]) for s in sc.sources], step=0.3,
                      camera=configs.orbit_camera(dims, (0.4, -0.6, 0.5), 1.1))
        for shape in ((8, 2, 1, 1, 0, 0), (4, 1, 1, 16, 4, 0), (4, 1, 1, 16, 0, 0)):
            with Context(device=0) as ctx:
                for c in range(16):
                    ctx.set_tile_shape(c, *shape)
                a = device.render_scene(ctx, sc, flags=DIRECT)
                b = device.render_scene(ctx, sc, flags=DERIVE)
            assert np.isfinite(a[0]).all() and a[1].max() > 0
            assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), (dims, shape)


def test_mixed_adjacency():
    """One source x-adjacent, another not: the launch keeps the value-by-value loads."""
    from paper_1611_09048_amd import DERIVE, DIRECT, Context, device
    sc = configs.pic3(dims=(15, 12, 9), width=64, height=48, dtype="f16")
    wide = relayout(sc.sources[1], pitch_align=2, order=(1, 0, 2))
    sc = sc.with_(sources=[sc.sources[0], dataclasses.replace(wide), sc.sources[2]])
    with Context(device=0) as ctx:
        a = device.render_scene(ctx, sc, flags=DIRECT)
        b = device.render_scene(ctx, sc, flags=DERIVE)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
