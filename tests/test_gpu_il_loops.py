"""The scan-point loops over plain FP32 values side by side (one scalar in place,
with and without guard layers; derived volumes of one, two and four sources)
against the general loop, bit for bit: a scalar stored with x adjacent takes the
x-pair loop, the same values stored in any other order or direction, or batched
with such a one, the general scalar loop; derived volumes against direct reads.
"""

import numpy as np
import pytest

from scenes import configs, fields, make_source, relayout
from scenes.layout import Scene

pytestmark = pytest.mark.gpu

SHAPES = [(8, 2, 1, 1, 0, 0), (8, 2, 2, 1, 0, 0), (8, 1, 1, 4, 0, 0), (8, 1, 1, 4, 4, 0), (4, 1, 1, 16, 4, 0),
          (4, 1, 1, 16, 0, 0), (1, 1, 1, 64, 0, 0), (8, 2, 1, 8, 0, 1)]


def scene(dims, guard, interp, n_src=1, seed=0, chain=""):
    rng = np.random.default_rng(1000 * seed + dims[0] + 10 * guard + interp)
    srcs = [make_source(f"s{k}", fields.uniform_random(rng, dims, guard, 1, 0.0, 1.0), guard=guard, chain=chain,
                        weight=0.9 - 0.2 * k, tf=configs.random_tf(rng, 5, 0.3)) for k in range(n_src)]
    return Scene(dims=dims, sources=srcs, camera=configs.orbit_camera(dims, (0.6, 0.5, -0.4), 1.1), width=53, height=45,
                 step=0.4, interpolation=interp, clip=[configs.random_clip_plane(rng, dims)] if dims[1] % 2 else [])


def render(sc, shape=None, flags=0):
    from paper_1611_09048_amd import Context, device
    with Context(device=0) as ctx:
        if shape:
            for c in range(16):
                ctx.set_tile_shape(c, *shape)
        return device.render_scene(ctx, sc, flags=flags)


def same(a, b):
    return np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("dims", [(1, 1, 1), (2, 1, 3), (3, 4, 2), (17, 12, 9), (40, 33, 21)])
@pytest.mark.parametrize("guard,interp", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_x_pairs_equal_the_general_scalar_loop(dims, guard, interp):
    sc = scene(dims, guard, interp)
    flipped = sc.with_(sources=[relayout(sc.sources[0], flip=(True, False, False))])
    turned = sc.with_(sources=[relayout(sc.sources[0], order=(2, 1, 0), flip=(False, True, False))])
    updown = sc.with_(sources=[relayout(sc.sources[0], flip=(False, True, True), pitch_align=4)])   # x pairs again
    for shape in SHAPES:
        a = render(sc, shape)
        assert np.isfinite(a[0]).all()
        for other in (flipped, turned, updown):
            assert same(a, render(other, shape)), shape
    assert a[1].max() > 0


@pytest.mark.parametrize("n_src", [1, 2, 3, 4])
@pytest.mark.parametrize("guard", [0, 1])
@pytest.mark.parametrize("interp", [0, 1])
def test_derived_loops_equal_direct(n_src, guard, interp):
    from paper_1611_09048_amd import DERIVE, DIRECT
    for dims in ((1, 1, 1), (19, 14, 23)):
        sc = scene(dims, guard, interp, n_src, seed=n_src, chain="mul(0.8) | add(0.05)")
        for shape in SHAPES:
            assert same(render(sc, shape, DIRECT), render(sc, shape, DERIVE)), (dims, shape)


def test_mixed_scalars_in_one_batch():
    """One launch over scalars of three forms equals each job rendered alone."""
    from paper_1611_09048_amd import Context, device
    a, b, c = scene((20, 15, 11), 1, 1, seed=1), scene((14, 9, 18), 0, 1, seed=2), scene((12, 22, 10), 1, 1, seed=3)
    scs = [a, b, c.with_(sources=[relayout(c.sources[0], flip=(True, True, False))])]
    with Context(device=0) as ctx:
        for cls in range(16):
            ctx.set_tile_shape(cls, 8, 2, 1, 4, 0, 0)
        vols = [device.upload_volume(ctx, s, k) for k, s in enumerate(scs)]
        imgs = [device.new_image(s) for s in scs]
        ctx.render([device.render_job(s, k, imgs[k]) for k, s in enumerate(scs)])
        batch = [i.cpu().numpy() for i in imgs]
        for k, s in enumerate(scs):
            ctx.render([device.render_job(s, k, imgs[k])])
            assert np.array_equal(batch[k], imgs[k].cpu().numpy())
        del vols


def test_frozen_without_guard_layers():
    """A frozen volume of guard-less sources reads its derived border layer."""
    from paper_1611_09048_amd import DIRECT, Context, device
    for n_src in (1, 2, 3, 4):
        sc = scene((13, 17, 10), 0, 1, n_src, seed=7 + n_src, chain="mul(0.8) | add(0.05)")
        with Context(device=0) as ctx:
            vol = device.upload_volume(ctx, sc, 0)
            img, ref = device.new_image(sc), device.new_image(sc)
            ctx.render([device.render_job(sc, 0, ref)], DIRECT)
            ctx.freeze_volume(0)
            ctx.render([device.render_job(sc, 0, img)])
            assert np.array_equal(img.cpu().numpy(), ref.cpu().numpy())
            del vol
