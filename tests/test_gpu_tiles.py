"""One workgroup per tile: an image of more tiles than one grid takes is launched in
parts.  Rays of a single scan point give the same pixel in every schedule, so 64
lanes per ray (16.8 M tiles, three launches) must equal one lane per ray."""

import pytest

from scenes import configs, fields, make_source
from scenes.layout import Camera, Scene

pytestmark = pytest.mark.gpu


def test_more_tiles_than_one_grid():
    import numpy as np
    import torch
    from paper_1611_09048_amd import Context, device
    rng = np.random.default_rng(5)
    src = make_source("s", fields.uniform_random(rng, (6, 6, 1), 1, 1, 0.2, 0.9), guard=1, tf=configs.random_tf(rng, 5, 0.6))
    cam = Camera(eye=(3.0, 3.0, -4.0), center=(3.0, 3.0, 0.5), up=(0.0, 1.0, 0.0), projection="orthographic",
                 ortho_height=5.9)
    sc = Scene(dims=(6, 6, 1), sources=[src], camera=cam, width=8192, height=8192, step=1.5, interpolation=1)
    with Context(device=0) as ctx:
        vol = device.upload_volume(ctx, sc, 0)
        one, many = device.new_image(sc), device.new_image(sc)
        ctx.render([device.render_job(sc, 0, one)])
        ctx.set_tile_shape(13, 1, 1, 1, 64, 0, 0)
        ctx.render([device.render_job(sc, 0, many)])
        torch.cuda.synchronize()
        assert float(one[..., 3].min()) > 0 and bool((one == many).all())
        del vol
