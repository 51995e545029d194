"""The pooled schedule with fewer rays than its waves take at first, about as many, and
several times as many: the tiled schedule's image and counts, bit for bit."""

import numpy as np
import pytest

from scenes import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [(3, 2), (61, 47), (380, 290), (1100, 900)])
@pytest.mark.parametrize("kind", ["scalar", "pic3", "pic3_f16_direct"])
@pytest.mark.parametrize("lanes", [2, 4, 8, 16])
def test_every_ray_is_handed_out_once(lanes, kind, size):
    from paper_1611_09048_amd import DIRECT, Context, device
    if kind.startswith("pic3"):
        sc, flags = configs.pic3(n=14, dtype="f16" if "f16" in kind else "f32", n_clip=1), DIRECT if "direct" in kind else 0
    else:
        sc, flags = configs.plain_scalar(n=14).with_(interpolation=1), 0
    sc = sc.with_(width=size[0], height=size[1], step=0.61, camera=configs.orbit_camera(sc.dims, (0.5, -0.7, 0.4), 0.6))
    got = []
    for pooled in (0, 1):
        with Context(device=0) as ctx:
            for c in range(16):
                ctx.set_tile_shape(c, 2, 1, 1, lanes, 0, pooled)
            keep = device.upload_volume(ctx, sc, 0)
            img, cnt = device.new_image(sc), device.new_counts(sc)
            for _ in range(2):
                img.fill_(-1.0)
                ctx.render([device.render_job(sc, 0, img, cnt)], flags)
            got.append((img.cpu().numpy(), cnt.cpu().numpy()))
            del keep
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
