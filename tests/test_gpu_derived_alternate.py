"""Calls of different kinds taking turns on one volume (trilinear, nearest, iso, fewer
sources) derive into one buffer, sized for the largest: every image is that of the
sources read in place, bit for bit."""

import dataclasses

import numpy as np
import pytest

from scenes import configs, relayout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("guard", [0, 1])
@pytest.mark.parametrize("dims", [(19, 22, 17), (24, 24, 24)])
def test_alternating_kinds_equal_direct(guard, dims):
    import torch
    from paper_1611_09048_amd import ASYNC, DERIVE, DIRECT, ISO, Context, device
    sc = configs.pic3(n=max(dims), width=96, height=72)
    cut = tuple(slice(1 - guard, 1 + n + guard) for n in reversed(dims))
    sc = sc.with_(dims=dims, camera=configs.orbit_camera(dims, (0.7, -0.5, 0.6)),
                  sources=[relayout(dataclasses.replace(s, guard=guard, values=s.values[cut])) for s in sc.sources])
    kinds = [dict(interpolation=1), dict(interpolation=0), dict(interpolation=1, mode=ISO, iso_values=[1.0, 0.2, 0.3]),
             dict(interpolation=1, enabled=[1, 0, 1])]
    with Context(device=0) as ctx:
        vol = device.upload_volume(ctx, sc, 0)
        want = []
        for kw in kinds:
            img, cnt = device.new_image(sc), device.new_counts(sc)
            ctx.render([device.render_job(sc, 0, img, cnt, **kw)], DIRECT)
            want.append((img.cpu().numpy(), cnt.cpu().numpy()))
            assert np.isfinite(want[-1][0]).all() and want[-1][1].max() > 0
        outs = []
        for k in (0, 1, 2, 3, 2, 0, 3, 1, 0):              # no wait in between: one buffer, one stream
            img, cnt = device.new_image(sc), device.new_counts(sc)
            ctx.render([device.render_job(sc, 0, img, cnt, **kinds[k])], DERIVE | ASYNC)
            outs.append((k, img, cnt))
        torch.cuda.synchronize()
        for k, img, cnt in outs:
            assert np.array_equal(img.cpu().numpy(), want[k][0]) and np.array_equal(cnt.cpu().numpy(), want[k][1]), k
        del vol
