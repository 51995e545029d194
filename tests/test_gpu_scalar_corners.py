"""A scalar's corners one by one and in pairs: the same job alone, which loads them one
by one, and in a launch whose other view keeps the pairs, must give the same image and
counts, bit for bit."""

import numpy as np
import pytest

import oracle
from parity import compare
from scenes import configs, fields
from scenes.layout import make_source

pytestmark = pytest.mark.gpu

OBLIQUE, ALONG_X = (0.5, -0.7, 0.55), (1.0, 0.02, 0.03)


@pytest.mark.parametrize("n_clip", [0, 2])
@pytest.mark.parametrize("dims", [(20, 20, 20), (2, 17, 33), (31, 5, 6)])
@pytest.mark.parametrize("guard", [0, 1])
@pytest.mark.parametrize("lanes", [4, 8])
def test_single_corners_and_pairs_agree(lanes, guard, dims, n_clip):
    from paper_1611_09048_amd import DIRECT, Context, device
    rng = np.random.default_rng(7)
    tf = configs.random_tf(rng, 4, 0.03 if lanes == 4 else 0.9)
    src = make_source("s", fields.gaussian_blobs(rng, dims, guard=guard, scale=0.3), guard=guard, tf=tf)
    clip = [configs.random_clip_plane(rng, dims) for _ in range(n_clip)]
    near = configs.plain_scalar(n=4).with_(
        dims=dims, sources=[src], width=203, height=151, interpolation=1, step=1.3, clip=clip,
        camera=configs.orbit_camera(dims, OBLIQUE, 0.7))
    along = near.with_(width=640, height=640, step=0.2, camera=configs.orbit_camera(dims, ALONG_X, 0.7))
    got = []
    with Context(device=0) as ctx:
        for c in range(16):
            ctx.set_tile_shape(c, 32 // lanes, 1, 1, lanes, 0, 0)
        keep = device.upload_volume(ctx, near, 0)
        for beside in (False, True):
            img, cnt = device.new_image(near), device.new_counts(near)
            jobs = [device.render_job(near, 0, img, cnt)]
            if beside:
                side = device.new_image(along)
                jobs.append(device.render_job(along, 0, side))
            ctx.render(jobs, DIRECT)
            got.append((img.cpu().numpy(), cnt.cpu().numpy()))
        del keep
    assert (got[0][1] > 0).mean() > 0.05
    assert np.array_equal(got[1][0], got[0][0]) and np.array_equal(got[1][1], got[0][1])
    compare(got[0][0].reshape(-1, 4), got[0][1].reshape(-1), oracle.render(near, threads=8),
            label=f"corners {lanes} {guard} {dims} {n_clip}")
