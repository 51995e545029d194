"""The derive pass for any 1 to 4 sources: one kernel per source count and widest
feature dimension, with the storage type and layout read at run time.  A derived
render equals the direct one bit for bit at every variant, on extents that leave
remainders of the 4-slice slabs, the 256-thread blocks and the stored (y, z)
pairs, and on a volume with more slabs than one grid axis holds.
"""

import numpy as np
import pytest

from scenes import configs, fields, make_source
from scenes.layout import Camera, Scene

pytestmark = pytest.mark.gpu

CHAINS = {1: "mul(0.7) | add(0.05)", 2: "add(0.1) | sum", 3: "length", 4: "mul(1.5,1,1,0.5) | length | pow(0.5)"}


def both(sc):
    from paper_1611_09048_amd import DERIVE, DIRECT, Context, device
    with Context(device=0) as ctx:
        return device.render_scene(ctx, sc, flags=DIRECT), device.render_scene(ctx, sc, flags=DERIVE)


@pytest.mark.parametrize("dims", [(1, 1, 1), (5, 2, 3), (33, 18, 21), (64, 31, 34)])
@pytest.mark.parametrize("f_dims", [(1,), (2,), (4,), (1, 1), (3, 2), (1, 4), (1, 1, 1), (3, 1, 3), (1, 3, 4),
                                    (1, 1, 1, 1), (1, 2, 3, 3), (1, 2, 3, 4)])
@pytest.mark.parametrize("guard", [0, 1])
def test_general_derive_equals_direct(dims, f_dims, guard):
    rng = np.random.default_rng(100 * len(f_dims) + sum(f_dims) + dims[0])
    srcs = []
    for k, f in enumerate(f_dims):
        vals = fields.uniform_random(rng, dims, guard, f, 0.0, 0.8)
        srcs.append(make_source(f"s{k}", vals, dtype=("f32", "f16", "bf16")[(k + f) % 3], guard=guard, chain=CHAINS[f],
                                weight=0.3 + 0.1 * k, tf=configs.random_tf(rng, 5, 0.4),
                                layout=("aos", "soa")[(k + len(f_dims)) % 2],
                                order=((0, 1, 2), (2, 0, 1))[k % 2], flip=(False, k % 2 == 1, False)))
    sc = Scene(dims=dims, sources=srcs, camera=configs.orbit_camera(dims, (0.7, -0.4, 0.5), 1.2), width=61, height=47,
               step=0.5, interpolation=1, clip=[configs.random_clip_plane(rng, dims)] if sum(dims) % 2 else [])
    (img, cnt), (img2, cnt2) = both(sc)
    assert np.isfinite(img).all() and cnt.max() > 0
    assert np.array_equal(img, img2) and np.array_equal(cnt, cnt2)


def test_more_slabs_than_one_grid_axis():
    dims = (1, 1, 131072 + 37)
    rng = np.random.default_rng(3)
    src = make_source("s", fields.uniform_random(rng, dims, 1, 1, 0.0, 1.0), guard=1, chain="mul(0.9)",
                      tf=configs.random_tf(rng, 5, 0.5), pitch_align=4)
    cam = Camera(eye=(-9.0, 0.5, dims[2] - 20.0), center=(0.5, 0.5, dims[2] - 20.0), up=(0.0, 1.0, 0.0),
                 projection="orthographic", ortho_height=2.0)
    sc = Scene(dims=dims, sources=[src], camera=cam, width=640, height=16, step=0.25, interpolation=1)
    (img, cnt), (img2, cnt2) = both(sc)
    assert cnt.max() > 0 and img[..., 3].max() > 0
    assert np.array_equal(img, img2) and np.array_equal(cnt, cnt2)
