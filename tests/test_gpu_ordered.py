"""One lane per ray, evaluated by groups of 4 or 16 lanes: the group size follows
the rays of a launch, so a job alone (16 lanes) and in a batch of its copies (4
lanes) must give the same image and counts, bit for bit, wherever a ray ends or
terminates inside a row, and both must agree with the oracle.
"""

import numpy as np
import pytest

import oracle
from parity import compare
from scenes import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ert", [0.999, 0.3, 1e-3, 1.0, 2.0])
@pytest.mark.parametrize("kind", ["near", "tri", "pic3", "pic3_direct", "pic3_f16_direct"])
def test_group_sizes_agree(kind, ert):
    from paper_1611_09048_amd import DERIVE, DIRECT, Context, device
    if kind in ("near", "tri"):
        sc = configs.plain_scalar(n=24, width=256, height=256).with_(interpolation=int(kind == "tri"))
    else:
        sc = configs.pic3(n=20, width=256, height=256, dtype="f16" if "f16" in kind else "f32", n_clip=1)
    sc = sc.with_(camera=configs.orbit_camera(sc.dims, (0.5, -0.7, 0.4), 0.75), step=0.37, ert_threshold=ert)
    flags = DIRECT if "direct" in kind else DERIVE if kind == "pic3" else 0
    with Context(device=0) as ctx:
        vol = device.upload_volume(ctx, sc, 0)
        n = 6                                             # 6 x 65,536 pixels: above the 4-lane line
        img = [device.new_image(sc) for _ in range(n + 1)]
        cnt = [device.new_counts(sc) for _ in range(n + 1)]
        jobs = [device.render_job(sc, 0, i, c) for i, c in zip(img, cnt)]
        ctx.render(jobs[:1], flags)
        ctx.render(jobs[1:], flags)
        ref, ref_n = img[0].cpu().numpy(), cnt[0].cpu().numpy()
        assert (ref_n > 0).mean() > 0.5
        for i, c in zip(img[1:], cnt[1:]):
            assert np.array_equal(i.cpu().numpy(), ref) and np.array_equal(c.cpu().numpy(), ref_n)
        del vol
    small = sc.with_(width=64, height=64)
    with Context(device=0) as ctx:
        a, b = device.render_scene(ctx, small, flags=flags)
    compare(a.reshape(-1, 4), b.reshape(-1), oracle.render(small, threads=8), label=f"ordered {kind} {ert}")
