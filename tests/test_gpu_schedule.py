"""One lane per ray, evaluated by one lane or by groups of 4 or 16: the choice follows
the rays and points of a launch, so the same job alone, beside a large transparent
view and beside a large opaque one runs in all three ways, and must give the same
image and counts, bit for bit."""

import dataclasses

import numpy as np
import pytest

import oracle
from parity import compare
from scenes import configs

pytestmark = pytest.mark.gpu

FLAT = {a: [(0.0, 0.9, 0.6, 0.3, a), (1.0, 0.2, 0.5, 0.8, a)] for a in (1e-4, 1.0)}


def with_tables(sc, alpha):
    return sc.with_(sources=[dataclasses.replace(s, tf=FLAT[alpha]) for s in sc.sources])


@pytest.mark.parametrize("ert", [0.999, 0.05, 2.0])
@pytest.mark.parametrize("kind", ["near", "tri", "pic3", "pic3_direct", "pic3_f16_direct", "mixed"])
def test_one_four_and_sixteen_lanes_agree(kind, ert):
    from paper_1611_09048_amd import DERIVE, DIRECT, Context, device
    pic3 = configs.pic3(n=20, width=256, height=256, dtype="f16" if "f16" in kind else "f32", n_clip=1)
    scalar = configs.plain_scalar(n=24, width=256, height=256).with_(interpolation=int(kind != "near"))
    place = dict(step=0.37, ert_threshold=ert)

    def near(s, **kw):
        return s.with_(camera=configs.orbit_camera(s.dims, (0.5, -0.7, 0.4), 0.75), **place, **kw)
    sc = near(scalar if kind in ("near", "tri", "mixed") else pic3)
    other = pic3 if kind == "mixed" else sc
    flags = DIRECT if "direct" in kind else DERIVE if kind == "pic3" else 0
    thin, opaque = (near(with_tables(other, a), width=800, height=800) for a in (1e-4, 1.0))
    with Context(device=0) as ctx:
        keep = [device.upload_volume(ctx, s, k) for k, s in enumerate((sc, thin, opaque))]
        got = []
        for beside in (None, (thin, 1), (opaque, 2)):
            img, cnt = device.new_image(sc), device.new_counts(sc)
            jobs = [device.render_job(sc, 0, img, cnt)]
            if beside:
                side = device.new_image(beside[0])
                jobs.append(device.render_job(beside[0], beside[1], side))
            ctx.render(jobs, flags)
            got.append((img.cpu().numpy(), cnt.cpu().numpy()))
        del keep
    assert np.isfinite(got[0][0]).all() and (got[0][1] > 0).mean() > 0.5
    for img, cnt in got[1:]:
        assert np.array_equal(img, got[0][0]) and np.array_equal(cnt, got[0][1])


@pytest.mark.parametrize("size", [(203, 151), (65, 40)])
@pytest.mark.parametrize("content", ["blob", "pic3"])
def test_opaque_view_agrees_with_the_oracle(content, size):
    """One lane per ray on its own: every ray ends at its first points."""
    from paper_1611_09048_amd import Context, device
    sc = configs.pic3(n=16) if content == "pic3" else configs.plain_scalar(n=16).with_(interpolation=1)
    sc = with_tables(sc, 1.0).with_(width=size[0], height=size[1], step=0.41,
                                    camera=configs.orbit_camera(sc.dims, (0.5, -0.7, 0.4), 0.75))
    with Context(device=0) as ctx:
        img, cnt = device.render_scene(ctx, sc)
    compare(img.reshape(-1, 4), cnt.reshape(-1), oracle.render(sc, threads=8), label=f"opaque {content} {size}")


@pytest.mark.parametrize("interpolation", [0, 1])
@pytest.mark.parametrize("kind", ["f32", "f16", "scalar"])
def test_iso_by_one_and_eight_lanes_agree(kind, interpolation):
    """Alone (8 lanes) and beside a large view (1 lane)."""
    from paper_1611_09048_amd import Context, device
    sc = configs.plain_scalar(n=20) if kind == "scalar" else configs.pic3(n=20, dtype=kind, n_clip=1)
    iso = [0.3] if kind == "scalar" else [1.0, 0.2, 0.15]
    sc = sc.with_(width=200, height=160, interpolation=interpolation, mode="iso",
                  camera=configs.orbit_camera(sc.dims, (0.5, -0.7, 0.4), 0.75),
                  sources=[dataclasses.replace(s, iso=v) for s, v in zip(sc.sources, iso)])
    large = sc.with_(width=1200, height=1200)
    with Context(device=0) as ctx:
        keep = device.upload_volume(ctx, sc, 0)
        got = []
        for beside in (False, True):
            img, cnt = device.new_image(sc), device.new_counts(sc)
            jobs = [device.render_job(sc, 0, img, cnt)]
            if beside:
                side = device.new_image(large)
                jobs.append(device.render_job(large, 0, side))
            ctx.render(jobs)
            got.append((img.cpu().numpy(), cnt.cpu().numpy()))
        del keep
    assert (got[0][0][..., 3] > 0).mean() > 0.1
    assert np.array_equal(got[1][0], got[0][0]) and np.array_equal(got[1][1], got[0][1])
