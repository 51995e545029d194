"""How many lanes evaluate a ray of the one-lane schedule, on the CPU (no device code
runs): one where rays are many and short, by their path or by the opacity of their
tables, a group of 4 or 16 where they are few or long."""

import re

import pytest

from cpu_library import cpu, cpu_lib  # noqa: F401

OPAQUE, HALF, THIN = 1.0, 0.5, 0.02


def volume(ctx, vid, n, alpha):
    from paper_1611_09048_amd import binding
    st = (4, 4 * n, 4 * n * n)
    ctx.set_sources(vid, (n, n, n), [binding.source_desc(name="s", f_dim=1, dtype="f32", comp=[1 << 20], stride=st,
                                                        guard=0)])
    ctx.set_transfer(vid, 0, [(0.0, 1, 1, 1, alpha), (1.0, 1, 1, 1, alpha)])


def view(vid, n, w, h, **kw):
    """The whole volume, two diagonals away: about 8 % of a frame's pixels lie in its rectangle."""
    from paper_1611_09048_amd import binding
    d, c = 2 * n * 3 ** 0.5, n / 2
    return binding.render_desc(volume_id=vid, width=w, height=h, eye=(c + d * 0.7, c + d * 0.57, c + d * 0.43),
                               center=(c, c, c), up=(0, 0, 1), out_rgba=1 << 30, interpolation=1, **kw)


def lanes(log):
    return [int(m.group(1)) for m in [re.search(r"raycast_kernelILb1ELi(\d+)E", line) for line in log()] if m]


@pytest.mark.parametrize("n,w,h,alpha,ert,want", [
    (64, 256, 256, THIN, 0, 16), (160, 1024, 768, THIN, 0, 16), (160, 3840, 2160, THIN, 0, 4),
    (64, 1920, 1080, HALF, 0, 4), (64, 1920, 1080, OPAQUE, 0, 1), (64, 3840, 2160, HALF, 0, 1),
    (160, 3840, 2160, OPAQUE, 0, 1), (160, 512, 512, OPAQUE, 0, 1), (16, 3840, 2160, THIN, 0, 1),
    (16, 512, 512, THIN, 0, 16), (160, 3840, 2160, OPAQUE, 2.0, 4), (160, 1024, 768, OPAQUE, 2.0, 16),
    (160, 1920, 1080, THIN, 0.01, 1)])
def test_lanes_follow_rays_and_points(cpu, n, w, h, alpha, ert, want):
    ctx, log = cpu
    volume(ctx, 0, n, alpha)
    log()
    ctx.render([view(0, n, w, h, ert_threshold=ert)])
    assert lanes(log) == [want]


@pytest.mark.parametrize("factor,step,w,want", [
    (1.0, 0.5, 400, 16), (0.4, 0.5, 700, 1), (1.0, 4.0, 700, 1), (0.4, 0.5, 190, 16), (0.4, 4.0, 240, 4)])
def test_close_views_and_long_steps(cpu, factor, step, w, want):
    """Where the rays are closer together than their points, and fill the chip, one lane reads fewer lines."""
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    n = 64
    volume(ctx, 0, n, THIN)
    log()
    d, c = factor * n * 3 ** 0.5, n / 2
    ctx.render([binding.render_desc(volume_id=0, width=w, height=w, eye=(c + d * 0.7, c + d * 0.57, c + d * 0.43),
                                    center=(c, c, c), up=(0, 0, 1), out_rgba=1 << 30, interpolation=1, step=step)])
    assert lanes(log) == [want]


def test_a_batch_is_one_launch_and_an_empty_rectangle_counts_nothing(cpu):
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    volume(ctx, 0, 64, OPAQUE)
    volume(ctx, 1, 160, THIN)
    away = binding.render_desc(volume_id=0, width=640, height=480, eye=(300, 32, 32), center=(600, 32, 32),
                               up=(0, 0, 1), out_rgba=1 << 30, interpolation=1)
    log()
    ctx.render([away])
    assert len(lanes(log)) <= 1
    ctx.render([view(0, 64, 1920, 1080), away])
    assert lanes(log) == [1]
    ctx.render([view(0, 64, 512, 512), view(1, 160, 512, 512)])
    assert lanes(log) == [16]
    volume(ctx, 2, 90, THIN)
    log()
    ctx.render([view(2, 90, 256, 256) for _ in range(26)])         # 180 thousand rays, 0.7 pixels a voxel
    assert lanes(log) == [16]


@pytest.mark.parametrize("n,w,h,shape,want", [
    (64, 256, 256, 1, 8), (64, 1920, 1080, 4, 8), (16, 3840, 2160, 1, 1), (32, 3840, 2160, 4, 1),
    (160, 3840, 2160, 1, 1), (16, 3840, 2160, 16, 8)])
def test_lanes_of_iso_jobs(cpu, n, w, h, shape, want):
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    for cls in range(16):
        ctx.set_tile_shape(cls, 64 // shape if shape > 8 else 8, 1, 1, shape)
    volume(ctx, 0, n, OPAQUE)
    log()
    ctx.render([view(0, n, w, h, mode=binding.ISO, iso_values=[0.5])])
    got = [int(m.group(1)) for m in [re.search(r"raycast_kernelILb0ELi(\d+)ELi\dELin[23]E", line) for line in log()] if m]
    assert got == [want]


def test_iso_batch_of_small_images(cpu):
    """Rays far apart (1.3 pixels a voxel): 8 lanes, however many they are."""
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    volume(ctx, 0, 48, OPAQUE)
    log()
    ctx.render([view(0, 48, 256, 256, mode=binding.ISO, iso_values=[0.5]) for _ in range(64)])
    got = [int(m.group(1)) for m in [re.search(r"raycast_kernelILb0ELi(\d+)ELi\dELin[23]E", line) for line in log()] if m]
    assert got == [8]


@pytest.mark.parametrize("guard,chain,want", [(1, "", "ELi0ELin3E"), (0, "", "ELi3ELin2E"), (1, "mul(2)", "ELi3ELin2E")])
def test_iso_kernel_of_the_sources(cpu, guard, chain, want):
    """Plain sources (FP32 scalars, guard layers, no chain) have a loop of 80 registers; the loop over any
    sources is bound to the registers of 3 waves per SIMD."""
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    n = 24
    ctx.set_sources(0, (n, n, n), [binding.source_desc(name="s", f_dim=1, dtype="f32", comp=[1 << 20], guard=guard,
                                                      stride=(4, 4 * (n + 2), 4 * (n + 2) ** 2), chain=chain)])
    log()
    ctx.render([view(0, n, 128, 96, mode=binding.ISO, iso_values=[0.5])], binding.DIRECT)
    assert [line for line in log() if "raycast_kernelILb0ELi8" + want in line]
