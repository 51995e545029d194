"""Which loop a tuned launch of a scalar with adjacent x neighbours runs, on the CPU (no
device code runs): corners in pairs, or one by one where four points of a ray next to
each other lie in rows of their own and the rays are close together."""

import re

import numpy as np
import pytest

from cpu_library import cpu, cpu_lib  # noqa: F401

SINGLE, PAIRS, PAIRS_CLAMP = 1, 7, 8
OBLIQUE, ALONG_X = (0.5, 0.6, 0.62), (1.0, 0.02, 0.03)


def define(ctx, vid, n, guard, alpha=0.02):
    from paper_1611_09048_amd import binding
    p = n + 2 * guard
    ctx.set_sources(vid, (n, n, n), [binding.source_desc(name="s", f_dim=1, dtype="f32", comp=[1 << 24],
                                                        stride=(4, 4 * p, 4 * p * p), guard=guard)])
    ctx.set_transfer(vid, 0, [(0.0, 1, 1, 1, alpha), (1.0, 1, 1, 1, alpha)])


def view(n, direction, diagonals, step, w=960, vid=0, **kw):
    from paper_1611_09048_amd import binding
    d = np.array(direction) / np.linalg.norm(direction)
    kw.setdefault("interpolation", 1)
    return binding.render_desc(volume_id=vid, width=w, height=w * 3 // 4, eye=tuple(n / 2 + diagonals * n * 3 ** 0.5 * d),
                               center=(n / 2,) * 3, up=(0, 0, 1), out_rgba=1 << 30, step=step, **kw)


def signatures(log):
    found = [re.search(r"raycast_kernelILb\dELi\d+ELi\d+ELi(n?\d+)E", line) for line in log()]
    return [int(m.group(1).replace("n", "-")) for m in found if m]


@pytest.mark.parametrize("lanes,guard,alpha,direction,diagonals,step,want", [
    (4, 1, 0.02, OBLIQUE, 0.6, 1.0, SINGLE), (4, 0, 0.02, OBLIQUE, 0.6, 1.0, SINGLE),
    (4, 1, 0.02, OBLIQUE, 0.6, 0.25, PAIRS), (4, 0, 0.02, OBLIQUE, 0.6, 0.25, PAIRS_CLAMP),
    (4, 1, 0.02, OBLIQUE, 0.6, 0.6, PAIRS), (4, 0, 0.02, OBLIQUE, 0.6, 0.6, SINGLE),
    (4, 1, 0.02, ALONG_X, 0.6, 1.0, PAIRS), (4, 1, 0.02, OBLIQUE, 4.0, 1.0, PAIRS),
    (8, 1, 0.02, OBLIQUE, 0.6, 1.0, PAIRS), (8, 0, 0.5, OBLIQUE, 0.6, 1.0, SINGLE),
    (8, 0, 0.5, OBLIQUE, 0.6, 0.25, PAIRS_CLAMP), (2, 1, 0.5, OBLIQUE, 0.6, 1.0, PAIRS),
    (16, 0, 0.5, OBLIQUE, 0.6, 1.0, PAIRS_CLAMP), (64, 1, 0.5, OBLIQUE, 0.6, 1.0, PAIRS)])
def test_loads_follow_the_view(cpu, lanes, guard, alpha, direction, diagonals, step, want):
    ctx, log = cpu
    for c in range(16):
        ctx.set_tile_shape(c, 64 // lanes // 2 if lanes < 32 else 1, 1, 1, lanes, 0, 0)
    define(ctx, 0, 64, guard, alpha)
    log()
    ctx.render([view(64, direction, diagonals, step)])
    assert signatures(log) == [want]


def test_untuned_nearest_and_iso_calls_keep_their_loops(cpu):
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    define(ctx, 0, 64, 1)
    log()
    ctx.render([view(64, OBLIQUE, 0.6, 1.0)])
    assert signatures(log) == [PAIRS]
    for c in range(16):
        ctx.set_tile_shape(c, 8, 1, 1, 4, 0, 0)
    ctx.render([view(64, OBLIQUE, 0.6, 1.0, interpolation=0)])
    assert signatures(log) == [PAIRS]
    ctx.render([view(64, OBLIQUE, 0.6, 1.0, mode=binding.ISO, iso_values=[0.5])])
    assert SINGLE not in signatures(log)


def test_a_batch_chooses_by_the_rays_of_its_jobs(cpu):
    ctx, log = cpu
    for c in range(16):
        ctx.set_tile_shape(c, 8, 1, 1, 4, 0, 0)
    define(ctx, 0, 64, 1)
    near, far = view(64, OBLIQUE, 0.6, 1.0, w=320), view(64, ALONG_X, 0.6, 0.25, w=960)
    for jobs, want in (([near] * 3, SINGLE), ([near, far], PAIRS), ([far, near], PAIRS)):
        log()
        ctx.render(jobs)
        assert set(signatures(log)) <= {want}
