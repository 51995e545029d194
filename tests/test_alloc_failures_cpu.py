"""Device allocations that fail, on the CPU (no device code runs): a call that can do
without the memory goes on, one that cannot says so, and the next call is not failed
by the error the runtime kept."""

import pytest

from cpu_library import cpu, cpu_lib  # noqa: F401
from test_derived_buffer_cpu import define, job


def test_render_without_derived_volume_or_ray_buffer(cpu):
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    dims = define(ctx, 3, 1)
    ctx.lib.fake_fail_malloc_from(0)
    for j in (job(binding, dims, interpolation=1), job(binding, dims, interpolation=0)):
        ctx.render([j], binding.DERIVE)                # neither: sources in place, rays set up by the ray kernel
        lines = log()
        assert not any("derive_kernel" in line for line in lines) and any("raycast_kernel" in line for line in lines)
    for cls in range(16):
        ctx.set_tile_shape(cls, 4, 1, 1, 4, 0, 1)
    ctx.render([job(binding, dims, interpolation=1)], binding.DIRECT)
    assert any("raycast_kernel" in line for line in log())          # not pooled: tiles
    ctx.lib.fake_fail_malloc_from(-1)
    ctx.render([job(binding, dims, interpolation=1)], binding.DERIVE)
    assert any("derive_kernel" in line for line in log())


def test_refusals_leave_the_context_usable(cpu):
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    dims = define(ctx, 1, 1)
    ctx.lib.fake_fail_malloc_from(1 << 16)
    big = binding.source_desc(name="s", f_dim=1, dtype="f32", comp=[1 << 20], stride=(4, 4 * 64, 4 * 64 * 64), guard=0,
                              persistent=False)
    with pytest.raises(binding.IsaacError) as e:       # no memory for the copy of a non-persistent source
        ctx.set_sources(1, (64, 64, 64), [big])
    assert e.value.code == -4
    ctx.render([job(binding, dims)])
    with pytest.raises(binding.IsaacError) as e:       # none for the serving images
        ctx.submit(job(binding, dims))
    assert e.value.code == -4
    ctx.render([job(binding, dims)])
