"""isaac_destroy gives back everything once, on the CPU (no device code runs), also with
requests not released and calls not known to be complete."""

from cpu_library import cpu, cpu_lib  # noqa: F401
from test_derived_buffer_cpu import define, job


def closed(ctx, log):
    log()
    ctx.close()
    return [line for line in log() if line.startswith("bad")]


def test_tickets_not_released(cpu):
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    dims = define(ctx, 2, 1)
    assert len(ctx.submit_batch([job(binding, dims) for _ in range(3)])) == 3
    assert closed(ctx, log) == []


def test_calls_that_allocate_nothing_still_pending(cpu):
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    dims = define(ctx, 1, 1)
    ctx.lib.fake_pending(1)
    for _ in range(3):
        ctx.render_noalloc([job(binding, dims)], binding.ASYNC)
        ctx.render([job(binding, dims)], binding.ASYNC)
    assert closed(ctx, log) == []
