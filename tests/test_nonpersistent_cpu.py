"""When a non-persistent field is copied before the render, on the CPU (no device code
runs): wherever something can reuse its memory before the render has read it, which is
any update() still to come in the call, of whatever volume, and the caller once an
asynchronous or served call has returned."""

import pytest

from cpu_library import cpu, cpu_lib  # noqa: F401

DIMS = (16, 12, 10)


def define(ctx, vid, loose, updates, soa=False):
    """Three sources; `loose` are not persistent, `updates` have an update()."""
    from paper_1611_09048_amd import binding
    c = 3
    st = (4, 64, 1024) if soa else (4 * c, 4 * c * 16, 4 * c * 16 * 12)
    comp = [[((k + 1) << 24) + (i << 20 if soa else 4 * i) for i in range(c)] for k in range(3)]
    ctx.set_sources(vid, DIMS, [binding.source_desc(
        name=f"s{k}", f_dim=c, dtype="f32", comp=comp[k], stride=st, guard=0, chain="length",
        persistent=k not in loose, update=(lambda user, enabled, p: None) if k in updates else None) for k in range(3)])


def job(vid, **kw):
    from paper_1611_09048_amd import binding
    c = [n / 2 for n in DIMS]
    return binding.render_desc(volume_id=vid, width=64, height=48, eye=(c[0] - 40, c[1], c[2]), center=c, up=(0, 0, 1),
                               out_rgba=1 << 30, interpolation=1, **kw)


def copies(log):
    lines = log()
    n = [i for i, line in enumerate(lines) if "strided_copy_kernel" in line]
    waited = [i for i in n if i + 1 < len(lines) and lines[i + 1] == "sync"]
    return len(n), len(waited)


@pytest.mark.parametrize("call", ["render", "noalloc"])
@pytest.mark.parametrize("loose,updates,want", [
    ((0,), (), 0), ((2,), (), 0), ((0, 1, 2), (), 0),
    ((0,), (0,), 0), ((2,), (2,), 0), ((2,), (0, 1, 2), 0),        # its own or earlier ones
    ((0,), (1,), 1), ((0,), (2,), 1), ((0, 1), (2,), 2),           # a later one
    ((0, 1, 2), (0, 1, 2), 2)])
def test_synchronous_calls(cpu, call, loose, updates, want):
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    define(ctx, 0, loose, updates)
    (ctx.render_noalloc if call == "noalloc" else ctx.render)([job(0)])
    assert copies(log) == (want, want)
    (ctx.render_noalloc if call == "noalloc" else ctx.render)([job(0)], binding.ASYNC)
    assert copies(log) == (len(loose), len(loose))


def test_updates_of_other_volumes_count(cpu):
    ctx, log = cpu
    define(ctx, 0, (0,), ())
    define(ctx, 1, (), (2,))
    define(ctx, 2, (1,), ())
    ctx.render([job(0), job(1), job(2)])                           # volume 1's update() comes between them
    assert copies(log) == (1, 1)
    ctx.render([job(1), job(0), job(2)])
    assert copies(log) == (0, 0)
    ctx.render([job(0), job(1, enabled=[1, 1, 0])])                # update() of a disabled source runs too
    assert copies(log) == (1, 1)


def test_separate_components_are_packed_and_disabled_sources_left_alone(cpu):
    ctx, log = cpu
    define(ctx, 0, (0, 1), (), soa=True)
    ctx.render([job(0)])
    assert copies(log) == (2, 0)                                   # nothing can reuse them: no wait
    ctx.render([job(0, enabled=[0, 1, 1])])
    assert copies(log) == (1, 0)


def test_served_calls_copy(cpu):
    ctx, log = cpu
    define(ctx, 0, (0, 2), ())
    assert ctx.submit(job(0)) is not None
    assert copies(log) == (2, 2)
