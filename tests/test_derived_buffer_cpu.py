"""The derived volume's buffer is kept from call to call while it is large enough, on
the CPU (no device code runs): calls of different kinds on one volume derive volumes
of different sizes (a guard layer for trilinear jobs, (y, z) pairs for three sources),
and a program that alternates them must not allocate, free or wait on each."""

import pytest

from cpu_library import cpu, cpu_lib  # noqa: F401


def define(ctx, n_src, guard):
    from paper_1611_09048_amd import binding
    dims, ext = (24, 23, 21), [n + 2 * guard for n in (24, 23, 21)]
    st = (4, 4 * ext[0], 4 * ext[0] * ext[1])
    src = [binding.source_desc(name=f"s{k}", f_dim=1, dtype="f32", comp=[(k + 1) << 20], stride=st, guard=guard,
                               chain="mul(0.5)") for k in range(n_src)]
    ctx.set_sources(0, dims, src)
    return dims


def job(binding, dims, **kw):
    c = [n / 2 for n in dims]
    return binding.render_desc(volume_id=0, width=64, height=48, eye=(c[0] - 60, c[1] + 5, c[2] + 4), center=c,
                               up=(0, 0, 1), out_rgba=1 << 30, **kw)


@pytest.mark.parametrize("guard", [0, 1])
@pytest.mark.parametrize("n_src", [1, 2, 3, 4])
def test_alternating_calls_keep_the_buffer(cpu, n_src, guard):
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    dims = define(ctx, n_src, guard)
    calls = [job(binding, dims, interpolation=1), job(binding, dims, interpolation=0),
             job(binding, dims, interpolation=1, mode=binding.ISO, iso_values=[0.5] * n_src),
             job(binding, dims, interpolation=1, enabled=[1] + [0] * (n_src - 1))]
    for j in calls:
        ctx.render([j], binding.DERIVE | binding.ASYNC)
    assert any("derive_kernel" in line for line in log())
    for _ in range(3):
        for j in calls:
            ctx.render([j], binding.DERIVE | binding.ASYNC)
            lines = log()
            assert any("derive_kernel" in line for line in lines)
            assert not [line for line in lines if line.split()[0] in ("malloc", "free", "sync")], lines
