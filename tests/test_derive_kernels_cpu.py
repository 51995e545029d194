"""Which derive pass a call launches, on the CPU (no device code runs): the one compiled
for a scalar and two vectors of one type, in either layout, the general one for the rest."""

import re

import pytest

from cpu_library import cpu, cpu_lib  # noqa: F401
from test_derived_buffer_cpu import job

DIMS = (24, 23, 21)


def define(ctx, kinds, guard=1):
    from paper_1611_09048_amd import binding
    ext = [n + 2 * guard for n in DIMS]
    src = []
    for k, (dtype, c) in enumerate(kinds):
        v = c * (4 if dtype == "f32" else 2)
        src.append(binding.source_desc(name=f"s{k}", f_dim=c, dtype=dtype, guard=guard, chain="length",
                                       comp=[((k + 1) << 20) + i * v // c for i in range(c)],
                                       stride=(v, v * ext[0], v * ext[0] * ext[1])))
    ctx.set_sources(0, DIMS, src)


@pytest.mark.parametrize("iso", [False, True])
@pytest.mark.parametrize("kinds,sig", [
    ([("f32", 1), ("f32", 3), ("f32", 3)], "2"), ([("f16", 1), ("f16", 3), ("f16", 3)], "3"),
    ([("bf16", 1), ("bf16", 3), ("bf16", 3)], "4"), ([("f32", 1), ("f16", 3), ("f32", 3)], "0"),
    ([("f32", 1), ("f32", 3)], "0"), ([("f32", 2)], "0"), ([("f32", 1)] + [("f32", 3)] * 3, "0")])
def test_derive_pass(cpu, kinds, sig, iso):
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    define(ctx, kinds)
    log()
    kw = dict(mode=binding.ISO, iso_values=[0.5] * len(kinds)) if iso else {}
    ctx.render([job(binding, DIMS, interpolation=1, **kw)], binding.DERIVE)
    got = [m.groups() for m in [re.search(r"derive_kernelILi(\d+)ELi(\d)ELi\dELb([01])E", line) for line in log()] if m]
    assert got == [(sig, str(len(kinds)), "1" if len(kinds) == 3 and not iso else "0")]
