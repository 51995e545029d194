"""Jobs on a frozen volume of three sources, on the CPU (no device code runs): without
guard layers every job reads the frozen values, whatever sources it uses and in iso
mode; with them the (y, z) pairs serve the jobs over all three."""

import re

import pytest

from cpu_library import cpu, cpu_lib  # noqa: F401
from test_derived_buffer_cpu import job


def kernel(log):
    return [m.group(1) for m in [re.search(r"raycast_kernelILb[01]ELi\d+ELi\dELi(n?\d+)E", line) for line in log()] if m]


# signatures (csrc/isaac_internal.h): 5 and 6 three derived values x fastest and in pairs, 1 one FP32 scalar, 0 any sources
@pytest.mark.parametrize("guard,all3,two,one,iso", [(0, "5", "0", "1", "n2"), (1, "6", "0", "0", "n2")])
def test_loops_on_a_frozen_volume(cpu, guard, all3, two, one, iso):
    from paper_1611_09048_amd import binding
    ctx, log = cpu
    dims = (24, 23, 21)
    ext = [n + 2 * guard for n in dims]
    ctx.set_sources(0, dims, [binding.source_desc(
        name=f"s{k}", f_dim=2, dtype="f16", comp=[(k + 1) << 20, ((k + 1) << 20) + 2], guard=guard, chain="length",
        stride=(4, 4 * ext[0], 4 * ext[0] * ext[1])) for k in range(3)])
    ctx.freeze_volume(0)
    log()
    for want, kw in ((all3, {}), (two, dict(enabled=[1, 0, 1])), (one, dict(enabled=[0, 1, 0])),
                     (iso, dict(mode=binding.ISO, iso_values=[0.5] * 3))):
        ctx.render([job(binding, dims, interpolation=1, **kw)])
        assert kernel(log) == [want], kw
