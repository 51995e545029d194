"""Pinned host memory of the JPEG encoder, on the CPU (no device code runs): how much a
frame holds before and after its stream is known, and a frame whose buffer cannot be
had is encoded all the same."""

import ctypes

import pytest

from cpu_library import cpu, cpu_lib  # noqa: F401


def encode(ctx, w, h, coded, in_host, capacity=None):
    """One frame whose stream has `coded` bytes, the first `in_host` of them in the pinned buffer."""
    ctx.lib.fake_graph_totals(8 * coded, 0, in_host)
    out = ctypes.create_string_buffer(capacity or coded + 4096)
    size = ctypes.c_size_t(0)
    rc = ctx.lib.isaac_encode_jpeg(ctx.h, 1 << 20, w, h, 90, out, len(out), ctypes.byref(size))
    return rc, size.value


@pytest.mark.parametrize("w,h", [(8, 8), (1920, 1080), (8192, 4096), (16384, 8192)])
def test_pinned_bytes_follow_the_stream(cpu, w, h):
    ctx, log = cpu
    base = ctx.lib.fake_host_bytes()
    assert encode(ctx, w, h, 5000, 5000)[0] == 0
    first = ctx.lib.fake_host_bytes() - base
    assert first <= max(64 << 10, min(8 << 20, w * h)) + (32 << 10)      # and the tables
    big = min(4 << 20, 128 * w * h)                                           # passes the first buffer, or not
    assert encode(ctx, w, h, big, min(big, 60000))[0] == 0
    assert ctx.lib.fake_host_bytes() - base <= max(first, big * 5 // 4 + (32 << 10))
    held = ctx.lib.fake_host_bytes() - base - (32 << 10)
    log()
    assert encode(ctx, w, h, big + big // 8, min(held, big + big // 8))[0] == 0
    assert not [line for line in log() if "malloc" in line]


def test_a_buffer_that_cannot_be_had(cpu):
    ctx, log = cpu
    ctx.lib.fake_fail_host_from(64 << 10)
    for _ in range(2):
        rc, size = encode(ctx, 1920, 1080, 300000, 0)
        assert rc == 0 and size > 300000, ctx.lib.isaac_last_error(ctx.h)
    ctx.lib.fake_fail_host_from(1 << 20)                                      # the first buffer, but not a larger one
    for _ in range(2):
        rc, size = encode(ctx, 1280, 720, 2000000, 250000)
        assert rc == 0 and size > 2000000, ctx.lib.isaac_last_error(ctx.h)
