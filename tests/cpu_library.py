"""The library's host code built without its device code, on a runtime that runs
nothing (tests/c/fake_hip.cpp): what a call allocates, waits for and launches, on the
CPU."""

import ctypes
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="session")
def cpu_lib(tmp_path_factory):
    from paper_1611_09048_amd import binding, build
    tmp = str(tmp_path_factory.mktemp("cpu_lib"))
    objs, undefined = [], set()
    for src in [os.path.join(build.CSRC, s) for s in build.SOURCES] + [os.path.join(ROOT, "tests", "c", "fake_hip.cpp")]:
        objs.append(os.path.join(tmp, os.path.basename(src) + ".o"))
        subprocess.run([build.hipcc(), f"--offload-arch={build.ARCH}", "--offload-host-only", "-O1", "-std=c++17",
                        "-fPIC", "-Wno-unused-value", "-I", os.path.join(ROOT, "include"), "-c", src, "-o", objs[-1]],
                       check=True, capture_output=True)
        out = subprocess.run(["nm", objs[-1]], check=True, capture_output=True, text=True).stdout
        undefined |= set(re.findall(r" U (__hip_fatbin\w*)", out))
    stub = os.path.join(tmp, "fatbin.c")                # no device code: the images' names stand for nothing
    with open(stub, "w") as f:
        f.write("".join(f"char {u}[8];\n" for u in sorted(undefined)))
    path = os.path.join(tmp, "libisaac_cpu.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-x", "c", stub, "-x", "none", *objs, "-o", path,
                    "-pthread"], check=True, capture_output=True)
    lib = binding.load(path)
    lib.fake_log.restype = ctypes.c_char_p
    lib.fake_host_bytes.restype = ctypes.c_ulonglong
    lib.fake_fail_host_from.argtypes = lib.fake_fail_malloc_from.argtypes = [ctypes.c_longlong]
    lib.fake_fail_call.argtypes = [ctypes.c_char_p]
    lib.fake_graph_totals.argtypes = [ctypes.c_ulonglong] * 3
    return lib


@pytest.fixture
def cpu(cpu_lib, monkeypatch):
    """(Context on the CPU library, function returning and clearing its log as a list of lines)."""
    from paper_1611_09048_amd import binding
    monkeypatch.setattr(binding, "_lib", cpu_lib)
    ctx = binding.Context(device=0, stream=None)

    def log():
        lines = cpu_lib.fake_log().decode().splitlines()
        cpu_lib.fake_clear()
        return lines
    log()
    yield ctx, log
    cpu_lib.fake_fail_host_from(-1)
    cpu_lib.fake_fail_malloc_from(-1)
    cpu_lib.fake_fail_call(b"")
    cpu_lib.fake_graph_totals(0, 0, 0)
    cpu_lib.fake_pending(0)
    log()
    ctx.close()
    assert not [line for line in log() if line.startswith("bad")]
