"""Host code of the batch when a launch or a capture fails: no work may be left on an extra stream that the
batch's stream does not wait for (a released region would be reused under it), and the batch's step parity stays
what its counters say.  The host code is built against a runtime that records its calls (fake_device.cpp)."""
import ctypes as C
import os
import subprocess

import pytest

from workloads import gen

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake") / "libbatch_host.so")
    csrc = os.path.join(ROOT, "paper_2501_01747_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-w", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + csrc, "-x", "c++", os.path.join(csrc, "adg_batch.hip"),
                    os.path.join(ROOT, "tests", "fake_device.cpp"), "-o", out], check=True)
    lib = C.CDLL(out)
    lib.fake_calls.restype = C.c_char_p
    lib.adg_batch_header_bytes.restype = C.c_size_t
    return lib


class FakeBatch:
    """Three groups: one-step instances of three orders, one instance each."""

    def __init__(self, lib, graph_steps=0):
        from paper_2501_01747_amd import adg   # (not with the module: a test run on a GPU loads torch's runtime first)

        self.lib, self.h, self.mem = lib, C.c_void_p(), C.create_string_buffer(1 << 20)
        base = (C.addressof(self.mem) + 255) & ~255
        assert lib.adg_batch_create(4, C.c_int64(1000), 0, C.c_void_p(base), C.c_size_t(1 << 19), C.c_void_p(7), C.byref(self.h)) == 0
        self.w = (C.c_double * 10000)()
        for order in (1, 2, 3):
            case, w0 = gen.case_c0(E=60, order_p=order, n_pe=2)
            p, slot = adg.Problem(case), C.c_int32()
            assert lib.adg_batch_add(self.h, C.byref(p.phys), C.byref(p.disc), C.byref(p.asyn), self.w, C.c_int64(w0.size), 0,
                                     C.c_int64(0), C.byref(slot)) == 0
        lib.adg_batch_set_graph(self.h, graph_steps)

    def step(self, n=1):
        return self.lib.adg_batch_step(self.h, n)

    def parity(self):
        st = (C.c_int64 * 4)()
        assert self.lib.adg_batch_poll(self.h, st, None) == 0
        return st[0]   # the copied-back counter of slot 0 is its own index, 0 or 1

    def close(self):
        self.lib.adg_batch_destroy(self.h)


def unjoined(calls, main):
    """Streams with a launch that no later event of theirs makes the main stream wait for."""
    busy, recorded = set(), set()
    for name, arg in (c.split(":") for c in calls.split()):
        if name in ("onestep", "detailed") and arg != main:
            busy.add(arg)
            recorded.discard(arg)
        elif name == "record":
            recorded.add(arg)
        elif name == "wait" and arg == main:
            busy -= recorded
        elif name == "sync":
            busy.discard(arg)
    return busy


@pytest.mark.parametrize("at", range(6))
def test_a_failed_launch_leaves_no_stream_behind(lib, at):
    b = FakeBatch(lib)
    assert b.step() == 0
    lib.fake_fail(b"onestep", at)
    assert b.step(2) != 0
    calls = lib.fake_calls().decode()
    assert "onestep" in calls and not unjoined(calls, "7"), calls
    lib.fake_fail(b"", -1)
    b.close()


@pytest.mark.parametrize("name,at", [("begin", 0), ("begin", 1), ("onestep", 4), ("end", 1), ("instantiate", 1)])
def test_a_failed_capture_keeps_the_parity(lib, name, at):
    b = FakeBatch(lib, graph_steps=3)
    lib.fake_fail(b"", -1)
    assert b.parity() == 0
    lib.fake_fail(name.encode(), at)
    assert b.step(3) != 0
    lib.fake_fail(b"", -1)
    assert b.parity() == 0
    assert b.step(3) == 0 and b.parity() == 1
    b.close()
