"""The autotuner's choice, on the host code of the solver built against a runtime that records its calls
(fake_device.cpp) and gives each kernel the time that the test wants."""
import ctypes as C
import os
import subprocess

import pytest

from workloads import gen

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LANE = 5


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake") / "libsolver_host.so")
    csrc = os.path.join(ROOT, "paper_2501_01747_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-D__align__(n)=",
                    "-DHIP_SYMBOL(s)=s", "-w", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"), "-I" + csrc, "-x", "c++",
                    os.path.join(csrc, "adg_api.hip"), os.path.join(ROOT, "tests", "fake_device.cpp"), "-o", out], check=True)
    lib = C.CDLL(out)
    lib.fake_calls.restype = C.c_char_p
    return lib


def tune(lib, untuned, ms, steps=0):
    """The choice and the calls of a tuning whose untuned kernel is `untuned`; ms: the times of the kernels 0..5."""
    from paper_2501_01747_amd import adg   # (not with the module: a test run on a GPU loads torch's runtime first)

    case, _ = gen.case_c1(E=16, n_pe=2, Lx=0.01 * 16 / 2048)
    p, h, mem = adg.Problem(case), C.c_void_p(), C.create_string_buffer(4096)
    base = (C.addressof(mem) + 255) & ~255
    assert lib.adg_create(C.byref(p.phys), C.byref(p.disc), C.byref(p.asyn), C.c_void_p(base), C.c_size_t(2048),
                          C.c_void_p(7), C.byref(h)) == 0
    lib.fake_kernels(untuned, (C.c_double * 6)(*ms))
    assert lib.adg_step(h, steps) == 0
    lib.fake_fail(b"", -1)
    c = C.c_int32()
    assert lib.adg_autotune(h, 4, C.byref(c)) == 0
    calls = lib.fake_calls().decode().split()
    lib.adg_destroy(h)
    return c.value, calls


# kernels (8,512) (8,256) (4,256) (4,512) (8,1024) and a lane per point
@pytest.mark.parametrize("untuned,ms,choice", [
    (3, [9.3, 11.0, 10.0, 9.1, 9.5, 18.0], 3),    # within 3 % of 8/512, and the untuned kernel: kept
    (0, [9.3, 11.0, 10.0, 9.1, 9.5, 18.0], 0),
    (3, [9.3, 11.0, 10.0, 9.4, 9.2, 18.0], 3),    # the fastest is not 3 % faster than the untuned one
    (3, [8.0, 11.0, 10.0, 9.4, 9.2, 18.0], 0),
    (LANE, [31.0, 99.0, 30.0, 32.0, 33.0, 30.5], 1),
    (LANE, [31.0, 99.0, 25.0, 32.0, 33.0, 30.5], 2),
])
def test_the_untuned_kernel_stays_unless_another_is_faster(lib, untuned, ms, choice):
    assert tune(lib, untuned, ms)[0] == choice


@pytest.mark.parametrize("steps", [0, 1])
def test_candidates_are_timed_as_steps_run_them(lib, steps):
    """With carried AT values, also before the first step: all but one launch that forms them."""
    _, calls = tune(lib, 0, [9.0] * 6, steps)
    timed = [c for c in calls if c.startswith(("carried", "gathered"))]
    assert len(timed) == 5 * (2 + 3 * 4) + (1 - steps)
    assert [c for c in timed if c.startswith("gathered")] == ([] if steps else ["gathered:0"])


def test_pinned_words_of_the_error_flags(lib):
    """One pinned block for all solvers of the process: none for the first read, then a word each from a
    solver's next read on, handed on after adg_destroy, and the flag copied where none is left."""
    from paper_2501_01747_amd import adg

    case, w0 = gen.case_c1(E=16, n_pe=2, Lx=0.01 * 16 / 2048)
    p, mem = adg.Problem(case), C.create_string_buffer(4096)
    base = (C.addressof(mem) + 255) & ~255
    w = (C.c_double * w0.size)()

    def solver():
        h = C.c_void_p()
        assert lib.adg_create(C.byref(p.phys), C.byref(p.disc), C.byref(p.asyn), C.c_void_p(base), C.c_size_t(2048),
                              C.c_void_p(7), C.byref(h)) == 0
        return h

    def read(h):
        assert lib.adg_get_state(h, w, C.c_int64(w0.size), 1) == 0
        return [c for c in lib.fake_calls().decode().split() if c.startswith("read")][-1]

    lib.fake_fail(b"", -1)
    many = [solver() for _ in range(70)]
    words = [read(h) for h in many]
    assert words[0] == "read:0" and len(set(words[1:65])) == 64 and set(words[65:]) == {"read:0"}
    assert [read(h) for h in many[1:65]] == words[1:65]
    lib.adg_destroy(many[5])
    assert read(many[0]) == words[5] and read(many[69]) == "read:0"
    assert lib.fake_calls().decode().split().count("pinned:0") == 1
    for h in many[:5] + many[6:]:
        lib.adg_destroy(h)
