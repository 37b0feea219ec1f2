"""Steps that the caller captures into a HIP graph of its own and replays, with eager steps, a new state and
reads between the replays: bit for bit what eager steps give, for even and odd numbers of steps."""
import numpy as np
import pytest

from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def adg():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2501_01747_amd import adg as lib

    return lib


def capture(obj, n):
    import torch

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=obj.stream):
        obj.step(n)
    return g


def problem(kind):
    if kind == "detailed" or kind == "detailed lserk4":
        case, w0 = gen.case_c1(E=70, order_p=2, n_pe=6, cfl=0.08, Lx=0.01 * 70 / 2048)
    elif kind == "limited":
        case, w0 = gen.case_shock(160, 2, n_pe=5)
    else:
        case, w0 = gen.case_c0(E=130, n_pe=8, pmf=(0.3, 0.4, 0.3), mode="sync" if kind == "sync" else "saa")
    if kind in ("rk2", "lserk4", "detailed lserk4"):
        case["disc"]["rk"] = kind.split()[-1]
    return case, w0


@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("kind", ["sync", "saa", "rk2", "lserk4", "limited", "detailed", "detailed lserk4"])
def test_solver_steps_in_a_graph(adg, kind, n):
    import torch

    case, w0 = problem(kind)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s, ref = adg.Solver(case), adg.Solver(case)
        s.set_state(w0)
        ref.set_state(w0)
        s.step(5)   # an odd alignment, with carried AT values
        ref.step(5)
        g = capture(s, n)
        done = 5
        for eager in (0, 2, 1, 0):
            g.replay()
            s.step(eager)
            ref.step(n + eager)
            done += n + eager
            assert s.step_count() == ref.step_count() == done
            np.testing.assert_array_equal(s.state(), ref.state())
        s.set_state(w0)   # replays from a new state need its alignment to be the captured one
        s.step(5)
        ref.set_state(w0)
        ref.step(5 + 2 * n)
        g.replay()
        g.replay()
        np.testing.assert_array_equal(s.state(), ref.state())
        s.close()
        ref.close()


def test_captured_steps_that_have_not_run(adg):
    """A capture alone changes nothing: the next eager step reads no values that its launches would carry."""
    import torch

    case, w0 = gen.case_c1(E=8200, order_p=1, n_pe=300, cfl=0.1, Lx=0.01 * 8200 / 2048)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s, ref = adg.Solver(case), adg.Solver(case)
        for x in (s, ref):
            x.set_state(w0)
            x.step(6)   # by the lane-per-point kernel, which carries nothing
            x.set_kernel_config(0)
        g = capture(s, 2)
        s.step(3)
        ref.step(3)
        np.testing.assert_array_equal(s.state(), ref.state())
        del g
        s.close()
        ref.close()


@pytest.mark.parametrize("n", [1, 2, 3])
def test_batch_steps_in_a_graph(adg, n):
    import torch

    cases = [gen.case_c0(E=90, n_pe=5, pmf=(0.3, 0.4, 0.3)), gen.case_shock(160, 2, n_pe=5),
             gen.case_c1(E=40, order_p=2, n_pe=4, cfl=0.08, Lx=0.01 * 40 / 2048), gen.case_c0(E=64, order_p=3, n_pe=3, cfl=0.04)]
    targets = [0, 0, 0, 7]
    heap = sum(adg.Batch.instance_bytes(c) for c, _ in cases)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        b, ref = (adg.Batch(4, 400, heap) for _ in range(2))
        slots = [[x.add(c, w, t) for (c, w), t in zip(cases, targets)] for x in (b, ref)]
        b.step(3)
        ref.step(3)
        b.set_group_streams(2)   # after a step, and before the capture: nothing is left to prepare
        g = capture(b, n)
        for eager in (0, 1, 2, 0):
            g.replay()
            b.step(eager)
            ref.step(n + eager)
            np.testing.assert_array_equal(b.poll()[0][slots[0]], ref.poll()[0][slots[1]])
            for x, y in zip(*slots):
                np.testing.assert_array_equal(b.state(x), ref.state(y))
        b.close()
        ref.close()


def test_steps_in_a_graph_of_a_solver_and_a_batch_that_have_their_own(adg):
    """Four steps captured where the library would replay its own graphs of two."""
    import torch

    c0, w0 = gen.case_c0(E=130, n_pe=8, pmf=(0.3, 0.4, 0.3))
    c1, w1 = gen.case_c1(E=40, order_p=2, n_pe=4, cfl=0.08, Lx=0.01 * 40 / 2048)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s, ref = adg.Solver(c0), adg.Solver(c0)
        b, bref = (adg.Batch(1, 40, adg.Batch.instance_bytes(c1)) for _ in range(2))
        for x in (s, ref):
            x.set_state(w0)
        for x in (b, bref):
            x.add(c1, w1)
        for x, r in ((s, ref), (b, bref)):
            x.set_graph(2)
            x.step(4)
            g = capture(x, 4)
            g.replay()
            x.step(3)
            g.replay()
            r.step(15)
        np.testing.assert_array_equal(s.state(), ref.state())
        np.testing.assert_array_equal(b.state(0), bref.state(0))
        assert s.step_count() == 15 and b.poll()[0][0] == 15
        for x in (s, ref, b, bref):
            x.close()
