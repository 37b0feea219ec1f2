"""A state into the device layout (blocks of 64 elements) and back, byte for byte, at the edges of a block,
from host and device memory; and the reset that goes with a new state."""
import numpy as np
import pytest

from _parity import check
from test_gpu_ns import mechanism_of
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def adg():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2501_01747_amd import adg as lib

    return lib


def any_state(shape, seed):
    """Doubles of any bit pattern, NaN and infinities among them."""
    return np.random.default_rng(seed).integers(-2**63, 2**63 - 1, size=shape, dtype=np.int64).view(np.float64)


# (E, N_p, species): 5 and 8 variables, and 19 of the largest mechanism (rows of 10 to 95 doubles)
@pytest.mark.parametrize("E,order_p,species", [(1, 1, 0), (63, 1, 0), (64, 2, 0), (65, 3, 0), (1000, 4, 0),
                                               (31, 2, 5), (129, 4, 5), (65, 4, 16), (64, 1, 16)])
def test_round_trip(adg, E, order_p, species):
    import torch

    if species:
        case, w0 = gen.case_c1(E=E, order_p=order_p, n_pe=1, mech=mechanism_of(species), Lx=0.01 * max(E, 8) / 2048)
    else:
        case, w0 = gen.case_c0(E=E, order_p=order_p, n_pe=1)
    for noalloc in (False, True):
        s = adg.Solver(case, noalloc=noalloc)
        host, dev = any_state(w0.shape, E), any_state(w0.shape, E + 1)
        s.set_state(host)
        out = torch.zeros(w0.shape, dtype=torch.float64, device="cuda")
        s.state_device(out)
        assert np.array_equal(out.cpu().numpy().view(np.int64), host.view(np.int64))
        s.set_state(torch.from_numpy(dev).cuda())
        assert np.array_equal(s.state().view(np.int64), dev.view(np.int64))
        s.close()


@pytest.mark.parametrize("model", ["onestep", "detailed"])
def test_new_state_starts_over(adg, model):
    """Steps from a second state are those of a new solver: no history, counter or error is left."""
    if model == "onestep":
        case, w0 = gen.case_c0(E=130, n_pe=8, pmf=(0.3, 0.4, 0.3))
    else:
        case, w0 = gen.case_c1(E=130, order_p=2, n_pe=8, cfl=0.08, Lx=0.01 * 130 / 2048)
    s, ref = adg.Solver(case), adg.Solver(case)
    bad = w0.copy()
    bad[:, 0, :] = -1.0
    s.set_state(bad)
    s.step(7)
    with pytest.raises(adg.AdgError):
        s.state()
    s.set_state(w0)
    ref.set_state(w0)
    s.step(9)
    ref.step(9)
    assert s.step_count() == 9
    assert np.array_equal(s.state(), ref.state())
    s.close()
    ref.close()


@pytest.mark.parametrize("graph_steps", [0, 3])
def test_batch_instances_at_their_own_counts(adg, orc, graph_steps):
    """One-step instances admitted at odd and even batch steps, one by a schedule of delays, one that stops
    at an odd count, each read after steps with and without graphs: the host knows which buffer is theirs."""
    sched = (np.arange(64 * 5, dtype=np.int8).reshape(64, 5) % 2).copy()
    specs = [dict(n_pe=5), dict(n_pe=5, mode="schedule", schedule=sched), dict(n_pe=3), dict(n_pe=4)]
    cases = [gen.case_c0(E=66 + 7 * i, order_p=2, pmf=(0.3, 0.4, 0.3), **{k: v for k, v in sp.items() if k != "schedule"})
             for i, sp in enumerate(specs)]
    cases[1][0]["async"].update(schedule=sched, L=2)
    targets = [0, 0, 5, 0]
    heap = sum(adg.Batch.instance_bytes(c) for c, _ in cases)
    b = adg.Batch(4, sum(c["disc"]["n_elem"] for c, _ in cases), heap)
    b.set_graph(graph_steps)
    slots, counts = [], []
    for (c, w), t in zip(cases, targets):
        slots.append(b.add(c, w, t))
        counts.append(0)
        b.step(7)
        counts = [min(n + 7, t or 999) for n, t in zip(counts, targets)]
        for (cc, ww), sl, n in zip(cases, slots, counts):
            o = orc.OracleSolver(cc, ww, 40)
            o.step(n)
            check(b.state(sl), o.state(), cc, 1e-10, f"after {n} steps")
    assert [int(x) for x in b.poll()[0]] == counts
    b.close()
