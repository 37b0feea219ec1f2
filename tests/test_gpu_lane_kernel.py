"""The lane-per-point detailed-chemistry kernel (batches of any size; single problems of more than
8192 elements, 12288 with more than 9 species) at the edges of its tiles (46, 37, 31 and 25 elements
for N_p = 1..4), with a PE interface at every face, and with equilibrium constants whose factors
leave the range of the factored form, against the oracle at the repository's parity bound (1e-10)."""
import numpy as np
import pytest

from _parity import check, var_errors
from test_gpu_ns import mechanism_of
from workloads import gen

pytestmark = pytest.mark.gpu

TILE = {1: 46, 2: 37, 3: 31, 4: 25}
CFL = {1: 0.1, 2: 0.08, 3: 0.04, 4: 0.01}


@pytest.fixture(scope="module")
def adg():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2501_01747_amd import adg as lib

    return lib


@pytest.fixture(scope="module")
def mech():
    return gen.c1_mechanism()


def run_batch(adg, orc, cases, steps):
    heap = sum(adg.Batch.instance_bytes(c) for c, _ in cases)
    b = adg.Batch(len(cases), sum(c["disc"]["n_elem"] for c, _ in cases), heap)
    slots = [b.add(c, w) for c, w in cases]
    b.step(steps)
    for (c, w), sl in zip(cases, slots):
        o = orc.OracleSolver(c, w, steps + 1)
        o.step(steps)
        print(f"[lane] E={c['disc']['n_elem']} Np={c['disc']['order_p']} PEs={c['async']['n_pe']} {c['disc']['bc']}", flush=True)
        check(b.state(sl), o.state(), c, 1e-10, "batch instance")
    b.close()


@pytest.mark.parametrize("bc", ["periodic", "transmissive"])
@pytest.mark.parametrize("order_p", [1, 2, 3, 4])
def test_tile_edges(adg, orc, mech, order_p, bc):
    """Meshes shorter than the halo, one element short of, equal to and past one and two tiles."""
    te = TILE[order_p]
    cases = []
    for E in (1, 2, 3, te - 1, te, te + 1, 2 * te, 2 * te + 1):
        c, w = gen.case_c1(E=E, order_p=order_p, n_pe=min(E, 3), mech=mech, cfl=CFL[order_p], Lx=0.01 * max(E, 8) / 2048, seed=E)
        c["disc"]["bc"] = bc
        cases.append((c, w))
    run_batch(adg, orc, cases, 8)


@pytest.mark.parametrize("order_p,at_order", [(2, 3), (3, 6)])
def test_every_face_a_pe_interface(adg, orc, mech, order_p, at_order):
    """More interfaces in a tile than the first wavefront takes in one round; AT orders of up to 6 levels."""
    cases = []
    for E, bc in ((2 * TILE[order_p] + 5, "periodic"), (TILE[order_p] + 2, "transmissive")):
        c, w = gen.case_c1(E=E, order_p=order_p, n_pe=E, mech=mech, cfl=0.2 * CFL[order_p], Lx=0.01 * E / 2048, seed=E,
                           at_order=at_order, pmf=(0.2, 0.4, 0.4))
        c["disc"]["bc"] = bc
        cases.append((c, w))
    run_batch(adg, orc, cases, 12)


def test_factors_beyond_the_factored_range(adg, orc, mech):
    """An enthalpy of -0.8 MJ/mol per atom A in every species leaves all reaction enthalpies as they are,
    but puts the largest species factor of the equilibrium constants (A2B) at exp(250) at 1000 K, where the
    kernel sums the exponents first: in a mesh between 950 and 1050 K, wavefronts of either form of the
    rates and of both kinds of points."""
    nasa = mech["nasa7"].copy()
    nasa[:, 5] -= 0.8e6 / gen.RU * mech["composition"][:, 0]
    shifted = dict(mech, nasa7=nasa)
    run_batch(adg, orc, [gen.case_c1(E=93, n_pe=4, mech=shifted, Lx=0.01 * 93 / 2048)], 10)


@pytest.mark.parametrize("ns,E,rk", [(9, 8215, "ssprk3"), (9, 8216, "lserk4"), (5, 8214, "rk2"), (16, 12307, "ssprk3")])
def test_single_problems(adg, orc, ns, E, rk):
    """Single problems past the size from which the kernel runs them by default, with a last tile of
    31, 1 and 30 elements and 16 species; then the decomposition changed in mid-run and back (the
    spread kernels' carried AT values are formed anew)."""
    mech = gen.c1_mechanism() if ns == 9 else mechanism_of(ns)
    case, w0 = gen.case_c1(E=E, n_pe=40, mech=mech, Lx=0.01 * E / 2048, cfl=0.02)
    case["disc"].update(rk=rk, bc="transmissive" if E % 2 else "periodic")
    s = adg.Solver(case)
    s.set_state(w0)
    o = orc.OracleSolver(case, w0, 8)
    s.step(5)
    s.set_kernel_config(0)
    s.step(1)
    s.set_kernel_config(1)
    s.step(1)
    o.step(7)
    assert float(np.max(var_errors(s.state(), o.state()))) < 1e-10
    check(s.state(), o.state(), case, 1e-10, "single")
    s.close()


@pytest.mark.parametrize("E,species", [(1, 9), (1023, 9), (1024, 9), (1025, 9), (1024, 16), (1025, 16)])
def test_untuned_choice_of_small_meshes(adg, orc, mech, E, species):
    """Either side of the last mesh that gives each of 256 CUs one tile of 4 elements: against the oracle,
    and bit for bit what the tile of 8 with 512 threads gives."""
    c, w = gen.case_c1(E=E, order_p=2, n_pe=min(E, 7), mech=mech if species == 9 else mechanism_of(species), cfl=0.08,
                       Lx=0.01 * max(E, 8) / 2048)
    got = []
    for config in (None, 0):
        s = adg.Solver(c)
        if config is not None:
            s.set_kernel_config(config)
        s.set_state(w)
        s.step(5)
        got.append(s.state())
        s.close()
    o = orc.OracleSolver(c, w, 6)
    o.step(5)
    check(got[0], o.state(), c, 1e-10, f"E={E} species={species}")
    assert np.array_equal(got[0], got[1])


def test_rates_at_the_ends_of_the_range_of_exp(adg, orc, mech):
    """Channels switched off by an activation energy of any size (the largest exponents a double holds, and
    some where only the forward rate is zero), in a batch and in a single problem of the size that takes
    this kernel, against the oracle."""
    Ea = mech["Ea"].copy()
    Ea[[0, 3, 7, 20]] = 1e300, 1e12, 3e8, 8e6
    off = dict(mech, Ea=Ea)
    run_batch(adg, orc, [gen.case_c1(E=E, n_pe=4, mech=off, Lx=0.01 * E / 2048) for E in (5, 70)], 10)
    case, w0 = gen.case_c1(E=8200, n_pe=4, mech=off, Lx=0.01 * 8200 / 2048)
    s = adg.Solver(case)
    s.set_state(w0)
    s.step(3)
    o = orc.OracleSolver(case, w0, 4)
    o.step(3)
    check(s.state(), o.state(), case, 1e-10, "single")
    s.close()


def test_reverse_rate_of_a_forward_rate_of_zero(adg, mech):
    """A reaction 2 X = 2 Y whose forward rate constant underflows at every temperature of the mesh but whose
    reverse one is e^26, Y lying 3.9 MJ/mol above X and the species' factors of the equilibrium constant
    within exp(250): the batched kernel against the single problem's, which forms the two constants apart.
    Bound: that of the other parity tests, 1e-10; without the reverse rate Y stays as it was."""
    ix, iy = mech["names"].index("A"), mech["names"].index("B")
    nasa, W = mech["nasa7"].copy(), mech["W"].copy()
    W[ix] = W[iy]
    nasa[ix] = (3.0, 1e-3, 0.0, 0.0, 0.0, -232e3, -20.0)
    nasa[iy] = (3.0, 1e-3, 0.0, 0.0, 0.0, 232e3, -20.0)
    nu_f, nu_r = (np.zeros((1, mech["n_species"]), np.int32) for _ in range(2))
    nu_f[0, ix] = nu_r[0, iy] = 2
    one = dict(mech, nasa7=nasa, W=W, n_reactions=1, nu_f=nu_f, nu_r=nu_r, A=np.array([np.exp(26.0)]),
               b=np.zeros(1), Ea=np.array([928e3 * gen.RU]))
    case, w0 = gen.case_c1(E=40, n_pe=2, mech=one, Lx=0.01 * 40 / 2048)
    s = adg.Solver(case)
    s.set_state(w0)
    s.step(10)
    b = adg.Batch(1, 40, adg.Batch.instance_bytes(case))
    sl = b.add(case, w0)
    b.step(10)
    got, ref = b.state(sl), s.state()
    b.close()
    s.close()
    y = ref[:, 3 + iy, 0] / w0[:, 3 + iy, 0]
    print("[lane] Y / Y(0):", y.min(), y.max(), flush=True)
    assert y.max() < 0.99
    check(got, ref, case, 1e-10, "reverse rate")


def test_chains_on_one_stream_and_on_two(adg, mech):
    """Enough tiles (538) for two chains of launches, of different orders: one launch for both on one stream
    and a stream each, bit for bit; the number of streams changed between steps."""
    cases = [gen.case_c1(E=E, order_p=p, n_pe=9, mech=mech, cfl=CFL[p], Lx=0.01 * E / 2048) for E, p in ((8000, 4), (10000, 1))]
    heap = sum(adg.Batch.instance_bytes(c) for c, _ in cases)
    got = []
    for streams in ((1, 1), (4, 4), (1, 2)):
        b = adg.Batch(2, 18000, heap)
        slots = [b.add(c, w) for c, w in cases]
        for n in streams:
            b.set_group_streams(n)
            b.step(2)
        assert b.profile(1)["detailed_stage"][1] == 3   # timed on one stream: a launch per stage
        got.append([b.state(sl) for sl in slots])
        b.close()
    for other in got[1:]:
        for x, y in zip(got[0], other):
            np.testing.assert_array_equal(x, y)


def test_inviscid(adg, orc, mech):
    run_batch(adg, orc, [gen.case_c1(E=E, order_p=p, n_pe=4, mech=mech, cfl=CFL[p], Lx=0.01 * E / 2048, viscous=0)
                         for E, p in ((70, 3), (47, 1))], 10)


def test_graphs_across_a_change_of_decomposition(adg, mech):
    """A large single problem stepped from graphs, by the lane-per-point kernel, by a spread one, which carries AT
    values from launch to launch, and by the former again: bit for bit the plain steps."""
    case, w0 = gen.case_c1(E=8215, n_pe=120, mech=mech, Lx=0.01 * 8215 / 2048, cfl=0.02)
    got = []
    for graph in (0, 2, 3):
        s = adg.Solver(case)
        s.set_graph(graph)
        s.set_state(w0)
        for config, n in ((None, 5), (0, 4), (1, 5), (0, 3)):
            if config is not None:
                s.set_kernel_config(config)
            s.step(n)
        assert s.step_count() == 17 and (s.graph_replays > 0) == (graph > 0)
        got.append(s.state())
        s.close()
    for w in got[1:]:
        np.testing.assert_array_equal(w, got[0])


def test_factors_beyond_the_factored_range_of_a_large_mechanism(adg, orc):
    """As above with 16 species: a single problem of a size that takes this kernel."""
    mech = mechanism_of(16)
    nasa = mech["nasa7"].copy()
    nasa[:, 5] -= 0.6e6 / gen.RU * mech["composition"][:, 0]
    case, w0 = gen.case_c1(E=12300, order_p=1, n_pe=5, mech=dict(mech, nasa7=nasa), Lx=0.01 * 12300 / 2048, cfl=0.05)
    s = adg.Solver(case)
    s.set_state(w0)
    s.step(3)
    o = orc.OracleSolver(case, w0, 4)
    o.step(3)
    check(s.state(), o.state(), case, 1e-10, "16 species")
    s.close()
