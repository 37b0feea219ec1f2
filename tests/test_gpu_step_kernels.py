"""The one-step model's whole-step kernel at the edges of its wavefront tiles (64 lanes less a halo
of one lane per RK stage on each side, two with the limiter: 58 and 52 owned elements for SSP-RK3, 60
and 56 for RK2, 54 and 44 for the five-stage scheme), against the oracle at the repository's parity
bound (1e-10)."""
import pytest

from _parity import check
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def adg():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2501_01747_amd import adg as lib

    return lib


OWNED = {"ssprk3": 58, "rk2": 60, "lserk4": 54}
# meshes shorter than the halo, and around one wavefront and one workgroup of four
SIZES = {rk: [1, 2, 4, n - 1, n, n + 1, 4 * n - 1, 4 * n + 1] for rk, n in OWNED.items()}


@pytest.mark.parametrize("bc,flux", [("periodic", "rusanov"), ("transmissive", "hllc")])
@pytest.mark.parametrize("rk,E", [(rk, E) for rk, sizes in SIZES.items() for E in sizes])
def test_whole_step_tiles(adg, orc, rk, E, bc, flux):
    """Every element its own PE on the short meshes (every face delayed), five PEs on the others."""
    order_p = 1 + E % 4
    case, w0 = gen.case_c0(E=E, order_p=order_p, n_pe=min(E, 5), mode="saa", pmf=(0.3, 0.4, 0.3),
                           cfl={1: 0.1, 2: 0.08, 3: 0.04, 4: 0.01}[order_p])
    case["disc"].update(bc=bc, flux=flux, rk=rk)
    s = adg.Solver(case)
    s.set_state(w0)
    o = orc.OracleSolver(case, w0, 13)
    s.step(12)
    o.step(12)
    check(s.state(), o.state(), case, 1e-10, f"{rk} E={E} {bc}")
    assert s.step_count() == 12
    s.close()


LIMITED = {"ssprk3": 52, "rk2": 56, "lserk4": 44}
LIM_SIZES = {rk: [1, 2, 3, 5, 2 * {"ssprk3": 3, "rk2": 2, "lserk4": 5}[rk] + 1, n - 1, n, n + 1, 2 * n + 1]
             for rk, n in LIMITED.items()}


@pytest.mark.parametrize("bc", ["periodic", "transmissive"])
@pytest.mark.parametrize("rk,E", [(rk, E) for rk, sizes in LIM_SIZES.items() for E in sizes])
def test_whole_step_limiter_tiles(adg, orc, rk, E, bc):
    """Every cell limited (no threshold that round-off could cross) on the smooth wave, with more delayed
    interfaces in a wavefront than one round of neighbour slots takes where the mesh allows."""
    order_p = 1 + (E + 1) % 4
    case, w0 = gen.case_c0(E=E, order_p=order_p, n_pe=min(E, 11), mode="saa", pmf=(0.3, 0.4, 0.3),
                           cfl={1: 0.1, 2: 0.05, 3: 0.02, 4: 0.005}[order_p], k_pre=1e2)
    case["disc"].update(bc=bc, flux="hllc" if E % 2 else "rusanov", rk=rk, limiter=1, indicator="all")
    s = adg.Solver(case)
    s.set_state(w0)
    o = orc.OracleSolver(case, w0, 11)
    s.step(10)
    o.step(10)
    check(s.state(), o.state(), case, 1e-10, f"limited {rk} E={E} {bc}")
    flags, total = s.flags()
    stages = {"ssprk3": 3, "rk2": 2, "lserk4": 5}[rk]
    assert flags.all() and total == 10 * stages * E
    s.close()


@pytest.mark.parametrize("limiter", [0, 1])
@pytest.mark.parametrize("e_act", [0.0, 3.0, 700.0, 1e7, 1e300])
def test_reaction_exponents(adg, orc, e_act, limiter):
    """Arrhenius exponents from 0 to where the rate underflows, and far beyond the bound that the kernel
    holds them to."""
    case, w0 = gen.case_c0(E=130, order_p=2, n_pe=4, cfl=0.05, k_pre=1e2)
    case["physics"]["e_act"] = e_act
    case["disc"].update(limiter=limiter, indicator="all", flux="hllc")
    s = adg.Solver(case)
    s.set_state(w0)
    o = orc.OracleSolver(case, w0, 13)
    s.step(12)
    o.step(12)
    check(s.state(), o.state(), case, 1e-10, f"e_act={e_act}")
    s.close()
