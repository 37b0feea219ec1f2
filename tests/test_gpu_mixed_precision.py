"""Mixed precision where it runs: FP32 modal operators in the single problem's kernels (N_p <= 3, up to 8192
elements), next to the discretisation error that their error has to stay a tenth of; and batches, whose kernel keeps
FP64 operators in either precision."""
import numpy as np
import pytest

from _parity import var_errors
from test_gpu_batch import CFL, ns_case, restrict_to_coarse
from workloads import gen

pytestmark = pytest.mark.gpu


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


@pytest.mark.parametrize("P", [1, 2, 3])
def test_single_problem_error_budget(adg, orc, mech, P):
    E, steps = 64, 120
    case, w0 = ns_case(mech, E, P, 8, "saa", 21)
    # the same run on twice the elements; both use the finer mesh's time step
    case2, w02 = gen.case_c1(E=2 * E, order_p=P, n_pe=8, mode="saa", mech=mech, seed=21, cfl=CFL[P], Lx=0.01 * E / 2048)
    case["disc"]["dt"] = case2["disc"]["dt"]
    o, o2 = orc.OracleSolver(case, w0, steps + 1), orc.OracleSolver(case2, w02, steps + 1)
    o.step(steps)
    o2.step(steps)
    ref = o.state()
    edisc = float(np.max(var_errors(ref, restrict_to_coarse(o2.state(), P))))
    got = {}
    for precision in ("fp64", "mixed"):
        c = dict(case, disc=dict(case["disc"], precision=precision))
        for config in (0, 1, 3):
            s = adg.Solver(c)
            s.set_kernel_config(config)
            s.set_state(w0)
            s.step(steps)
            got[precision, config] = s.state()
            s.close()
    for config in (0, 1, 3):
        e64 = float(np.max(var_errors(got["fp64", config], ref)))
        emx = float(np.max(var_errors(got["mixed", config], ref)))
        print(f"[mixed-single] Np={P} config {config} fp64 {e64:.2e} mixed {emx:.2e} discretisation {edisc:.2e} "
              f"ratio {emx / edisc:.3f}", flush=True)
        assert e64 < 1e-10
        assert 10 * e64 < emx < 0.1 * edisc   # FP32 operators ran, and stay within the budget


@pytest.mark.parametrize("P", [1, 2, 3, 4])
def test_batches_keep_fp64_operators(adg, mech, P):
    case, w0 = ns_case(mech, 40, P, 4, "saa", 22)
    out = []
    for precision in ("fp64", "mixed"):
        b = adg.Batch(1, 40, adg.Batch.instance_bytes(case), precision=precision)
        sl = b.add(case, w0)
        b.step(15)
        out.append(b.state(sl))
        b.close()
    np.testing.assert_array_equal(*out)
