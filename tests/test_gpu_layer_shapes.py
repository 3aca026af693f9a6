"""Default schedules of flat grids with a layer, and the thresholds of the longer
line counts in every mode, against the oracle.  Tolerances as for every static solve:
FP64 1e-11 relative L2, FP32 2e-5."""
import pytest

from oracle import dirac_oracle as O
from paper_1909_02894_amd import workloads as W
from tests.helpers import oracle_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_02894_amd import dirac
    return dirac


@pytest.mark.parametrize("prec,n1,n2,kinds", [
    (0, 512, 256, "l"), (0, 256, 512, "l"), (0, 2048, 256, "l"), (0, 2048, 512, "l"), (0, 512, 1024, "l"),
    (0, 1024, 1024, "lcf"), (0, 2048, 1024, "lcf"), (0, 4096, 256, "lf"), (0, 4096, 512, "lf"),
    (1, 1024, 256, "l"), (1, 256, 1024, "l"), (1, 2048, 512, "l"), (1, 2048, 1024, "l"), (1, 512, 4096, "lcf"),
    (1, 1024, 4096, "lcf"), (1, 2048, 2048, "l"), (1, 64, 8192, "lcf"), (1, 512, 8192, "lc")])
def test_default_thresholds(D, prec, n1, n2, kinds):
    for k in kinds:
        print(f"[layer shapes] {n1}x{n2} prec={prec} {k}", flush=True)
        spec = W.curved_bump(n=64, seed=9, m=0.5) if k == "c" else W.flat_small(n=64)
        spec.n1, spec.n2 = n1, n2
        spec.pml_width = 0 if k == "f" else min(n1, n2) // 16
        psi0 = W.random_spinor(n1, n2, 3)
        s = D.Solver.from_spec(spec, precision=prec)
        s.set_initial_spinor(psi0)
        s.step_n(2)
        ref = O.run(psi0, O.build_tables(oracle_problem(spec)), 2)
        assert O.rel_l2(s.get_spinor(), ref) < (1e-11 if prec == 0 else 2e-5), (k, s.schedule(0), s.schedule(1))
        s.close()
