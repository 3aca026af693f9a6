"""Scheme I at the vector lengths where its reduction and update kernels change their
work split: fewer entries than one workgroup's threads, exactly one entry per thread
of the whole launch, several; vectors below, inside and above the written-through
range.  Tolerance as in the Scheme I parity tests: both sides solve to 1e-14."""
import numpy as np
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


@pytest.mark.parametrize("n1,n2", [(16, 16), (32, 16), (256, 256), (64, 1024), (512, 256), (1024, 1024)])
def test_cn_vector_lengths(D, n1, n2):
    print(f"[cn] {n1}x{n2}", flush=True)
    spec = W.curved_bump(n=64, seed=9, m=0.5)
    spec.n1, spec.n2 = n1, n2
    spec.pml_width = max(1, min(n1, n2) // 16)
    psi0 = W.random_spinor(n1, n2, 3)
    s = D.Solver.from_spec(spec, precision=D.FP64, scheme=D.SCHEME_CN_GMRES, gmres_restart=20, gmres_rtol=1e-14)
    s.set_initial_spinor(psi0)
    s.step_n(2)
    T = O.build_tables(oracle_problem(spec))
    assert O.rel_l2(s.get_spinor(), O.cn_run(psi0, T, 2)) < 1e-11
    s2 = D.Solver.from_spec(spec, precision=D.FP64, scheme=D.SCHEME_CN_GMRES, gmres_restart=20, gmres_rtol=1e-14)
    s2.set_initial_spinor(psi0)
    s2.step_n(2)
    assert np.array_equal(s2.get_spinor(), s.get_spinor())
