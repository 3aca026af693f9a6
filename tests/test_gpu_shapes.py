"""Kernel shapes chosen by grid size, as created (no tuning): the plain step's
default schedules and store modes on both sides of their line-count thresholds, and
the corrected second-order step's one- and two-component kernels, against the
oracle.  Tolerances as for every static solve: FP64 1e-11 relative L2, FP32 2e-5."""
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


def check(D, n1, n2, prec, kind, scheme, step2):
    print(f"[shapes] {n1}x{n2} prec={prec} {kind} scheme={scheme}", flush=True)
    spec = W.flat_small(n=64) if kind != "curved" else W.curved_bump(n=64, seed=9, m=0.5)
    spec.n1, spec.n2 = n1, n2
    spec.pml_width = 0 if kind == "flat" else max(1, min(n1, n2) // 16)
    psi0 = W.random_spinor(n1, n2, 3)
    s = D.Solver.from_spec(spec, precision=prec, scheme=scheme)
    s.set_initial_spinor(psi0)
    s.step_n(3)
    ref = O.run(psi0, O.build_tables(oracle_problem(spec, step2=step2)), 3)
    assert O.rel_l2(s.get_spinor(), ref) < (1e-11 if prec == 0 else 2e-5)
    s.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n1,n2", [(16, 16), (512, 32), (32, 512), (1024, 64), (1024, 256), (256, 1024), (2048, 512),
                                   (16, 2048)])
def test_default_shapes(D, n1, n2, prec):
    for kind in ("curved", "flat"):
        check(D, n1, n2, prec, kind, D.SCHEME_EXP_SPLIT, O.STEP2_PLAIN)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n1,n2", [(16, 16), (16, 512), (512, 16), (64, 128), (1024, 512), (32, 1024)])
def test_corrected_step_shapes(D, n1, n2, prec):
    for kind in ("curved", "layer"):
        check(D, n1, n2, prec, kind, D.SCHEME_EXP_SPLIT_2BIS, O.STEP2BIS_CORRECTED)
