"""Column launches whose workgroups take several tiles in turn, against the oracle, with
one tile per workgroup (512 lines of two), a few, lines in groups of four, padded rows;
and against the same radix with a workgroup per tile, bitwise.  Tolerances as for every
static solve: FP64 1e-11 relative L2, FP32 2e-5."""
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


def make(D, n1, n2, prec, kind):
    print(f"[stream] {n1}x{n2} prec={prec} {kind}", flush=True)
    spec = W.flat_small(n=64) if kind != "curved" else W.curved_bump(n=64, seed=9, m=0.5)
    spec.n1, spec.n2 = n1, n2
    spec.pml_width = 0 if kind == "flat" else min(n1, n2) // 16
    s = D.Solver.from_spec(spec, precision=prec)
    psi0 = W.random_spinor(n1, n2, 3)
    s.set_initial_spinor(psi0)
    return spec, s, psi0


@pytest.mark.parametrize("kind", ["curved", "layer", "flat"])
@pytest.mark.parametrize("prec,n1,n2,sy", [(0, 512, 2048, (16, 2, 2)), (0, 1024, 2048, (16, 2, 2)),
                                           (1, 512, 4096, (16, 2, 2)), (1, 1024, 4096, (16, 2, 2)),
                                           (1, 2048, 2048, (16, 4, 2)), (1, 4096, 2048, (16, 4, 2))])
def test_streamed_columns(D, prec, n1, n2, sy, kind):
    spec, s, psi0 = make(D, n1, n2, prec, kind)
    s.set_schedule(1, *sy)
    s.step_n(2)
    ref = O.run(psi0, O.build_tables(oracle_problem(spec)), 2)
    assert O.rel_l2(s.get_spinor(), ref) < (1e-11 if prec == 0 else 2e-5)
    s.close()


@pytest.mark.parametrize("kind", ["curved", "layer", "flat"])
@pytest.mark.parametrize("n1,n2,sy,other", [(1024, 4096, (16, 2, 2), (16, 2, 1)), (2048, 2048, (16, 4, 2), (16, 4, 1))])
def test_streamed_columns_same_bits(D, n1, n2, sy, other, kind):
    got = []
    for sched in (sy, other):
        _, s, _ = make(D, n1, n2, 1, kind)
        s.set_schedule(1, *sched)
        s.step_n(3)
        s.step_n(1)
        got.append(s.get_spinor())
        s.close()
    assert np.array_equal(got[0], got[1])
