"""Write-through state stores leave the same bits as ordinary ones: every row and
column schedule of FP64 and FP32 lines, rows of 4096 points and more among them, in
the modes chosen explicitly, each on a solver of its own created anew."""
import numpy as np
import pytest

from paper_1909_02894_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def D():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_02894_amd import dirac
    return dirac


def solve(D, spec, prec, psi0, d, sched, mode):
    s = D.Solver.from_spec(spec, precision=prec)
    s.set_schedule(d, *sched)
    s.set_store_mode(mode)
    assert s.store_mode() == mode
    s.set_initial_spinor(psi0)
    s.step_n(2)
    out = s.get_spinor()
    s.close()
    return out


@pytest.mark.parametrize("prec,n1,n2,d", [(0, 4096, 32, 0), (1, 4096, 32, 0), (1, 8192, 16, 0), (0, 2048, 16, 0),
                                          (0, 1024, 64, 0), (0, 512, 64, 0), (0, 64, 1024, 1), (0, 64, 512, 1)])
def test_store_modes_same_bits(D, prec, n1, n2, d):
    psi0 = W.random_spinor(n1, n2, seed=n1 + d)
    for kind in ("curved", "layer"):
        spec = W.curved_bump(n=32, seed=31 + n1 + d, m=0.7, pml_width=6) if kind == "curved" else W.flat_small(n=32)
        spec.n1, spec.n2, spec.pml_width = n1, n2, 6
        spec.a1, spec.a2 = 20.0 * n1 / max(n1, n2), 20.0 * n2 / max(n1, n2)
        for sched in D.schedules(n1 if d == 0 else n2, prec, d):
            print(f"[store mode] {n1}x{n2} prec={prec} {kind} {sched}", flush=True)
            ref = solve(D, spec, prec, psi0, d, sched, 0)
            for mode in (3, 1 << d, 3):
                assert np.array_equal(solve(D, spec, prec, psi0, d, sched, mode), ref), (kind, sched, mode)
