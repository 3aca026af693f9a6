"""States with padded rows (n1 >= 4096 points) and the row lengths below:
upload, download, device upload, the tuner's save and restore, stepping and the
observables against the oracle.

Tolerances as for every static solve: FP64 1e-11 relative L2, FP32 2e-5 (state)
and 1e-6 (norms, quadratic in rounded data)."""
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


@pytest.mark.parametrize("n1,n2,prec", [(2048, 32, 0), (4096, 16, 0), (4096, 64, 0), (4096, 32, 1), (8192, 16, 1),
                                        (16, 4096, 0)])
def test_row_pitch(D, n1, n2, prec):
    import torch
    print(f"[layout] {n1}x{n2} prec={prec}", flush=True)
    spec = W.curved_bump(n=64, seed=5, m=0.5)
    spec.n1, spec.n2, spec.pml_width = n1, n2, min(n1, n2) // 16
    rng = np.random.default_rng(7)
    psi0 = W.initial_spinor(spec) * (1 + 0.1 * rng.random((n2, n1, 1)))
    stored = psi0 if prec == 0 else psi0.astype(np.complex64).astype(np.complex128)
    s = D.Solver.from_spec(spec, precision=prec)
    s.set_initial_spinor(psi0)
    assert np.array_equal(s.get_spinor(), stored)
    s.set_initial_spinor(np.zeros_like(psi0))
    dev = torch.from_numpy(np.ascontiguousarray(psi0)).cuda()
    s.set_initial_spinor_device(dev)
    assert np.array_equal(s.get_spinor(), stored)
    s.autotune(2)
    s.time_directions(2)
    assert np.array_equal(s.get_spinor(), stored)
    T = O.build_tables(oracle_problem(spec))
    s.step_n(3)
    ref = O.run(psi0, T, 3)
    assert O.rel_l2(s.get_spinor(), ref) < (1e-11 if prec == 0 else 2e-5)
    got = s.observables()
    dA = (2 * spec.a1 / n1) * (2 * spec.a2 / n2)
    l2 = dA * float((np.abs(ref) ** 2).sum())
    assert abs(got["norm_l2"] - l2) < (1e-11 if prec == 0 else 1e-6) * l2 and got["finite"] == 1
    s.close()
