"""Device uploads from an array that is aligned to its doubles only (a view one double
into a buffer), into padded and unpadded states of both precisions."""
import numpy as np
import pytest

from paper_1909_02894_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n1,n2", [(4096, 16), (2048, 16), (64, 32)])
def test_upload_from_an_odd_double(n1, n2, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_02894_amd import dirac as D
    print(f"[upload] {n1}x{n2} prec={prec}", flush=True)
    spec = W.flat_small(n=64)
    spec.n1, spec.n2 = n1, n2
    psi = W.random_spinor(n1, n2, 11)
    buf = torch.zeros(4 * n1 * n2 + 1, dtype=torch.float64, device="cuda")
    buf[1:] = torch.from_numpy(psi.view(np.float64).ravel())
    view = buf[1:]
    assert view.data_ptr() % 16 == 8
    s = D.Solver.from_spec(spec, precision=prec)
    s.set_initial_spinor_device(view)
    got = s.get_spinor()
    s.close()
    assert np.array_equal(got, psi if prec == 0 else psi.astype(np.complex64).astype(np.complex128))
