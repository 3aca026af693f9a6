"""3-D direction kernels at every line length along every axis (the shortest to
the longest, several and one line per workgroup, staged and unstaged twiddles),
flat, flat with a layer and curved, against the 3-D oracle.  Tolerances as for
every 3-D solve: FP64 1e-11 relative L2, FP32 2e-5."""
import numpy as np
import pytest

from oracle import dirac3_oracle as O3
from oracle import dirac_oracle as O
from tests.test_gpu_3d import TOL32, TOL64, D, gpu3  # noqa: F401  (D: the module fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [(16, 16, 16), (32, 128, 16), (256, 16, 32), (16, 512, 16), (1024, 16, 16),
                               (16, 1024, 16), (16, 16, 1024), (64, 16, 512)])
def test_3d_line_lengths(D, n, prec):  # noqa: F811
    rng = np.random.default_rng(11)
    psi0 = rng.standard_normal(n[::-1] + (4,)) + 1j * rng.standard_normal(n[::-1] + (4,))
    for metric, width in ((O.METRIC_FLAT, 0), (O.METRIC_FLAT, 2), (O3.METRIC_PAPER_EXP3, 2)):
        print(f"[3d shapes] {n} prec={prec} metric={metric} layer={width}", flush=True)
        p = O3.Problem3(n1=n[0], n2=n[1], n3=n[2], a1=6.0, a2=5.0, a3=7.0, dt=0.02, c=1.1, m=0.8, metric=metric,
                        spin=O.SPIN_PAPER if metric != O.METRIC_FLAT else O.SPIN_NONE, pml_width=width)
        _, g = gpu3(D, p, psi0, 3, precision=prec)
        assert O.rel_l2(g, O3.run3(psi0, O3.build_tables3(p), 3)) < (TOL64 if prec == 0 else TOL32)
